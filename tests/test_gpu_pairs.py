"""The backprojection contracts each unordered (e, r) pair once, with the sum
of the pair's two weighted residuals.  These cases give the two orders of a
pair different data and weights, down to whole 32 x 32 blocks that are zero in
one order only, on rings whose block count is even (two blocks half a ring
apart), odd, and one.

The FP32 contractions that run on the FP16 matrix cores in two pieces are
checked here too, at the edges of their tiles and of FP16's range.
"""
import dataclasses

import numpy as np
import pytest
import torch

import workload as W
from _parity import close
from oracle import born

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = {"f64": 1e-10, "f32": 1e-5, "f16": 2e-3, "bf16": 1e-2}   # as the dense contraction tests


@pytest.fixture(scope="module")
def rb():
    import paper_2511_16633_amd as m
    return m


def _geom(nx, ny, m):
    g = W.centred_grid(nx, 0.5e-3, m, 12e-3, 1500.0)
    return dataclasses.replace(g, ny=ny, y0=-0.5 * (ny - 1) * 0.5e-3)


def _tables(rb, geom, freqs, dtype, seed):
    T, A, B, _, _, _ = W.random_tables(geom, seed=seed)
    f32 = torch.float32
    z = np.zeros((geom.m, geom.m))
    tab = {k: torch.as_tensor(v, device=DEV, dtype=t) for k, v, t in
           (("T", T, None), ("amp", A, f32), ("att", B, f32), ("T_rx", z, None), ("amp_rx", z, f32), ("att_rx", z, f32))}
    Gr = torch.empty((len(freqs), geom.m, geom.n_pixels), dtype=rb._binding.TORCH_DTYPES[rb.DTYPES[dtype]], device=DEV)
    Gi = torch.empty_like(Gr)
    sc = torch.empty(len(freqs), dtype=f32, device=DEV)
    rb.build_green(geom, tab, freqs, 1.0, dtype, Gr, Gi, sc)
    G = [born.green(T, A.astype(np.float64), B.astype(np.float64), f) for f in freqs]
    return Gr, Gi, sc, G


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16", "f16"])
@pytest.mark.parametrize("shape", [(9, 7, 4), (8, 8, 32), (16, 8, 64), (13, 10, 96), (16, 16, 128), (12, 11, 256),
                                   (8, 9, 515), (8, 8, 640)])
def test_adjoint_of_unsymmetric_data_and_weights(rb, dtype, shape):
    nx, ny, m = shape
    geom = _geom(nx, ny, m)
    freqs = [3e5, 7e5]
    print(f"[gpu-test] unsymmetric adjoint {dtype} {shape}", flush=True)
    Gr, Gi, sc, G = _tables(rb, geom, freqs, dtype, 5)
    rng = np.random.default_rng(m)
    D = W.random_residual(2, m, 6)
    w = rng.uniform(0.0, 2.0, (2, m, m))
    nb = (m + 31) // 32
    for k in range(2):   # about half of the blocks zero in this order, and the first emitter block row
        for i in range(nb):
            for j in range(nb):
                if i == 0 and nb > 1 or rng.random() < 0.5 and nb > 2:
                    w[k, 32 * i:32 * i + 32, 32 * j:32 * j + 32] = 0.0
    if m == 4:
        w[1] = 0.0       # a frequency without a weight
    g_o, h_o = np.zeros(geom.n_pixels), np.zeros(geom.n_pixels)
    for k, f in enumerate(freqs):
        g_o += born.born_adjoint(G[k], w[k] * D[k], f, geom.h ** 2)
        h_o += born.hessian_diag(G[k], w[k], f, geom.h ** 2)
    d = torch.as_tensor(np.stack([D.real, D.imag], -1), device=DEV)
    wd = torch.as_tensor(w, device=DEV)
    for hess in (True, False):
        grad = torch.zeros(geom.n_pixels, dtype=torch.float64, device=DEV)
        hd = torch.zeros_like(grad) if hess else None
        rb.born_adjoint_weighted(geom, Gr, Gi, sc, dtype, freqs, d, wd, grad, hd)
        close(grad.cpu().numpy(), g_o, TOL[dtype], f"grad {dtype} {shape} hess={hess}")
        if hess:
            close(hd.cpu().numpy(), h_o, TOL[dtype], f"hdiag {dtype} {shape}")


def _random_g(nf, m, N, seed):
    rng = np.random.default_rng(seed)
    mag = np.exp(rng.uniform(np.log(1e-2), 0.0, (nf, m, N)))      # two decades
    ph = rng.uniform(0.0, 2 * np.pi, (nf, m, N))
    return (mag * np.cos(ph)).astype(np.float32), (mag * np.sin(ph)).astype(np.float32)


def _gradient(rb, geom, gr, gi, freqs, D, w):
    grad = torch.zeros(geom.n_pixels, dtype=torch.float64, device=DEV)
    rb.born_adjoint_weighted(geom, torch.as_tensor(gr, device=DEV), torch.as_tensor(gi, device=DEV), None, "f32", freqs,
                             torch.as_tensor(np.stack([D.real, D.imag], -1), device=DEV),
                             torch.as_tensor(w, device=DEV), grad, None)
    return grad.cpu().numpy()


# FP32 gradients large enough for the FP16 matrix cores (k_adjoint_split): odd
# pixel counts and rows that are not 16-byte aligned, the last tile holding 1
# to 127 pixels, rings of whole and partial 32- and 128-element blocks, one and
# several emitter passes per workgroup.  2e-6 is 40 times 2^-24 sqrt(2 rounding
# steps per MFMA of a 1024-receiver row): the FP32 kernel's own bound is 1e-5.
@pytest.mark.parametrize("shape", [(137, 143, 256), (160, 128, 300), (200, 181, 130), (190, 190, 515), (129, 257, 192),
                                   (183, 180, 65), (257, 256, 96)])
def test_fp32_gradient_in_two_fp16_pieces(rb, shape):
    nx, ny, m = shape
    geom, freqs = _geom(nx, ny, m), [3e5, 7e5]
    print(f"[gpu-test] split gradient {shape}", flush=True)
    gr, gi = _random_g(2, m, geom.n_pixels, 7)
    D = W.random_residual(2, m, 8)
    w = np.random.default_rng(9).uniform(0.0, 2.0, (2, m, m))
    w[:, :32, 32:64] = w[:, 32:64, :32] = 0.0
    ref = sum(born.born_adjoint(gr[k] + 1j * gi[k].astype(np.float64), w[k] * D[k], f, geom.h ** 2)
              for k, f in enumerate(freqs))
    close(_gradient(rb, geom, gr, gi, freqs, D, w), ref, 2e-6, f"split gradient {shape}")


def test_fp32_gradient_outside_the_fp16_range(rb):
    """Pixels whose tables a 16-element sample misjudges or that FP16 cannot
    hold: each pixel must be as exact as an FP32 contraction makes it, whatever
    its neighbours hold (errors relative to the pixel's own value)."""
    nx, ny, m = 140, 144, 256
    geom, freqs = _geom(nx, ny, m), [4e5]
    N = geom.n_pixels
    print("[gpu-test] split gradient, wide-ranging tables", flush=True)
    gr, gi = _random_g(1, m, N, 10)
    s = np.ones((m, N), np.float32)
    s[:, :4096] = np.float32(2.0) ** np.random.default_rng(11).integers(-60, 40, 4096)   # any scale per pixel
    s[::16, 5000:5100] = 0.0           # sampled elements see nothing
    s[::16, 6000:6050] = 1e-6          # ... or a millionth
    s[7, 7000:7003] = 3e5              # one element far above the sample
    s[:, 8000:8200] = 0.0              # uncovered by every element
    gr, gi = gr * s, gi * s
    D = W.random_residual(1, m, 12)
    w = np.ones((1, m, m))
    g = gr[0] + 1j * gi[0].astype(np.float64)
    ref = born.born_adjoint(g, D[0], freqs[0], geom.h ** 2)
    size = (2 * np.pi * freqs[0]) ** 2 * geom.h ** 2 * (np.abs(g) * (np.abs(D[0]) @ np.abs(g))).sum(0)
    got = _gradient(rb, geom, gr, gi, freqs, D, w)
    assert np.all(got[8000:8200] == 0.0)
    ok = size > 0
    # |error| <= 2^-24 (sqrt(256) additions + 2 roundings) of the sum of magnitudes
    assert np.max(np.abs(got - ref)[ok] / size[ok]) <= 18 * 2.0 ** -24
    bad = gr.copy()
    bad[0, 9, 33] = np.nan
    bad[0, 9, 9033] = np.inf
    nan = _gradient(rb, geom, bad, gi, freqs, D, w)
    assert not np.isfinite(nan[33]) and not np.isfinite(nan[9033])
    keep = np.ones(N, bool)
    keep[[33, 9033]] = False
    assert np.max(np.abs(nan - ref)[keep & ok] / size[keep & ok]) <= 18 * 2.0 ** -24


def _forward(rb, geom, gr, gi, freqs, delta):
    d = torch.zeros((len(freqs), geom.m, geom.m, 2), dtype=torch.float64, device=DEV)
    rb.born_forward(geom, torch.as_tensor(gr, device=DEV), torch.as_tensor(gi, device=DEV), None, "f32", freqs,
                    torch.as_tensor(delta, device=DEV), d)
    return torch.view_as_complex(d).cpu().numpy()


# Pixel counts with rows of whole 16-byte pieces and without, a last chunk of 1
# to 32 pixels, one and several pixel splits; rings of one 128-element tile, a
# tile and two elements, and three tiles.
@pytest.mark.parametrize("shape", [(64, 80, 128), (67, 71, 130), (97, 103, 128), (75, 59, 300), (160, 129, 256)])
@pytest.mark.parametrize("kind", ["dense", "point", "zero"])
def test_fp32_forward_in_two_fp16_pieces(rb, shape, kind):
    nx, ny, m = shape
    geom, freqs = _geom(nx, ny, m), [3e5, 7e5]
    print(f"[gpu-test] split forward {shape} {kind}", flush=True)
    gr, gi = _random_g(2, m, geom.n_pixels, 13)
    delta = W.random_delta(geom.n_pixels, 14)
    if kind == "point":
        delta[:-1] = 0.0             # the last pixel alone
    if kind == "zero":
        delta[:] = 0.0
    got = _forward(rb, geom, gr, gi, freqs, delta)
    for k, f in enumerate(freqs):
        ref = born.born_forward(gr[k] + 1j * gi[k].astype(np.float64), delta, f, geom.h ** 2)
        assert np.array_equal(got[k], got[k].T)
        if kind == "zero":
            assert np.all(got[k] == 0.0)
        else:
            close(got[k].view(np.float64), ref.view(np.float64), 2e-6, f"split forward {shape} {kind} k={k}")


def test_fp32_forward_outside_the_fp16_range(rb):
    """Rows that a sample of their pixels misjudges, or of any scale: every pair
    as exact as an FP32 contraction makes it, relative to its sum of magnitudes."""
    nx, ny, m = 70, 74, 160
    geom, freqs = _geom(nx, ny, m), [4e5]
    N = geom.n_pixels
    print("[gpu-test] split forward, wide-ranging tables", flush=True)
    gr, gi = _random_g(1, m, N, 15)
    s = np.ones((m, N), np.float32)
    s[:32] = (np.float32(2.0) ** np.random.default_rng(16).integers(-30, 20, 32))[:, None]
    sampled = np.arange(256) * N // 256
    s[40, sampled] = 0.0               # the sample sees nothing
    s[41, sampled] = 1e-5              # ... or a hundred-thousandth
    s[42, 777] = 4e4                   # one pixel far above the rest
    s[150] = 0.0                       # an element that covers nothing
    gr, gi = gr * s, gi * s
    delta = W.random_delta(N, 17)
    g = gr[0] + 1j * gi[0].astype(np.float64)
    c = (2 * np.pi * freqs[0]) ** 2 * geom.h ** 2
    ref = c * (g * delta) @ g.T
    size = c * (np.abs(g) * np.abs(delta)) @ np.abs(g).T
    got = _forward(rb, geom, gr, gi, freqs, delta)[0]
    assert np.all(got[150] == 0.0) and np.all(got[:, 150] == 0.0)
    ok = size > 0
    # |error| <= 2^-24 (sqrt(5180) additions + 2 roundings) of the sum of magnitudes
    assert np.max(np.abs(got - ref)[ok] / size[ok]) <= 74 * 2.0 ** -24
    bad = gr.copy()
    bad[0, 50, 3] = np.inf
    nan = _forward(rb, geom, bad, gi, freqs, delta)[0]
    assert not np.any(np.isfinite(nan[50])) and not np.any(np.isfinite(nan[:, 50]))
    keep = np.ones(m, bool)
    keep[50] = False
    keep = np.outer(keep, keep) & ok
    assert np.max(np.abs(nan - ref)[keep] / size[keep]) <= 74 * 2.0 ** -24


# 16-bit tables with rows that are not 16-byte aligned (odd and even pixel
# counts, a last chunk of 1 to 31 pixels) and, aligned, large enough for the
# same 256 x 128 tiles by direct loads (a last pair of steps of 64, 8 and 24
# pixels); rings of a part of a tile, a tile and two elements, and three rows of
# tiles.
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", [(33, 31, 65), (50, 41, 130), (61, 67, 258), (41, 45, 520), (256, 256, 512), (199, 168, 512),
                                   (181, 184, 700)])
def test_16bit_forward_in_wide_tiles(rb, dtype, shape):
    nx, ny, m = shape
    geom, freqs = _geom(nx, ny, m), [3e5]
    print(f"[gpu-test] wide 16-bit forward {dtype} {shape}", flush=True)
    gr, gi = _random_g(1, m, geom.n_pixels, 18)
    td = rb._binding.TORCH_DTYPES[rb.DTYPES[dtype]]
    tr, ti = torch.as_tensor(gr, device=DEV).to(td), torch.as_tensor(gi, device=DEV).to(td)
    delta = W.random_delta(geom.n_pixels, 19)
    d = torch.zeros((1, m, m, 2), dtype=torch.float64, device=DEV)
    sc = torch.tensor([0.25], dtype=torch.float32, device=DEV)
    rb.born_forward(geom, tr, ti, sc, dtype, freqs, torch.as_tensor(delta, device=DEV), d)
    got = torch.view_as_complex(d).cpu().numpy()[0]
    g = 0.25 * (tr[0].double().cpu().numpy() + 1j * ti[0].double().cpu().numpy())
    ref = born.born_forward(g, delta, freqs[0], geom.h ** 2)
    assert np.array_equal(got, got.T)
    close(got.view(np.float64), ref.view(np.float64), TOL[dtype], f"wide forward {dtype} {shape}")


# The outlier selection of small rings runs in one block per frequency: rings
# of 1024 pairs (one stripe of its threads), of 10000 (a part of the last) and
# of 16384 (all it holds), and one beyond, with ties across the threshold that
# spread over all stripes, so that the flat index decides which are zeroed.
@pytest.mark.parametrize("m", [32, 100, 128, 130])
def test_outlier_selection_with_ties(rb, m):
    from oracle import invert
    p = W.custom(33, 0.5e-3, m, 8e-3, 90, [[2.4e5, 3.1e5]], seed=23)
    topts = W.resolve_trace_opts(p.geom, p.c_start, 90)
    f = p.freq_sets[0]
    print(f"[gpu-test] outlier ties m={m}", flush=True)
    pm = p.p_meas[0].copy()
    sel = np.flatnonzero(invert.receiver_mask(m, p.inv.recv_fraction).reshape(-1))
    kz = int(np.floor(p.inv.outlier_fraction * sel.size))
    rng = np.random.default_rng(m)
    for k in range(2):
        big = np.abs(pm[k]).max()
        tied = rng.choice(sel, size=2 * kz, replace=False)
        pm[k].reshape(-1)[tied] = 2.0 * big * np.exp(0.3j)
        pm[k].reshape(-1)[tied[:kz // 2]] *= 1.5          # half above the ties
    ref, _ = invert.invert_frequency_set(p.geom, topts, p.inv, p.c_start, p.alpha0, f, pm)
    c_in = torch.as_tensor(p.c_start.reshape(-1), device=DEV)
    c_out = torch.empty_like(c_in)
    rb.invert_frequency_set(p.geom, topts, p.inv, "f64", c_in, torch.as_tensor(p.alpha0.reshape(-1), device=DEV), f,
                            torch.as_tensor(np.stack([pm.real, pm.imag], -1), device=DEV), c_out)
    dc = c_out.cpu().numpy() - p.c_start.reshape(-1)
    dc_o = ref.reshape(-1) - p.c_start.reshape(-1)
    # the bound of the tied-outlier test at 64 elements; one pair more or less moves the update by 1e-3
    assert np.linalg.norm(dc - dc_o) <= 1e-6 * np.linalg.norm(dc_o)


# FP64: forward tiles of 64 pairs and 16 pixels (whole, partial and single
# steps, one and several tiles, several splits), backprojection tiles of 64 and,
# from 512 workgroups of them on, 128 pixels.  A sum of n products in FP64 is
# off by at most about n 2^-53 of the sum of their magnitudes: 3.6e-11 for the
# longest here (4 N = 2.6e5 products a pair, 8 m^2 = 3.2e5 a pixel).
@pytest.mark.parametrize("shape", [(3, 5, 4), (4, 4, 64), (21, 13, 65), (40, 25, 130), (17, 15, 200), (257, 256, 33)])
def test_fp64_tiles(rb, shape):
    nx, ny, m = shape
    geom, freqs = _geom(nx, ny, m), [3e5, 7e5]
    N = geom.n_pixels
    print(f"[gpu-test] FP64 tiles {shape}", flush=True)
    rng = np.random.default_rng(N + m)
    G = rng.uniform(-1, 1, (2, m, N)) + 1j * rng.uniform(-1, 1, (2, m, N))
    gr, gi = (torch.as_tensor(np.ascontiguousarray(v), device=DEV) for v in (G.real, G.imag))
    delta = rng.uniform(-1, 1, N)
    D = W.random_residual(2, m, 8)
    w = rng.uniform(0.5, 2.0, (2, m, m))
    wd = w * D
    out = torch.empty((2, m, m, 2), dtype=torch.float64, device=DEV)
    rb.born_forward(geom, gr, gi, None, "f64", freqs, torch.as_tensor(delta, device=DEV), out)
    grad = torch.zeros(N, dtype=torch.float64, device=DEV)
    hd = torch.zeros_like(grad)
    rb.born_adjoint_weighted(geom, gr, gi, None, "f64", freqs, torch.as_tensor(np.stack([D.real, D.imag], -1), device=DEV),
                             torch.as_tensor(w, device=DEV), grad, hd)
    g_o, g_b = np.zeros(N), np.zeros(N)
    h_o = np.zeros(N)
    for k, f in enumerate(freqs):
        want = born.born_forward(G[k], delta, f, geom.h ** 2)
        bound = np.abs(born.born_forward(np.abs(G[k]), np.abs(delta), f, geom.h ** 2))
        got = out[k].cpu().numpy() @ [1, 1j]
        assert (np.abs(got - want) <= 4e-11 * bound).all()
        g_o += born.born_adjoint(G[k], wd[k], f, geom.h ** 2)
        h_o += born.hessian_diag(G[k], w[k], f, geom.h ** 2)
        a = np.abs(G[k])
        g_b += 4e-11 * (2 * np.pi * f) ** 2 * geom.h ** 2 * np.einsum("ex,er,rx->x", a, np.abs(wd[k]), a, optimize=True)
    assert (np.abs(grad.cpu().numpy() - g_o) <= g_b).all()
    assert (np.abs(hd.cpu().numpy() - h_o) <= 4e-11 * h_o).all()


# 16-bit backprojection by direct loads (rows of whole 16-byte pieces, rings of
# whole 32-element blocks) and through registers: a last tile of one 16-byte
# piece, of odd pixels and of one pixel; one, two and many receiver chunks.
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("shape", [(34, 4, 32), (40, 10, 64), (43, 3, 64), (33, 13, 70), (20, 20, 288), (53, 5, 300)])
def test_16bit_gradient_rows(rb, dtype, shape):
    nx, ny, m = shape
    geom, freqs = _geom(nx, ny, m), [3e5, 7e5]
    N = geom.n_pixels
    print(f"[gpu-test] 16-bit gradient rows {dtype} {shape}", flush=True)
    Gr, Gi, sc, G = _tables(rb, geom, freqs, dtype, 15)
    D = W.random_residual(2, m, 16)
    w = np.random.default_rng(N + m).uniform(0.0, 2.0, (2, m, m))
    g_o = sum(born.born_adjoint(G[k], w[k] * D[k], f, geom.h ** 2) for k, f in enumerate(freqs))
    h_o = sum(born.hessian_diag(G[k], w[k], f, geom.h ** 2) for k, f in enumerate(freqs))
    d, wd = (torch.as_tensor(v, device=DEV) for v in (np.stack([D.real, D.imag], -1), w))
    for hess in (True, False):
        grad = torch.zeros(N, dtype=torch.float64, device=DEV)
        hd = torch.zeros_like(grad) if hess else None
        rb.born_adjoint_weighted(geom, Gr, Gi, sc, dtype, freqs, d, wd, grad, hd)
        close(grad.cpu().numpy(), g_o, TOL[dtype], f"grad {dtype} {shape} hess={hess}")
        if hess:
            close(hd.cpu().numpy(), h_o, TOL[dtype], f"hdiag {dtype} {shape}")


# The banded Hessian diagonal at the edges of its block variants (rings up to
# 128, 256, 512, 768 and 1024 elements, above; groups with and without a
# partial last one), of its last pixels' block, of the band (none, one pair,
# part of a group, the whole ring) and of its chunks of zeroed pairs.  Each
# pixel's value is a sum of at most about 200 dependent FP32 (FP64) additions
# of terms whose magnitudes add up to `mag`: 200 2^-24 = 1.2e-5.
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16", "f16"])
@pytest.mark.parametrize("m, dmin, nz", [(5, 0, 3), (33, 5, 70), (64, 64, 0), (129, 1, 513), (250, 32, 1100),
                                         (257, 33, 2049), (500, 62, 5000), (513, 100, 1), (770, 97, 9000),
                                         (1024, 128, 8193), (1030, 129, 600)])
def test_banded_hessian_blocks(rb, dtype, m, dmin, nz):
    geom, freqs = _geom(9, 5, m), [3e5, 7e5]
    N = geom.n_pixels
    print(f"[gpu-test] banded Hessian {dtype} m={m} dmin={dmin} zeroed={nz}", flush=True)
    rng = np.random.default_rng(m)
    td = rb._binding.TORCH_DTYPES[rb.DTYPES[dtype]]
    gr, gi = (torch.as_tensor(rng.uniform(-1, 1, (2, m, N)), device=DEV).to(td) for _ in range(2))
    sc = np.array([0.5, 2.0]) if dtype in ("bf16", "f16") else np.ones(2)
    scale = torch.as_tensor(sc, dtype=torch.float32, device=DEV) if dtype in ("bf16", "f16") else None
    cap = max(nz, 1) + 3
    pairs = rng.integers(0, m, (2, cap, 2)).astype(np.int32)
    pairs[:, 0] = (m, 0)          # out of range: ignored
    n = np.array([nz, max(nz - 1, 0)], dtype=np.int32)
    hd = torch.zeros(N, dtype=torch.float64, device=DEV)
    rb.born_hessian_banded(geom, gr, gi, scale, dtype, freqs, dmin, torch.as_tensor(pairs, device=DEV),
                           torch.as_tensor(n, device=DEV), hd)
    i = np.arange(m)
    dist = np.abs(i[:, None] - i[None, :])
    sel = (np.minimum(dist, m - dist) >= dmin).astype(np.float64)
    want, mag = np.zeros(N), np.zeros(N)
    for k, f in enumerate(freqs):
        G = (gr[k].double().cpu().numpy() + 1j * gi[k].double().cpu().numpy()) * sc[k]
        z = np.zeros((m, m))
        p = pairs[k, 1:n[k]]
        np.add.at(z, (p[:, 0], p[:, 1]), 1.0)
        want += born.hessian_diag(G, sel - z, f, geom.h ** 2)
        mag += born.hessian_diag(G, 2.0 + z, f, geom.h ** 2)
    assert (np.abs(hd.cpu().numpy() - want) <= (200 * 2.0 ** (-53 if dtype == "f64" else -24)) * mag).all()


# FP32 gradient and Hessian diagonal where the gradient takes the FP16 cores:
# the diagonal is a contraction of its own, with tiles of 64 pixels (the last of
# 1 to 64), one and several emitter passes per workgroup.
@pytest.mark.parametrize("shape", [(183, 180, 65), (129, 257, 192), (160, 128, 300)])
def test_fp32_hessian_beside_split_gradient(rb, shape):
    nx, ny, m = shape
    geom, freqs = _geom(nx, ny, m), [3e5, 7e5]
    N = geom.n_pixels
    print(f"[gpu-test] FP32 Hessian beside split gradient {shape}", flush=True)
    gr, gi = _random_g(2, m, N, 21)
    D = W.random_residual(2, m, 22)
    w = np.random.default_rng(23).uniform(0.0, 2.0, (2, m, m))
    w[:, :32, 32:64] = 0.0
    grad, hd = (torch.ones(N, dtype=torch.float64, device=DEV) for _ in range(2))   # both are added to
    rb.born_adjoint_weighted(geom, torch.as_tensor(gr, device=DEV), torch.as_tensor(gi, device=DEV), None, "f32", freqs,
                             torch.as_tensor(np.stack([D.real, D.imag], -1), device=DEV),
                             torch.as_tensor(w, device=DEV), grad, hd)
    G = [gr[k] + 1j * gi[k].astype(np.float64) for k in range(2)]
    g_o = sum(born.born_adjoint(G[k], w[k] * D[k], f, geom.h ** 2) for k, f in enumerate(freqs))
    h_o = sum(born.hessian_diag(G[k], w[k], f, geom.h ** 2) for k, f in enumerate(freqs))
    close(grad.cpu().numpy() - 1.0, g_o, TOL["f32"], f"grad {shape}")
    close(hd.cpu().numpy() - 1.0, h_o, TOL["f32"], f"hdiag {shape}")
