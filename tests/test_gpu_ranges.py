"""FP32 contractions on operands of a wide range.  The contractions of larger
rings run on the FP16 matrix cores in two pieces per operand; FP16 holds 40
binary orders, FP32 more than 250, and a call must return what FP32 operands
give whatever part of a table its sums use.  Errors are measured against each
result's sum of magnitudes: sums of n random products rounded to FP32 are off
by about 2^-24 (sqrt(n) additions and 2 roundings) of it at most.
"""
import dataclasses

import numpy as np
import pytest
import torch

import workload as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def rb():
    import paper_2511_16633_amd as m
    return m


def _geom(nx, ny, m):
    g = W.centred_grid(nx, 0.5e-3, m, 12e-3, 1500.0)
    return dataclasses.replace(g, ny=ny, y0=-0.5 * (ny - 1) * 0.5e-3)


def _random_g(m, N, seed):
    rng = np.random.default_rng(seed)
    mag = np.exp(rng.uniform(np.log(1e-2), 0.0, (m, N)))
    ph = rng.uniform(0.0, 2 * np.pi, (m, N))
    return mag * np.cos(ph), mag * np.sin(ph)


def _forward(rb, geom, gr, gi, f, delta):
    d = torch.zeros((1, geom.m, geom.m, 2), dtype=torch.float64, device=DEV)
    rb.born_forward(geom, torch.as_tensor(gr[None], dtype=torch.float32, device=DEV),
                    torch.as_tensor(gi[None], dtype=torch.float32, device=DEV), None, "f32", [f],
                    torch.as_tensor(delta, device=DEV), d)
    return torch.view_as_complex(d).cpu().numpy()[0]


def _check_forward(rb, geom, gr, gi, delta, rows=None):
    f = 4e5
    gr, gi = gr.astype(np.float32), gi.astype(np.float32)
    g = gr + 1j * gi.astype(np.float64)
    c = (2 * np.pi * f) ** 2 * geom.h ** 2
    got = _forward(rb, geom, gr, gi, f, delta)
    rows = np.arange(geom.m) if rows is None else rows
    ref = c * (g[rows] * delta) @ g[rows].T
    size = c * (np.abs(g[rows]) * np.abs(delta)) @ np.abs(g[rows]).T
    err = np.abs(got[np.ix_(rows, rows)] - ref)
    ok = size > 0
    assert np.all(err[~ok] == 0.0)
    worst = float(np.max(err[ok] / size[ok]))
    print(f"[gpu-test] worst error {worst:.2e} of the sum of magnitudes", flush=True)
    assert worst <= (np.sqrt(geom.n_pixels) + 2) * 2.0 ** -24
    return got


# Tables that are loud where delta is zero (near the elements, outside of the
# support) and quiet where it counts, by 60 to 200 dB; two and three blocks of
# 128 rows, rows of whole 16-byte pieces and not.
@pytest.mark.parametrize("shape", [(96, 90, 130), (93, 97, 300)])
@pytest.mark.parametrize("db", [60, 100, 140, 200])
def test_forward_loud_where_delta_is_zero(rb, shape, db):
    nx, ny, m = shape
    geom = _geom(nx, ny, m)
    N = geom.n_pixels
    print(f"[gpu-test] forward, loud where delta is zero, {shape} {db} dB", flush=True)
    gr, gi = _random_g(m, N, 1)
    rng = np.random.default_rng(2)
    counts = rng.random(N) < 0.5
    s = np.where(counts, 10.0 ** (-db / 20), 1.0)
    delta = W.random_delta(N, 3) * counts
    _check_forward(rb, geom, gr * s, gi * s, delta)


# The same with a delta that is small, not zero, where the table is loud, and
# with a delta that falls off without end; one pixel alone; both with an element
# that covers nothing.
@pytest.mark.parametrize("shape", [(96, 90, 130), (93, 97, 300)])
@pytest.mark.parametrize("kind", ["small", "tail", "point"])
def test_forward_of_a_wide_ranging_delta(rb, shape, kind):
    nx, ny, m = shape
    geom = _geom(nx, ny, m)
    N = geom.n_pixels
    print(f"[gpu-test] forward, wide-ranging delta, {shape} {kind}", flush=True)
    gr, gi = _random_g(m, N, 4)
    gr[7] = gi[7] = 0.0
    rng = np.random.default_rng(5)
    delta = W.random_delta(N, 6)
    if kind == "small":
        loud = rng.random(N) < 0.3
        s = np.where(loud, 1e6, 1.0)
        gr, gi = gr * s, gi * s
        delta = delta * np.where(loud, 1e-11, 1.0)
    elif kind == "tail":
        x, y = np.meshgrid(np.arange(nx) - nx / 2, np.arange(ny) - ny / 2)
        delta = delta * np.exp(-0.5 * (x ** 2 + y ** 2) / 25.0).reshape(-1)
    else:
        delta[:] = 0.0
        delta[N // 2 + 3] = 1e-8
        gr[:, N // 2 + 3] *= 1e-7
        gi[:, N // 2 + 3] *= 1e-7
    _check_forward(rb, geom, gr, gi, delta)


def test_forward_keeps_infinities_to_their_rows(rb):
    geom = _geom(96, 90, 200)
    print("[gpu-test] forward, one infinite value", flush=True)
    gr, gi = _random_g(200, geom.n_pixels, 7)
    gr[50, 333] = np.inf
    rows = np.delete(np.arange(200), 50)
    with np.errstate(invalid="ignore"):
        got = _check_forward(rb, geom, gr, gi, W.random_delta(geom.n_pixels, 8), rows)
    assert not np.any(np.isfinite(got[50])) and not np.any(np.isfinite(got[:, 50]))


# FP32 tables of one sign, whose sums only grow: what the kernel keeps in FP32
# are the sums of at most 16 pixels (a rounding per 4, each at most 2^-24 of a
# partial sum, rms 0.42 2^-24: together 0.6 2^-24 of the 16 pixels' sum), and the N /
# 16 of them, and the rounded products, are as good as independent: 1.4 2^-24 /
# sqrt(N / 16) is 8e-9 at the smallest grid here, and a third of 2^-24 far above
# it.  Sums of 512 pixels would be off by 2.7 2^-24 each.
@pytest.mark.parametrize("shape", [(41, 82, 20), (40, 80, 16), (72, 36, 80), (96, 76, 144)])
def test_forward_of_small_grids_sums_in_fp64(rb, shape):
    nx, ny, m = shape
    geom, f = _geom(nx, ny, m), 4e5
    N = geom.n_pixels
    print(f"[gpu-test] forward of one sign {shape}", flush=True)
    rng = np.random.default_rng(9)
    gr = rng.uniform(0.5, 1.0, (m, N)).astype(np.float32)
    delta = rng.uniform(0.5e-8, 1e-8, N)
    got = _forward(rb, geom, gr, np.zeros_like(gr), f, delta)
    g = gr.astype(np.float64)
    ref = (2 * np.pi * f) ** 2 * geom.h ** 2 * (g * delta) @ g.T
    rel = float(np.linalg.norm(got.real - ref) / np.linalg.norm(ref))
    print(f"[gpu-test] {rel:.2e}", flush=True)
    assert np.all(got.imag == 0.0) and rel <= 2.0 ** -24 / 3


# The same where the 16 pixels' sums are added in FP64 within a split: a last step of
# 12 and of 4 pixels, the largest grid that takes this kernel (64 pixels for each of 16
# splits a compute unit, 256 of them) and the next, which adds at most 80 pixels in
# FP32: 20 roundings, 1.1 2^-24 of their sum, / sqrt(N / 80), 2 % of 2^-24.
@pytest.mark.parametrize("shape", [(34, 30, 64), (20, 33, 33), (512, 512, 16), (516, 512, 16)])
def test_forward_sums_of_steps(rb, shape):
    test_forward_of_small_grids_sums_in_fp64(rb, shape)


def _check_gradient(rb, geom, gr, gi, D, w, pixels=slice(None)):
    f = 4e5
    gr, gi = gr.astype(np.float32), gi.astype(np.float32)
    g = gr + 1j * gi.astype(np.float64)
    c = (2 * np.pi * f) ** 2 * geom.h ** 2
    grad = torch.zeros(geom.n_pixels, dtype=torch.float64, device=DEV)
    rb.born_adjoint_weighted(geom, torch.as_tensor(gr[None], device=DEV), torch.as_tensor(gi[None], device=DEV), None,
                             "f32", [f], torch.as_tensor(np.stack([D.real, D.imag], -1)[None], device=DEV),
                             torch.as_tensor(np.ascontiguousarray(w[None]), device=DEV), grad, None)
    ref = c * (np.conj(g) * ((w * D) @ np.conj(g))).sum(0).real
    size = c * (np.abs(g) * (np.abs(w * D) @ np.abs(g))).sum(0)
    err, size = np.abs(grad.cpu().numpy() - ref)[pixels], size[pixels]
    ok = size > 0
    assert np.all(err[~ok] == 0.0)
    worst = float(np.max(err[ok] / size[ok]))
    print(f"[gpu-test] worst error {worst:.2e} of the sum of magnitudes", flush=True)
    assert worst <= (np.sqrt(geom.m) + 2) * 2.0 ** -24


# Elements that are loud at a pixel and carry no weight beside quiet ones that
# do, by 60 to 200 dB: any of the elements, and the near part of the ring under
# a receiver selection.  One and several emitter passes per workgroup.
@pytest.mark.parametrize("shape", [(190, 190, 96), (140, 144, 256)])
@pytest.mark.parametrize("db", [60, 100, 140, 200])
@pytest.mark.parametrize("kind", ["unweighted", "ring"])
def test_gradient_loud_where_the_weight_is_zero(rb, shape, db, kind):
    nx, ny, m = shape
    geom = _geom(nx, ny, m)
    N = geom.n_pixels
    print(f"[gpu-test] gradient, loud where the weight is zero, {shape} {db} dB {kind}", flush=True)
    gr, gi = _random_g(m, N, 10)
    rng = np.random.default_rng(11)
    D = W.random_residual(1, m, 12)[0]
    if kind == "unweighted":
        loud = rng.random(m) < 0.3
        loud[::m // 16] = True
        s = np.where(loud, 1.0, 10.0 ** (-db / 20))[:, None]
        w = np.outer(~loud, ~loud) * rng.uniform(0.5, 1.0, (m, m))
    else:
        i = np.arange(m)
        d = np.abs(i[:, None] - i[None, :])
        d = np.minimum(d, m - d)
        s = 10.0 ** (-db / 20 * d[rng.integers(0, m, N)].T / (m // 2))
        w = (d >= m // 8).astype(np.float64)
    _check_gradient(rb, geom, gr * s, gi * s, D, w)


# Tables and residuals far from 1 whose gradient is not.
@pytest.mark.parametrize("shape", [(190, 190, 96), (140, 144, 256)])
@pytest.mark.parametrize("kind", ["large", "small"])
def test_gradient_of_any_scale(rb, shape, kind):
    nx, ny, m = shape
    geom = _geom(nx, ny, m)
    print(f"[gpu-test] gradient, {kind} tables, {shape}", flush=True)
    gr, gi = _random_g(m, geom.n_pixels, 13)
    D = W.random_residual(1, m, 14)[0]
    if kind == "large":
        gr, gi, D = gr * 2.0 ** 112, gi * 2.0 ** 112, D * 2.0 ** -110
    else:
        gr, gi, D = gr * 2.0 ** -55, gi * 2.0 ** -55, D * 2.0 ** 60
    _check_gradient(rb, geom, gr, gi, D, np.ones((m, m)))


# Residuals that are loud at elements which do not reach half of the pixels, at
# those: the others' sums are of a few loud terms, which the bound is not for.
@pytest.mark.parametrize("shape", [(190, 190, 96), (140, 144, 256)])
@pytest.mark.parametrize("db", [60, 120, 180, 240])
def test_gradient_of_a_wide_ranging_residual(rb, shape, db):
    nx, ny, m = shape
    geom = _geom(nx, ny, m)
    N = geom.n_pixels
    print(f"[gpu-test] gradient, wide-ranging residual, {shape} {db} dB", flush=True)
    gr, gi = _random_g(m, N, 13)
    D = W.random_residual(1, m, 14)[0]
    c = [3, m // 2, m - 1]
    D[c] *= 10.0 ** (db / 20)
    D[:, c] *= 10.0 ** (db / 20)
    gr[c, :N // 2] = gi[c, :N // 2] = 0.0
    _check_gradient(rb, geom, gr, gi, D, np.ones((m, m)), slice(0, N // 2))


# The FP32 Hessian diagonal of a small ring.  The sum over the receivers is one of
# up to m / 4 FP32 additions of growing sums (rms 0.42 2^-24 sqrt(m / 12): 1.2 2^-24
# at 100 elements), with its products' roundings 1.4 2^-24, different for every
# emitter, over whom it is summed in FP64: 0.14 2^-24, and twice that is allowed.
# With the emitters' terms summed in FP32 by eight threads (16 additions each, 1.0
# 2^-24, together 0.35) it would be more.
@pytest.mark.parametrize("shape", [(92, 92, 100), (190, 190, 100), (80, 40, 100)])
def test_fp32_hessian_of_small_rings_sums_in_fp64(rb, shape):
    nx, ny, m = shape
    geom, f = _geom(nx, ny, m), 4e5
    N = geom.n_pixels
    print(f"[gpu-test] FP32 Hessian diagonal {shape}", flush=True)
    rng = np.random.default_rng(15)
    gr, gi = (rng.uniform(0.5, 1.0, (1, m, N)).astype(np.float32) for _ in range(2))
    D = W.random_residual(1, m, 16)
    w = rng.uniform(0.5, 1.0, (1, m, m))
    grad, hd = (torch.zeros(N, dtype=torch.float64, device=DEV) for _ in range(2))
    rb.born_adjoint_weighted(geom, torch.as_tensor(gr, device=DEV), torch.as_tensor(gi, device=DEV), None, "f32", [f],
                             torch.as_tensor(np.stack([D.real, D.imag], -1), device=DEV),
                             torch.as_tensor(w, device=DEV), grad, hd)
    p = gr[0].astype(np.float64) ** 2 + gi[0].astype(np.float64) ** 2
    c = (2 * np.pi * f) ** 2 * geom.h ** 2
    ref = c * c * (p * (w[0] @ p)).sum(0)
    rel = float(np.linalg.norm(hd.cpu().numpy() - ref) / np.linalg.norm(ref))
    print(f"[gpu-test] {rel:.2e}", flush=True)
    assert rel <= 0.28 * 2.0 ** -24


# The 16-bit Hessian diagonal under weights that vary.  Contracted in both orders of
# a pair, its error is that of m rounded |G|^2 (uniform over half a last place of
# numbers of any mantissa: rms 0.42 2^-p, p the type's bits), each on 1 / m of the
# sum: 0.42 2^-p / sqrt(m), and m^2 rounded weights, sqrt(m) times less.  Contracted
# once per pair, it must not be more.
@pytest.mark.parametrize("dtype, bits", [("bf16", 8), ("f16", 11)])
@pytest.mark.parametrize("shape", [(72, 72, 48), (88, 88, 64), (96, 64, 96), (72, 72, 130), (60, 61, 227)])
def test_16bit_hessian_of_varied_weights(rb, dtype, bits, shape):
    nx, ny, m = shape
    geom, f = _geom(nx, ny, m), 4e5
    N = geom.n_pixels
    print(f"[gpu-test] 16-bit Hessian diagonal {dtype} {shape}", flush=True)
    rng = np.random.default_rng(17)
    td = torch.bfloat16 if dtype == "bf16" else torch.float16
    mag, ph = np.exp2(rng.uniform(-1.0, 0.0, (1, m, N))), rng.uniform(0.0, 2 * np.pi, (1, m, N))
    gr, gi = (torch.as_tensor(v, device=DEV).to(td) for v in (mag * np.cos(ph), mag * np.sin(ph)))
    D = W.random_residual(1, m, 18)
    w = rng.uniform(0.5, 1.0, (1, m, m))
    grad, hd = (torch.zeros(N, dtype=torch.float64, device=DEV) for _ in range(2))
    rb.born_adjoint_weighted(geom, gr, gi, torch.ones(1, device=DEV), dtype, [f],
                             torch.as_tensor(np.stack([D.real, D.imag], -1), device=DEV),
                             torch.as_tensor(w, device=DEV), grad, hd)
    p = (gr[0].double() ** 2 + gi[0].double() ** 2).cpu().numpy()
    c = (2 * np.pi * f) ** 2 * geom.h ** 2
    ref = c * c * (p * (w[0] @ p)).sum(0)
    rel = float(np.linalg.norm(hd.cpu().numpy() - ref) / np.linalg.norm(ref))
    print(f"[gpu-test] {rel * 2.0 ** bits * np.sqrt(m):.3f} of 2^-{bits} / sqrt(m)", flush=True)
    assert rel <= 0.45 * 2.0 ** -bits / np.sqrt(m)


# The 16-bit gradient of residuals that are reciprocal but for noise.  Contracted in
# both orders of a pair, its two values are rounded apart (rms 0.42 2^-p each): 0.30
# 2^-p of their sum, and of the gradient, a sum of independent such terms.  Contracted
# once per pair, it must not be more (rounded once: 0.42).
@pytest.mark.parametrize("dtype, bits", [("bf16", 8), ("f16", 11)])
@pytest.mark.parametrize("shape", [(72, 72, 64), (72, 72, 130), (60, 61, 200), (64, 40, 256)])
def test_16bit_gradient_of_reciprocal_residuals(rb, dtype, bits, shape):
    nx, ny, m = shape
    geom, f = _geom(nx, ny, m), 4e5
    N = geom.n_pixels
    print(f"[gpu-test] 16-bit gradient, reciprocal residual {dtype} {shape}", flush=True)
    rng = np.random.default_rng(19)
    td = torch.bfloat16 if dtype == "bf16" else torch.float16
    mag, ph = np.exp2(rng.uniform(-1.0, 0.0, (1, m, N))), rng.uniform(0.0, 2 * np.pi, (1, m, N))
    gr, gi = (torch.as_tensor(v, device=DEV).to(td) for v in (mag * np.cos(ph), mag * np.sin(ph)))
    D = rng.standard_normal((m, m)) + 1j * rng.standard_normal((m, m))
    D = (D + D.T) * (1.0 + 0.05 * rng.standard_normal((m, m)))
    grad = torch.zeros(N, dtype=torch.float64, device=DEV)
    rb.born_adjoint_weighted(geom, gr, gi, torch.ones(1, device=DEV), dtype, [f],
                             torch.as_tensor(np.stack([D.real, D.imag], -1)[None], device=DEV),
                             torch.ones((1, m, m), dtype=torch.float64, device=DEV), grad, None)
    g = (gr[0].double() + 1j * gi[0].double()).cpu().numpy()
    ref = (2 * np.pi * f) ** 2 * geom.h ** 2 * (np.conj(g) * (D @ np.conj(g))).sum(0).real
    rel = float(np.linalg.norm(grad.cpu().numpy() - ref) / np.linalg.norm(ref))
    print(f"[gpu-test] {rel * 2.0 ** bits:.3f} of 2^-{bits}", flush=True)
    assert rel <= 0.33 * 2.0 ** -bits
