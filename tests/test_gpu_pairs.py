"""The backprojection contracts each unordered (e, r) pair once, with the sum
of the pair's two weighted residuals.  These cases give the two orders of a
pair different data and weights, down to whole 32 x 32 blocks that are zero in
one order only, on rings whose block count is even (two blocks half a ring
apart), odd, and one."""
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
