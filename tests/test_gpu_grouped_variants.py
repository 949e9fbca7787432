"""Grouped single steps whose problems take the backprojection's other
variants: FP32 rings on the FP16 matrix cores in two pieces (more than 64
elements, more workgroups than compute units), one of them so absorbing that
its tables leave FP16's range and go to the FP32 list, and 16-bit rings of
whole 32-element blocks on pixel counts divisible by 8 (direct loads).  Each
problem's result is bitwise the one it has alone, and that of the FP64 oracle
to the type's accuracy."""
import numpy as np
import pytest

import workload as W
from oracle import invert

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (grid n, ny, m, ring radius, rays, frequencies, seed, dtype, absorption times)
PROBLEMS = [(140, 144, 96, 34e-3, 220, [2.5e5, 3.1e5], 61, "f32", 1.0),
            (137, 141, 130, 33e-3, 220, [2.4e5, 3.3e5], 62, "f32", 1.0),
            (130, 130, 100, 31e-3, 220, [2.6e5, 3.0e5, 3.4e5], 63, "f32", 400.0),
            (64, 64, 64, 14e-3, 120, [2.4e5, 3.0e5], 64, "bf16", 1.0),
            (56, 64, 96, 13e-3, 120, [2.7e5], 65, "bf16", 1.0),
            (64, 40, 64, 14e-3, 120, [2.2e5, 2.9e5], 66, "f16", 1.0),
            (57, 61, 70, 13e-3, 120, [2.9e5], 67, "f16", 1.0)]
TOL = {"f32": 1e-4, "bf16": 1e-2, "f16": 2e-3}   # rel-L2 of the update, as the precision tests


@pytest.fixture(scope="module")
def rb():
    import paper_2511_16633_amd as m
    m.lib()
    return m


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


def _problem(spec):
    n, ny, m, R, nr, fs, seed, dtype, absorb = spec
    p = W.custom(n, 0.5e-3, m, R, nr, [fs], seed=seed, ny=ny)
    return p, W.resolve_trace_opts(p.geom, p.c_start, nr), absorb * p.alpha0


def _job(rb, spec):
    p, topts, alpha = _problem(spec)
    f, dtype = p.freq_sets[0], spec[7]
    ws = torch.empty(rb.invert_workspace_bytes(p.geom, topts, len(f), dtype), dtype=torch.uint8, device=DEV)
    return {"g": p.geom, "t": topts, "o": p.inv, "dtype": dtype, "c_in": _t(p.c_start.reshape(-1)),
            "alpha0": _t(alpha.reshape(-1)), "freqs": f,
            "p_meas": _t(np.stack([p.p_meas[0].real, p.p_meas[0].imag], -1)),
            "c_out": torch.empty(p.geom.n_pixels, dtype=torch.float64, device=DEV), "ws": ws}


def test_grouped_variants_equal_alone(rb):
    print(f"[gpu-test] grouped variants, {len(PROBLEMS)} problems", flush=True)
    alone = []
    for spec in PROBLEMS:
        j = _job(rb, spec)
        nrm = rb.invert_frequency_set(j["g"], j["t"], j["o"], j["dtype"], j["c_in"], j["alpha0"], j["freqs"],
                                      j["p_meas"], j["c_out"], ws=j["ws"])
        alone.append((j["c_out"].cpu().numpy(), nrm))
    jobs = [_job(rb, spec) for spec in PROBLEMS]
    norms = rb.invert_frequency_sets_grouped(jobs)
    for spec, j, (c_a, n_a), n_g in zip(PROBLEMS, jobs, alone, norms):
        assert np.array_equal(j["c_out"].cpu().numpy(), c_a), f"{spec} differs grouped and alone"
        assert n_g == n_a


@pytest.mark.parametrize("i", range(len(PROBLEMS)))
def test_variant_against_the_oracle(rb, i):
    spec = PROBLEMS[i]
    print(f"[gpu-test] variant against the oracle {spec}", flush=True)
    p, topts, alpha = _problem(spec)
    ref, _ = invert.invert_frequency_set(p.geom, topts, p.inv, p.c_start, alpha, p.freq_sets[0], p.p_meas[0])
    j = _job(rb, spec)
    rb.invert_frequency_set(j["g"], j["t"], j["o"], j["dtype"], j["c_in"], j["alpha0"], j["freqs"], j["p_meas"],
                            j["c_out"], ws=j["ws"])
    dc = j["c_out"].cpu().numpy() - p.c_start.reshape(-1)
    dc_o = ref.reshape(-1) - p.c_start.reshape(-1)
    rel = float(np.linalg.norm(dc - dc_o) / np.linalg.norm(dc_o))
    print(f"[gpu-test] rel-L2 of the update {rel:.3e}", flush=True)
    assert rel <= TOL[spec[7]]
