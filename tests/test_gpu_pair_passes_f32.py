"""Single-precision pair passes at every number of lanes per particle, with
particle counts whose last chunk is ragged and one and two species: steepest
descent (whole groups of list entries loaded past a list's end), force adjoint
and reverse sweep (blocks of 256 threads up to four lanes, 1,024 above) against
the oracle, with the tolerances of test_gpu_parity.py and test_gpu_adjoint.py.
"""
import numpy as np
import pytest

import oracle
from paper_2406_04210_amd import workloads as W
from test_gpu_adjoint import (CASES, FP32, TOL_ROLL, TOL_TH, TOL_VJP, check_theta, rel_err, rollout_case_mixture,
                              vjp_tie_allowance)

pytestmark = pytest.mark.gpu
LANES = [1, 2, 4, 8, 16]


@pytest.fixture(scope="module")
def ljmd():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_04210_amd import ljmd as L
    return L


@pytest.mark.parametrize("lanes", LANES)
@pytest.mark.parametrize("n,two", [(777, False), (1501, True)])
def test_steepest_descent(ljmd, lanes, n, two):
    w = W.config_mixture(n=n, seed_index=2) if two else W.random_dense(n, 0.8442, seed=22, min_dist=0.7)
    s = ljmd.System(n, w.box, w.params, precision=FP32, lanes=lanes)
    s.set_state(w.x, np.zeros_like(w.x), w.species)
    fm = s.minimize_sd(30, 0.01, 0.6).cpu().numpy()
    xu = s.unwrapped_positions().cpu().numpy()
    r = oracle.minimize_sd(w.x, w.species, w.box, w.params, 30, delta=0.01, clamp=0.6)
    assert np.abs(fm - r["fmax"][:30]).max() <= 1e-5 * r["fmax"][0]
    assert np.abs(xu - r["x"]).max() <= 1e-4


@pytest.mark.parametrize("lanes", LANES)
@pytest.mark.parametrize("case", CASES[1:], ids=[c[0] for c in CASES[1:]])
def test_force_vjp(ljmd, lanes, case):
    name, x, sp, box, p = case
    s = ljmd.System(len(x), box, p, precision=FP32, lanes=lanes)
    s.set_state(x, np.zeros_like(x), sp)
    g = np.random.default_rng(31).standard_normal(x.shape)
    gx, gth = (t.cpu().numpy() for t in s.force_vjp(g))
    ox, ge, gs = oracle.force_vjp(x, sp, box, p, g)
    err = rel_err(gx, ox, vjp_tie_allowance(x, sp, box, p, g, FP32))
    print(f"vjp {name} lanes={lanes} max rel err {err:.3e}", flush=True)
    assert err <= TOL_VJP[FP32], err
    check_theta(gth, ge, gs, p.nspecies, TOL_TH[FP32], f"{name} lanes={lanes}")


@pytest.mark.parametrize("lanes", LANES)
def test_reverse_sweep(ljmd, lanes):
    x, v, sp, box, p = rollout_case_mixture()
    x, v, sp = x[:-3], v[:-3], sp[:-3]  # 497: a ragged last chunk at every number of lanes
    rng = np.random.default_rng(63)
    lam_x, lam_v = rng.standard_normal(x.shape), rng.standard_normal(x.shape)
    s = ljmd.System(len(x), box, p, precision=FP32, lanes=lanes)
    s.set_state(x, v, sp)
    s.vv_forward(12, 5)
    gx0, gv0, gth = (t.cpu().numpy() for t in s.vv_backward(lam_x, lam_v))
    ox, ov, ge, gs = oracle.vv_adjoint(x, v, sp, box, p, 12, lam_x, lam_v)
    assert np.abs(gx0 - ox).max() <= TOL_ROLL[FP32] * np.abs(ox).max()
    assert np.abs(gv0 - ov).max() <= TOL_ROLL[FP32] * np.abs(ov).max()
    ref = np.concatenate([ge, gs])
    assert np.all(np.abs(gth - ref) <= TOL_ROLL[FP32] * (np.abs(ref) + 1.0))
