"""Launch shapes above 65,536 particles: the step kernel in blocks of
256 or of 1024 threads, by how evenly either loads the compute units, and the
list build with a wave per cell, on both sides of each line (256 compute
units).

Expected values: the same box as a batch of one, which always runs in blocks of
1024 and adds every sum in the same order, so forces and observables are equal
bit for bit; the oracle's forces for two species (tolerance of
test_gpu_parity.py); four lanes per particle for the thermostat; the oracle's
lists.
"""
import numpy as np
import pytest

import oracle
from force_metrics import bound_key, force_errors, reference, report, tie_allowance
from paper_2406_04210_amd import workloads as W

pytestmark = pytest.mark.gpu
FP32_DS = 1


@pytest.fixture(scope="module")
def ljmd():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_04210_amd import ljmd as L
    return L


def disordered(n):
    w = W.thermostat_fluid(n, seed_index=3)
    rng = np.random.default_rng(n)
    return w, (w.x + 0.03 * rng.standard_normal(w.x.shape)) % w.box, rng


@pytest.mark.parametrize("n", [65537, 98304, 98305, 131073, 229376, 229377, 262145, 327680, 327681])
def test_step_blocks_repeat_a_batch_of_one(ljmd, n):
    w, x, _ = disordered(n)
    s = ljmd.System(n, w.box, w.params, precision=FP32_DS)
    s.set_state(x, w.v, w.species)
    b = ljmd.Batch([n], [w.box[0]], w.params)
    b.set_state(x, w.v, w.species)
    assert np.array_equal(b.forces().cpu().numpy(), s.forces().cpu().numpy())
    obs = s.run(3).cpu().numpy()
    assert np.array_equal(b.run(3, observe=True).cpu().numpy()[0, :6], obs[-1, :6])
    s.run(2, observe=False)
    b.run(2)
    assert np.array_equal(b.forces().cpu().numpy(), s.forces().cpu().numpy())


@pytest.mark.parametrize("n", [131073])
def test_step_blocks_two_species(ljmd, n):
    w, x, rng = disordered(n)
    p = W.binary_mixture_params()
    sp = (rng.uniform(size=n) < 0.2).astype(np.int32)
    s = ljmd.System(n, w.box, p, precision=FP32_DS)
    s.set_state(x, w.v, sp)
    ref, _, _, A = reference(x, sp, w.box, p, FP32_DS)
    m = report(f"step blocks n={n}", force_errors(s.forces().cpu().numpy(), ref, A,
                                                  tie_allowance(x, sp, w.box, p, FP32_DS)))
    assert m[bound_key(FP32_DS)] <= 1e-5, m


@pytest.mark.parametrize("n", [65537, 100001])
def test_step_blocks_thermostat(ljmd, n):
    w, x, _ = disordered(n)
    out = []
    for lanes in (2, 4):
        s = ljmd.System(n, w.box, w.params, precision=FP32_DS, lanes=lanes)
        s.set_thermostat(1.0, 20.0, 7)
        s.set_state(x, w.v, w.species)
        f = s.forces().cpu().numpy()
        s.run(3, observe=False)
        out.append(s.get_state()[1].cpu().numpy())
    # Both draw the same collisions; a step adds at most a force error of 1e-5
    # of the largest force on either side, times dt / m.
    tol = 3 * 2 * 1e-5 * np.abs(f).max() * w.params.dt / min(w.params.mass)
    assert np.abs(out[0] - out[1]).max() <= tol


def test_list_build_of_a_wave_per_cell(ljmd):
    n = 270000  # 13,824 cells
    w, x, _ = disordered(n)
    s = ljmd.System(n, w.box, w.params, precision=FP32_DS)
    s.set_state(x, w.v, w.species)
    cnt, ids = s.neighbors(cap=192)
    s.sync()
    oc, on = oracle.build_lists(x, w.species, w.box, w.params, mode=1, cap=192)
    cnt, ids = cnt.cpu().numpy(), ids.cpu().numpy()
    assert np.array_equal(cnt, oc)
    k = np.arange(192)[None, :] < cnt[:, None]
    big = np.int64(n)
    assert np.array_equal(np.sort(np.where(k, ids, big), 1), np.sort(np.where(k, on, big), 1))


@pytest.mark.parametrize("lanes", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("n", [513, 1024])
def test_pair_passes_by_lanes(ljmd, n, lanes):
    """Force adjoint, reverse sweep and steepest descent at every number of
    lanes per particle (their blocks follow it), FP64: against the oracle's
    adjoint and against the default four lanes. Sums of about 80 terms in
    another order: 1e-12 of the largest value, and 1e-10 after several steps."""
    w, x, rng = disordered(n)
    g = rng.standard_normal((n, 3))

    def passes(k):
        s = ljmd.System(n, w.box, w.params, precision=0, lanes=k)
        s.set_state(x, w.v, w.species)
        gx, gth = (t.cpu().numpy() for t in s.force_vjp(g))
        s.vv_forward(4, 2)
        back = [t.cpu().numpy() for t in s.vv_backward(g, 0.1 * g)]
        s.set_state(x, w.v, w.species)
        fm = s.minimize_sd(4).cpu().numpy()
        return gx, gth, back, fm, s.get_state()[0].cpu().numpy()

    gx, gth, back, fm, xr = passes(lanes)
    ox, ge, gs = oracle.force_vjp(x, w.species, w.box, w.params, g)
    assert np.abs(gx - ox).max() <= 1e-12 * np.abs(ox).max()
    assert abs(gth[0] - ge[0]) <= 1e-12 * np.abs(ox).max() * n and abs(gth[3] - gs[0]) <= 1e-12 * np.abs(ox).max() * n
    _, _, back4, fm4, xr4 = passes(4)
    for a, b in zip(back, back4):
        assert np.abs(a - b).max() <= 1e-10 * max(1.0, np.abs(b).max())
    assert np.abs(fm - fm4).max() <= 1e-10 * fm4.max()
    assert np.abs(xr - xr4).max() <= 1e-10 * w.box[0]


@pytest.mark.parametrize("prec", [0, FP32_DS])
@pytest.mark.parametrize("n", [65, 1537, 2049, 8000, 12289])
def test_all_pairs_splits(ljmd, n, prec):
    """All-to-all forces, energy and a step where the number of splits of the
    partners changes: one, one less or many more than two blocks per compute
    unit need, ragged last splits (tolerances of test_gpu_allpairs.py). The
    positions are off the lattice: pairs exactly half a box apart have no
    nearest image."""
    w = W.all_pairs_fluid(n=n, seed_index=3)
    x = (w.x + 0.03 * np.random.default_rng(n).standard_normal(w.x.shape)) % w.box
    s = ljmd.System(n, w.box, w.params, precision=prec)
    s.set_state(x, w.v, w.species)
    f = s.forces().cpu().numpy()
    o = s.observables()
    ref, U, Wv, A = reference(x, w.species, w.box, w.params, prec)
    m = report(f"all pairs n={n} prec={prec}", force_errors(f, ref, A))
    assert m[bound_key(prec)] <= (1e-12 if prec == 0 else 1e-5), m
    tol = 1e-12 if prec == 0 else 5e-6
    assert abs(o["U"] - U) <= tol * abs(U) and abs(o["W"] - Wv) <= tol * abs(Wv)
    obs = s.run(2).cpu().numpy()
    v = s.get_state()[1].cpu().numpy()
    K = 0.5 * (v ** 2).sum()
    assert abs(obs[-1, 1] - K) <= 2e-6 * K
