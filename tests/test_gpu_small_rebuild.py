"""List rebuild of small boxes in one launch (every home cell's block scans
all particles): lists against the oracle's, as sets and bit for bit in the
membership decision, at the edges of its range (12,288 particles is the
largest size it takes) and with ragged shares; and the refusal of an
overfull cell.
"""
import numpy as np
import pytest

import oracle
from paper_2406_04210_amd import workloads as W

pytestmark = pytest.mark.gpu
FP64, FP32_DS = 0, 1


@pytest.fixture(scope="module")
def ljmd():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_04210_amd import ljmd as L
    return L


@pytest.mark.parametrize("prec", [FP64, FP32_DS])
@pytest.mark.parametrize("n,two", [(163, False), (1023, True), (1025, False), (12288, True), (12289, False)])
def test_small_rebuild_lists(ljmd, prec, n, two):
    w = W.thermostat_fluid(n, seed_index=3)
    rng = np.random.default_rng(n)
    x = (w.x + 0.05 * rng.standard_normal(w.x.shape)) % w.box
    sp, p = w.species, w.params
    if two:
        p = W.binary_mixture_params()
        sp = (rng.uniform(size=n) < 0.2).astype(np.int32)
    s = ljmd.System(n, w.box, p, precision=prec)
    s.set_state(x, w.v, sp)
    for _ in range(2):
        cnt, ids = s.neighbors(cap=256)
        s.sync()
        cnt, ids = cnt.cpu().numpy(), ids.cpu().numpy()
        oc, on = oracle.build_lists(x, sp, w.box, p, mode=0 if prec == FP64 else 1, cap=256)
        assert np.array_equal(cnt, oc)
        for i in range(n):
            assert set(ids[i, : cnt[i]].tolist()) == set(on[i, : oc[i]].tolist()), i
        # Again where a run without resorts rebuilt the lists itself.
        obs = s.run(30).cpu().numpy()
        last = int(np.nonzero(obs[:, 6])[0][-1]) + 1
        s = ljmd.System(n, w.box, p, precision=prec, sort_interval=0)
        s.set_state(x, w.v, sp)
        s.run(last, observe=False)
        x = s.get_state()[0].cpu().numpy()


@pytest.mark.parametrize("prec", [FP64, FP32_DS])
def test_small_rebuild_refuses_an_overfull_cell(ljmd, prec):
    p = W.single_species_params()
    L = 3 * (p.rcut[0] + p.skin) * 1.01
    rng = np.random.default_rng(5)
    x = np.concatenate([rng.uniform(0.0, L, size=(100, 3)), rng.uniform(0.1, 0.3 * L, size=(60, 3))])
    s = ljmd.System(len(x), (L, L, L), p, precision=prec, nbr_capacity=384, cell_capacity=32)
    with pytest.raises(ljmd.LJMDError) as err:
        s.set_state(x, np.zeros_like(x), np.zeros(len(x), dtype=np.int32))
    assert err.value.code == -8                       # LJMD_ECELL


@pytest.mark.parametrize("prec", [FP64, FP32_DS])
@pytest.mark.parametrize("cells,two", [(3, False), (5, True)])
def test_reduced_build_with_crowded_cells(ljmd, prec, cells, two):
    # Just above the one-launch size, a dilute gas with a long cutoff: hundreds
    # of particles per cell (several batches of home particles, queues that
    # fill and are moved up many times), with 3 cells per axis (wrapped gap to
    # the groups' boxes) and 5 (signed gap).
    n, L = 12500, 60.0
    p = W.binary_mixture_params() if two else W.single_species_params()
    p.rcut[:] = L / cells / 1.001 - p.skin
    rng = np.random.default_rng(40 + cells)
    x = rng.uniform(0.0, L, size=(n, 3))
    sp = (rng.uniform(size=n) < 0.2).astype(np.int32) if two else np.zeros(n, dtype=np.int32)
    s = ljmd.System(n, (L, L, L), p, precision=prec)
    s.set_state(x, np.zeros_like(x), sp)
    cnt, ids = s.neighbors(cap=2304)
    s.sync()
    cnt, ids = cnt.cpu().numpy(), ids.cpu().numpy()
    oc, on = oracle.build_lists(x, sp, (L, L, L), p, mode=0 if prec == FP64 else 1, cap=2304)
    assert 64 < oc.max() <= 2304
    assert np.array_equal(cnt, oc)
    for i in rng.choice(n, 1500, replace=False):
        assert np.array_equal(np.sort(ids[i, : cnt[i]]), np.sort(on[i, : oc[i]])), i
