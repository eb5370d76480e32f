"""List build of a box of more cells than twelve blocks of four waves per compute
unit hold (256 compute units): a wave per cell, lists against the oracle's.
"""
import numpy as np
import pytest

import oracle
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
