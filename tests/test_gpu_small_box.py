"""The step kernels' form for small boxes (256-thread blocks,
pipelined pair loop; two lanes per particle in FP32, four in FP64) at the edges of its tiles and of
its range: ragged last blocks and rows of partial sums, the largest size it
takes (256 particles per compute unit) and the first it does not.

Expected values: the oracle's forces of the fixed-point positions (tolerance
of test_gpu_parity.py, tests/force_metrics.py; 1e-12 of the rms force against
its plain forces in FP64); and, in FP32 with one species, the
forces and observables of the same box as a batch of one, which the form for
large boxes steps: both add every sum in the same order, so they are equal
bit for bit.
"""
import numpy as np
import pytest

from force_metrics import bound_key, force_errors, reference, report, tie_allowance
from paper_2406_04210_amd import workloads as W

pytestmark = pytest.mark.gpu
FP64, FP32 = 0, 1


@pytest.fixture(scope="module")
def ljmd():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_04210_amd import ljmd as L
    return L


def disordered(n, two):
    w = W.thermostat_fluid(n, seed_index=3)
    rng = np.random.default_rng(n)
    x = (w.x + 0.03 * rng.standard_normal(w.x.shape)) % w.box
    sp, p = w.species, w.params
    if two:
        p = W.binary_mixture_params()
        sp = (rng.uniform(size=n) < 0.2).astype(np.int32)
    return x, w.v, sp, w.box, p


@pytest.mark.parametrize("prec", [FP64, FP32])
@pytest.mark.parametrize("n,two", [(150, False), (255, True), (257, False), (1025, True), (4095, False),
                                   (65536, False), (65537, True)])
def test_small_box_forces_and_observables(ljmd, n, two, prec):
    x, v, sp, box, p = disordered(n, two)
    s = ljmd.System(n, box, p, precision=prec)
    s.set_state(x, v, sp)
    f = s.forces().cpu().numpy()
    ref, _, _, A = reference(x, sp, box, p, prec)
    m = report(f"small box n={n} two={two} prec={prec}", force_errors(f, ref, A, tie_allowance(x, sp, box, p, prec)))
    assert m[bound_key(prec)] <= (1e-12 if prec == FP64 else 1e-5), m
    # Every row of partial sums of every step is written: the observed steps
    # of a run agree with the kinetic energy of the state it ends in.
    obs = s.run(3).cpu().numpy()
    _, vv, _ = s.get_state()
    vv = vv.cpu().numpy()
    K = 0.5 * (vv ** 2).sum()
    assert abs(obs[-1, 1] - K) <= 2e-6 * K
    assert np.array_equal(obs[:, 7], [1.0, 2.0, 3.0])
    if prec == FP32 and not two:
        b = ljmd.Batch([n], [box[0]], p)
        b.set_state(x, v, sp)
        assert np.array_equal(b.forces().cpu().numpy(), f)
        ob = b.run(3, observe=True).cpu().numpy()
        assert np.array_equal(ob[0, :6], obs[-1, :6])
