"""Boxes of many cells and few particles: the forms of the list build on both
sides of the lines that cells draw, and a box of millions of cells.
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


def gas(n, edge, dim, seed):
    """n particles at a Maxwellian of T = 1 on sites of a square or cubic lattice
    that fills the box, kept by a seeded permutation and jittered; where the
    sites are far apart, two particles 1.1 apart at each."""
    rng = np.random.default_rng(seed)
    pairs = n % 2 == 0 and edge / np.ceil((n / 2) ** (1.0 / dim)) > 3.5
    k = n // 2 if pairs else n
    m = int(np.ceil(k ** (1.0 / dim) - 1e-9))
    a = edge / m
    g = np.stack(np.meshgrid(*[np.arange(m)] * dim, indexing="ij"), -1).reshape(-1, dim)
    room = 0.5 * (a - 3.2) if pairs else min(0.4, max(0.02, 0.4 * (a - 0.95)))
    c = a * g[np.sort(rng.permutation(len(g))[:k])] + rng.uniform(-room, room, (k, dim))
    if pairs:
        d = rng.standard_normal((k, dim))
        d *= 0.55 / np.linalg.norm(d, axis=1)[:, None]
        c = np.concatenate([c - d, c + d])
    x, v = np.zeros((n, 3)), np.zeros((n, 3))
    x[:, :dim] = c % edge
    v[:, :dim] = rng.standard_normal((n, dim))
    return x, v


def check_lists(s, x, sp, box, p, prec):
    cnt, ids = s.neighbors(cap=128)
    s.sync()
    cnt, ids = cnt.cpu().numpy(), ids.cpu().numpy()
    oc, on = oracle.build_lists(x, sp, box, p, mode=0 if prec == FP64 else 1, cap=128)
    assert np.array_equal(cnt, oc)
    k = np.arange(128)[None, :] < cnt[:, None]
    far = np.int64(len(x))
    assert np.array_equal(np.sort(np.where(k, ids, far), 1), np.sort(np.where(k, on, far), 1))


@pytest.mark.parametrize("prec", [FP64, FP32_DS])
@pytest.mark.parametrize("n,cells,dim", [
    (500, 11, 3), (500, 12, 3), (6000, 10, 3), (6000, 11, 3), (12288, 8, 3), (12288, 9, 3),
    (4500, 38, 2), (4500, 39, 2), (8000, 41, 2), (8000, 42, 2), (3000, 30, 3), (12288, 60, 3)])
def test_lists_by_cells(ljmd, prec, n, cells, dim):
    edge = 2.8 * 1.001 * cells
    x, v = gas(n, edge, dim, n + cells)
    p = W.single_species_params()
    p.dim = dim
    box = (edge, edge, edge if dim == 3 else 10.0)
    sp = np.zeros(n, dtype=np.int32)
    s = ljmd.System(n, box, p, precision=prec, sort_interval=0)
    assert ljmd.cell_grid(s.params) == (cells, cells, cells if dim == 3 else 1)
    s.set_state(x, v, sp)
    check_lists(s, x, sp, box, p, prec)
    # Again where the run rebuilt the lists itself.
    obs = s.run(25).cpu().numpy()
    last = int(np.nonzero(obs[:, 6])[0][-1]) + 1
    s.set_state(x, v, sp)
    s.run(last, observe=False)
    check_lists(s, s.get_state()[0].cpu().numpy(), sp, box, p, prec)


@pytest.mark.parametrize("prec", [FP64, FP32_DS])
def test_millions_of_cells(ljmd, prec):
    # 164 cells along each edge: a block of 1,024 threads for each would be more
    # threads than a launch may have.
    n, cells = 300, 164
    edge = 2.8 * 1.001 * cells
    x, v = gas(n, edge, 3, 7)
    p = W.single_species_params()
    s = ljmd.System(n, (edge,) * 3, p, precision=prec, cell_capacity=8)
    assert np.prod(ljmd.cell_grid(s.params)) * 1024 >= 1 << 32
    s.set_state(x, v, np.zeros(n, dtype=np.int32))
    cnt = s.neighbors(cap=16)[0].cpu().numpy()
    assert np.array_equal(cnt, oracle.build_lists(x, np.zeros(n, dtype=np.int32), (edge,) * 3, p,
                                                  mode=0 if prec == FP64 else 1, cap=16)[0])
    assert cnt.min() == 1
    obs = s.run(20).cpu().numpy()
    s.sync()
    assert obs[:, 6].any()
    r = oracle.run_nve(x, v, np.zeros(n, dtype=np.int32), (edge,) * 3, p, 20)
    tol = 1e-10 if prec == FP64 else 1e-4  # as test_gpu_parity.py
    assert np.abs(s.unwrapped_positions().cpu().numpy() - r["x"]).max() <= tol


@pytest.mark.parametrize("prec,two", [(FP64, False), (FP64, True), (FP32_DS, False), (FP32_DS, True)])
@pytest.mark.parametrize("n,cells,dim", [(20735, 24, 3), (20736, 24, 3), (5000, 23, 3), (19860, 31, 3),
                                         (15000, 55, 3), (20000, 190, 2)])
def test_lists_of_many_cells(ljmd, prec, two, n, cells, dim):
    # A wave per cell (up to 12,288 cells, or at least two particles for three
    # cells), and a grid that strides over them: on both sides of either line,
    # and where one wave takes fourteen.
    edge = 2.8 * 1.001 * cells
    x, v = gas(n, edge, dim, n + cells)
    p = W.binary_mixture_params() if two else W.single_species_params()
    p.rcut[:] = 2.5
    p.dim = dim
    box = (edge, edge, edge if dim == 3 else 10.0)
    sp = (np.random.default_rng(n).uniform(size=n) < 0.2).astype(np.int32) if two else np.zeros(n, dtype=np.int32)
    s = ljmd.System(n, box, p, precision=prec)
    assert ljmd.cell_grid(s.params) == (cells, cells, cells if dim == 3 else 1)
    s.set_state(x, v, sp)
    check_lists(s, x, sp, box, p, prec)


@pytest.mark.parametrize("n,cells", [(17575, 13), (17576, 13), (117648, 49), (117649, 49)])
def test_fp64_lists_with_and_without_the_reduction(ljmd, n, cells):
    # Eight particles a cell are the line below which every candidate is tested
    # exactly (2,197 cells), and one a cell lies far below it (striding grid).
    edge = 2.8 * 1.001 * cells
    x, v = gas(n, edge, 3, n)
    p = W.single_species_params()
    box = (edge,) * 3
    sp = np.zeros(n, dtype=np.int32)
    s = ljmd.System(n, box, p, precision=FP64)
    s.set_state(x, v, sp)
    check_lists(s, x, sp, box, p, FP64)


@pytest.mark.parametrize("prec", [FP64, FP32_DS])
@pytest.mark.parametrize("cells,kw", [((55, 40, 61), {}), ((45, 45, 45), dict(lanes=4)), ((45, 45, 45), dict(lanes=16)),
                                      ((24, 24, 24), dict(cell_split=2)), ((21, 30, 24), dict(cell_split=2, lanes=1))])
def test_dilute_lists_of_other_layouts(ljmd, prec, cells, kw):
    # The striding grid in boxes that are not cubic, at other numbers of lanes,
    # and over half-size cells with the 125-cell stencil.
    n = 14000
    edges = 2.8 * 1.001 * np.array(cells)
    x, v = gas(n, edges.min(), 3, sum(cells))
    x *= edges / edges.min()  # stretched: the nearest pairs are no closer
    p = W.single_species_params()
    sp = np.zeros(n, dtype=np.int32)
    s = ljmd.System(n, edges, p, precision=prec, **kw)
    k = kw.get("cell_split", 1)
    grid = ljmd.cell_grid(s.params)
    assert all(k * c <= g <= k * (c + 1) for c, g in zip(cells, grid)) and np.prod(grid) > 12288
    s.set_state(x, v, sp)
    check_lists(s, x, sp, edges, p, prec)
    obs = s.run(15).cpu().numpy()
    s.sync()
    assert np.isfinite(obs).all()
