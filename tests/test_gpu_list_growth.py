"""List overflow and recovery in inhomogeneous boxes: a dense droplet whose
particles' lists exceed the capacity, in a box of many more cells than run at
once, so that some blocks of a list build end, and report the overflow, while
others start. The lists grow and the build is done again: everything equals,
bit for bit, a system that had the room from the start.
"""
import numpy as np
import pytest

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


def droplet(dim, edge, inside, spacing, outside):
    """inside sites a side at `spacing` in the middle of a box of the given
    edge, and the sites of a lattice of spacing `outside` around them."""
    side = inside * spacing
    lo = 0.5 * (edge - side)
    a = lo + spacing * (np.arange(inside) + 0.5)
    m = int(edge / outside)
    b = edge / m * (np.arange(m) + 0.5)
    x = [np.stack(np.meshgrid(*[c] * dim, indexing="ij"), -1).reshape(-1, dim) for c in (a, b)]
    far = np.abs(x[1] - 0.5 * edge).max(axis=1) > 0.5 * side + outside
    x = np.concatenate([x[0], x[1][far]])
    rng = np.random.default_rng(inside)
    x += 0.03 * rng.standard_normal(x.shape)
    v = rng.standard_normal(x.shape)
    z = np.zeros((len(x), 3 - dim))
    return np.concatenate([x, z], 1), np.concatenate([v, z], 1)


# Two dimensions: 38 x 38 cells; three: 21 x 21 x 21.
BOXES = {"2d": (2, 107.8, 55, 1.05, 2.4, 16), "3d": (3, 60.0, 20, 1.1, 3.6, 48)}


@pytest.mark.parametrize("prec", [FP64, FP32_DS])
@pytest.mark.parametrize("box", sorted(BOXES))
def test_droplet_overflow_is_recovered(ljmd, box, prec):
    dim, edge, inside, spacing, outside, cap = BOXES[box]
    x, v = droplet(dim, edge, inside, spacing, outside)
    n = len(x)
    p = W.single_species_params()
    p.dim = dim
    edges = (edge, edge, edge if dim == 3 else 10.0)
    out = []
    for c, room in ((4 * cap, 0), (cap, 4 * cap)):
        s = ljmd.System(n, edges, p, precision=prec, nbr_capacity=c, nbr_capacity_max=room, sort_interval=7,
                        cell_capacity=64)
        print(f"droplet {box} prec={prec} n={n} cells={ljmd.cell_grid(s.params)} capacity={c}", flush=True)
        s.set_state(x, v, np.zeros(n, dtype=np.int32))
        f = s.forces().cpu().numpy()
        obs = s.run(20).cpu().numpy()
        o = s.observables()
        assert o["max_fill"] > cap
        out.append((f, obs, s.unwrapped_positions().cpu().numpy()))
    assert o["nbr_capacity"] > cap
    assert np.isfinite(out[0][1]).all()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
