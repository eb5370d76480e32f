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


def clusters(edge, spacings, outside, seed):
    """Cubic pieces of simple cubic lattices, one per spacing, at places of a
    3 x 3 x 3 grid, in a lattice of spacing `outside`."""
    rng = np.random.default_rng(seed)
    third = edge / 3.0
    places = np.stack(np.meshgrid(*[np.arange(3)] * 3, indexing="ij"), -1).reshape(-1, 3)
    side = 0.6 * third
    m = int(edge / outside)
    far = (np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3) + 0.5) * (edge / m)
    x = []
    for place, a in zip(places[rng.permutation(27)[: len(spacings)]], spacings):
        c = third * (place + 0.5)
        k = int(side / a)
        x.append(c + a * (np.stack(np.meshgrid(*[np.arange(k)] * 3, indexing="ij"), -1).reshape(-1, 3) - 0.5 * (k - 1)))
        far = far[np.abs(far - c).max(axis=1) > 0.5 * side + outside]
    x = np.concatenate(x + [far])
    return x + 0.02 * rng.standard_normal(x.shape)


@pytest.mark.parametrize("prec", [FP64, FP32_DS])
@pytest.mark.parametrize("edge,outside", [(45.0, 3.0), (118.0, 1.7), (118.0, 4.0)])
def test_growth_knows_the_longest_list(ljmd, edge, outside, prec):
    # Clusters of several densities: whichever list overflows first, the lists
    # grow once, by the longest of them all.
    x = clusters(edge, [1.3, 1.2, 1.1, 1.05, 1.0, 0.97, 0.95, 0.92], outside, 3)
    n, v, sp = len(x), np.zeros_like(x), np.zeros(len(x), dtype=np.int32)
    p = W.single_species_params()
    cap, room = 32, 512
    for seed in range(3):
        order = np.random.default_rng(seed).permutation(n)
        ref = ljmd.System(n, (edge,) * 3, p, precision=prec, nbr_capacity=256, cell_capacity=128)
        ref.set_state(x[order], v, sp)
        longest = ref.observables()["max_fill"]
        s = ljmd.System(n, (edge,) * 3, p, precision=prec, nbr_capacity=cap, nbr_capacity_max=room,
                        cell_capacity=128)
        s.set_state(x[order], v, sp)
        o = s.observables()
        print(f"clusters n={n} cells={ljmd.cell_grid(s.params)} prec={prec} longest={longest} "
              f"capacity={o['nbr_capacity']} builds={o['rebuilds']}", flush=True)
        assert o["rebuilds"] == 2
        assert 64 < longest <= 256
        assert o["nbr_capacity"] == -(-max(longest + 16, int(np.ceil(1.25 * longest))) // 16) * 16
        assert np.array_equal(s.forces().cpu().numpy(), ref.forces().cpu().numpy())
