"""The projected potential over its cell lists and factor tables: cells as
small as a tile's reach and one cell for the whole grid, positions outside the
cell and on its edges, more listed atoms than one table holds, species of 1 to
4 Gaussians and of different reach, and an empty list, against the FP64 oracle.

Tolerance: a term is the product of two FP32 exponentials (2 x 2^-23 with
their arguments' rounding) and up to 200 of them are added (random roundings,
14 x 2^-24): 2e-6 of the largest value."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

SPECIES = (W.Species((20.0,), (0.3,)), W.Species((20.0, 5.0), (0.3, 0.8)),
           W.Species((9.0, 3.0, 2.0, -1.0), (0.2, 0.35, 0.5, 0.7)))


def _check(pos, idx, species, L, S, n):
    import paper_1706_08563_amd as P
    g = P.prism_grid_init((L, L, 2.0 * S), 2.0, n)
    V = P.prism_project_potential(pos, idx, species, g).cpu().numpy().astype(np.float64)
    if len(pos) == 0:
        assert not V.any()
        return
    ref = O.projected_potential(pos, idx, species, (L, L, 2.0 * S), 2.0, n)
    assert np.max(np.abs(V - ref)) <= 2e-6 * np.max(np.abs(ref))


@pytest.mark.parametrize("species", [SPECIES[:1], SPECIES[:2], SPECIES])
@pytest.mark.parametrize("n,L,S,atoms", [(64, 9.7, 2, 40),        # one cell, the reach wraps around it
                                         (128, 40.0, 3, 300),     # several cells
                                         (64, 40.0, 40, 400),     # few cells for the many slices
                                         (256, 60.0, 1, 2000),    # up to 9 cells per tile, many tables
                                         (64, 12.0, 2, 0)])
def test_potential_cells(species, n, L, S, atoms):
    rng = np.random.default_rng(atoms + n)
    pos = rng.uniform(-1.3, 2.3, size=(atoms, 3)) * np.array([L, L, 2.0 * S])
    idx = rng.integers(0, len(species), size=atoms).astype(np.int32)
    _check(pos, idx, species, L, S, n)


def test_potential_cell_edges_and_clusters():
    L, n = 30.0, 128
    edge = np.array([[0.0, 0.0, 0.0], [L, L, 2.0], [-1e-17, 5.0, 1.0], [np.nextafter(L, 0), 7.0, 4.0], [L / 2, L, 3.9]])
    rng = np.random.default_rng(3)
    heap = np.concatenate([rng.normal(0.0, 0.4, size=(150, 2)) + 14.9, rng.uniform(0, 4, size=(150, 1))], axis=1)
    pos = np.concatenate([edge, heap])
    for kind in (np.int32, np.int64, list):
        idx = np.arange(len(pos)) % 3
        _check(pos, idx.tolist() if kind is list else idx.astype(kind), SPECIES, L, 2, n)


def test_potential_repeats_bit_for_bit():
    import torch
    import paper_1706_08563_amd as P
    rng = np.random.default_rng(9)
    pos = rng.uniform(0.0, 1.0, size=(4000, 3)) * np.array([50.0, 50.0, 8.0])
    idx = np.zeros(4000, np.int32)
    g = P.prism_grid_init((50.0, 50.0, 8.0), 2.0, 256)
    a, b = (P.prism_project_potential(pos, idx, SPECIES[1:2], g) for _ in range(2))
    assert torch.equal(a, b)
