"""Host atoms as prism_atom records (no GPU): the same values, and the same
refusals, as one ctypes assignment per atom."""
import ctypes

import numpy as np
import pytest


def _one_by_one(pos, idx):
    from paper_1706_08563_amd._lib import prism_atom
    pos = np.ascontiguousarray(pos, dtype=np.float64)
    out = []
    for i in range(len(pos)):
        a = prism_atom()
        a.x, a.y, a.z = (float(np.squeeze(pos[i, k])) for k in range(3))
        a.species = int(idx[i])
        out.append((a.x, a.y, a.z, a.species))
    return out


POS = np.arange(15.0).reshape(5, 3) * 0.37


@pytest.mark.parametrize("pos,idx", [
    (POS, [0, 1, 2, 1, 0]), (POS.tolist(), (1, 0, 1, 0, 1)), (POS, np.array([3, 1, 2, 1, 0, 9], dtype=np.uint8)),
    (np.c_[POS, POS], np.array([0, 1, 0, 1, 0], dtype=np.int64)), (POS.reshape(5, 3, 1), [0] * 5),
    (POS.astype(np.float32), np.array([0.0, 1.9, 2.0, 0.0, 1.0])), (POS, np.array([[1], [0], [1], [0], [1]])),
    (POS, [2 ** 40 + 1, -1, 2 ** 70, True, 0]), (POS, np.array([2 ** 40 + 1, -1, 5, 0, 2 ** 32], dtype=np.int64)),
    (POS[::-1], {0: 1, 1: 0, 2: 2, 3: 0, 4: 1}), (np.asfortranarray(POS), [1] * 5), (np.zeros((0, 3)), [])])
@pytest.mark.filterwarnings("ignore::DeprecationWarning")
def test_records_equal_single_assignments(pos, idx):
    from paper_1706_08563_amd import api
    from paper_1706_08563_amd._lib import prism_atom
    rec, n = api._atom_records(pos, idx)
    atoms = rec.ctypes.data_as(ctypes.POINTER(prism_atom))
    assert n == len(pos) and rec.flags.c_contiguous and rec.itemsize * 4 == ctypes.sizeof(prism_atom)
    assert [(atoms[i].x, atoms[i].y, atoms[i].z, atoms[i].species) for i in range(n)] == _one_by_one(pos, idx)


@pytest.mark.parametrize("pos,idx", [(POS[:, :1], [0] * 5), (POS[:, :2], [0] * 5), (POS[:, :0], [0] * 5), (POS[:, 0], [0] * 5),
                                     (POS, [0, 1]), (POS, np.array([0, 1]))])
def test_missing_coordinates_and_species_are_refused(pos, idx):
    """A single column of positions is not taken for x = y = z."""
    import paper_1706_08563_amd as P
    grid = P.prism_grid_init((25.0, 25.0, 4.0), 2.0, 64)
    with pytest.raises(IndexError):
        P.prism_project_potential(pos, idx, [], grid, device="cpu")
