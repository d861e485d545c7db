"""The one-pass read of the Miller list (largest |m| per axis for the grid rule)
gives the rule of the oracle for lists of every length modulo its block size,
with the largest index anywhere in the list (CPU: fock_exchange_grid reads no
device)."""
import numpy as np
import pytest

from oracle import exx
from paper_1305_7313_amd import fock as F

SIZES = (24, 48, 64, 72, 96, 128)
PLANES = {(24, 24), (48, 48), (48, 64), (64, 64), (72, 72), (96, 96), (96, 128)}


@pytest.mark.parametrize("npw", [1, 2, 7, 8, 9, 16, 335, 336, 337, 345, 1009])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_largest_index_anywhere(npw, axis):
    rng = np.random.default_rng(npw)
    a = np.diag([10.0, 11.0, 12.0])
    for where in {0, npw // 2, npw - 1}:
        for top in (11, -15):
            m = rng.integers(-3, 4, (npw, 3)).astype(np.int32)
            m[where, axis] = top
            need = [4 * int(np.abs(m[:, k]).max()) + 1 for k in range(3)]
            assert need == list(exx.exchange_grid_need(a, m, 0.0))
            got = F.fock_exchange_grid(F.Cell(a, (24, 24, 24), m))
            grids = [(x, y, z) for x in SIZES for y, z in PLANES if x >= need[0] and y >= need[1] and z >= need[2]]
            assert np.prod(got) == min(np.prod(g) for g in grids)
            assert all(g >= n for g, n in zip(got, need))
