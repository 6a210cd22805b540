"""Sizes of device workspaces that the library decides on the host, by its own functions."""
import ctypes as ct

import pytest

import paper_2207_04636_amd as P


def _fn(name, *args):
    f = getattr(P.load(), name)
    f.restype, f.argtypes = ct.c_int64, [ct.c_int64] * len(args)
    return f(*args)


@pytest.mark.parametrize("R", [64, 24 ** 3, 48 ** 3, 80 * 40 * 40, 108 ** 3, 1953088, 1953152, 160 ** 3, 256 ** 3])
def test_full_exchange_chunk(R):
    """A chunk of A (rows x R doubles) takes 256 MB or less, or one 128-row tile up to 2 GB, or
    64 rows: never more than the larger of 2 GB and 64 rows."""
    rows = _fn("_ZN3rps15full_chunk_rowsEl", R)
    assert rows >= 64 and rows % 64 == 0
    assert rows * R * 8 <= max(2_000_000_000, 64 * R * 8)
    assert rows <= 128 or (rows % 128 == 0 and rows * R * 8 <= 256 << 20)


@pytest.mark.parametrize("K,tiles,outputs", [
    (8000, 320, 32 * 416 ** 2),         # 32 atoms: several pieces
    (700, 20, 8 * 104 ** 2), (200, 3, 100), (0, 0, 0), (6500, 3520, 64 * 832 ** 2),
    (100_000, 768 * 5 + 40, 59_000_000),     # without a cap: several pieces of 472 MB each
])
def test_atom_block_pieces_fit_the_workspace(K, tiles, outputs):
    """Partials of the atom blocks' products: one copy, or as many as fit the 512 MB that the
    other split products keep to."""
    cap = 64 << 20
    z = _fn("_ZN3rps13sparse_piecesEllll", K, tiles, outputs, cap)
    assert z >= 1 and (z == 1 or (z * outputs <= cap and K // z >= 256))
    if (K, tiles) == (8000, 320):
        assert z > 1
    if K == 100_000:
        assert z == 1 and _fn("_ZN3rps13sparse_piecesEllll", K, tiles, outputs, 1 << 40) > 1
