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
