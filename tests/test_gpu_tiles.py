"""Edges of the kernels' tiles: sizes at which a tile, a split or a remainder starts or
ends, each against the FP64 oracle (or a plain numpy product) on small cells.

Tolerances: FP64 results differ from the oracle only in summation order.  A sum of K
products carries at most K eps relative to the sum of their magnitudes; with K up to a
few thousand grid points and magnitudes within 100 of the result that stays under 1e-10,
and random rounding keeps it far below, so the bar of the Coulomb tests (1e-11) is used."""
import dataclasses
import sys

import numpy as np
import pytest

import rps_inputs as ri
from oracle import basis, coulomb, grid

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def lib():
    import paper_2207_04636_amd as P
    P.load()
    return P


def _s_cell(nfunc, mesh, nocc, lmax=0, cid=90):
    """nfunc shells of s (up to l = lmax) functions at random places of a 4-bohr cell."""
    w = ri.tiny_s_cell(nfunc=nfunc, mesh=8, L=4.0, nocc=nocc, naux=4, cid=cid, lmax=lmax)
    return dataclasses.replace(w, mesh=np.asarray(mesh))


def _coefficients(w, seed=0):
    rng = np.random.default_rng(seed)
    return np.ascontiguousarray(np.linalg.qr(rng.standard_normal((w.nbas, w.nocc)))[0])


# ---- Coulomb matrix by the GEMM path: lower output tiles of 128 x 64, K split over the grid
@pytest.mark.parametrize("nfunc,mesh", [
    (17, (8, 8, 8)),          # one narrow tile (padded N = 32)
    (64, (5, 7, 9)),          # exactly one 64-wide tile, ragged grid (315 points)
    (65, (9, 8, 8)),          # a second column tile
    (128, (10, 9, 8)),        # a full row panel
    (129, (8, 8, 10)),        # a second row panel
    (200, (16, 15, 12)),      # ragged tiles, several K splits
])
def test_coulomb_lower_tiles(lib, nfunc, mesh, monkeypatch):
    monkeypatch.setenv("RPS_COULOMB_GEMM", "1")
    w = _s_cell(nfunc, mesh, nocc=min(5, nfunc))
    _say(f"case: Coulomb tiles N={w.nbas} mesh={mesh}")
    Phi = basis.eval_basis(w)
    C = _coefficients(w)
    Jref, Eref, _ = coulomb.build_j(Phi, C, w.lattice, w.mesh)
    pts = np.linspace(0, w.ngrid - 1, w.naux).astype(np.int64)
    with lib.Context.from_workload(w, points=pts) as ctx:
        J, E = ctx.build_coulomb(C)
    assert np.abs(J - Jref).max() < 1e-11 * np.abs(Jref).max()
    assert abs(E - Eref) < 1e-11 * abs(Eref)
    assert np.array_equal(J, J.T)
