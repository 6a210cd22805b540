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


# ---- point selection: pivots of the sketched Gram matrices
def _greedy(Phi_c, K, seed, streams):
    """Pivots of the Gram matrix of the sketched pair products, and the residual of each."""
    from scipy.linalg import lapack
    from oracle import isdf
    p = isdf.sketch_size(min(K, len(Phi_c)), Phi_c.shape[1])
    A, B = (Phi_c @ isdf.orthonormal_sketch(Phi_c.shape[1], p, seed, s) for s in streams)
    L, piv, _, _ = lapack.dpstrf((A @ A.T) * (B @ B.T), lower=1, tol=0.0)
    return piv[:K] - 1, np.diag(L)[:K] ** 2


def _checked(got, want, resid):
    """Equal pivots while the residual stands well above rounding: an element of the updated
    diagonal carries about k eps of the first pivot (1e-13 of it), so two candidates can
    only change places when they are within 1e-7 of each other there."""
    k = int(np.argmax(resid < 1e-6 * resid[0])) if (resid < 1e-6 * resid[0]).any() else len(resid)
    assert k > 8 and np.array_equal(got[:k], want[:k])
    return k


@pytest.mark.parametrize("mesh,naux", [
    ((8, 8, 8), 31),          # one panel of pivots, less than a panel wide
    ((16, 8, 8), 33),         # 1024 candidates: the largest set of the one-workgroup panel
    ((5, 5, 41), 64),         # 1025 candidates: one launch per pivot
    ((13, 12, 11), 65),
])
def test_global_selection_pivots(lib, mesh, naux):
    w = dataclasses.replace(ri.tiny_cell(), mesh=np.asarray(mesh), naux=naux)
    _say(f"case: global selection, {w.ngrid} candidates, {naux} pivots")
    want, resid = _greedy(basis.eval_basis(w), naux, w.sketch_seed(), (0, 1))
    with lib.Context.from_workload(w, seed=w.sketch_seed(), select=lib.SELECT_GLOBAL) as ctx:
        got = ctx.points()
    _say(f"  {_checked(got, want, resid)} of {naux} pivots compared")


@pytest.mark.parametrize("w", [
    dataclasses.replace(ri.tiny_cell(), mesh=np.array([12, 11, 10])),            # 2 sets of about 660
    ri.diamond_supercell((1, 1, 1), (16, 15, 14), 2, c=3.0, cid=71),             # 8 sets of about 420
    ri.diamond_supercell((2, 1, 1), (24, 13, 13), 2, c=5.2, cid=72),             # a union of more than 1024
], ids=["2-atoms", "8-atoms", "16-atoms"])
def test_voronoi_selection_pivots(lib, w):
    """The sets of all atoms at once without their Gram matrices, then their union."""
    seed, Phi = w.sketch_seed(), basis.eval_basis(w)
    owner, Rh = basis.voronoi(w), []
    for I, NI in enumerate(w.funcs_per_atom()):
        kap = np.flatnonzero(owner == I)
        piv, resid = _greedy(Phi[kap], min(len(kap), int(np.ceil(w.naux / w.nbas * NI - 1e-9)) + 10), seed,
                             (2 + 2 * I, 3 + 2 * I))
        assert (resid > 1e-12 * resid[0]).all()       # the reference itself is well above rounding
        Rh.append(kap[piv])
    Rh = np.concatenate(Rh)
    _say(f"case: Voronoi selection, {w.natom} atoms, {len(Rh)} candidates, {w.naux} points")
    want, resid = _greedy(Phi[Rh], w.naux, seed, (0, 1))
    with lib.Context.from_workload(w, seed=seed) as ctx:
        got = ctx.points()
        assert ctx.info()["n_candidates"] == len(Rh)
    _say(f"  {_checked(got, Rh[want], resid)} of {w.naux} points compared")


# ---- full exchange matrix: A in chunks of interpolation points, workspace kept between calls
def test_full_exchange_chunks_and_workspace(lib):
    """K_full C = K_occ (both FP64, so within rounding of sums of N_g and N_aux terms) on a
    cell whose A takes two chunks (256 and 160 points), for several n in turn on one context
    (the kept workspace grows and is reused), and for the FP32 context's stored V."""
    w = ri.diamond_cell(4.0)
    with lib.Context.from_workload(w, seed=w.sketch_seed()) as ctx:
        S, pts = ctx.overlap(), ctx.points()
        for nocc in (3, 16, 33, 16):
            C = ri.lowdin(np.random.default_rng(nocc).standard_normal((w.nbas, nocc)), S)
            _say(f"case: full exchange, config 2 c=4, n={nocc}")
            Kf, (K, _) = ctx.build_full(C), ctx.build(C)
            assert np.array_equal(Kf, ctx.build_full(C))
            assert np.abs(Kf - Kf.T).max() < 1e-11 * np.abs(Kf).max()
            assert np.abs(Kf @ C - K).max() < 1e-10 * np.abs(K).max()
    with lib.Context.from_workload(w, points=pts, precision=lib.PREC_FP32) as ctx:
        _say("case: full exchange, FP32 context")
        K32 = ctx.build_full(C)
    assert np.abs(K32 - Kf).max() < 1e-6 * np.abs(Kf).max()     # V rounded to 24 bits


# ---- streaming passes: the M1 pass's last round of workgroups cut along the points
@pytest.mark.parametrize("prec,nocc", [("fp32", 16), ("bf16x3", 16), ("fp32", 33), ("fp64", 20), ("fp64", 65)])
def test_streaming_pass_tail(lib, prec, nocc, monkeypatch):
    """48^3 grid (864 blocks of 128 rows): at the FP32 and split-BF16 forms' residency the last
    round is partly empty, so its blocks run in pieces beside whole ones.  Against the FP64
    fused kernels (n <= 64) or the GEMM form, which share nothing with the passes; the bars are
    those of the precision forms (1e-6 Ha, 1e-6 of max|K|) and 1e-11 for FP64."""
    w = ri.diamond_cell(4.0)
    with lib.Context.from_workload(w, seed=w.sketch_seed()) as ctx:
        pts = ctx.points()
        C = ri.lowdin(np.random.default_rng(nocc).standard_normal((w.nbas, nocc)), ctx.overlap())
        if nocc > 64:
            monkeypatch.setenv("RPS_GENERAL_GEMM", "1")
        Kref, Eref = ctx.build(C)
    monkeypatch.delenv("RPS_GENERAL_GEMM", raising=False)
    monkeypatch.setenv("RPS_BUILD_PATH", "general")
    p = {"fp64": lib.PREC_FP64, "fp32": lib.PREC_FP32, "bf16x3": lib.PREC_BF16X3}[prec]
    with lib.Context.from_workload(w, points=pts, precision=p) as ctx:
        K, E = ctx.build(C)
        K2, E2 = ctx.build(C)
    dk = np.abs(K - Kref).max() / np.abs(Kref).max()
    _say(f"case: streaming pass tail {prec} n={nocc} dE={E - Eref:.2e} dK={dk:.2e}")
    assert np.array_equal(K, K2) and E == E2
    if prec == "fp64":
        assert dk < 1e-11 and abs(E - Eref) < 1e-11 * abs(Eref)
    else:
        assert dk < 1e-6 and abs(E - Eref) < 1e-6


# ---- FP32 products of the GEMM form: 96- and 64-wide tiles, splits of K joined or cut
@pytest.mark.parametrize("nocc", [65, 81, 96, 97, 150, 160, 176, 193, 200])
def test_gemm_form_tiles(lib, nocc, monkeypatch):
    """n around the edges of the 64- and 96-wide tiles (padded n 80, 96, 112, 160, 176, 208),
    several chunks with a ragged last one; against the FP64 form, with the bars of the
    precision forms (1e-6 Ha, 1e-6 of max|K|)."""
    monkeypatch.setenv("RPS_GENERAL_GEMM", "1")
    monkeypatch.setenv("RPS_GEMM_RCHUNK", "2048")
    w = ri.diamond_supercell((2, 1, 1), (36, 17, 18), 2, c=4.0, cid=73)
    rng = np.random.default_rng(nocc)
    with lib.Context.from_workload(w, seed=w.sketch_seed()) as ctx:
        pts = ctx.points()
        C = ri.lowdin(rng.standard_normal((w.nbas, nocc)), ctx.overlap()) * (16 / nocc) ** 0.5
        Kref, Eref = ctx.build(C)
    with lib.Context.from_workload(w, points=pts, precision=lib.PREC_FP32) as ctx:
        K, E = ctx.build(C)
        K2, E2 = ctx.build(C)
    dk = np.abs(K - Kref).max() / np.abs(Kref).max()
    _say(f"case: GEMM form n={nocc} dE={E - Eref:.2e} dK={dk:.2e}")
    assert np.array_equal(K, K2) and E == E2
    assert dk < 1e-6 and abs(E - Eref) < 1e-6


# ---- screened basis: atom blocks padded to multiples of 8, products in pieces along the grid
@pytest.mark.parametrize("w,nocc,eps", [
    (ri.diamond_supercell((1, 1, 1), (24, 24, 23), 2, c=4.0, cid=74), 17, 1e-2),      # |kappa| about 1650, ragged
    (ri.diamond_supercell((2, 1, 1), (33, 16, 15), 2, c=4.0, cid=75), 65, 1e-3),
    (ri.tiny_cell(), 3, 3e-2),                                                        # pieces of K1 and J
    (_s_cell(9, (6, 7, 5), nocc=2, lmax=2), 2, 3e-1),                                 # blocks of few functions
], ids=["8-atoms", "16-atoms", "2-atoms", "9-atoms"])
def test_screened_blocks(lib, w, nocc, eps, monkeypatch):
    """K and J from the atom blocks against the screened values in dense form (FP64 both,
    other summation orders: 1e-11), through the general path."""
    monkeypatch.setenv("RPS_BUILD_PATH", "general")
    monkeypatch.setenv("RPS_COULOMB_GEMM", "1")
    C = np.linalg.qr(np.random.default_rng(5).standard_normal((w.nbas, nocc)))[0].copy()
    pts = np.linspace(0, w.ngrid - 1, 6).astype(np.int64)
    out = []
    for blocks in ("1", "0"):
        monkeypatch.setenv("RPS_SCREENED_BLOCKS", blocks)
        kw = dict(seed=w.sketch_seed()) if w.naux > 10 else dict(points=pts[:w.naux])
        with lib.Context.from_workload(w, basis_eps=eps, **kw) as ctx:
            out.append((*ctx.build(C), *ctx.build_coulomb(C), ctx.info()["basis_fill"]))
    (K, E, J, EJ, fill), (K0, E0, J0, EJ0, _) = out
    _say(f"case: screened blocks N={w.nbas} n={nocc} fill={fill:.3f}")
    assert 0.0 < fill < 1.0
    assert np.abs(K - K0).max() < 1e-11 * np.abs(K0).max() and abs(E - E0) < 1e-11 * abs(E0)
    assert np.abs(J - J0).max() < 1e-11 * np.abs(J0).max() and abs(EJ - EJ0) < 1e-11 * abs(EJ0)


# ---- Coulomb matrix of small bases: lower tiles shared by a pair of waves, groups of four rows
@pytest.mark.parametrize("nfunc,mesh", [
    (1, (4, 4, 4)), (16, (4, 5, 13)), (17, (9, 8, 7)), (33, (8, 8, 9)), (49, (12, 11, 10)), (65, (16, 16, 17)),
    (81, (15, 16, 10)), (97, (20, 18, 16)), (112, (24, 24, 24)), (113, (9, 10, 8)), (128, (32, 30, 31)),
])
def test_coulomb_small_basis(lib, nfunc, mesh):
    """One case per padded N up to 128 with grids from one 64-row block to several groups per
    pair of waves (and lengths that do and do not take the plane transform)."""
    w = _s_cell(nfunc, mesh, nocc=min(3, nfunc), cid=91)
    _say(f"case: small Coulomb N={w.nbas} mesh={mesh}")
    Phi = basis.eval_basis(w)
    C = _coefficients(w)
    Jref, Eref, _ = coulomb.build_j(Phi, C, w.lattice, w.mesh)
    pts = np.linspace(0, w.ngrid - 1, w.naux).astype(np.int64)
    with lib.Context.from_workload(w, points=pts) as ctx:
        J, E = ctx.build_coulomb(C)
        J2, E2 = ctx.build_coulomb(C)
    assert np.abs(J - Jref).max() < 1e-11 * np.abs(Jref).max()
    assert abs(E - Eref) < 1e-11 * abs(Eref)
    assert np.array_equal(J, J2) and E == E2


# ---- FP64 exchange with n <= 16: orbitals formed in the V-streaming kernel, fit-fit line folded in
@pytest.mark.parametrize("w,nocc,shape", [
    (_s_cell(1, (4, 4, 4), 1), 1, None),                                  # one tile of everything
    (dataclasses.replace(_s_cell(17, (5, 7, 9), 3), naux=40), 3, None),   # ragged last grid tile
    (dataclasses.replace(_s_cell(64, (9, 8, 8), 16), naux=128), 16, None),
    (dataclasses.replace(_s_cell(128, (16, 15, 12), 15), naux=160), 15, None),
    (ri.diamond_supercell((1, 1, 1), (16, 17, 18), 2, naux=192), 16, None),      # 1.5 g subtiles per wave
    (ri.diamond_supercell((1, 1, 1), (16, 17, 18), 2, naux=448), 9, "3,1"),      # 4, odd number of R tiles
    (ri.diamond_supercell((1, 1, 1), (16, 17, 18), 2, naux=640), 16, "2,1"),     # 5
    (ri.diamond_supercell((1, 1, 1), (16, 17, 18), 2, naux=704), 16, None),      # two uneven g blocks
    (ri.diamond_supercell((1, 1, 1), (16, 17, 18), 2, naux=320), 13, "2,4"),     # the last g block empty
    (ri.diamond_supercell((1, 1, 1), (28, 35, 32), 2, naux=704), 11, "1,2"),    # line 3 in its own kernel (scratch)
])
def test_fused_fp64_orbitals_in_kernel(lib, w, nocc, shape, monkeypatch):
    """All three variants and the no-allocation build against the 4x4x4-instruction kernels,
    which read U from memory and form the fit-fit line by themselves (same points, same V)."""
    import torch
    if shape:
        monkeypatch.setenv("RPS_FUSED_SHAPE", shape)
    w = dataclasses.replace(w, nocc=nocc)
    C = _coefficients(w, seed=nocc)
    variants = (lib.VARIANT_RPS, lib.VARIANT_PS, lib.VARIANT_THC)
    with lib.Context.from_workload(w, seed=w.sketch_seed()) as ctx:
        pts = ctx.points()
        got = [ctx.build(C, variant=v) for v in variants]
        again = ctx.build(C)
        Cd = torch.from_numpy(C).cuda()
        Kd = torch.empty_like(Cd)
        ed = torch.zeros(1, dtype=torch.float64, device="cuda")
        ctx.build_noalloc(Cd, Kd, ed)
        torch.cuda.synchronize()
        assert np.array_equal(Kd.cpu().numpy(), got[0][0]) and float(ed[0]) == got[0][1]
    monkeypatch.setenv("RPS_FP64_MFMA", "m4")
    with lib.Context.from_workload(w, points=pts) as ctx:
        ref = [ctx.build(C, variant=v) for v in variants]
    assert np.array_equal(again[0], got[0][0]) and again[1] == got[0][1]
    for (K, E), (Kr, Er), v in zip(got, ref, variants):
        dk = np.abs(K - Kr).max() / np.abs(Kr).max()
        _say(f"case: FP64 fused N={w.nbas} n={nocc} N_aux={w.naux} variant {v} dE={E - Er:.2e} dK={dk:.2e}")
        assert dk < 1e-11 and abs(E - Er) < 1e-11 * abs(Er)


# ---- set-up: Cholesky panels and triangular solves in 64-row blocks, 512-row outer blocks
@pytest.mark.parametrize("naux", [1, 16, 63, 64, 65, 200, 520])
def test_setup_solve_blocks(lib, naux):
    """V and W against the oracle's LAPACK solve on a ragged grid, with the bar of the set-up's
    parity tests: both solves carry the metric's condition number times eps, up to 1e-8."""
    from oracle import isdf
    w = ri.diamond_supercell((1, 1, 1), (11, 13, 14), 2, naux=naux)
    with lib.Context.from_workload(w, seed=w.sketch_seed()) as ctx:
        pts = ctx.points()
        V, W = ctx.array(1), ctx.array(2)
    st = isdf.setup(w, basis.eval_basis(w), points=pts)
    _say(f"case: set-up solve N_aux={naux} dV={np.abs(V - st['V']).max() / np.abs(st['V']).max():.2e}")
    assert np.abs(V - st["V"]).max() < 1e-8 * np.abs(st["V"]).max()
    assert np.abs(W - st["W"]).max() < 1e-8 * np.abs(st["W"]).max()
