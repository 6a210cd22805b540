"""Device memory that outlives a call of the full exchange matrix: one pool for all contexts,
at most 1 GB per device, given back with the last context."""
import sys
import threading
import time

import numpy as np
import pytest

import rps_inputs as ri

pytestmark = pytest.mark.gpu

MB = 1 << 20


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def lib():
    import paper_2207_04636_amd as P
    P.load()
    return P


def test_full_exchange_memory_is_shared_and_bounded(lib):
    """Five contexts with about 300 MB of workspace each, in turn and then in threads of their
    own: equal results, and never more than 1 GB (and the runtime's own few MB) held between
    calls; nothing once the contexts are gone."""
    import torch
    w = ri.diamond_cell(4.0)
    C = np.linalg.qr(np.random.default_rng(3).standard_normal((w.nbas, 16)))[0].copy()

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    with lib.Context.from_workload(w, seed=w.sketch_seed()) as ctx:
        pts = ctx.points()
        ctx.build_full(C)
    start = free()      # the library's code and constants are loaded
    ctxs = [lib.Context.from_workload(w, points=pts) for _ in range(5)]
    try:
        before = free()
        K = [c.build_full(C) for c in ctxs]
        _say(f"case: five contexts in turn, {(before - free()) / MB:.0f} MB held")
        assert before - free() <= 1100 * MB
        assert all(np.array_equal(K[0], k) for k in K[1:])
        out = [None] * 5

        def work(i):
            torch.cuda.set_device(0)
            out[i] = [ctxs[i].build_full(C) for _ in range(3)]

        threads = [threading.Thread(target=work, args=(i,)) for i in range(5)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert all(np.array_equal(K[0], k) for o in out for k in o)
        _say(f"  in threads, {(before - free()) / MB:.0f} MB held")
        assert before - free() <= 1100 * MB
    finally:
        for c in ctxs:
            c.close()
    _say(f"  contexts gone, {(start - free()) / MB:.0f} MB held")
    assert start - free() <= 100 * MB


def test_full_exchange_of_a_large_grid(lib):
    """More than 1.9 million points: A in chunks of 64 rows (a half-empty output tile), three
    of them.  K_full C = K_occ within the rounding of FP64 sums over grid and points."""
    import dataclasses
    w = ri.tiny_s_cell(nfunc=9, mesh=8, L=4.0, nocc=3, naux=130, cid=92, lmax=1)
    w = dataclasses.replace(w, mesh=np.array([125, 125, 126]))
    rng = np.random.default_rng(7)
    C = np.linalg.qr(rng.standard_normal((w.nbas, 3)))[0].copy()
    pts = np.sort(rng.choice(w.ngrid, w.naux, replace=False)).astype(np.int64)
    q = 1.0 + rng.random((w.naux, 1))
    V = (q * np.cos(1e-5 * np.arange(w.ngrid))[None, :]).copy()
    W = 1.0 + rng.random((w.naux, w.naux))
    W = 0.5 * (W + W.T)
    with lib.Context.from_potentials(w, pts, V, W) as ctx:
        Kf, (K, _) = ctx.build_full(C), ctx.build(C)
    _say(f"case: full exchange, {w.ngrid} points, |K_full C - K| {np.abs(Kf @ C - K).max() / np.abs(K).max():.1e}")
    assert np.abs(Kf @ C - K).max() < 1e-10 * np.abs(K).max()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_no_orbitals_held_where_the_kernel_forms_them(lib, prec):
    """n <= 16, N <= 128: U stays in the kernel, so a build's workspace on a large grid with few
    points is below the size that U alone would have."""
    import dataclasses
    w = ri.tiny_s_cell(nfunc=9, mesh=8, L=4.0, nocc=3, naux=4, cid=93, lmax=1)
    w = dataclasses.replace(w, mesh=np.array([64, 64, 64]))
    C = np.linalg.qr(np.random.default_rng(8).standard_normal((w.nbas, 3)))[0].copy()
    pts = np.array([5, 70001, 140003, 210007])
    with lib.Context.from_workload(w, points=pts, precision=lib.PREC_FP64 if prec == "fp64" else lib.PREC_FP32) as ctx:
        before = ctx.info()["device_bytes"]
        K, E = ctx.build(C)
        for v in (lib.VARIANT_PS, lib.VARIANT_THC):
            ctx.build(C, variant=v)
        grown = ctx.info()["device_bytes"] - before
    _say(f"case: workspace of a build, {prec}: {grown / MB:.1f} MB, U would be {w.ngrid * 16 * 8 / MB:.1f} MB")
    assert grown < w.ngrid * 16 * 8
    assert np.isfinite(K).all() and np.isfinite(E)


def test_build_after_a_failed_allocation(lib, monkeypatch):
    """A build whose workspace does not fit returns an error and leaves no half of it behind: the
    builds after it, of the size that was there before and of the refused one once there is
    room, are those of a context of their own.  Idle workspace of the full exchange matrix is
    given back before the library reports that there is no memory."""
    import torch
    monkeypatch.setenv("RPS_BUILD_PATH", "general")
    w = ri.diamond_cell(4.0)
    rng = np.random.default_rng(9)

    def take_all_but_64_mb():
        hold, still = [], 0
        for _ in range(40):        # memory freed before comes back a moment later: until none does
            torch.cuda.empty_cache()
            free = torch.cuda.mem_get_info()[0]
            still = still + 1 if free <= 80 * MB else 0
            if still == 6:
                break
            if free > 80 * MB:
                hold.append(torch.empty(free - 64 * MB, dtype=torch.uint8, device="cuda"))
            time.sleep(0.1)
        _say(f"  {torch.cuda.mem_get_info()[0] / MB:.0f} MB free")
        assert still == 6
        return hold

    C16, C96 = (np.linalg.qr(rng.standard_normal((w.nbas, n)))[0].copy() for n in (16, 96))
    with lib.Context.from_workload(w, seed=w.sketch_seed()) as ctx:
        pts = ctx.points()
        want = [ctx.build(C16), ctx.build(C96), ctx.build_coulomb(C16), ctx.build_coulomb(C96)]
        full = ctx.build_full(C16)
    with lib.Context.from_workload(w, points=pts) as ctx:
        ctx.build(C16)
        ctx.build_coulomb(C16)
        _say("case: build without room for its workspace")
        hold, refused = [], False
        for _ in range(2):        # (contexts of other tests may have left idle workspace: gone after the first try)
            hold += take_all_but_64_mb()        # a part of what n = 96 adds (about 230 MB)
            try:
                ctx.build(C96)
                ctx.build(C16)
            except lib.RpsError:
                refused = True
                break
        assert refused
        got = [ctx.build(C16)]
        del hold
        torch.cuda.empty_cache()
        got += [ctx.build(C96), ctx.build_coulomb(C16), ctx.build_coulomb(C96)]
        for (K, E), (Kw, Ew) in zip(got, [want[0], want[1], want[2], want[3]]):
            assert np.array_equal(K, Kw) and E == Ew
        # the pool's idle block makes room for a build
        assert np.array_equal(ctx.build_full(C16), full)
        ctx.build(C16)
        hold = take_all_but_64_mb()
        K, E = ctx.build(C96)
        assert np.array_equal(K, want[1][0]) and E == want[1][1]
        del hold
        torch.cuda.empty_cache()
