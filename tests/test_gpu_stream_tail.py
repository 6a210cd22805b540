"""The streaming M1 pass's last round of workgroups, cut along the interpolation points."""
import sys

import numpy as np
import pytest

import rps_inputs as ri

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def lib():
    import paper_2207_04636_amd as P
    P.load()
    return P


@pytest.fixture(scope="module")
def cell(lib):
    """1088 row blocks of 128 points.  256 compute units hold 256, 512, 768 or 1024 workgroups of
    eight waves at once (one to four each), and 1088 leaves 64 or 320 blocks over: whatever the
    kernel's registers allow, a last round that is cut in two or more pieces."""
    w = ri.diamond_supercell((1, 1, 1), (64, 64, 34), 2, naux=576, cid=94)
    assert w.ngrid == 1088 * 128
    with lib.Context.from_workload(w, seed=w.sketch_seed()) as ctx:
        return w, ctx.points(), ctx.overlap()


@pytest.mark.parametrize("prec,nocc", [("fp32", 16), ("fp32", 33), ("fp32", 48), ("bf16x3", 16), ("bf16x3", 40),
                                       ("fp64", 20), ("fp64", 64)])
def test_streaming_pass_tail_runs(lib, cell, prec, nocc, monkeypatch, capfd):
    """The plan says that the tail is cut, and the build agrees with the FP64 fused kernels, which
    share nothing with the passes: 1e-6 Ha and 1e-6 of max|K| for the precision forms, 1e-11
    for FP64 (other summation orders only)."""
    w, pts, S = cell
    C = ri.lowdin(np.random.default_rng(nocc).standard_normal((w.nbas, nocc)), S)
    with lib.Context.from_workload(w, points=pts) as ctx:
        Kref, Eref = ctx.build(C)
    monkeypatch.setenv("RPS_BUILD_PATH", "general")
    monkeypatch.setenv("RPS_VERBOSE", "1")
    p = {"fp64": lib.PREC_FP64, "fp32": lib.PREC_FP32, "bf16x3": lib.PREC_BF16X3}[prec]
    with lib.Context.from_workload(w, points=pts, precision=p) as ctx:
        capfd.readouterr()
        K, E = ctx.build(C)
        K2, E2 = ctx.build(C)
        lines = [s for s in capfd.readouterr().err.splitlines() if "M1 pass" in s]
    dk = np.abs(K - Kref).max() / np.abs(Kref).max()
    _say(f"case: streaming pass tail {prec} n={nocc}: {lines} dE={E - Eref:.2e} dK={dk:.2e}")
    whole, pieces = int(lines[0].split()[4]), int(lines[0].split()[-2])
    assert len(lines) == 1 and 0 < whole < 1088 and pieces > 1
    assert np.array_equal(K, K2) and E == E2
    if prec == "fp64":
        assert dk < 1e-11 and abs(E - Eref) < 1e-11 * abs(Eref)
    else:
        assert dk < 1e-6 and abs(E - Eref) < 1e-6
