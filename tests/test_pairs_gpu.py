"""Two iterations per update (bf16, k at least 256 and N - k at least 2048, up to 2560 for k
from 683 to 1279 and k from 1280 to 2047): the k x k products of tm_fast.hip against the fp64 oracle at the edges of the
tiles and of the rule, for even and odd iteration counts, and equal bits from single, batched
and grouped calls that run different tiles."""
import importlib.util
import os

import numpy as np
import pytest

from oracle import turbomuon as O
from gpu_helpers import (BF16_TOL, EO_RATIO_TOL, SCHEDULE5, eo_ratio, from_device, log,
                         make_input, relF, to_device)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2512_04632_amd import _lib as tm  # noqa: E402


ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def one(X, iters, precond, coeffs=None):
    t = to_device(X, "bf16")
    tm.orthogonalize(t, iters, coeffs, precond)
    return t


# (k, N): the edges of the rule (256 x 2304, 640 x 2688, 768 x 3072 and 1280 x 2560 are in,
# 256 x 2303, 255 x 2400, 640 x 2687, 768 x 3071, 1279 x 2560 and 1281 x 2560 out), tile
# remainders on either side, ragged N
SHAPES = [(256, 2304), (257, 2304), (300, 2701), (512, 2048), (513, 2048), (513, 2100),
          (575, 2333), (577, 2900), (640, 3000), (1280, 2560), (1281, 2560),
          (255, 2400), (256, 2303), (300, 2348), (640, 2687), (640, 2688), (768, 3071), (768, 3072),
          (1279, 2560)]


@pytest.mark.parametrize("k,N", SHAPES)
@pytest.mark.parametrize("precond,iters,coeffs", [("aol", 4, None), ("aol", 2, None), ("aol", 3, None),
                                                  ("frobenius", 5, None), ("schatten4", 4, None),
                                                  ("aol", 5, SCHEDULE5)])
def test_pairs_match_oracle(k, N, precond, iters, coeffs):
    for tall in (False, True):
        m, n = (N, k) if tall else (k, N)
        log(f"case: pairs {m}x{n} {precond} t={iters} schedule={coeffs is not None}")
        X = make_input(m, n, 0.8, 17 * k + N, "bf16")
        G = from_device(one(X, iters, precond, coeffs))
        R = O.orthogonalize(X, iters, coeffs, precond)
        e = relF(G, R)
        log(f"relF={e:.3e}")
        assert e <= BF16_TOL
        if coeffs is None:   # the schedule's own polar error is near zero
            assert abs(eo_ratio(G, R) - 1) <= EO_RATIO_TOL


@pytest.mark.parametrize("k,N,iters,precond", [
    (k, N, t, p) for k, N in ((255, 2400), (256, 2303), (256, 2304), (640, 2687), (640, 2688), (768, 3071),
                              (768, 3072), (1000, 3560), (1279, 3838), (1279, 3839), (1280, 2559), (1280, 2560),
                              (1535, 4000), (1536, 3071), (1536, 3072), (1000, 5096))
    for t, p in ((2, "aol"), (3, "aol"), (4, "aol"), (5, "frobenius"), (8, "frobenius"), (4, "none"))])
def test_benchmark_counts_the_updates_that_run(k, N, iters, precond):
    """bench.py holds its own copy of the rule: the updates launched by one matrix (at most one
    full wave of tiles, so one launch each) are those that it counts."""
    log(f"case: updates of {k}x{N} t={iters} {precond}")
    spec = importlib.util.spec_from_file_location("tm_bench", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    t = (torch.randn((k, N), device="cuda") / (k ** 0.5 + N ** 0.5)).bfloat16()
    tm.timing_reset()
    tm.timing_enable(True)
    try:
        tm.orthogonalize(t, iters, None, precond)
        torch.cuda.synchronize()
    finally:
        tm.timing_enable(False)
    ran = tm.timing_read("update")[1]
    tm.timing_reset()
    assert ran == bench.run_flops(k, N, iters, "bf16", precond)["updates"]


def test_mixed_group_equals_single_calls_bitwise():
    """Pairs, step-by-step and fused-range matrices in one call: every launch covers other
    matrices, with other tiles, than the single calls'."""
    log("case: mixed group vs single calls, bitwise")
    shapes = [(768, 3072), (515, 515), (64, 576), (129, 1153), (1001, 777), (300, 375), (2048, 640),
              (1300, 2700), (2900, 640), (1300, 3400),
              (768, 3072), (40, 41)]
    Xs = [make_input(m, n, 0.8, i, "bf16") for i, (m, n) in enumerate(shapes)]
    for precond, iters, part in (("aol", 4, Xs), ("frobenius", 5, Xs), ("schatten4", 3, Xs),
                                 ("aol", 4, [Xs[0], Xs[2], Xs[11]])):   # pairs and fused only
        ts = [to_device(X, "bf16") for X in part]
        tm.orthogonalize_grouped(ts, iters, None, precond)
        for i, X in enumerate(part):
            assert torch.equal(ts[i], one(X, iters, precond)), (precond, X.shape)


@pytest.mark.parametrize("N", [2100, 2700])   # step by step, in pairs
@pytest.mark.parametrize("scale", [30.0, 1e3])
def test_large_coefficients_stay_finite(scale, N):
    """Coefficients whose k x k matrices could leave fp16's range take the bf16
    step-by-step form: linear steps (scale, 0, 0) multiply by scale each."""
    log(f"case: linear steps of {scale}")
    X = make_input(520, N, 0.8, 5, "bf16")
    co = [(scale, 0.0, 0.0)] * 4
    G = from_device(one(X, 4, "aol", co))
    R = O.orthogonalize(X, 4, co, "aol")
    assert np.isfinite(G).all() and relF(G, R) <= BF16_TOL


@pytest.mark.parametrize("N", [2048, 2600])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_non_finite_input_stays_visible(bad, N):
    """One NaN or infinity reaches every output, as in the step-by-step form (its row sum
    scales every row)."""
    log(f"case: {bad} in the input")
    X = make_input(512, N, 0.8, 6, "bf16")
    X[5, 7] = bad
    assert np.isnan(from_device(one(X, 4, "aol"))).all()


@pytest.mark.parametrize("N", [2200, 2700])
def test_zero_rows_and_zero_matrix(N):
    log("case: zero rows, zero matrix")
    X = make_input(530, N, 0.8, 7, "bf16")
    X[3] = 0.0
    X[529] = 0.0
    G = from_device(one(X, 4, "aol"))
    R = O.orthogonalize(X, 4, None, "aol")
    assert relF(G, R) <= BF16_TOL and not G[3].any() and not G[529].any()
    assert not from_device(one(0.0 * X, 4, "frobenius")).any()


@pytest.mark.parametrize("precond", ["aol", "frobenius", "schatten4"])
@pytest.mark.parametrize("tall", [False, True])
def test_small_rows_keep_their_directions(precond, tall):
    """Rows at 1e-9 of the others (their entries of A are below fp16's normal numbers): each comes
    out within the tolerance of the whole matrix, by itself."""
    log(f"case: rows at 1e-9, {precond} tall={tall}")
    X = make_input(520, 2700, 0.8, 8, "bf16")
    small = [0, 77, 300, 519]
    X[small] *= 2.0 ** -30
    G = from_device(one(X.T if tall else X, 4, precond))
    G = G.T if tall else G
    R = O.orthogonalize(X, 4, None, precond)
    assert relF(G, R) <= BF16_TOL
    for i in small:
        assert np.linalg.norm(G[i] - R[i]) <= BF16_TOL * np.linalg.norm(R[i]), i


def test_failed_allocation_leaves_a_mixed_group_untouched(monkeypatch):
    """Pairs beside matrices of the fused range, which need no workspace: still nothing is
    enqueued when the pairs' workspace cannot be had."""
    log("case: forced workspace allocation failure, 768 x 3072 and 64 x 576")
    Xs = [make_input(768, 3072, 0.8, 1, "bf16"), make_input(64, 576, 0.8, 2, "bf16")]
    ts = [to_device(X, "bf16") for X in Xs]
    keep = [t.clone() for t in ts]
    torch.cuda.synchronize()
    tm.release_workspaces()
    monkeypatch.setenv("TM_TEST_FAIL_ALLOC", "1")
    with pytest.raises(tm.TurboMuonError):
        tm.orthogonalize_grouped(ts, 4, None, "aol")
    torch.cuda.synchronize()
    assert all(torch.equal(t, k) for t, k in zip(ts, keep))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shapes", [
    [(70, 100), (100, 1500), (300, 310)],                        # fewer tiles than XCDs in an entry
    [(200, 260)] * 9 + [(1000, 600)] + [(130, 2000)] * 3,        # the longest products last
    [(300, 500)] * 20 + [(500, 1999)] * 5 + [(1000, 1200)] * 2,  # more than two waves of tiles
    [(300, 400), (250, 900), (900, 1000)] + [(2048, 2048)] * 4,  # larger tiles than the single calls'
    [(100 + 17 * i, 160 + 31 * i) for i in range(20)],           # too many entries for shares
])
@pytest.mark.parametrize("precond", ["aol", "schatten4"])   # two reductions of the first Gram
def test_mixed_lengths_equal_single_calls(dtype, shapes, precond):
    """Entries of different K in one launch: every XCD takes an eighth of each, the long ones
    first; a tile left out or done for another matrix would show in the bits, and so would an
    element whose products or sums depend on the tile size."""
    log(f"case: mixed lengths {dtype} {precond}, {len(shapes)} matrices, the last {shapes[-1]}")
    ts = [to_device(make_input(m, n, 0.8, 40 + i, dtype), dtype) for i, (m, n) in enumerate(shapes)]
    ref = [t.clone() for t in ts]
    tm.orthogonalize_grouped(ts, 3, None, precond)
    for t, r in zip(ts, ref):
        tm.orthogonalize(r, 3, None, precond)
    torch.cuda.synchronize()
    for i, (t, r) in enumerate(zip(ts, ref)):
        assert torch.equal(t, r), i
