"""Two iterations per update (bf16, N at least 9 k from k = 256 on, 4 k from 512 on, 2 k
from 1280 on and 1.5 k from 3072 on): the k x k products of tm_fast.hip against the fp64 oracle at the edges of the tiles
and of the rule, for even and odd iteration counts, and equal bits from single, batched and
grouped calls that run different tiles."""
import numpy as np
import pytest

from oracle import turbomuon as O
from gpu_helpers import (BF16_TOL, EO_RATIO_TOL, SCHEDULE5, eo_ratio, from_device, log,
                         make_input, relF, to_device)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2512_04632_amd import _lib as tm  # noqa: E402


def one(X, iters, precond, coeffs=None):
    t = to_device(X, "bf16")
    tm.orthogonalize(t, iters, coeffs, precond)
    return t


# (k, N): the edges of the rule (256 x 2304, 512 x 2048 and 1280 x 2560 are in, 257 x 2304,
# 513 x 2048 and 1281 x 2560 out), tile remainders on either side, ragged N
SHAPES = [(256, 2304), (257, 2304), (300, 2701), (512, 2048), (513, 2048), (513, 2100),
          (575, 2333), (577, 2900), (640, 3000), (1280, 2560), (1281, 2560)]


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


def test_mixed_group_equals_single_calls_bitwise():
    """Pairs, step-by-step and fused-range matrices in one call: every launch covers other
    matrices, with other tiles, than the single calls'."""
    log("case: mixed group vs single calls, bitwise")
    shapes = [(768, 3072), (515, 515), (64, 576), (129, 1153), (1001, 777), (300, 375), (2048, 640),
              (1300, 2700),
              (768, 3072), (40, 41)]
    Xs = [make_input(m, n, 0.8, i, "bf16") for i, (m, n) in enumerate(shapes)]
    for precond, iters, part in (("aol", 4, Xs), ("frobenius", 5, Xs), ("schatten4", 3, Xs),
                                 ("aol", 4, [Xs[0], Xs[2], Xs[9]])):   # pairs and fused only
        ts = [to_device(X, "bf16") for X in part]
        tm.orthogonalize_grouped(ts, iters, None, precond)
        for i, X in enumerate(part):
            assert torch.equal(ts[i], one(X, iters, precond)), (precond, X.shape)


@pytest.mark.parametrize("scale", [30.0, 1e3])
def test_large_coefficients_stay_finite(scale):
    """Coefficients whose k x k matrices could leave fp16's range take the bf16
    step-by-step form: linear steps (scale, 0, 0) multiply by scale each."""
    log(f"case: linear steps of {scale}")
    X = make_input(520, 2100, 0.8, 5, "bf16")
    co = [(scale, 0.0, 0.0)] * 4
    G = from_device(one(X, 4, "aol", co))
    R = O.orthogonalize(X, 4, co, "aol")
    assert np.isfinite(G).all() and relF(G, R) <= BF16_TOL


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_non_finite_input_stays_visible(bad):
    """One NaN or infinity reaches every output, as in the step-by-step form (its row sum
    scales every row)."""
    log(f"case: {bad} in the input")
    X = make_input(512, 2048, 0.8, 6, "bf16")
    X[5, 7] = bad
    assert np.isnan(from_device(one(X, 4, "aol"))).all()


def test_zero_rows_and_zero_matrix():
    log("case: zero rows, zero matrix")
    X = make_input(530, 2200, 0.8, 7, "bf16")
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
