"""Two iterations per update (bf16, k > 32 and N >= 1.25 k outside the fused kernel's
range): the k x k products of tm_fast.hip against the fp64 oracle at the edges of the tiles
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


# (k, N): the smallest k, tile remainders on either side, the ratio's edge (160 x 200 is
# in, 161 x 200 is out), a k with several 64 tiles and a ragged N
SHAPES = [(33, 1300), (63, 1111), (65, 1000), (128, 400), (160, 200), (161, 200),
          (193, 777), (257, 513), (320, 1024)]


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
              (768, 3072), (40, 41)]
    Xs = [make_input(m, n, 0.8, i, "bf16") for i, (m, n) in enumerate(shapes)]
    for precond, iters in (("aol", 4), ("frobenius", 5), ("schatten4", 3)):
        ts = [to_device(X, "bf16") for X in Xs]
        tm.orthogonalize_grouped(ts, iters, None, precond)
        for i, X in enumerate(Xs):
            assert torch.equal(ts[i], one(X, iters, precond)), (precond, shapes[i])


@pytest.mark.parametrize("scale", [30.0, 1e3])
def test_large_coefficients_stay_finite(scale):
    """Coefficients whose k x k matrices could leave fp16's range take the bf16
    step-by-step form: linear steps (scale, 0, 0) multiply by scale each."""
    log(f"case: linear steps of {scale}")
    X = make_input(96, 400, 0.8, 5, "bf16")
    co = [(scale, 0.0, 0.0)] * 4
    G = from_device(one(X, 4, "aol", co))
    R = O.orthogonalize(X, 4, co, "aol")
    assert np.isfinite(G).all() and relF(G, R) <= BF16_TOL


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_non_finite_input_stays_visible(bad):
    """One NaN or infinity reaches every output, as in the step-by-step form (its row sum
    scales every row)."""
    log(f"case: {bad} in the input")
    X = make_input(128, 512, 0.8, 6, "bf16")
    X[5, 7] = bad
    assert np.isnan(from_device(one(X, 4, "aol"))).all()


def test_zero_rows_and_zero_matrix():
    log("case: zero rows, zero matrix")
    X = make_input(130, 520, 0.8, 7, "bf16")
    X[3] = 0.0
    X[129] = 0.0
    G = from_device(one(X, 4, "aol"))
    R = O.orthogonalize(X, 4, None, "aol")
    assert relF(G, R) <= BF16_TOL and not G[3].any() and not G[129].any()
    assert not from_device(one(0.0 * X, 4, "frobenius")).any()
