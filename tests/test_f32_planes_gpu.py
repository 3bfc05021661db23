"""fp32 storage on the fp16 matrix cores (every matrix as two fp16 planes; k >= 64): against
the fp64 oracle at tile remainders, both orientations, every scale, with row scales far
apart, and the step back to the fp32 matrix instructions."""
import numpy as np
import pytest

from oracle import turbomuon as O
from gpu_helpers import SCHEDULE5, from_device, log, make_input, relF, to_device

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
from paper_2512_04632_amd import _lib as tm  # noqa: E402

# A product's operands carry 22 bits or more and its fp32 sums a few units of 2^-24; the
# small directions of AOL(X) grow by up to a^t = 3.44^4 = 140: 140 * 2^-22 = 3e-5.
TOL = 3e-5


def one(X, iters, precond, coeffs=None):
    t = to_device(X, "f32")
    tm.orthogonalize(t, iters, coeffs, precond)
    return from_device(t)


@pytest.mark.parametrize("k,N", [(64, 64), (65, 65), (64, 1000), (96, 301), (127, 128), (130, 515),
                                 (257, 400), (320, 1024)])
@pytest.mark.parametrize("precond,iters,coeffs", [("aol", 4, None), ("aol", 1, None), ("aol", 3, None),
                                                  ("frobenius", 5, None), ("schatten4", 2, None),
                                                  ("aol", 5, SCHEDULE5)])
def test_planes_match_oracle(k, N, precond, iters, coeffs):
    for tall in (False, True):
        m, n = (N, k) if tall else (k, N)
        log(f"case: planes {m}x{n} {precond} t={iters} schedule={coeffs is not None}")
        X = make_input(m, n, 0.8, 13 * k + N, "f32")
        e = relF(one(X, iters, precond, coeffs), O.orthogonalize(X, iters, coeffs, precond))
        log(f"relF={e:.3e}")
        assert e <= TOL


@pytest.mark.parametrize("tall", [False, True])
@pytest.mark.parametrize("precond,decades", [("aol", 6), ("frobenius", 3), ("frobenius", 7), ("schatten4", 7)])
def test_small_rows_keep_their_bits(tall, precond, decades):
    """Rows 10^-decades .. 10^decades of the others' size: the planes of X are scaled row by
    row and a lo plane underflows only after its hi plane, and under a uniform scale rows below
    2^-18 are worked on at that size, so the smallest rows of X1 (AOL: 10^-decades, the uniform
    scales: 10^-2 decades) come out with the accuracy of the largest."""
    log(f"case: row scales far apart, {precond} {decades} tall={tall}")
    X = make_input(96, 500, 0.8, 3, "f32")
    X = (X * np.logspace(-decades, decades, 96)[:, None]).astype(np.float32).astype(np.float64)
    R = O.orthogonalize(X, 4, None, precond)
    G = one(X.T if tall else X, 4, precond)
    G = G.T if tall else G
    for i in range(96):
        assert np.linalg.norm(G[i] - R[i]) <= TOL * np.linalg.norm(R[i]), i


@pytest.mark.parametrize("precond,iters", [("frobenius", 1), ("frobenius", 5), ("schatten4", 4)])
@pytest.mark.parametrize("k,N", [(64, 64), (300, 1000), (1000, 1100)])
def test_few_small_rows_under_a_uniform_scale(k, N, precond, iters):
    """Rows far below the others, in several blocks of the scale vector and at the tiles' edges."""
    log(f"case: few small rows, {k}x{N} {precond} t={iters}")
    X = make_input(k, N, 0.8, 9, "f32")
    small = sorted({0, 31, 63, k // 2, k - 1})
    X[small] *= np.array([2.0 ** -e for e in (20, 30, 40, 24, 50)])[: len(small), None]
    X[small[1]] *= 2.0 ** -10
    R = O.orthogonalize(X, iters, None, precond)
    G = one(X, iters, precond)
    assert relF(G, R) <= TOL
    for i in small:
        assert np.linalg.norm(G[i] - R[i]) <= TOL * np.linalg.norm(R[i]), i


@pytest.mark.parametrize("precond", ["aol", "frobenius"])
def test_small_columns_keep_their_bits(precond):
    """Columns at 2^-20 of the others: entries of about 2^-25 (400 columns), held to 2^-50 between
    the iterations."""
    log(f"case: small columns, {precond}")
    X = make_input(96, 400, 0.8, 4, "f32")
    X[:, ::7] *= 2.0 ** -20
    R = O.orthogonalize(X, 4, None, precond)
    G = one(X, 4, precond)
    for j in range(0, 400, 7):
        assert np.linalg.norm(G[:, j] - R[:, j]) <= TOL * np.linalg.norm(R[:, j]), j


def test_large_coefficients_keep_the_fp32_instructions():
    log("case: linear steps of 1e3 in fp32")
    X = make_input(96, 400, 0.8, 5, "f32")
    co = [(1e3, 0.0, 0.0)] * 4
    assert relF(one(X, 4, "aol", co), O.orthogonalize(X, 4, co, "aol")) <= 1e-4


def test_group_of_small_and_large_fp32():
    """Matrices on the planes and on the fp32 instructions in one call, zero matrices and
    rows among them."""
    log("case: mixed fp32 group")
    shapes = [(512, 700), (17, 33), (768, 3072), (63, 500), (500, 64), (1, 1)]
    Xs = [make_input(m, n, 0.8, i, "f32") for i, (m, n) in enumerate(shapes)]
    Xs[0][5] = 0.0
    Xs[4][:] = 0.0
    ts = [to_device(X, "f32") for X in Xs]
    tm.orthogonalize_grouped(ts, 4, None, "aol")
    for X, t in zip(Xs, ts):
        G = from_device(t)
        if not X.any():
            assert not G.any()
        else:
            assert relF(G, O.orthogonalize(X, 4, None, "aol")) <= 1e-4
    assert not from_device(ts[0])[5].any()


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_non_finite_input_stays_visible(bad):
    log(f"case: {bad} in an fp32 input")
    X = make_input(96, 300, 0.8, 6, "f32")
    X[5, 7] = bad
    assert np.isnan(one(X, 4, "aol")).all()


@pytest.mark.parametrize("precond,iters", [("frobenius", 1), ("frobenius", 4), ("schatten4", 1), ("schatten4", 4)])
@pytest.mark.parametrize("tall", [False, True])
@pytest.mark.parametrize("norm", [1e-3, 1e-7, 1.0, 1e6])   # norm^4, the Schatten-4 sum, is a normal fp32 number
def test_zero_rows_of_matrices_of_any_norm(precond, iters, tall, norm):
    """A uniform scale of 1 / norm reaches the zero rows too (a dead unit): the first factor's
    diagonal there is a s r kScaleY, which must stay finite in fp16 for any norm."""
    log(f"case: zero rows, {precond} t={iters} tall={tall} norm={norm}")
    X = make_input(100, 330, 0.8, 11, "f32")
    X = (X * (norm / np.linalg.norm(X))).astype(np.float32).astype(np.float64)
    X[[0, 63, 64, 99]] = 0.0
    G = one(X.T if tall else X, iters, precond)
    G = G.T if tall else G
    assert np.isfinite(G).all() and not G[[0, 63, 64, 99]].any()
    assert relF(G, O.orthogonalize(X, iters, None, precond)) <= TOL
