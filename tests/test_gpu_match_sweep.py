"""The integer sweep of the matching at the sizes and values where it can go
wrong: set sizes around the chunk (16 rows), group (64 queries) and sample
(every row below 64 rows, then one in four) borders, descriptor lengths around
the padding, rows out of the integer range (as queries and as candidates), lists
longer than a query's registers and than its list, sets of equal rows, and the
two forms (both directions, one-sided) on the same sets.  Correspondences, d1
and d2 must equal the oracle's bit for bit."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def K():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_15615_amd import kmg

    kmg.load()
    torch.cuda.set_device(0)
    return kmg


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def check(K, orc, X, Y):
    X, Y = X.astype(np.float32), Y.astype(np.float32)
    mm = orc.mutual_match(X, Y)
    out = K.match(dev(X), dev(Y))
    np.testing.assert_array_equal(out.pairs.cpu().numpy(), mm["pairs"])
    np.testing.assert_array_equal(out.d1.cpu().numpy(), mm["d1"].astype(np.float32))
    np.testing.assert_array_equal(out.d2.cpu().numpy(), mm["d2"].astype(np.float32))
    return out


def rows(rng, n, dim):
    return rng.gamma(0.7, 10.0, (n, dim))


@pytest.mark.parametrize("shape", [(15, 17), (16, 16), (63, 64), (64, 63), (65, 129), (255, 257), (1023, 1025)])
def test_borders(K, orc, shape):
    rng = np.random.default_rng(sum(shape))
    Y = rows(rng, shape[1], 33)
    X = np.abs(Y[rng.integers(0, shape[1], shape[0])] * (1 + 0.05 * rng.standard_normal((shape[0], 33))))
    check(K, orc, X, Y)


@pytest.mark.parametrize("dim", [7, 8, 9, 36, 37, 63])
def test_lengths(K, orc, dim):
    rng = np.random.default_rng(dim)
    check(K, orc, rows(rng, 300, dim), rows(rng, 333, dim))


@pytest.mark.parametrize("n_far", [1, 20, 300])
def test_rows_out_of_range(K, orc, n_far):
    # rows far beyond the range that the scale holds, some with their twin among the far rows of
    # the other set, some nearest to ordinary rows; more of them than the short exact scan takes
    rng = np.random.default_rng(n_far)
    X, Y = rows(rng, 1500, 33), rows(rng, 1400, 33)
    far = rng.choice(1400, n_far, replace=False)
    X[far] *= 10.0 ** rng.uniform(1.5, 3.0, (n_far, 1))
    half = far[: (n_far + 1) // 2]
    Y[half] = X[half] * (1 + 1e-3 * rng.standard_normal((half.size, 33)))
    check(K, orc, X, np.abs(Y))


@pytest.mark.parametrize("n_same", [40, 200, 900])
def test_dense_clusters(K, orc, n_same):
    # n_same rows closer together than the rounding, beside spread ones: lists of n_same rows
    # (registers hold 64, a list a few hundred, the rest is scanned exactly)
    rng = np.random.default_rng(n_same)
    X, Y = rows(rng, 1200, 33), rows(rng, 1300, 33)
    centre = rows(rng, 1, 33)
    X[100:100 + n_same // 2] = centre + 1e-4 * rng.random((n_same // 2, 33))
    Y[50:50 + n_same] = centre + 1e-4 * rng.random((n_same, 33))
    check(K, orc, X, Y)


def test_equal_rows(K, orc):
    rng = np.random.default_rng(3)
    one = rows(rng, 1, 33)
    check(K, orc, np.repeat(one, 700, 0), np.repeat(one, 100, 0))
    check(K, orc, np.zeros((90, 33)), np.zeros((70, 33)))


@pytest.mark.parametrize("shape", [(1024, 1023), (1024, 1025), (2049, 2048), (3000, 1100)])
@pytest.mark.parametrize("norms", ["equal", "spread", "huge", "tiny", "bad"])
def test_norm_order(K, orc, shape, norms):
    # sets around the borders of the tiles that rows are ordered in by norm: all norms equal (nothing
    # is skipped), over six decades (nearly all is), with squares beyond FP32's range at either end, and
    # with rows that are not numbers (no row is their nearest)
    rng = np.random.default_rng(sum(shape))
    Y = rows(rng, shape[1], 33)
    X = np.abs(Y[rng.integers(0, shape[1], shape[0])] * (1 + 0.05 * rng.standard_normal((shape[0], 33))))
    if norms == "equal":
        X, Y = (v / np.linalg.norm(v, axis=1, keepdims=True) for v in (X, Y))
    if norms == "spread":
        X, Y = (v * 10.0 ** rng.uniform(-3, 3, (v.shape[0], 1)) for v in (X, Y))
    if norms in ("huge", "tiny"):
        s = 1e18 if norms == "huge" else 1e-22
        X, Y = X * s, Y * s
    if norms == "bad":
        X[::97, 5], Y[::89, 7], Y[3::60, 1] = np.nan, np.nan, np.inf
    check(K, orc, X, Y)


def test_forms_agree(K):
    # above the size from which matching is one-sided: the same pairs and distances both ways
    from synth import synthetic_descriptors

    X, Y, _ = synthetic_descriptors(26000, 21000, item=21)
    out = {}
    try:
        for form in (0, 1):
            K.set_tuning({"match_form": form})
            out[form] = K.match(dev(X), dev(Y))
    finally:
        K.set_tuning(None)
    for k in ("pairs", "d1", "d2"):
        assert torch.equal(getattr(out[0], k), getattr(out[1], k)), k
