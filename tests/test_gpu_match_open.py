"""The exact scan of the queries that the integer sweep cannot serve, at the
numbers of them per set where lanes are shared differently (up to 8, 16, 32 and
64 to a group, and one more), and lists around the numbers of entries that are
gathered at a time.  Correspondences, d1 and d2 must equal the oracle's bit for
bit, with equal distances among the rows."""

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


def check(K, orc, X, Y):
    X, Y = np.ascontiguousarray(X, np.float32), np.ascontiguousarray(Y, np.float32)
    mm = orc.mutual_match(X, Y)
    out = K.match(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda())
    np.testing.assert_array_equal(out.pairs.cpu().numpy(), mm["pairs"])
    np.testing.assert_array_equal(out.d1.cpu().numpy(), mm["d1"].astype(np.float32))
    np.testing.assert_array_equal(out.d2.cpu().numpy(), mm["d2"].astype(np.float32))


@pytest.mark.parametrize("far", [(1, 16), (8, 9), (9, 8), (16, 17), (17, 33), (32, 1), (33, 64), (64, 65), (130, 7)])
@pytest.mark.parametrize("dim", [33, 50])
def test_open_queries(K, orc, far, dim):
    # far rows of the two sets, every second one with a twin in the other set (and a second
    # copy of the twin, at the same distance)
    rng = np.random.default_rng(far[0] * 100 + far[1] + dim)
    n = 4001
    X, Y = rng.random((n, dim)), rng.random((n + 6, dim))
    at = rng.choice(n, far[0] + far[1], replace=False)
    ax, ay = at[: far[0]], at[far[0]:]
    X[ax] += 40.0 * (1 + rng.random((far[0], 1)))
    Y[ay] += 40.0 * (1 + rng.random((far[1], 1)))
    both = min(far[0], far[1]) // 2
    if both:
        Y[ay[:both]] = X[ax[:both]]
        Y[ay[both: 2 * both]] = X[ax[:both]]
    check(K, orc, X, Y)


@pytest.mark.parametrize("n_same", [15, 16, 17, 63, 64, 65, 66, 127, 129, 255, 256, 257, 258, 320])
def test_list_lengths(K, orc, n_same):
    # n_same rows closer together than the rounding, some of them equal, beside spread ones
    rng = np.random.default_rng(n_same)
    X, Y = rng.random((900, 33)), rng.random((1000, 33))
    c = rng.random(33)
    X[100:140] = c + 1e-6 * rng.random((40, 33))
    Y[300:300 + n_same] = c + 1e-6 * rng.random((n_same, 33))
    Y[310] = Y[300]
    check(K, orc, X, Y)
