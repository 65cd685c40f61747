"""Exact scans of queries whose lists overflowed: the rows are read in norm order
and those whose norms no query of a group can reach are passed over.  Clusters
closer together than the integers resolve, of one norm, of several, all about the
norms of other rows, with equal rows far apart in the order (the smaller index
wins a tie), beside queries out of the integer range, which read every row.
Correspondences, d1 and d2 must equal the oracle's bit for bit."""

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


@pytest.mark.parametrize("dim", [33, 50])
@pytest.mark.parametrize("far", [0, 3])            # rows out of range on each side
@pytest.mark.parametrize("factors", [(1.0,), (0.3, 1.0, 1.7), (1.0, 1.0 + 1e-6)])
@pytest.mark.parametrize("shape", [(700, 2047), (1500, 2049), (2064, 1025)])
def test_clusters(K, orc, dim, far, factors, shape):
    rng = np.random.default_rng(dim + 10 * far + shape[0] + len(factors))
    X, Y = (rng.gamma(0.7, 10.0, (n, dim)) for n in shape)
    centre = rng.gamma(0.7, 10.0, dim)
    for Z in (X, Y):
        at = rng.permutation(Z.shape[0])[: Z.shape[0] * 3 // 4]
        for k, part in enumerate(np.array_split(at, len(factors))):
            Z[part] = factors[k] * (centre + 1e-3 * rng.random((part.size, dim)))
            Z[part[::7]] = Z[part[0]]  # equal rows all over the set
        if far:
            Z[rng.permutation(Z.shape[0])[:far]] *= 60.0
    check(K, orc, X, Y)
