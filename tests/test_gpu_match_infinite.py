"""Rows at an infinite distance are nobody's nearest (as in the oracle, where a
distance has to be below infinity to count), however few or many such rows a set
has and whichever scan meets them."""

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


@pytest.mark.parametrize("n", [2, 9, 40, 700])
@pytest.mark.parametrize("finite", [0, 1, 5])  # rows of the second set that are finite
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3e38])
def test_infinite_rows(K, orc, n, finite, value):
    rng = np.random.default_rng(n)
    X, Y = (rng.gamma(0.7, 10.0, (n, 33)).astype(np.float32) for _ in range(2))
    Y[min(finite, n):, 4] = value
    for a, b in ((X, Y), (Y, X), (Y, Y)):
        mm = orc.mutual_match(a, b)
        out = K.match(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda())
        np.testing.assert_array_equal(out.pairs.cpu().numpy(), mm["pairs"])
        np.testing.assert_array_equal(out.d1.cpu().numpy(), mm["d1"].astype(np.float32))
        np.testing.assert_array_equal(out.d2.cpu().numpy(), mm["d2"].astype(np.float32))
