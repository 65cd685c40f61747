"""Matching a few rows with very many: the sample of the large set is dealt to
more wavefronts the fewer queries there are (one segment of it per sort tile of
1,024 rows, up to 32, more tiles to a segment beyond).  Correspondences, d1 and
d2 must equal the oracle's, both ways round."""

import numpy as np
import pytest

import synth

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


@pytest.fixture(scope="module")
def rows():
    X, Y, _ = synth.synthetic_descriptors(34000, 700, item=9)
    return X, Y


@pytest.mark.parametrize("shape", [(1, 34000), (64, 34000), (65, 33793), (200, 32768), (200, 32769), (700, 9217),
                                   (3, 8192), (130, 8193)])
def test_uneven(K, orc, rows, shape):
    a, b = rows[1][: shape[0]], rows[0][-shape[1]:]
    for x, y in ((a, b), (b, a)):
        x, y = np.ascontiguousarray(x), np.ascontiguousarray(y)
        mm = orc.mutual_match(x, y)
        out = K.match(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
        np.testing.assert_array_equal(out.pairs.cpu().numpy(), mm["pairs"])
        np.testing.assert_array_equal(out.d1.cpu().numpy(), mm["d1"].astype(np.float32))
        np.testing.assert_array_equal(out.d2.cpu().numpy(), mm["d2"].astype(np.float32))
