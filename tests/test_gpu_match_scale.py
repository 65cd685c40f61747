"""The matching's integer scale beside a few rows of another order of magnitude
(or that are no numbers), among the rows that the scale is taken from: the
answers are the oracle's, and the other queries take no more work than without
those rows."""

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


def match(K, orc, X, Y):
    mm = orc.mutual_match(X, Y)
    out = K.match(torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda())
    np.testing.assert_array_equal(out.pairs.cpu().numpy(), mm["pairs"])
    np.testing.assert_array_equal(out.d1.cpu().numpy(), mm["d1"].astype(np.float32))
    np.testing.assert_array_equal(out.d2.cpu().numpy(), mm["d2"].astype(np.float32))
    return out.n_fallback


@pytest.mark.parametrize("factor", [1e2, 1e6, 1e15, 1e30, np.nan, np.inf])
@pytest.mark.parametrize("n_odd", [1, 12])
def test_few_odd_rows(K, orc, factor, n_odd):
    X, Y, _ = synth.synthetic_descriptors(1300, 1260, item=31)  # every tenth row is among those of the scale
    base = match(K, orc, X, Y)
    X, Y = X.copy(), Y.copy()
    for Z in (X, Y):
        Z[:: 10][:n_odd] *= np.float32(factor)
    odd = match(K, orc, X, Y)
    print(f"more than four exact scores: {base} queries, {odd} with {n_odd} rows x{factor} a side")
    assert odd <= base + 2 * n_odd + (X.shape[0] + Y.shape[0]) // 20


@pytest.mark.parametrize("n", [1, 2, 9, 10, 11, 127, 128, 129])
@pytest.mark.parametrize("share", [0.05, 0.12, 0.5])
def test_shares(K, orc, n, share):
    # few rows, some to half of them a thousand times the others
    rng = np.random.default_rng(n)
    X, Y = (rng.gamma(0.7, 10.0, (k, 33)) * np.where(rng.random((k, 1)) < share, 1e3, 1.0) for k in (n, n + 1))
    match(K, orc, X.astype(np.float32), Y.astype(np.float32))
