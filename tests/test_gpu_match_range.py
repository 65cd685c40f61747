"""Rows at the border of the integer range of the matching: their integer norm
lies a few units on either side of it while rounding has lengthened or shortened
them by up to half a unit per value, and a query's two ordinary neighbours are
nearer, about as near, or farther than such a row.  Sets of 256 rows in all, so
that every row counts for the centre and the scale and both can be laid out
here.  Correspondences, d1 and d2 must equal the oracle's bit for bit."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

RANGE = 32600.0     # largest integer norm that takes part in the sweep
RMS = 4.0           # ... which is this many root mean square norms
UNIT = 2.0 ** -10   # the scale that the rows below are laid out for


@pytest.fixture(scope="module")
def K():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_15615_amd import kmg

    kmg.load()
    torch.cuda.set_device(0)
    return kmg


def border_vector(dim, steps):
    """The nearly equal integers whose norm is the first above RANGE, then `steps` values one more
    (or one less)."""
    v = np.full(dim, np.floor(RANGE / np.sqrt(dim)))
    i = 0
    while v @ v <= RANGE * RANGE:
        v[i] += 1
        i += 1
    for k in range(abs(steps)):
        v[-1 - k % dim] += np.sign(steps)
    return v


def lay_out(rng, dim, far, n):
    """n rows of which the first are `far` (in units, about the centre), the others such that the centre
    is where it is and the scale is UNIT."""
    m = (n - len(far)) // 2
    lean = -far.sum(0) / (2 * m)
    u = rng.standard_normal((m, dim))
    u = np.concatenate([u, -u])
    want = n * (RANGE / RMS) ** 2 - (far ** 2).sum() - 2 * m * (lean @ lean)
    assert want > 0
    u *= np.sqrt(want / (u ** 2).sum())
    rows = 24.0 + UNIT * np.concatenate([far, u + lean])
    assert rows.min() > 0
    return rows.astype(np.float32)


def integers(rows):
    """What the matching makes of the rows: integer vectors, and the rows themselves in units."""
    x = rows.astype(np.float64)
    x = x - x.mean(0)
    s = np.sqrt((x ** 2).sum(1).mean()) * RMS / RANGE
    return np.rint(x / s), x / s


@pytest.mark.parametrize("dim", [8, 33, 64])
@pytest.mark.parametrize("steps", [-2, 0, 2])        # integer norms just below and above the range
@pytest.mark.parametrize("frac", [-0.49, 0.0, 0.49])  # what rounding did to every value of the row
@pytest.mark.parametrize("near", [-30.0, -0.5, 0.5, 1.2, 30.0])  # ordinary rows: farther than the border row by
def test_border_rows(K, orc, dim, steps, frac, near):
    rng = np.random.default_rng(dim * 100 + steps)
    border = border_vector(dim, steps) + frac
    query = np.rint(border) - np.rint(430.0 / np.sqrt(dim))
    d = np.linalg.norm(border - query)
    side = rng.standard_normal((2, dim))
    side -= np.outer(side @ query, query) / (query @ query)
    side *= np.array([[d + near], [d + near + 0.3]]) / np.linalg.norm(side, axis=1, keepdims=True)
    far = np.stack([query, query + side[0], query + side[1], border])
    rows = lay_out(rng, dim, far, 256)
    q, x = integers(rows)
    if frac != 0.0:
        assert np.abs(np.abs(x[3] - q[3]) - 0.49).max() < 0.02  # the layout came out as meant
    if steps == 0 and frac == -0.49:
        assert np.linalg.norm(q[3]) > RANGE > np.linalg.norm(x[3])
    order = rng.permutation(253)
    X = np.concatenate([rows[:1], rows[4:104]])  # the query, and the border row among the partners, and the reverse
    Y = np.concatenate([rows[1:4], rows[104:]])[np.argsort(order[:155])]
    for a, b in ((X, Y), (Y, X)):
        mm = orc.mutual_match(a, b)
        out = K.match(torch.from_numpy(np.ascontiguousarray(a)).cuda(), torch.from_numpy(np.ascontiguousarray(b)).cuda())
        np.testing.assert_array_equal(out.pairs.cpu().numpy(), mm["pairs"])
        np.testing.assert_array_equal(out.d1.cpu().numpy(), mm["d1"].astype(np.float32))
        np.testing.assert_array_equal(out.d2.cpu().numpy(), mm["d2"].astype(np.float32))
