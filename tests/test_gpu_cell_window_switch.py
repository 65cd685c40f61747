"""Neighbour lists at the two sizes between which the cells of the search start to
share windows: a table of twice the points, rounded up to a power of two, has
2^17 slots for 65,536 points (every cell hashed by itself) and 2^18 for 65,537
(windows); as one cloud and as a batch's clouds together."""

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


def lattice(m, seed):
    rng = np.random.default_rng(seed)
    side = 42
    cells = rng.choice(side ** 3, m, replace=False)  # a nearly full cube about the origin
    xyz = np.stack([cells // side ** 2, cells // side % side, cells % side]).astype(np.float64) - side / 2
    return (xyz + rng.uniform(-0.2, 0.2, xyz.shape)).astype(np.float32)


@pytest.mark.parametrize("m", [65535, 65536, 65537])
@pytest.mark.parametrize("radius", [0.9, 1.6])
def test_lists(K, orc, m, radius):
    xyz = lattice(m, m)
    off, idx = orc.radius_search(xyz, radius, grid=True)
    out = K.normals(torch.from_numpy(xyz).cuda(), K.make_params(0.5, radius, radius))
    np.testing.assert_array_equal(out.off.cpu().numpy(), off)
    np.testing.assert_array_equal(out.idx.cpu().numpy(), idx)


@pytest.mark.parametrize("m", [65536, 65537])
def test_batch_table(K, m):
    # two clouds in one table of that size: descriptors and correspondences of the per-stage calls
    p = K.make_params(0.05, 1.2, 1.6)
    xyz = lattice(m, 3)
    clouds = [(torch.from_numpy(np.ascontiguousarray(x)).cuda(), p) for x in (xyz[:, :30000], xyz[:, 30000:])]
    b = K.Batch(1, m, 40 * m, 11)
    b.upload(clouds)
    b.run()
    r = b.results()[0]
    assert r.status == K.KMG_OK
    s, t = (K.faster_pfh(x, p) for x, _ in clouds)
    for side, c in enumerate((s, t)):
        fp, jj = b.descriptors(side, r.kept[side], r.n_j[side])
        assert torch.equal(fp, c.feats.fpfh) and torch.equal(jj, c.feats.j_idx)
    mt = K.match(s.feats.fpfh, t.feats.fpfh, s.feats.j_idx, t.feats.j_idx)
    assert torch.equal(r.pairs, mt.pairs) and torch.equal(r.d1, mt.d1) and torch.equal(r.d2, mt.d2)
