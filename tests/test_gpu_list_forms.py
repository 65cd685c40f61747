"""Neighbour lists around the lengths where the pass that writes them changes (928
entries) or its sort (1,024), and around a row of the batch form's pad: the lists of the
per-stage calls, and descriptors and correspondences of a batch in both search
forms, which must equal the per-stage calls'."""

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
    yield kmg
    kmg.set_tuning(None)


def balls(rng, sizes):
    """Balls of diameter 0.9, 3 apart: within a ball all points are neighbours at radius 1."""
    out = []
    for k, n in enumerate(sizes):
        b = rng.normal(size=(3, n))
        b *= rng.random(n) ** (1 / 3) * 0.45 / np.linalg.norm(b, axis=0)
        b[0] += 3.0 * (k % 8)
        b[1] += 3.0 * (k // 8)
        out.append(b)
    return np.concatenate(out, 1).astype(np.float32)


SIZES = [5, 927, 928, 929, 1000, 1023, 1024, 1025, 1100, 2100, 40, 3]


def test_lists_of_all_passes(K):
    rng = np.random.default_rng(1)
    xyz = balls(rng, SIZES)
    order = rng.permutation(xyz.shape[1])
    group = np.repeat(np.arange(len(SIZES)), SIZES)[order]
    out = K.normals(torch.from_numpy(np.ascontiguousarray(xyz[:, order])).cuda(), K.make_params(0.05, 0.5, 1.0))
    off, idx = out.off.cpu().numpy(), out.idx.cpu().numpy()
    np.testing.assert_array_equal(np.diff(off), np.array(SIZES)[group])
    members = [np.flatnonzero(group == k) for k in range(len(SIZES))]
    np.testing.assert_array_equal(idx, np.concatenate([members[g] for g in group]))


@pytest.mark.parametrize("copies", [1, 3])  # raw points a voxel: rows of the pad shorter than the lists, and longer
@pytest.mark.parametrize("form", [0, 1])
def test_batch_equals_stages(K, copies, form):
    rng = np.random.default_rng(2)
    p = K.make_params(1e-4, 0.6, 1.0, tau_num=3, tau_lin=0.99)
    clouds = []
    for sizes in ([930, 300], [928, 64], [1025, 33], [1024, 5]):
        pts = np.repeat(balls(rng, sizes), copies, axis=1)  # copies of a point fall into its voxel
        clouds.append((torch.from_numpy(np.ascontiguousarray(pts)).cuda(), p))
    raw = sum(int(c[0].shape[1]) for c in clouds)
    K.set_tuning({"search_form": form})
    try:
        b = K.Batch(2, raw, 1000 * raw, 11)
        b.upload(clouds)
        b.run()
        res = b.results()
        single = [K.faster_pfh(x, p) for x, _ in clouds]
        for i, r in enumerate(res):
            assert r.status == K.KMG_OK
            s, t = single[2 * i], single[2 * i + 1]
            m = K.match(s.feats.fpfh, t.feats.fpfh, s.feats.j_idx, t.feats.j_idx)
            assert r.kept == (s.xyz.shape[1], t.xyz.shape[1])
            assert r.n_j == (s.feats.j_idx.numel(), t.feats.j_idx.numel()) and min(r.n_j) > 0
            for side, c in enumerate((s, t)):
                fp, jj = b.descriptors(2 * i + side, r.kept[side], r.n_j[side])
                assert torch.equal(fp, c.feats.fpfh) and torch.equal(jj, c.feats.j_idx)
            assert torch.equal(r.pairs, m.pairs) and torch.equal(r.d1, m.d1) and torch.equal(r.d2, m.d2)
    finally:
        K.set_tuning(None)
