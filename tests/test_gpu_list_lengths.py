"""Neighbour lists around the longest that the common fill pass holds in LDS (928
entries) and around the powers of two of its sorting: balls of n points that are
all neighbours of each other, among a few lone points.  Lists must be complete
and ascending, in the per-stage call and in the batch form."""

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


@pytest.mark.parametrize("n", [32, 33, 64, 65, 128, 129, 256, 257, 927, 928, 929, 1024, 1025])
def test_ball(K, n):
    rng = np.random.default_rng(n)
    ball = rng.normal(size=(3, n))
    ball *= rng.random(n) ** (1 / 3) * 0.45 / np.linalg.norm(ball, axis=0)
    lone = np.stack([np.arange(7) * 5.0 + 20, np.zeros(7), np.zeros(7)])
    xyz = np.concatenate([lone[:, :3], ball, lone[:, 3:]], axis=1).astype(np.float32)
    out = K.normals(torch.from_numpy(xyz).cuda(), K.make_params(0.05, 0.5, 1.0))
    lens = np.r_[np.ones(3), np.full(n, n), np.ones(4)].astype(np.int64)
    np.testing.assert_array_equal(out.off.cpu().numpy(), np.r_[0, np.cumsum(lens)])
    idx = out.idx.cpu().numpy()
    np.testing.assert_array_equal(idx[:3], [0, 1, 2])
    np.testing.assert_array_equal(idx[3:3 + n * n].reshape(n, n), np.tile(np.arange(3, 3 + n), (n, 1)))
