"""The FPFH sum where its groups of lanes change: rows of 21 to 63 values (three
points per wavefront up to 42, then two), lists around the 21 and 32 places of a
round, and every choice of rows per step, on one cloud.  Bit-equal over the
choices; against the oracle within half a float32 unit or 1e-4 per bin."""

import numpy as np
import pytest

import synth
from test_gpu_parity import K, check_features, dev, kparams  # noqa: F401 (K is the fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def cloud(n, seed=2):
    # two sheets, thin enough in places for short lists
    rng = np.random.default_rng(seed)
    x, y = rng.uniform(0, 3, n), rng.uniform(0, 3, n) ** 2 / 3
    return np.stack([x, y, np.where(rng.random(n) < 0.5, 0.1 * np.sin(3 * x), 0.4 + 0.2 * y * y)]).astype(np.float32)


@pytest.mark.parametrize("bins", [7, 8, 14, 15, 21])
def test_row_lengths(K, orc, bins):
    p = synth.Params(voxel=0.05, r_normal=0.2, r_fpfh=0.25, n_bins=bins)
    out, sp, _, _ = check_features(K, orc, cloud(2500), p, np.array([1.0, 1.0, 9.0]))
    assert out.j_idx.numel() > 500


@pytest.mark.parametrize("rows", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("bins", [11, 16])
def test_rows_per_step(K, rows, bins):
    p = synth.Params(voxel=0.05, r_normal=0.2, r_fpfh=0.3, n_bins=bins)
    kp = kparams(K, p, np.array([1.0, 1.0, 9.0]))
    xyz = dev(cloud(2501, 3))
    nr = K.normals(xyz, kp)
    lens = (nr.off[1:] - nr.off[:-1]).cpu().numpy()
    assert {20, 21, 22, 31, 32, 33, 42, 43} <= set(lens.tolist())
    want = K.fpfh(xyz, nr.normals, nr.flags.clone(), nr.off, nr.idx, kp).fpfh.clone()
    try:
        K.set_tuning({"fpfh_rows": rows})
        got = K.fpfh(xyz, nr.normals, nr.flags.clone(), nr.off, nr.idx, kp).fpfh
    finally:
        K.set_tuning(None)
    assert torch.equal(got, want)
