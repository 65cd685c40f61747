"""Neighbour lists from cell tables on both sides of the size from which cells
share windows (2^18 slots: 131,072 points), where windows fill up: lattices with
about one point per cell and several, so that cells collide in their windows.
Lists must equal the oracle's."""

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


@pytest.mark.parametrize("m", [131072, 131073, 150000])
@pytest.mark.parametrize("radius", [0.9, 1.6])
def test_lists(K, orc, m, radius):
    rng = np.random.default_rng(m)
    side = 54
    cells = rng.choice(side**3, m, replace=False)  # a nearly full cube about the origin
    xyz = np.stack([cells // side**2, cells // side % side, cells % side]).astype(np.float64) - side / 2
    xyz = (xyz + rng.uniform(-0.2, 0.2, xyz.shape)).astype(np.float32)
    off, idx = orc.radius_search(xyz, radius, grid=True)
    p = K.make_params(0.5, radius, radius)
    out = K.normals(torch.from_numpy(xyz).cuda(), p)
    np.testing.assert_array_equal(out.off.cpu().numpy(), off)
    np.testing.assert_array_equal(out.idx.cpu().numpy(), idx)
