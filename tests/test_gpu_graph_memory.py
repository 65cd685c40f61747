"""A compatibility graph holds memory for about the entries it has, not for the
capacity that its call started from."""

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


@pytest.mark.parametrize("k", [1, 2, 70, 3000])
@pytest.mark.parametrize("wrong", [0.0, 0.9])
def test_adjacency_storage(K, k, wrong):
    rng = np.random.default_rng(k)
    src = rng.uniform(0.0, 50.0, (3, k)).astype(np.float32)
    tgt = src.copy()
    bad = rng.random(k) < wrong
    tgt[:, bad] = rng.uniform(0.0, 50.0, (3, int(bad.sum())))
    at = torch.arange(k, dtype=torch.int32, device="cuda")
    d = torch.ones(k, device="cuda")
    g = K.corr_graph(torch.from_numpy(src).cuda(), torch.from_numpy(tgt).cuda(), torch.stack([at, at], 1), d, 2 * d,
                     n_tau=3000, beta=0.45)
    entries = int(g.off[-1])
    assert g.adj.numel() == entries
    assert g.adj.untyped_storage().nbytes() <= 4 * max(64 * k, 2 * entries)
    # every right correspondence is compatible with every other
    right = np.flatnonzero(~bad)
    deg = (g.off[1:] - g.off[:-1]).cpu().numpy()
    sel = g.sel.cpu().numpy()
    assert (deg[np.isin(sel, right)] >= right.size - 1).all()
