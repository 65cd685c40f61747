"""Counts brought back through pinned host slots: calls from several threads on
streams of their own (each wait sees its own report), more of them at once than
the pool keeps slots, and a capacity error between good calls.  Results must
equal those of the same calls made one after the other."""

import threading

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


def chain(K, raw, p, ws):
    c = K.faster_pfh(raw, p, ws)
    m = K.match(c.feats.fpfh, c.feats.fpfh, c.feats.j_idx, c.feats.j_idx, ws=ws)
    return [c.kept_idx, c.normals.off, c.normals.idx, c.normals.flags, c.feats.j_idx, c.feats.fpfh, m.pairs, m.d1]


@pytest.mark.parametrize("threads", [2, 20])
def test_threads(K, threads):
    p = K.make_params(0.3, 0.75, 1.25)
    raws, want = [], []
    for t in range(threads):
        rng = np.random.default_rng(t)
        n = 600 + 37 * t
        xyz = rng.uniform(-4.0, 4.0, (3, n)).astype(np.float32)
        xyz[2] = 0.2 * np.sin(xyz[0]) + 0.02 * rng.standard_normal(n)
        raws.append(torch.from_numpy(xyz).cuda())
        want.append(chain(K, raws[t], p, K.Workspace()))
    torch.cuda.synchronize()
    bad = []

    def work(t):
        try:
            s, ws = torch.cuda.Stream(), K.Workspace()
            with torch.cuda.stream(s):
                for _ in range(5):
                    got = chain(K, raws[t], p, ws)
                    s.synchronize()
                    bad.extend((t, i) for i, (g, w) in enumerate(zip(got, want[t])) if not torch.equal(g, w))
        except Exception as e:  # a thread's failure must fail the test
            bad.append((t, repr(e)))

    ts = [threading.Thread(target=work, args=(t,)) for t in range(threads)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad, bad[:5]


def test_capacity_between(K):
    rng = np.random.default_rng(1)
    a = torch.from_numpy(rng.random((400, 33), dtype=np.float32)).cuda()
    first = K.match(a, a)
    with pytest.raises(Exception):
        K.voxelize(torch.full((3, 10), 1e30, device="cuda"), 1e-3)
    again = K.match(a, a)
    assert torch.equal(first.pairs, again.pairs) and torch.equal(first.d1, again.d1)
