"""The graph and k-core kernels where their forms change: ranking around the
tiles of 256 keys with many equal ratios, Eq. (3) at pairs that lie exactly on
the threshold or beyond FP32's range (the FP32 decision gives way to FP64), rows
around the neighbours that a wavefront holds in registers, and sweeps that end
in each chunk.  Bit-exact against the oracle."""

import numpy as np
import pytest

from oracle import pose
from test_gpu_graph import K, check_graph, csr_of, dev  # noqa: F401 (K is the fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("k", [1, 255, 256, 257, 512, 513, 1500])
def test_rank_tiles(K, k):
    rng = np.random.default_rng(k)
    src = rng.uniform(-9, 9, (3, 400)).astype(np.float32)
    tgt = rng.uniform(-9, 9, (3, 400)).astype(np.float32)
    pairs = rng.integers(0, 400, (k, 2)).astype(np.int32)
    d2 = np.full(k, 2.0, np.float32)
    d1 = rng.integers(0, 7, k).astype(np.float32) * np.float32(0.25)  # seven ratios
    d2[::50], d1[::100] = 0.0, 0.0
    for n_tau in sorted({1, max(k // 2, 1), k}):
        check_graph(K, src, tgt, pairs, d1, d2, n_tau, 0.6)


@pytest.mark.parametrize("step,scale", [(0.25, 1.0), (0.1, 1.0), (0.25, 1e-20), (0.25, 1e18), (0.25, 1e25)])
def test_threshold(K, step, scale):
    # points on a lattice: gaps of exactly 2 beta (FP64 of the same FP32 coordinates decides)
    rng = np.random.default_rng(3)
    src = (rng.integers(-8, 9, (3, 500)) * step * scale).astype(np.float32)
    tgt = (rng.integers(-8, 9, (3, 500)) * step * scale).astype(np.float32)
    pairs = rng.integers(0, 500, (700, 2)).astype(np.int32)
    d1, d2 = rng.random(700).astype(np.float32), np.ones(700, np.float32)
    check_graph(K, src, tgt, pairs, d1, d2, 700, step * scale)


@pytest.mark.parametrize("n", [2048, 2049, 2050, 2200])
def test_long_rows(K, n):
    # a clique whose rows straddle the registers' 2,048 neighbours, and pendant vertices
    adj = np.zeros((n + 60, n + 60), bool)
    adj[:n, :n] = True
    adj[n:, 5] = True
    adj |= adj.T
    np.fill_diagonal(adj, False)
    off, idx = csr_of(adj)
    kc = K.max_kcore(dev(off), dev(idx), n + 60)
    core = np.r_[np.full(n, n - 1), np.ones(60)]
    np.testing.assert_array_equal(kc.core.cpu().numpy(), core)
    np.testing.assert_array_equal(kc.members.cpu().numpy(), np.arange(n))
    assert kc.max_core == n - 1


@pytest.mark.parametrize("length", [4, 20, 36, 60, 84, 97, 130])
def test_chunks_of_sweeps(K, length):
    # paths peel from both ends, a vertex or more a sweep: convergence in each chunk and past the last
    n = length + 12
    adj = np.zeros((n, n), bool)
    order = np.arange(length)[::-1]
    adj[order[:-1], order[1:]] = True
    adj[length:, length:] = True
    adj |= adj.T
    np.fill_diagonal(adj, False)
    off, idx = csr_of(adj)
    kc = K.max_kcore(dev(off), dev(idx), n)
    np.testing.assert_array_equal(kc.core.cpu().numpy(), pose.core_numbers(adj))
    np.testing.assert_array_equal(kc.members.cpu().numpy(), pose.max_kcore(adj))


@pytest.mark.parametrize("seed", range(3))
def test_one_way_rows(K, seed):
    # rows that do not name each other: still the greatest fixed point of the h-index operator
    rng = np.random.default_rng(seed)
    n = 700
    adj = rng.random((n, n)) < 0.05
    np.fill_diagonal(adj, False)
    off, idx = csr_of(adj)
    h = adj.sum(1)
    while True:
        new = h.copy()
        for v in range(n):
            w = np.sort(h[adj[v]])[::-1]
            new[v] = min(h[v], int((w >= np.arange(1, w.size + 1)).sum()))
        if (new == h).all():
            break
        h = new
    kc = K.max_kcore(dev(off), dev(idx), n)
    np.testing.assert_array_equal(kc.core.cpu().numpy(), h)
