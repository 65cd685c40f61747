"""Core numbers of graphs whose rows straddle the lengths where a sweep changes its
form (256 and 2,048 neighbours), rows of all lengths side by side, and sparse ones."""

import numpy as np
import pytest

from oracle import pose
from test_gpu_graph import K, csr_of, dev  # noqa: F401 (K is the fixture)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def check(K, adj):
    off, idx = csr_of(adj)
    kc = K.max_kcore(dev(off), dev(idx), adj.shape[0])
    core = pose.core_numbers(adj)
    np.testing.assert_array_equal(kc.core.cpu().numpy(), core)
    np.testing.assert_array_equal(kc.members.cpu().numpy(), np.flatnonzero(core == core.max()))
    assert kc.max_core == core.max()


@pytest.mark.parametrize("n", [64, 65, 255, 256, 257, 258, 320, 2049])
def test_cliques(K, n):
    # a clique of n (rows of n - 1), one of a third of it, a bridge and pendant vertices
    m = n // 3
    adj = np.zeros((n + m + 40, n + m + 40), bool)
    adj[:n, :n] = True
    adj[n:n + m, n:n + m] = True
    adj[0, n] = True
    adj[n + m:, 3] = True
    adj |= adj.T
    np.fill_diagonal(adj, False)
    check(K, adj)


@pytest.mark.parametrize("density", [0.002, 0.02, 0.2, 0.6])
def test_random(K, density):
    rng = np.random.default_rng(int(1000 * density))
    n = 1300
    # vertices of very different degrees
    p = rng.random(n) ** 2
    adj = rng.random((n, n)) < density * 2 * np.sqrt(p[:, None] * p[None, :])
    adj = np.triu(adj, 1)
    check(K, adj | adj.T)
