"""The work count of per-stage timing: the query-row products that the matching's
sample and sweep evaluated, all of them where no chunk can be passed over by its
norms, far fewer where the norms are spread, none while timing is off."""

import ctypes as C

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
    kmg.load().kmg_timing_enable(0)


def work(K, X, Y):
    lib = K.load()
    x, y = (torch.from_numpy(np.ascontiguousarray(Z, np.float32)).cuda() for Z in (X, Y))
    ws = K.Workspace()
    lib.kmg_timing_enable(1)
    K.match(x, y, ws=ws)
    n = lib.kmg_timing_work(None, 0)
    w = (C.c_int64 * n)()
    lib.kmg_timing_work(w, n)
    lib.kmg_timing_enable(0)
    names = [lib.kmg_stage_name(i).decode() for i in range(n)]
    return int(w[names.index("match_topk")])


def all_products(nq, n):
    """A chunk is 16 rows; the sweep takes every chunk for each 16 queries, the sample one chunk in four
    (of sets of 64 rows and more, fewer than 1,024) for each 64."""
    chunks = -(-n // 16)
    sampled = chunks if n < 64 else -(-chunks // 4)
    return 256 * (-(-nq // 16) * chunks + 4 * -(-nq // 64) * sampled)


@pytest.mark.parametrize("shape", [(300, 400), (17, 50), (640, 64)])
def test_equal_norms(K, shape):
    rng = np.random.default_rng(1)
    X, Y = (rng.gamma(0.7, 10.0, (n, 33)) for n in shape)
    X, Y = (Z / np.linalg.norm(Z, axis=1, keepdims=True) for Z in (X, Y))
    assert work(K, X, Y) == all_products(*shape) + all_products(*shape[::-1])


def test_spread_norms(K):
    rng = np.random.default_rng(2)
    Y = rng.gamma(0.7, 10.0, (2000, 33)) * 10.0 ** rng.uniform(-1, 1, (2000, 1))
    X = Y * (1 + 1e-3 * rng.standard_normal(Y.shape))
    n = work(K, X, Y)
    assert 0 < n < all_products(2000, 2000) and n % 256 == 0
