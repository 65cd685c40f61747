"""Sets for which the matching's tiles are more than 32 bits number: refused with
KMG_ERR_WORKSPACE, never answered with no correspondences.  Two sets of 12 million
rows in both directions in full are ceil(12e6 / 64) = 187,500 query groups against
ceil(12e6 / 16 / 128) = 5,860 runs of chunks each way, 2.2e9 tiles."""

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N = 12_000_000


@pytest.fixture(scope="module")
def K():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2409_15615_amd import kmg

    kmg.load()
    torch.cuda.set_device(0)
    yield kmg
    kmg.set_tuning(None)


def test_too_many_tiles(K):
    assert 2 * -(-N // 64) * -(-N // (16 * 128)) > 2 ** 31
    x = torch.rand((N, 4), device="cuda")
    K.set_tuning({"match_form": 1})
    try:
        with pytest.raises(K.KmgError) as e:
            K.match(x, x, ws=K.Workspace())
    finally:
        K.set_tuning(None)
    assert e.value.status == K.KMG_ERR_WORKSPACE
    small = x[:3000].contiguous()
    assert K.match(small, small).pairs.shape[0] == 3000
