"""Every tile of the prefill's matrix products, launched directly (a plan's choice moves when its constants do)."""
import pytest

from tests import gemm_calls as gc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    return t


@pytest.fixture(scope="module")
def lib():
    from paper_2609_34045_amd import stage
    return stage.load_library()


@pytest.mark.parametrize("tile,rows", [(0, 32), (1, 64)])
def test_row_tiles_take_k_in_one_order(torch, lib, tile, rows):
    """Equal rows of A in different row tiles get the same bits: a tile's start in K depends on its columns alone."""
    n, k = 384, 320
    g = torch.Generator(device="cuda").manual_seed(3)
    a = torch.randn(rows, k, generator=g, device="cuda").half().repeat(128 // rows, 1).contiguous()
    w = torch.randn(n, k, generator=g, device="cuda").half()
    c, err = torch.zeros(128, n, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    assert gc.launch_gemm(lib, gc.RESID, tile, 1, a, w, None, 128, n, k, c, None, err, None) == 0
    torch.cuda.synchronize()
    for r in range(rows, 128, rows):
        assert torch.equal(c[r:r + rows], c[:rows]), r
