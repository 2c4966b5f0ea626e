"""The tiles of the linear layers that share a compute unit (11: three 64 x 64, 12: two 128 x 128), on the inputs of the tests that
force the other tiles, and at the edges of their rings: stage counts around three (11) and two (12), many more tiles than fit the chip."""
import pytest
import torch

from paper_2412_00876_amd import binding as P
from tests import test_gpu_linear_tiles as T


@pytest.mark.gpu
@pytest.mark.parametrize("tile", [11, 12])
@pytest.mark.parametrize("M,N,K,act,res", [(1, 8, 64, 0, False), (129, 264, 128, 1, False), (161, 256, 192, 0, True), (257, 520, 256, 2, True),
                                           (63, 64, 320, 1, True), (65, 136, 384, 0, False), (70, 72, 1088, 1, True)])
def test_every_epilogue(tile, M, N, K, act, res):
    T.test_every_tile(tile, M, N, K, act, res)


@pytest.mark.gpu
@pytest.mark.parametrize("tile", [11, 12])
@pytest.mark.parametrize("M,N,K", [(5000, 1032, 64), (4099, 2048, 512), (20000, 136, 256)])
def test_many_tiles(tile, M, N, K):
    """Several rounds of blocks: the bits of the 256 x 256 tile (a sum runs along K in one order in all tiles)."""
    g = torch.Generator(device="cuda").manual_seed(6)
    x, w = (torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16) for s in ((M, K), (N, K)))
    w = w * K ** -0.5
    out = []
    for t in (8, tile):
        y = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
        with T._Forced(t):
            P.dllava_linear(x, K, M, K, w, None, N, 1, None, y, N, P.BF16)
        out.append(y.view(torch.int16))
    assert torch.equal(*out) and out[0].any()
