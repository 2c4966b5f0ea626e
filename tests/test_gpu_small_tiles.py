"""The tiles of one head / 128 units (9: x 192 rows, 10: x 64 rows) of the projection and scoring kernels, on the inputs of
the tests that force the other tiles."""
import pytest
import torch

from paper_2412_00876_amd import binding as P
from tests import test_gpu_edges as E
from tests import test_gpu_qkv as Q
from tests import test_gpu_score_generic as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [9, 10])
@pytest.mark.parametrize("H,d", [(3, 256), (2, 704), (4, 4096)])
def test_projection(tile, H, d):
    Q.test_projection_tiles_forced(tile, H, d)


@pytest.mark.parametrize("tile", [9, 10])
@pytest.mark.parametrize("d,dh", [(512, 320), (64, 40), (4096, 1024), (704, 130)])
def test_score(tile, d, dh):
    E.test_score_tiles_forced(tile, d, dh)


@pytest.mark.parametrize("tile", [9, 10])
def test_score_spans(tile):
    E.test_score_many_short_spans(1024, tile)


@pytest.mark.parametrize("tile", [0, 1, 4, 5, 6, 7, 8, 9, 10])
@pytest.mark.parametrize("dh", [1, 40, 130, 384])
def test_score_infinite_last_unit(tile, dh):
    P.dllava_set_launch_override(P.LAUNCH_SCORE_TILE, tile)
    try:
        G._infinite_last_unit(100, 64, dh, torch.bfloat16, P.BF16)
    finally:
        P.dllava_set_launch_override(P.LAUNCH_SCORE_TILE, 0)
