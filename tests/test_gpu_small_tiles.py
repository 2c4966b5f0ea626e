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


def test_projection_work_follows_the_rows_there_are():
    """`rows` is an upper bound on off[B].  With four times the rows the call may pick a wider tile, but the tiles that exist go
    to all dies alike: when they were dealt out by the bound, 1500 of 6000 rows took 2.8 times as long as 1500 of 1500."""
    H, d, total = 16, 2048, 1500
    g = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16)  # noqa: E731
    x, W = rnd(4 * total, d), [rnd(H * 128, d) * d ** -0.5 for _ in range(3)]
    pages_of = (total + 15) // 16
    off, pos = (torch.tensor(v, dtype=torch.int32, device="cuda") for v in ([0, total], range(4 * total)))

    def project(rows):
        cache = P.KVCache(torch.zeros((pages_of, 2, H, 16, 128), dtype=torch.bfloat16, device="cuda"),
                          torch.arange(pages_of, dtype=torch.int32, device="cuda").reshape(1, -1), torch.zeros(1, dtype=torch.int32, device="cuda"))
        Q = torch.zeros((4 * total, H, 128), dtype=torch.bfloat16, device="cuda")
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ms = []
        for _ in range(10):
            ev[0].record()
            for _ in range(10):
                P.dllava_qkv_project(x, d, rows, d, 1, off, pos, *W, 10000.0, Q, cache, None, P.BF16)
            ev[1].record()
            torch.cuda.synchronize()
            ms.append(ev[0].elapsed_time(ev[1]))
        return min(ms), Q, cache.pages

    t1, Q1, p1 = project(total)
    t4, Q4, p4 = project(4 * total)
    assert torch.equal(Q1.view(torch.int16), Q4.view(torch.int16)) and torch.equal(p1.view(torch.int16), p4.view(torch.int16))
    assert not Q4[total:].any()
    assert t4 < 1.7 * t1, (t1, t4)


@pytest.mark.parametrize("tile", [1, 4, 5, 6, 7, 8, 9, 10])
@pytest.mark.parametrize("dh", [128, 300])
def test_score_vectors_at_any_address(tile, dh):
    """Bias and output weights one element off their alignment (read through LDS) give the bits of aligned ones (read by fours)."""
    M, d = 130, 128
    g = torch.Generator(device="cuda").manual_seed(9)
    rnd = lambda *s, dtype=torch.bfloat16: torch.randn(s, generator=g, device="cuda", dtype=dtype)  # noqa: E731
    x, W1, b1, W2 = rnd(M, d), rnd(dh, d), rnd(dh + 1, dtype=torch.float32), rnd(2 * dh + 1)
    ws = torch.zeros(P.dllava_score_workspace(M, d, dh, P.BF16), dtype=torch.uint8, device="cuda")
    out = []
    P.dllava_set_launch_override(P.LAUNCH_SCORE_TILE, tile)
    try:
        for off in (0, 1):
            bias, weights = torch.zeros(dh + 1, device="cuda"), torch.zeros(2 * dh + 1, dtype=torch.bfloat16, device="cuda")
            bias[off:off + dh], weights[off:off + 2 * dh] = b1[:dh], W2[:2 * dh]
            D = torch.zeros((M, 2), device="cuda")
            P.dllava_score(x, d, M, 0, None, None, None, d, dh, W1, bias[off:], weights[off:], None, P.BF16, D, ws)
            out.append(D)
    finally:
        P.dllava_set_launch_override(P.LAUNCH_SCORE_TILE, 0)
    assert out[0].abs().max() > 0 and torch.equal(*out)
