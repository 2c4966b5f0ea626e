"""dllava_linear through every tile of its kernel (dllava_set_launch_override forces each): row and feature counts
that end inside a tile, stage counts around the depth of the operand ring, all epilogues."""
import numpy as np
import pytest
import torch

from oracle import dllava_ref as R
from oracle import predictor_ref as PR
from paper_2412_00876_amd import binding as P
from synth import rng
from synth import workloads as W
from tests.test_gpu_predictor import _assert_same_rounding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _dev(a):
    return torch.from_numpy(a.view(np.int16).copy()).to(DEV).view(torch.bfloat16)


@pytest.mark.parametrize("tile", [1, 2, 3, 9, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("M,N,K,act,res", [(1, 8, 64, 0, False), (129, 264, 128, 1, False), (161, 256, 192, 0, True), (257, 520, 256, 2, True),
                                           (193, 248, 320, 1, True), (449, 512, 704, 0, False), (70, 72, 1088, 1, True)])
def test_every_tile(tile, M, N, K, act, res):
    x = W.store(rng.normal(3, "x", (M, K)), "bf16")
    w = W.store(rng.normal(3, "w", (N, K)) / np.sqrt(K), "bf16")
    b = rng.normal(3, "b", (N,)).astype(np.float32)
    r = W.store(rng.normal(3, "r", (M, N)), "bf16")
    ref = PR.linear(R.widen(x, "bf16"), w, b, "bf16")
    g = R.widen(r, "bf16")
    if act == 1:
        ref = R.gelu(ref)
    if act == 2:
        ref = ref * (g / (1.0 + np.exp(-g)))
    elif res:
        ref = ref + g
    ldy = N + 8
    y = torch.zeros((M + 1, ldy), dtype=torch.bfloat16, device=DEV)
    rd = torch.zeros((M, ldy), dtype=torch.bfloat16, device=DEV)
    rd[:, :N] = _dev(r)
    P.dllava_set_launch_override(P.LAUNCH_LINEAR_TILE, tile)
    try:
        P.dllava_linear(_dev(x), K, M, K, _dev(w), torch.from_numpy(b).to(DEV), N, act, rd if res else None, y, ldy, P.BF16)
        torch.cuda.synchronize()
    finally:
        P.dllava_set_launch_override(P.LAUNCH_LINEAR_TILE, 0)
    got = y.view(torch.int16).cpu().numpy().view(np.uint16)
    assert (got[:, N:] == 0).all() and (got[M] == 0).all()   # nothing written beside the M x N block
    _assert_same_rounding(got[:M, :N], ref, f"linear {M}x{K}x{N} tile {tile}")


TILES = [1, 2, 3, 9, 4, 5, 6, 7, 8, 11, 12]


class _Forced:
    def __init__(self, tile):
        self.tile = tile

    def __enter__(self):
        P.dllava_set_launch_override(P.LAUNCH_LINEAR_TILE, self.tile)

    def __exit__(self, *_):
        P.dllava_set_launch_override(P.LAUNCH_LINEAR_TILE, 0)


@pytest.mark.parametrize("act", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(129, 264, 128), (70, 72, 1088), (257, 520, 256)])
def test_in_place_from_wide_rows(M, N, K, act):
    """x with rows further apart than K, y in the place of the residual (or the gate): through every tile the bits of a call
    with packed x and a buffer of its own, which the test above holds to the oracle.  A sum runs along K in one order in
    all tiles."""
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.randn(s, generator=g, device=DEV, dtype=torch.bfloat16)  # noqa: E731
    x, w, r, b = rnd(M, K + 24), rnd(N, K) * K ** -0.5, rnd(M, N + 8), torch.randn(N, generator=g, device=DEV)
    packed = x[:, :K].contiguous()
    want = torch.zeros_like(r)
    P.dllava_linear(packed, K, M, K, w, b, N, act, r, want, N + 8, P.BF16)
    for tile in TILES:
        y = r.clone()
        with _Forced(tile):
            P.dllava_linear(x, K + 24, M, K, w, b, N, act, y, y, N + 8, P.BF16)
        assert torch.equal(y[:, :N].view(torch.int16), want[:, :N].view(torch.int16)), tile
        assert torch.equal(y[:, N:].view(torch.int16), r[:, N:].view(torch.int16)), tile


@pytest.mark.parametrize("n_vis,d", [([130, 0, 300], 128), ([33, 31, 1, 64, 7], 64), ([520], 192)])
def test_image_predictor_through_every_tile(n_vis, d):
    """Rows gathered from ragged spans, q | k | v into three matrices, the output projection and the second layer of the MLP in
    the place of their residual: the same bits through every tile, and those of the automatic pick held to the oracle by
    the predictor's own tests."""
    from tests import harness as h
    from tests.test_gpu_predictor import _span_rows, _wl, _workspace, upload
    B = len(n_vis)
    w = _wl(d, [3] * B, n_vis, [5] * B, 6)
    desc = upload(h, W.paper_predictor(w, 2), d)
    hidden = h.to_dev(W.store(rng.normal(w.seed, "hid", (w.sumN, d)) * 1.5, "bf16"), "bf16")
    M = len(_span_rows(w))
    i32 = lambda a: torch.from_numpy(np.asarray(a, np.int32)).to(DEV)  # noqa: E731
    spans = (i32(w.seq_off), i32(w.vis_start), i32(w.vis_len))
    out = []
    for tile in [0] + TILES:
        D = torch.full((M, 2), float("nan"), device=DEV)
        with _Forced(tile):
            P.dllava_predict(hidden, d, M, B, *spans, desc, P.BF16, D, _workspace(h, M, B, 2))
        out.append(D)
    assert torch.isfinite(out[0]).all()
    for tile, D in zip(TILES, out[1:]):
        assert torch.equal(D, out[0]), tile
