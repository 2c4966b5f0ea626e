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
