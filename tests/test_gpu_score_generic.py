"""dllava_score on the precision-generic kernel: all of its forms (4, 8 or 16 waves, one or four rows per block, one to eight
hidden units per wave), hidden units that end inside a wave's group or a block's round, rows shorter and longer than one pass of a wave, spans with gaps and logits rows beyond the spans.
(bfloat16 comes here when d is no multiple of 64.)"""
import numpy as np
import pytest
import torch

from paper_2412_00876_amd import binding as P
from synth import rng

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,d,dh", [(1, 8, 1), (3, 248, 7), (7, 520, 129), (512, 72, 9), (513, 264, 130), (1030, 40, 137), (515, 4104, 5), (9, 16376, 3),
                                    (5, 512, 20), (300, 264, 47), (2049, 136, 33), (600, 8200, 40), (1025, 4096, 9),
                                    (2, 16384, 130), (300, 16384, 33), (600, 16384, 3)])
def test_matches_float64(M, d, dh, dtype):
    f32 = dtype == torch.float32
    t = lambda name, shape, s=1.0: torch.from_numpy(rng.normal(11, name, shape) * s).to(dtype)
    rows = 2 * M + 5
    x, W1, W2 = t("x", (rows, d + 8)), t("w1", (dh, d), d ** -0.5), t("w2", (2, dh))
    b1, b2 = (torch.from_numpy(rng.normal(11, n, s).astype(np.float32)) for n, s in (("b1", (dh,)), ("b2", (2,))))
    n0 = (M + 1) // 2
    spans = [(0, 2, n0), (n0 + 3, 1, 0), (n0 + 3, 1, max(M - n0 - 1, 0))]   # first row of the sequence, start in it, length
    src = np.concatenate([np.arange(o + s, o + s + n) for o, s, n in spans])
    so, vs, vl = (torch.tensor(c, dtype=torch.int32, device=DEV) for c in zip(*spans))
    out = torch.full((M + 1, 2), 7.0, device=DEV)
    code = P.F32 if f32 else P.BF16
    ws = torch.zeros(max(256, P.dllava_score_workspace(M, d, dh, code)), dtype=torch.uint8, device=DEV)
    P.dllava_score(x.to(DEV), d + 8, M, 3, so, vs, vl, d, dh, W1.to(DEV), b1.to(DEV), W2.to(DEV), b2.to(DEV), code, out, ws)
    got = out.cpu().double()
    pre = x[src][:, :d].double() @ W1.double().T + b1.double()
    h = torch.nn.functional.gelu(pre)
    ref = h @ W2.double().T + b2.double()
    # float32 sums: each of the d + 2 roundings of a unit's sum and of the dh + 2 of a logit is at most 2^-24 of the sum of
    # magnitudes up to it; GELU's slope is at most 1.13 and its own error 4e-7 of its argument's magnitude
    e = 2.0 ** -24
    mag = x[src][:, :d].double().abs() @ W1.double().abs().T + b1.double().abs()
    tol = ((1.13 * (d + 2) * e + 4e-7) * mag) @ W2.double().abs().T + (dh + 20) * e * (h.abs() @ W2.double().abs().T + b2.double().abs())
    n = len(src)
    assert n < M or M == 1
    assert ((got[:n] - ref).abs() <= tol).all(), f"worst {((got[:n] - ref).abs() / tol).max():.2f} of the bound"
    assert (got[n:] == 7.0).all()   # rows beyond the spans are not written


def test_few_hidden_units_are_cheap():
    """A row with two hidden units is a fraction of the work of a row with 128.  On blocks of 16 waves it took nearly half the
    time of one."""
    M, d, ms = 20000, 512, {}
    x = torch.randn(M, d, device=DEV)
    for dh in (2, 128):
        W1, W2, out = torch.randn(dh, d, device=DEV), torch.randn(2, dh, device=DEV), torch.zeros(M, 2, device=DEV)
        ws = torch.zeros(P.dllava_score_workspace(M, d, dh, P.F32), dtype=torch.uint8, device=DEV)
        ev, t = [torch.cuda.Event(enable_timing=True) for _ in range(2)], []
        for _ in range(10):
            ev[0].record()
            for _ in range(10):
                P.dllava_score(x, d, M, 0, None, None, None, d, dh, W1, None, W2, None, P.F32, out, ws)
            ev[1].record()
            torch.cuda.synchronize()
            t.append(ev[0].elapsed_time(ev[1]))
        ms[dh] = min(t)
    assert ms[2] < 0.3 * ms[128], ms


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,dh", [(3, 1), (3, 5), (7, 13), (600, 130)])
def test_infinite_last_unit(M, dh, dtype):
    """The last hidden unit overflows and is repeated in the places past dh: the logits are infinite, not NaN.  They are
    NaN in the one row that holds one."""
    d, code = 72, P.F32 if dtype == torch.float32 else P.BF16
    _infinite_last_unit(M, d, dh, dtype, code)


def _infinite_last_unit(M, d, dh, dtype, code):
    x, W1, W2 = torch.zeros(M, d, dtype=dtype), torch.zeros(dh, d, dtype=dtype), torch.ones(2, dh, dtype=dtype)
    x[:, 0], W1[-1, 0], W2[1, -1] = 1e30, 1e30, -2.0
    x[1, 1] = float("nan")
    out = torch.zeros((M, 2), device=DEV)
    ws = torch.zeros(P.dllava_score_workspace(M, d, dh, code), dtype=torch.uint8, device=DEV)
    P.dllava_score(x.to(DEV), d, M, 0, None, None, None, d, dh, W1.to(DEV), None, W2.to(DEV), None, code, out, ws)
    assert out[1].isnan().all()
    other = torch.arange(M, device=DEV) != 1
    assert (out[other, 0] == float("inf")).all() and (out[other, 1] == -float("inf")).all()
