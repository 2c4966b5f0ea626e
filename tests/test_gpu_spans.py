"""Rows gathered from vision spans: dllava_score and dllava_predict over spans give the bits of a call on the rows themselves, for
few and many sequences, on each of their row mappings (a table in LDS up to 1024 sequences in the tile kernels, one pass over
the sequences otherwise); and looking the rows up does not dominate the call."""
import numpy as np
import pytest
import torch

from paper_2412_00876_amd import binding as P
from synth import workloads as W
from tests import harness as h
from tests.test_gpu_predictor import upload

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _spans(B, longest, seed):
    """Lengths from -2 (counts as empty) to `longest`, gaps before and after every span: tensors, source rows, rows of x."""
    rs = np.random.RandomState(seed)
    n = rs.randint(-2, longest + 1, size=B)
    n[rs.randint(B)] = longest
    start, room = rs.randint(0, 4, size=B), rs.randint(0, 3, size=B)
    off = np.concatenate([[0], np.cumsum(start + np.maximum(n, 0) + room)])
    rows = np.concatenate([np.arange(off[b] + start[b], off[b] + start[b] + max(n[b], 0)) for b in range(B)])
    return tuple(torch.tensor(a, dtype=torch.int32, device=DEV) for a in (off, start, n)), torch.from_numpy(rows).to(DEV), int(off[-1]) + 1


@pytest.mark.parametrize("B,longest", [(1, 700), (5, 300), (70, 20), (1024, 3), (1030, 3), (1500, 0)])
@pytest.mark.parametrize("dtype,d,dh", [(torch.float32, 64, 40), (torch.bfloat16, 128, 130), (torch.bfloat16, 72, 9)])
def test_score(B, longest, dtype, d, dh):
    spans, rows, n_rows = _spans(B, max(longest, 1), B + d)
    code = P.F32 if dtype == torch.float32 else P.BF16
    g = torch.Generator(device=DEV).manual_seed(B)
    rnd = lambda *s: torch.randn(s, generator=g, device=DEV).to(dtype)  # noqa: E731
    x, W1, W2 = rnd(n_rows, d + 8), rnd(dh, d) * d ** -0.5, rnd(2, dh)
    total = len(rows)
    for extra in (0, 70):                              # rows beyond the spans: left as they are
        M = total + extra
        ws = torch.zeros(P.dllava_score_workspace(M, d, dh, code), dtype=torch.uint8, device=DEV)
        got, want = (torch.full((M, 2), 7.0, device=DEV) for _ in range(2))
        P.dllava_score(x, d + 8, M, B, *spans, d, dh, W1, None, W2, None, code, got, ws)
        packed = torch.cat([x[rows], x[rows[-1:]].expand(extra, -1)]).contiguous()
        P.dllava_score(packed, d + 8, M, 0, None, None, None, d, dh, W1, None, W2, None, code, want, ws)
        # at most 64 bfloat16 rows of a plain call go to another kernel
        assert torch.equal(got[:total], want[:total]) or (M <= 64 and torch.allclose(got[:total], want[:total], atol=1e-4))
        assert (got[total:] == 7.0).all()


@pytest.mark.parametrize("B,longest,nb", [(3, 200, 0), (70, 20, 0), (1030, 3, 0), (1030, 3, 1)])
def test_predict(B, longest, nb):
    """Without blocks every row is on its own: the bits of a plain call.  With blocks the attention couples the rows of a span:
    only that rows are found and finite is checked here, against the same call with the sequences packed."""
    spans, rows, n_rows = _spans(B, longest, B)
    d, total = 128, len(rows)
    desc = upload(h, W.paper_predictor(W.make("pp", "bf16", d, 2, 64, 1, [0], [64], [0], 0.5, 1, seed=4), nb), d)
    x = torch.randn(n_rows, d, generator=torch.Generator(device=DEV).manual_seed(1), device=DEV).to(torch.bfloat16)
    n = spans[2].clamp(min=0)
    packed = (torch.cat([torch.zeros_like(n[:1]), n.cumsum(0, dtype=torch.int32)]), torch.zeros_like(n), n)
    ws = torch.zeros(P.dllava_predict_workspace(total, B, nb), dtype=torch.uint8, device=DEV)
    out = []
    for src, sp in ((x, (B, *spans)), (x[rows].contiguous(), (B, *packed) if nb else (0, None, None, None))):
        D = torch.full((total, 2), float("nan"), device=DEV)
        P.dllava_predict(src, d, total, *sp, desc, P.BF16, D, ws)
        out.append(D)
    assert torch.isfinite(out[0]).all() and torch.equal(*out)


@pytest.mark.parametrize("dtype,d,dh,bound", [(torch.float32, 512, 128, 15.0), (torch.bfloat16, 5120, 1280, 8.0)])
def test_finding_rows_is_not_the_call(dtype, d, dh, bound):
    """3300 rows in 1100 spans against the same rows plain: 5 and 3 times the time.  One row after another it was 39 and 18."""
    B, code, ms = 1100, P.F32 if dtype == torch.float32 else P.BF16, []
    M, i32 = 3 * B, lambda a: torch.tensor(a, dtype=torch.int32, device=DEV)  # noqa: E731
    x, W1, W2, D = torch.randn(5 * B, d, device=DEV).to(dtype), torch.randn(dh, d, device=DEV).to(dtype), torch.randn(2, dh, device=DEV).to(dtype), torch.zeros(M, 2, device=DEV)
    ws = torch.zeros(P.dllava_score_workspace(M, d, dh, code), dtype=torch.uint8, device=DEV)
    for sp in ((0, None, None, None), (B, i32(list(range(0, 5 * B + 1, 5))), i32([1] * B), i32([3] * B))):
        ev, t = [torch.cuda.Event(enable_timing=True) for _ in range(2)], []
        for _ in range(8):
            ev[0].record()
            for _ in range(5):
                P.dllava_score(x, d, M, *sp, d, dh, W1, None, W2, None, code, D, ws)
            ev[1].record()
            torch.cuda.synchronize()
            t.append(ev[0].elapsed_time(ev[1]))
        ms.append(min(t))
    assert ms[1] < bound * ms[0], ms
