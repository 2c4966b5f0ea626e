"""The output-text predictor on at most 64 rows: row counts around the groups of 8 rows that its head is compiled for (8, 16, 32 and a
second block of 32), with and without biases, against the oracle; rows past the spans stay as they were."""
import numpy as np
import pytest
import torch

import paper_2412_00876_amd as P
from oracle import predictor_ref as PR
from synth import rng
from synth import workloads as W

pytestmark = pytest.mark.gpu


def _predictor(h, Pw, d):
    dev = lambda v: None if v is None else h.to_dev(v, "bf16") if v.dtype == np.uint16 else torch.from_numpy(v).to(h.DEV)  # noqa: E731
    return P.Predictor(d, {k: dev(v) for k, v in Pw.items() if k != "blocks"}, [])


@pytest.mark.parametrize("bias", [True, False])
@pytest.mark.parametrize("M", [1, 7, 8, 9, 15, 16, 17, 24, 25, 31, 32, 33, 40, 41, 63, 64])
def test_rows(M, bias):
    from tests import harness as h
    d = 128
    w = W.make("pp", "bf16", d, 2, 64, 1, [0], [M], [0], 0.5, 1, seed=900 + M)
    Pw = W.paper_predictor(w, 0)
    x = W.store(rng.normal(w.seed, "x", (M, d)) * 1.5, "bf16")
    given = {k: (v if bias or not k.startswith("b_") else np.zeros_like(v)) for k, v in Pw.items()}
    ref = PR.predict(x, None, given, "bf16")
    if not bias:
        given = {k: (None if k.startswith("b_") else v) for k, v in given.items()}
    logits = torch.full((M + 3, 2), 7.0, dtype=torch.float32, device=h.DEV)
    ws = torch.full((P.dllava_predict_workspace(M, 0, 0),), 0x7f, dtype=torch.uint8, device=h.DEV)
    P.dllava_predict(h.to_dev(x, "bf16"), d, M, 0, None, None, None, _predictor(h, given, d), P.BF16, logits, ws)
    got = logits.cpu().numpy()
    # three stored tensors: the bounds of predictor logits
    assert np.abs(got[:M] - ref).max() <= 2e-2 and np.abs(got[:M] - ref).mean() <= 2e-3
    assert (got[M:] == 7.0).all()


@pytest.mark.parametrize("lens,M", [([3, 0, 4], 8), ([3, 0, 4], 20), ([9, 24], 40), ([1], 64)])
def test_rows_past_the_spans(lens, M):
    from tests import harness as h
    d, n = 64, sum(lens)
    w = W.make("pp", "bf16", d, 2, 64, 1, [0], [M], [0], 0.5, 1, seed=77)
    Pw = W.paper_predictor(w, 0)
    p = _predictor(h, Pw, d)
    x = W.store(rng.normal(w.seed, "x", (n, d)), "bf16")
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device=h.DEV)  # noqa: E731
    off = [0]
    for k in lens:
        off.append(off[-1] + k)
    logits = torch.full((M, 2), 7.0, dtype=torch.float32, device=h.DEV)
    ws = torch.full((P.dllava_predict_workspace(M, len(lens), 0),), 0x7f, dtype=torch.uint8, device=h.DEV)
    P.dllava_predict(h.to_dev(x, "bf16"), d, M, len(lens), i32(off), i32([0] * len(lens)), i32(lens), p, P.BF16, logits, ws)
    got = logits.cpu().numpy()
    assert np.abs(got[:n] - PR.predict(x, None, Pw, "bf16")).max() <= 2e-2
    assert (got[n:] == 7.0).all()
