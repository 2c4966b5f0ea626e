"""dllava_masked_attn takes the visible keys in front of an item's 128 queries from a list where they are at most three quarters of
all keys there: list lengths around its 32-key tiles and around that line, against the oracle and against the walk over all keys,
which a workspace of the mask words alone leads to."""
import math
import os
import re
import subprocess

import numpy as np
import pytest
import torch

import paper_2412_00876_amd as P
from oracle import dllava_ref as R
from tests.test_gpu_masked_attn import _H, _qkv
from tests.test_gpu_parity import _assert_out_close


def _masks(lens, seen):
    """Of the first 128 keys of a sequence seen[b] are visible, of the others a third."""
    out = []
    for b, n in enumerate(lens):
        rs = np.random.RandomState(7 * n + seen[b])
        keep = (rs.rand(n) < 1 / 3).astype(np.uint8)
        head = np.zeros(min(n, 128), np.uint8)
        head[rs.permutation(len(head))[:seen[b]]] = 2
        keep[:len(head)] = head
        out.append(keep)
    return np.concatenate(out)


def _call(h, q, k, v, off, keep, H, Dh, words_only):
    rows, B = q.shape[0], len(off) - 1
    ws = torch.full((P.dllava_masked_attn_workspace(rows, B),), 0xff, dtype=torch.uint8, device=h.DEV)  # as a list: rows far outside
    if words_only:
        ws = ws[:((rows // 32 + B + 2) * 4 + 255) // 256 * 256]
    O = torch.full((rows, H, Dh), float("nan"), dtype=torch.bfloat16, device=h.DEV)
    P.dllava_masked_attn(q, k, v, B, torch.from_numpy(off).to(h.DEV), rows, H, Dh, 1.0 / math.sqrt(Dh), torch.from_numpy(keep).to(h.DEV), O, P.BF16, ws)
    return O


@pytest.mark.gpu
@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("blocks", [0, 2])
@pytest.mark.parametrize("lens,seen", [
    ([129, 160, 161, 192, 193, 255, 256, 257], [0, 1, 31, 32, 33, 64, 65, 95]),
    ([130, 385, 0, 300, 513], [96, 97, 0, 128, 63]),
    ([140 + b % 50 for b in range(70)], [(11 * b) % 129 for b in range(70)]),   # more than 64: one item per block
])
def test_list_lengths(lens, seen, blocks, Dh):
    h = _H()
    rows, H = int(sum(lens)), 3
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    q, k, v = _qkv(60 + Dh, rows, H, Dh)
    keep = _masks(lens, seen)
    dev = [h.to_dev(x, "bf16") for x in (q, k, v)]
    P.dllava_set_launch_override(P.LAUNCH_PREFILL_BLOCKS, blocks)
    try:
        O, again, walk = (_call(h, *dev, off, keep, H, Dh, only) for only in (False, False, True))
        torch.cuda.synchronize()
    finally:
        P.dllava_set_launch_override(P.LAUNCH_PREFILL_BLOCKS, 0)
    assert torch.equal(O.view(torch.int16), again.view(torch.int16))
    ref = R.masked_attn(q, k, v, off, keep, 1.0 / math.sqrt(Dh), "bf16")
    _assert_out_close(h.as_f64(O), ref, "bf16", "listed keys")
    _assert_out_close(h.as_f64(walk), ref, "bf16", "all keys")
    # the first 128 queries of a sequence have no list: the same tiles, the same bits
    first = torch.from_numpy(np.concatenate([np.arange(n) < 128 for n in lens])).to(h.DEV)
    assert torch.equal(O[first].view(torch.int16), walk[first].view(torch.int16))


def test_no_register_is_kept_in_an_accumulator():
    """Fragments on their way from LDS are registers that the compiler takes as loaded: none may be moved to an accumulation register
    for want of room.  Those in use are the outputs, the queries and K: 64 at heads of 64, 128 at heads of 128."""
    from paper_2412_00876_amd import build
    src = os.path.join(build.CSRC, "masked_mfma.hip")
    r = subprocess.run([build.HIPCC, *build.COMMON, *build.HIP_FLAGS, "-Rpass-analysis=kernel-resource-usage", "-c", src, "-o", os.devnull],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    names = re.findall(r"Function Name: \S*masked_mfma_kernelILi(\d+)E", r.stderr)
    agprs = re.findall(r"AGPRs: (\d+)", r.stderr)
    assert dict(zip(names, agprs)) == {"64": "64", "128": "128"}
