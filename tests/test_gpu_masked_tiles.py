"""The matrix-core kernel of dllava_masked_attn at the edges of its tiles: sequence lengths around the 16-row groups, 32-key
tiles and 128-row items, few blocks with many items each (dllava_set_launch_override), key tiles that are hidden whole."""
import math

import numpy as np
import pytest
import torch

import paper_2412_00876_amd as P
from oracle import dllava_ref as R
from synth import rng
from tests.test_gpu_masked_attn import _H, _qkv, _run
from tests.test_gpu_parity import _assert_out_close


@pytest.mark.gpu
@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("blocks", [0, 1, 3])
@pytest.mark.parametrize("lens", [[1, 15, 16, 17, 31, 32, 33], [127, 128, 129, 0, 95], [160, 257, 385]])
def test_tile_edges(lens, blocks, Dh):
    h = _H()
    rows, H = int(sum(lens)), 3
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    q, k, v = _qkv(70 + Dh, rows, H, Dh)
    keep = rng.bernoulli(71, "keep", (rows,), 0.4).astype(np.uint8)
    for b, n in enumerate(lens):       # runs of hidden keys that fill whole tiles, and one such tile at the start
        keep[off[b]:off[b] + min(n, 40)] = 0
        keep[off[b] + min(n, 64):off[b] + min(n, 130)] = 0
    P.dllava_set_launch_override(P.LAUNCH_PREFILL_BLOCKS, blocks)
    try:
        O = _run(h, q, k, v, off, keep, H, Dh)
        again = _run(h, q, k, v, off, keep, H, Dh)
        torch.cuda.synchronize()
    finally:
        P.dllava_set_launch_override(P.LAUNCH_PREFILL_BLOCKS, 0)
    _assert_out_close(h.as_f64(O), R.masked_attn(q, k, v, off, keep, 1.0 / math.sqrt(Dh), "bf16"), "bf16", f"masked {lens}")
    assert torch.equal(O.view(torch.int16), again.view(torch.int16))   # same bits every time


def test_masked_kernel_does_not_spill():
    """The kernel counts its outstanding vector-memory operations; scratch traffic would add to them."""
    import re
    import subprocess
    import os
    from paper_2412_00876_amd import build
    src = os.path.join(build.CSRC, "masked_mfma.hip")
    r = subprocess.run([build.HIPCC, *build.COMMON, *build.HIP_FLAGS, "-Rpass-analysis=kernel-resource-usage", "-c", src, "-o", os.devnull],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    scratch = re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)
    assert len(scratch) >= 2 and set(scratch) == {"0"}
