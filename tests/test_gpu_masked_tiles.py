"""The matrix-core kernel of dllava_masked_attn at the edges of its tiles: sequence lengths around the 16-row groups, 32-key
tiles and 128-row items, few blocks with many items each (dllava_set_launch_override), key tiles that are hidden whole."""
import math

import numpy as np
import pytest
import torch

import paper_2412_00876_amd as P
from oracle import dllava_ref as R
from synth import rng
from synth import workloads as W
from tests.test_gpu_masked_attn import _H, _qkv, _run
from tests.test_gpu_parity import _assert_out_close
from tests.test_gpu_prefill_tiles import growing, growing_reference


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


@pytest.mark.gpu
@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("slope", ["steep", "some", "falling"])
def test_growing_maximum(Dh, slope):
    """The reference of the exponentials moves from tile to tile, with whole hidden tiles and hidden keys between: odd and even numbers
    of visible tiles, so that the walk ends on a tile of its own or on one without keys."""
    h = _H()
    H, lens = 2, [200, 33, 96, 161, 288, 321]
    q, k, v, _ = growing(190 + Dh, lens, H, Dh, slope)
    scale = 1.0 / math.sqrt(Dh)                                          # the one that _run passes
    q = W.store(R.widen(q, "bf16") * (8.0 / Dh / scale), "bf16")
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    pos = np.concatenate([np.arange(n) for n in lens])
    keep = rng.bernoulli(191, "keep", (len(pos),), 0.7).astype(np.uint8)
    keep[(pos // 32 % 4 == 1) | (pos // 32 == 6)] = 0
    O = h.as_f64(_run(h, q, k, v, off, keep, H, Dh))

    def seen(a, b):
        n = b - a
        return np.tril(np.broadcast_to(keep[a:b] != 0, (n, n)) | np.eye(n, dtype=bool))

    ref = growing_reference(q, k, v, off, seen, scale, slope, Dh)
    assert np.allclose(ref, R.masked_attn(q, k, v, off, keep, scale, "bf16"), rtol=1e-9, atol=1e-12)
    _assert_out_close(O, ref, "bf16", f"growing maximum, masked {Dh} {slope}")


@pytest.mark.gpu
@pytest.mark.parametrize("lens", [[1], [31, 32, 33, 0, 64, 65], [0, 0, 7, 0], [1000, 5, 96], [(37 * b) % 70 for b in range(130)]])
def test_mask_words(lens):
    """The packed masks that the kernel reads, as they stand in the workspace: word t of sequence b at off[b] / 32 + b + t."""
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rows, B = int(off[-1]), len(lens)
    keep = (np.arange(rows) * 2654435761 >> 7 & 3 != 0).astype(np.uint8) * 5     # any non-zero byte is "kept"
    d = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    x = torch.zeros((rows, 1, 64), dtype=torch.bfloat16, device="cuda")
    ws = torch.full((P.dllava_masked_attn_workspace(rows, B),), 0xa5, dtype=torch.uint8, device="cuda")
    P.dllava_masked_attn(x, x, x, B, d(off), rows, 1, 64, 0.125, d(keep), torch.zeros_like(x), P.BF16, ws)
    words = ws.cpu().numpy().view(np.uint32)
    for b, n in enumerate(lens):
        bits = np.zeros((n + 31) // 32 * 32, np.uint8)
        bits[:n] = keep[off[b]:off[b + 1]] != 0
        want = np.packbits(bits, bitorder="little").view(np.uint32)
        assert (words[off[b] // 32 + b:][:len(want)] == want).all(), b


@pytest.mark.gpu
@pytest.mark.parametrize("B", [65, 128, 193])
@pytest.mark.parametrize("Dh", [64, 128])
def test_many_sequences(B, Dh):
    """Above 64 sequences a block finds its item by scans of 64: the same bits as calls of at most 64 sequences, which number
    their items another way."""
    rs = np.random.RandomState(B)
    lens = np.where(rs.rand(B) < 0.2, 0, rs.randint(1, 300, size=B))
    lens[[0, 63, 64, B - 1]] = [129, 0, 257, 1]
    H, off = 2, np.concatenate([[0], np.cumsum(lens)])
    g = torch.Generator(device="cuda").manual_seed(B)
    q, k, v = (torch.randn((int(off[-1]), H, Dh), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    keep = (torch.rand(int(off[-1]), generator=g, device="cuda") < 0.4).to(torch.uint8)

    def run(first, last):
        a, z = int(off[first]), int(off[last])
        O = torch.zeros((z - a, H, Dh), dtype=torch.bfloat16, device="cuda")
        ws = torch.zeros(P.dllava_masked_attn_workspace(z - a, last - first), dtype=torch.uint8, device="cuda")
        P.dllava_masked_attn(q[a:z].contiguous(), k[a:z].contiguous(), v[a:z].contiguous(), last - first,
                             torch.tensor(off[first:last + 1] - a, dtype=torch.int32, device="cuda"), z - a, H, Dh, Dh ** -0.5, keep[a:z].contiguous(),
                             O, P.BF16, ws)
        return O

    parts = torch.cat([run(b, min(b + 64, B)) for b in range(0, B, 64)])
    assert torch.equal(run(0, B).view(torch.int16), parts.view(torch.int16)) and parts.any()


@pytest.mark.gpu
def test_time_of_many_short_sequences():
    """500 sequences of one row take 4 times as long as 64.  When every block walked the sequences it was 18 times."""
    t = []
    for B in (64, 500):
        x = torch.randn((B, 8, 64), device="cuda").to(torch.bfloat16)
        off, keep = torch.arange(B + 1, dtype=torch.int32, device="cuda"), torch.ones(B, dtype=torch.uint8, device="cuda")
        O, ws = torch.zeros_like(x), torch.zeros(P.dllava_masked_attn_workspace(B, B), dtype=torch.uint8, device="cuda")
        ev, ms = [torch.cuda.Event(enable_timing=True) for _ in range(2)], []
        for _ in range(8):
            ev[0].record()
            for _ in range(10):
                P.dllava_masked_attn(x, x, x, B, off, B, 8, 64, 0.125, keep, O, P.BF16, ws)
            ev[1].record()
            torch.cuda.synchronize()
            ms.append(ev[0].elapsed_time(ev[1]))
        t.append(min(ms))
    assert t[1] < 12 * t[0], t


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
