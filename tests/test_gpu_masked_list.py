"""dllava_masked_attn takes the visible keys in front of an item's 128 queries from a list where that spares enough of the 32-key tiles
that have a visible key, else it walks those: list lengths around its tiles and around that line, against the oracle and against the
walk, which a workspace of the mask words alone leads to; which keys either route reads; counts and list as they stand in the workspace."""
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
    # an entry that is read without having been written is key 0: a wrong result, nothing outside K and V
    ws = torch.zeros(P.dllava_masked_attn_workspace(rows, B), dtype=torch.uint8, device=h.DEV)
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


def _scattered(n, rs):
    """A third visible; of the hidden keys the first 128 are marked."""
    keep = (rs.rand(n) < 1 / 3).astype(np.uint8)
    return keep, (keep == 0) & (np.arange(n) < 128)


def _whole_tiles(n, rs):
    """Three of the first eight tiles hidden whole, and marked; everything else visible."""
    hidden = np.isin(np.arange(n) // 32, (1, 6, 7))
    return (~hidden).astype(np.uint8), hidden


@pytest.mark.gpu
@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("mask,first,words_only,clean", [(_scattered, 128, False, True), (_scattered, 128, True, False),
                                                         (_whole_tiles, 256, False, True), (_whole_tiles, 256, True, True)])
def test_hidden_rows_that_are_not_read(mask, first, words_only, clean, Dh):
    """V of the marked hidden keys is NaN, which reaches every query whose tiles hold one (0 times NaN).  Queries of later items: the list
    holds visible keys only, and a tile without a visible key is left out on either route; the walk over partly visible tiles reads
    the marked ones, which shows that this test can tell."""
    h = _H()
    lens, H = [first + 140, 700], 2
    rows, off = sum(lens), np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    q, k, v = _qkv(90 + Dh, rows, H, Dh)
    keep, marked = (np.concatenate(x) for x in zip(*(mask(n, np.random.RandomState(n)) for n in lens)))
    dirty = v.copy()
    dirty[marked] = 0x7fc0
    later = np.concatenate([np.arange(n) >= first for n in lens])
    O = h.as_f64(_call(h, *(h.to_dev(x, "bf16") for x in (q, k, dirty)), off, keep, H, Dh, words_only))[later]
    if clean:
        _assert_out_close(O, R.masked_attn(q, k, v, off, keep, 1.0 / math.sqrt(Dh), "bf16")[later], "bf16", "later queries")
    else:
        assert np.isnan(O).all()


@pytest.mark.gpu
@pytest.mark.parametrize("Dh", [64, 128])
def test_full_tiles_between_hidden_ones_are_walked(Dh):
    """Every other tile hidden whole, of the others 31 keys visible: less than half of the keys, but no fewer tiles from a list.  The
    same tiles as without a list, so the same bits."""
    h = _H()
    lens, H = [900, 130, 257], 2
    rows, off = sum(lens), np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    pos = np.concatenate([np.arange(n) for n in lens])
    keep = ((pos // 32 % 2 == 1) & (pos % 32 != 5)).astype(np.uint8)
    q, k, v = _qkv(95 + Dh, rows, H, Dh)
    dev = [h.to_dev(x, "bf16") for x in (q, k, v)]
    O, walk = (_call(h, *dev, off, keep, H, Dh, only) for only in (False, True))
    assert torch.equal(O.view(torch.int16), walk.view(torch.int16))
    _assert_out_close(h.as_f64(O), R.masked_attn(q, k, v, off, keep, 1.0 / math.sqrt(Dh), "bf16"), "bf16", "every other tile")


@pytest.mark.gpu
@pytest.mark.parametrize("lens", [[1, 31, 32, 33, 0, 127, 128, 129], [700, 255, 256, 257, 1030], [5000], [(37 * b) % 300 for b in range(90)]])
def test_counts_and_list(lens):
    """As they stand in the workspace: for word 4i of a sequence the visible keys in front of it, in the place of word 4i - 1 the words in
    front of 4i that are not zero; the visible keys in order, as bytes from the sequence's first row."""
    h = _H()
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rows, B, H, Dh = int(off[-1]), len(lens), 3, 64
    rs = np.random.RandomState(rows)
    keep = np.concatenate([(rs.rand(n) < 0.3) & (rs.rand(n // 32 + 1) < 0.7).repeat(32)[:n] for n in lens]).astype(np.uint8) * 7
    x = torch.zeros((rows, H, Dh), dtype=torch.bfloat16, device=h.DEV)
    ws = torch.zeros(P.dllava_masked_attn_workspace(rows, B), dtype=torch.uint8, device=h.DEV)
    P.dllava_masked_attn(x, x, x, B, torch.from_numpy(off).to(h.DEV), rows, H, Dh, 0.125, torch.from_numpy(keep).to(h.DEV), torch.zeros_like(x), P.BF16, ws)
    got = ws.cpu().numpy().view(np.uint32)
    slots = ((rows // 32 + B + 2) * 4 + 255) // 256 * 64
    for b, n in enumerate(lens):
        at, k = slots + off[b] // 32 + b, keep[off[b]:off[b + 1]] != 0
        for word in range(0, (n + 31) // 32, 4):
            assert got[at + word] == k[:32 * word].sum(), (b, word)
            if word:
                assert got[at + word - 1] == k[:32 * word].reshape(-1, 32).any(1).sum(), (b, word)
        listed = got[2 * slots + off[b] + 32 * b:][:k.sum()]
        assert (listed == np.flatnonzero(k) * (H * Dh * 2)).all(), b


@pytest.mark.gpu
def test_rows_that_span_4_gib():
    """Places in the list are 32 bits: a sequence whose rows span more walks its tiles.  The bits of the same heads in a call of
    their own."""
    n, H, Dh = 400, 65535, 128   # 256 rows of 16 MiB - 256 bytes: the last items' keys lie on both sides of 4 GiB
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.randn((n, 64, Dh), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    keep = (torch.rand(n, generator=g, device="cuda") < 1 / 3).to(torch.uint8)
    off = torch.tensor([0, n], dtype=torch.int32, device="cuda")

    def run(heads, ws):
        q_, k_, v_ = (t.repeat(1, 1024, 1)[:, :heads].contiguous() if heads > 64 else t for t in (q, k, v))
        O = torch.zeros_like(q_)
        P.dllava_masked_attn(q_, k_, v_, 1, off, n, heads, Dh, Dh ** -0.5, keep, O, P.BF16, ws)
        torch.cuda.synchronize()
        return O.view(torch.int16)

    full = torch.zeros(P.dllava_masked_attn_workspace(n, 1), dtype=torch.uint8, device="cuda")
    big, want = run(H, full), run(64, full[:((n // 32 + 3) * 4 + 255) // 256 * 256])
    assert want.any() and torch.equal(big[:, :64], want) and torch.equal(big[:, -63:], want[:, :63])


def test_no_register_is_kept_in_an_accumulator():
    """Fragments on their way from LDS are registers that the compiler takes as loaded: none may be moved to an accumulation register
    for want of room.  Those in use are the outputs, the queries and K: 64 at heads of 64, 128 at heads of 128."""
    from paper_2412_00876_amd import build
    src = os.path.join(build.CSRC, "masked_mfma.hip")
    r = subprocess.run([build.HIPCC, *build.COMMON, *build.HIP_FLAGS, "-Rpass-analysis=kernel-resource-usage", "-c", src, "-o", os.devnull],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    names = re.findall(r"Function Name: \S*masked_mfma_kernelILi(\d+)E", r.stderr)
    assert sorted(names) == ["128", "128", "64", "64"]
    agprs = re.findall(r"AGPRs: (\d+)", r.stderr)
    assert dict(zip(names, agprs)) == {"64": "64", "128": "128"}
    # spilled scalars would be moves to and from lanes of a vector register in the tile loop
    assert re.findall(r"SGPRs Spill: (\d+)", r.stderr) == ["0"] * 4
