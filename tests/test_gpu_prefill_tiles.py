"""The software-pipelined attention kernel of prefill_tiles.hip, forced through dllava_set_launch_override (the library takes it
for long sequences only): even and odd numbers of key tiles per wave, sequence lengths around the 32-key tiles and the items, few
blocks with many items each, keys in pages and in rows, the unmasked form, a maximum that keeps growing along the keys."""
import math
import os
import re
import subprocess

import numpy as np
import pytest
import torch

import paper_2412_00876_amd as P
from oracle import dllava_ref as R
from oracle import predictor_ref as PR
from synth import rng
from synth import workloads as W
from tests.test_gpu_parity import _assert_out_close

TILES, SHORT = 16, 32      # added to the waves of LAUNCH_PREFILL_WAVES: this kernel, the one for short sequences, whatever the size


def _run(q, k, v, lens, H, Dh, form, waves, blocks, scale, kernel=TILES):
    """q, k, v: bfloat16 bit patterns as the oracle takes them.  Page slots past a sequence's end hold NaN."""
    from tests import harness as h
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rows, B = int(off[-1]), len(lens)
    d = lambda a: h.to_dev(a, "bf16")  # noqa: E731
    qd, kd, vd, od = d(q), d(k), d(v), torch.from_numpy(off).to(h.DEV)
    cache = None
    if form == "paged":
        mp = max(1, (max(lens) + 15) // 16)
        pages = torch.full((B * mp, 2, H, 16, Dh), float("nan"), dtype=torch.bfloat16, device=h.DEV)
        table = torch.from_numpy(np.random.RandomState(1).permutation(B * mp).astype(np.int32).reshape(B, mp)).to(h.DEV)
        for b, n in enumerate(lens):
            for j in range(0, n, 16):
                m, pg = min(16, n - j), int(table[b, j // 16])
                pages[pg, 0, :, :m] = kd[off[b] + j:off[b] + j + m].transpose(0, 1)
                pages[pg, 1, :, :m] = vd[off[b] + j:off[b] + j + m].transpose(0, 1)
        cache, kd, vd = P.KVCache(pages, table, torch.tensor(lens, dtype=torch.int32, device=h.DEV)), None, None
    out = []
    P.dllava_set_launch_override(P.LAUNCH_PREFILL_WAVES, kernel + waves)
    P.dllava_set_launch_override(P.LAUNCH_PREFILL_BLOCKS, blocks)
    try:
        for _ in range(2):
            O = torch.full((rows, H, Dh), float("nan"), dtype=torch.bfloat16, device=h.DEV)
            if form == "full":
                P.dllava_span_attn(qd, kd, vd, B, od, rows, H, Dh, scale, O, P.BF16)
            else:
                P.dllava_prefill_attn(qd, kd, vd, cache, B, od, rows, H, Dh, scale, O, P.BF16)
            out.append(O)
        torch.cuda.synchronize()
    finally:
        P.dllava_set_launch_override(P.LAUNCH_PREFILL_WAVES, 0)
        P.dllava_set_launch_override(P.LAUNCH_PREFILL_BLOCKS, 0)
    assert torch.equal(out[0].view(torch.int16), out[1].view(torch.int16))   # same bits every time
    return h.as_f64(out[0]), off


def _reference(q, k, v, off, H, Dh, form, scale):
    if form != "full":
        return R.prefill_attn(q, k, v, off, scale, "bf16")
    ref = np.zeros((len(q), H * Dh))
    f = lambda a: R.widen(a, "bf16").reshape(len(a), H * Dh)  # noqa: E731
    for a, b in zip(off[:-1], off[1:]):
        if b > a:
            ref[a:b] = PR.attention(f(q[a:b]), f(k[a:b]), f(v[a:b]), heads=H)
    return ref.reshape(len(q), H, Dh)


def _qkv(seed, rows, H, Dh):
    return tuple(W.store(rng.normal(seed, t, (rows, H, Dh)), "bf16") for t in "qkv")


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["paged", "rows", "full"])
@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("waves,blocks", [(4, 0), (4, 1), (4, 3), (2, 0), (2, 3), (1, 0), (1, 7)])
@pytest.mark.parametrize("lens", [[1, 15, 16, 17, 31, 32, 33, 48], [127, 128, 129, 0, 95, 64], [160, 257, 385]])
def test_tile_edges(lens, waves, blocks, Dh, form):
    H, rows = 3, int(sum(lens))
    q, k, v = _qkv(80 + Dh, rows, H, Dh)
    O, off = _run(q, k, v, lens, H, Dh, form, waves, blocks, 1.0 / math.sqrt(Dh))
    _assert_out_close(O, _reference(q, k, v, off, H, Dh, form, 1.0 / math.sqrt(Dh)), "bf16", f"{form} {lens}")


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["paged", "rows", "full"])
@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("spread", [1.0, 6.0])
@pytest.mark.parametrize("lens", [[1, 31, 33, 64, 97], [160, 257, 385], [1500, 700]])
def test_the_bits_of_the_kernel_for_short_sequences(lens, spread, Dh, form):
    """The two kernels differ in when they do things, not in what they add up in which order: a sequence's outputs do not depend on the
    length from which the library takes the other one.  spread 6: scores of +-36 powers of two or so, the reference moves often."""
    H, rows = 2, int(sum(lens))
    q, k, v = _qkv(120 + Dh, rows, H, Dh)
    q = W.store(R.widen(q, "bf16") * spread, "bf16")
    for waves in (1, 2, 4):
        here, _ = _run(q, k, v, lens, H, Dh, form, waves, 0, 1.0 / math.sqrt(Dh))
        there, _ = _run(q, k, v, lens, H, Dh, form, waves, 0, 1.0 / math.sqrt(Dh), SHORT)
        assert np.array_equal(here, there), (waves, int((here != there).sum()), here.size)


def growing(seed, lens, H, Dh, slope):
    """q, k, v and a scale whose scores grow along the keys: steep, by about 11 powers of two per 32-key tile, more than the 8 from
    which the reference of the exponentials moves; some, the same for every fourth query and a thirtieth of it for the others;
    falling, downwards: the reference never moves again.  Values have a mean per tile, so that every tile's share shows."""
    q, k, v = (R.widen(a, "bf16") for a in _qkv(seed, sum(lens), H, Dh))
    q, at = np.abs(q), 0
    for n in lens:
        pos = np.arange(n)
        ramp = (pos[::-1] if slope == "falling" else pos) / 32.0 * 1.2
        k[at:at + n] = 0.05 * k[at:at + n] + ramp[:, None, None]
        v[at:at + n] = 0.25 * v[at:at + n] + (pos // 32 % 3 - 1.0)[:, None, None]
        if slope == "some":
            q[at:at + n][pos % 4 != 2] /= 32
        at += n
    return tuple(W.store(a, "bf16") for a in (q, k, v)) + (8.0 / Dh,)


def online(q, k, v, seen, scale, rescale=True):
    """Attention of one sequence and head as the kernels do it, in float64: 32 queries at a time over the 32-key tiles of which they see
    any key (seen [n, n]), the reference of the exponentials moved for all 32 when one of them is past it by more than 8 powers
    of two.  Returns the outputs, and for every tile but a group's first whether it moved the reference.  rescale=False: with the
    mistake of leaving the outputs and the sum as they are when it moves."""
    n = len(q)
    x = np.where(seen, q @ k.T * (scale * math.log2(math.e)), -np.inf)
    O, moved = np.zeros((n, v.shape[1])), []
    for i in range(0, n, 32):
        m, l, o, first = np.full(min(32, n - i), -1e30), 0.0, 0.0, True
        for j in range(0, n, 32):
            t = x[i:i + 32, j:j + 32]
            if not np.isfinite(t).any():
                continue
            move = bool((t.max(1) > m + 8).any())
            if move:
                old, m = m, np.maximum(m, t.max(1))
                if rescale:
                    l, o = l * np.exp2(old - m), o * np.exp2(old - m)[:, None]
            if not first:
                moved.append(move)
            first = False
            p = np.exp2(t - m[:, None])
            l, o = l + p.sum(1), o + p @ v[j:j + t.shape[1]]
        O[i:i + 32] = o / l[:, None]
    return O, moved


def growing_reference(q, k, v, off, seen_of, scale, slope, what):
    """The oracle's outputs for inputs of growing(), after checking on the host that they do what they are for: the reference moves
    in every tile but last ones of few keys (steep), in most (some), in none (falling); and leaving the old tiles' share as it was would show."""
    q, k, v = (R.widen(a, "bf16") for a in (q, k, v))
    ref, moves, wrong = np.zeros(q.shape), [], 0
    for a, b in zip(off[:-1], off[1:]):
        for h in range(q.shape[1]):
            seen = seen_of(a, b)
            s = np.where(seen, q[a:b, h] @ k[a:b, h].T * scale, -np.inf)
            w = np.exp(s - s.max(1, keepdims=True))
            ref[a:b, h] = w / w.sum(1, keepdims=True) @ v[a:b, h]
            out, moved = online(q[a:b, h], k[a:b, h], v[a:b, h], seen, scale)
            assert np.allclose(out, ref[a:b, h], rtol=1e-9, atol=1e-12)
            planted = online(q[a:b, h], k[a:b, h], v[a:b, h], seen, scale, rescale=False)[0]
            moves += moved
            wrong += int((np.abs(planted - ref[a:b, h]) > 4 * (2.0 ** -8 * np.abs(ref[a:b, h]) + 2e-3)).any(1).sum())
    if slope == "falling":
        assert not any(moves) and wrong == 0, what
    else:
        assert sum(moves) >= (0.8 if slope == "steep" else 0.6) * len(moves) and len(moves) > 30 and wrong > 40, (what, sum(moves), len(moves), wrong)
    return ref


@pytest.mark.gpu
@pytest.mark.parametrize("form", ["paged", "rows", "full"])
@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("slope", ["steep", "some", "falling"])
def test_growing_maximum(Dh, form, slope):
    """The reference of the exponentials moves in every tile, while the products of the tile before are pending, or never again; even
    and odd numbers of tiles."""
    H, lens = 2, [200, 33, 96, 161]
    q, k, v, scale = growing(90 + Dh, lens, H, Dh, slope)
    O, off = _run(q, k, v, lens, H, Dh, form, 4, 0, scale)
    seen = lambda a, b: np.ones((b - a, b - a), bool) if form == "full" else np.tril(np.ones((b - a, b - a), bool))  # noqa: E731
    ref = growing_reference(q, k, v, off, seen, scale, slope, (form, Dh))
    _assert_out_close(O, ref, "bf16", f"growing maximum {form} {Dh} {slope}")


@pytest.mark.gpu
@pytest.mark.parametrize("Dh", [64, 128])
def test_many_sequences(Dh):
    """Above 64 sequences: one item per block, found by scans."""
    H, lens = 2, [(37 * b) % 150 for b in range(80)]
    q, k, v = _qkv(100 + Dh, int(sum(lens)), H, Dh)
    O, off = _run(q, k, v, lens, H, Dh, "paged", 4, 0, 1.0 / math.sqrt(Dh))
    _assert_out_close(O, _reference(q, k, v, off, H, Dh, "paged", 1.0 / math.sqrt(Dh)), "bf16", "80 sequences")


@pytest.mark.gpu
@pytest.mark.parametrize("Dh", [64, 128])
def test_special_values_pass_through(Dh):
    """An infinity in a query, a NaN in a value and a key of zeros: not-a-number results where the definition gives them, the other
    rows as without them."""
    from tests import harness as h
    H, lens = 1, [130]
    q, k, v = (R.widen(a, "bf16") for a in _qkv(110 + Dh, 130, H, Dh))
    clean, _ = _run(*(W.store(a, "bf16") for a in (q, k, v)), lens, H, Dh, "rows", 4, 0, 0.1)
    q[70, 0, 3] = np.inf
    v[100, 0, 5] = np.nan
    O, _ = _run(*(W.store(a, "bf16") for a in (q, k, v)), lens, H, Dh, "rows", 4, 0, 0.1)
    bad = np.isnan(O)
    assert bad[70].all() and bad[101:, 0, 5].all() and not bad[:70].any() and not bad[71:100, 0, :5].any()
    keep = [i for i in range(96) if i != 70]      # rows of key tiles without the NaN
    assert np.array_equal(O[keep], clean[keep])


def test_tiles_kernels_do_not_spill():
    """The kernels count their outstanding vector-memory operations; scratch traffic would add to them."""
    from paper_2412_00876_amd import build
    r = subprocess.run([build.HIPCC, *build.COMMON, *build.HIP_FLAGS, "-Rpass-analysis=kernel-resource-usage", "--cuda-device-only", "-c",
                        os.path.join(build.CSRC, "prefill_tiles.hip"), "-o", os.devnull], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    scratch = re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)
    assert len(scratch) == 18 and set(scratch) == {"0"}
