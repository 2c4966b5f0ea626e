"""The attention kernels' instructions written as such (products, loads into LDS): the compiler does not see what they need between them
and plain instructions, so the built assembly is read here.  Straight-line distances, label to label included."""
import os
import re
import subprocess

import pytest

# Wait states that the hardware does not insert by itself: an instruction is one, s_nop n is n + 1; a product occupies the matrix
# cores for 8, in which no other product starts.
PRODUCT = 8
AFTER_PRODUCT = 12       # a product's result before a plain instruction that touches it
BASE_OF_LOAD = 5         # a scalar register written by a vector instruction before a load that takes it as its base


def _registers(operand):
    out = set()
    for kind, one, lo, hi in re.findall(r"\b([vas])(?:(\d+)\b|\[(\d+):(\d+)\])", operand):
        out |= {(kind, i) for i in range(int(one or lo), int(one or hi) + 1)}
    return out


def _instructions(text):
    for line in text.splitlines():
        line = line.split(";")[0].strip()
        if line and not line.startswith(".") and not line.endswith(":"):
            name, _, rest = line.partition(" ") if " " in line else line.partition("\t")
            yield name, [o.strip() for o in re.split(r",(?![^\[]*\])", rest)]


def violations(text):
    out, now, products, scalars = [], 0, {}, {}          # register -> wait state at which its writer was over / was issued
    for name, operands in _instructions(text):
        if name in ("s_endpgm", "s_branch"):
            products, scalars = {}, {}
            continue
        touched = set().union(*(_registers(o) for o in operands)) if operands else set()
        if name.startswith("v_mfma"):
            now += PRODUCT - 1                            # the one before it has left the cores
            for r in _registers(operands[0]):
                products[r] = now
        else:
            for r in touched:
                if r in products and now - products[r] - 1 < AFTER_PRODUCT:
                    out.append(f"{name} {', '.join(operands)}: {r} {now - products[r] - 1} wait states after the product")
            if name.startswith("global_load_lds"):
                for r in _registers(operands[1]):
                    if r in scalars and now - scalars[r] - 1 < BASE_OF_LOAD:
                        out.append(f"{name} {', '.join(operands)}: {r} {now - scalars[r] - 1} wait states after it was written")
            written = _registers(operands[0]) if operands else set()
            for r in written:
                products.pop(r, None)
                scalars.pop(r, None)
                if r[0] == "s" and name.startswith("v_"):
                    scalars[r] = now
        now += int(operands[0], 0) + 1 if name == "s_nop" else 1
    return out


def test_the_reader_finds_them():
    load = "\ts_mov_b32 m0, s9\n\ts_nop 0\n\tglobal_load_lds_dwordx4 v1, s[4:5]\n"
    product = "\tv_mfma_f32_32x32x16_bf16 v[16:31], a[0:3], a[4:7], v[16:31]\n"
    assert violations("\tv_readfirstlane_b32 s5, v2\n" + load)
    assert violations("\tv_readfirstlane_b32 s5, v2\n\ts_nop 1\n" + load)
    assert not violations("\tv_readfirstlane_b32 s5, v2\n\ts_nop 2\n" + load)
    assert not violations("\tv_readfirstlane_b32 s5, v2\n\ts_add_u32 s4, s6, s7\n\ts_addc_u32 s5, s5, s8\n" + load)
    assert violations(product + "\tv_max_f32_e32 v1, v2, v20\n") and violations(product + "\ts_nop 10\n\tv_mov_b32_e32 v16, v1\n")
    assert not violations(product + "\ts_nop 11\n\tv_max_f32_e32 v1, v2, v20\n")
    other = "\tv_mfma_f32_32x32x16_bf16 a[16:31], v[0:3], v[4:7], a[16:31]\n"
    assert violations(product + other + "\tv_max_f32_e32 v1, v2, v20\n") and not violations(product + 2 * other + "\tv_max_f32_e32 v1, v2, v20\n")
    assert violations(product + other + other + "\tv_accvgpr_read_b32 v1, a20\n")


@pytest.mark.parametrize("source", ["prefill_tiles.hip", "masked_mfma.hip"])
def test_distances_in_the_built_kernels(source, tmp_path):
    from paper_2412_00876_amd import build
    out = tmp_path / "kernels.s"
    r = subprocess.run([build.HIPCC, *build.COMMON, *build.HIP_FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(out)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    text = out.read_text()
    assert text.count("v_mfma_f32_32x32x16_bf16") > 100 and text.count("global_load_lds_dwordx4") > 10
    found = violations(text)
    assert not found, found[:10]
