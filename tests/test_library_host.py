"""CPU-side checks of the C-ABI library: it loads, exports every symbol the header declares, its pure host
queries behave, and argument errors are reported on the host before anything is launched."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2412_00876_amd", "lib", "libdllava.so")
HDR = os.path.join(ROOT, "include", "dllava.h")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_2412_00876_amd import build
        build.build(verbose=False)
    import paper_2412_00876_amd.binding as b
    return b


def _declared_functions():
    src = open(HDR).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(dllava_[a-z_]+)\s*\(", src)))


def test_every_declared_symbol_is_exported(lib):
    names = _declared_functions()
    assert {"dllava_score", "dllava_select_compact", "dllava_prefill_attn", "dllava_decode_attn_append"} <= set(names)
    raw = C.CDLL(LIB)
    for n in names:
        assert hasattr(raw, n), n
    assert set(lib.EXPORTS) == set(names)


def test_version_and_workspace_queries(lib):
    assert lib.dllava_version() >= 100
    for q in (lib.dllava_score_workspace(16, 4096, 1024, lib.BF16), lib.dllava_score_workspace(9216, 4096, 1024, lib.BF16),
              lib.dllava_select_compact_workspace(16, 10800), lib.dllava_decode_workspace(16, 32, 128, 78),
              lib.dllava_decode_step_workspace(16, 32, 128, 78, 4096, 1024, lib.BF16)):
        assert q > 0 and q % 256 == 0
    # monotone in the problem size
    assert lib.dllava_select_compact_workspace(16, 20000) > lib.dllava_select_compact_workspace(16, 10000)
    assert lib.dllava_decode_workspace(32, 40, 128, 50) > lib.dllava_decode_workspace(16, 32, 128, 50)
    assert lib.dllava_score_workspace(0, 4096, 1024, lib.BF16) >= 256
    assert lib.dllava_decode_step_workspace(16, 32, 128, 78, 4096, 1024, lib.BF16) >= \
        lib.dllava_decode_workspace(16, 32, 128, 78) + lib.dllava_score_workspace(16, 4096, 1024, lib.BF16)


def _expect(lib, status, fn, *args):
    rc = fn(*args)
    assert rc == status, (rc, lib.lib().dllava_last_error().decode())
    assert lib.lib().dllava_last_error().decode() != ""


def test_argument_errors_are_reported_on_the_host(lib):
    L = lib.lib()
    EINVAL, ENULL, ESHAPE, EDTYPE, EWORKSPACE = -1, -2, -3, -4, -6
    fake = C.c_void_p(0x1000)       # never dereferenced: every call below must fail validation first
    # score
    _expect(lib, EDTYPE, L.dllava_score, fake, 64, 4, 0, None, None, None, 64, 16, fake, None, fake, None, 7, fake, fake, 1 << 20, None)
    _expect(lib, ESHAPE, L.dllava_score, fake, 63, 4, 0, None, None, None, 63, 16, fake, None, fake, None, 1, fake, fake, 1 << 20, None)
    _expect(lib, ENULL, L.dllava_score, None, 64, 4, 0, None, None, None, 64, 16, fake, None, fake, None, 1, fake, fake, 1 << 20, None)
    _expect(lib, EWORKSPACE, L.dllava_score, fake, 64, 4, 0, None, None, None, 64, 16, fake, None, fake, None, 1, fake, None, 0, None)
    # select_compact
    cache = lib._KvCache(0x1000, 0x1000, 0x1000, 4, 2, 16, 2, 64, 1)
    args = lambda mode, ratio, thr, d, dtype, ws, wsb: (fake, 2, fake, fake, fake, 40, mode, ratio, thr, fake, fake, d, None, None,
                                                         None, None, None, fake, fake, fake, None, dtype, ws, wsb, None)
    _expect(lib, EINVAL, L.dllava_select_compact, *args(0, 1.5, 0.0, 64, 1, fake, 1 << 20))
    _expect(lib, EINVAL, L.dllava_select_compact, *args(0, float("nan"), 0.0, 64, 1, fake, 1 << 20))
    _expect(lib, EINVAL, L.dllava_select_compact, *args(1, 0.5, float("nan"), 64, 1, fake, 1 << 20))
    _expect(lib, EINVAL, L.dllava_select_compact, *args(3, 0.5, 0.0, 64, 1, fake, 1 << 20))
    _expect(lib, ESHAPE, L.dllava_select_compact, *args(0, 0.5, 0.0, 36, 1, fake, 1 << 20))
    _expect(lib, EWORKSPACE, L.dllava_select_compact, *args(0, 0.5, 0.0, 64, 1, fake, 16))
    _expect(lib, EDTYPE, L.dllava_select_compact, *args(0, 0.5, 0.0, 64, 9, fake, 1 << 20))
    # prefill
    _expect(lib, ESHAPE, L.dllava_prefill_attn, fake, fake, fake, None, 1, fake, 8, 2, 96, 0.1, fake, 1, None)
    _expect(lib, EINVAL, L.dllava_prefill_attn, fake, fake, fake, None, 1, fake, 8, 2, 64, -1.0, fake, 1, None)
    _expect(lib, ENULL, L.dllava_prefill_attn, fake, None, None, None, 1, fake, 8, 2, 64, 0.1, fake, 1, None)
    bad = lib._KvCache(0x1000, 0x1000, 0x1000, 4, 2, 32, 2, 64, 1)          # page_size 32
    _expect(lib, ESHAPE, L.dllava_prefill_attn, fake, None, None, C.byref(bad), 1, fake, 8, 2, 64, 0.1, fake, 1, None)
    # decode
    _expect(lib, ENULL, L.dllava_decode_attn_append, fake, fake, fake, 2, None, 0.0, None, C.byref(cache), 0.1, fake, None, None, fake, 1 << 24, None)
    _expect(lib, EWORKSPACE, L.dllava_decode_attn_append, fake, fake, fake, 2, fake, 0.0, None, C.byref(cache), 0.1, fake, None, None, fake, 64, None)
    _expect(lib, ENULL, L.dllava_decode_attn_append, fake, fake, fake, 2, fake, 0.0, None, None, 0.1, fake, None, None, fake, 1 << 24, None)
    _expect(lib, EINVAL, L.dllava_decode_attn_append, fake, fake, fake, 2, fake, float("nan"), None, C.byref(cache), 0.1, fake, None, None, fake, 1 << 24, None)
    # decode, one-launch form: (x, ldx, d, dh, W1, b1, W2, b2, q, k, v, k_prev, v_prev, logits_prev, keep_prev_override, B, threshold,
    #                           cache, scale, o, logits, keep_prev_out, err_flag, workspace, bytes, stream)
    step = lambda **kw: tuple({**dict(x=fake, ldx=64, d=64, dh=16, W1=fake, b1=None, W2=fake, b2=None, q=fake, k=fake, v=fake,
                                      kp=None, vp=None, lp=None, ov=None, B=2, thr=0.0, cache=C.byref(cache), scale=0.1, o=fake,
                                      logits=fake, ko=None, err=None, ws=fake, wsb=1 << 24, st=None), **kw}.values())
    _expect(lib, ENULL, L.dllava_decode_step, *step(W1=None))                              # x without its predictor
    _expect(lib, ENULL, L.dllava_decode_step, *step(x=None, q=None))                       # no scoring, but q is still required
    _expect(lib, EWORKSPACE, L.dllava_decode_step, *step(x=None, wsb=64))
    _expect(lib, ENULL, L.dllava_decode_step, *step(logits=None))
    _expect(lib, ENULL, L.dllava_decode_step, *step(lp=C.c_void_p(0x2000)))                 # previous logits without previous K/V
    _expect(lib, EINVAL, L.dllava_decode_step, *step(kp=fake, vp=fake, lp=fake))            # logits_prev == logits
    _expect(lib, EWORKSPACE, L.dllava_decode_step, *step(wsb=64))
    _expect(lib, ENULL, L.dllava_decode_step, *step(cache=None))
    _expect(lib, EINVAL, L.dllava_decode_step, *step(scale=0.0))
    _expect(lib, ENULL, L.dllava_decode_commit, fake, fake, None, None, 2, 0.0, C.byref(cache), None, None, None)
    _expect(lib, EINVAL, L.dllava_decode_commit, fake, fake, fake, None, 2, float("nan"), C.byref(cache), None, None, None)
    # projection: (x, ldx, rows, d, B, off, pos, Wq, Wk, Wv, rope_base, Q_out, cache, err_flag, dtype, stream)
    proj = lambda **kw: tuple({**dict(x=fake, ldx=64, rows=8, d=64, B=2, off=fake, pos=fake, Wq=fake, Wk=fake, Wv=fake, base=10000.0,
                                      Q=fake, cache=C.byref(cache), err=None, dtype=1, st=None), **kw}.values())
    _expect(lib, ENULL, L.dllava_qkv_project, *proj(Wk=None))
    _expect(lib, ENULL, L.dllava_qkv_project, *proj(pos=None))                              # rotation asked for, no positions
    _expect(lib, EDTYPE, L.dllava_qkv_project, *proj(dtype=0))                              # cache is bfloat16
    _expect(lib, ESHAPE, L.dllava_qkv_project, *proj(d=60, ldx=60))
    _expect(lib, EINVAL, L.dllava_qkv_project, *proj(ldx=32))
    _expect(lib, EINVAL, L.dllava_qkv_project, *proj(base=float("nan")))
    _expect(lib, ENULL, L.dllava_qkv_project, *proj(cache=None))


def test_noop_sizes_return_ok_without_a_gpu(lib):
    L = lib.lib()
    fake = C.c_void_p(0x1000)
    assert L.dllava_score(fake, 64, 0, 0, None, None, None, 64, 16, fake, None, fake, None, 1, fake, None, 0, None) == 0
    cache = lib._KvCache(0x1000, 0x1000, 0x1000, 4, 2, 16, 2, 64, 1)
    assert L.dllava_decode_attn_append(fake, fake, fake, 0, fake, 0.0, None, C.byref(cache), 0.1, fake, None, None, None, 0, None) == 0
    assert L.dllava_prefill_attn(fake, fake, fake, None, 0, fake, 0, 2, 64, 0.1, fake, 1, None) == 0
    assert L.dllava_qkv_project(fake, 64, 0, 64, 2, fake, fake, fake, fake, fake, 10000.0, fake, C.byref(cache), None, 1, None) == 0
    assert L.dllava_decode_commit(fake, fake, fake, None, 0, 0.0, C.byref(cache), None, None, None) == 0


def test_product_path_has_no_cpu_fallback():
    """The package must not import the oracle (or anything else that could stand in for the kernels)."""
    pkg = os.path.join(ROOT, "paper_2412_00876_amd")
    for fn in os.listdir(pkg):
        if fn.endswith(".py"):
            src = open(os.path.join(pkg, fn)).read()
            assert "oracle" not in src, fn


def test_build_module_imports_without_loading_the_library():
    """The package loads the binding (and the shared library) on first use only, so the build module can be imported
    on a tree where the library does not exist yet or is older than the binding."""
    import subprocess
    import sys
    code = ("import sys; import paper_2412_00876_amd.build as b; "
            "assert 'paper_2412_00876_amd.binding' not in sys.modules; assert callable(b.build); print('ok')")
    out = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stderr


def test_prefill_kernel_does_not_spill():
    """The matrix-core prefill kernel waits for its asynchronous tile loads with explicit counts of outstanding
    vector-memory operations; register spills inside its loop would add scratch traffic to that count.  The
    compiler's resource report must show no scratch memory for any variant of the kernel."""
    import subprocess
    from paper_2412_00876_amd import build
    src = os.path.join(build.CSRC, "prefill_mfma.hip")
    cmd = [build.HIPCC, "-O3", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", build.CSRC, "--offload-arch=gfx950",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Rpass-analysis=kernel-resource-usage",
           "--cuda-device-only", "-c", src, "-o", os.devnull]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S*prefill_mfma_kernel\S*)", r.stderr)
    scratch = re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)
    assert len(names) >= 6 and len(scratch) == len(re.findall(r"Function Name:", r.stderr))
    blocks = r.stderr.split("Function Name: ")[1:]
    for b in blocks:
        if "prefill_mfma_kernel" in b.split()[0]:
            assert re.search(r"ScratchSize \[bytes/lane\]: 0\b", b), b[:400]


def test_ring_kernels_do_not_spill():
    """The loops of the tile products count their loads in the same way; here scratch traffic would also stand between their
    matrix instructions."""
    import subprocess
    from concurrent.futures import ThreadPoolExecutor
    from paper_2412_00876_amd import build

    def report(source):
        r = subprocess.run([build.HIPCC, *build.COMMON, *build.HIP_FLAGS, "-Rpass-analysis=kernel-resource-usage", "--cuda-device-only", "-c",
                            os.path.join(build.CSRC, source), "-o", os.devnull], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return [b for b in r.stderr.split("Function Name: ")[1:] if re.search("_ring_kernel|lin_shared_kernel", b.split()[0])]

    with ThreadPoolExecutor(3) as ex:
        kernels = list(ex.map(report, ("score_mfma.hip", "qkv_project.hip", "predictor.hip")))
    assert [len(k) for k in kernels] == [8, 8, 11]     # every tile
    for b in sum(kernels, []):
        assert re.search(r"ScratchSize \[bytes/lane\]: 0\b", b), b[:400]


def test_score_workspace_is_monotonic_in_rows(lib):
    """A workspace sized for the largest row count must serve every smaller one."""
    for d, dh in ((4096, 1024), (256, 64), (64, 1)):
        sizes = [lib.dllava_score_workspace(m, d, dh, lib.BF16) for m in (1, 16, 17, 64, 65, 200, 5000, 100000)]
        assert sizes == sorted(sizes), (d, dh, sizes)


def test_score_workspace_of_narrow_rows(lib):
    """d % 8 == 0 is all that dllava_score asks for: widths below one k-step of the matrix-core forms have a workspace too,
    alone and inside a decode step, and a query without units answers."""
    for d in (8, 40, 56):
        for dh in (1, 10, 1024):
            sizes = [lib.dllava_score_workspace(m, d, dh, lib.BF16) for m in (1, 64, 65, 100, 100000)]
            assert sizes[0] >= 256 and sizes == sorted(sizes), (d, dh, sizes)
            assert lib.dllava_decode_step_workspace(3, 4, 64, 8, d, dh, lib.BF16) > sizes[0]
    assert lib.dllava_score_workspace(100, 64, 0, lib.BF16) > 0


def test_predictor_entry_points_validate_on_the_host(lib):
    L = lib.lib()
    EINVAL, ENULL, ESHAPE, EDTYPE, EWORKSPACE = -1, -2, -3, -4, -6
    fake = C.c_void_p(0x1000)       # never dereferenced: every call below must fail validation first
    p = lib._Predictor()
    p.d, p.n_blocks = 128, 0
    p.W_in = p.W_h1 = p.W_h2 = p.W_h3 = 0x1000
    big = 1 << 30
    call = lambda pp, dtype, ldx, M, ws, wsb, x=fake: (x, ldx, M, 0, None, None, None, pp, dtype, fake, ws, wsb, None)
    _expect(lib, ENULL, L.dllava_predict, *call(None, 1, 128, 4, fake, big))
    _expect(lib, EDTYPE, L.dllava_predict, *call(C.byref(p), 0, 128, 4, fake, big))       # float32 is not offered
    _expect(lib, ESHAPE, L.dllava_predict, *call(C.byref(p), 1, 120, 4, fake, big))       # ldx < d
    _expect(lib, EWORKSPACE, L.dllava_predict, *call(C.byref(p), 1, 128, 4, None, 0))
    _expect(lib, EWORKSPACE, L.dllava_predict, *call(C.byref(p), 1, 128, 4, fake, 64))
    _expect(lib, ENULL, L.dllava_predict, *call(C.byref(p), 1, 128, 4, fake, big, x=None))
    assert L.dllava_predict(*call(C.byref(p), 1, 128, 0, None, 0)) == 0                   # M == 0: nothing to do
    q = lib._Predictor()
    q.d, q.n_blocks = 100, 0
    q.W_in = q.W_h1 = q.W_h2 = q.W_h3 = 0x1000
    _expect(lib, ESHAPE, L.dllava_predict, *call(C.byref(q), 1, 128, 4, fake, big))       # d % 64
    q.d, q.n_blocks = 128, 5
    _expect(lib, EINVAL, L.dllava_predict, *call(C.byref(q), 1, 128, 4, fake, big))
    q.n_blocks = 1                                                                       # a block without matrices
    _expect(lib, ENULL, L.dllava_predict, *call(C.byref(q), 1, 128, 4, fake, big))
    # spans need all three arrays
    _expect(lib, ENULL, L.dllava_predict, fake, 128, 4, 1, fake, None, None, C.byref(p), 1, fake, fake, big, None)
    # workspace query: grows with the rows, image form needs more than the text form
    assert lib.dllava_predict_workspace(1000, 4, 2) > lib.dllava_predict_workspace(1000, 4, 0) > 0
    assert lib.dllava_predict_workspace(2000, 4, 2) > lib.dllava_predict_workspace(1000, 4, 2)
    assert lib.dllava_predict_workspace(1000, 4, 2) % 256 == 0
    # the layers
    _expect(lib, ESHAPE, L.dllava_linear, fake, 100, 4, 100, fake, None, 64, 0, None, fake, 64, 1, None)   # K % 64
    _expect(lib, ESHAPE, L.dllava_linear, fake, 128, 4, 128, fake, None, 60, 0, None, fake, 64, 1, None)   # N % 8
    _expect(lib, ESHAPE, L.dllava_linear, fake, 128, 4, 128, fake, None, 64, 0, None, fake, 56, 1, None)   # ldy < N
    _expect(lib, EINVAL, L.dllava_linear, fake, 128, 4, 128, fake, None, 64, 3, None, fake, 64, 1, None)   # act
    _expect(lib, ENULL, L.dllava_linear, fake, 128, 4, 128, fake, None, 64, 2, None, fake, 64, 1, None)    # gated form without a gate
    _expect(lib, ESHAPE, L.dllava_rms_norm, fake, 64, 4, 60, None, 1e-5, fake, 64, 1, None)                # d % 8
    _expect(lib, ESHAPE, L.dllava_rms_norm, fake, 64, 4, 16384, None, 1e-5, fake, 16384, 1, None)          # d too large
    _expect(lib, ESHAPE, L.dllava_rms_norm, fake, 56, 4, 64, None, 1e-5, fake, 64, 1, None)                # ldx < d
    _expect(lib, EINVAL, L.dllava_rms_norm, fake, 64, 4, 64, None, -1.0, fake, 64, 1, None)
    _expect(lib, EDTYPE, L.dllava_rms_norm, fake, 64, 4, 64, None, 1e-5, fake, 64, 0, None)
    _expect(lib, ENULL, L.dllava_rms_norm, None, 64, 4, 64, None, 1e-5, fake, 64, 1, None)
    _expect(lib, EDTYPE, L.dllava_linear, fake, 128, 4, 128, fake, None, 64, 0, None, fake, 64, 0, None)
    _expect(lib, ENULL, L.dllava_linear, fake, 128, 4, 128, None, None, 64, 0, None, fake, 64, 1, None)
    _expect(lib, EINVAL, L.dllava_linear, C.c_void_p(0x1008), 128, 4, 128, fake, None, 64, 0, None, fake, 64, 1, None)
    _expect(lib, ENULL, L.dllava_layer_norm, None, 4, None, None, fake, 1, None)
    _expect(lib, EDTYPE, L.dllava_layer_norm, fake, 4, None, None, fake, 0, None)
    _expect(lib, ESHAPE, L.dllava_span_attn, fake, fake, fake, 1, fake, 8, 8, 96, 0.1, fake, 1, None)
    _expect(lib, ENULL, L.dllava_span_attn, fake, fake, fake, 1, None, 8, 8, 64, 0.1, fake, 1, None)
    _expect(lib, EINVAL, L.dllava_span_attn, fake, fake, fake, 1, fake, 8, 8, 64, float("nan"), fake, 1, None)


def test_masked_attn_validates_on_the_host(lib):
    L = lib.lib()
    EINVAL, ENULL, ESHAPE, EDTYPE, EWORKSPACE = -1, -2, -3, -4, -6
    fake = C.c_void_p(0x1000)
    big = 1 << 20
    call = lambda Dh, scale, keep, dtype, ws, wsb: (fake, fake, fake, 2, fake, 64, 4, Dh, scale, keep, fake, dtype, ws, wsb, None)
    _expect(lib, EDTYPE, L.dllava_masked_attn, *call(64, 0.1, fake, 0, fake, big))
    _expect(lib, ESHAPE, L.dllava_masked_attn, *call(96, 0.1, fake, 1, fake, big))
    _expect(lib, EINVAL, L.dllava_masked_attn, *call(64, 0.0, fake, 1, fake, big))
    _expect(lib, ENULL, L.dllava_masked_attn, *call(64, 0.1, None, 1, fake, big))
    _expect(lib, EWORKSPACE, L.dllava_masked_attn, *call(64, 0.1, fake, 1, None, 0))
    _expect(lib, EWORKSPACE, L.dllava_masked_attn, *call(64, 0.1, fake, 1, fake, 8))
    assert lib.dllava_masked_attn_workspace(64, 2) % 256 == 0
    assert lib.dllava_masked_attn_workspace(1 << 20, 16) >= (1 << 20) // 32 * 4


def test_compact_validates_on_the_host(lib):
    L = lib.lib()
    EINVAL, ENULL, ESHAPE, EDTYPE = -1, -2, -3, -4
    fake = C.c_void_p(0x1000)
    cache = lib._KvCache(0x1000, 0x1000, 0x1000, 4, 2, 16, 2, 64, 1)
    call = lambda sumN, hid, hid_out, d, K, V, c, dtype, idx=fake: (2, fake, idx, fake, sumN, hid, hid_out, d, None, None, K, V,
                                                                    c, None, dtype, None)
    _expect(lib, EDTYPE, L.dllava_compact, *call(40, fake, fake, 64, None, None, None, 5))
    _expect(lib, ESHAPE, L.dllava_compact, *call(40, fake, fake, 36, None, None, None, 1))
    _expect(lib, ENULL, L.dllava_compact, *call(40, fake, None, 64, None, None, None, 1))        # hidden without hidden_out
    _expect(lib, ENULL, L.dllava_compact, *call(40, None, None, 0, fake, None, C.byref(cache), 1))  # K without V
    _expect(lib, ENULL, L.dllava_compact, *call(40, None, None, 0, fake, fake, None, 1))         # K/V without a cache
    _expect(lib, ENULL, L.dllava_compact, *call(40, fake, fake, 64, None, None, None, 1, idx=None))
    _expect(lib, EINVAL, L.dllava_compact, *call(-1, fake, fake, 64, None, None, None, 1))
    assert L.dllava_compact(*call(0, fake, fake, 64, None, None, None, 1)) == 0                  # nothing to move


def test_few_rows_linear_and_rope_validate_on_the_host(lib):
    L = lib.lib()
    EINVAL, ENULL, ESHAPE, EDTYPE, EWORKSPACE = -1, -2, -3, -4, -6
    fake = C.c_void_p(0x1000)
    big = 1 << 28
    call = lambda M, K, N, act, res, ws, wsb, dtype=1: (fake, K, M, K, fake, None, N, act, res, fake, N, dtype, ws, wsb, None)
    _expect(lib, ESHAPE, L.dllava_linear_few, *call(65, 128, 64, 0, None, fake, big))        # too many rows for this form
    _expect(lib, ESHAPE, L.dllava_linear_few, *call(4, 100, 64, 0, None, fake, big))
    _expect(lib, ESHAPE, L.dllava_linear_few, *call(4, 128, 40, 0, None, fake, big))         # N % 32
    _expect(lib, ENULL, L.dllava_linear_few, *call(4, 128, 64, 2, None, fake, big))
    _expect(lib, EWORKSPACE, L.dllava_linear_few, *call(4, 128, 64, 0, None, None, 0))
    _expect(lib, EWORKSPACE, L.dllava_linear_few, *call(4, 128, 64, 0, None, fake, 16))
    _expect(lib, EDTYPE, L.dllava_linear_few, *call(4, 128, 64, 0, None, fake, big, dtype=0))
    assert lib.dllava_linear_few_workspace(4096, 4096) % 256 == 0
    assert lib.dllava_linear_few_workspace(11008, 4096) >= 4096               # at least the counters
    assert lib.dllava_linear_few_workspace(256, 4096) >= 4096 + 2 * 64 * 256 * 4  # few feature groups: sums handed over
    _expect(lib, ESHAPE, L.dllava_rope, fake, fake, 4, 2, 63, 10000.0, 1, None)
    _expect(lib, EINVAL, L.dllava_rope, fake, fake, 4, 2, 64, 0.0, 1, None)
    _expect(lib, ENULL, L.dllava_rope, fake, None, 4, 2, 64, 10000.0, 1, None)
    _expect(lib, EDTYPE, L.dllava_rope, fake, fake, 4, 2, 64, 10000.0, 0, None)


def test_fused_decode_projections_validate_on_the_host(lib):
    L = lib.lib()
    EINVAL, ENULL, ESHAPE, EDTYPE, EWORKSPACE = -1, -2, -3, -4, -6
    fake = C.c_void_p(0x1000)
    big = 1 << 28
    qkv = lambda M=4, d=128, H=2, Dh=64, pos=fake, base=10000.0, dtype=1, ws=fake, wsb=big: (
        fake, d, M, d, fake, fake, fake, H, Dh, pos, base, fake, fake, fake, dtype, ws, wsb, None)
    _expect(lib, ESHAPE, L.dllava_qkv_few, *qkv(M=65))
    _expect(lib, ESHAPE, L.dllava_qkv_few, *qkv(d=100))
    _expect(lib, ESHAPE, L.dllava_qkv_few, *qkv(Dh=12))
    _expect(lib, ESHAPE, L.dllava_qkv_few, *qkv(Dh=48))
    _expect(lib, EINVAL, L.dllava_qkv_few, *qkv(base=0.0))
    _expect(lib, ENULL, L.dllava_qkv_few, *qkv(pos=None))
    _expect(lib, EDTYPE, L.dllava_qkv_few, *qkv(dtype=0))
    _expect(lib, EWORKSPACE, L.dllava_qkv_few, *qkv(ws=None, wsb=0))
    gated = lambda M=4, d=128, F=96, dtype=1, ws=fake, wsb=big: (fake, d, M, d, fake, fake, F, fake, F, dtype, ws, wsb, None)
    _expect(lib, ESHAPE, L.dllava_gated_few, *gated(F=40))
    _expect(lib, ESHAPE, L.dllava_gated_few, *gated(M=100))
    _expect(lib, EDTYPE, L.dllava_gated_few, *gated(dtype=0))
    _expect(lib, EWORKSPACE, L.dllava_gated_few, *gated(wsb=32))
    assert lib.dllava_decode_proj_workspace(3 * 4096, 4096) >= 4096 and lib.dllava_decode_proj_workspace(3 * 4096, 4096) % 256 == 0
    assert lib.dllava_decode_proj_workspace(96, 4096) >= 4096 + 2 * 64 * 96 * 4


def test_few_rows_workspaces_over_a_sweep_of_shapes(lib):
    """Counters first (4096 bytes), then at most 8 parts of 64 rows of float32 sums; 256-byte multiples; wide outputs,
    whose input width is not cut across blocks, need the counters only."""
    L = lib.lib()
    for K in (64, 512, 4096, 5120, 11008, 13824):
        for N in list(range(32, 1025, 32)) + [2048, 4096, 5120, 8192, 11008, 12288, 15360, 22016, 27648]:
            for q in (L.dllava_linear_few_workspace, L.dllava_decode_proj_workspace):
                b = q(N, K)
                assert b % 256 == 0 and 4096 <= b <= 4096 + 8 * 64 * N * 4 + 256, (N, K, b)
    assert L.dllava_linear_few_workspace(4096, 4096) == 4096        # 256 blocks of 16 features, 8 waves along K
    assert L.dllava_linear_few_workspace(5120, 13824) == 4096       # 160 blocks of 32 features, 8 waves along K
    assert L.dllava_decode_proj_workspace(3 * 4096, 4096) == 4096   # 384 blocks of 32 features
    assert L.dllava_decode_proj_workspace(2 * 11008, 4096) == 4096
    assert L.dllava_linear_few_workspace(0, 4096) == 4096 and L.dllava_decode_proj_workspace(64, 0) == 4096


def test_launch_forms_of_attention(tmp_path):
    """DLLAVA_LAUNCH_PREFILL_WAVES: the documented values are taken, every other one is as good as none."""
    import subprocess

    from paper_2412_00876_amd import build
    checks = []
    for v in list(range(80)) + [128, 1000, 1 << 20, (1 << 31) - 1]:
        waves, kernel = v % 16, v - v % 16
        ok = waves in (0, 1, 2, 4) and kernel in (0, 16, 32)
        checks.append(f"constexpr ForcedForm f{v} = forced_form({v}); static_assert(f{v}.waves == {waves if ok else 0} && "
                      f"f{v}.tiles == {int(ok and kernel == 16)} && f{v}.few == {int(ok and kernel == 32)}, \"{v}\");")
    src = tmp_path / "forms.cpp"
    src.write_text('#include "prefill_args.h"\nusing namespace dllava;\n' + "\n".join(checks) + "\n")
    r = subprocess.run([build.HIPCC, *build.COMMON, "--cuda-host-only", "-x", "hip", "-fsyntax-only", str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
