"""The few-rows layers at the edges of their line ring and row groups: input widths of 1 to 19 lines of 64 elements (waves with no
line, with fewer than the ring holds, with remainders), 1 to 64 rows, and weights past the size from which they are read past the caches."""
import pytest
import torch

import paper_2412_00876_amd as P

pytestmark = pytest.mark.gpu


def _close(y, ref, K):
    """One rounding to bfloat16 (8 significant bits: half a step is at most 2^-8 of the value) of a float32 sum of K products of
    bfloat16 numbers (exact in float32; the sum's own error at most K steps of 2^-24 of its terms, which are below 4 together)."""
    y, ref = y.double(), ref.double()
    assert ((y - ref).abs() <= 2.0 ** -8 * 1.01 * ref.abs() + K * 2.0 ** -24 * 4).all(), float((y - ref).abs().max())


def _inputs(seed, M, K, N):
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
    W = (torch.randn((N, K), generator=g, device="cuda") / K ** 0.5).to(torch.bfloat16)
    return x, W, x.double() @ W.double().T


@pytest.mark.parametrize("M", [1, 7, 8, 9, 16, 17, 25, 32, 33, 64])
@pytest.mark.parametrize("lines", [1, 3, 4, 5, 8, 9, 16, 17, 19])
def test_linear_few_rings(M, lines):
    for N in (32, 4096, 5120):          # 16 features and 8 waves per block, 32 and 4, 32 and 8
        K = 64 * lines
        x, W, ref = _inputs(M + lines, M, K, N)
        y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        ws = torch.zeros(P.dllava_linear_few_workspace(N, K), dtype=torch.uint8, device="cuda")
        P.dllava_linear_few(x, K, M, K, W, None, N, 0, None, y, N, P.BF16, ws)
        _close(y, ref, K)


@pytest.mark.parametrize("M", [1, 8, 9, 17, 33, 64])
def test_weights_past_the_caches(M):
    """64 MiB of weights and more, and the same rows on a part of them that is below that: the same bits."""
    N, K = 8256, 4096
    x, W, ref = _inputs(M, M, K, N)
    ws = torch.zeros(max(P.dllava_linear_few_workspace(N, K), P.dllava_linear_few_workspace(8160, K)), dtype=torch.uint8, device="cuda")
    y, part = (torch.full((M, n), float("nan"), dtype=torch.bfloat16, device="cuda") for n in (N, 8160))
    P.dllava_linear_few(x, K, M, K, W, None, N, 0, None, y, N, P.BF16, ws)
    P.dllava_linear_few(x, K, M, K, W, None, 8160, 0, None, part, 8160, P.BF16, ws)
    _close(y, ref, K)
    assert torch.equal(y[:, :8160].contiguous().view(torch.int16), part.view(torch.int16))


@pytest.mark.parametrize("M", [1, 9, 33])
@pytest.mark.parametrize("d,H", [(256, 4), (4160, 65)])
def test_qkv_and_gated_rings(M, d, H):
    """d = 4160: 99 MiB of q|k|v and an odd number of lines."""
    Dh, F = 64, 8192 if d > 256 else 96
    g = torch.Generator(device="cuda").manual_seed(M)
    x = torch.randn((M, d), generator=g, device="cuda").to(torch.bfloat16)
    mk = lambda n: (torch.randn((n, d), generator=g, device="cuda") / d ** 0.5).to(torch.bfloat16)  # noqa: E731
    Wq, Wk, Wv, Wg, Wu = mk(H * Dh), mk(H * Dh), mk(H * Dh), mk(F), mk(F)
    ws = torch.zeros(max(P.dllava_decode_proj_workspace(3 * H * Dh, d), P.dllava_decode_proj_workspace(2 * F, d)), dtype=torch.uint8, device="cuda")
    q, k, v = (torch.zeros((M, H, Dh), dtype=torch.bfloat16, device="cuda") for _ in range(3))
    pos = torch.zeros(M, dtype=torch.int32, device="cuda")          # position 0: no rotation
    P.dllava_qkv_few(x, d, M, d, Wq, Wk, Wv, H, Dh, pos, 1e4, q, k, v, P.BF16, ws)
    for out, Wm in ((q, Wq), (k, Wk), (v, Wv)):
        _close(out.reshape(M, -1), x.double() @ Wm.double().T, d)
    y = torch.zeros((M, F), dtype=torch.bfloat16, device="cuda")
    P.dllava_gated_few(x, d, M, d, Wg, Wu, F, y, F, P.BF16, ws)
    gate = (x.double() @ Wg.double().T).to(torch.bfloat16).double()
    up = x.double() @ Wu.double().T
    # the gate is rounded as if stored: a value next to a rounding boundary may go to its other side
    tol = (up.abs() * 1.2 * 2.0 ** -8 * gate.abs() + 2.0 ** -8 * (up * gate).abs() + 1e-4)
    assert ((y.double() - up * gate * torch.sigmoid(gate)).abs() <= tol).all()
