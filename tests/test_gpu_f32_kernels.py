"""The fp32 matrix-core kernels (GEMM tiles of 64 and of 32 rows, attention) at the edges of their tiles and of their
range, against float64 arithmetic; and the two GEMM kernels against each other, bit for bit."""
import numpy as np
import pytest

import otas_synth as synth
from tests import harness as hz

pytestmark = pytest.mark.gpu


def _context(lib, D, H, dtype):
    import torch
    cfg = synth.Config("f32", L=1, D=D, H=H, F=8, dtype=dtype, B=1, n0=2)
    return hz.make_context(cfg)[0], torch.float32 if dtype == "f32" else torch.bfloat16


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N,K", [(8, 8), (24, 40), (192, 768), (72, 1000), (2304, 136)])
def test_fp32_gemm_tile_edges_and_row_independence(lib, dtype, N, K):
    """Rows 0 .. m - 1 of a product must not depend on how many rows follow them: M = 1 .. 65 runs the small tiles,
    M = 12000 the large ones for every N here.  Error of the sum: at most K roundings of 2^-24 each on terms of total
    size sum |x w|, plus the rounding of the result (bf16: 2^-9 of it)."""
    import torch
    ctx, dt = _context(lib, 64, 1, dtype)
    g = torch.Generator(device="cuda").manual_seed(N + K)
    M = 12000
    x = torch.randn((M, K), generator=g, device="cuda").to(dt)
    w = torch.randn((N, K), generator=g, device="cuda").to(dt)
    b = torch.randn(N, generator=g, device="cuda").to(dt)
    res = torch.randn((M, N), generator=g, device="cuda")
    out = {}
    for m in (1, 31, 33, 64, 65, M):
        y = torch.full((m, N), float("nan"), device="cuda")
        ctx.otas_linear_kernel(1, x[:m].contiguous(), w, b, res[:m].contiguous(), m, N, K, 2, y)
        out[m] = y
    xd, wd = x.double(), w.double()
    ref = xd @ wd.T + b.double() + res.double()
    bound = (K + 8) * 2.0 ** -24 * (xd.abs() @ wd.abs().T + b.double().abs() + res.double().abs())
    assert bool(((out[M].double() - ref).abs() <= bound).all())
    for m in (1, 31, 33, 64, 65):
        assert torch.equal(out[m], out[M][:m]), m
    ctx.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D,H", [(8, 2), (24, 2), (64, 1), (200, 2), (256, 2)])
def test_fp32_attention_tile_edges(lib, dtype, D, H):
    """Head widths 4, 12, 64, 100 and 128 (the bf16 model takes this kernel where it has no other), sequences around the
    32-row and 32-key blocks and the four waves, with and without the size bias, in one ragged batch each."""
    import torch
    ctx, dt = _context(lib, D, H, dtype)
    dh = D // H
    if dtype == "bf16" and dh in (64, 80, 96, 128):
        pytest.skip("the bf16 kernel takes this width")
    ns = [1, 31, 32, 33, 128, 129, 300]
    off = np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)
    T = int(off[-1])
    g = torch.Generator(device="cuda").manual_seed(D)
    qkv = torch.randn((T, 3 * D), generator=g, device="cuda").to(dt)
    sizes = torch.randint(1, 9, (T,), generator=g, device="cuda", dtype=torch.int32)
    for flags in (0, lib.OTAS_FLAG_SIZE_BIAS):
        o = torch.full((T, D), float("nan"), device="cuda", dtype=dt)
        ctx.otas_attention(qkv, sizes, off, flags, o)
        for q, n in enumerate(ns):
            r = slice(int(off[q]), int(off[q + 1]))
            x = qkv[r].double().cpu()
            Q, Kk, V = (x[:, i * D:(i + 1) * D].reshape(n, H, dh).transpose(0, 1) for i in range(3))
            s = Q @ Kk.transpose(1, 2) / dh ** 0.5
            if flags:
                s = s + sizes[r].double().cpu().log()
            ref = (torch.softmax(s, -1) @ V).transpose(0, 1).reshape(n, D).numpy()
            got = o[r].double().cpu().numpy()
            # logits of size <= 30 in fp32: 30 * 2^-23 of the weights; a bf16 result adds its own rounding
            assert np.abs(got - ref).max() <= (2e-5 if dtype == "f32" else 2.0 ** -8) * np.abs(ref).max(), (flags, n)
    ctx.close()


@pytest.mark.parametrize("H", [1, 4])
def test_fp32_attention_keys_without_weight_and_infinite_values(lib, H):
    """A row's whole key block may have no weight: sizes 0 under the size bias, or logits that overflow to -inf.  Such keys
    get weight 0, wherever they lie among the blocks and the waves.  An infinite value reaches the rows that weigh it
    and its own column only, also as the last key of a sequence that ends inside a block."""
    import torch
    D, n = 128, 170
    dh = D // H
    ctx, _ = _context(lib, D, H, "f32")
    g = torch.Generator(device="cuda").manual_seed(H)
    qkv = torch.randn((n, 3 * D), generator=g, device="cuda")
    one = torch.ones(n, dtype=torch.int32, device="cuda")

    def check(x, sizes, flags):
        o = torch.full((n, D), float("nan"), device="cuda")
        ctx.otas_attention(x, sizes, np.array([0, n], dtype=np.int32), flags, o)
        x = x.cpu()
        Q, Kk, V = (x[:, i * D:(i + 1) * D].reshape(n, H, dh).transpose(0, 1) for i in range(3))
        s = (Q @ Kk.transpose(1, 2)).double() / dh ** 0.5      # products in 32 bits: the overflow is the point
        if flags:
            s = s + sizes.cpu().double().log()
        ref = (torch.softmax(s, -1) @ V.double()).transpose(0, 1).reshape(n, D)
        got = o.cpu().double()
        assert torch.equal(torch.isinf(got), torch.isinf(ref)) and not bool(torch.isnan(got).any())
        fin = ~torch.isinf(ref)
        assert float((got - ref)[fin].abs().max()) <= 2e-5 * float(ref[fin].abs().max())     # as in the test above

    for lo, hi in [(0, 32), (32, 64), (0, 160), (128, 170), (5, 170)]:
        sizes = one.clone()
        sizes[lo:hi] = 0
        check(qkv, sizes, lib.OTAS_FLAG_SIZE_BIAS)
        x = qkv.clone()
        x[:, :D:dh] = 1e25                       # first column of every head's queries ...
        x[lo:hi, D:2 * D:dh] = -1e25             # ... times the keys': -1e50
        x[:lo, D:2 * D:dh] = 0
        x[hi:, D:2 * D:dh] = 0
        check(x, one, 0)
    x = qkv.clone()
    x[n - 1, 2 * D + 3] = float("inf")
    check(x, one, 0)
    ctx.close()


@pytest.mark.parametrize("N,K", [(8, 8), (8, 128), (72, 128), (136, 256), (200, 384), (768, 640), (64, 3072)])
def test_fp32_gemm_large_tiles_every_epilogue(lib, N, K):
    """M just past what the small tiles take (512 tiles of 32 x 32, 600 where K is no multiple of 128): one to 24 k-tiles a quarter, a ragged last
    tile in both directions, no epilogue / GELU / residual, against float64 and, bit for bit, the small tiles' rows."""
    import torch
    ctx, dt = _context(lib, 64, 1, "f32")
    g = torch.Generator(device="cuda").manual_seed(N + K)
    M = 32 * ((600 if K % 128 else 512) // ((N + 31) // 32) + 1) + 7
    x, w = torch.randn((M, K), generator=g, device="cuda"), torch.randn((N, K), generator=g, device="cuda")
    b, res = torch.randn(N, generator=g, device="cuda"), torch.randn((M, N), generator=g, device="cuda")
    xd, wd = x.double(), w.double()
    lin = xd @ wd.T + b.double()
    # at most K roundings of 2^-24 on terms of total size sum |x w|; GELU's slope is below 1.13 and its own error a few units
    size = xd.abs() @ wd.abs().T + b.double().abs()
    for epi, ref, bound in ((0, lin, (K + 8) * 2.0 ** -24 * size),
                            (1, torch.nn.functional.gelu(lin), 1.13 * (K + 16) * 2.0 ** -24 * size),
                            (2, lin + res.double(), (K + 8) * 2.0 ** -24 * (size + res.double().abs()))):
        out = {}
        for m in (33, M):
            out[m] = torch.full((m, N), float("nan"), device="cuda")
            ctx.otas_linear_kernel(1, x[:m].contiguous(), w, b, res[:m].contiguous() if epi == 2 else None, m, N, K, epi, out[m])
        assert bool(((out[M].double() - ref).abs() <= bound).all()), epi
        assert torch.equal(out[33], out[M][:33]), epi
    ctx.close()


@pytest.mark.parametrize("which", ["x", "w"])
def test_fp32_gemm_operands_that_do_not_begin_on_16_bytes(lib, which):
    """A view four bytes into a buffer takes the kernel that stages through registers: the same rows bit for bit."""
    import torch
    ctx, dt = _context(lib, 64, 1, "f32")
    M, N, K = 2500, 256, 256                     # 632 tiles of 32 x 32: past the small ones with either kernel
    g = torch.Generator(device="cuda").manual_seed(9)
    x, w = torch.randn((M, K), generator=g, device="cuda"), torch.randn((N, K), generator=g, device="cuda")
    b = torch.randn(N, generator=g, device="cuda")
    shift = lambda t: torch.cat([t.new_zeros(1), t.flatten()])[1:].view(t.shape)
    want, got = torch.empty((M, N), device="cuda"), torch.full((M, N), float("nan"), device="cuda")
    ctx.otas_linear_kernel(1, x, w, b, None, M, N, K, 0, want)
    xs, ws = (shift(x), w) if which == "x" else (x, shift(w))
    assert (xs.data_ptr() | ws.data_ptr()) & 15 == 4
    ctx.otas_linear_kernel(1, xs, ws, b, None, M, N, K, 0, got)
    assert torch.equal(want, got)
    ctx.close()
