"""Batches whose QKV projection and hidden rows share one workspace buffer: a query's rows are those of the query alone,
for which the two lie apart."""
import ctypes

import numpy as np
import pytest

import otas_synth as synth
from tests import harness as hz

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,D,H,F,n,B", [
    ("bf16", 128, 1, 512, 400, 48),    # F > 3 D; metric rows in the workspace (more than 293 tokens at metric width 128)
    ("bf16", 256, 2, 384, 300, 49),    # F < 3 D: the rows left beside the shared buffer are the hidden rows' number
    ("f32", 128, 2, 512, 70, 141),     # 9870 rows, just past the line (32 MB) in f32
])
def test_shared_activation_buffer_changes_nothing(lib, dtype, D, H, F, n, B):
    """Rows do not depend on the batch in these shapes (no split over K), so bit for bit; lanes own rows of every buffer."""
    import torch
    cfg = synth.Config("shared", L=3, D=D, H=H, F=F, dtype=dtype, B=1, n0=n, strategies=[(0, 12)], seed=31)
    ctx, _ = hz.make_context(cfg)
    assert B * n * (3 * D + F) * (4 if dtype == "f32" else 2) > 32 << 20
    g = torch.Generator().manual_seed(5)
    x0 = torch.randn((B * n, D), generator=g).to("cuda").to(ctx.torch_dtype)
    off = np.arange(B + 1, dtype=np.int32) * n
    R = [n // 3 + q % 3 for q in range(B)]     # the later blocks are below the line
    alone = {q: hz.gpu_forward(ctx, x0[q * n:(q + 1) * n].contiguous(), [0, n], [R[q]]) for q in (0, 1, B // 2, B - 1)}
    for lanes in (1, 3):
        ctx.otas_set_lanes(lanes)
        got = hz.gpu_forward(ctx, x0, off, R)
        for q, ref in alone.items():
            assert np.array_equal(got["x"][q], ref["x"][0]) and np.array_equal(got["sizes"][q], ref["sizes"][0]), (lanes, q)
            for a, b in zip(got["trace"][q], ref["trace"][0]):
                assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    ctx.close()


@pytest.mark.parametrize("path", ["merge", "lanes", "grow"])
@pytest.mark.parametrize("dtype,D,H,F,n", [("bf16", 128, 1, 512, 400), ("bf16", 256, 2, 384, 300), ("f32", 128, 2, 512, 70)])
def test_a_pass_stays_inside_the_bytes_it_asks_for(lib, dtype, D, H, F, n, path):
    """Workspaces of exactly the reported size between guard bytes, for batches whose blocks are below, around and above the line
    at which projection and hidden rows share a buffer, F on both sides of 3 D, metric rows in the spare part of it: no
    guard byte changes."""
    import torch
    cfg = synth.Config("guard", L=3, D=D, H=H, F=F, dtype=dtype, B=1, n0=n, seed=31)
    ctx, _ = hz.make_context(cfg)
    ctx.otas_set_lanes(3 if path == "lanes" else 1)
    rows = (32 << 20) // ((3 * D + F) * (4 if dtype == "f32" else 2))        # of a block at the line
    guard = 1 << 16
    for B in (3, rows // n, rows // n + 1, 2 * rows // n):
        P = 2 if path == "grow" else 0
        off = np.arange(B + 1, dtype=np.int32) * (n + P)
        T = B * (n + 3 * P)                                       # two layers insert P rows each
        x0 = torch.randn((B * (n + P), D), generator=torch.Generator().manual_seed(B)).to("cuda").to(ctx.torch_dtype)
        buf = torch.full((ctx.otas_workspace_bytes(B, T) + 2 * guard,), 0xA5, dtype=torch.uint8, device="cuda")
        ws = buf[guard:-guard]
        r, left = n // 3, n + 3 * P
        for _ in range(0 if P else 3):                            # a third of the tokens a layer while the length allows
            left -= min(r, (left - 1) // 2)
        x_out = torch.empty((B * left, D), device="cuda")
        sizes = torch.empty(B * left, dtype=torch.int32, device="cuda")
        if path == "grow":
            prompts = torch.randn((3, B * P, D), generator=torch.Generator().manual_seed(1)).to("cuda").to(ctx.torch_dtype)
            ctx.otas_encoder_forward_deep(x0, off, lib.OTAS_PROMPT_GROW, prompts, np.arange(B + 1, dtype=np.int32) * P, ws,
                                          x_out, sizes)
        else:
            ctx.otas_encoder_forward(x0, off, [r] * B, 0, ws, x_out, sizes)
        assert bool(torch.isfinite(x_out).all()) and bool((sizes >= 1).all())
        assert bool((buf[:guard] == 0xA5).all()) and bool((buf[-guard:] == 0xA5).all()), B
    ctx.close()


@pytest.mark.parametrize("D,F", [(72, 136), (64, 8)])
def test_weights_read_ahead_change_nothing(lib, D, F):
    """Up to 4096 rows merge-apply's launch also reads FC1's weight (here of 153 and 8 cache lines): the rows are those of a
    batch that is above the line after every merge."""
    import torch
    n, r, B, L = 30, 5, 220, 2
    assert B * (n - L * r) > 4096 > n
    cfg = synth.Config("warm", L=L, D=D, H=1, F=F, dtype="bf16", B=1, n0=n, seed=5)
    ctx, _ = hz.make_context(cfg)
    x0 = torch.randn((B * n, D), generator=torch.Generator().manual_seed(2)).to("cuda").to(ctx.torch_dtype)
    many = hz.gpu_forward(ctx, x0, np.arange(B + 1, dtype=np.int32) * n, [r] * B)
    for q in (0, B - 1):
        one = hz.gpu_forward(ctx, x0[q * n:(q + 1) * n].contiguous(), [0, n], [r])
        assert np.array_equal(one["x"][0], many["x"][q]) and np.array_equal(one["sizes"][0], many["sizes"][q])
    ctx.close()


class WarmWeight(ctypes.Structure):
    _fields_ = [("w", ctypes.c_void_p), ("bytes", ctypes.c_int64), ("wgs", ctypes.c_int)]


@pytest.mark.parametrize("wgs,lines", [(64, 8), (64, 153), (64, 64 * 256 + 1), (128, 100 * 1024)])
@pytest.mark.parametrize("M,D", [(1, 64), (30, 72), (197, 768), (5, 1280)])
def test_launches_with_and_without_read_ahead(lib, M, D, wgs, lines):
    """Merge-apply and both forms of the split-K reduce, each with and without the workgroups that read a weight: fewer lines
    than workgroups, a line past whole rounds of them, a weight of more than 8 MB; the same bits, the weight as it was."""
    import paper_2401_05031_amd as otas
    import torch
    so = ctypes.CDLL(otas.lib_path())
    g = torch.Generator(device="cuda").manual_seed(M + D + lines)
    rand = lambda *shape: torch.randn(shape, generator=g, device="cuda")
    w = torch.randint(-99, 99, (lines * 32,), generator=g, device="cuda", dtype=torch.int32)
    x, part, S = rand(2 * M, D), rand(3, M, D), 3
    gamma, beta, bias = (rand(D).to(torch.bfloat16) for _ in range(3))
    src = torch.arange(2 * M, device="cuda", dtype=torch.int32)       # row j: the average of rows 2 j and 2 j + 1
    ptr = torch.arange(M, device="cuda", dtype=torch.int32) * 2
    p = lambda t: ctypes.c_void_p(t.data_ptr() if t is not None else None)
    stream, kept = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), w.clone()

    def launches(warm):
        xo, y = torch.full((3, M, D), float("nan"), device="cuda"), torch.zeros((2, M, D), device="cuda", dtype=torch.bfloat16)
        sizes = torch.zeros(M, device="cuda", dtype=torch.int32)
        assert so._ZN4otas21launch_merge_apply_lnEiPKfPKiS3_S3_lliPfPiPKvS7_PvfP12ihipStream_tRKNS_10WarmWeightE(
            1, p(x), p(None), p(src), p(ptr), ctypes.c_int64(2 * M), ctypes.c_int64(M), D, p(xo[0]), p(sizes), p(gamma),
            p(beta), p(y[0]), ctypes.c_float(1e-6), stream, ctypes.byref(warm)) == 0
        for i, (ga, be, out) in enumerate([(gamma, beta, y[1]), (None, None, None)]):
            assert so._ZN4otas23launch_splitk_reduce_lnEPKfiPKvS1_PfliS3_S3_PvfP12ihipStream_tRKNS_10WarmWeightE(
                p(part), S, p(bias), p(x), p(xo[1 + i]), ctypes.c_int64(M), D, p(ga), p(be), p(out), ctypes.c_float(1e-6),
                stream, ctypes.byref(warm)) == 0
        return xo, y, sizes

    plain, warm = launches(WarmWeight(None, 0, 0)), launches(WarmWeight(w.data_ptr(), lines * 128, wgs))
    assert all(torch.equal(a, b) for a, b in zip(plain, warm)) and torch.equal(w, kept)
    assert torch.equal(plain[0][1], plain[0][2]) and bool((plain[2] == 2).all())
