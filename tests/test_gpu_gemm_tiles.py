"""The 256-column GEMM kernels at every tile height, at the edges of their tiles, loops and output rules."""
import numpy as np
import pytest

import otas_synth as synth
from tests import harness as hz

pytestmark = pytest.mark.gpu
ROWS = {4: 192, 5: 256, 6: 320, 8: 160, 9: 224, 10: 288}


def _context():
    cfg = synth.config("vitb_plain")
    cfg.L = 1
    return hz.make_context(cfg)[0]


@pytest.mark.parametrize("K", [128, 192, 256, 448])
@pytest.mark.parametrize("kernel", sorted(ROWS))
def test_tile_heights_at_their_edges(lib, kernel, K):
    """Two to seven k-tiles; one row short of, at and past one and two tiles, one of them inside a wave's last 16 rows; ragged
    columns; all epilogues.  Against float64 (K + 8 roundings of 2^-24 on the terms' absolute sum, GELU's slope below 1.13,
    the rounding of a bf16 output), and bit for bit against the 128 x 128 kernel: K is walked in the same order."""
    import torch
    ctx, bm = _context(), ROWS[kernel]
    g = torch.Generator(device="cuda").manual_seed(K + kernel)
    for M, N in [(1, 8), (bm - 1, 264), (bm, 256), (bm + 1, 200), (2 * bm + bm // 2 + 5, 520)]:
        x, w, b = (torch.randn(s, generator=g, device="cuda").to(torch.bfloat16) for s in ((M, K), (N, K), (N,)))
        res = torch.randn((M, N), generator=g, device="cuda")
        xd, wd, bd = x.double(), w.double(), b.double()
        lin, mag = xd @ wd.T + bd, xd.abs() @ wd.abs().T + bd.abs()
        for epi in (0, 1, 2):
            out = {}
            for k in (kernel, 3):
                out[k] = torch.full((M, N), float("nan"), dtype=torch.float32 if epi == 2 else torch.bfloat16, device="cuda")
                ctx.otas_linear_kernel(k, x, w, b, res if epi == 2 else None, M, N, K, epi, out[k])
            want = torch.nn.functional.gelu(lin) if epi == 1 else lin + res.double() if epi == 2 else lin
            bound = (K + 8) * 2.0 ** -24 * 1.13 * (mag + (res.double().abs() if epi == 2 else 0))
            if epi != 2:
                bound = bound + 2.0 ** -8 * want.abs() + 1e-7
            assert bool(((out[kernel].double() - want).abs() <= bound).all()), (M, N, epi)
            assert torch.equal(out[kernel], out[3]), (M, N, epi)
    ctx.close()


MB = 1 << 20


@pytest.mark.parametrize("epi,N,line", [(0, 1024, 160 * MB), (1, 2048, 160 * MB)])
@pytest.mark.parametrize("kernel", sorted(ROWS))
def test_outputs_on_both_sides_of_the_streaming_rule(lib, kernel, epi, N, line):
    """Outputs of just the bytes at which the rule changes, one row fewer and one more: stored past the L2's replacement or
    not, the same rows as the 128 x 128 kernel's."""
    import torch
    ctx, K, most = _context(), 128, line // (2 * N) + 1
    g = torch.Generator(device="cuda").manual_seed(N)
    x, w, b = (torch.randn(s, generator=g, device="cuda").to(torch.bfloat16) for s in ((most, K), (N, K), (N,)))
    want = torch.empty((most, N), dtype=torch.bfloat16, device="cuda")
    ctx.otas_linear_kernel(3, x, w, b, None, most, N, K, epi, want)
    for M in (most - 2, most - 1, most):
        out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        ctx.otas_linear_kernel(kernel, x, w, b, None, M, N, K, epi, out)
        assert torch.equal(out, want[:M]), M
    ctx.close()


def test_a_large_models_hidden_rows_past_the_caches(lib):
    """A model of more than 128 MB of weights and one of fewer layers, the same weights layer by layer: the hidden rows of 16 to
    64 MB are stored past the L2's replacement in the first only.  After its one layer the small model's rows are the large
    one's after its first, on both sides of both lines."""
    import torch
    D, F, n = 768, 3072, 128
    cfg = synth.Config("stream", L=1, D=D, H=12, F=F, dtype="bf16", B=1, n0=n, seed=3)
    one, layers = hz.make_context(cfg)
    many = lib.Context.from_host_weights(10, D, 12, F, lib.OTAS_BF16, cfg.ln_eps, cfg.n_lead, layers * 10)
    for B in (21, 22, 85, 86):                      # 15.75, 16.5, 63.75 and 64.5 MB
        assert (2 * B * n * F > 16 * MB) == (B >= 22) and (2 * B * n * F > 64 * MB) == (B == 86)
        x0 = torch.randn((B * n, D), generator=torch.Generator().manual_seed(B)).to("cuda")
        off = np.arange(B + 1, dtype=np.int32) * n
        a = hz.gpu_forward(one, x0, off, [0] * B, trace=False, layer_range=(0, 1))
        b = hz.gpu_forward(many, x0, off, [0] * B, trace=False, layer_range=(0, 1))
        assert all(np.array_equal(p, q) for p, q in zip(a["x"], b["x"])), B
    one.close()
    many.close()


@pytest.mark.parametrize("epi", [0, 1, 2])
@pytest.mark.parametrize("K", [64, 96, 128, 192, 256, 320, 384])
def test_small_tiles_whose_last_stage_the_epilogue_takes(lib, K, epi):
    """64 x 64 tiles, several per CU: the ring's last k-tile lies in each of its four stages, all but the last of which become
    the epilogue's staging area while other waves may still read.  Twenty launches, each bit for bit the kernel's that
    walks K in steps of 32 and has no tile smaller than 128 x 128."""
    import torch
    ctx, M, N = _context(), 12549, 136
    g = torch.Generator(device="cuda").manual_seed(K)
    x, w, b = (torch.randn(s, generator=g, device="cuda").to(torch.bfloat16) for s in ((M, K), (N, K), (N,)))
    res = torch.randn((M, N), generator=g, device="cuda") if epi == 2 else None
    want = torch.full((M, N), float("nan"), dtype=torch.float32 if epi == 2 else torch.bfloat16, device="cuda")
    ctx.otas_linear_kernel(2, x, w, b, res, M, N, K, epi, want)
    got = torch.empty_like(want)
    for _ in range(20):
        got.fill_(float("nan"))
        ctx.otas_linear_kernel(7, x, w, b, res, M, N, K, epi, got)
        assert torch.equal(got, want)
    ctx.close()


def _against_float64(out, x, w, b, res, epi):
    """K + 8 roundings of 2^-24 on the terms' absolute sum, GELU's slope below 1.13, the rounding of a bf16 output."""
    import torch
    xd, wd, bd, K = x.double(), w.double(), b.double(), x.shape[1]
    lin, mag = xd @ wd.T + bd, xd.abs() @ wd.abs().T + bd.abs()
    want = torch.nn.functional.gelu(lin) if epi == 1 else lin + res.double() if epi == 2 else lin
    bound = (K + 8) * 2.0 ** -24 * 1.13 * (mag + (res.double().abs() if epi == 2 else 0))
    if epi != 2:
        bound = bound + 2.0 ** -8 * want.abs() + 1e-7
    return bool(((out.double() - want).abs() <= bound).all())


# tile of kernel 7 -> shapes that are run in it, whole tiles and ragged ones; K of five to twelve k-tiles and of 48
SMALL = {1: [(1, 8, 320), (32, 32, 384), (197, 200, 448), (65, 1000, 768), (33, 40, 3072)],
         2: [(197, 2304, 768), (220, 2048, 640), (190, 2056, 576)],
         0: [(64, 64, 128), (250, 2304, 768), (700, 1000, 64), (130, 72, 192)],
         3: [(576, 2304, 768), (481, 2304, 384), (500, 2360, 320)]}


@pytest.mark.parametrize("epi", [0, 1, 2])
@pytest.mark.parametrize("tile", sorted(SMALL))
def test_tiles_of_the_small_kernel(lib, tile, epi):
    """Kernel 7 in each of its tiles (which one a shape takes is asked of the library) against float64, and bit for bit against the
    K-step-32 kernel, which walks K in the same order in tiles of 128 x 128."""
    import ctypes
    import torch
    pick = ctypes.CDLL(lib.lib_path())._ZN4otas15pick_small_tileEliii
    pick.argtypes, pick.restype = [ctypes.c_int64] + [ctypes.c_int] * 3, ctypes.c_int
    ctx = _context()
    g = torch.Generator(device="cuda").manual_seed(10 * tile + epi)
    for M, N, K in SMALL[tile]:
        assert pick(M, N, K, 1) == tile, (M, N, K)
        x, w, b = (torch.randn(s, generator=g, device="cuda").to(torch.bfloat16) for s in ((M, K), (N, K), (N,)))
        res = torch.randn((M, N), generator=g, device="cuda") if epi == 2 else None
        out = {}
        for k in (7, 2):
            out[k] = torch.full((M, N), float("nan"), dtype=torch.float32 if epi == 2 else torch.bfloat16, device="cuda")
            ctx.otas_linear_kernel(k, x, w, b, res, M, N, K, epi, out[k])
        assert _against_float64(out[7], x, w, b, res, epi), (M, N, K)
        assert torch.equal(out[7], out[2]), (M, N, K)
    ctx.close()


@pytest.mark.parametrize("epi", [0, 1, 2])
@pytest.mark.parametrize("M,N,K,rows", [(1920, 2304, 128, 160), (1921, 2176, 192, 160), (2079, 2304, 256, 160), (1406, 3072, 768, 160),
                                        (3599, 2296, 320, 160), (1281, 2304, 192, 128), (159, 136, 128, 128), (1920, 2304, 832, 128)])
def test_tiles_of_128_and_160_rows(lib, M, N, K, rows, epi):
    """Kernel 3 where the fullest CU has a tile fewer with 160 rows and where it has not; the last tile of one row, one row short
    and whole; two k-tiles to twelve."""
    import ctypes
    import torch
    wide = ctypes.CDLL(lib.lib_path())._ZN4otas9wide_rowsEliii
    wide.argtypes, wide.restype = [ctypes.c_int64] + [ctypes.c_int] * 3, ctypes.c_int
    assert wide(M, N, K, 1) == rows
    ctx = _context()
    g = torch.Generator(device="cuda").manual_seed(M)
    x, w, b = (torch.randn(s, generator=g, device="cuda").to(torch.bfloat16) for s in ((M, K), (N, K), (N,)))
    res = torch.randn((M, N), generator=g, device="cuda") if epi == 2 else None
    out = {}
    for k in (3, 2):
        out[k] = torch.full((M, N), float("nan"), dtype=torch.float32 if epi == 2 else torch.bfloat16, device="cuda")
        ctx.otas_linear_kernel(k, x, w, b, res, M, N, K, epi, out[k])
    assert _against_float64(out[3], x, w, b, res, epi)
    assert torch.equal(out[3], out[2])
    ctx.close()


@pytest.mark.parametrize("M,N,K,S", [(21, 768, 3072, 8), (32, 768, 3072, 8), (100, 768, 3072, 8), (165, 768, 3072, 8),
                                     (400, 768, 3072, 8), (950, 768, 3072, 6), (1406, 768, 3072, 4), (2000, 768, 3072, 4)])
def test_partial_products_in_every_tile(lib, M, N, K, S):
    """The partial products of a split, whichever tile they run in, are the products of the pieces of K bit for bit."""
    import ctypes
    import torch
    split = ctypes.CDLL(lib.lib_path())._ZN4otas20launch_linear_splitkEPKvS1_PfliiiP12ihipStream_t
    vp = ctypes.c_void_p
    split.argtypes, split.restype = [vp, vp, vp, ctypes.c_int64] + [ctypes.c_int] * 3 + [vp], ctypes.c_int
    ctx = _context()
    g = torch.Generator(device="cuda").manual_seed(M)
    x, w = (torch.randn(s, generator=g, device="cuda").to(torch.bfloat16) for s in ((M, K), (N, K)))
    part = torch.full((S, M, N), float("nan"), device="cuda")
    torch.cuda.synchronize()
    assert split(x.data_ptr(), w.data_ptr(), part.data_ptr(), M, N, K, S, torch.cuda.current_stream().cuda_stream) == 0
    zero, none = torch.zeros((M, N), device="cuda"), torch.zeros(N, dtype=torch.bfloat16, device="cuda")
    for i, (xs, ws) in enumerate(zip(x.chunk(S, 1), w.chunk(S, 1))):
        want = torch.full((M, N), float("nan"), device="cuda")
        ctx.otas_linear_kernel(2, xs.contiguous(), ws.contiguous(), none, zero, M, N, K // S, 2, want)
        assert torch.equal(part[i], want), i
    ctx.close()
