"""bf16 attention in every way the library cuts up its work: row blocks whose keys several waves share, staged pieces, waves per row
block, row blocks of a head on one XCD."""
import ctypes

import numpy as np
import pytest

import otas_synth as synth
from tests import harness as hz

pytestmark = pytest.mark.gpu


class Shape(ctypes.Structure):
    _fields_ = [("kc", ctypes.c_int), ("nw", ctypes.c_int), ("kg", ctypes.c_int), ("by_head", ctypes.c_bool)]


def _shape(lib, dh, H, ns, others=0):
    f = ctypes.CDLL(lib.lib_path())._ZN4otas15attention_shapeEiiiiii
    f.argtypes, f.restype = [ctypes.c_int] * 6, Shape
    s = f(dh, H, len(ns), max(ns), sum(-(-n // 128) for n in ns if 2 * n > max(ns)), others)
    return s.kc, s.nw, s.kg, s.by_head


# (keys staged at a time, waves, waves that share a row block, a head's row blocks on one XCD) -> (head width, heads, lengths).  Lengths at
# and beside the edges of key blocks (32), row blocks (32, 64, 128, 256) and staged pieces (128, 256).
CASES = {
    (128, 4, 4, False): [(64, 4, [65]), (64, 2, [128, 1, 33, 32, 97]), (80, 4, [97, 31, 128, 129]), (80, 2, [197])],
    (128, 4, 4, True): [(80, 2, [577, 160, 1])],
    (256, 4, 4, False): [(64, 4, [197, 1, 33, 32, 129]), (64, 2, [700]), (64, 4, [256, 31, 64, 65])],
    (256, 4, 4, True): [(64, 4, [700, 2]), (64, 2, [513, 1, 257, 256]), (64, 3, [300, 270, 301])],
    (256, 8, 4, False): [(64, 12, [197, 65, 64, 1, 129]), (64, 4, [161, 160, 129, 128, 2, 97, 63, 130, 191, 150, 1, 140, 256, 31])],
    (256, 8, 4, True): [(64, 12, [257, 1, 129, 65]), (64, 12, [400, 193, 2])],
    (256, 8, 1, False): [(64, 12, [197, 193, 256, 1, 225, 32, 33, 100, 129, 160, 161]), (64, 12, [160, 129, 1, 31, 64, 97, 128, 65]), (64, 12, [400, 385, 512, 511, 480, 450])],
    (256, 8, 1, True): [(64, 4, [1000, 897, 1024, 998] * 4)],
    (128, 8, 1, False): [(80, 4, [197, 129, 256, 1, 33, 200] * 2), (96, 2, [130, 256]), (128, 1, [200, 3])],
    (128, 4, 1, False): [(64, 12, [197, 193, 256, 1, 225, 32, 33, 100]), (64, 12, [161, 160] * 4), (64, 4, [300, 257, 384, 290, 31, 1] * 8), (64, 3, [100, 128, 1, 65, 33] * 20), (64, 2, [64, 1, 32]),
                         (64, 4, [400, 385, 512, 511, 257, 1, 129, 480] * 3),                          (80, 4, [267, 257, 100, 5] * 12)],
    (128, 4, 1, True): [(64, 4, [770, 1000, 1024, 897] * 4), (64, 3, [300, 257, 129, 1] * 51 + [300]), (80, 4, [300, 257, 1] * 21)],
}


@pytest.mark.parametrize("bias", [False, True])
@pytest.mark.parametrize("shape", sorted(CASES), ids=str)
def test_attention_however_it_is_cut_up(lib, shape, bias):
    """Against float64, and every query bit for bit what it is alone.  A weight exp(s - m) is rounded to bf16 (2^-9 of itself) before it
    meets the values, the output once more; twice that covers the fp32 sums (1024 terms), the exponential's error and the row sum, which
    takes the weights unrounded.  Sizes of 0, over whole blocks of keys and here and there, take a key's weight away."""
    import torch
    for dh, H, ns in CASES[shape]:
        assert _shape(lib, dh, H, ns) == shape, (dh, H, ns)
        D = dh * H
        cfg = synth.Config("attn", L=1, D=D, H=H, F=2 * D, dtype="bf16", B=1, n0=8, strategies=[(0, 0)], seed=11)
        ctx, _ = hz.make_context(cfg)
        off = np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)
        g = torch.Generator(device="cuda").manual_seed(dh + H + len(ns))
        qkv = torch.randn((int(off[-1]), 3 * D), generator=g, device="cuda").mul_(1.5).to(torch.bfloat16)
        sizes = torch.randint(1, 9, (int(off[-1]),), generator=g, device="cuda", dtype=torch.int32)
        for q in range(0, len(ns), 2):
            sizes[int(off[q]) + 32:min(int(off[q]) + 96, int(off[q + 1]))] = 0
            sizes[int(off[q]) + 1:int(off[q + 1]):7] = 0
        flags = lib.OTAS_FLAG_SIZE_BIAS if bias else 0
        o = torch.full((int(off[-1]), D), float("nan"), dtype=torch.bfloat16, device="cuda")
        ctx.otas_attention(qkv, sizes, off, flags, o)
        for q, n in enumerate(ns):
            rows = slice(int(off[q]), int(off[q + 1]))
            Q, K, V = qkv[rows].double().view(n, 3, H, dh).permute(1, 2, 0, 3)
            s = Q @ K.transpose(1, 2) * dh ** -0.5
            if bias:
                s = s + sizes[rows].double().log()
            p = s.softmax(-1)
            want, mag = p @ V, p @ V.abs()
            got = o[rows].double().view(n, H, dh).transpose(0, 1)
            assert bool(((got - want).abs() <= 2.0 ** -8 * (mag + want.abs())).all()), (dh, H, q, n)
            if q < 12:
                alone = torch.full((n, D), float("nan"), dtype=torch.bfloat16, device="cuda")
                ctx.otas_attention(qkv[rows].contiguous(), sizes[rows].contiguous(), [0, n], flags, alone)
                assert torch.equal(o[rows], alone), (dh, H, q, n)
        ctx.close()


# queries of a batch -> how attention is cut up beside its selection (12 heads; 24 or 46 tokens merged)
FUSED = {(65, 2): (128, 4, 1, False), (197, 1): (256, 8, 1, False), (197, 24): (256, 8, 1, False), (300, 2): (256, 4, 4, True),
         (300, 20): (128, 4, 1, True), (257, 3): (256, 8, 4, True), (577, 12): (128, 4, 1, True), (500, 16): (256, 8, 1, True)}


@pytest.mark.parametrize("bias", [False, True])
@pytest.mark.parametrize("n,B", sorted(FUSED))
def test_attention_beside_a_selection(lib, n, B, bias):
    """Two blocks of B queries, which all merge but the last.  Each query's rows, sizes and edges are bit for bit those of the query alone,
    whose attention is cut up otherwise; and the one that merges nothing has the bits of a pass without selections, whose attention is
    the one that the test above compares with float64."""
    import torch
    H, r = 12, 24
    D = 64 * H
    cfg = synth.Config("fused", L=2, D=D, H=H, F=768, dtype="bf16", B=1, n0=8, seed=B + n)
    ctx, _ = hz.make_context(cfg)
    assert ctx.otas_splitk_factor(B * n, D, cfg.F, 8) == 1
    how = ctypes.CDLL(lib.lib_path())._ZN4otas18attention_plan_howEiiiiib

    class Parts(ctypes.Structure):
        _fields_ = [("na", ctypes.c_int), ("nb", ctypes.c_int)]
    how.argtypes, how.restype = [ctypes.c_int] * 5 + [ctypes.c_bool], Parts
    p = how(1, B, n, D, H, True)
    assert p.na > 0 and _shape(lib, 64, H, [n] * B, B * p.na * p.nb) == FUSED[n, B]
    g = torch.Generator(device="cuda").manual_seed(n)
    x0 = torch.randn((B * n, D), generator=g, device="cuda").to(torch.bfloat16)
    off = np.arange(B + 1, dtype=np.int32) * n
    R = [r] * (B - 1) + [0 if B > 1 else r]
    flags = lib.OTAS_FLAG_SIZE_BIAS if bias else 0
    got = hz.gpu_forward(ctx, x0, off, R, flags)
    for q in sorted({0, B // 2, B - 1}):
        alone = hz.gpu_forward(ctx, x0[q * n:(q + 1) * n].contiguous(), off[:2], [R[q]], flags)
        assert np.array_equal(got["x"][q], alone["x"][0]) and np.array_equal(got["sizes"][q], alone["sizes"][0]), q
        for a, b in zip(got["trace"][q], alone["trace"][0]):
            assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    ctx.close()


def test_lanes_and_batches_leave_the_bits_of_bf16_passes(lib):
    """No launch is split over K here, so that a query's rows are the same bits in any batch and on any number of lanes, though its attention
    is cut up otherwise in each."""
    import torch
    H, B = 2, 40
    cfg = synth.Config("lanes", L=3, D=64 * H, H=H, F=256, dtype="bf16", B=1, n0=8, seed=3)
    ctx, _ = hz.make_context(cfg)
    assert ctx.otas_splitk_factor(200, cfg.D, cfg.F, 8) == 1
    ns = [(200, 65, 129, 257)[q % 4] for q in range(B)]
    off = np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)
    assert _shape(lib, 64, H, ns)[2] == 1 and _shape(lib, 64, H, ns[:5])[2] == 4
    g = torch.Generator(device="cuda").manual_seed(8)
    x0 = torch.randn((int(off[-1]), cfg.D), generator=g, device="cuda").to(torch.bfloat16)
    for R in ([0] * B, [(0, 11, 5)[q % 3] for q in range(B)]):
        ctx.otas_set_lanes(1)
        want = hz.gpu_forward(ctx, x0, off, R)
        for lanes in (2, 5, 8):
            ctx.otas_set_lanes(lanes)
            got = hz.gpu_forward(ctx, x0, off, R)
            for q in range(B):
                assert np.array_equal(got["x"][q], want["x"][q]) and np.array_equal(got["sizes"][q], want["sizes"][q]), (lanes, q)
        ctx.otas_set_lanes(1)
        for q in range(6):
            alone = hz.gpu_forward(ctx, x0[int(off[q]):int(off[q + 1])].contiguous(), [0, ns[q]], [R[q]])
            assert np.array_equal(alone["x"][0], want["x"][q]), q
    ctx.close()
