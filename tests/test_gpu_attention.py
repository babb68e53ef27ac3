"""bf16 attention in every way the library cuts up its work: key groups, staged pieces, waves per row block."""
import numpy as np
import pytest

import otas_synth as synth
from tests import harness as hz

pytestmark = pytest.mark.gpu

# Which one a launch takes depends on the heads, the number of queries and the longest ones (attention_shape).  Lengths at
# and beside the edges of key blocks (32), groups' shares, row blocks (32, 64, 128, 256) and staged pieces (128, 256).
CASES = {
    "four groups, blocks of 32 rows": [(64, 4, [65]), (64, 2, [197, 1, 33, 32]), (64, 4, [700, 2]), (80, 4, [97, 31, 128, 129]),
                                       (80, 2, [577, 160, 1])],
    "four groups, blocks of 64 rows": [(64, 4, [300, 1, 33, 64, 65, 256, 31, 129]), (64, 3, [161, 160, 129, 128, 2, 97, 63, 130, 191, 150, 1, 140, 155])],
    "two groups": [(64, 4, [197, 193, 256, 1, 225, 32, 33, 100, 130, 161] * 2), (64, 6, [577, 640, 515, 197, 64, 1, 31, 290, 200, 33])],
    "pieces of 256": [(64, 4, [400, 385, 512, 511, 257, 1, 129, 480] * 3), (64, 4, [770, 1000, 1024, 897] * 4)],
    "heads dealt to the XCDs": [(64, 3, [300, 257, 129, 1] * 51 + [300]), (64, 3, [300, 270, 301]), (80, 4, [300, 257, 1] * 21)],
    "pieces of 128": [(64, 4, [300, 257, 384, 290, 31, 1] * 8), (80, 4, [267, 257, 100, 5] * 12), (64, 3, [100, 128, 1, 65, 33] * 20)],
}


@pytest.mark.parametrize("bias", [False, True])
@pytest.mark.parametrize("name", sorted(CASES))
def test_attention_however_it_is_cut_up(lib, name, bias):
    """Against float64.  A weight exp(s - m) is rounded to bf16 (2^-9 of itself) before it meets the values, the output once more;
    twice that covers the fp32 sums (1024 terms), the exponential's error and the row sum, which takes the weights unrounded."""
    import torch
    for dh, H, ns in CASES[name]:
        D = dh * H
        cfg = synth.Config("attn", L=1, D=D, H=H, F=2 * D, dtype="bf16", B=1, n0=8, strategies=[(0, 0)], seed=11)
        ctx, _ = hz.make_context(cfg)
        off = np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)
        g = torch.Generator(device="cuda").manual_seed(dh + H + len(ns))
        qkv = torch.randn((int(off[-1]), 3 * D), generator=g, device="cuda").mul_(1.5).to(torch.bfloat16)
        sizes = torch.randint(1, 9, (int(off[-1]),), generator=g, device="cuda", dtype=torch.int32)
        o = torch.full((int(off[-1]), D), float("nan"), dtype=torch.bfloat16, device="cuda")
        ctx.otas_attention(qkv, sizes, off, lib.OTAS_FLAG_SIZE_BIAS if bias else 0, o)
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
        ctx.close()


@pytest.mark.parametrize("n", [200, 300, 577])
@pytest.mark.parametrize("B", [1, 2, 5, 11])
def test_heads_dealt_to_the_xcds_beside_a_selection(lib, B, n):
    """Equal queries are equal rows, whichever workgroups worked on them, and the one that merges nothing has the rows (bf16, up to
    four roundings of 2^-8 of a row's largest) of a pass without selections."""
    cfg = synth.Config("fused", L=1, D=384, H=6, F=768, dtype="bf16", B=1, n0=8, seed=B + n)
    ctx, _ = hz.make_context(cfg)
    import torch
    tok = torch.randn((n, cfg.D), generator=torch.Generator().manual_seed(n)).to("cuda").to(torch.bfloat16)
    x0, off = tok.repeat(B + 1, 1), np.arange(B + 2, dtype=np.int32) * n
    got = hz.gpu_forward(ctx, x0, off, [8] * B + [0])
    plain = hz.gpu_forward(ctx, tok, off[:2], [0])["x"][0]
    for q in range(1, B):
        assert np.array_equal(got["x"][q], got["x"][0]) and np.array_equal(got["trace"][q][0], got["trace"][0][0])
    assert np.abs(got["x"][B] - plain).max() <= 2.0 ** -6 * np.abs(plain).max()
    kept = np.setdiff1d(np.arange(n), np.concatenate(got["trace"][0][0]))   # rows that the merge left alone come in order
    rows = np.setdiff1d(np.arange(n), got["trace"][0][0][0])
    assert np.abs(got["x"][0][np.searchsorted(rows, kept)] - plain[kept]).max() <= 2.0 ** -6 * np.abs(plain).max()
    ctx.close()
