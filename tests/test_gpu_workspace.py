"""Batches whose QKV projection and hidden rows share one workspace buffer: a query's rows are those of the query alone,
for which the two lie apart."""
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


def test_workspace_bytes_never_shrink_as_a_batch_grows(lib):
    """A workspace sized for a program's largest batch serves its smaller ones, on both sides of the line."""
    cfg = synth.config("tiny")
    ctx, _ = hz.make_context(cfg)
    line = (32 << 20) // (4 * (3 * cfg.D + cfg.F))
    sizes = [ctx.otas_workspace_bytes(4, T) for T in range(line - 2048, line + 2048, 64)]
    assert sizes == sorted(sizes)
    ctx.close()


@pytest.mark.parametrize("D,F", [(72, 136), (64, 8)])
def test_weights_read_ahead_change_nothing(lib, D, F):
    """Up to 2048 rows merge-apply's launch also reads FC1's weight (here of 153 and 8 cache lines, dealt to eight parts):
    the rows are those of a batch above the line."""
    import torch
    n, B = 30, 80
    cfg = synth.Config("warm", L=2, D=D, H=1, F=F, dtype="bf16", B=1, n0=n, seed=5)
    ctx, _ = hz.make_context(cfg)
    x0 = torch.randn((B * n, D), generator=torch.Generator().manual_seed(2)).to("cuda").to(ctx.torch_dtype)
    many = hz.gpu_forward(ctx, x0, np.arange(B + 1, dtype=np.int32) * n, [5] * B)
    for q in (0, B - 1):
        one = hz.gpu_forward(ctx, x0[q * n:(q + 1) * n].contiguous(), [0, n], [5])
        assert np.array_equal(one["x"][0], many["x"][q]) and np.array_equal(one["sizes"][0], many["sizes"][q])
    ctx.close()
