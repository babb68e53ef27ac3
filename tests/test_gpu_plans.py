"""The small integer arrays of a call go to the GPU in the kernels' arguments up to a number of queries and through the
device plan buffer beyond it: both sides of that line give the same rows, edges and sizes."""
import ctypes

import numpy as np
import pytest

import otas_synth as synth
from tests import harness as hz

pytestmark = pytest.mark.gpu


def _queries(cfg, B, seed):
    rng = np.random.default_rng(seed)
    n = rng.integers(2, 9, B)
    base = synth.query_tokens(cfg, 0)
    return [np.ascontiguousarray(base[(11 * q) % 180:(11 * q) % 180 + n[q]]) for q in range(B)], rng


@pytest.mark.parametrize("B", [1, 2, 255, 480])
def test_encoder_plan_expanded_on_the_device_equals_the_copied_one(lib, B):
    """B queries (plan expanded by the first LayerNorm: 480 is the most) against the same B queries followed by enough
    others to make the host build and copy the plan; fp32, where rows do not depend on the batch: bit for bit."""
    cfg = synth.config("tiny")
    ctx, _ = hz.make_context(cfg)
    toks, rng = _queries(cfg, 500, 3)
    R = rng.integers(0, 4, 500).tolist()
    prm = [np.zeros((0, cfg.D), dtype=np.float32)] * 500
    x0, off = hz.gpu_prepend(ctx, toks, prm)
    many = hz.gpu_forward(ctx, x0, off, R)
    few = hz.gpu_forward(ctx, x0[:int(off[B])].contiguous(), off[:B + 1], R[:B])
    plain = hz.gpu_forward(ctx, x0[:int(off[B])].contiguous(), off[:B + 1], [0] * B)
    for q in range(B):
        assert np.array_equal(few["x"][q], many["x"][q]) and np.array_equal(few["sizes"][q], many["sizes"][q])
        for a, b in zip(few["trace"][q], many["trace"][q]):
            assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
        assert (plain["sizes"][q] == 1).all()
    ctx.close()


@pytest.mark.parametrize("mode", [1, 2])
def test_per_layer_prompting_plan_on_both_sides(lib, mode):
    import torch
    cfg = synth.config("tiny")
    ctx, _ = hz.make_context(cfg)
    toks, rng = _queries(cfg, 500, 5)
    P = [min(int(p), len(t) - 1) for p, t in zip(rng.integers(0, 3, 500), toks)]
    off = np.concatenate([[0], np.cumsum([len(t) for t in toks])]).astype(np.int32)
    prm_off = np.concatenate([[0], np.cumsum(P)]).astype(np.int32)
    x = torch.from_numpy(np.concatenate(toks)).to("cuda")
    prompts = torch.randn((cfg.L, int(prm_off[-1]), cfg.D), generator=torch.Generator().manual_seed(1)).to("cuda")
    got = {}
    for B in (480, 500):
        T, TP = int(off[B]), int(prm_off[B])
        rows = T + (TP * (cfg.L - 1) if mode == 2 else 0)
        out = torch.full((rows, cfg.D), float("nan"), device="cuda")
        sizes = torch.zeros(rows, dtype=torch.int32, device="cuda")
        ws = torch.empty(ctx.otas_workspace_bytes(B, max(T, rows)), dtype=torch.uint8, device="cuda")
        ctx.otas_encoder_forward_deep(x[:T].contiguous(), off[:B + 1], mode, prompts[:, :TP].contiguous(), prm_off[:B + 1],
                                      ws, out, sizes)
        assert bool((sizes == 1).all())
        got[B] = out
    assert torch.equal(got[480], got[500][:got[480].shape[0]])
    ctx.close()


@pytest.mark.parametrize("B", [239, 240])
def test_prepend_merge_and_heads_plans_on_both_sides(lib, B):
    """239 queries are the most whose prepend and merge plans fit the arguments."""
    import torch
    cfg = synth.config("tiny")
    ctx, _ = hz.make_context(cfg)
    toks, rng = _queries(cfg, B, 7)
    prm = [synth.query_tokens(cfg, 1)[q % 50:q % 50 + q % 3] for q in range(B)]
    x0, off = hz.gpu_prepend(ctx, toks, prm)
    ref = np.concatenate([np.concatenate([t[:1], p, t[1:]]) for t, p in zip(toks, prm)])
    assert np.array_equal(x0.cpu().numpy(), ref)
    T = int(off[-1])
    metric = torch.randn((T, 12), generator=torch.Generator().manual_seed(2)).to("cuda")
    r = rng.integers(0, 4, B).tolist()
    n_out = [int(off[q + 1] - off[q]) - min(r[q], (int(off[q + 1] - off[q]) - 1) // 2) for q in range(B)]
    ws = torch.empty(ctx.otas_merge_workspace_bytes(B, T), dtype=torch.uint8, device="cuda")
    out = torch.full((sum(n_out), cfg.D), float("nan"), device="cuda")
    sizes = torch.zeros(sum(n_out), dtype=torch.int32, device="cuda")
    oo = ctx.otas_token_merge(x0, metric, 12, None, off, r, ws, out, sizes)
    assert np.array_equal(np.diff(oo), n_out)
    for q in (0, 1, B // 2, B - 1):     # alone, through the arguments
        lo, hi = int(off[q]), int(off[q + 1])
        o1 = torch.full((n_out[q], cfg.D), float("nan"), device="cuda")
        s1 = torch.zeros(n_out[q], dtype=torch.int32, device="cuda")
        ctx.otas_token_merge(x0[lo:hi].contiguous(), metric[lo:hi].contiguous(), 12, None, [0, hi - lo], [r[q]], ws, o1, s1)
        assert torch.equal(o1, out[int(oo[q]):int(oo[q + 1])]) and torch.equal(s1, sizes[int(oo[q]):int(oo[q + 1])])
    g = torch.Generator().manual_seed(4)
    for classes in ([1, 7, 33], [64] * (150 if B == 240 else 3)):     # 150 tasks: the records alone pass the line
        heads = [(torch.randn((k, cfg.D), generator=g).to("cuda"), torch.randn(k, generator=g).to("cuda")) for k in classes]
        gam, bet = torch.ones(cfg.D, device="cuda"), torch.zeros(cfg.D, device="cuda")
        task = [q % len(classes) for q in range(B)]
        lg = torch.full((B, 70), float("nan"), device="cuda")
        ctx.otas_task_heads(x0, off, task, heads, gam, bet, lg)
        first = x0[torch.from_numpy(off[:-1].astype(np.int64)).to("cuda")].double()
        h = torch.nn.functional.layer_norm(first, (cfg.D,), eps=1e-6)
        for q in range(B):
            k = classes[task[q]]
            want = heads[task[q]][0].double() @ h[q] + heads[task[q]][1].double()
            # D + 8 roundings of 2^-24 on sums of |w h|; |h| of a normalised row sums to less than D
            bound = (cfg.D + 8) * 2.0 ** -24 * (heads[task[q]][0].double().abs() @ h[q].abs() + 1.0)
            assert bool(((lg[q, :k].double() - want).abs() <= bound).all()) and bool((lg[q, k:] == 0).all())
    ctx.close()


def test_heads_of_more_queries_than_a_second_grid_dimension_holds(lib):
    import torch
    cfg = synth.config("tiny")
    ctx, _ = hz.make_context(cfg)
    B, g = 70000, torch.Generator().manual_seed(6)
    x = torch.randn((B, cfg.D), generator=g).to("cuda")
    heads = [(torch.randn((k, cfg.D), generator=g).to("cuda"), torch.randn(k, generator=g).to("cuda")) for k in (3, 2)]
    gam, bet = torch.ones(cfg.D, device="cuda"), torch.zeros(cfg.D, device="cuda")
    lg = torch.full((B, 3), float("nan"), device="cuda")
    ctx.otas_task_heads(x, np.arange(B + 1, dtype=np.int32), np.arange(B, dtype=np.int32) % 2, heads, gam, bet, lg)
    h = torch.nn.functional.layer_norm(x.double(), (cfg.D,), eps=1e-6)
    for t, (w, b) in enumerate(heads):
        k, got = w.shape[0], lg[t::2]
        bound = (cfg.D + 8) * 2.0 ** -24 * (h[t::2].abs() @ w.double().abs().T + 1.0)      # as in the test above
        assert bool(((got[:, :k].double() - (h[t::2] @ w.double().T + b.double())).abs() <= bound).all())
        assert bool((got[:, k:] == 0).all())
    ctx.close()


@pytest.mark.parametrize("n", [2, 64, 65, 66, 197, 257, 513, 577, 1024])
def test_selection_shared_by_workgroups_gives_the_same_edges(lib, n):
    """bf16, head width 64: the best matches of a query are found by as many workgroups as the batch leaves room for, down
    to one block of 32 A and 32 B tokens each.  The same query in batches of 1, 3, 20 and 150: the same edges, ranks,
    sizes.  One query is shorter than the longest, so that some of its workgroups have no tokens."""
    cfg = synth.config("tiny")
    cfg.D, cfg.H, cfg.F, cfg.dtype, cfg.n0, cfg.L = 256, 4, 512, "bf16", n, 1
    ctx, _ = hz.make_context(cfg)
    tok, short = synth.query_tokens(cfg, 3)[:n], synth.query_tokens(cfg, 4)[:max(2, n // 3)]
    none = np.zeros((0, cfg.D), dtype=np.float32)
    r = max(0, (n - 1) // 3)
    want = {}
    for B in (1, 3, 20, 150):
        toks = [tok] + [short] * (B > 1) + [tok] * max(0, B - 2)
        x0, off = hz.gpu_prepend(ctx, toks, [none] * B)
        got = hz.gpu_forward(ctx, x0, off, [r] * B)
        for q in range(B):
            tr, sizes = want.setdefault(q == 1, (got["trace"][q], got["sizes"][q]))
            assert np.array_equal(got["sizes"][q], sizes)
            for a, b in zip(got["trace"][q], tr):
                assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])
    ctx.close()


def _check_edges(n, r, src, dst, sizes):
    """r distinct unprotected A tokens, each merged into an existing B token, and no token lost."""
    assert len(src) == r and len(np.unique(src)) == r
    assert (src % 2 == 0).all() and (src >= 2).all() and (src < n).all()
    assert (dst % 2 == 1).all() and (dst >= 1).all() and (dst < n).all()
    assert int(sizes.sum()) == n and (sizes >= 1).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [3, 65, 197, 600])
def test_merge_of_tokens_that_compare_with_none(lib, dtype, n):
    """NaN similarities (a broken or overflowing token) still give a merge: every index a later kernel reads with stays
    inside the query, the tokens that can be compared rank first, the leading token is never merged.  As an
    operator, and in the encoder (one workgroup per query, and as many as a lone query gets)."""
    import torch
    cfg = synth.config("tiny")
    cfg.D, cfg.H, cfg.F, cfg.dtype, cfg.n0, cfg.L = 256, 4, 512, dtype, n, 1
    ctx, _ = hz.make_context(cfg)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(n)
    r = (n - 1) // 2                                               # all that the length allows
    a_bad, all_b = [2] if n < 5 else [2, n // 2 // 2 * 2, (n - 1) // 2 * 2], list(range(1, n, 2))
    for bad in ([], a_bad, all_b, a_bad + all_b, list(range(n))):
        x = torch.randn((n, cfg.D), generator=g, device="cuda").to(dt)
        metric = torch.randn((n, 64), generator=g, device="cuda").to(dt)
        metric[bad] = float("nan")
        ws = torch.empty(ctx.otas_merge_workspace_bytes(1, n), dtype=torch.uint8, device="cuda")
        out = torch.full((n - r, cfg.D), float("nan"), device="cuda", dtype=dt)
        sizes = torch.zeros(n - r, dtype=torch.int32, device="cuda")
        src, dst = (torch.full((r,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
        ctx.otas_token_merge(x, metric, 64, None, [0, n], [r], ws, out, sizes, src, dst)
        src, dst = src.cpu().numpy(), dst.cpu().numpy()
        _check_edges(n, r, src, dst, sizes.cpu().numpy())
        assert bool(torch.isfinite(out).all())
        if bad == a_bad:                                           # the A tokens that compare with none come last
            assert sorted(src[r - len(a_bad):]) == sorted(a_bad) and (dst[r - len(a_bad):] == 1).all()
        tok = x.float().cpu().numpy()
        tok[bad] = float("nan")
        for B in (1, 100):
            toks = [x.float().cpu().numpy()] * B
            toks[B // 2] = tok
            x0, off = hz.gpu_prepend(ctx, toks, [np.zeros((0, cfg.D), dtype=np.float32)] * B)
            got = hz.gpu_forward(ctx, x0, off, [r] * B)
            for q in range(B):
                _check_edges(n, r, *got["trace"][q][0], got["sizes"][q])
                assert q == B // 2 or np.isfinite(got["x"][q]).all()
    ctx.close()


@pytest.mark.parametrize("dtype,D,dm", [("bf16", 768, 64), ("bf16", 136, 100), ("f32", 192, 128), ("f32", 104, 4)])
@pytest.mark.parametrize("ns", [[129], [128, 129, 1], [0, 197, 2, 196, 0, 33, 130], [577, 400], [1024], [131] * 64])
def test_merge_shared_out_equals_one_workgroup_a_query(lib, dtype, D, dm, ns):
    """Up to 64 queries with one of 129 tokens or more share their work between workgroups; with more queries each has one.
    Rows, sizes, offsets and edges bit for bit, with and without sizes and edges, some queries removing nothing."""
    import ctypes
    import torch
    cfg = synth.Config("op", L=1, D=D, H=8 if D == 768 else 2, F=128, dtype=dtype, B=1, n0=2, seed=17)
    ctx, _ = hz.make_context(cfg)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    more = ns + [3] * (65 - len(ns))
    off = np.concatenate([[0], np.cumsum(more)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(len(ns) + ns[0])
    x = torch.randn((int(off[-1]), D), generator=g, device="cuda").to(dt)
    metric = torch.randn((int(off[-1]), dm), generator=g, device="cuda").to(dt)
    sizes = torch.randint(1, 5, (int(off[-1]),), generator=g, device="cuda", dtype=torch.int32)
    r = [(0, n // 3, n, 1)[(q + len(ns)) % 4] for q, n in enumerate(more)]

    def run(B, sz, traced, static=False):
        T = int(off[B])
        out = torch.full((T, D), float("nan"), device="cuda", dtype=dt)
        so, src, dst = (torch.full((T,), -1, dtype=torch.int32, device="cuda") for _ in range(3))
        ws = torch.full((ctx.otas_merge_workspace_bytes(B, T),), 0xff, dtype=torch.uint8, device="cuda")
        args = (x[:T].contiguous(), metric[:T].contiguous(), dm, sz[:T].contiguous() if sz is not None else None, off[:B + 1], r[:B])
        tr = (src, dst) if traced else (None, None)
        o = ctx.otas_token_merge_static(*args, out, so, *tr) if static else ctx.otas_token_merge(*args, ws, out, so, *tr)
        return out, so, src, dst, np.asarray(o)

    B = len(ns)
    in_two = ctypes.CDLL(lib.lib_path())._ZN4otas18token_merge_in_twoEiii
    in_two.argtypes, in_two.restype = [ctypes.c_int] * 3, ctypes.c_bool
    assert (in_two(B, max(ns), dm) or max(ns) * dm > 64 * 1024) and not in_two(65, max(ns), dm)   # (B tokens that LDS does not hold)
    for sz in (None, sizes):
        want = run(65, sz, True)
        end, edges = int(want[4][B]), int(off[B]) - int(want[4][B])
        # (without a workspace a query whose metric rows do not fit in LDS is refused)
        for traced, static in ((True, False), (False, False), (True, True))[:3 if max(ns) * (dm + 4) * 4 < 150 * 1024 else 2]:
            got = run(B, sz, traced, static)
            assert np.array_equal(got[4], want[4][:B + 1])
            assert torch.equal(got[0][:end], want[0][:end]) and torch.equal(got[1][:end], want[1][:end])
            assert bool((got[1][end:] == -1).all()) and bool(got[0][end:].isnan().all())
            for a, b in zip(got[2:4], want[2:4]):
                assert torch.equal(a[:edges], b[:edges] if traced else torch.full_like(a[:edges], -1))
                assert bool((a[edges:] == -1).all())
    ctx.close()


@pytest.mark.parametrize("D,H", [(192, 3), (200, 2)])
def test_fp32_selection_beside_attention_equals_the_plan_kernel(lib, D, H):
    """f32 models: a query alone runs its selection beside attention, in as many workgroups as its tokens have blocks, and
    its lists beside the projection; in this batch, whose projection is too large for the small tiles and no multiple of
    128 wide, the plan is a kernel of its own.  Rows, sizes and edges bit for bit."""
    import torch
    cfg = synth.Config("fused", L=2, D=D, H=H, F=256, dtype="f32", B=1, n0=2, seed=17)
    ctx, _ = hz.make_context(cfg)
    ns = [2, 3, 33, 64, 65, 66, 129, 577, 1024, 300, 300, 300, 300, 300]
    off = np.concatenate([[0], np.cumsum(ns)]).astype(np.int32)
    x0 = torch.randn((int(off[-1]), D), generator=torch.Generator().manual_seed(3)).to("cuda")
    R = [1, 1, 4, 8, 32, 5, 64, 23, 400, 16, 0, 149, 7, 9]
    many = hz.gpu_forward(ctx, x0, off, R)
    for q, n in enumerate(ns):
        one = hz.gpu_forward(ctx, x0[int(off[q]):int(off[q + 1])].contiguous(), [0, n], [R[q]])
        assert np.array_equal(one["x"][0], many["x"][q]) and np.array_equal(one["sizes"][0], many["sizes"][q]), n
        for a, b in zip(one["trace"][0], many["trace"][q]):
            assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), n
    ctx.close()


class PlanTail(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("in_off", "out_off", "reff", "troff", "src_list", "row_ptr", "trace_src",
                                               "trace_dst", "best", "bcol")] + [
        ("stride", ctypes.c_int64), ("nb", ctypes.c_int), ("B", ctypes.c_int)]


@pytest.mark.parametrize("shift", ["", "x", "w"])
@pytest.mark.parametrize("M,D,B", [(600, 192, 3), (3200, 192, 40), (3201, 192, 40), (3300, 192, 40), (2048, 256, 8), (2080, 256, 8),
                                   (2400, 256, 8), (8200, 256, 100), (8200, 256, 510), (1206, 768, 6), (200, 72, 200)])
def test_fp32_lists_beside_the_projection_where_they_are_said_to_fit(lib, M, D, B, shift):
    """Row counts on both sides of the small tiles (512 tiles, 600 where the large ones are staged), few and many queries,
    operands four bytes into a buffer: where linear_plan_tail_fits says so the launch takes the shape, whose rows are then the
    plain launch's and whose lists (nothing merges) name every row once; where the large tiles are staged it refuses."""
    import torch
    so = ctypes.CDLL(lib.lib_path())
    fits = so._ZN4otas21linear_plan_tail_fitsEiPKvS1_liii
    fits.restype, vp = ctypes.c_bool, ctypes.c_void_p
    cfg = synth.config("tiny")
    ctx, _ = hz.make_context(cfg)
    g = torch.Generator(device="cuda").manual_seed(M + B)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda")
    off4 = lambda t: torch.cat([t.new_zeros(1), t.flatten()])[1:].view(t.shape)
    x, w, b, res = rand(M, D), rand(D, D), rand(D), rand(M, D)
    x, w = off4(x) if shift == "x" else x, off4(w) if shift == "w" else w
    want, got = torch.empty((M, D), device="cuda"), torch.full((M, D), float("nan"), device="cuda")
    ctx.otas_linear_kernel(0, x, w, b, res, M, D, D, 2, want)
    ints = lambda a: torch.as_tensor(a, dtype=torch.int32).to("cuda")
    off, zero = ints(np.linspace(0, M, B + 1).astype(np.int64)), ints([0] * B)
    lists, ptr = ints([-1] * M), ints([-1] * (M + 1))
    best, col = rand(M), ints([0] * M)
    p = lambda t: vp(t.data_ptr())
    pt = PlanTail(*(t.data_ptr() for t in (off, off, zero, zero, lists, ptr)), None, None, best.data_ptr(), col.data_ptr(), M, 1, B)
    ok = fits(0, p(x), p(w), ctypes.c_int64(M), D, D, B)
    small, dma = -(-M // 32) * -(-D // 32), D % 128 == 0 and not shift
    assert ok or small > (512 if dma else 600)
    status = so._ZN4otas23launch_linear_plan_tailEiPKvS1_S1_PKfPvliiRKNS_8PlanTailEiP12ihipStream_t(
        0, p(x), p(w), p(b), p(res), p(got), ctypes.c_int64(M), D, D, ctypes.byref(pt), -(-M // B),
        vp(torch.cuda.current_stream().cuda_stream))
    assert status == 0 if ok or dma else status == 1           # hipErrorInvalidValue
    if status == 0:
        assert torch.equal(got, want)
        assert lists.tolist() == list(range(M)) and ptr[:M].tolist() == list(range(M))
    else:
        assert bool(torch.isnan(got).all()) and bool((lists == -1).all())
    ctx.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("p,shift", [(16, 0), (8, 0), (4, 0), (16, 1), (6, 0)])
def test_patches_and_rows_by_16_bytes_and_by_elements(lib, dtype, p, shift):
    """Patch sizes that are a multiple of 16 bytes' elements and not, pointers that begin on 16 bytes and not (shift in
    elements): both forms of the two kernels give the tokens of torch's unfold, product and sum; a grid of 5 x 7 patches, 4
    channels, so that a workgroup's last threads and a band's last patch are partial."""
    import torch
    cfg = synth.config("tiny")
    cfg.dtype = dtype
    ctx, _ = hz.make_context(cfg)
    dt, B, C, Hi, Wi = ctx.torch_dtype, 3, 4, 5 * p, 7 * p
    N, kp = 35, C * p * p
    g = torch.Generator(device="cuda").manual_seed(p)

    def draw(*shape):                               # begins `shift` elements past a 16-byte boundary
        n = int(np.prod(shape))
        buf = torch.empty(n + 8, dtype=dt, device="cuda")
        buf.copy_(torch.randn(n + 8, generator=g, device="cuda"))
        return buf[shift:shift + n].view(shape)

    img, cls, pos = draw(B, C, Hi, Wi), draw(cfg.D), draw(1 + N, cfg.D)
    w = (torch.randn((cfg.D, kp), generator=g, device="cuda") * 0.05).to(dt)
    b = torch.randn(cfg.D, generator=g, device="cuda").to(dt)
    ws = torch.empty(ctx.otas_patch_embed_workspace_bytes(B, C, Hi, Wi, p), dtype=torch.uint8, device="cuda")
    toks = draw(B * (1 + N), cfg.D).fill_(float("nan"))
    ctx.otas_patch_embed(img, p, w, b, cls, pos, ws, toks)
    rows = torch.nn.functional.unfold(img.double(), p, stride=p).transpose(1, 2)
    proj, mag = rows @ w.double().T + b.double(), rows.abs() @ w.double().abs().T + b.double().abs()
    eps = 2.0 ** -24 if dtype == "f32" else 2.0 ** -8
    got = toks.double().view(B, 1 + N, cfg.D)
    # the projection's sum in fp32, its rounding to the model's type, one more addition with its rounding
    want = proj + pos[1:].double()
    bound = (kp + 8) * 2.0 ** -24 * mag + eps * (proj.abs() + want.abs()) + 1e-6
    assert bool(((got[:, 1:] - want).abs() <= bound).all())
    lead = (cls.float() + pos[0].float()).to(dt)
    assert all(torch.equal(toks.view(B, 1 + N, cfg.D)[q, 0], lead) for q in range(B))
    ctx.close()


def test_more_images_than_a_grid_has_threads_for(lib):
    """A launch has fewer than 2^32 threads, 256 for the rows of a band of patches however short they are: 2^23 + 3 images of two channels
    of 4 x 4 pixels in one patch are more.  So are 2^26 + 6 token rows with a wave each.  (One patch an image: the patch matrix is the images.)"""
    import ctypes
    import torch
    so, vp, i32 = ctypes.CDLL(lib.lib_path()), ctypes.c_void_p, ctypes.c_int
    patchify, finish = so._ZN4otas15launch_patchifyEiPKvPviiiiiP12ihipStream_t, so._ZN4otas19launch_embed_finishEiPKvS1_S1_PviiiiP12ihipStream_t
    patchify.argtypes, finish.argtypes = [i32, vp, vp] + [i32] * 5 + [vp], [i32] + [vp] * 4 + [i32] * 4 + [vp]
    stream = torch.cuda.current_stream().cuda_stream
    B = (1 << 23) + 3
    img = torch.randint(-9, 9, (B, 32), dtype=torch.int8, device="cuda").to(torch.bfloat16)
    out = torch.full_like(img, float("nan"))
    assert patchify(1, img.data_ptr(), out.data_ptr(), B, 2, 4, 4, 4, stream) == 0
    assert torch.equal(out, img)
    del img, out
    B, D = (1 << 25) + 3, 8
    proj = torch.randint(-9, 9, (B, D), dtype=torch.int8, device="cuda").to(torch.bfloat16)
    cls, pos = (torch.randint(-9, 9, s, dtype=torch.int8, device="cuda").to(torch.bfloat16) for s in ((D,), (2, D)))
    toks = torch.full((B, 2, D), float("nan"), dtype=torch.bfloat16, device="cuda")
    assert finish(1, proj.data_ptr(), cls.data_ptr(), pos.data_ptr(), toks.data_ptr(), B, 1, D, 1, stream) == 0
    assert bool((toks[:, 0] == cls + pos[0]).all()) and torch.equal(toks[:, 1], proj + pos[1])


@pytest.mark.parametrize("n", [2, 3, 16, 17, 31, 32, 33, 34, 49, 63, 64, 65, 100])
def test_selection_in_tiles_of_16_and_of_32(lib, n):
    """Queries of up to 64 tokens have one block of 32 tokens of either kind, which the selection beside attention (eight waves)
    compares in tiles of 16 x 16; otas_token_merge (sixteen waves) in tiles of 32 x 32.  The same edges from the same keys: both
    heads are given the same ones, whose mean is that of one."""
    import torch
    D, dh = 128, 64
    cfg = synth.Config("tiles", L=1, D=D, H=2, F=128, dtype="bf16", B=1, n0=n, seed=n)
    layers = synth.all_weights(cfg)
    layers[0]["w_qkv"][D + dh:2 * D] = layers[0]["w_qkv"][D:D + dh]
    layers[0]["b_qkv"][D + dh:2 * D] = layers[0]["b_qkv"][D:D + dh]
    ctx, _ = hz.make_context(cfg, layers)
    g = torch.Generator(device="cuda").manual_seed(n)
    x0 = torch.randn((n, D), generator=g, device="cuda").to(torch.bfloat16)
    r = max(1, n // 3)
    got = hz.gpu_forward(ctx, x0, [0, n], [r])
    w = {k: torch.from_numpy(np.ascontiguousarray(v)).to("cuda").to(torch.bfloat16) for k, v in layers[0].items()}
    h = torch.empty((n, D), dtype=torch.bfloat16, device="cuda")
    qkv = torch.empty((n, 3 * D), dtype=torch.bfloat16, device="cuda")
    ctx.otas_layer_norm(x0, w["ln1_g"], w["ln1_b"], n, h)
    ctx.otas_linear(h, w["w_qkv"], w["b_qkv"], None, n, 3 * D, D, 0, qkv)
    metric = qkv[:, D:D + dh].contiguous()
    assert torch.equal(metric, qkv[:, D + dh:2 * D])
    ws = torch.empty(ctx.otas_merge_workspace_bytes(1, n), dtype=torch.uint8, device="cuda")
    xo, so = torch.empty((n, D), dtype=torch.bfloat16, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")
    src, dst = (torch.full((n,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    off = ctx.otas_token_merge(x0, metric, dh, None, [0, n], [r], ws, xo, so, src, dst)
    k = n - int(off[1])
    assert k == min(r, (n - cfg.n_lead) // 2)
    s, d = got["trace"][0][0]
    assert np.array_equal(np.asarray(s), src[:k].cpu().numpy()) and np.array_equal(np.asarray(d), dst[:k].cpu().numpy())
    ctx.close()
