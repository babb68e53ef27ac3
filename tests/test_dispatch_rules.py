"""Pure-host rules of the dispatch, through the built library (no GPU)."""
import ctypes
import os

import paper_2401_05031_amd as otas


def _library():
    if not os.path.exists(otas.lib_path()):
        from paper_2401_05031_amd import build
        build.build(verbose=False)
    return ctypes.CDLL(otas.lib_path())


def test_split_counts_of_the_second_linear_are_fixed():
    """How many partial products the MLP's second linear is summed from sets the order of additions, hence the bits of a
    pass: the counts are pinned on the rows a ViT-B pass with r = 16 has in its layers (batches of 1, 7, 24 and 64) and
    on some of ViT-L and ViT-H."""
    split = _library()._ZN4otas13splitk_factorEiliii
    split.argtypes = [ctypes.c_int, ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    split.restype = ctypes.c_int
    want = {(768, 3072, 1): [8] * 11,
            (768, 3072, 7): [6, 6, 6, 6, 6, 6, 8, 8, 8, 8, 8],
            (768, 3072, 24): [2, 2, 3, 3, 3, 4, 4, 4, 6, 6, 8],
            (768, 3072, 64): [1, 1, 1, 1, 1, 1, 1, 2, 3, 4, 6]}
    for (N, K, B), counts in want.items():
        assert [split(1, B * (197 - 16 * (l + 1)), N, K, 8) for l in range(11)] == counts, B
    assert [split(1, M, 1024, 4096, 8) for M in (128, 1000, 2000, 4000, 25216)] == [8, 8, 4, 2, 1]
    assert [split(1, M, 1280, 5120, 8) for M in (128, 1000, 2000, 4000, 67072)] == [8, 4, 2, 1, 1]
    assert split(1, 1344, 768, 3072, 4) == 4 and split(0, 1344, 768, 3072, 8) == 1 and split(1, 1344, 768, 1536, 8) == 1


class FusedPlan(ctypes.Structure):
    _fields_ = [("na", ctypes.c_int), ("nb", ctypes.c_int)]


def test_workgroups_of_the_selection():
    """Queries of 0 and 1 tokens have no pair to compare: not taken, whatever asks.  From 2 tokens on the selection has at
    least one workgroup and no more of either kind than there are blocks of 32 tokens."""
    how = _library()._ZN4otas18attention_plan_howEiiiiib
    how.argtypes = [ctypes.c_int] * 5 + [ctypes.c_bool]
    how.restype = FusedPlan
    for B in (1, 7, 200):
        for elsewhere in (False, True):
            for max_n in (-1, 0, 1, 1025):
                assert how(1, B, max_n, 256, 4, elsewhere).na == 0
        for max_n in (2, 3, 64, 65, 66, 197, 1024):
            p = how(1, B, max_n, 256, 4, True)
            assert 1 <= p.na <= ((max_n + 1) // 2 + 31) // 32 and 1 <= p.nb <= (max_n // 2 + 31) // 32


class AttnShape(ctypes.Structure):
    _fields_ = [("kc", ctypes.c_int), ("nw", ctypes.c_int), ("kg", ctypes.c_int), ("by_head", ctypes.c_bool)]


def test_how_attention_is_cut_up():
    """Waves share row blocks while every block has a CU of its own; 256 rows a workgroup beyond 256 rows, on its own, where every
    query has as many blocks and the rounds of the CUs are halved.  12 heads of width 64."""
    shape = _library()._ZN4otas15attention_shapeEiiiiii
    shape.argtypes, shape.restype = [ctypes.c_int] * 6, AttnShape

    def form(ns, others=0, H=12, dh=64):
        s = shape(dh, H, len(ns), max(ns), sum(-(-n // 128) for n in ns if 2 * n > max(ns)), others)
        return s.kc, s.nw, s.kg

    rows128, rows256 = (128, 4, 1), (256, 8, 1)
    assert [form([n]) for n in (64, 65, 128, 129, 577)] == [rows128] + [(128, 4, 4)] * 2 + [(256, 4, 4)] * 2
    assert [form([197] * B) for B in (3, 4, 5, 6, 10, 11)] == [(256, 4, 4)] + [(256, 8, 4)] * 2 + [rows128] * 2 + [rows256]
    assert [form([160] * B) for B in (4, 5, 7, 8, 10)] == [(256, 4, 4)] + [(256, 8, 4)] * 2 + [rows256] * 2 and form([161] * 8) == rows128
    assert [form([577] * B) for B in (1, 2, 3)] == [(256, 4, 4), (256, 8, 4), rows128]
    assert [form([400] * B) for B in (4, 5, 6, 10, 11, 16, 17, 21, 22, 26, 27, 32)] == \
        [rows128] * 2 + [rows256] * 2 + [rows128] * 2 + [rows256] * 2 + [rows128] * 2 + [rows256] * 2
    assert form([400] * 7 + [384]) == form([400, 197] * 4) == rows128 and form([400] * 7 + [385]) == rows256
    assert form([577] + [128] * 32) == form([197] + [98] * 64, H=16, dh=80)[:1] + (4, 1) == rows128   # few long ones in a full chip
    # beside a selection: not up to 256 rows
    assert form([197], 16) == rows256 and form([101], 16) == rows128 and form([577], 16) == (256, 4, 4) and form([400] * 5, 64) == rows256


def _choice():
    choice = _library()._ZN4otas20linear_kernel_choiceEiliii
    choice.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 3
    return choice


# the ids of otas_linear_kernel
K128, H160, H192, H224, H256, H288, H320, T64 = 3, 8, 4, 9, 5, 10, 6, 7


def test_kernels_of_the_products_of_a_block_are_fixed():
    """What the cost model picks for QKV, FC1, the projection and the second linear at a range of rows: a change of its
    constants shows here."""
    rows = (200, 700, 1500, 2600, 4000, 6000, 9000, 12000, 15000, 20000, 30000, 50000)
    want = {768: [[T64, T64, K128, K128, H160, H224, H192, H224, H288, H256, H288, H256],
                  [T64, T64, K128, K128, H192, H288, H224, H288, H256, H320, H288, H320],
                  [T64, T64, T64, T64, T64, K128, K128, H160, H192, H256, H192, H320],
                  [T64, T64, T64, T64, T64, K128, K128, H160, H192, H256, H192, H320]],
            1024: [[T64, T64, K128, K128, H192, H288, H224, H288, H256, H320, H288, H320],
                   [T64, T64, K128, H192, H256, H192, H288, H256, H320, H320, H320, H320],
                   [T64, T64, T64, T64, T64, K128, H160, H192, H256, H320, H256, H288],
                   [T64, T64, T64, T64, K128, K128, H160, H192, H256, H320, H256, H288]],
            1280: [[T64, T64, K128, H160, H256, H192, H288, H256, H320, H320, H320, H320],
                   [T64, K128, K128, H224, H160, H256, H256, H320, H320, H320, H320, H320],
                   [T64, T64, T64, K128, K128, K128, H192, H256, H320, H224, H320, H256],
                   [T64, T64, T64, K128, K128, K128, H192, H256, H320, H224, H320, H256]]}
    choice = _choice()
    for D, lists in want.items():
        products = [(3 * D, D, 0), (4 * D, D, 1), (D, D, 2), (D, 4 * D, 2)]
        assert [[choice(1, M, N, K, epi) for M in rows] for N, K, epi in products] == lists, D


def test_small_tiles_stay_within_four_workgroups_per_cu():
    """The 64 x 64 kernel's cost is known for up to 1024 tiles; past them it is not picked, whatever the width."""
    choice = _choice()
    for D in (128, 192, 256, 512, 768, 1280):
        for N, K, epi in ((3 * D, D, 0), (4 * D, D, 1), (D, D, 2), (D, 4 * D, 2)):
            most = 1024 // ((N + 63) // 64) * 64        # rows
            assert choice(1, most + 1, N, K, epi) != T64 and choice(1, 64, N, K, epi) == T64
            assert all(choice(1, M, N, K, epi) != T64 for M in (2 * most + 5, 10 * most, 100 * most))


def test_which_outputs_go_past_the_caches():
    """More than 160 MB always; behind GELU 16 to 64 MB if the model has more than 128 MB of weights."""
    streams = _library()._ZN4otas14streams_outputEliil
    streams.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int64]
    streams.restype = ctypes.c_bool
    MB, N = 1 << 20, 1024                            # 2 KB a row
    for epi in (0, 1):
        for model in (0, 128 * MB, 128 * MB + 1):
            large = epi == 1 and model > 128 * MB
            for mb, want in [(16, False), (64, large), (160, False)]:
                assert streams(mb * 512, N, epi, model) == want, (epi, model, mb)
            for mb, want in [(16, large), (64, False), (160, True)]:
                assert streams(mb * 512 + 1, N, epi, model) == want, (epi, model, mb)
