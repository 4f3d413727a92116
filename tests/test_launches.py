"""CPU-side checks of what the library launches: which kernels serve a call, that every launch stays
within the runtime's limits, and that scratch memory which was enough stays enough."""
import pytest

import launches as L
from paper_2503_00022_amd import binding as kv


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    from paper_2503_00022_amd import build
    build.ensure_built()
    recorder = L.build_recorder(tmp_path_factory.mktemp("recorder"))
    return lambda calls, lib=kv.LIB_PATH: L.record(recorder, lib, calls)


def up(n):
    return (n + 255) // 256 * 256


@pytest.mark.parametrize("B,Hq,Hkv,S,D,dtype", [
    (2, 8, 2, 300, 128, 1), (8, 32, 8, 2049, 128, 2), (4, 32, 8, 32768, 128, 1), (1, 8, 8, 131073, 64, 0),
    (1, 8, 8, 268000000, 64, 1),       # 2^23 blocks of 256 keys in 8 heads: side by side 2^32 threads and more
    (3, 2, 1, 2147483000, 128, 2),
])
def test_append_needs_one_pair_per_256_keys(record, B, Hq, Hkv, S, D, dtype):
    """The decoding step's scratch memory: a logit per query head and key, and a (maximum, sum) pair per
    query head and 256 keys.  That much is asked for, is enough, and a byte less is refused."""
    sh = kv.Shape(B, Hq, Hkv, S, D, dtype, 1)
    cap = (S + 15) // 16 * 16
    need = up(B * Hq * S * 4) + up(B * Hq * ((S + 255) // 256) * 8)
    assert kv.kvcrush_scores_append_workspace(sh, cap) == need
    (st, ran), (short, none) = record([L.append(sh, cap, need, 16), L.append(sh, cap, need - 1, 16)])
    assert st == kv.OK and short == kv.ERR_WORKSPACE and not none
    assert "append_logits" in ran[0].kernel and "append_update" in ran[1].kernel and len(ran) == 2


def kernels(ran):
    """The names of the launched kernels, without their template arguments."""
    import re
    return [re.search(r"(?<=\d)[a-z][a-z_]*_kernel", l.kernel).group(0) for l in ran]


@pytest.mark.parametrize("Hs,unit,B,S,budget,n_imp,rows,buckets", [
    # where the general kernels measured less, in whole or for one of the two steps (us, general / short)
    (1, 16, 64, 32768, 16384, 8192, "general", "general"),   # 86 / 148: 512 short vectors in each of 64 sequences
    (8, 2, 16, 8192, 2048, 1536, "general", "general"),      # 16-bit vectors
    (128, 2, 1, 2048, 512, 512, "general", "general"),       # 48 / 68: no representatives
    (128, 2, 1, 2048, 256, 0, "general", "short"),           # no importance to add up
    (8, 16, 1, 2048, 512, 384, "general", "short"),          # few tokens, few long vectors
    (4, 8, 4, 8192, 4096, 2048, "general", "short"),         # 256 buckets a sequence, 1024 in all
    (4, 8, 8, 8192, 4096, 2048, "general", "general"),       # 2048 in all
    # where the short path does
    (8, 16, 1, 32768, 1024, 768, "short", "short"),          # 72 / 46
    (128, 8, 1, 32768, 8192, 6144, "short", "short"),        # 422 / 312
    (1, 8, 1, 32768, 4096, 0, "short", "general"),           # 47 / 39
    (64, 8, 8, 8192, 2048, 2048, "short", "general"),        # more rows than compute units
])
def test_units_take_the_path_that_measured_less(record, Hs, unit, B, S, budget, n_imp, rows, buckets):
    a = kv.make_select_args(B, Hs, S, budget, n_imp, 0, "mean", 1, unit=unit)
    need = kv.kvcrush_select_workspace(a)
    (st, ran), (st2, less), (st3, static) = record([L.select(a, need), L.select(a, need - 1), L.select_static(a)])
    names = kernels(ran)
    assert st == kv.OK and ("row_select_kernel" in names) == (rows == "short")
    assert ("topk_mask_kernel" in names) == (rows == "general")
    assert ("medoid_units_emit_kernel" in names) == (buckets == "short") and ("emit_kernel" in names) == (buckets == "general")
    # with a byte less than is asked for: the general kernels, which need less
    assert st2 == kv.OK and kernels(less)[0] == "topk_mask_kernel" and kernels(less)[-1] == "emit_kernel"
    assert st3 in (kv.OK, kv.ERR_WORKSPACE)


def test_units_on_the_static_scratch_array(record):
    """kvcrush_select_static takes units whose queried size, which counts the faster kernels' tables, exceeds the
    array as long as the general kernels fit; tokens of that size are refused."""
    a = kv.make_select_args(8, 8, 32768, 4096, 3072, 0, "mean", 1, unit=16)
    tokens = kv.make_select_args(16, 8, 32768, 4096, 3072, 0, "mean", 1)
    large = kv.make_select_args(32, 8, 32768, 4096, 3072, 0, "mean", 1, unit=16)
    assert min(kv.kvcrush_select_workspace(x) for x in (a, tokens, large)) > kv.SELECT_STATIC_MAX_BYTES
    (st, ran), (st2, none), (st3, none3) = record([L.select_static(x) for x in (a, tokens, large)])
    assert st == kv.OK and kernels(ran)[0] == "topk_mask_kernel"
    assert st2 == st3 == kv.ERR_WORKSPACE and not none and not none3


@pytest.mark.parametrize("B,Hs,S,budget,n_imp,route", [
    # (us: general path / rows and tail apart / one launch)
    (1, 8, 512, 128, 64, ["select_one_kernel"]),                          # 21.0 / 10.1 / 8.2
    (2, 2, 700, 160, 120, ["select_one_kernel"]),                         # 20.4 / 9.7 / 8.9
    (1, 32, 512, 128, 64, ["row_select_kernel", "select_one_kernel"]),    # 28.1 / 11.9 / 13.7
    (1, 8, 2048, 512, 300, ["row_select_kernel", "select_one_kernel"]),   # 23.4 / 12.8 / 20.2
    (256, 8, 2048, 512, 300, ["select_one_kernel"]),                      # 99.6 / 36.6 / 24.0
    (1, 8, 4096, 1024, 512, ["row_select_kernel", "select_one_kernel"]),  # 24.9 / 17.3
    (1, 8, 512, 128, 128, ["select_one_kernel"]), (1, 32, 4096, 99, 99, ["row_select_kernel"]),  # the important tokens alone
    (1, 16, 8192, 99, 99, ["row_select_kernel"]), (1, 32, 8192, 99, 99, ["slice_hist_kernel", "row_select_kernel"]),
    (1, 4, 1300, 20, 10, ["row_select_kernel"] + 2 * ["group"] + ["medoid_emit_kernel"]),        # buckets of 129
    (1, 8, 8192, 2048, 1500, ["row_select_kernel"] + 2 * ["group"] + ["medoid_emit_kernel"]),    # 26.6, 24.4 without slices
    (1, 32, 8192, 2048, 1500, ["slice_hist_kernel", "row_select_kernel"] + 2 * ["group"] + ["medoid_emit_kernel"]),  # 35.7, 37.4
    (1, 8, 16384, 4096, 3072, ["slice_hist_kernel", "row_select_kernel"] + 2 * ["group"] + ["medoid_emit_kernel"]),  # 30.6, 32.6
])
def test_selection_takes_the_launches_that_measured_less(record, B, Hs, S, budget, n_imp, route):
    a = kv.make_select_args(B, Hs, S, budget, n_imp, 0, "mean", 1)
    need = kv.kvcrush_select_workspace(a)
    (st, ran), (st2, none), (st3, static) = record([L.select(a, need), L.select(a, need - 1), L.select_static(a)])
    assert st == kv.OK and st2 == kv.ERR_WORKSPACE and not none
    assert len(ran) == len(route) and all(k == r or r == "group" and k.startswith("group_") for k, r in zip(kernels(ran), route))
    assert st3 == kv.ERR_WORKSPACE or (st3 == kv.OK and static == ran)


@pytest.mark.parametrize("B,Hq,Hkv,S,D,dtype,rg,window,lse,colsum", [
    # (us, tiled / short, pass A and pass B)
    (32, 32, 8, 128, 128, 1, 1, 0, "tiled", "tiled"),     # 13 / 41, 21 / 20: many sequences of short prompts
    (128, 4, 4, 200, 128, 1, 1, 0, "tiled", "tiled"),     # 18 / 39, 19 / 40
    (8, 32, 32, 256, 64, 2, 0, 0, "tiled", "tiled"),      # 9 / 12, 10 / 12
    (2, 32, 8, 700, 128, 1, 1, 0, "tiled", "short"),      # 16 / 25, 29 / 16
    (1, 8, 8, 512, 64, 0, 0, 0, "short", "short"),        # 43 / 10, 45 / 10
    (2, 8, 2, 700, 128, 1, 1, 0, "short", "short"),       # 15 / 9, 28 / 15
    (1, 4, 4, 3000, 128, 0, 1, 0, "short", "short"),      # 393 / 67, 116 / 70
    (1, 4, 4, 4000, 64, 0, 1, 0, "short", "short"),       # 295 / 50, 69 / 52
    (8, 32, 8, 1024, 128, 1, 1, 0, "tiled", "tiled"),     # 44 / 176, 63 / 91
    (1, 32, 8, 16384, 128, 1, 1, 0, "tiled", "tiled"),
    (1, 4, 2, 700, 128, 1, 1, 64, "tiled", "tiled"),      # an observation window
    (1, 1, 1, 17600, 64, 0, 0, 0, "tiled", "tiled"),      # 151525 tiles: beyond what was measured
])
def test_scores_take_the_kernels_that_measured_less(record, B, Hq, Hkv, S, D, dtype, rg, window, lse, colsum):
    sh = kv.Shape(B, Hq, Hkv, S, D, dtype, rg, window)
    need = kv.kvcrush_scores_workspace(sh)
    other = kv.Shape(B, Hq, Hkv, S, D, dtype, 1 - rg, window)
    calls = [L.scores(sh, ws_bytes=need), L.scores(sh, lse=True, ws_bytes=need), L.row_lse(sh), L.row_lse(other), L.row_lse(sh, 0)]
    out = record(calls)
    assert all(st == kv.OK for st, _ in out)
    both, given, alone, alone2, bare = (kernels(ran) for _, ran in out)
    assert both[0] == alone[0] == alone2[0] == bare[0] == {"short": "lse_short_kernel", "tiled": "lse_kernel"}[lse]
    assert given[0] == {"short": "colsum_short_kernel", "tiled": "colsum_kernel"}[colsum] and given[0] in both
    # the normalisers do not depend on how the score rows are reduced, nor on who asks for them
    assert out[2][1] == out[3][1] == out[0][1][:len(out[2][1])]


def test_no_short_kernel_beyond_the_measured_sizes(record):
    """Of many sizes up to the largest that a call accepts: the short kernels' grids stay below 2^32 threads
    (the recorder refuses more, as the runtime does) and no prompt of 150000 tiles or more takes them."""
    import random
    rng = random.Random(4)
    shapes = []
    for _ in range(400):
        G, Hkv = rng.choice([1, 2, 3, 4, 8]), rng.choice([1, 2, 8, 32])
        B = rng.choice([1, 8, 64, 2000])
        shapes.append(kv.Shape(B, Hkv * G, Hkv, int(2 ** rng.uniform(0, 22)), rng.choice([64, 128]), rng.randint(0, 2), rng.randint(0, 1)))
    for sh, (st, ran) in zip(shapes, record([L.scores(sh) for sh in shapes])):
        n = (sh.S + 31) // 32
        short = any("short" in k for k in kernels(ran))
        assert not (short and sh.B * sh.Hq * n * (n + 1) // 2 > 150000)
        assert st == kv.OK or any(l.grid[0] * l.block > 0xFFFFFFFF for l in ran) or not ran


@pytest.mark.parametrize("B,Hq,Hkv,S,D,window,slices", [
    # pass A in us with that many slices a query block (one slice where it is not the choice)
    (1, 8, 2, 7000, 64, 0, 3),         # 56 (80): 220 blocks of up to 109 tiles
    (1, 8, 8, 6000, 128, 0, 3),        # 60 (76)
    (1, 4, 4, 11000, 128, 0, 3),       # 86 (134)
    (1, 32, 8, 2048, 128, 0, 1),       # 33 (40 with two): 256 blocks of up to 31 tiles
    (2, 24, 8, 16000, 128, 32, 10),    # 59 (183; 61 with four): a window, 48 blocks of 248 tiles
    (1, 12, 4, 16000, 128, 32, 42),    # 27 (182)
    (1, 32, 8, 16384, 128, 0, 1),      # more blocks than the chip takes at once
])
def test_slices_of_the_normaliser_pass(record, B, Hq, Hkv, S, D, window, slices):
    sh = kv.Shape(B, Hq, Hkv, S, D, 1, 1, window)
    (st, ran), (st2, bare) = record([L.row_lse(sh), L.row_lse(sh, 0)])
    assert st == st2 == kv.OK and kernels(bare) == ["lse_kernel"]
    assert ran[0].grid[0] == slices * bare[0].grid[0]
    assert kernels(ran) == ["lse_kernel"] + (["lse_combine_kernel"] if slices > 1 else [])


@pytest.mark.parametrize("B,Hq,Hkv,S,rg,cut", [
    (2, 32, 32, 2048, 0, False),       # 512 whole pieces of up to 32 steps: 57 us, 66 in pieces of up to 24
    (1, 32, 8, 2048, 1, True),         # 84 in pieces of 72 steps, 44
    (8, 32, 8, 1024, 1, True),         # 84, 71
    (1, 32, 8, 5000, 1, True),         # pieces of 72 steps: more than one a key block
])
def test_pieces_of_the_column_sums(record, B, Hq, Hkv, S, rg, cut):
    sh = kv.Shape(B, Hq, Hkv, S, 128, 1, rg)
    (st, ran), = record([L.scores(sh)])
    assert st == kv.OK and ("colsum_reduce_kernel" in kernels(ran)) == cut
    rows = B * (Hkv if rg else Hq)
    if not cut:
        assert [l.grid[0] for l in ran if "colsum_kernel" in l.kernel] == [rows * ((S + 255) // 256)]


@pytest.mark.parametrize("B,Hq,Hkv,S,D,rg,whole,cut", [
    # pass B in us, whole pieces -> cut for one a place of the chip
    (1, 16, 4, 5564, 128, 1, 272, 508),     # 120 -> 81
    (1, 32, 8, 4439, 128, 1, 368, 504),     # 118 -> 99
    (1, 8, 8, 8623, 128, 1, 416, 704),      # 107 -> 91
    (1, 32, 8, 4090, 128, 1, 352, 352),     # 94: 656 pieces take 102
    (1, 20, 5, 5145, 128, 1, 335, 335),     # 99: 525 take 113
    (1, 32, 8, 4003, 128, 1, 352, 352),     # 93: 528 take 103
    (1, 24, 3, 4286, 128, 1, 249, 249),     # 100: 357 take 109
    (1, 4, 4, 10880, 128, 1, 388, 628),     # 80 -> 74
    (1, 8, 8, 7720, 128, 1, 392, 856),      # 93 -> 75
    (1, 32, 32, 4096, 128, 0, 512, 512),    # every place taken by whole pieces
])
def test_pieces_fill_the_places_of_the_chip(record, B, Hq, Hkv, S, D, rg, whole, cut):
    sh = kv.Shape(B, Hq, Hkv, S, D, 1, rg)
    need = kv.kvcrush_scores_workspace(sh)
    (st, ran), (st2, less) = record([L.scores(sh, lse=True, ws_bytes=need), L.scores(sh, lse=True, ws_bytes=need - 1)])
    grid = lambda ls: [l.grid[0] for l in ls if "colsum_kernel" in l.kernel]
    assert st == kv.OK and grid(ran) == [cut]
    assert st2 == kv.ERR_WORKSPACE and not less if whole == cut else st2 == kv.OK and grid(less) == [whole]


@pytest.mark.parametrize("B,H,S,window,wgs,lse_turn,colsum_turn", [
    # a score row a head: workgroups of pass A, and the first piece of each row that runs in turned order (None: none)
    (1, 32, 3584, 0, 448, 8, None), (1, 32, 4096, 0, 512, 8, 8), (1, 32, 4097, 0, 544, None, None),
    (1, 3, 38100, 0, 447, None, None), (1, 37, 3300, 0, 481, 7, 7), (3, 8, 5100, 0, 480, 11, None),
    (3, 27, 1500, 0, 486, None, 4),           # 24 tiles are the least: 20 before the last block, 24 to the whole sequence
    (1, 32, 4096, 4000, 512, None, None),     # a window's pieces do not fall evenly
])
def test_order_of_the_workgroups(record, B, H, S, window, wgs, lse_turn, colsum_turn):
    """Launches of 448 to 512 workgroups of falling lengths start the second 256 in turned order, from the first piece
    that lies wholly behind them."""
    sh = kv.Shape(B, H, H, S, 128, 1, 0, window)
    (st, lse), (st2, ran) = record([L.row_lse(sh, 0), L.scores(sh, lse=True)])
    assert st == st2 == kv.OK and lse[0].grid[0] == wgs
    for launch, turn in ((lse[0], lse_turn), (ran[0], colsum_turn)):
        length, n_bh, n_pieces, got = launch.order
        assert (length, n_bh, n_pieces * n_bh) == (S, B * H, launch.grid[0])
        assert got == (n_pieces if turn is None else turn)
        if turn is not None:
            assert (turn - 1) * n_bh < 256 <= turn * n_bh


def test_the_sizes_of_the_tiled_tests_are_tiled(record):
    """test_gpu_parity.py's cases for the tiled kernels run those, whatever the rules become."""
    from test_gpu_parity import EXTREME_TILED, TILED_CASES
    code = {"f32": kv.F32, "bf16": kv.BF16, "f16": kv.F16}
    cases = [(c[:7], c[7:]) for c in TILED_CASES]
    cases += [((1, Hq, Hkv, S, D, dt, rg), None) for Hq, Hkv, S, D, dt in EXTREME_TILED for rg in (0, 1)]
    cases.append(((1, 8, 2, 7000, 128, "bf16", True), (True, True)))       # test_scores_deterministic
    out = record([L.scores(kv.Shape(B, Hq, Hkv, S, D, code[dt], int(rg))) for (B, Hq, Hkv, S, D, dt, rg), _ in cases])
    for (shape, expected), (st, ran) in zip(cases, out):
        names = kernels(ran)
        assert st == kv.OK and {"lse_kernel", "colsum_kernel"} <= set(names), shape
        if expected:
            assert ("lse_combine_kernel" in names, "colsum_reduce_kernel" in names) == expected, shape


def test_scores_with_less_scratch_than_the_finer_pieces_need(record):
    """One buffer for prompts of several lengths, sized for the longest: a shorter prompt that asks for more is
    cut coarser, with the same kernels otherwise; what even that needs is the limit."""
    for B, Hq, Hkv, S in [(1, 32, 8, 2100), (1, 32, 8, 1500), (2, 8, 8, 3500), (1, 4, 4, 4400)]:
        sh = kv.Shape(B, Hq, Hkv, S, 128, kv.BF16, 1)
        need = kv.kvcrush_scores_workspace(sh)
        (st, fine), (st2, coarse) = record([L.scores(sh, ws_bytes=need), L.scores(sh, ws_bytes=need - 1)])
        assert st == st2 == kv.OK and len({k for k in kernels(fine) + kernels(coarse) if k.startswith("lse")} & {"lse_kernel", "lse_short_kernel"}) == 1
        if "colsum_kernel" in kernels(fine):
            grid = lambda ran: [l.grid[0] for l in ran if "colsum_kernel" in l.kernel][0]
            assert grid(coarse) < grid(fine)
        else:
            assert fine == coarse
        (st3, none), = record([L.scores(sh, ws_bytes=B * Hq * S * 4 - 1)])
        assert st3 == kv.ERR_WORKSPACE and not none
