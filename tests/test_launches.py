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


def test_append_logits_in_two_steps_from_1024_workgroups_on(record):
    """The sizes of test_gpu_parity.py's test of the same name, on either side of the line."""
    calls = [L.append(kv.Shape(B, Hq, Hkv, S, D, dt, 1), S) for B, Hq, Hkv, S, D, dt in [
        (16, 8, 8, 2049, 128, 1), (32, 160, 4, 2176, 64, 2), (16, 16, 8, 2177, 64, 1), (15, 8, 8, 2049, 128, 1), (14, 8, 8, 2049, 128, 1)]]
    blocks = [ran[0].block for _, ran in record(calls)]
    assert blocks == [256, 256, 256, 256, 512]


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


@pytest.mark.parametrize("B,Hq,Hkv,S,D,window,slices", [
    # pass A in us with that many slices a query block (one slice where it is not the choice)
    (1, 8, 2, 7000, 64, 0, 3),         # 56 (80): 220 blocks of up to 109 tiles
    (1, 8, 8, 6000, 128, 0, 3),        # 60 (76)
    (1, 4, 4, 11000, 128, 0, 3),       # 86 (134)
    (1, 32, 8, 2048, 128, 0, 1),       # 33 (40 with two): 256 blocks of up to 31 tiles
    (2, 24, 8, 16000, 128, 32, 10),    # 59 (183; 63 with five): a window, 48 blocks of 248 tiles
    (1, 12, 4, 16000, 128, 32, 42),    # 28 (182)
    (1, 32, 8, 16384, 128, 0, 1),      # more blocks than the chip takes at once
])
def test_slices_of_the_normaliser_pass(record, B, Hq, Hkv, S, D, window, slices):
    sh = kv.Shape(B, Hq, Hkv, S, D, 1, 1, window)
    (st, ran), (st2, bare) = record([L.row_lse(sh), L.row_lse(sh, 0)])
    assert st == st2 == kv.OK and kernels(bare) == ["lse_kernel"]
    assert ran[0].grid[0] == slices * bare[0].grid[0]
    assert kernels(ran) == ["lse_kernel"] + (["lse_combine_kernel"] if slices > 1 else [])


@pytest.mark.parametrize("B,Hq,Hkv,S,rg,cut", [
    (2, 32, 32, 2048, 0, False),       # 512 whole pieces of up to 32 steps: 58 us, 65 in pieces of up to 24
    (1, 32, 8, 2048, 1, True),         # 65 uncut, 41
    (8, 32, 8, 1024, 1, True),         # 61 uncut, 51
    (1, 32, 8, 5000, 1, True),         # pieces of 72 steps: more than one a key block
])
def test_pieces_of_the_column_sums(record, B, Hq, Hkv, S, rg, cut):
    sh = kv.Shape(B, Hq, Hkv, S, 128, 1, rg)
    (st, ran), = record([L.scores(sh)])
    assert st == kv.OK and ("colsum_reduce_kernel" in kernels(ran)) == cut
    rows = B * (Hkv if rg else Hq)
    if not cut:
        assert [l.grid[0] for l in ran if "colsum_kernel" in l.kernel] == [rows * ((S + 255) // 256)]
