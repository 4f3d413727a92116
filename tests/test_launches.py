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
