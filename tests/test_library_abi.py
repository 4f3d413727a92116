"""CPU-side checks of the C-ABI library: it loads, exports every function the
header declares, and rejects bad arguments on the host before any launch (no
compute call is made here)."""
import ctypes
import os
import re

import pytest

from paper_2503_00022_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "kvcrush.h")


@pytest.fixture(scope="module")
def lib():
    from paper_2503_00022_amd import build
    build.ensure_built()
    return binding.load()


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(kvcrush_[a-z_0-9]+)\s*\(", text)))


def test_header_functions_are_exported(lib):
    names = declared_functions()
    assert set(names) == set(binding.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None


def test_version_and_status_strings(lib):
    assert binding.kvcrush_version() >= 100
    assert binding.status_string(0) == "ok"
    for s in range(1, 5):
        assert binding.status_string(s) not in ("ok", "unknown status")
    assert binding.status_string(99) == "unknown status"


def test_workspace_sizes(lib):
    sh = binding.Shape(1, 32, 8, 16384, 128, binding.BF16, 1)
    assert binding.kvcrush_scores_workspace(sh) >= 32 * 16384 * 4
    assert binding.kvcrush_scores_workspace(binding.Shape(1, 30, 8, 16, 128, 1, 1)) == 0   # Hq % Hkv != 0
    a = binding.make_select_args(1, 8, 16384, 4096, 3072)
    need = binding.kvcrush_select_workspace(a)
    nw = 16384 // 64
    assert need >= (9 * nw + nw) * 8 + 16384 * 4 + 16384 * 8
    assert binding.kvcrush_select_workspace(binding.make_select_args(1, 8, 100, 101, 5)) == 0  # budget > S


FAKE = ctypes.c_void_p(0x1000)  # aligned, never dereferenced: validation fails first


def test_scores_rejects_bad_arguments(lib):
    def call(shape, q=FAKE, k=FAKE, lse=None, scores=FAKE, ws=FAKE, ws_bytes=1 << 40):
        return lib.kvcrush_scores(ctypes.byref(shape), q, k, lse, scores, ws, ws_bytes, None)

    good = dict(B=1, Hq=4, Hkv=2, S=64, D=128, dtype=1, reduce_groups=0)

    def shape(**kw):
        d = dict(good, **kw)
        return binding.Shape(d["B"], d["Hq"], d["Hkv"], d["S"], d["D"], d["dtype"], d["reduce_groups"])

    assert call(shape(S=0)) == binding.ERR_INVALID_ARG
    assert call(shape(Hq=5)) == binding.ERR_INVALID_ARG
    assert call(shape(dtype=7)) == binding.ERR_INVALID_ARG
    assert call(shape(dtype=3)) == binding.ERR_INVALID_ARG
    assert call(shape(reduce_groups=2)) == binding.ERR_INVALID_ARG
    assert call(shape(D=96)) == binding.ERR_UNSUPPORTED
    assert call(shape(), q=None) == binding.ERR_INVALID_ARG
    assert call(shape(), q=ctypes.c_void_p(0x1004)) == binding.ERR_INVALID_ARG      # misaligned
    assert call(shape(), ws=None) == binding.ERR_WORKSPACE
    assert call(shape(), ws_bytes=16) == binding.ERR_WORKSPACE
    # memory layouts: all-zero strides are the packed layout; otherwise positive multiples of 16 bytes
    def strided(q=(0, 0, 0), k=(0, 0, 0), **kw):
        sh = shape(**kw)
        sh.q_stride[:], sh.k_stride[:] = q, k
        return sh
    # (accepted layouts are probed through the size query: no call here may reach a launch)
    assert lib.kvcrush_scores_workspace(ctypes.byref(strided(q=(64 * 4 * 128, 128, 4 * 128)))) > 0   # [B,S,Hq,D]
    assert lib.kvcrush_scores_workspace(ctypes.byref(strided(q=(64 * 4 * 128, 128, 0)))) == 0
    assert call(strided(q=(64 * 4 * 128, 128, 0))) == binding.ERR_INVALID_ARG          # partly given
    assert call(strided(k=(64 * 2 * 128, 128, 127))) == binding.ERR_INVALID_ARG        # rows overlap their own values
    assert call(strided(k=(64 * 2 * 128, 132, 2 * 128))) == binding.ERR_INVALID_ARG    # head stride not 16-byte
    assert call(strided(q=(-1, 128, 512))) == binding.ERR_INVALID_ARG
    assert call(strided(q=(1 << 30, 128, 1 << 24))) == binding.ERR_INVALID_ARG         # token stride over 2^24 bytes
    # launch-size limits: refused on the host, before anything is enqueued
    assert call(shape(B=70000, Hq=1, Hkv=1)) == binding.ERR_UNSUPPORTED               # second grid dimension
    assert call(shape(B=1, Hq=32, Hkv=8, S=1 << 24, reduce_groups=1), ws_bytes=1 << 62) == binding.ERR_UNSUPPORTED   # pass-B pieces
    assert call(shape(B=4096, Hq=8, Hkv=8, S=1 << 24), ws_bytes=1 << 62) == binding.ERR_UNSUPPORTED     # pass-A blocks


def test_select_rejects_bad_arguments(lib):
    def call(args, scores=FAKE, idx=FAKE, ws=FAKE, ws_bytes=1 << 40):
        return lib.kvcrush_select(ctypes.byref(args), scores, idx, None, None, ws, ws_bytes, None)

    mk = binding.make_select_args
    assert call(mk(1, 8, 100, 101, 10)) == binding.ERR_INVALID_ARG           # budget > S
    assert call(mk(1, 8, 100, 50, 51)) == binding.ERR_INVALID_ARG            # n_important > budget
    assert call(mk(1, 8, 100, 50, 10, bit_topk=101)) == binding.ERR_INVALID_ARG
    assert call(mk(1, 0, 100, 50, 10)) == binding.ERR_INVALID_ARG
    assert call(mk(1, 1025, 100, 50, 10)) == binding.ERR_UNSUPPORTED         # more than 1024 bits per vector
    assert call(mk(1, 64, 128, 64, 32, unit=32)) == binding.ERR_UNSUPPORTED  # 64 rows x 32 tokens = 2048 bits
    assert call(mk(1, 8, 100, 48, 16, unit=8)) == binding.ERR_INVALID_ARG    # 100 tokens are not whole units
    assert call(mk(1, 8, 96, 50, 16, unit=8)) == binding.ERR_INVALID_ARG     # nor is a budget of 50
    assert call(mk(1, 8, 96, 48, 12, unit=8)) == binding.ERR_INVALID_ARG     # nor 12 important tokens
    assert call(mk(1, 8, 96, 48, 16, unit=-2)) == binding.ERR_INVALID_ARG
    assert call(mk(1, 8, 100, 50, 10, anchor=9)) == binding.ERR_INVALID_ARG
    assert call(mk(1, 8, 100, 50, 10, anchor="explicit")) == binding.ERR_INVALID_ARG  # no anchor_bits
    # the grouping's counter table must fit a workgroup's LDS: (bits + 1) x 4 x ceil(items / 1024) <= 30720
    big = mk(1, 128, 70000, 1000, 500)
    assert binding.kvcrush_select_workspace(big) == 0 and call(big) == binding.ERR_UNSUPPORTED
    assert binding.kvcrush_select_workspace(mk(1, 128, 60000, 1000, 500)) > 0
    assert binding.kvcrush_select_workspace(mk(1, 8, 900000, 1000, 500)) == 0
    assert binding.kvcrush_select_workspace(mk(1, 8, 800000, 1000, 500)) > 0
    assert call(mk(1, 8, 100, 50, 10), scores=None) == binding.ERR_INVALID_ARG
    assert call(mk(1, 8, 100, 50, 10), ws=None) == binding.ERR_WORKSPACE
    assert call(mk(1, 8, 100, 50, 10), ws_bytes=64) == binding.ERR_WORKSPACE


def test_compact_rejects_bad_arguments(lib):
    def call(B=1, Hkv=2, S=64, D=128, dtype=1, budget=16, k=FAKE, v=FAKE, idx=FAKE, bt=None, bs=16,
             ko=FAKE, vo=FAKE):
        return lib.kvcrush_compact(B, Hkv, S, D, dtype, budget, k, v, idx, bt, bs, ko, vo, None)

    assert call(budget=65) == binding.ERR_INVALID_ARG
    assert call(budget=-1) == binding.ERR_INVALID_ARG
    assert call(dtype=3) == binding.ERR_INVALID_ARG
    assert call(dtype=2, k=None) == binding.ERR_INVALID_ARG     # fp16 is a known type; the null pointer is not
    assert call(D=4) == binding.ERR_UNSUPPORTED                 # 8-byte rows cannot be moved as 16-byte vectors
    assert call(k=None) == binding.ERR_INVALID_ARG
    assert call(ko=ctypes.c_void_p(0x1008)) == binding.ERR_INVALID_ARG
    assert call(S=70, bt=FAKE, bs=16) == binding.ERR_INVALID_ARG  # S not a multiple of the block size
    assert call(budget=0, k=None, v=None, idx=None, ko=None, vo=None) == binding.OK   # nothing to do


def test_score_kernels_keep_their_registers():
    """The hand-scheduled kernels of stage 1 are built for two waves per SIMD with
    no register spills; either one slipping costs a multiple of their run time
    and no numerical test would notice."""
    from paper_2503_00022_amd import build
    report = build.resource_usage("scores.hip")
    hot = {name: r for name, r in report.items() if "lse_kernel" in name or "colsum_kernel" in name}
    assert len(hot) == 24, sorted(report)          # {lse, colsum} x {bf16, fp16, fp32} x {D = 64, 128} x {packed, strided}
    for name, r in hot.items():
        assert r["VGPRs Spill"] == 0 and r["SGPRs Spill"] == 0 and r["ScratchSize"] == 0, (name, r)
        assert r["Occupancy"] >= 2, (name, r)
        assert r["LDS Size"] <= 80 * 1024, (name, r)   # two workgroups share a compute unit's 160 KiB


def test_short_prompt_and_decoding_kernels_keep_their_registers():
    """The same for the short-prompt kernels, whose stationary rows and closing sums are arrays that only
    stay in registers while every index is known, and for the decoding step's matrix-core kernel."""
    from paper_2503_00022_amd import build
    short = {n: r for n, r in build.resource_usage("scores.hip").items() if "_short_kernel" in n}
    assert len(short) == 24, sorted(short)         # {lse, colsum} x {bf16, fp16, fp32} x {D = 64, 128} x {packed, strided}
    for name, r in short.items():
        assert r["VGPRs Spill"] == 0 and r["SGPRs Spill"] == 0 and r["ScratchSize"] == 0, (name, r)
        assert r["LDS Size"] <= 160 * 1024, (name, r)       # one workgroup of eight (fp32, D = 128: four) waves a compute unit
        assert r["Occupancy"] >= 1, (name, r)
    append = {n: r for n, r in build.resource_usage("decode.hip").items() if "append_" in n}
    assert len([n for n in append if "mfma" in n]) == 4, sorted(append)   # {bf16, fp16} x {D = 64, 128}
    for name, r in append.items():
        assert r["VGPRs Spill"] == 0 and r["SGPRs Spill"] == 0 and r["ScratchSize"] == 0, (name, r)
        assert "mfma" not in name or (r["Occupancy"] >= 4 and r["LDS Size"] <= 80 * 1024), (name, r)


def test_struct_layouts_match_the_header(tmp_path):
    """The ctypes mirrors of the header's structs have the C compiler's sizes and
    field offsets (a C program that includes the header prints them)."""
    import subprocess
    structs = {"kvcrush_shape": binding.Shape, "kvcrush_select_args": binding.SelectArgs}
    lines = []
    for cname, cls in structs.items():
        lines.append(f'printf("{cname} %zu\\n", sizeof({cname}));')
        for fname, _ in cls._fields_:
            lines.append(f'printf("{cname}.{fname} %zu\\n", offsetof({cname}, {fname}));')
    src = tmp_path / "layout.c"
    src.write_text('#include <stdio.h>\n#include <stddef.h>\n#include "kvcrush.h"\nint main(void) {\n'
                   + "\n".join(lines) + "\nreturn 0; }\n")
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-std=c99", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)],
                   check=True)
    out = dict(l.split() for l in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines())
    for cname, cls in structs.items():
        assert int(out[cname]) == ctypes.sizeof(cls)
        for fname, _ in cls._fields_:
            assert int(out[f"{cname}.{fname}"]) == getattr(cls, fname).offset, (cname, fname)
    # and the header names no field the mirror lacks
    text = re.sub(r"/\*.*?\*/", "", open(HEADER).read(), flags=re.S)
    for cname, cls in structs.items():
        body = re.search(r"typedef struct \{([^{}]*)\} " + cname + ";", text).group(1)
        names = re.findall(r"(\w+)\s*(?:\[\d+\])?\s*[,;]", body)
        assert names == [f for f, _ in cls._fields_], (cname, names)


def test_select_protected_ends_validation(lib):
    def ws(**kw):
        d = dict(B=1, Hs=8, S=1000, budget=200, n_important=100, n_sink=32, n_recent=64)
        d.update(kw)
        return binding.kvcrush_select_workspace(binding.make_select_args(
            d["B"], d["Hs"], d["S"], d["budget"], d["n_important"], n_sink=d["n_sink"], n_recent=d["n_recent"]))
    assert ws() > 0
    assert ws(n_sink=150, n_recent=51) == 0        # protected tokens exceed the budget
    assert ws(n_important=105) == 0                # more important tokens than the middle's budget
    assert ws(n_sink=-1) == 0
    assert ws(n_sink=100, n_recent=100, n_important=0) > 0   # budget == protected: legal
    # the workspace is sized by the middle, which is never longer than the sequence
    assert ws() <= ws(n_sink=0, n_recent=0)


def make_shape(base, overrides):
    d = dict(base, **overrides)
    shape = binding.Shape(*[d.get(f, 0) for f, _ in binding.Shape._fields_ if not f.endswith("_stride")])
    for f in ("q_stride", "k_stride"):
        getattr(shape, f)[:] = d.get(f, (0, 0, 0))
    return shape


def test_window_pool_and_row_lse_validation(lib):
    sh = lambda **kw: make_shape(dict(B=1, Hq=4, Hkv=2, S=4096, D=128, dtype=1, reduce_groups=1, obs_window=0), kw)
    # a window shrinks the partial-sum part of the workspace, never grows the total past the full one
    assert 0 < binding.kvcrush_scores_workspace(sh(obs_window=64)) <= binding.kvcrush_scores_workspace(sh()) + (1 << 20)
    assert binding.kvcrush_scores_workspace(sh(obs_window=-1)) == 0
    assert binding.kvcrush_scores_workspace(sh(softmax_scale=-0.5)) == 0
    assert binding.kvcrush_scores_workspace(sh(softmax_scale=float("nan"))) == 0
    assert binding.kvcrush_scores_workspace(sh(softmax_scale=0.102)) == binding.kvcrush_scores_workspace(sh())
    # few heads: the normaliser pass wants scratch memory for key slices
    assert binding.kvcrush_row_lse_workspace(sh(obs_window=64)) > 0
    assert binding.kvcrush_row_lse_workspace(sh(B=8, Hq=32, Hkv=8, S=16384)) == 0      # enough workgroups already
    assert binding.kvcrush_row_lse_workspace(sh(dtype=0, obs_window=64)) == 0          # fp32 path never slices
    call = lambda shape, ws, n: lib.kvcrush_row_lse(ctypes.byref(shape), FAKE, FAKE, FAKE, ws, n, None)
    assert call(sh(obs_window=64), FAKE, 16) == binding.ERR_WORKSPACE
    assert call(sh(obs_window=64), ctypes.c_void_p(0x1004), 1 << 40) == binding.ERR_WORKSPACE
    assert call(sh(D=96), None, 0) == binding.ERR_UNSUPPORTED
    pool = lambda rows=2, S=64, kernel=3, a=FAKE, b=ctypes.c_void_p(0x100000): \
        lib.kvcrush_pool_scores(rows, S, kernel, a, b, None)
    assert pool(kernel=2) == binding.ERR_INVALID_ARG
    assert pool(kernel=1025) == binding.ERR_INVALID_ARG
    assert pool(S=0) == binding.ERR_INVALID_ARG
    assert pool(b=FAKE) == binding.ERR_INVALID_ARG                       # in place
    assert pool(b=ctypes.c_void_p(0x1000 + 256)) == binding.ERR_INVALID_ARG   # overlapping
    assert pool(a=None) == binding.ERR_INVALID_ARG
    assert pool(rows=0, a=None, b=None) == binding.OK


def test_decode_entry_points_validation(lib):
    sh = lambda **kw: make_shape(dict(B=2, Hq=8, Hkv=2, S=300, D=128, dtype=1, reduce_groups=1, obs_window=0), kw)
    need = binding.kvcrush_scores_append_workspace(sh(), 320)
    assert need >= 2 * 8 * 300 * 4
    assert binding.kvcrush_scores_append_workspace(sh(), 299) == 0        # capacity below the valid length
    assert binding.kvcrush_scores_append_workspace(sh(obs_window=8), 320) == 0
    call = lambda shape, cap=320, q=FAKE, k=FAKE, sc=FAKE, ws=FAKE, n=1 << 40, bt=None, bs=16: \
        lib.kvcrush_scores_append(ctypes.byref(shape), cap, None, q, k, bt, bs, sc, ws, n, None)
    assert call(sh(), cap=100) == binding.ERR_INVALID_ARG
    assert call(sh(Hq=7)) == binding.ERR_INVALID_ARG
    assert call(sh(D=32)) == binding.ERR_UNSUPPORTED
    assert call(sh(), q=None) == binding.ERR_INVALID_ARG
    assert call(sh(), k=ctypes.c_void_p(0x1002)) == binding.ERR_INVALID_ARG
    assert call(sh(), ws=None) == binding.ERR_WORKSPACE
    assert call(sh(), n=need - 1) == binding.ERR_WORKSPACE
    assert call(sh(), cap=330, bt=FAKE, bs=16) == binding.ERR_INVALID_ARG     # capacity is not whole blocks
    assert call(sh(), bt=FAKE, bs=0) == binding.ERR_INVALID_ARG
    other = ctypes.c_void_p(0x200000)
    cc = lambda B=1, Hkv=2, Hs=2, D=128, dtype=1, cs=100, cd=80, budget=40, k=FAKE, v=FAKE, sc=FAKE, idx=FAKE, \
        ko=other, vo=other, so=other: lib.kvcrush_compact_cache(B, Hkv, Hs, D, dtype, cs, cd, budget, k, v, sc, idx,
                                                                 ko, vo, so, None)
    assert cc(budget=81) == binding.ERR_INVALID_ARG          # does not fit the destination
    assert cc(budget=101, cd=200) == binding.ERR_INVALID_ARG  # more than the source holds
    assert cc(dtype=5) == binding.ERR_INVALID_ARG
    assert cc(D=4) == binding.ERR_UNSUPPORTED
    assert cc(ko=FAKE) == binding.ERR_INVALID_ARG            # in place
    assert cc(sc=None) == binding.ERR_INVALID_ARG
    assert cc(budget=0, k=None, v=None, sc=None, idx=None, ko=None, vo=None, so=None) == binding.OK
    cb = lambda B=1, S=64, budget=32, bs=16, idx=FAKE, bt=FAKE, out=other: \
        lib.kvcrush_compact_block_table(B, S, budget, bs, idx, bt, out, None)
    assert cb(budget=40) == binding.ERR_INVALID_ARG          # not whole blocks
    assert cb(S=70) == binding.ERR_INVALID_ARG
    assert cb(out=None) == binding.ERR_INVALID_ARG
    assert cb(budget=0, idx=None, bt=None, out=None) == binding.OK
    # strided score rows in the selection
    mk = binding.make_select_args
    assert binding.kvcrush_select_workspace(mk(1, 8, 100, 50, 10, score_stride=99)) == 0
    assert binding.kvcrush_select_workspace(mk(1, 8, 100, 50, 10, score_stride=128)) > 0


def test_decode_step_validation(lib):
    sh = lambda **kw: make_shape(dict(B=2, Hq=8, Hkv=2, S=300, D=128, dtype=1, reduce_groups=1, obs_window=0), kw)
    need = binding.kvcrush_scores_append_workspace(sh(), 320)
    call = lambda shape, cap=320, q=FAKE, kn=FAKE, vn=FAKE, k=FAKE, v=FAKE, sc=FAKE, ws=FAKE, n=1 << 40: \
        lib.kvcrush_decode_step(ctypes.byref(shape), cap, q, kn, vn, k, v, sc, ws, n, None)
    for name in ("q", "kn", "vn", "k", "v", "sc"):
        assert call(sh(), **{name: None}) == binding.ERR_INVALID_ARG
        assert call(sh(), **{name: ctypes.c_void_p(0x1002)}) == binding.ERR_INVALID_ARG
    assert call(sh(), cap=100) == binding.ERR_INVALID_ARG
    assert call(sh(D=32)) == binding.ERR_UNSUPPORTED
    assert call(sh(), ws=None) == call(sh(), n=need - 1) == binding.ERR_WORKSPACE


def test_pipeline_classes_validate_before_touching_the_gpu(lib):
    """The buffer-owning wrappers import without a GPU and reject a capacity that cannot hold the cache."""
    import torch
    from paper_2503_00022_amd import pipeline
    k = torch.zeros(1, 2, 8, 64, dtype=torch.bfloat16)
    sc = torch.zeros(1, 2, 8)
    with pytest.raises(ValueError):
        pipeline.DecodeCache(k, k, sc, budget=8, n_important=4, capacity=8)
    with pytest.raises(ValueError):
        pipeline.DecodeCache(k, k, sc, budget=4, n_important=2, capacity=6)
    with pytest.raises(RuntimeError):
        lc = object.__new__(pipeline.LayerCompressor)      # no buffers: only the guard is exercised
        lc._graph = None
        lc.replay()


def test_decode_cache_in_host_memory_is_refused(lib, monkeypatch):
    """A cache and rows in host memory: an append raises, and no host address is handed to the library."""
    import torch
    from paper_2503_00022_amd import pipeline
    monkeypatch.setattr(binding, "_decode_step", lambda *a, **kw: pytest.fail("host addresses given to the library"))
    k = torch.zeros(1, 2, 8, 64, dtype=torch.bfloat16)
    cache = pipeline.DecodeCache(k, k, torch.zeros(1, 2, 8), budget=4, n_important=2, capacity=16)
    with pytest.raises(ValueError, match="GPU memory"):
        cache.append(torch.zeros(1, 8, 64, dtype=torch.bfloat16), k[:, :, 0].contiguous(), k[:, :, 0].contiguous())
    assert cache.n == 8 and cache._append_ws is None       # no longer than before, and no workspace in host memory kept


def test_decode_step_refuses_any_tensor_in_host_memory(lib, monkeypatch):
    """Each operand of the step, the workspace included, has to live in GPU memory."""
    import torch

    class OnGpu(torch.Tensor):          # host memory that says otherwise: nothing here gets as far as a kernel
        device = torch.device("cuda", 0)

    monkeypatch.setattr(binding, "_decode_step", lambda *a, **kw: pytest.fail("host addresses given to the library"))
    mk = lambda *s, dtype=torch.bfloat16: torch.zeros(*s, dtype=dtype)
    args = dict(q_new=mk(1, 8, 64), k_new=mk(1, 2, 64), v_new=mk(1, 2, 64), k_cache=mk(1, 2, 16, 64), v_cache=mk(1, 2, 16, 64),
                scores_cache=mk(1, 2, 16, dtype=torch.float32), workspace=mk(4096, dtype=torch.uint8))
    for name in args:
        given = {n: t if n == name else t.as_subclass(OnGpu) for n, t in args.items()}
        with pytest.raises(ValueError, match=f"{name} must live in GPU memory"):
            binding.kvcrush_decode_step(**given, S=9, reduce_groups=True)


def test_calibration_library_is_separate_from_the_product():
    """The benchmark's calibration kernel is built into a library of its own; the product library
    exports nothing of it."""
    from paper_2503_00022_amd import build
    build.ensure_built()
    bench = ctypes.CDLL(build.BENCH_LIB_PATH)
    assert hasattr(bench, "kvcrush_bench_mfma_ceiling") and hasattr(bench, "kvcrush_bench_mfma_operand_bytes")
    bench.kvcrush_bench_mfma_operand_bytes.restype = ctypes.c_size_t
    assert bench.kvcrush_bench_mfma_operand_bytes() == 64 * 1024
    bench.kvcrush_bench_mfma_ceiling.restype = ctypes.c_double
    bench.kvcrush_bench_mfma_ceiling.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32, ctypes.c_void_p,
                                                 ctypes.c_void_p]
    assert bench.kvcrush_bench_mfma_ceiling(None, 1, 1, None, None) == 0.0       # refused before any launch
    product = binding.load()
    assert not hasattr(product, "kvcrush_bench_mfma_ceiling")


def test_mix_calibration_kernel_keeps_its_matrix_instructions(tmp_path):
    """The mix ceiling is quoted in matrix FLOP/s: its loop must really hold 32 MFMAs (two 64 x 32
    blocks) and 64 each of fma / exp2 / add per trip.  Its operands never change, so a compiler that
    is allowed to would compute one block and reuse it; the count is checked in the generated code."""
    import subprocess
    from paper_2503_00022_amd import build
    src = os.path.join(build.CSRC, "bench", "mix_ceiling.hip")
    out = tmp_path / "mix.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-S", "-o", str(out), src],
                   check=True, capture_output=True)
    text = out.read_text()
    body = text[text.index("mix_ceiling_kernel"):]
    body = body[:body.index("s_endpgm")]
    assert body.count("v_mfma_f32_32x32x16_bf16") == 32
    assert body.count("v_exp_f32") == 64 and body.count("v_fma_f32") >= 64


def test_score_loops_wait_only_where_they_must(tmp_path):
    """The pipelined loops of the two score kernels (16-bit operands) hold 96 MFMAs a trip (three
    unrolled steps).  Their tile copies are kept out of the compiler's sight so that it does not
    wait for them at the next LDS read: inside a trip there is one `vmcnt(0)` per step (the loop's
    own, before its barrier) and no LDS wait that drains every read in flight except the one that
    goes with each barrier.  A compiler or source change that brings the conservative waits back
    costs several per cent and no numerical test would notice."""
    import re
    import subprocess
    from paper_2503_00022_amd import build
    src = os.path.join(build.CSRC, "scores.hip")
    out = tmp_path / "scores.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-fPIC", "-shared")]
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *flags, "--cuda-device-only", "-I",
                    os.path.join(ROOT, "include"), "-I", build.CSRC, "-S", "-o", str(out), src],
                   check=True, capture_output=True)
    text = out.read_text()
    checked = 0
    # every kernel's text, cut into basic blocks at the compiler's labels
    for kern in re.split(r"\n(?=_Z\S+:)", text):
        name = kern.split(":", 1)[0]
        if not ("lse_kernel" in name or "colsum_kernel" in name) or "ILb1E" not in name:
            continue                                   # 16-bit instantiations only (the fp32 path is not pipelined)
        body = kern[:kern.index("s_endpgm")] if "s_endpgm" in kern else kern
        blocks = re.split(r"\n(?=\.LBB\d+_\d+:)", body)
        D = 128 if "ELi128E" in name else 64
        per_half = D // 8                              # MFMAs of one 64 x 32 block
        n_mfma = lambda b: len(re.findall(r"v_mfma_f32_32x32x16", b))
        if "colsum_kernel" in name:
            loops = [b for b in blocks if n_mfma(b) == 6 * per_half]                     # one straight block a trip
            assert len(loops) == 1, (name, [n_mfma(b) for b in blocks])
            loop = loops[0]
        else:
            # pass A's trip is six blocks of one half step each (a rarely taken re-basing branch ends each)
            idx = [i for i, b in enumerate(blocks) if n_mfma(b) == per_half and "s_cbranch_vccnz" in b]
            assert len(idx) >= 6, (name, len(idx))
            loop = "\n".join(blocks[idx[0]:idx[5] + 2])
        assert loop.count("s_waitcnt vmcnt(0)") == 3, (name, loop.count("s_waitcnt vmcnt(0)"))
        assert loop.count("s_barrier") == 3, name
        lgkm = [int(n) for n in re.findall(r"s_waitcnt lgkmcnt\((\d+)\)", loop)]
        assert lgkm.count(0) <= 3, (name, lgkm)        # only the drain in front of each barrier
        if D == 128:
            assert sum(1 for n in lgkm if n >= 2) >= 36, (name, lgkm)   # fragment waits leave reads in flight
        assert "global_load_lds_dwordx4" in loop
        checked += 1
    assert checked == 16, checked   # {lse, colsum} x {bf16, fp16} x {D = 64, 128} x {packed, strided}
