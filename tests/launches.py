"""What the library's host code launches for a call, without a GPU: a child process loads
launch_recorder.cpp ahead of libkvcrush.so and makes the calls with addresses that nothing reads."""
import collections
import ctypes
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
FAKE, FAKE2 = 0x10000000, 0x70000000000      # aligned addresses, never dereferenced
Launch = collections.namedtuple("Launch", "kernel grid block lds order")    # order: S, n_bh, n_pieces, turn of the score kernels


def build_recorder(folder):
    path = os.path.join(str(folder), "launch_recorder.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-shared", "-fPIC", "-o", path,
                    os.path.join(HERE, "launch_recorder.cpp")], check=True)
    return path


def scores(shape, lse=False, ws_bytes=1 << 60):
    return ["kvcrush_scores", bytes(shape).hex(), ["struct", FAKE, FAKE, FAKE if lse else 0, FAKE2, FAKE, ws_bytes, 0]]


def row_lse(shape, ws_bytes=1 << 60):
    return ["kvcrush_row_lse", bytes(shape).hex(), ["struct", FAKE, FAKE, FAKE2, FAKE if ws_bytes else 0, ws_bytes, 0]]


def append(shape, capacity, ws_bytes=1 << 60, block_size=0):
    return ["kvcrush_scores_append", bytes(shape).hex(),
            ["struct", capacity, 0, FAKE, FAKE, FAKE if block_size else 0, block_size, FAKE2, FAKE, ws_bytes, 0]]


def select(args, ws_bytes=1 << 60):
    return ["kvcrush_select", bytes(args).hex(), ["struct", FAKE, FAKE2, 0, 0, FAKE, ws_bytes, 0]]


def select_static(args):
    return ["kvcrush_select_static", bytes(args).hex(), ["struct", FAKE, FAKE2, 0, 0, 0]]


def record(recorder, lib_path, calls):
    """[(status, [Launch, ...]), ...] of the calls made with the functions above."""
    out = subprocess.run([sys.executable, os.path.abspath(__file__), recorder, lib_path], input=json.dumps(calls), text=True,
                         check=True, capture_output=True).stdout
    return [(st, [Launch(k, tuple(g), b, lds, tuple(o)) for k, g, b, lds, o in ls]) for st, ls in json.loads(out)]


def _child(recorder, lib_path):
    rec = ctypes.CDLL(recorder, mode=ctypes.RTLD_GLOBAL)
    rec.recorded.restype = ctypes.c_char_p
    lib = ctypes.CDLL(lib_path)
    result = []
    for name, struct, args in json.load(sys.stdin):
        buf = ctypes.create_string_buffer(bytes.fromhex(struct))
        rec.forget()
        # (every argument is an integer or a pointer: passing each as 64 bits fits the calling convention)
        st = getattr(lib, name)(*[buf if a == "struct" else ctypes.c_uint64(a) for a in args])
        launches = []
        for line in rec.recorded().decode().splitlines():
            kernel, gx, gy, gz, bx, lds, _, *order = line.split()
            launches.append([kernel, [int(gx), int(gy), int(gz)], int(bx), int(lds), [int(x) for x in order]])
        result.append([st, launches])
    json.dump(result, sys.stdout)


if __name__ == "__main__":
    _child(sys.argv[1], sys.argv[2])
