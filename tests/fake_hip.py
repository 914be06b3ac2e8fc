"""Runs Python code against libpm.so with tests/fake_hip.cpp in the HIP runtime's place.

The code runs in a process of its own (a library binds its runtime once); its
names: np, api, scenes, log() (the runtime's calls since the last log(), one
list of words each), fail(name, nth, code), memory(bytes), used(), fake (the
stand-in itself), new_stream(), unjoined(calls, stream).
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
OOM, INVALID = 2, 1  # hipErrorOutOfMemory, hipErrorInvalidValue

PRELUDE = """
import ctypes, sys
sys.path.insert(0, {root!r})
fake = ctypes.CDLL({lib!r}, ctypes.RTLD_GLOBAL)
fake.fake_take_log.restype = ctypes.c_char_p
fake.fake_fail.argtypes = [ctypes.c_char_p, ctypes.c_long, ctypes.c_int]
fake.fake_memory.argtypes = [ctypes.c_size_t]
fake.fake_used.restype = ctypes.c_size_t
fake.fake_last_block.restype = ctypes.c_void_p
fake.fake_capture.argtypes = [ctypes.c_ssize_t, ctypes.c_int]
fake.fake_take_log()
import numpy as np
from paper_1505_06022_amd import api, scenes
OOM, INVALID = {oom}, {invalid}
def log():
    return [l.split() for l in fake.fake_take_log().decode().splitlines()]
def fail(name, nth, code):
    fake.fake_fail(name.encode(), nth, code)
def memory(size):
    fake.fake_memory(size)
def used():
    return fake.fake_used()
class Stream:
    def __init__(self):
        s = ctypes.c_void_p()
        assert fake.hipStreamCreateWithFlags(ctypes.byref(s), 1) == 0
        self.cuda_stream = s.value
def new_stream():
    return Stream()
def unjoined(calls, stream):
    '''Streams with work that the work enqueued on `stream` after these calls would not wait for.'''
    done, seen, events = dict(), dict(), dict()  # per stream: its work, the work of others it follows
    for c in calls:
        if c[0] in ("launch", "copy", "fill", "graph"):
            done[c[-1]] = done.get(c[-1], 0) + 1
        elif c[0] == "record":
            s = dict(seen.get(c[2], dict()))
            s[c[2]] = done.get(c[2], 0)
            events[c[1]] = s
        elif c[0] == "wait":
            mine = seen.setdefault(c[1], dict())
            for k, v in events.get(c[2], dict()).items():
                mine[k] = max(mine.get(k, 0), v)
    return [s for s, n in done.items() if s != str(stream) and seen.get(str(stream), dict()).get(s, 0) < n]
"""


def build(folder) -> str:
    out = os.path.join(str(folder), "libfake_hip.so")
    hipcc = os.environ.get("HIPCC") or "/opt/rocm/bin/hipcc"
    subprocess.run([hipcc, "-std=c++17", "-O1", "-fPIC", "-shared", "-x", "hip", "--offload-host-only",
                    os.path.join(HERE, "fake_hip.cpp"), "-o", out], check=True)
    return out


def run(lib: str, code: str) -> str:
    """Output of the code; an assertion that fails in it fails the caller."""
    text = PRELUDE.format(root=os.path.dirname(HERE), lib=lib, oom=OOM, invalid=INVALID) + code
    r = subprocess.run([sys.executable, "-c", text], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def kernels(library: str) -> dict:
    """Name -> metadata (registers, LDS) of the kernels that this repository's build put into a library."""
    import struct

    import msgpack
    data, out, at = open(library, "rb").read(), {}, 0
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        (n,), p = struct.unpack_from("<Q", data, at + 24), at + 32
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in name:
                out.update(_elf_kernels(data[at + offset:at + offset + size], struct, msgpack))
        at += 24
    return out


def _elf_kernels(elf, struct, msgpack):
    sections, = struct.unpack_from("<Q", elf, 40)
    size, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, sections + i * size + 4)
        offset, length = struct.unpack_from("<QQ", elf, sections + i * size + 24)
        if kind == 7:  # a note: name and description, each padded to four bytes
            names, desc, _ = struct.unpack_from("<III", elf, offset)
            start = offset + 12 + (names + 3) // 4 * 4
            meta = msgpack.unpackb(elf[start:start + desc], strict_map_key=False)
            return {k[".name"]: k for k in meta["amdhsa.kernels"]}
    return {}
