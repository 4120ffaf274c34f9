"""Runs pieces of test code in a process of their own in which libcutgraph.so
runs on tests/fake_hip.cpp: no GPU, no kernel is executed, and the launches,
allocations and event calls that the library makes are read from a log."""
from __future__ import annotations

import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
_fake = None


def _build() -> str:
    global _fake
    if _fake is None:
        _fake = os.path.join(tempfile.mkdtemp(prefix="fake_hip_"), "libfake_hip.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                        "-I/opt/rocm/include", os.path.join(HERE, "fake_hip.cpp"), "-o", _fake],
                       check=True, capture_output=True, timeout=300)
    return _fake


_PRELUDE = """
import ctypes as C, json, os, re, sys, types
fake = C.CDLL({fake!r}, C.RTLD_GLOBAL)
fake.fake_log.restype = C.c_char_p
fake.fake_used.restype = C.c_size_t
fake.fake_limit.argtypes = fake.fake_left.argtypes = [C.c_size_t]
fake.fake_capturing.argtypes = [C.c_void_p, C.c_int]
fake.fake_block.argtypes, fake.fake_block.restype = [C.c_void_p], C.c_size_t
sys.modules["torch"] = types.ModuleType("torch")   # the binding imports it for its runtime alone
import importlib.util
spec = importlib.util.spec_from_file_location("_lib", {lib!r})
L = importlib.util.module_from_spec(spec)
spec.loader.exec_module(L)


class Buf:
    '''An operand that no kernel reads: an address and a row length.'''
    def __init__(self, ld, ptr=1 << 40):
        self.ld, self.ptr = ld, ptr
    def data_ptr(self):
        return self.ptr
    def dim(self):
        return 2
    def stride(self, k):
        return self.ld


def graph(m, flags=0, load=0, alg=None):
    import tempfile
    with tempfile.TemporaryDirectory() as d:
        path = os.path.join(d, "g.cgb")
        L.cut_graph_build(L.CUT_ALG_MAJORANA if alg is None else alg, m, path, 0, flags)
        return L.cut_graph_load(path, 0, load)


def log(clear=True):
    lines = fake.fake_log().decode().splitlines()
    if clear:
        fake.fake_clear()
    return lines


def kernels(lines):
    '''(name, stream) of every launch'''
    return [(re.split("<", l.split(" ", 3)[3])[0], l.split(" ")[1]) for l in lines if l.startswith("kernel ")]


def out(v):
    print("RESULT " + json.dumps(v))
"""


def run(code: str, timeout: int = 300):
    """Runs `code` (which sees L, fake, Buf, graph, log, kernels, out) and returns what it passed to out()."""
    lib = os.path.join(ROOT, "paper_2609_14831_amd", "_lib.py")
    src = _PRELUDE.format(fake=_build(), lib=lib) + code
    r = subprocess.run([sys.executable, "-c", src], capture_output=True, text=True, timeout=timeout, cwd=ROOT)
    assert r.returncode == 0, (r.returncode, r.stdout[-2000:], r.stderr[-4000:])
    got = [l for l in r.stdout.splitlines() if l.startswith("RESULT ")]
    assert got, r.stdout[-2000:]
    return json.loads(got[-1][len("RESULT "):])
