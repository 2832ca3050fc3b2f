"""The library's host code without a GPU: the host halves of ``csrc/*.hip`` (kernels left out) linked against the stand-in
for the runtime in ``host_runtime.cpp``; ``host_probe.hip`` reaches what has no entry point.  "Device" pointers are those of numpy arrays."""

from __future__ import annotations

import ctypes
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

import numpy as np

from paper_1803_03288_amd import build as build_mod

HERE = os.path.dirname(os.path.abspath(__file__))
I32, I64 = ctypes.c_int32, ctypes.c_int64


def build_host_lib(where: str) -> str:
    """Compiles into the folder ``where``; returns the path of the shared library."""
    flags = ["-O1", "-std=c++17", "-fPIC", "-w", "-I", os.path.join(build_mod.ROOT, "include"), "-I", build_mod.CSRC]

    def compile_one(src):
        obj = os.path.join(where, os.path.basename(src) + ".o")
        cmd = [build_mod.HIPCC, "--cuda-host-only", "--offload-arch=gfx950"] if src.endswith(".hip") else \
            ["g++", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(os.path.dirname(os.path.dirname(build_mod.HIPCC)), "include")]
        subprocess.run(cmd + flags + ["-c", src, "-o", obj], check=True, stderr=subprocess.PIPE)
        return obj

    with ThreadPoolExecutor(8) as ex:
        objs = list(ex.map(compile_one, build_mod.sources() + [os.path.join(HERE, f) for f in ("host_runtime.cpp", "host_probe.hip")]))
    # each object refers to its device code under a name of its own; there is none here
    undefined = subprocess.run(["nm", "-u"] + objs, check=True, stdout=subprocess.PIPE, text=True).stdout
    names = sorted({w for w in undefined.split() if w.startswith("__hip_fatbin_")})
    stub = os.path.join(where, "fatbin.c")
    with open(stub, "w") as f:
        f.writelines(f"const char {n}[8];\n" for n in names)
    out = os.path.join(where, "libtictac_host.so")
    subprocess.run(["gcc", "-c", "-fPIC", stub, "-o", stub + ".o"], check=True)
    # (-Bsymbolic: the stand-in is used, not a runtime that the process has loaded already)
    subprocess.run(["g++", "-shared", "-Wl,-Bsymbolic", "-o", out] + objs + [stub + ".o", "-lpthread"], check=True)
    return out


class HostLib:
    """The loaded library: the C calls by name (``lib.tictac_...``), the stand-in's controls, and a few shorthands."""

    def __init__(self, path: str):
        self.L = ctypes.CDLL(path)
        self.L.tictac_last_error.restype = ctypes.c_char_p
        for f in ("host_count", "host_group_bytes", "host_fail_new_left", "host_fail_device_left"):
            getattr(self.L, f).restype = I64
        for f in ("host_fail_device", "host_device_limit", "host_fail_new", "host_slow_copies"):
            getattr(self.L, f).argtypes = [I64]

    def __getattr__(self, name):
        return getattr(self.L, name)

    def count(self, what: str) -> int:
        return self.L.host_count(what.encode())

    def error(self) -> str:
        return self.L.tictac_last_error().decode()

    def build(self, d):
        """``(status, handle)``"""
        rp, ci, ri = (np.ascontiguousarray(x, dtype=np.int32) for x in (d.row_ptr, d.col_idx, d.recv_ids))
        h = ctypes.c_void_p()
        rc = self.L.tictac_build_deps(I32(d.n_ops), ptr(rp), ptr(ci), I32(ri.size), ptr(ri), None, ctypes.byref(h))
        return rc, h

    def free(self, h):
        assert self.L.tictac_dag_free(h) == 0

    def tac(self, h, d, B, room=None):
        """``tictac_tac_simulate`` on ``B`` samples of ones; ``room`` keeps the arrays for the next call."""
        room = {} if room is None else room
        if room.get("B") != B:
            room.update(B=B, op=np.ones((B, d.n_compute)), rv=np.ones((B, d.n_recv)), order=np.zeros((B, d.n_recv), np.int32),
                        out=np.zeros((5, B)))
        return self.L.tictac_tac_simulate(h, I32(B), ptr(room["op"]), ptr(room["rv"]), ptr(room["order"]), None, None, None,
                                          *(ptr(x) for x in room["out"]), None)

    def launches(self):
        """``[(kernel, workgroups, threads, LDS bytes, words that a fill fills)]`` since they were last forgotten."""
        out, name = [], ctypes.create_string_buffer(256)
        v = [I64() for _ in range(4)]
        i = 0
        while self.L.host_launch(I64(i), name, I64(256), *(ctypes.byref(x) for x in v)):
            out.append((name.value.decode(),) + tuple(x.value for x in v))
            i += 1
        return out

    def kernels(self):
        return [l[0] for l in self.launches()]


def ptr(a: np.ndarray) -> ctypes.c_void_p:
    return ctypes.c_void_p(a.ctypes.data)
