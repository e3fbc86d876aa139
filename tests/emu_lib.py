"""Builds the drivers of tests/emu (the library's sources compiled with g++
against the host emulation of the device operations) and loads them with
ctypes."""
import ctypes
import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_dir = tempfile.TemporaryDirectory(prefix="emu_")


EMU = os.path.join(ROOT, "tests", "emu")
CSRC = os.path.join(ROOT, "paper_2107_00075_amd", "csrc")
FLAGS = ["-std=c++17", "-fwrapv", "-fPIC", "-fno-reorder-blocks", "-pthread", "-w", "-I", EMU, "-I", CSRC,
         "-I", os.path.join(ROOT, "include")]


def load(driver: str) -> ctypes.CDLL:
    so = os.path.join(_dir.name, driver + ".so")
    if not os.path.exists(so):
        subprocess.check_call(["g++", *FLAGS, "-O1", "-shared", "-x", "c++", os.path.join(EMU, driver + ".cpp"), "-o", so])
    return ctypes.CDLL(so)


def load_library() -> ctypes.CDLL:
    """The library's sources as one shared object on host memory."""
    so = os.path.join(_dir.name, "library.so")
    if not os.path.exists(so):
        srcs = [os.path.join(CSRC, s) for s in ("rounds.hip", "setup.hip", "keys.hip", "api.hip", "batch.hip", "server.cpp")]
        srcs += [os.path.join(EMU, s) for s in ("library_host.cpp", "library_core.cpp", "library_inc.cpp")]

        def compile_one(src):
            obj = os.path.join(_dir.name, os.path.basename(src) + ".o")
            subprocess.check_call(["g++", *FLAGS, "-O1", "-x", "c++", "-c", src, "-o", obj])
            return obj

        with ThreadPoolExecutor(4) as ex:
            objs = list(ex.map(compile_one, srcs))
        subprocess.check_call(["g++", "-shared", "-pthread", *objs, "-o", so])
    return ctypes.CDLL(so)


def ptr(a):
    return None if a is None else a.ctypes.data_as(ctypes.c_void_p)


def core_run(lib, g, seed=1, prio=None, init=None, max_rounds=0, order=1):
    """All rounds of a distance-1 graph in the core kernels: colors, rounds,
    vertex visits, stopped at max_rounds.  order: the wavefronts' order."""
    rp, ci = (np.ascontiguousarray(a, dtype=np.int32) for a in (g.row_ptr, g.col))
    init = None if init is None else np.ascontiguousarray(init, dtype=np.int32)
    prio = None if prio is None else np.ascontiguousarray(prio, dtype=np.uint32)
    colors = np.zeros(g.n, np.int32)
    rounds, visits, left = ctypes.c_int32(), ctypes.c_int64(), ctypes.c_int32()
    err = lib.core_run(g.n, ptr(rp), ptr(ci), ctypes.c_uint32(seed), ptr(prio), ptr(init), max_rounds,
                       ctypes.c_uint64(order), ptr(colors), ctypes.byref(rounds), ctypes.byref(visits),
                       ctypes.byref(left))
    assert err & ~0x800 == 0, hex(err)  # (0x800: the wide stage handed over)
    return colors, rounds.value, visits.value, left.value
