"""The launch plan of the library (csrc/plan.hpp), compiled by itself: the cut that a call gets, and whether it runs as one launch."""

import ctypes
import functools
import os
import subprocess
import tempfile
from collections import namedtuple

import paper_2510_18413_amd as A
from paper_2510_18413_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))
Cut = namedtuple("Cut", "tile parts n_tiles scratch")


def _compiled(source):
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, source + ".so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-fPIC", "-shared", "-I", str(B.ROOT / "include"),
                        "-I", str(B.CSRC), os.path.join(HERE, source + ".cpp"), "-o", so], check=True)
        return ctypes.CDLL(so)


@functools.lru_cache(maxsize=1)
def _lib():
    return _compiled("scan_plan")


@functools.lru_cache(maxsize=1)
def one_launch_lib():
    lib = _compiled("one_launch_plan")
    lib.one_launch_lds.restype = ctypes.c_int64
    return lib


STEP, TOPK, DISTANCES, STATIC = range(4)


def cut(cfg, batch, max_seq_len, use=STEP):
    got = (ctypes.c_int64 * 4)()
    _lib().scan_plan(ctypes.byref(cfg), ctypes.c_int32(batch), ctypes.c_int64(max_seq_len), ctypes.c_int32(use), got)
    return Cut(*got)


def waves(cfg, batch, max_seq_len, k, use=STEP, paged=False):
    """Waves of the workgroups of a step or top-k that runs as one launch, 0 for two kernels."""
    return one_launch_lib().one_launch_waves(ctypes.byref(cfg), batch, ctypes.c_int64(max_seq_len), k, use, int(paged))


def config(heads, kv_heads, batch=1, context=1, **kw):
    return A.Config.make(heads, kv_heads, max(1, batch * context), **kw)


def heads_per_part(group, shift):
    return _lib().heads_per_part(group, shift)


def sparse_parts(heads, k, d):
    """Workgroups per head of the stand-alone attention; -1 for one of sixteen waves."""
    return _lib().sparse_parts(ctypes.c_int64(heads), ctypes.c_int32(k), d)
