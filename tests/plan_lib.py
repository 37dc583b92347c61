"""The library's launch rules on the CPU (plan_harness.cpp, built once per process with the C++ compiler)."""
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
SPLITS = ("eight_waves", "four_waves", "two_key_groups")


@functools.lru_cache(maxsize=None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "plan.so")
        subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC", "-o", so,
                        os.path.join(HERE, "plan_harness.cpp")], check=True)
        return ctypes.CDLL(so)   # stays mapped


def _cu(docs):
    return np.concatenate([[0], np.cumsum(docs)]).astype(np.int32)


def _call(fn, *args, n_out=2):
    out = [ctypes.c_int() for _ in range(n_out)]
    fn(*args, *(ctypes.byref(o) for o in out))
    return tuple(o.value for o in out)


def forward_split(docs, hq, hkv, d, dtype, step_begin, n_steps, n_cu=256):
    """(split, query heads that share a workgroup)"""
    cu = _cu(docs)
    split, pack = _call(_lib().plan_forward, int(cu[-1]), step_begin, n_steps, hq // hkv, hkv, len(docs),
                        cu.ctypes.data_as(ctypes.c_void_p), int(dtype == "bf16"), d, n_cu)
    return SPLITS[split], 1 << pack


def backward_split(cu, hq, hkv, d, step_begin, n_steps, n_cu=256):
    """(32-row query blocks per chunk, parts of the (step, head) list); cu: int32 array"""
    return _call(_lib().plan_backward, int(cu[-1] - cu[0]), step_begin, n_steps, hq // hkv, hkv, len(cu) - 1,
                 cu.ctypes.data_as(ctypes.c_void_p), d, n_cu)


def backward_launch(docs, hq, hkv, d, step_begin, n_steps, n_cu=256):
    """(32-row query blocks per chunk, parts of the (step, head) list, key groups of a dQ tile) of a launch of one run of documents"""
    cu = _cu(docs)
    return _call(_lib().plan_backward_launch, int(cu[-1]), step_begin, n_steps, hq // hkv, hkv, len(docs),
                 cu.ctypes.data_as(ctypes.c_void_p), d, n_cu, n_out=3)


def backward_splits_of_runs(cu, first, n_docs, n_steps, hq, hkv, d, n_cu=256):
    """[(32-row query blocks per chunk, parts of the list)] of runs of documents, 16 to a launch"""
    ints = [np.ascontiguousarray(x, dtype=np.int32) for x in (first, n_docs, n_steps, cu)]
    out = np.zeros((2, len(first)), dtype=np.int32)
    ptr = lambda x: x.ctypes.data_as(ctypes.c_void_p)
    _lib().plan_backward_runs(len(first), *map(ptr, ints), hq // hkv, hkv, d, n_cu, ptr(out[0]), ptr(out[1]))
    return [tuple(x) for x in out.T.tolist()]


def later_blocks_apart(tokens, hq, hkv, d, step_begin, n_steps, n_cu=256):
    """whether the preprocess launch makes the later blocks' dK, dV (16-bit)"""
    return bool(_lib().plan_later_blocks(tokens, step_begin, n_steps, hq // hkv, hkv, d, n_cu))


def f32_direct(docs, hq, hkv, d, step_begin, n_steps, n_cu=256, q_st=None, kv_st=None):
    """whether the fp32 forward and backward take their operands straight from memory; q_st, kv_st: elements from row to row"""
    cu = _cu(docs)
    strides = [ctypes.c_int64(heads * d if st is None else st) for heads, st in ((hq, q_st), (hkv, kv_st))]
    return tuple(map(bool, _call(_lib().plan_f32_direct, int(cu[-1]), step_begin, n_steps, hq // hkv, hkv, len(docs),
                                 cu.ctypes.data_as(ctypes.c_void_p), d, n_cu, *strides)))


def projection_tiles(tokens, hidden_in, features, n_cu=256, largest_fits=True):
    """[(tokens, features, workgroups per compute unit) of a tile] of the launches"""
    tiles, f_first = (ctypes.c_int * 6)(), ctypes.c_int()
    n = _lib().plan_projection(ctypes.c_int64(tokens), hidden_in, features, int(largest_fits), n_cu, tiles, ctypes.byref(f_first))
    return [tuple(tiles[3 * i:3 * i + 3]) for i in range(n)]


def projection_first_features(tokens, hidden_in, features, n_cu=256):
    """features of the first launch"""
    tiles, f_first = (ctypes.c_int * 6)(), ctypes.c_int()
    _lib().plan_projection(ctypes.c_int64(tokens), hidden_in, features, 1, n_cu, tiles, ctypes.byref(f_first))
    return f_first.value


def projection_group(tokens, kind, features, n_cu=256):
    """token tiles of one feature tile that are dealt to an XCD together (kind: place in the table of tiles)"""
    return _lib().plan_projection_group(ctypes.c_int64(tokens), kind, features, n_cu)
