"""ctypes over tests/native/kernel_hooks.cpp: planners, and single projection launches by a given plan."""
import ctypes as C
import os

from paper_2604_13519_amd import binding
from paper_2604_13519_amd.build import HOOKS_PATH, build_library, build_test_hooks

PARTIAL, ARGMAX, SWIGLU = 0, 1, 2
ROWS = 100                                    # plan ids from here on: the many-row kernel, + 4 x row tiles + configuration
SHAPES = ((1, 4, 1), (2, 4, 1), (1, 8, 1), (2, 8, 1), (2, 4, 2), (1, 2, 4), (2, 1, 4))     # skinny: tiles a wave, column sets, k-waves
SHAPE_MODES = ((0, 1), (0, 1, 2), (0, 1), (0, 1, 2), (0, 1, 2), (1,), (2,))
CONFIGS = ((8, 1), (4, 2), (2, 4))            # many rows: column sets, k-waves

_lib = None


def lib():
    global _lib
    if _lib is None:
        if not os.path.exists(HOOKS_PATH):
            if not os.path.exists(binding.LIB_PATH):
                build_library(verbose=False)
            build_test_hooks(verbose=False)
        _lib = C.CDLL(HOOKS_PATH)
    return _lib


def plan(R, N, K, mode, part_elems=0, amax_parts=0, n_cu=256):
    i, s = C.c_int(-1), C.c_int(-1)
    lib().hook_plan(n_cu, R, N, K, mode, C.c_long(part_elems), amax_parts, C.byref(i), C.byref(s))
    return i.value, s.value


def cols_per_group(pid):
    if pid >= ROWS:
        return CONFIGS[(pid - ROWS) % 4][0] * 64
    return SHAPES[pid][0] * SHAPES[pid][1] * 16


def units(n_keys, max_M, hq, hkv, n_cu=256):
    """[(sequence, split, first block, end)], splits per sequence, and the room the workspace has for them."""
    n = len(n_keys)
    room = lib().hook_max_units(n_cu, n)
    u, s = (C.c_int * (4 * room))(), (C.c_int * n)()
    count = lib().hook_units(n_cu, hq, hkv, n, (C.c_int * n)(*n_keys), max_M, u, s)
    return [tuple(u[4 * i:4 * i + 4]) for i in range(count)], list(s), room
