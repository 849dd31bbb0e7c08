"""Rooms that wavefronts fill in blocks (csrc/room.h), on the host: up to the largest room, every request gets
consecutive items inside the room that no other request has, or none."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2202_06088_amd", "csrc")

# take_items of one lane: the counter is an argument, the rest as in the kernels
SRC = r"""
#include "room.h"
extern "C" int take(int64_t* counter, int64_t cap, int n, int* cur, int* end) {
    if (!neuvv::items_fit(*cur, *end, n)) {
        if (*end < 0) return -1;
        const int64_t first = *counter;
        *counter += neuvv::item_block(cap);
        neuvv::open_block(first, cap, *cur, *end);
        if (!neuvv::items_fit(*cur, *end, n)) {
            *end = -1;
            return -1;
        }
    }
    const int at = *cur;
    *cur += n;
    return at;
}
"""


@pytest.fixture(scope="module")
def take(tmp_path_factory):
    d = tmp_path_factory.mktemp("rooms")
    (d / "take.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fwrapv", "-D__host__=", "-D__device__=",
                           "-D__forceinline__=inline", "-shared", "-fPIC", "-I", CSRC, str(d / "take.cpp"), "-o",
                           str(d / "take.so")])
    lib = ctypes.CDLL(str(d / "take.so"))
    lib.take.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p]
    return lib.take


@pytest.mark.parametrize("cap", [0, 1, 127, 128, 129, 100_000, 2**20, 2**31 - 2049, 2**31 - 128, 2**31 - 64, 2**31 - 2,
                                 2**31 - 1])
def test_requests_stay_in_the_room(take, cap):
    rng = np.random.default_rng(cap % 1000)
    start = max(0, cap - 40_000)   # the last blocks of the room
    counter = ctypes.c_int64(start - start % 2048)
    waves = [(ctypes.c_int32(0), ctypes.c_int32(0)) for _ in range(12)]
    used, full = [], 0
    while full < 12 * 5 and len(used) < 5000:
        cur, end = waves[rng.integers(12)]
        n = int(rng.integers(0, 129))
        at = take(ctypes.addressof(counter), cap, n, ctypes.addressof(cur), ctypes.addressof(end))
        if at < 0:
            full += 1
            continue
        assert at + n <= cap, (at, n)
        if n:
            used.append((at, at + n))
    used.sort()
    assert all(a[1] <= b[0] for a, b in zip(used, used[1:]))
    assert cap < 128 or used   # (the room's last requests found it exhausted: the loop's end)
