"""Rooms that wavefronts fill in blocks (csrc/room.h), on the host: up to the largest room, every request gets
consecutive items inside the room that no other request has, or none; and the room that an adjoint asks for."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2202_06088_amd", "csrc")

# take_items of one lane: the counter is an argument, the rest as in the kernels
SRC = r"""
#include "room.h"
extern "C" int take(int64_t* counter, int64_t cap, int records, int n, int* cur, int* end) {
    const int block = records ? neuvv::record_block(cap) : neuvv::item_block(cap);
    if (!neuvv::items_fit(*cur, *end, n)) {
        if (*end < 0) return -1;
        const int64_t first = *counter;
        *counter += block;
        neuvv::open_block(first, cap, block, *cur, *end);
        if (!neuvv::items_fit(*cur, *end, n)) {
            *end = -1;
            return -1;
        }
    }
    const int at = *cur;
    *cur += n;
    return at;
}
extern "C" void records(int64_t n_rays, int64_t trace_cap, int64_t* out) {
    const neuvv::RecordRoom r = neuvv::record_room(n_rays, trace_cap);
    out[0] = r.most;
    out[1] = r.least;
}
// the room that a device with memory for `memory` records gives; error: another failure at the first try
extern "C" int room(int64_t most, int64_t least, int64_t memory, int error, int64_t* cap, int* tries) {
    *tries = 0;
    return neuvv::take_room(neuvv::RecordRoom{most, least}, *cap,
                            [&](int64_t n) { ++*tries; return error ? error : (n <= memory ? 0 : 2); },
                            [](int e) { return e == 2; });
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("rooms")
    (d / "take.cpp").write_text(SRC)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fwrapv", "-D__host__=", "-D__device__=",
                           "-D__forceinline__=inline", "-shared", "-fPIC", "-I", CSRC, str(d / "take.cpp"), "-o",
                           str(d / "take.so")])
    lib = ctypes.CDLL(str(d / "take.so"))
    lib.take.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p]
    lib.records.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_void_p]
    lib.room.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.c_int32, ctypes.c_void_p, ctypes.c_void_p]
    return lib


@pytest.mark.parametrize("records", [0, 1])
@pytest.mark.parametrize("cap", [0, 1, 127, 128, 129, 100_000, 2**20, 2**31 - 2049, 2**31 - 128, 2**31 - 64, 2**31 - 2,
                                 2**31 - 1])
def test_requests_stay_in_the_room(lib, cap, records):
    take = lib.take
    rng = np.random.default_rng(cap % 1000)
    start = max(0, cap - 40_000)   # the last blocks of the room
    counter = ctypes.c_int64(start - start % 2048)
    waves = [(ctypes.c_int32(0), ctypes.c_int32(0)) for _ in range(12)]
    used, full = [], 0
    while full < 12 * 5 and len(used) < 5000:
        cur, end = waves[rng.integers(12)]
        n = int(rng.integers(0, 129))
        at = take(ctypes.addressof(counter), cap, records, n, ctypes.addressof(cur), ctypes.addressof(end))
        if at < 0:
            full += 1
            continue
        assert at + n <= cap, (at, n)
        if n:
            used.append((at, at + n))
    used.sort()
    assert all(a[1] <= b[0] for a, b in zip(used, used[1:]))
    assert cap < 128 or used   # (the room's last requests found it exhausted: the loop's end)


@pytest.mark.parametrize("n", [0, 1, 64, 4096, 2**16, 2**17, 200_000, 2**19 - 1, 2**19, 2**19 + 1, 2**20, 2**22, 2**24,
                               2**30 - 1, 2**30, 2**31, 2**40])
@pytest.mark.parametrize("trace", [0, 1, 2**20, 2**23, 2**31 - 1])
def test_records_of_a_call(lib, n, trace):
    """Sixteen records a ray up to 256 MiB of them, and never fewer than two a ray, the trace's room and 2^20."""
    out = (ctypes.c_int64 * 2)()
    lib.records(n, trace, ctypes.addressof(out))
    most, least = out
    assert least == min(max(2 * n, trace, 2**20), 2**31 - 1)
    assert most == max(least, min(16 * n, 2**23))


@pytest.mark.parametrize("most,least", [(2**23, 2**21), (2**23, 2**20), (2**20, 2**20), (0, 0), (3 * 2**20 + 5, 2**20)])
@pytest.mark.parametrize("memory", [2**31, 2**23, 2**23 - 1, 3 * 2**20, 2**21, 2**20, 2**20 - 1, 0])
def test_records_that_memory_allows(lib, most, least, memory):
    """A call asks for less where there is no memory for the most, and fails only where the least does not fit."""
    cap, tries = ctypes.c_int64(-1), ctypes.c_int32(0)
    rc = lib.room(most, least, memory, 0, ctypes.addressof(cap), ctypes.addressof(tries))
    assert rc == (0 if least <= memory else 2) and tries.value <= 5
    assert rc != 0 or least <= cap.value <= min(most, memory) and 2 * cap.value + 1 >= min(most, memory)
    assert lib.room(most, least, memory, 7, ctypes.addressof(cap), ctypes.addressof(tries)) == 7 and tries.value == 1
