"""The device walk (csrc/neuvv_device.h), compiled for the host with the few builtins it uses: from any ray, also one
with zeros, infinities, NaN or components near the ends of float32, it stays inside the grid and ends, and its segments
lie in order; for ordinary rays the leaves are those that the ray crosses."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2202_06088_amd.voctree import build_node_table

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2202_06088_amd", "csrc")

SHIM = r"""
#pragma once
#include <cmath>
#include <cstdint>
#include <cstring>
#define __host__
#define __device__
#define __forceinline__ inline
struct int4 { int x, y, z, w; };
struct float4 { float x, y, z, w; };
static inline int __popc(uint32_t v) { return __builtin_popcount(v); }
static inline void sincosf_(float x, float* s, float* c) { *s = std::sin(x); *c = std::cos(x); }
#define sincosf sincosf_
static inline double rcp_host(double d) { return 1.0 / d; }
static inline float rcpf_host(float d) { return 1.0f / d; }
#define __builtin_amdgcn_rcp rcp_host
#define __builtin_amdgcn_rcpf rcpf_host
"""

SRC = r"""
#include "shim.h"
#include "neuvv_device.h"
using namespace neuvv;
// One ray; IDENT: no instance. Writes up to `room` segments {leaf, a, b}; returns their number, -1 when the walk leaves
// the grid, -2 when it does not end, -3 when segments are out of order.
template <bool IDENT>
static int walk(const TreeArgs& tr, const InstArgs& in, const float* o, const float* d, int room, int* leaf, double* ab) {
    RaySetup rs;
    ray_geometry<IDENT>(tr, in, o, d, rs);
    Walk w;
    walk_begin(tr, rs, w);
    int n = 0;
    const int G = 1 << tr.depth;
    double last = -1.0;
    for (int visit = 0; visit < 3 * G + 8; ++visit) {
        if (!w.done)
            for (int a = 0; a < 3; ++a)
                if ((w.m[a] ^ rs.flip[a]) < 0 || (w.m[a] ^ rs.flip[a]) >= G) return -1;
        float delta, umid;
        double sa, sb;
        const int l = walk_next<1>(tr, rs, w, delta, umid, sa, sb);
        if (l == -2) continue;
        if (l == -1) return n;
        if (l < 0 || l >= tr.n_leaves) return -1;
        if (!(sa < sb) || sa < last) return -3;
        last = sb;
        if (n < room) {
            leaf[n] = l;
            ab[2 * n] = sa;
            ab[2 * n + 1] = sb;
        }
        ++n;
    }
    return -2;
}
extern "C" void walks(int depth, const int4* nodes, int64_t n_leaves, const int* dir, const int* box, const float* place,
                      int64_t n, const float* o, const float* d, int room, int* count, int* leaf, double* ab) {
    TreeArgs tr{};
    tr.nodes = nodes;
    tr.dir = dir;
    tr.depth = depth;
    tr.n_leaves = n_leaves;
    for (int a = 0; a < 3; ++a) {
        tr.box_lo[a] = box[a];
        tr.box_hi[a] = box[3 + a];
    }
    InstArgs in{};
    if (place) {
        for (int k = 0; k < 9; ++k) in.rot[k] = place[k];
        for (int k = 0; k < 3; ++k) in.trans[k] = place[9 + k];
        in.scale = place[12];
    }
    for (int64_t r = 0; r < n; ++r)
        count[r] = place ? walk<false>(tr, in, o + 3 * r, d + 3 * r, room, leaf + r * room, ab + 2 * r * room)
                         : walk<true>(tr, in, o + 3 * r, d + 3 * r, room, leaf + r * room, ab + 2 * r * room);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("walk")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text('#include "shim.h"\n')
    (d / "shim.h").write_text(SHIM)
    (d / "walk.cpp").write_text(SRC)
    # clang++: the header uses its vector types
    subprocess.check_call(["/opt/rocm/llvm/bin/clang++", "-O2", "-std=c++17", "-mfma", "-ffp-contract=off", "-shared",
                           "-fPIC", "-Wno-everything", "-I", str(d), "-I", CSRC, str(d / "walk.cpp"), "-o",
                           str(d / "walk.so")])
    return ctypes.CDLL(str(d / "walk.so"))


def directory(depth, leaf_ijk, nodes):
    """The brick directory from its definition: per 4^3 region its last-level node row, else -(1 + log2 edge) of the
    largest aligned empty cube around it."""
    E = 1 if depth <= 2 else 1 << (depth - 2)
    occ = np.zeros((1 << depth,) * 3, bool)
    occ[tuple(leaf_ijk.T)] = True
    out = np.empty(E ** 3, np.int32)

    def descend(i, j, k):
        row, lo, edge = 0, np.zeros(3, int), depth
        p = np.array([i, j, k])
        while True:
            bits = 1 if edge == depth and depth & 1 else 2
            child = edge - bits
            if child == 0:
                return row
            q = (p - lo) >> child
            b = int((q[0] & 1) | (q[1] & 1) << 1 | (q[2] & 1) << 2)
            if bits == 2:
                b = int((q[0] & 1) | (q[1] & 1) << 1 | (q[2] & 1) << 2 | (q[0] >> 1) << 3 | (q[1] >> 1) << 4 | (q[2] >> 1) << 5)
            mask = (int(nodes[row, 0]) & 0xffffffff) | (int(nodes[row, 1]) & 0xffffffff) << 32
            if not mask >> b & 1:
                return None
            row = int(nodes[row, 2]) + bin(mask & ((1 << b) - 1)).count("1")
            lo = lo + (q << child)
            edge = child

    for k in range(E):
        for j in range(E):
            for i in range(E):
                c = (4 * i, 4 * j, 4 * k)
                if occ[c[0]:c[0] + 4, c[1]:c[1] + 4, c[2]:c[2] + 4].any():
                    out[(k * E + j) * E + i] = descend(*c)
                    continue
                s = 2
                while s < depth:
                    a = [v >> (s + 1) << (s + 1) for v in c]
                    if occ[a[0]:a[0] + (2 << s), a[1]:a[1] + (2 << s), a[2]:a[2] + (2 << s)].any():
                        break
                    s += 1
                out[(k * E + j) * E + i] = -(1 + s)
    return out


def make_tree(depth, n, seed):
    rng = np.random.default_rng(seed)
    G = 1 << depth
    cells = rng.choice(G ** 3, size=min(n, G ** 3), replace=False)
    ijk = np.stack([cells % G, cells // G % G, cells // (G * G)], 1).astype(np.int32)
    nodes, slots, box = build_node_table(depth, ijk, with_box=True)
    return ijk, np.ascontiguousarray(nodes), slots, np.asarray(box, np.int32), directory(depth, ijk, nodes)


def run(lib, depth, tree, o, d, place=None, room=256):
    ijk, nodes, slots, box, dirs = tree
    n = o.shape[0]
    o, d = np.ascontiguousarray(o, np.float32), np.ascontiguousarray(d, np.float32)
    count, leaf, ab = np.empty(n, np.int32), np.full((n, room), -1, np.int32), np.zeros((n, room, 2))
    p = lambda a: None if a is None else a.ctypes.data_as(ctypes.c_void_p)
    lib.walks(depth, p(nodes), ctypes.c_int64(len(ijk)), p(dirs), p(box), p(place), ctypes.c_int64(n), p(o), p(d), room,
              p(count), p(leaf), p(ab))
    return count, leaf, ab


TREES = [(1, 3), (2, 1), (2, 40), (3, 60), (4, 300), (5, 2000), (6, 900)]
PLACES = [None, np.array([0, -1, 0, 1, 0, 0, 0, 0, 1, 3.5, -2, 1, 0.7], np.float32),
          np.array([1, 0, 0, 0, 1, 0, 0, 0, 1, 0, 0, 0, 1e-30], np.float32),
          np.array([1, 0, 0, 0, 1, 0, 0, 0, 1, 1e30, 0, 0, 1e30], np.float32),
          np.zeros(13, np.float32) + np.array([0] * 12 + [1], np.float32)]   # (a rotation of zeros)


@pytest.mark.parametrize("place", range(len(PLACES)))
@pytest.mark.parametrize("depth,n", TREES)
def test_any_ray_stays_in_the_grid_and_ends(lib, depth, n, place):
    tree, rng, G = make_tree(depth, n, depth), np.random.default_rng(100 * depth + place), 1 << depth
    odd = np.array([0.0, -0.0, 1.0, -1.0, np.nan, np.inf, -np.inf, 1e-45, -1e-45, 1e-38, 1e-30, -1e-20, 1e-10, 1e10, -1e20,
                    1e30, 3.4e38, -3.4e38, 0.5, G, G - 1, G / 2, -G, G + 1e-3, np.nextafter(np.float32(G), np.float32(0))],
                   np.float32)
    m = 20_000
    o = np.where(rng.random((m, 3)) < 0.5, rng.choice(odd, (m, 3)), rng.uniform(-G, 2 * G, (m, 3)).astype(np.float32))
    d = np.where(rng.random((m, 3)) < 0.5, rng.choice(odd, (m, 3)), rng.normal(size=(m, 3)).astype(np.float32))
    o[::3] = np.round(o[::3])   # on planes, edges and corners
    count, _, _ = run(lib, depth, tree, o.astype(np.float32), d.astype(np.float32), PLACES[place])
    assert count.min() >= 0, (count.min(), o[count.argmin()], d[count.argmin()])


@pytest.mark.parametrize("depth,n", TREES)
def test_segments_are_the_leaves_crossed(lib, depth, n):
    """Against the clip of every leaf's cube in extended precision: the same leaves, in order, with the same bounds."""
    tree, rng, G = make_tree(depth, n, depth), np.random.default_rng(depth), 1 << depth
    ijk, _, slots, _, _ = tree
    m = 300
    o = (G / 2 + rng.normal(size=(m, 3)) * G).astype(np.float32)
    d = (rng.uniform(0, G, (m, 3)) - o).astype(np.float32)
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    count, leaf, ab = run(lib, depth, tree, o, d)
    O, D = o.astype(np.longdouble)[:, None, :], d.astype(np.longdouble)[:, None, :]
    t0, t1 = (ijk[None] - O) / D, (ijk[None] + 1 - O) / D
    a, b = np.minimum(t0, t1).max(2), np.maximum(t0, t1).min(2)
    a = np.maximum(a, 0)
    assert count.max() > 0
    for r in range(m):
        want = np.flatnonzero(b[r] - a[r] > 1e-9)
        want = want[a[r][want].argsort()]
        clear = count[r] - ((ab[r, :count[r], 1] - ab[r, :count[r], 0]) <= 1e-9).sum()
        long = np.flatnonzero((ab[r, :count[r], 1] - ab[r, :count[r], 0]) > 1e-9)
        assert clear == len(want) and np.array_equal(leaf[r, long], slots[want])
        assert np.abs(ab[r, long, 0] - a[r][want]).max(initial=0) < 1e-9
        assert np.abs(ab[r, long, 1] - b[r][want]).max(initial=0) < 1e-9
