// Building blocks shared by the render kernels (render_kernels.h, render_pp.hip):
// payload gathers, work queues, cull passes and candidate lists, launch
// sizing. Device code for gfx950.
#pragma once

#include <hip/hip_runtime.h>

#include <math.h>

#include "launch.h"
#include "neuvv_device.h"
#include "room.h"

namespace neuvv {

constexpr int kBlock = 256;

// Cells a lane's walk visits per iteration of the wavefront's loop at most: a
// lane with a sample to evaluate must not wait for lanes crossing long empty
// stretches (without a budget an iteration lasts as long as its slowest lane's
// stretch), but a second visit for the lanes still without a sample costs less
// than another round of the loop. Forward kernels, 1 / 2 / 3 / 4 visits: ring
// 922 / 883 / 880 / 876 us, 1920 x 1080 view 198 / 165 / 160 / 157 us, stereo frame
// 216 / 193 / 187 / 185 us, but 64 x 64 thumbnail 54 / 57 / 62 / 64 us, where a
// wavefront has a SIMD to itself.
constexpr int kWalkBudget = 2;

template <int DT>
struct StoreTraits;
template <>
struct StoreTraits<0> { static constexpr int V = 4; };
template <>
struct StoreTraits<1> { static constexpr int V = 8; };
template <>
struct StoreTraits<2> { static constexpr int V = 8; };

template <int DT>
__device__ __forceinline__ void unpack16(const uint4& v, float (&out)[StoreTraits<DT>::V]) {
    if constexpr (DT == 0) {
        out[0] = __uint_as_float(v.x);
        out[1] = __uint_as_float(v.y);
        out[2] = __uint_as_float(v.z);
        out[3] = __uint_as_float(v.w);
    } else {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint16_t lo = (uint16_t)(w[i] & 0xffffu), hi = (uint16_t)(w[i] >> 16);
            if constexpr (DT == 1) {
                out[2 * i] = (float)__builtin_bit_cast(_Float16, lo);
                out[2 * i + 1] = (float)__builtin_bit_cast(_Float16, hi);
            } else {
                out[2 * i] = __uint_as_float((uint32_t)lo << 16);
                out[2 * i + 1] = __uint_as_float((uint32_t)hi << 16);
            }
        }
    }
}

// Gathers R values of leaf `slot` from a [ceil(R/V)][N][V] array (layout 0) or
// a [N][ceil(R/V)][V] array (layout 1).
template <int DT, int R>
__device__ __forceinline__ void load_leaf(const void* base, int64_t N, int64_t slot, int layout,
                                          float (&out)[R]) {
    constexpr int V = StoreTraits<DT>::V;
    constexpr int NG = (R + V - 1) / V;
    const int64_t stride = layout ? 1 : N;
    const uint4* p = reinterpret_cast<const uint4*>(base) + (layout ? slot * NG : slot);
    uint4 raw[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) raw[g] = p[(int64_t)g * stride];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        float tmp[V];
        unpack16<DT>(raw[g], tmp);
#pragma unroll
        for (int e = 0; e < V; ++e)
            if (g * V + e < R) out[g * V + e] = tmp[e];
    }
}

// Value e of the R-value row of leaf `slot` (layouts as in load_leaf).
template <int DT, int R>
__device__ __forceinline__ float leaf_elem(const void* base, int64_t N, int64_t slot, int e, int layout) {
    constexpr int V = StoreTraits<DT>::V;
    constexpr int NG = (R + V - 1) / V;
    const int g = e / V, r = e - (e / V) * V;
    const int64_t vec = layout ? slot * NG + g : (int64_t)g * N + slot;
    if constexpr (DT == 0) {
        return reinterpret_cast<const float*>(base)[vec * 4 + r];
    } else {
        const uint16_t u = reinterpret_cast<const uint16_t*>(base)[vec * 8 + r];
        if constexpr (DT == 1) return (float)__builtin_bit_cast(_Float16, u);
        else return __uint_as_float((uint32_t)u << 16);
    }
}

// Per-sample transcendentals on the hardware base-2 exponential, base-2
// logarithm and reciprocal (about 1 ulp each) instead of the correctly
// rounded library sequences, which cost several times the instructions.
// exp_hw: e^x = 2^(x log2 e); relative error 1 ulp plus |x| * 6e-8 from
// rounding the scaled argument (below 1e-6 for the |x| < 15 of colour
// logits and optical depths).
__device__ __forceinline__ float exp_hw(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504088896341f); }
__device__ __forceinline__ float sigmoid_f(float x) { return __builtin_amdgcn_rcpf(1.0f + exp_hw(-x)); }
// log(1 + e), e in [0, 1]: the logarithm of the rounded u = 1 + e, scaled by
// e / (u - 1) to undo the rounding of u (a few ulp).
__device__ __forceinline__ float log1p_hw(float e) {
    const float u = 1.0f + e;
    const float lg = __builtin_amdgcn_logf(u) * 0.693147180559945309f;
    return u == 1.0f ? e : lg * (e * __builtin_amdgcn_rcpf(u - 1.0f));
}
__device__ __forceinline__ float softplus_f(float x) { return fmaxf(x, 0.0f) + log1p_hw(exp_hw(-fabsf(x))); }
// Density activation of Eq. 5 (relu = 0: softplus, the workloads' reading;
// relu != 0: ReLU as Eq. 5 prints it) and its derivative (0 at x <= 0 for ReLU).
// relu is a kernel argument, so the branch is uniform.
__device__ __forceinline__ float density_f(float x, int relu) { return relu ? fmaxf(x, 0.0f) : softplus_f(x); }
__device__ __forceinline__ float density_dx(float x, int relu) { return relu ? (x > 0.0f ? 1.0f : 0.0f) : sigmoid_f(x); }
// Opacity a = 1 - e^-od and transmittance factor e = e^-od of an optical
// depth od >= 0 (Eq. 8). Below od = 1/4 the series of 1 - e^-od to the
// seventh power (truncation below 2e-9 relative) keeps a accurate where
// 1 - e would cancel; above it a = 1 - e loses at most 3e-7 relative.
__device__ __forceinline__ void absorb(float od, float& a, float& e) {
    const float s = od * fmaf(od, fmaf(od, fmaf(od, fmaf(od, fmaf(od, fmaf(od, 1.0f / 5040.0f, -1.0f / 720.0f),
                                                                      1.0f / 120.0f), -1.0f / 24.0f), 1.0f / 6.0f),
                                         -0.5f), 1.0f);
    const float x = exp_hw(-od);
    const bool small = od < 0.25f;
    a = small ? s : 1.0f - x;
    e = small ? 1.0f - s : x;
}

// What one time for every ray makes common to all of them, in LDS: the radial
// factors of the HH basis, the density-basis row and the local time. A ray's
// setup is then its geometry and the products with its harmonics, without the
// table reads (two dependent latencies in every refill of a wavefront), the
// frame arithmetic and the sine and cosine; the values are those ray_basis
// makes (same expressions).
template <int C>
struct CommonTime {
    float g[10];
    float b[C];
    float tau;
};
// Call with the whole block; the caller synchronises.
template <int C>
__device__ __forceinline__ void stage_common_time(const TreeArgs& tr, const InstArgs& in, float t, CommonTime<C>& s) {
    int i0, i1;
    float f, tau;
    time_setup(tr, in, t, i0, i1, f, &tau);
    if (threadIdx.x == 0) {
        float g[10];
        hh_radial((1.0f - f) * tr.gamma[i0] + f * tr.gamma[i1], g);
#pragma unroll
        for (int k = 0; k < 10; ++k) s.g[k] = g[k];
        s.tau = tau;
    }
    if (threadIdx.x < C)
        s.b[threadIdx.x] = (1.0f - f) * tr.basis[(int64_t)i0 * C + threadIdx.x] +
                           f * tr.basis[(int64_t)i1 * C + threadIdx.x];
}
// The first K HH values of a unit direction at the common time.
template <int K, int C>
__device__ __forceinline__ void common_basis(const CommonTime<C>& s, const float (&dir)[3], float (&h)[K]) {
    float g[10], hall[30];
#pragma unroll
    for (int k = 0; k < 10; ++k) g[k] = s.g[k];
    hh_assemble(g, dir[0], dir[1], dir[2], hall);
#pragma unroll
    for (int k = 0; k < K; ++k) h[k] = hall[k];
}

__device__ __forceinline__ int lane_rank(uint64_t mask) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Dynamic chunk distribution: kQueues counters, 128 bytes apart, one per XCD.
// The chunk range [0, n_chunks) is cut into kQueues contiguous parts. In the
// candidate form a cull pass has listed the rays worth walking of part x in
// list[lo_x * 64 ...] (count[x] of them), and chunks are 64 consecutive
// entries of that list.
constexpr int kQueues = 8;
constexpr int kQueueStride = 16;

struct ChunkCursor {
    int home;       // this block's XCD
    int tried;      // queues drained so far (wave-uniform)
    int pos;        // slots of the current chunk handed out; 64 = take a new chunk
    int px0;        // x of the tile's first pixel (images)
    int len;        // candidate form: entries in the current chunk
    int64_t base;   // ray index of the chunk's first slot (candidate form: list index)
};

__device__ __forceinline__ ChunkCursor chunk_cursor() {
    ChunkCursor c;
    c.home = (int)(blockIdx.x & (kQueues - 1));
    c.tried = 0;
    c.pos = kWave;
    c.px0 = 0;
    c.len = 0;
    c.base = 0;
    return c;
}

// Moves the (converged) wavefront to its next chunk; false when every queue
// is drained. One lane takes the ticket; the result is wave-uniform.
__device__ __forceinline__ bool next_chunk(const RayArgs& ra, ChunkCursor& cc) {
    const int64_t n_chunks = (ra.n_slots + 63) >> 6;
    const int leader = __builtin_ctzll(__ballot(1));
    while (cc.tried < kQueues) {
        const int x = (cc.home + cc.tried) & (kQueues - 1);
        const int64_t lo = n_chunks * x / kQueues, hi = n_chunks * (x + 1) / kQueues;
        const int64_t cnt = ra.list ? (int64_t)ra.count[x * kQueueStride] : 0;   // (on its way with the ticket)
        unsigned long long t = 0;
        if ((int)(threadIdx.x & 63) == leader) t = atomicAdd(ra.queue + x * kQueueStride, 1ull);
        const uint32_t t_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)t);
        const uint32_t t_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(t >> 32));
        const int64_t t64 = (int64_t)(((uint64_t)t_hi << 32) | t_lo);
        if (ra.list) {
            if (t64 * 64 < cnt) {
                cc.pos = 0;
                cc.base = lo * 64 + t64 * 64;
                cc.len = cnt - t64 * 64 < 64 ? (int)(cnt - t64 * 64) : 64;
                return true;
            }
            ++cc.tried;
            continue;
        }
        const int64_t k = lo + t64;
        if (k < hi) {
            cc.pos = 0;
            if (ra.img_w > 0) {
                const int64_t ty = k / ra.tiles_x, tx = k - ty * ra.tiles_x;
                cc.px0 = (int)(tx * 8);
                cc.base = ty * 8 * (int64_t)ra.img_w + cc.px0;
            } else {
                cc.base = k * 64;
            }
            return true;
        }
        ++cc.tried;
    }
    return false;
}

// Ray index of slot `within` (0..63) of the current chunk, -1 for padding.
__device__ __forceinline__ int64_t chunk_ray(const RayArgs& ra, const ChunkCursor& cc, int within) {
    if (ra.list) return within < cc.len ? (int64_t)ra.list[cc.base + within] : -1;
    int64_t r;
    if (ra.img_w > 0) {
        if (cc.px0 + (within & 7) >= ra.img_w) return -1;
        r = cc.base + (int64_t)(within >> 3) * ra.img_w + (within & 7);
    } else {
        r = cc.base + within;
    }
    return r < ra.n ? r : -1;
}

// True when a candidate-form launch has no candidates at all (every block
// then leaves before staging anything; the same answer for every thread).
__device__ __forceinline__ bool no_candidates(const RayArgs& ra) {
    if (!ra.list) return false;
    unsigned long long total = 0;
#pragma unroll
    for (int x = 0; x < kQueues; ++x) total += ra.count[x * kQueueStride];
    return total == 0;
}

__device__ __forceinline__ void write_miss(const RenderOut& out, int64_t ray) {
    if (out.rgb) store3(out.rgb + 3 * ray, 0.0f, 0.0f, 0.0f);
    if (out.alpha) out.alpha[ray] = 0.0f;
    if (out.depth) out.depth[ray] = INFINITY;
    if (out.nsamp) out.nsamp[ray] = 0;
    if (out.last_leaf) out.last_leaf[ray] = -1;
}

__device__ __forceinline__ float readlane_f(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

template <typename KernelT>
static int grid_for(KernelT kernel, const RayArgs& ra) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kBlock, 0) != hipSuccess || per_cu <= 0)
        per_cu = 2;
    const int64_t chunks = (ra.n_slots + 63) / 64;
    const int64_t want = (chunks + (kBlock / kWave) - 1) / (kBlock / kWave);
    const int64_t cap = (int64_t)per_cu * device_cu_count();
    const int64_t g = want < cap ? want : cap;
    return (int)(g > 0 ? g : 1);
}

// Blocks of a reduction over the leaves, persistent: as many as are resident
// (where three fit, a fourth that had to wait for its place made the per-point
// reduction take 419 instead of 367 us, that of 30 coefficients 153 instead of
// 127 us), no more than its wavefronts have batches of at least `least` leaves.
template <typename KernelT>
static int leaf_grid(KernelT kernel, int64_t n_leaves, int least = kWave) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, kBlock, 0) != hipSuccess || per_cu <= 0)
        per_cu = 2;
    const int64_t per_block = (int64_t)(kBlock / kWave) * least;
    const int64_t want = (n_leaves + per_block - 1) / per_block, cap = (int64_t)per_cu * device_cu_count();
    return (int)(want < cap ? want : cap);
}

// Work-queue counters of one launch: 1 KiB of stream-ordered scratch, zeroed
// by a one-block kernel (no memset node, so the sequence may be captured in a
// graph) and freed after the render kernel in stream order. The candidate
// form adds kQueues counts (the second KiB) and a list of n_chunks * 64
// int32 ray indices.
// extra: nullptr, or one more counter to clear.
static __global__ void zero_queue_kernel(unsigned long long* q, unsigned long long* extra) {
    q[threadIdx.x] = 0ull;
    if (extra && threadIdx.x == 0) *extra = 0ull;
}

// Cull pass of the candidate form: each wavefront tests kCullGroup chunks of
// one XCD part at a time (64 slots per chunk, one per lane), reserves room for
// the rays it keeps with one atomic on the part's count (atomics on one
// address serialise, so the groups are large), and lists them in slot order.
// MODE 0 (forward): keep the rays the plain-float box test cannot reject and
// write the miss outputs of the others. MODE 4: keep the rays hit.keep(ray) accepts
// and write the miss outputs of the others (no ray loads). MODE 1 (adjoint):
// keep the rays whose forward composited a sample (the others carry no
// gradient); with a trace (head not NULL) the rays that have one go on a second
// list, and only the others on the first. The
// pass is bound by the 24 bytes of ray per slot it reads; at high occupancy
// it runs near HBM bandwidth, where the render kernel's refill rounds would
// take one memory latency per round for every ray. A group is a chain of
// dependent steps (loads, tests, one atomic, list stores), so it is kept to what
// a lane can hold in flight: 8 rays (a segment of an image has that many rows),
// 4 in launches of fewer than kCullSmall chunks that are not images, where a
// group's chain is longer than the work is deep. Forward culls, 4 and 8 rays:
// 65,536 rays 5.3 and 8.3 us, 262,144 6.0 and 8.8, 1,048,576 11.0 and 11.8,
// 2,097,152 25.8 and 23.8, 4,194,304 39.1 and 39.2. With 32 chunks to a group,
// whose loads waited one by one behind the stores of the test before, 518,400
// rays took 25 us and 867,000 took 31 us; now 9.5 and 16 us.
constexpr int kCullGroup = 8;
constexpr int kCullGroupSmall = 4;
constexpr int64_t kCullSmall = 16384;

// Coarse test of one placed tree (the forward's cull).
template <bool IDENT>
struct TreeHit {
    TreeArgs tr;
    InstArgs in;
    __device__ __forceinline__ bool operator()(const float o[3], const float d[3]) const {
        return ray_may_hit<IDENT>(tr, in, o, d);
    }
};

// What the adjoint's cull reads and its second list (MODE 1).
struct CullAdjoint {
    const int32_t* nsamp;
    const int32_t* head;           // nullptr: no trace
    int32_t* list2;
    unsigned long long* count2;
};

// The cull of one ray in two halves, so that the loads of all rays of a lane's
// group are in flight before the first test (a test's miss stores would keep
// the later loads behind them).
template <int MODE>
struct CullIn {
    f3v o, d;         // MODE 0
    int ns, head;     // MODE 1 (head: -1 without a trace)
    bool keep;        // MODE 4
};
template <int MODE, class Hit>
__device__ __forceinline__ void cull_load(const Hit& hit, const RayArgs& ra, const CullAdjoint& adj, int64_t ray,
                                          CullIn<MODE>& in) {
    if constexpr (MODE == 0) {
        in.o = load3(ra.o + 3 * ray);
        in.d = load3(ra.d + 3 * ray);
    } else if constexpr (MODE == 1) {
        in.ns = adj.nsamp[ray];
        in.head = adj.head ? adj.head[ray] : -1;
    } else {
        in.keep = hit.keep(ray);
    }
}
template <int MODE, class Hit>
__device__ __forceinline__ void cull_test(const Hit& hit, const RenderOut& out, const CullIn<MODE>& in, int64_t ray,
                                          bool& k, bool& k2) {
    if constexpr (MODE == 0) {
        const float o[3] = {in.o.x, in.o.y, in.o.z};
        const float d[3] = {in.d.x, in.d.y, in.d.z};
        k = hit(o, d);
        if (!k) write_miss(out, ray);
    } else if constexpr (MODE == 1) {
        k = in.ns > 0 && in.head < 0;
        k2 = in.ns > 0 && in.head >= 0;
    } else {
        k = in.keep;
        if (!k) write_miss(out, ray);
    }
}

// Room for n list entries of part x: one atomic by one lane. Wave-uniform.
__device__ __forceinline__ int64_t list_room(unsigned long long* count, int x, int n) {
    unsigned long long b = 0;
    if ((threadIdx.x & 63) == 0) b = atomicAdd(count + x * kQueueStride, (unsigned long long)n);
    const uint32_t b_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
    const uint32_t b_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
    return (int64_t)(((uint64_t)b_hi << 32) | b_lo);
}

// Adds the lanes' samples to a counter, one atomic per wavefront.
__device__ __forceinline__ void add_samples(unsigned long long* total, int64_t v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) atomicAdd(total, (unsigned long long)v);
}

template <int MODE, class Hit, int GROUP = kCullGroup>
static __global__ __launch_bounds__(kBlock) void cull_kernel(Hit hit, RayArgs ra, RenderOut out, CullAdjoint adj,
                                                              int32_t* list, unsigned long long* count) {
    const int lane = threadIdx.x & 63;
    const int x = (int)(blockIdx.x & (kQueues - 1));
    const int64_t n_chunks = (ra.n_slots + 63) >> 6;
    const int64_t lo = n_chunks * x / kQueues, hi = n_chunks * (x + 1) / kQueues;
    const int64_t nw = (int64_t)(gridDim.x / kQueues) * (kBlock / kWave);
    const int64_t wi = (int64_t)(blockIdx.x / kQueues) * (kBlock / kWave) + (threadIdx.x >> 6);
    if (ra.img_w > 0) {
        // Images: a wavefront takes a segment of up to 8 horizontally adjacent
        // tiles and walks its 8 pixel rows, one row of 64 pixels per pass, so
        // its ray loads and miss stores are contiguous; the rays kept are then
        // listed tile by tile in slot order from the per-row ballots.
        if (hi <= lo) return;
        // (list form: fewer than 2^31 rays, so tile and segment indices fit 32 bits)
        const uint32_t tiles_x = (uint32_t)ra.tiles_x;
        const uint32_t ty_lo = (uint32_t)lo / tiles_x, ty_hi = (uint32_t)(hi - 1) / tiles_x;
        const uint32_t nseg = (tiles_x + 7) / 8;
        const uint32_t n_seg = (ty_hi - ty_lo + 1) * nseg;
        const int jt = lane >> 3;   // tile of the lane within the segment
        for (uint32_t sg = (uint32_t)wi; sg < n_seg; sg += (uint32_t)nw) {
            const uint32_t ty = ty_lo + sg / nseg, j = sg - (sg / nseg) * nseg;
            const int64_t row0 = (int64_t)ty * tiles_x;
            int64_t kx0 = 8 * (int64_t)j, kx1 = kx0 + 8 < tiles_x ? kx0 + 8 : tiles_x;
            if (kx0 < lo - row0) kx0 = lo - row0;
            if (kx1 > hi - row0) kx1 = hi - row0;
            if (kx0 >= kx1) continue;   // wave-uniform
            const int64_t tx = 8 * (int64_t)j + jt;
            const int64_t px = 8 * tx + (lane & 7);
            const bool lane_ok = tx >= kx0 && tx < kx1 && px < ra.img_w;
            uint64_t keep[8], keep2[8];
            int total = 0, total2 = 0;
            int64_t samples = 0;   // MODE 1: the lane's
            CullIn<MODE> in[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int64_t ray = (8 * (int64_t)ty + r) * ra.img_w + px;
                if (lane_ok && ray < ra.n) cull_load<MODE>(hit, ra, adj, ray, in[r]);
            }
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int64_t ray = (8 * (int64_t)ty + r) * ra.img_w + px;
                bool k = false, k2 = false;
                if (lane_ok && ray < ra.n) cull_test<MODE>(hit, out, in[r], ray, k, k2);
                keep[r] = __ballot(k);
                total += __popcll(keep[r]);
                if constexpr (MODE == 1) {
                    if (k || k2) samples += in[r].ns;
                    keep2[r] = __ballot(k2);
                    total2 += __popcll(keep2[r]);
                }
            }
            // lists the kept rays: per lane its tile's kept-slot mask (bit 8r + column) and
            // the rays kept in the segment's earlier tiles
            auto emit = [&](const uint64_t(&kp)[8], int n, int32_t* ls, unsigned long long* ct) {
                const int64_t at = lo * 64 + list_room(ct, x, n);
                uint64_t tm = 0ull;
                int before = 0;
                const uint64_t below = jt ? (~0ull >> (64 - 8 * jt)) : 0ull;
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    tm |= ((kp[r] >> (8 * jt)) & 0xffull) << (8 * r);
                    before += __popcll(kp[r] & below);
                }
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    if ((kp[r] >> lane) & 1ull) {
                        const int within = 8 * r + (lane & 7);
                        const int64_t ray = (8 * (int64_t)ty + r) * ra.img_w + px;
                        ls[at + before + __popcll(tm & ((1ull << within) - 1ull))] = (int32_t)ray;
                    }
                }
            };
            if (total) emit(keep, total, list, count);   // wave-uniform
            if constexpr (MODE == 1) {
                if (total2) emit(keep2, total2, adj.list2, adj.count2);
                if (total + total2) add_samples(count + x * kQueueStride + 1, samples);
            }
        }
        return;
    }
    for (int64_t c0 = lo + wi * GROUP; c0 < hi; c0 += nw * GROUP) {
        uint64_t keep[GROUP], keep2[GROUP];
        int32_t rays[GROUP];
        int total = 0, total2 = 0;
        int64_t samples = 0;   // MODE 1: the lane's
        CullIn<MODE> in[GROUP];
#pragma unroll
        for (int j = 0; j < GROUP; ++j) {
            const int64_t ray = c0 + j < hi ? slot_to_ray(ra, (c0 + j) * 64 + lane) : -1;
            rays[j] = (int32_t)ray;
            if (ray >= 0) cull_load<MODE>(hit, ra, adj, ray, in[j]);
        }
#pragma unroll
        for (int j = 0; j < GROUP; ++j) {
            bool k = false, k2 = false;
            if (rays[j] >= 0) cull_test<MODE>(hit, out, in[j], rays[j], k, k2);
            keep[j] = __ballot(k);
            total += __popcll(keep[j]);
            if constexpr (MODE == 1) {
                if (k || k2) samples += in[j].ns;
                keep2[j] = __ballot(k2);
                total2 += __popcll(keep2[j]);
            }
        }
        auto emit = [&](const uint64_t(&kp)[GROUP], int n, int32_t* ls, unsigned long long* ct) {
            int64_t at = lo * 64 + list_room(ct, x, n);
#pragma unroll
            for (int j = 0; j < GROUP; ++j) {
                if ((kp[j] >> lane) & 1ull) ls[at + lane_rank(kp[j])] = rays[j];
                at += __popcll(kp[j]);
            }
        };
        if (total) emit(keep, total, list, count);   // wave-uniform
        if constexpr (MODE == 1) {
            if (total2) emit(keep2, total2, adj.list2, adj.count2);
            if (total + total2) add_samples(count + x * kQueueStride + 1, samples);
        }
    }
}

template <int MODE, class Hit>
static hipError_t launch_cull_hit(const Hit& hit, const RayArgs& ra, const RenderOut& out, const CullAdjoint& adj,
                                  int32_t* list, unsigned long long* count, hipStream_t st) {
    const int64_t n_chunks = (ra.n_slots + 63) >> 6;
    const bool small = ra.img_w <= 0 && n_chunks < kCullSmall;
    const int group = small ? kCullGroupSmall : kCullGroup;
    const int64_t groups = (n_chunks / kQueues + 1 + group - 1) / group;   // per part, at most
    int64_t blocks = (groups + (kBlock / kWave) - 1) / (kBlock / kWave);
    const int64_t cap = (int64_t)device_cu_count() * 2;
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    const dim3 grid((unsigned)(blocks * kQueues));
    if (small)
        hipLaunchKernelGGL((cull_kernel<MODE, Hit, kCullGroupSmall>), grid, dim3(kBlock), 0, st, hit, ra, out, adj, list,
                           count);
    else
        hipLaunchKernelGGL((cull_kernel<MODE, Hit>), grid, dim3(kBlock), 0, st, hit, ra, out, adj, list, count);
    return hipGetLastError();
}

// Runs launch(ra) with the launch's queue counters set; rays are the slots.
// ws: caller-provided scratch of at least list_scratch_bytes(n_slots) bytes
// (nothing is allocated), or nullptr to take it from the pool. extra: a counter
// that starts at zero with the launch, or nullptr.
template <typename Launch>
static hipError_t with_queue(const RayArgs& ra_in, hipStream_t st, Launch&& launch, void* ws = nullptr,
                             unsigned long long* extra = nullptr) {
    RayArgs ra = ra_in;
    void* q = ws;
    hipError_t e = ws ? hipSuccess : work_alloc(&q, kQueues * kQueueStride * sizeof(unsigned long long), st);
    if (e != hipSuccess) return e;
    ra.queue = static_cast<unsigned long long*>(q);
    hipLaunchKernelGGL(zero_queue_kernel, dim3(1), dim3(kQueues * kQueueStride), 0, st, ra.queue, extra);
    e = hipGetLastError();
    if (e == hipSuccess) e = launch(ra);
    const hipError_t f = ws ? hipSuccess : work_free(q, st);
    return e != hipSuccess ? e : f;
}

static_assert(2 * kQueues * kQueueStride * sizeof(unsigned long long) == kListHeaderBytes,
              "candidate-list header size");

// Candidate form: cull(list, count) lists the rays, then launch(ra) runs over
// them. Ray indices must fit int32; larger launches take the slot form (the
// render kernels then test every ray themselves). ws and extra as in with_queue.
template <typename Cull, typename Launch>
static hipError_t with_list(const RayArgs& ra_in, hipStream_t st, Cull&& cull, Launch&& launch,
                            void* ws = nullptr, unsigned long long* extra = nullptr) {
    if (ra_in.n > (int64_t)INT32_MAX) return with_queue(ra_in, st, launch, ws, extra);
    const size_t qbytes = kListHeaderBytes;
    RayArgs ra = ra_in;
    void* q = ws;
    hipError_t e = ws ? hipSuccess : work_alloc(&q, list_scratch_bytes(ra_in.n_slots), st);
    if (e != hipSuccess) return e;
    ra.queue = static_cast<unsigned long long*>(q);
    unsigned long long* count = ra.queue + kQueues * kQueueStride;
    int32_t* list = reinterpret_cast<int32_t*>(static_cast<char*>(q) + qbytes);
    ra.count = count;
    ra.list = list;
    hipLaunchKernelGGL(zero_queue_kernel, dim3(1), dim3(2 * kQueues * kQueueStride), 0, st, ra.queue, extra);
    e = hipGetLastError();
    if (e == hipSuccess) e = cull(list, count);
    if (e == hipSuccess) e = launch(ra);
    const hipError_t f = ws ? hipSuccess : work_free(q, st);
    return e != hipSuccess ? e : f;
}

// Candidate form of a forward: the cull pass of one placed tree. The counter of
// out's trace, if it has one, starts at zero.
template <typename Launch>
static hipError_t with_candidates(const TreeArgs& tr, const InstArgs& in, const RayArgs& ra_in, const RenderOut& out,
                                  hipStream_t st, Launch&& launch, void* ws = nullptr) {
    return with_list(
        ra_in, st,
        [&](int32_t* list, unsigned long long* count) {
            if (in.identity)
                return launch_cull_hit<0>(TreeHit<true>{tr, in}, ra_in, out, CullAdjoint{}, list, count, st);
            return launch_cull_hit<0>(TreeHit<false>{tr, in}, ra_in, out, CullAdjoint{}, list, count, st);
        },
        launch, ws, out.trace.head ? out.trace.counter : nullptr);
}

// ----------------------------------------------------------------------------
// records of the two-phase adjoint (see RecordArgs)

// LDS rows per wavefront for the transposition of finished leaf rows
constexpr int kFlushSlots = 16;

// Clears hdr (n_hdr counters) and sets the n leaf heads to "no record".
static __global__ void adjoint_init_kernel(unsigned long long* hdr, int n_hdr, int32_t* head, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) head[i] = -1;
    if (i < n_hdr) hdr[i] = 0ull;
}

// Wave-uniform allocation of n (<= 128) consecutive items of a room of cap
// items, out of blocks of BLOCK(cap) taken from its counter. [cur, end) is what is left of
// the wavefront's current block, end = -1 once the room is exhausted. Returns
// the first item, or -1 when there is no room. A request that fails has left
// the counter above cap. Call with every lane of the wavefront active.
template <int (*BLOCK)(int64_t) = item_block>
__device__ __forceinline__ int take_items(unsigned long long* counter, int64_t cap, int n, int& cur, int& end) {
    if (!items_fit(cur, end, n)) {
        if (end < 0) return -1;
        const int block = BLOCK(cap);
        unsigned long long b = 0;
        if ((threadIdx.x & 63) == 0) b = atomicAdd(counter, (unsigned long long)block);
        const uint32_t b_lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
        const uint32_t b_hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
        open_block((int64_t)(((uint64_t)b_hi << 32) | b_lo), cap, block, cur, end);
        if (!items_fit(cur, end, n)) {
            end = -1;
            return -1;
        }
    }
    const int at = cur;
    cur += n;
    return at;
}

// Linking one iteration's records into their leaves' lists. The records of
// the lanes with a sample (mask hm) are consecutive in lane order. A run is a
// maximal sequence of such lanes, consecutive in that order, on one leaf: its
// first lane links the whole run with one atomic exchange of the leaf's head
// (the head becomes the run's last record, and the first record links to the
// old head), and every other lane links its record to the record before it.
// count: the run's length for its first lane, 0 for the others. Call with
// every lane of the wavefront active.
struct RecordRun {
    int count;
};
__device__ __forceinline__ RecordRun record_run(uint64_t hm, bool has, int leaf) {
    const int lane = threadIdx.x & 63;
    const uint64_t below = (1ull << lane) - 1ull;
    const uint64_t hb = hm & below;
    const int pred = hb ? 63 - __builtin_clzll(hb) : lane;   // the previous lane with a sample
    const int pleaf = __builtin_amdgcn_ds_bpermute(pred << 2, leaf);
    const bool start = has && (hb == 0ull || pleaf != leaf);
    const uint64_t starts = __ballot(start);
    RecordRun r{0};
    if (start) {
        const uint64_t later = starts & ~((2ull << lane) - 1ull);   // starts above this lane (none: lane 63)
        const uint64_t upto = later ? (1ull << __builtin_ctzll(later)) - 1ull : ~0ull;
        r.count = __popcll(hm & upto & ~below);
    }
    return r;
}

// The list that the records of one iteration, the first of which is `at`, join
// for a leaf: the leaf's only one, or one of 2^split picked by the record's
// index, so that the records of a leaf spread over all of them.
__device__ __forceinline__ int64_t record_list(const RecordArgs& rec, int64_t n_leaves, int leaf, int at) {
    if (rec.split == 0) return leaf;
    return (int64_t)(((uint32_t)at * 0x9E3779B1u) >> (32 - rec.split)) * n_leaves + leaf;
}

// Whether every sample of the call is sure to get a record: the samples and
// rays the cull pass counted, an unused block for every wavefront that takes
// rays (of the persistent grids of the walk and the replay: no more than chunks
// of rays), and the up to 63 items that a request leaves behind at a block's end. Then nothing is scattered, and a call that
// writes its gradient rows (fresh) may leave them uninitialised until the
// reduction stores them, each once; else they are cleared before anything is
// added. The same answer for every thread of the call's kernels.
__device__ __forceinline__ bool records_fit(const RecordArgs& rec) {
    if (!rec.head) return false;
    int64_t samples = 0, waves = 0;
#pragma unroll
    for (int list = 0; list < 2; ++list) {
        int64_t chunks = 0;
#pragma unroll
        for (int x = 0; x < kQueues; ++x) {   // (the replaying rays' counts lie two groups of lines on)
            const unsigned long long* c = rec.counts + (list * 2 * kQueues + x) * kQueueStride;
            chunks += ((int64_t)c[0] + 63) >> 6;
            samples += (int64_t)c[1];
        }
        waves += chunks < rec.max_waves ? chunks : rec.max_waves;
    }
    const int64_t block = record_block(rec.cap);
    return samples >= 0 && (samples / (block - 63) + 1 + waves) * block <= rec.cap;
}

// Clears the n float4 of a fresh call's gradient rows unless the reduction will
// write every one of them.
static __global__ __launch_bounds__(kBlock) void fresh_clear_kernel(RecordArgs rec, float4* rows, int64_t n) {
    if (records_fit(rec)) return;
    for (int64_t i = blockIdx.x * (int64_t)kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock)
        rows[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}

// Basis gradients of a reduction with one time for every ray: n components per
// wavefront (lane c: component c) are summed in float64 over the block and the
// grid, and basis_finish_kernel adds the sums to the two frames' rows. (They
// are sums over all leaves of terms of either sign: added to the rows block by
// block in float32, their last bits differed by up to 4e-7 from run to run.)
// s: n doubles of LDS, zero and synchronised; at: the components' place in
// basis_sum. Call with the whole block.
__device__ __forceinline__ void basis_add(const RecordArgs& rec, double* s, int at, int n, double v) {
    if ((int)(threadIdx.x & 63) < n) atomicAdd(s + (threadIdx.x & 63), v);
    __syncthreads();
    if ((int)threadIdx.x < n) unsafeAtomicAdd(rec.basis_sum + at + threadIdx.x, s[threadIdx.x]);
}
// One block: adds the sums of C density and Cg hyperangle components.
static __global__ void basis_finish_kernel(TreeArgs tr, InstArgs in, float t, RecordArgs rec, int C, float* grad_basis,
                                           int Cg, float* grad_basis_g) {
    const int c = threadIdx.x;
    const bool dens = c < C;
    float* grad = dens ? grad_basis : grad_basis_g;
    if (c >= C + Cg || !grad) return;
    int i0, i1;
    float f;
    time_setup(tr, in, t, i0, i1, f);
    const int n = dens ? C : Cg, e = dens ? c : c - C;
    const double v = rec.basis_sum[c];
    unsafeAtomicAdd(grad + (int64_t)i0 * n + e, (float)((1.0 - (double)f) * v));
    if (f != 0.0f) unsafeAtomicAdd(grad + (int64_t)i1 * n + e, (float)((double)f * v));
}

// Hands leaves with records to the idle lanes of a reduction wavefront.
// Wavefront w takes 64-leaf batches w, w + W, ...; a batch's heads are read in
// one load (lane = leaf) and its leaves with records are compacted into a
// per-wavefront LDS queue of {leaf, first record}, from which idle lanes take
// entries in lane order.
struct LeafFeeder {
    int64_t batch;     // next batch of this wavefront
    int64_t n_waves;
    int cnt, pos;      // wave-uniform: queue entries, entries handed out
    bool more;         // wave-uniform: batches may be left
};

__device__ __forceinline__ LeafFeeder leaf_feeder(int wave_in_block) {
    LeafFeeder f;
    f.batch = (int64_t)blockIdx.x * (kBlock / kWave) + wave_in_block;
    f.n_waves = (int64_t)gridDim.x * (kBlock / kWave);
    f.cnt = f.pos = 0;
    f.more = true;
    return f;
}

// Gradient rows of calls with one time for every ray are stored non-temporally:
// what they would push out of L2 are the lines of records that a wavefront's
// lists share (per-point step's reduction of 1 GB of rows 442 -> 419 us, the
// ring's of 512 MB 413 -> 403 us, 256 MB of 30 coefficients 149 -> 127 us). A
// training batch with a time per ray touches few rows and reads them next: kept
// in the caches, its reduction takes 36 instead of 35 us, the unpacking after it
// 34 instead of 48 us. Zero rows follow the size of all rows: what the 256 MB
// last-level cache can hold with what follows is stored as usual.
constexpr int64_t kStreamRows = 192ll << 20;
template <bool STREAM>
__device__ __forceinline__ void store_row_value(float* at, float v) {
    if constexpr (STREAM) __builtin_nontemporal_store(v, at);
    else *at = v;
}
__device__ __forceinline__ void store_row4_zero(float4* at, bool stream) {
    typedef float v4 __attribute__((ext_vector_type(4)));
    if (stream) __builtin_nontemporal_store(v4{0.0f, 0.0f, 0.0f, 0.0f}, reinterpret_cast<v4*>(at));
    else *at = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
}

// Writes zero rows of ROW floats for the leaves of the batch at b0 (of up to
// `batch` leaves) whose bit is set in m: sixteen bytes per lane, whole rows per
// instruction.
template <int ROW>
__device__ __forceinline__ void zero_batch_rows(float* rows, int64_t b0, uint64_t m, int64_t n_leaves,
                                                int batch = kWave) {
    constexpr int per = ROW / 4;   // float4 per row
    const bool stream = n_leaves * (int64_t)(ROW * sizeof(float)) > kStreamRows;
    float4* p = reinterpret_cast<float4*>(rows + b0 * ROW);
    for (int i = threadIdx.x & 63; i < batch * per; i += kWave)
        if ((m >> (i / per)) & 1ull) store_row4_zero(p + i, stream);
}

// Gives idle lanes (leaf < 0) a leaf and its first record while leaves are left.
// q: this wavefront's LDS queue of kWave entries. fresh: the rows (of ROW floats)
// of leaves without records are written here, as zeros. Call with every lane active.
template <int ROW>
__device__ __forceinline__ void feed_leaves(LeafFeeder& f, const RecordArgs& rec, int64_t n_leaves, int2* q,
                                            int& leaf, int& first, bool fresh, float* rows) {
    const int lane = threadIdx.x & 63;
    for (;;) {
        const uint64_t idle = __ballot(leaf < 0);
        if (!idle || !f.more) break;
        if (f.pos >= f.cnt) {
            const int64_t b0 = f.batch * kWave;
            f.batch += f.n_waves;
            if (b0 >= n_leaves) {
                f.more = false;
                break;
            }
            const int64_t L = b0 + lane;
            const int h = L < n_leaves ? rec.head[L] : -1;
            const uint64_t m = __ballot(h >= 0);
            if (fresh) zero_batch_rows<ROW>(rows, b0, __ballot(L < n_leaves) & ~m, n_leaves);
            __builtin_amdgcn_wave_barrier();
            if (h >= 0) q[lane_rank(m)] = make_int2((int)L, h);
            __builtin_amdgcn_wave_barrier();
            f.cnt = __popcll(m);
            f.pos = 0;
            continue;
        }
        const int avail = f.cnt - f.pos, n_idle = __popcll(idle);
        if (leaf < 0) {
            const int r = lane_rank(idle);
            if (r < avail) {
                const int2 e = q[f.pos + r];
                leaf = e.x;
                first = e.y;
            }
        }
        f.pos += n_idle < avail ? n_idle : avail;
    }
}

// Scratch of one adjoint call, taken from the pool in one piece and initialised
// by one kernel: the queues and list counts of the rays that walk and of those
// that replay their trace, the lists, the counter of records, the leaf heads
// and the records (32 bytes each, as many of the room as the device has memory
// for; with none rec stays empty: per-sample atomics only). One cull pass then lists the rays. (An allocation,
// a clearing kernel and a cull pass per list and another of each for the
// records cost an adjoint of four 1920 x 1080 layers about 25 us a layer.)
struct AdjointScratch {
    RayArgs walk, replay;
    RecordArgs rec;
    void* mem;
};
struct NoHit {};
// Whether an adjoint with room for cap records replays a trace with room for
// `samples`: only where every traced sample may get a record. The replay keeps
// no basis and makes one for each sample it has to scatter, so with few records
// or none the rays walk instead, whose lanes hold their basis (a 1920 x 1080
// step without records 2236 us replayed, 929 us walked; a per-point 960 x 540
// step 2666 and 1217 us).
static bool replays(const TraceArgs& trace, int64_t samples, int64_t cap) { return trace.head && cap > 0 && cap >= samples; }
static hipError_t adjoint_begin(const TreeArgs& tr, const RayArgs& ra, const int32_t* nsamp, const int32_t* trace_head,
                                const RecordRoom& room, hipStream_t st, AdjointScratch& s, int split = 0) {
    s = AdjointScratch{ra, ra, RecordArgs{}, nullptr};
    const bool listed = ra.n <= (int64_t)INT32_MAX;   // else the slot form: the walking kernel tests every ray
    if (trace_head && !listed) return hipErrorInvalidValue;
    constexpr int kCounters = kQueues * kQueueStride;
    constexpr int n_hdr = 4 * kCounters + kQueueStride + 64;   // (the last 64 start as the float64 zeros of basis_sum)
    constexpr size_t hdr = ((size_t)n_hdr * sizeof(unsigned long long) + 255) & ~(size_t)255;
    const size_t list_b = listed ? (size_t)((ra.n_slots + 63) >> 6) * 64 * sizeof(int32_t) : 0;
    const size_t lists = trace_head ? 2 * list_b : list_b;
    const int64_t n_heads = room.most > 0 ? tr.n_leaves << split : 0;
    const size_t head_b = ((size_t)n_heads * sizeof(int32_t) + 255) & ~(size_t)255;
    int64_t cap = 0;
    hipError_t e = take_room(
        room, cap, [&](int64_t records) { return work_alloc(&s.mem, hdr + lists + head_b + (size_t)records * 2 * sizeof(int4), st); },
        [](hipError_t a) { return a == hipErrorOutOfMemory; });
    if (e != hipSuccess) {
        s.mem = nullptr;
        return e;
    }
    char* p = static_cast<char*>(s.mem);
    auto* counters = reinterpret_cast<unsigned long long*>(p);
    auto* list = reinterpret_cast<int32_t*>(p + hdr);
    auto* list2 = reinterpret_cast<int32_t*>(p + hdr + list_b);
    s.walk.queue = counters;
    s.replay.queue = counters + 2 * kCounters;
    if (cap > 0) {
        s.rec.counter = counters + 4 * kCounters;
        s.rec.counts = counters + kCounters;
        s.rec.basis_sum = reinterpret_cast<double*>(counters + 4 * kCounters + kQueueStride);
        s.rec.head = reinterpret_cast<int32_t*>(p + hdr + lists);
        s.rec.rec = reinterpret_cast<int4*>(p + hdr + lists + head_b);
        s.rec.split = split;
        s.rec.cap = cap;
    }
    const int64_t n_init = n_heads > n_hdr ? n_heads : n_hdr;
    hipLaunchKernelGGL(adjoint_init_kernel, dim3((unsigned)((n_init + 255) / 256)), dim3(256), 0, st, counters, n_hdr,
                       s.rec.head, n_heads);
    e = hipGetLastError();
    if (e == hipSuccess && listed) {
        s.walk.list = list;
        s.walk.count = counters + kCounters;
        s.replay.list = list2;
        s.replay.count = counters + 3 * kCounters;
        const CullAdjoint adj{nsamp, trace_head, list2, counters + 3 * kCounters};
        e = launch_cull_hit<1>(NoHit{}, ra, RenderOut{}, adj, list, counters + kCounters, st);
    }
    return e;
}
// Before a fresh call's rays: its rows of `row` floats are cleared where the
// reduction cannot be relied on to write them, or adds several lists to each.
static hipError_t fresh_begin(const TreeArgs& tr, const BackwardIO& io, int row, const RecordArgs& rec, hipStream_t st) {
    const int64_t n = tr.n_leaves * (int64_t)(row / 4);
    if (n <= 0) return hipSuccess;
    if (rec.split > 0) return launch_zero_rows(io.grad_leaf, 4 * n, st);
    const int64_t want = (n + kBlock - 1) / kBlock, cap = (int64_t)device_cu_count() * 4;
    hipLaunchKernelGGL(fresh_clear_kernel, dim3((unsigned)(want < cap ? want : cap)), dim3(kBlock), 0, st, rec,
                       reinterpret_cast<float4*>(io.grad_leaf), n);
    return hipGetLastError();
}
// The kernels over an adjoint's rays: walk for those on the first list, replay
// (if any ray may replay) for those on the second.
template <class Kernel>
static hipError_t adjoint_rays(Kernel walk, Kernel replay_kernel, bool replay, int row, const TreeArgs& tr,
                               const InstArgs& in, const BackwardIO& io, AdjointScratch& s, hipStream_t st) {
    const int walk_grid = grid_for(walk, s.walk), replay_grid = replay ? grid_for(replay_kernel, s.replay) : 0;
    s.rec.max_waves = (walk_grid > replay_grid ? walk_grid : replay_grid) * (kBlock / kWave);
    hipError_t e = io.fresh ? fresh_begin(tr, io, row, s.rec, st) : hipSuccess;
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(walk, dim3(walk_grid), dim3(kBlock), 0, st, tr, in, s.walk, io, s.rec);
    e = hipGetLastError();
    if (e != hipSuccess || !replay) return e;
    hipLaunchKernelGGL(replay_kernel, dim3(replay_grid), dim3(kBlock), 0, st, tr, in, s.replay, io, s.rec);
    return hipGetLastError();
}
static hipError_t adjoint_end(const AdjointScratch& s, hipError_t e, hipStream_t st) {
    const hipError_t f = s.mem ? work_free(s.mem, st) : hipSuccess;
    return e != hipSuccess ? e : f;
}

}  // namespace neuvv
