// Device-side building blocks of the VOctree renderer (gfx950).
//
//  * float64 ray geometry, so that segment lengths inside leaves keep float32
//               relative accuracy even when the ray parameter is thousands of
//               leaf units large (evaluation and compositing are float32);
//  * hh_all:    the first 30 real 4-D hyperspherical harmonics (Sec. 4.1,
//               Eq. 2-3, Appendix A.2) as closed-form polynomials;
//  * RaySetup:  instance transform and re-timing of one ray (Eq. 13), clip to
//               the tree box, per-ray HH basis and density-basis row (Eq. 4, 5);
//  * walk_next: the next occupied leaf along the ray (Sec. 4.3 "Rendering"),
//               skipping whole empty octree cubes; the octree is stored two
//               levels per node (64-bit occupancy mask + base index), a
//               directory maps each 4^3 region of leaf cells to its
//               last-level node (a "brick") or to the largest empty cube
//               around it, and the current brick's node is kept in registers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace neuvv {

constexpr int kMaxDepth = 12;
constexpr int kWave = 64;

// 12-byte vector access to a ray's origin or direction, or a pixel's colour
// (one dwordx3 memory instruction instead of three).
typedef float f3v __attribute__((ext_vector_type(3)));
__device__ __forceinline__ f3v load3(const float* p) {
    f3v v;
    __builtin_memcpy(&v, p, 12);
    return v;
}
__device__ __forceinline__ void store3(float* p, float x, float y, float z) {
    const f3v v = {x, y, z};
    __builtin_memcpy(p, &v, 12);
}

// ----------------------------------------------------------------------------
// float64 geometry. A wave64 v_add/mul/fma_f64 issues in the four cycles of an
// unpacked float32 one on gfx950 (78 TFLOP/s either way), so one float64
// instruction replaces the 8 to 20 of the same operation on a compensated
// float32 pair, which the walk used before, and carries 53 bits instead of 48.
// Measured against the pairs: forward call of one 1920 x 1080 view 0.29 -> 0.20 ms,
// stereo frame of 2 x 2048 x 2048 rays with its camera rays 0.53 -> 0.35 ms,
// ring step of 16.6 M rays 2.24 -> 2.11 ms.

// 1/d: the hardware estimate (about 24 bits) refined by two Newton steps.
__device__ __forceinline__ double rcp64(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
    return __builtin_fma(r, __builtin_fma(-d, r, 1.0), r);
}

// ----------------------------------------------------------------------------
// Real 4-D hyperspherical harmonics H_nlm(d, gamma) = g_nl(gamma) Y_lm(d)
// with g_nl = A_nl sin^l(gamma) C^{l+1}_{n-l}(cos gamma), A_nl =
// (2l)!! sqrt(2 (n+1) (n-l)! / (pi (n+l+1)!)), and Y_lm the orthonormal real
// spherical harmonic of the unit direction d = (x, y, z), polar axis z, no
// Condon-Shortley phase (cos m phi for m > 0, sin |m| phi for m < 0). Order:
// n = 0.., l = 0..n, m = -l..l. Constants are the closed forms evaluated.
// Radial factors g_nl of the hyperangle gamma, n + l <= 3 (order g00, g10, g11,
// g20, g21, g22, g30, g31, g32, g33).
__device__ __forceinline__ void hh_radial(float gam, float (&g)[10]) {
    float s, c;
    sincosf(gam, &s, &c);
    const float c2 = c * c, s2 = s * s;
    g[0] = 0.7978845608028654f;                        // sqrt(2/pi)
    g[1] = 1.5957691216057308f * c;                    // 2 sqrt(2/pi) cos
    g[2] = 0.9213177319235613f * s;                    // 2 sqrt(2/(3pi)) sin
    g[3] = 0.7978845608028654f * (4.0f * c2 - 1.0f);   // sqrt(2/pi) U_2
    g[4] = 2.256758334191025f * s * c;                 // (1/sqrt(pi)) sin * 4 cos
    g[5] = 1.009253008808064f * s2;                    // 8/sqrt(20 pi) sin^2
    g[6] = 0.7978845608028654f * c * (8.0f * c2 - 4.0f);    // sqrt(2/pi) U_3
    g[7] = 0.41202581549140227f * s * (12.0f * c2 - 2.0f);  // 2 sqrt(2/(15pi)) sin C^2_2
    g[8] = 2.854598585844434f * c * s2;                // 8/sqrt(90 pi) sin^2 * 6 cos
    g[9] = 1.0789368501515768f * s2 * s;               // 48/sqrt(630 pi) sin^3
}

// The 30 HH values from the radial factors and the unit direction (x, y, z):
// h = g_nl Y_lm with real spherical harmonics up to degree 3.
__device__ __forceinline__ void hh_assemble(const float (&g)[10], float x, float y, float z, float (&h)[30]) {
    const float x2 = x * x, y2 = y * y, z2 = z * z;
    const float Y00 = 0.28209479177387814f;
    const float k1 = 0.4886025119029199f;
    const float Y1n1 = k1 * y, Y10 = k1 * z, Y11 = k1 * x;
    const float k2 = 1.0925484305920792f;
    const float Y2n2 = k2 * x * y, Y2n1 = k2 * y * z, Y20 = 0.31539156525252005f * (3.0f * z2 - 1.0f);
    const float Y21 = k2 * x * z, Y22 = 0.5462742152960396f * (x2 - y2);
    const float k33 = 0.5900435899266435f, k31 = 0.4570457994644658f;
    const float Y3n3 = k33 * y * (3.0f * x2 - y2), Y3n2 = 2.890611442640554f * x * y * z;
    const float Y3n1 = k31 * y * (5.0f * z2 - 1.0f), Y30 = 0.3731763325901154f * z * (5.0f * z2 - 3.0f);
    const float Y31 = k31 * x * (5.0f * z2 - 1.0f), Y32 = 1.445305721320277f * z * (x2 - y2);
    const float Y33 = k33 * x * (x2 - 3.0f * y2);
    h[0] = g[0] * Y00;
    h[1] = g[1] * Y00;
    h[2] = g[2] * Y1n1; h[3] = g[2] * Y10; h[4] = g[2] * Y11;
    h[5] = g[3] * Y00;
    h[6] = g[4] * Y1n1; h[7] = g[4] * Y10; h[8] = g[4] * Y11;
    h[9] = g[5] * Y2n2; h[10] = g[5] * Y2n1; h[11] = g[5] * Y20; h[12] = g[5] * Y21; h[13] = g[5] * Y22;
    h[14] = g[6] * Y00;
    h[15] = g[7] * Y1n1; h[16] = g[7] * Y10; h[17] = g[7] * Y11;
    h[18] = g[8] * Y2n2; h[19] = g[8] * Y2n1; h[20] = g[8] * Y20; h[21] = g[8] * Y21; h[22] = g[8] * Y22;
    h[23] = g[9] * Y3n3; h[24] = g[9] * Y3n2; h[25] = g[9] * Y3n1; h[26] = g[9] * Y30;
    h[27] = g[9] * Y31; h[28] = g[9] * Y32; h[29] = g[9] * Y33;
}

__device__ __forceinline__ void hh_all(float x, float y, float z, float gam, float (&h)[30]) {
    float g[10];
    hh_radial(gam, g);
    hh_assemble(g, x, y, z, h);
}

// Per-point hyperangle form (Eq. 6), first 14 functions (all n <= 2): the
// direction factors are per ray, the radial factors per sample.
// Y = (Y1-1, Y10, Y11, Y2-2, Y2-1, Y20, Y21, Y22) of the unit direction; Y00 is
// the constant 1 / (2 sqrt(pi)).
constexpr float kY00 = 0.28209479177387814f;
__device__ __forceinline__ void sh_deg2(float x, float y, float z, float (&Y)[8]) {
    const float k1 = 0.4886025119029199f, k2 = 1.0925484305920792f;
    Y[0] = k1 * y; Y[1] = k1 * z; Y[2] = k1 * x;
    Y[3] = k2 * x * y; Y[4] = k2 * y * z; Y[5] = 0.31539156525252005f * (3.0f * z * z - 1.0f);
    Y[6] = k2 * x * z; Y[7] = 0.5462742152960396f * (x * x - y * y);
}
// g = (g00, g10, g11, g20, g21, g22)(gamma) and their derivatives in gamma,
// from s = sin(gamma), c = cos(gamma); same closed forms as hh_all.
__device__ __forceinline__ void radial_n2(float s, float c, float (&g)[6], float (&dg)[6]) {
    const float a0 = 0.7978845608028654f, a1 = 1.5957691216057308f, b1 = 0.9213177319235613f;
    const float d1 = 2.256758334191025f, e2 = 1.009253008808064f;
    g[0] = a0;                         dg[0] = 0.0f;
    g[1] = a1 * c;                     dg[1] = -a1 * s;
    g[2] = b1 * s;                     dg[2] = b1 * c;
    g[3] = a0 * (4.0f * c * c - 1.0f); dg[3] = -8.0f * a0 * c * s;
    g[4] = d1 * s * c;                 dg[4] = d1 * (c * c - s * s);
    g[5] = e2 * s * s;                 dg[5] = 2.0f * e2 * s * c;
}
// h_k = g_{n(k) l(k)} Y_{l(k) m(k)} in the canonical order of the first 14.
__device__ __forceinline__ void hh14(const float (&g)[6], const float (&Y)[8], float (&h)[14]) {
    h[0] = g[0] * kY00;
    h[1] = g[1] * kY00;
    h[2] = g[2] * Y[0]; h[3] = g[2] * Y[1]; h[4] = g[2] * Y[2];
    h[5] = g[3] * kY00;
    h[6] = g[4] * Y[0]; h[7] = g[4] * Y[1]; h[8] = g[4] * Y[2];
    h[9] = g[5] * Y[3]; h[10] = g[5] * Y[4]; h[11] = g[5] * Y[5]; h[12] = g[5] * Y[6]; h[13] = g[5] * Y[7];
}

// ----------------------------------------------------------------------------
// kernel-side descriptions of the tree, instance and rays

struct TreeArgs {
    const int4* nodes;   // [n_nodes] {mask lo, mask hi, first child, 0}
    const void* hh;
    const void* wsig;
    const float* basis;
    const float* gamma;
    int64_t n_nodes;
    int64_t n_leaves;
    int32_t depth;
    int32_t T;
    int32_t box_lo[3];   // occupied-cell bounds: rays are clipped to [lo, hi)
    int32_t box_hi[3];
    int32_t layout;      // 0: vectors structure-of-arrays, 1: leaf-major rows of vectors
    int32_t Cg;          // per-point hyperangle weights per leaf (0: the global table gamma)
    const void* wgam;    // [N] rows of Cg weights, storage dtype and layout of wsig
    const float* basis_g;   // [T][Cg] hyperangle basis
    const float4* edit;     // nullptr, or [N][2] rows {r, g, b, sigma_d}, {t_d, owner, 0, 0} (appearance edits)
    int32_t relu;           // density activation of Eq. 5: 0 softplus, 1 ReLU
    const int32_t* dir;     // brick directory (directory_entries(depth) entries; see walk_next)
};

struct InstArgs {
    float rot[9];
    float trans[3];
    float scale;
    float time_offset;
    int32_t wrap;
    int32_t identity;
};

struct RayArgs {
    const float* o;
    const float* d;
    const float* t;      // nullptr: t_scalar for every ray
    float t_scalar;
    int32_t img_w;       // > 0: rays form a row-major image of this width
    int32_t tiles_x;
    int64_t n;
    int64_t n_slots;     // work slots (64 per 8x8 tile when img_w > 0, else n)
    int32_t refill_min;  // idle lanes that trigger a refill of the wavefront
    unsigned long long* queue;   // work-queue counters of the launch (set by the launcher)
    // candidate form (set by the launcher): the rays a cull pass kept, listed in
    // the slot range of their XCD part, with the per-part counts; nullptr: the
    // work items are the slots themselves
    const int32_t* list;
    const unsigned long long* count;
};

// Work slot -> ray index, -1 when the slot is padding of a ragged tile.
__device__ __forceinline__ int64_t slot_to_ray(const RayArgs& ra, int64_t slot) {
    if (ra.img_w <= 0) return slot < ra.n ? slot : -1;
    int64_t tile = slot >> 6;
    int within = (int)(slot & 63);
    int64_t ty = tile / ra.tiles_x, tx = tile - ty * ra.tiles_x;
    int64_t px = tx * 8 + (within & 7), py = ty * 8 + (within >> 3);
    if (px >= ra.img_w) return -1;
    int64_t r = py * ra.img_w + px;
    return r < ra.n ? r : -1;
}

// Per-ray constants: local ray x_l(u) = O + u D with the world parameter u,
// reciprocal direction, box interval [u_in, u_out), frame interpolation.
struct RaySetup {
    // the walk's ray, mirrored on the axes it moves down: D >= 0, inv = 1/D > 0 (0 and +inf on an
    // axis it does not move along), flip = -1 on a mirrored axis, else 0
    double O[3], D[3], inv[3];
    int flip[3];
    double u_in, u_out;
    float len_local;   // |D|: leaf units per unit of u
    float len_world;   // |d|: world distance per unit of u
    float dir[3];      // unit local direction
    int i0, i1;
    float f;
    float tau;         // local time after re-timing (appearance edits are gated on it)
    bool hit;
};

// Re-timing (Eq. 13): tau = t + offset, wrapped into [0, T) or clamped into
// [0, T-1]; frames i0 = floor(tau), i1 = min(i0 + 1, T - 1), weight f = tau - i0
// (0 on the held last frame). tau is float64 so f is accurate.
__device__ __forceinline__ void time_setup(const TreeArgs& tr, const InstArgs& in, float t, int& i0_out,
                                           int& i1_out, float& f_out, float* tau_out = nullptr) {
    const int T = tr.T;
    const double Td = (double)T;
    double tau = (double)t + (double)in.time_offset;
    if (in.wrap) {
        tau = __builtin_fma(-__builtin_floor(tau / Td), Td, tau);
        if (tau < 0.0) tau += Td;
        if (!(tau < Td)) tau -= Td;
        if (tau < 0.0) tau = 0.0;
    } else {
        if (tau < 0.0) tau = 0.0;
        if (tau > Td - 1.0) tau = Td - 1.0;
    }
    int i0 = (int)__builtin_floor(tau);
    i0 = i0 < 0 ? 0 : (i0 > T - 1 ? T - 1 : i0);
    float f = (float)(tau - (double)i0);
    if (i0 == T - 1) f = 0.0f;
    i0_out = i0;
    i1_out = i0 + 1 < T ? i0 + 1 : T - 1;
    f_out = f;
    if (tau_out) *tau_out = (float)tau;
}

// IDENT: the instance is the identity (known at compile time), so the local
// ray is the world ray.
// Coarse reject in plain float against the occupied box grown by one leaf on
// every side: float rounding of the clip is far below that margin for any
// local coordinate below ~1e5, so a ray rejected here misses the exact box.
// Returns false only for such rays.
template <bool IDENT>
__device__ __forceinline__ bool ray_may_hit(const TreeArgs& tr, const InstArgs& in, const float o[3],
                                            const float d[3]) {
    float of[3], dfl[3];
    if constexpr (IDENT) {
#pragma unroll
        for (int a = 0; a < 3; ++a) { of[a] = o[a]; dfl[a] = d[a]; }
    } else {
        const float is = 1.0f / in.scale;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            of[a] = ((o[0] - in.trans[0]) * in.rot[a] + (o[1] - in.trans[1]) * in.rot[3 + a] +
                     (o[2] - in.trans[2]) * in.rot[6 + a]) * is;
            dfl[a] = (d[0] * in.rot[a] + d[1] * in.rot[3 + a] + d[2] * in.rot[6 + a]) * is;
        }
    }
    float tn = 0.0f, tf = INFINITY;
    bool pass = true, small = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        small = small && fabsf(of[a]) < 1.0e5f;
        const float lo = (float)tr.box_lo[a] - 1.0f, hi = (float)tr.box_hi[a] + 1.0f;
        if (dfl[a] == 0.0f) {
            pass = pass && of[a] >= lo && of[a] < hi;
        } else {
            const float iv = __builtin_amdgcn_rcpf(dfl[a]);   // 1 ulp: far inside the margin
            const float t0 = (lo - of[a]) * iv, t1 = (hi - of[a]) * iv;
            tn = fmaxf(tn, fminf(t0, t1));
            tf = fminf(tf, fmaxf(t0, t1));
        }
    }
    return !small || (pass && tn < tf);
}

// Local direction of a ray (D = R^T d / s), |D| (leaf units per unit of the ray
// parameter), |d| and the unit local direction; dmax = the largest |D| component.
template <bool IDENT>
__device__ __forceinline__ void ray_direction(const InstArgs& in, const float d[3], RaySetup& rs, float& dmax) {
    if constexpr (IDENT) {
#pragma unroll
        for (int a = 0; a < 3; ++a) rs.D[a] = (double)d[a];
    } else {
        const double is = rcp64((double)in.scale);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            double ad = (double)d[0] * (double)in.rot[a];
            ad = __builtin_fma((double)d[1], (double)in.rot[3 + a], ad);
            ad = __builtin_fma((double)d[2], (double)in.rot[6 + a], ad);
            rs.D[a] = ad * is;
        }
    }
    float dl2 = 0.0f, dw2 = 0.0f;
    dmax = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        float v = (float)rs.D[a];
        dl2 += v * v;
        dw2 += d[a] * d[a];
        dmax = fmaxf(dmax, fabsf(v));
    }
    rs.len_local = sqrtf(dl2);
    rs.len_world = sqrtf(dw2);
    const float inv_len = rs.len_local > 0.0f ? 1.0f / rs.len_local : 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) rs.dir[a] = (float)rs.D[a] * inv_len;
    if (!(rs.len_local > 0.0f)) rs.dir[2] = 1.0f;
}

// Exact geometry of a ray (float64): everything of RaySetup but its time; call
// for rays ray_may_hit accepts.
template <bool IDENT>
__device__ __forceinline__ void ray_geometry(const TreeArgs& tr, const InstArgs& in, const float o[3],
                                             const float d[3], RaySetup& rs) {
    float dmax;
    ray_direction<IDENT>(in, d, rs, dmax);
    if constexpr (IDENT) {
#pragma unroll
        for (int a = 0; a < 3; ++a) rs.O[a] = (double)o[a];
    } else {
        double diff[3];
#pragma unroll
        for (int b = 0; b < 3; ++b) diff[b] = (double)o[b] - (double)in.trans[b];
        const double is = rcp64((double)in.scale);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            double ao = diff[0] * (double)in.rot[a];
            ao = __builtin_fma(diff[1], (double)in.rot[3 + a], ao);
            ao = __builtin_fma(diff[2], (double)in.rot[6 + a], ao);
            rs.O[a] = ao * is;
        }
    }
    bool hit = rs.len_local > 0.0f;
    // clip to the occupied-cell box [lo, hi) (no occupied cell lies outside it).
    // Direction components below 1e-20 of the largest are treated as zero: their
    // plane crossings lie beyond any representable ray parameter.
    double u_in = 0.0, u_out = 0.0;
    bool have_out = false;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const bool zero = fabsf((float)rs.D[a]) <= 1.0e-20f * dmax;
        const bool neg = !zero && rs.D[a] < 0.0;
        const double lo_p = (double)tr.box_lo[a], hi_p = (double)tr.box_hi[a];
        if (zero) {
            if (rs.O[a] < lo_p || !(rs.O[a] < hi_p)) hit = false;
            rs.flip[a] = 0;
            rs.D[a] = 0.0;
            rs.inv[a] = (double)INFINITY;
            continue;
        }
        const double inv = rcp64(rs.D[a]);
        const double t0 = (lo_p - rs.O[a]) * inv, t1 = (hi_p - rs.O[a]) * inv;
        const double lo = neg ? t1 : t0, hi = neg ? t0 : t1;
        if (u_in < lo) u_in = lo;
        if (!have_out || hi < u_out) { u_out = hi; have_out = true; }
        rs.flip[a] = neg ? -1 : 0;
        rs.O[a] = neg ? -rs.O[a] : rs.O[a];
        rs.D[a] = neg ? -rs.D[a] : rs.D[a];
        rs.inv[a] = neg ? -inv : inv;
    }
    if (!have_out || !(u_in < u_out)) hit = false;
    rs.u_in = u_in;
    rs.u_out = u_out;
    rs.hit = hit;
}

// Geometry and time of a ray.
template <bool IDENT>
__device__ __forceinline__ void ray_setup(const TreeArgs& tr, const InstArgs& in, const float o[3],
                                          const float d[3], float t, RaySetup& rs) {
    ray_geometry<IDENT>(tr, in, o, d, rs);
    time_setup(tr, in, t, rs.i0, rs.i1, rs.f, &rs.tau);
}

// ----------------------------------------------------------------------------
// octree walk

struct Walk {
    int m[3];        // leaf-level cell containing the ray just after the entry point, mirrored: cell ^ flip
    double u;        // ray parameter of the entry point
    bool done;
    int brick;       // directory entry of the brick whose node is held below, -1: none
    uint32_t bm_lo, bm_hi;
    int bbase;
};

// Node levels of a depth-D tree: L = ceil(D/2); level w is a cube of edge
// 2^node_edge(D, w) split into child cells of edge 2^(node_edge - node_bits).
__device__ __forceinline__ int node_bits(int D, int w) { return (w == 0 && (D & 1)) ? 1 : 2; }
__device__ __forceinline__ int node_edge(int D, int w) { return w == 0 ? D : D - (D & 1 ? 1 : 2) - 2 * (w - 1); }
// The brick directory: one int32 per 4^3 region of leaf cells, E^3 entries
// with E = 2^(D-2) (E = 1 for D <= 2, where the root is the only node),
// entry (k E + j) E + i for the region with corner (4i, 4j, 4k): the row of
// the region's last-level node when the region holds a leaf, else -(1 + s)
// where 2^s is the edge of the largest aligned cube around the region that
// holds no leaf, the cube at which a descent from the root would stop.
__host__ __device__ __forceinline__ int64_t directory_edge(int D) { return D <= 2 ? 1 : (int64_t)1 << (D - 2); }
__host__ __device__ __forceinline__ int64_t directory_entries(int D) {
    const int64_t e = directory_edge(D);
    return e * e * e;
}

__device__ __forceinline__ void walk_begin(const TreeArgs& tr, const RaySetup& rs, Walk& w) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        // the half-open cell just after the entry point: floor along the mirrored axis
        const int c = (int)__builtin_floor(__builtin_fma(rs.u_in, rs.D[a], rs.O[a])) ^ rs.flip[a];
        w.m[a] = (c < tr.box_lo[a] ? tr.box_lo[a] : (c > tr.box_hi[a] - 1 ? tr.box_hi[a] - 1 : c)) ^ rs.flip[a];
    }
    w.u = rs.u_in;
    w.done = !rs.hit;
    w.brick = -1;
    w.bm_lo = w.bm_hi = 0u;
    w.bbase = 0;
}

// Advances to the next occupied leaf segment of positive length. Returns its
// slot and writes delta (leaf units), umid (ray parameter of the segment
// midpoint) and the segment's bounds [seg_a, seg_b) in the ray parameter; returns -1 when the ray has left the box. With kBudget > 0 at
// most kBudget cells are visited per call, and -2 says that the budget ran out
// before a segment was found (the next call resumes the walk): lanes of a
// wavefront in long empty stretches then stop holding back the lanes that
// have a sample to evaluate.
//
// A cell visit reads nothing while the walk stays in the brick whose node it
// holds. Entering another 4^3 region, it reads the region's directory entry
// and, when the region holds a leaf, the brick's node row: at most two
// dependent loads, where a descent from the deepest common ancestor took up
// to one per node level (and a wavefront as many loop iterations as its
// deepest lane).
//
// Every decision of the walk (which face a node is left through, which cell
// the ray enters, whether it leaves the box) is taken in float64 directly, the
// same instructions for every lane. (Float estimates with error bounds, redone
// in compensated pairs where a bound was met, cost a visit about four times
// the instructions, and some lane of a wavefront met a bound in 27 % of its
// iterations.) The walk runs in coordinates mirrored on the axes the ray moves
// down, so that it only ever moves up: a step needs no selects by direction,
// and a cell is turned back (one xor per axis) only to look it up. It ends by
// construction: every visit moves up by a cell at least, and none back.
// It never leaves the grid either: the box's far planes give u_out by the
// same expression, which grows with the plane, so a step past them has ue >= u_out.
template <int kBudget = 0>
__device__ __forceinline__ int walk_next(const TreeArgs& tr, const RaySetup& rs, Walk& w, float& delta,
                                         float& umid, double& seg_a, double& seg_b) {
    const int eb = tr.depth <= 2 ? 0 : tr.depth - 2;   // log2 of the directory's edge
    int budget = kBudget;
    while (!w.done) {
        if (kBudget > 0 && budget-- == 0) return -2;
        // the cell's brick, or the empty cube around its region; sh = log2 of the
        // edge of the empty cube or cell reached (0 for a leaf)
        int leaf = -1;
        int sh = 0;
        {
            const int x = w.m[0] ^ rs.flip[0], y = w.m[1] ^ rs.flip[1], z = w.m[2] ^ rs.flip[2];
            const int bid = ((((z >> 2) << eb) + (y >> 2)) << eb) + (x >> 2);
            bool held = bid == w.brick;
            if (!held) {
                const int e = tr.dir[bid];
                if (e >= 0) {
                    const int4 v = tr.nodes[e];
                    w.brick = bid;
                    w.bm_lo = (uint32_t)v.x;
                    w.bm_hi = (uint32_t)v.y;
                    w.bbase = v.z;
                    held = true;
                } else {
                    sh = -e - 1;
                }
            }
            if (held) {
                // child q of the brick node: bit 0 of x, y, z, then bit 1 of x, y, z; the last picks the mask's half
                const uint32_t q = (x & 1) | ((y & 1) << 1) | ((z & 1) << 2) | ((x & 2) << 2) | ((y & 2) << 3);
                const bool top = (z & 2) != 0;
                const uint32_t half = top ? w.bm_hi : w.bm_lo;
                if ((half >> q) & 1u)
                    leaf = w.bbase + (top ? __popc(w.bm_lo) : 0) + __popc(half & ((1u << q) - 1u));
                else   // an empty cell; its 2^3 group (one byte of the mask) may be empty as a whole
                    sh = ((half >> (q & 24u)) & 0xffu) == 0u ? 1 : 0;
            }
        }
        const int S = 1 << sh;
        // Exit face of the cell (or empty node) of edge S: the smallest crossing of
        // its far planes, the first axis on a tie. An axis the ray does not move
        // along has inv = +inf and its far plane above O, so it is never left.
        int plane[3];
        double t[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            plane[a] = (w.m[a] & -S) + S;
            t[a] = ((double)plane[a] - rs.O[a]) * rs.inv[a];
        }
        const bool y_first = t[1] < t[0];
        const double t01 = y_first ? t[1] : t[0];
        const bool z_first = t[2] < t01;
        const double ue = z_first ? t[2] : t01;
        w.done = !(ue < rs.u_out);   // leaving the box
        bool produced = false;
        if (leaf >= 0) {
            const double ux = w.done ? rs.u_out : ue;
            if (w.u < ux) {
                delta = (float)(ux - w.u) * rs.len_local;
                umid = 0.5f * ((float)w.u + (float)ux);
                seg_a = w.u;
                seg_b = ux;
                produced = delta > 0.0f;
            }
        }
        // The next cell: across the exit plane on the exit axis; on the other
        // axes the cell of the position at the exit, within the node.
        const bool ex[3] = {!z_first && !y_first, !z_first && y_first, z_first};
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            int c = (int)__builtin_floor(__builtin_fma(ue, rs.D[b], rs.O[b]));
            c = c < plane[b] - 1 ? c : plane[b] - 1;
            c = c > w.m[b] ? c : w.m[b];
            w.m[b] = ex[b] ? plane[b] : c;
        }
        w.u = ue;
        if (produced) return leaf;
    }
    return -1;
}

// The same without the segment's bounds [seg_a, seg_b).
template <int kBudget = 0>
__device__ __forceinline__ int walk_next(const TreeArgs& tr, const RaySetup& rs, Walk& w, float& delta,
                                         float& umid) {
    double a, b;
    return walk_next<kBudget>(tr, rs, w, delta, umid, a, b);
}

}  // namespace neuvv
