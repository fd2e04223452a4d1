// Ray-marching emission (App. B), its pose Jacobian with the fused normal-
// equation reduction, anchor normals, and the adjoint w.r.t. map means.
//
// Work split of render and render_jacobian: four lanes per ray (a quad), an
// 8x2 pixel strip per wave, an 8x8 tile per workgroup, blockIdx.y = frame.
// A single frame is only ~10^5 rays, so the march is latency-bound: the four
// lanes of a ray evaluate interleaved samples (lane s takes k0 + s + 4 j, a few
// per trip) and two DPP quad permutations find the first crossing of the trip, which shortens each ray's chain of dependent gathers four-fold and
// gives the GPU four times more waves to overlap.  Samples in bricks whose
// occupancy is <= 0 everywhere are decided without touching the map
// (free-space bits in LDS; every cell reads the dilated bit of its base
// corner's 2x2x2 block of bricks).  At the hit the quad splits the
// double-precision shading and the Jacobian by channel: lane 0 occupancy /
// depth, lanes 1-3 one colour each.
//
// The adjoint takes four lanes per ray as well (8x8 pixels per workgroup):
// from the given hit index it recomputes the two samples, nothing to march,
// and lane s scatters the gradient of plane s.
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"

namespace prism {

constexpr int kLanes = 4;       // lanes per ray in render / render_jacobian
// Samples per lane per trip of the march.  With free-space bits it starts just
// before the first occupied brick and ends within a trip or two, and short
// trips evaluate fewer samples past the crossing (8-frame render at 256^3,
// 320x240: 59.5 us with 2, 61.9 with 3, 64.2 with 4); without bits every
// sample reads the map and long trips keep more loads in flight.
constexpr int kPerLaneBits = 2, kPerLaneNoBits = 4;

template <typename T, bool Pool>
__device__ __forceinline__ float occ_at(const GridC& g, const T* occ, const Cell& c) {
    float v[8];
    corners<T, Pool>(g, occ, c, g.occ_out, g.pocc, v);
    return trilerp(v, c.w);
}

// Occupancy of a cell that straddles the grid's boundary (on every axis one
// of its two corner planes is inside; dense maps): corners outside take the
// outside value.  A brick-order element index is a sum of one term per
// axis, ((x >> 3) * brick stride + (x & 7) * voxel stride), so the two
// candidates per axis are formed once, from coordinates clamped into the
// grid (a clamped corner is loaded and then replaced), and each corner is
// three adds away: a few dozen instructions instead of eight corners each
// tested and indexed on its own.
template <typename T>
__device__ __forceinline__ float occ_partial(const GridC& g, const T* occ, const Cell& c) {
    const unsigned bs[3] = {512u, 512u * (unsigned)g.nb, 512u * (unsigned)(g.nb * g.nb)};
    const unsigned vs[3] = {1u, 8u, 64u};
    unsigned off[3][2];
    bool ok[3][2];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const int x = c.i[a] + d;    // in [-1, n] for a straddling cell
            ok[a][d] = (unsigned)x < (unsigned)g.n;
            const unsigned xc = (unsigned)min(max(x, 0), g.n - 1);
            off[a][d] = (__umul24(xc >> 3, bs[a]) + (xc & 7u) * vs[a]) * (unsigned)sizeof(T);
        }
    float v[8];
    const gptr<T> pl = as_global(occ);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int dx = q & 1, dy = (q >> 1) & 1, dz = q >> 2;
        const float x = ldg(pl, off[0][dx] + off[1][dy] + off[2][dz]);
        v[q] = (ok[0][dx] && ok[1][dy] && ok[2][dz]) ? x : g.occ_out;
    }
    return trilerp(v, c.w);
}

// Free-space bits.  A sample's occupancy is proven <= 0 when every corner of
// its cell lies inside the grid and in bricks whose largest occupancy mean is
// <= 0: each lerp of values <= 0 with a weight in [0, 1] is <= 0 under
// round-to-nearest (rounding is monotonic and 0 is representable), so the
// single-precision recipe would have produced a value <= 0 as well and the
// sample cannot be the hit when tau == 0.  Most marched samples are decided
// by the bits alone, so that path takes only the cell's base corner and its
// brick: every cell inside the grid reads the one dilated bit of the 2x2x2
// bricks from its base brick, whether or not the cell spans bricks (a spanned
// brick is in that block; a cell within one brick loses little from the
// coarser test), so the plain bits are not needed here.  The corner addressing
// and the weights are formed only for samples that read the map.
__device__ __forceinline__ bool bit_of(lds_u32* bits, int b) { return (bits[b >> 5] >> (b & 31)) & 1u; }

// grid coordinate of a marched sample and its cell's base corner
struct SamplePos {
    float gc[3];
    int i[3];
};

__device__ __forceinline__ SamplePos sample_pos(const RayCoef& rc, float fk) {
    SamplePos p;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        p.gc[a] = sample_gc(rc, fk, a);
        p.i[a] = floor_i32(p.gc[a]);
    }
    return p;
}

// occupancy of a marched sample that the bits do not decide
template <typename T, bool Pool>
__device__ __forceinline__ float march_sample(const GridC& g, const T* occ, const SamplePos& p) {
    const float* gc = p.gc;
    const int* i = p.i;
    const unsigned lim = (unsigned)(g.n - 1);
    if (max(max((unsigned)i[0], (unsigned)i[1]), (unsigned)i[2]) < lim) {
        // all 8 corners inside: indices >= 0 and < 2^10, so 24-bit products
        const unsigned bx = (unsigned)i[0] >> 3, by = (unsigned)i[1] >> 3, bz = (unsigned)i[2] >> 3;
        const int b0 = (int)(__umul24(bz, (unsigned)(g.nb * g.nb)) + __umul24(by, (unsigned)g.nb) + bx);
        const int lx = i[0] & 7, ly = i[1] & 7, lz = i[2] & 7;
        CellAddr a;
        a.b0 = b0;
        a.base = (b0 << 9) | (lz << 6) | (ly << 3) | lx;
        a.dx = lx == 7 ? 512 - 7 : 1;
        a.dy = ly == 7 ? 512 * g.nb - 56 : 8;
        a.dz = lz == 7 ? 512 * g.nb * g.nb - 448 : 64;
        a.cross = (lx == 7) | (ly == 7) | (lz == 7);
        // inside the grid g >= 0, where g - floor(g) is exact and fract(g) equals it
        float w[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) w[q] = __builtin_amdgcn_fractf(gc[q]);
        float v[8];
        if constexpr (Pool)
            corners_pool(g, as_global(occ), a, g.pocc, v);
        else
            corners_in_g(as_global(occ), a, v);
        return trilerp(v, w);
    }
    // Every corner outside the grid (on some axis both i and i + 1 are): the
    // blend of 8 equal outside values is that value, lerp(a, a, w) = a.
    if (max(max((unsigned)i[0] + 1u, (unsigned)i[1] + 1u), (unsigned)i[2] + 1u) > (unsigned)g.n) return g.occ_out;
    Cell cl;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        cl.i[q] = i[q];
        cl.w[q] = gc[q] - (float)i[q];
    }
    if constexpr (!Pool) return occ_partial(g, occ, cl);
    return occ_at<T, Pool>(g, occ, cl);
}

// double-precision sample point k of the ray with direction dir (world)
__device__ __forceinline__ void grid_coord64(const GridD& gd, const CamD& cd, const Pose64& P, const double dir[3],
                                             int k, double gc[3]) {
    double dk = cd.dn + (double)k * cd.step;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double p = P.t[a] + dk * dir[a];
        gc[a] = (p - gd.o[a]) * gd.inv_s - 0.5;
    }
}

__device__ __forceinline__ void cross3(const float a[3], const float b[3], float o[3]) {
    o[0] = a[1] * b[2] - a[2] * b[1];
    o[1] = a[2] * b[0] - a[0] * b[2];
    o[2] = a[0] * b[1] - a[1] * b[0];
}

struct BlockPose {
    Pose64 d;
    Pose32 f;
};

// sixteen bytes of free-space bits in global memory (the dilated ones start
// at any word)
typedef unsigned uint4u __attribute__((ext_vector_type(4), aligned(4)));

// The prologue of a marching workgroup, one barrier: thread 0's pose loads
// are issued first and are in flight while every thread copies the dilated
// free-space bits to LDS (free_lds_words words, which the launch allocates;
// none: no skipping, NULL).  gbits: the map's two bitmaps, the dilated one
// last.  (Copying both, as the march of cells within one brick could use,
// took a 384^3 map's workgroup 27 KB instead of 13.5, hence one workgroup
// less per CU.)
__device__ __forceinline__ lds_u32* block_setup(const GridC& g, const unsigned* __restrict__ gbits, unsigned* lbits,
                                                const prism_pose* pose, BlockPose* sp) {
    prism_pose raw;
    if (threadIdx.x == 0) raw = *pose;
    const int nwords = free_words(g.nb), nl = gbits ? free_lds_words(nwords) : 0;
    if (nl) {
        const unsigned* src = gbits + nwords;
        const int n4 = nl >> 2;
        for (int i = threadIdx.x; i < n4; i += blockDim.x) {
            const uint4u v = reinterpret_cast<const uint4u*>(src)[i];
            reinterpret_cast<uint4*>(lbits)[i] = make_uint4(v[0], v[1], v[2], v[3]);
        }
        for (int i = (n4 << 2) + threadIdx.x; i < nl; i += blockDim.x) lbits[i] = src[i];
    }
    if (threadIdx.x == 0) {
        quat_to_rot64(raw, sp->d.R);
        for (int i = 0; i < 3; ++i) sp->d.t[i] = raw.t[i];
        sp->f = to32(sp->d);
    }
    __syncthreads();
    return nl ? (lds_u32*)lbits : nullptr;
}

__device__ __forceinline__ const BlockPose& block_pose(const prism_pose* pose, BlockPose* sp) {
    if (threadIdx.x == 0) {
        sp->d = load_pose64(pose);
        sp->f = to32(sp->d);
    }
    __syncthreads();
    return *sp;
}

// ---------------------------------------------------------------------------
// quad (four lanes per ray) march and shading
// ---------------------------------------------------------------------------
// minimum over the four lanes of a quad (DPP quad permutations: lanes 1,0,3,2
// then 2,3,0,1; a lane whose partner is inactive keeps its own value)
__device__ __forceinline__ int quad_min(int x) {
    x = min(x, __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false));
    x = min(x, __builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false));
    return x;
}

// lane 0 of each quad to all four lanes (DPP quad_perm 0,0,0,0; whole quads
// are active together)
__device__ __forceinline__ float quad_bcast0f(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x00, 0xF, 0xF, false));
}

// sum over the quad (DPP quad permutations 1,0,3,2 then 2,3,0,1; every lane
// ends with (x0 + x1) + (x2 + x3) up to the order of each addition)
__device__ __forceinline__ double quad_xchg(double x, int ctrl_is_2301) {
    const long long b = __double_as_longlong(x);
    int lo, hi;
    if (ctrl_is_2301) {
        lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), 0x4E, 0xF, 0xF, false);
        hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x4E, 0xF, 0xF, false);
    } else {
        lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), 0xB1, 0xF, 0xF, false);
        hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0xB1, 0xF, 0xF, false);
    }
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double quad_sum(double x) {
    x += quad_xchg(x, 0);
    x += quad_xchg(x, 1);
    return x;
}

__device__ __forceinline__ double quad_bcast0(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), 0x00, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x00, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// first sample index from `start` on whose occupancy exceeds tau (strictly),
// or -1; every lane of the quad returns the same value
template <typename T, bool Pool, bool Bits>
__device__ __forceinline__ int march_quad_b(const GridC& g, const CamC& c, const RayCoef& rc, const T* occ,
                                            lds_u32* fb, int s, int start) {
    constexpr int kPerLane = Bits ? kPerLaneBits : kPerLaneNoBits, G = kLanes * kPerLane;
    // the sample index as a float, advanced exactly (K < 2^24); the last trip's
    // samples past K - 1 are evaluated like any other and ignored
    float fk0 = (float)(start + s);
    // The sample recipe is monotone in k on every axis, so once a sample's
    // cell lies past the grid on an axis the ray moves away from it along,
    // so do all later cells: their occupancy is the outside value.  When that
    // value cannot cross tau the ray has no first crossing left.  The test
    // per axis: cell index < lo (ray not moving up) or >= hi (not moving down).
    const bool stop_outside = !(g.occ_out > c.tau);
    int lo[3], hi[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = rc.B[a] <= 0.0f ? -1 : INT_MIN;
        hi[a] = rc.B[a] >= 0.0f ? g.n : INT_MAX;
    }
    for (int k0 = start; k0 < c.K; k0 += G, fk0 += (float)G) {
        float f[kPerLane];
        bool gone = false;
        if constexpr (Bits) {
            // the round's free-space tests first, as straight-line code, so its
            // LDS reads are in flight together (a sample outside the grid reads
            // word 0 and ignores it); then the samples the bits do not decide,
            // whose position is formed again (a few instructions, fewer live
            // registers than keeping it)
            const unsigned lim = (unsigned)(g.n - 1);
            unsigned word[kPerLane];
            int b0[kPerLane];
            bool in[kPerLane];
#pragma unroll
            for (int j = 0; j < kPerLane; ++j) {
                const SamplePos p = sample_pos(rc, fk0 + (float)(j * kLanes));
                const int* i = p.i;
                in[j] = max(max((unsigned)i[0], (unsigned)i[1]), (unsigned)i[2]) < lim;
                const int b = (int)(__umul24((unsigned)i[2] >> 3, (unsigned)(g.nb * g.nb)) +
                                    __umul24((unsigned)i[1] >> 3, (unsigned)g.nb) + ((unsigned)i[0] >> 3));
                b0[j] = in[j] ? b : 0;
                word[j] = fb[b0[j] >> 5];
                if (j == kPerLane - 1) {
#pragma unroll
                    for (int a = 0; a < 3; ++a) gone |= (i[a] < lo[a]) | (i[a] >= hi[a]);
                }
            }
#pragma unroll
            for (int j = 0; j < kPerLane; ++j) {
                const bool fr = in[j] && __builtin_amdgcn_ubfe(word[j], (unsigned)b0[j], 1u);
                f[j] = fr ? -1.0f
                          : march_sample<T, Pool>(g, occ, sample_pos(rc, fk0 + (float)(j * kLanes)));
            }
        } else {
#pragma unroll
            for (int j = 0; j < kPerLane; ++j) {
                const SamplePos p = sample_pos(rc, fk0 + (float)(j * kLanes));
                f[j] = march_sample<T, Pool>(g, occ, p);
                if (j == kPerLane - 1) {
#pragma unroll
                    for (int a = 0; a < 3; ++a) gone |= (p.i[a] < lo[a]) | (p.i[a] >= hi[a]);
                }
            }
        }
        int first = 0x7fffffff;
#pragma unroll
        for (int j = kPerLane - 1; j >= 0; --j) {
            int k = k0 + j * kLanes + s;
            if (k < c.K && f[j] > c.tau) first = k;
        }
        first = quad_min(first);
        if (first != 0x7fffffff) return first;
        // lane 3 holds the trip's last sample (DPP quad_perm 3,3,3,3)
        if (stop_outside && __builtin_amdgcn_update_dpp(0, (int)gone, 0xFF, 0xF, 0xF, false)) return -1;
    }
    return -1;
}

// the march with or without the workgroup's free-space bits (one uniform
// branch per ray instead of one per sample)
template <typename T, bool Pool>
__device__ __forceinline__ int march_quad(const GridC& g, const CamC& c, const RayCoef& rc, const T* occ, lds_u32* fb,
                                          int s, int start) {
    if (fb) return march_quad_b<T, Pool, true>(g, c, rc, occ, fb, s, start);
    return march_quad_b<T, Pool, false>(g, c, rc, occ, fb, s, start);
}

// This lane's share of the shading at a valid hit: plane s (0 occupancy,
// 1..3 colour) at samples k*-1 and k*, in double precision, plus the
// double-precision interpolation weights.
struct QuadShade {
    double v0, v1;          // plane s at samples k*-1, k*
    double f0, f1;          // occupancy at k*-1, k* (from lane 0)
    double alpha, value;    // alpha and this lane's output (depth or colour)
    float w0[3], w1[3];
    float d0, d1;
    float cv0[8], cv1[8];   // plane s at the corners of the two cells (as corners() gives them)
};

// Trilinear value of one plane in double precision at a marched sample:
// cell from the decision recipe, weights from the double-precision grid
// coordinate, blended along x, then y, then z (seven linear blends, each one
// fused multiply-add; the same trilinear interpolant as the sum of the
// corners weighted by products of 1-D hat weights, to rounding).  The
// corners are the ones corners() gathered; a corner outside the grid takes
// the double-precision outside value.
__device__ __forceinline__ double lerp64(double a, double b, double w) { return __builtin_fma(w, b - a, a); }

__device__ __forceinline__ double tri64c(const GridC& g, const float v[8], const double gc[3], const int cell[3],
                                         double outv) {
    const double w0 = gc[0] - (double)cell[0], w1 = gc[1] - (double)cell[1], w2 = gc[2] - (double)cell[2];
    // a cell inside the grid (the usual case) needs no test per corner
    const unsigned lim = (unsigned)(g.n - 1);
    const bool inside = (unsigned)cell[0] < lim && (unsigned)cell[1] < lim && (unsigned)cell[2] < lim;
    double V[8];
    if (inside) {
#pragma unroll
        for (int q = 0; q < 8; ++q) V[q] = (double)v[q];
    } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            int i = cell[0] + (q & 1), j = cell[1] + ((q >> 1) & 1), k = cell[2] + (q >> 2);
            bool in = (unsigned)i < (unsigned)g.n && (unsigned)j < (unsigned)g.n && (unsigned)k < (unsigned)g.n;
            V[q] = in ? (double)v[q] : outv;
        }
    }
    const double l00 = lerp64(V[0], V[1], w0), l10 = lerp64(V[2], V[3], w0);
    const double l01 = lerp64(V[4], V[5], w0), l11 = lerp64(V[6], V[7], w0);
    return lerp64(lerp64(l00, l10, w1), lerp64(l01, l11, w1), w2);
}

template <typename T, bool Pool>
__device__ __forceinline__ QuadShade shade_quad(const GridC& g, const GridD& gd, const CamD& cd, const Pose64& P,
                                                int u, int v, const T* map, const Cell& c0, const Cell& c1, int k,
                                                int s) {
    // values only from here (the hit index and cells are decided): the
    // double-precision arithmetic may fuse multiplies and adds
#pragma clang fp contract(fast)
    QuadShade q;
    double rc[3], dir[3], gc0[3], gc1[3];
    pixel_dir64(cd, u, v, rc);
#pragma unroll
    for (int a = 0; a < 3; ++a) dir[a] = P.R[a][0] * rc[0] + P.R[a][1] * rc[1] + P.R[a][2] * rc[2];
    grid_coord64(gd, cd, P, dir, k - 1, gc0);
    grid_coord64(gd, cd, P, dir, k, gc1);
    double d0 = cd.dn + (double)(k - 1) * cd.step;
    double d1 = cd.dn + (double)k * cd.step;
    const T* pl = map + (long long)s * g.nvox;
    double outv = s == 0 ? gd.occ_out : gd.rgb_out;
    float outv32 = s == 0 ? g.occ_out : g.rgb_out, priorv = s == 0 ? g.pocc : g.prgb;
    // the lane's plane at both cells, gathered once (the Jacobian row reuses them)
    corners<T, Pool>(g, pl, c0, outv32, priorv, q.cv0);
    corners<T, Pool>(g, pl, c1, outv32, priorv, q.cv1);
    q.v0 = tri64c(g, q.cv0, gc0, c0.i, outv);
    q.v1 = tri64c(g, q.cv1, gc1, c1.i, outv);
    q.f0 = quad_bcast0(q.v0);
    q.f1 = quad_bcast0(q.v1);
    q.alpha = (cd.tau - q.f0) / (q.f1 - q.f0);
    q.value = s == 0 ? q.alpha * d1 + (1.0 - q.alpha) * d0 : q.alpha * q.v1 + (1.0 - q.alpha) * q.v0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        q.w0[a] = (float)(gc0[a] - (double)c0.i[a]);
        q.w1[a] = (float)(gc1[a] - (double)c1.i[a]);
    }
    q.d0 = (float)d0;
    q.d1 = (float)d1;
    return q;
}

// This lane's row of the 4x6 Jacobian d(depth, r, g, b)/d(delta), k* fixed.
// Lane 0 forms d(alpha)/d(delta) from the occupancy gradients and shares it.
__device__ __forceinline__ void jac_row_quad(const GridC& g, const QuadShade& q, const float dir[3], int s,
                                             float row[6]) {
    float a0[3], a1[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) { a0[i] = q.d0 * dir[i]; a1[i] = q.d1 * dir[i]; }
    float G0[3], G1[3], cr[3], r0[6], r1[6];
    trigrad(q.cv0, q.w0, G0);
    trigrad(q.cv1, q.w1, G1);
#pragma unroll
    for (int i = 0; i < 3; ++i) { G0[i] *= g.inv_s; G1[i] *= g.inv_s; r0[i] = G0[i]; r1[i] = G1[i]; }
    cross3(a0, G0, cr);
#pragma unroll
    for (int i = 0; i < 3; ++i) r0[3 + i] = cr[i];
    cross3(a1, G1, cr);
#pragma unroll
    for (int i = 0; i < 3; ++i) r1[3 + i] = cr[i];
    // lane 0: d(alpha) = -[(1-alpha) df0 + alpha df1] / (f1 - f0)
    float al = (float)q.alpha;
    float inv_den = (float)(1.0 / (q.f1 - q.f0));
    float dal[6];
#pragma unroll
    for (int m = 0; m < 6; ++m) dal[m] = quad_bcast0f(-((1.0f - al) * r0[m] + al * r1[m]) * inv_den);
    if (s == 0) {
#pragma unroll
        for (int m = 0; m < 6; ++m) row[m] = (q.d1 - q.d0) * dal[m];
    } else {
        float dc = (float)(q.v1 - q.v0);
#pragma unroll
        for (int m = 0; m < 6; ++m) row[m] = dc * dal[m] + al * r1[m] + (1.0f - al) * r0[m];
    }
}

// tile of workgroup blk: 8x8 pixels from (u0, v0)
struct Tile {
    int u0, v0;
};

__device__ __forceinline__ Tile tile_of(const CamC& c, int blk) {
    // blk / tiles per row through the high half of a product with
    // floor(2^32 / tiles) + 1, exact for blk * tiles < 2^32 (blk <= 2^20, at
    // most 2^10 tiles per row; one tile per row: 0 stands for 2^32)
    const int by = c.tiles_inv ? (int)__umulhi((unsigned)blk, c.tiles_inv) : blk;
    return Tile{(blk - by * ((c.W + 7) >> 3)) << 3, by << 3};
}

// quad tile mapping: 8x8 pixels per 256-thread workgroup, 8x2 per wave
__device__ __forceinline__ void quad_pixel(const Tile& tl, int& u, int& v, int& s) {
    const int t = threadIdx.x, r = t >> 2;    // r: 0..63 ray of the tile
    s = t & 3;
    u = tl.u0 + (r & 7);
    v = tl.v0 + (r >> 3);
}

// A sample index below which no ray of the tile can cross tau, from the
// dilated bits (fb; tau == 0).  The 64 rays of a tile run close together, so
// the free space before them is the same: lane l tests the box that holds all
// rays' samples 2l and 2l + 1, and the march starts at the first sample whose
// box is not proven free.  A pixel direction is affine in (u, v), so per axis
// the box at depth e is the centre ray's coordinate +- e h with h the spread
// of a half tile; the margin covers the rounding of the single-precision
// recipe (2^-18 of the magnitudes it sums, 64 ulp) and of this bound.  A box
// is free when it lies inside the grid and the dilated bits of all its base
// bricks (at most two per axis) are set, or when it lies off the grid on some
// axis, where every sample takes the outside value.  About 90 instructions in
// one wavefront of four (K <= 128) against 140 in each for a round of the march.
__device__ __forceinline__ int tile_start(const GridC& g, const CamC& c, const Pose32& P, const Tile& tl,
                                          lds_u32* fb, int* starts) {
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (128 * wv < c.K) {
        const int k = 2 * (int)threadIdx.x;
        const float e0 = (c.dn + (float)k * c.dstep) * g.inv_s, e1 = e0 + c.dstep * g.inv_s;
        const float rx = ((float)tl.u0 + 4.0f - c.cx) * c.ifx, ry = ((float)tl.v0 + 4.0f - c.cy) * c.ify;
        int lo[3], hi[3];
        bool off = false;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float d = P.R[a][0] * rx + P.R[a][1] * ry + P.R[a][2];
            const float h = 3.5f * (fabsf(P.R[a][0] * c.ifx) + fabsf(P.R[a][1] * c.ify));
            const float t0 = (P.t[a] - g.o[a]) * g.inv_s - 0.5f;
            const float m = (fabsf(P.t[a]) + fabsf(g.o[a])) * g.inv_s + e1 * (fabsf(d) + h);
            const float eps = 0.0078125f + 3.814697265625e-6f * m;
            lo[a] = floor_i32(t0 - eps + fminf(e0 * (d - h), e1 * (d - h)));
            hi[a] = floor_i32(t0 + eps + fmaxf(e0 * (d + h), e1 * (d + h)));
            off |= hi[a] < -1 || lo[a] >= g.n;
        }
        const unsigned lim = (unsigned)(g.n - 1);
        const bool in = max(max((unsigned)lo[0], (unsigned)lo[1]), (unsigned)lo[2]) < lim &&
                        max(max((unsigned)hi[0], (unsigned)hi[1]), (unsigned)hi[2]) < lim;
        const int sx = (hi[0] >> 3) - (lo[0] >> 3), sy = (hi[1] >> 3) - (lo[1] >> 3), sz = (hi[2] >> 3) - (lo[2] >> 3);
        bool free = false;
        if (in && max(max(sx, sy), sz) <= 1) {
            const int b = ((lo[2] >> 3) * g.nb + (lo[1] >> 3)) * g.nb + (lo[0] >> 3);
            const int oy = sy ? g.nb : 0, oz = sz ? g.nb * g.nb : 0;
            free = true;
#pragma unroll
            for (int q = 0; q < 8; ++q)
                free &= bit_of(fb, b + ((q & 1) ? sx : 0) + ((q & 2) ? oy : 0) + ((q & 4) ? oz : 0));
        }
        free |= off && !(g.occ_out > c.tau);
        const unsigned long long stop = __ballot(!free);
        if ((threadIdx.x & 63) == 0) starts[wv] = stop ? 128 * wv + 2 * __builtin_ctzll(stop) : INT_MAX;
    } else if ((threadIdx.x & 63) == 0) {
        starts[wv] = 128 * wv;
    }
    __syncthreads();
    // (all 512 samples free: the rest is marched)
    return min(min(min(starts[0], starts[1]), min(starts[2], starts[3])), 512);
}

// ---------------------------------------------------------------------------
// render
// ---------------------------------------------------------------------------
// workgroup blk (8x8 pixel tile) of frame `frame`, rendered at *pose
template <typename T, bool Pool>
__device__ __forceinline__ void render_block(int blk, int frame, const GridC& g, const CamC& c, const GridD& gd,
                                             const CamD& cd, const T* __restrict__ map,
                                             const unsigned* __restrict__ gbits, const prism_pose* __restrict__ pose,
                                             float* __restrict__ depth, float* __restrict__ rgb,
                                             uint8_t* __restrict__ mask, int32_t* __restrict__ hit_k) {
    __shared__ BlockPose sp;
    extern __shared__ __align__(16) unsigned lbits[];
    lds_u32* const fb = block_setup(g, gbits, lbits, pose, &sp);
    const BlockPose& P = sp;
    __shared__ int starts[4];
    const Tile tl = tile_of(c, blk);
    const int start = fb ? tile_start(g, c, P.f, tl, fb, starts) : 0;
    int u, v, s;
    quad_pixel(tl, u, v, s);
    if (u >= c.W || v >= c.H) return;   // whole quads leave together
    float dir[3];
    ray_dir32(c, P.f, u, v, dir);
    const RayCoef rc = ray_coef(g, c, P.f, dir);
    int k = march_quad<T, Pool>(g, c, rc, map, fb, s, start);
    long long pix = (long long)frame * c.W * c.H + (long long)v * c.W + u;
    if (s == 0) {
        if (hit_k) hit_k[pix] = k;
        mask[pix] = k >= 1 ? 1 : 0;
    }
    if (k >= 1) {
        Cell c0 = sample_cell(rc, k - 1), c1 = sample_cell(rc, k);
        QuadShade q = shade_quad<T, Pool>(g, gd, cd, P.d, u, v, map, c0, c1, k, s);
        if (s == 0)
            depth[pix] = (float)q.value;
        else
            rgb[3 * pix + s - 1] = (float)q.value;
    } else {
        if (s == 0)
            depth[pix] = 0.0f;
        else
            rgb[3 * pix + s - 1] = 0.0f;
    }
}

template <typename T, bool Pool>
// at least 6 waves per SIMD (80 VGPRs, no spills): the march hides gather
// latency with waves; 7 or 8 would spill the double-precision shading
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void k_render(GridC g, CamC c, GridD gd, CamD cd, const T* __restrict__ map,
                                                const unsigned* __restrict__ gbits,
                                                const prism_pose* __restrict__ poses,
                                                float* __restrict__ depth, float* __restrict__ rgb,
                                                uint8_t* __restrict__ mask, int32_t* __restrict__ hit_k) {
    render_block<T, Pool>(blockIdx.x, blockIdx.y, g, c, gd, cd, map, gbits, poses + blockIdx.y, depth, rgb, mask, hit_k);
}

// batched: every filter renders its next anchor from its updated map at its
// posterior mean
template <typename T, bool Pool>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void k_render_batch(BatchArgs b) {
    const int a = batch_agent(b, blockIdx.x);
    const AgentDesc& D = *b.d[a];
    render_block<T, Pool>(blockIdx.x - b.start[a], 0, D.g, D.c, D.gd, D.cd, (const T*)D.map, D.bits, &D.S->pose, D.a_depth,
                    D.a_rgb, D.a_mask, nullptr);
}

// ---------------------------------------------------------------------------
// normals of a rendered depth image
// ---------------------------------------------------------------------------
__device__ __forceinline__ void normals_block(int blk, const CamC& c, int n_frames, const float* __restrict__ depth,
                                              const uint8_t* __restrict__ mask, float disc,
                                              float* __restrict__ normals, uint8_t* __restrict__ nmask,
                                              const int* __restrict__ counts, int ngroups,
                                              int64_t* __restrict__ n_updated,
                                              int64_t* __restrict__ n_updated_total) {
    // in a filter step, the first workgroup also totals the preceding map
    // update (before any thread returns: the sum synchronises the workgroup)
    __shared__ long long part[4];
    if (n_updated && blk == 0) sum_counts_block(counts, ngroups, n_updated, part, n_updated_total);
    long long npix = (long long)c.W * c.H;
    long long gid = (long long)blk * blockDim.x + threadIdx.x;
    if (gid >= npix * n_frames) return;
    long long f = gid / npix;
    int p = (int)(gid - f * npix);
    int u = p % c.W, v = p / c.W;
    const float* D = depth + f * npix;
    const uint8_t* M = mask + f * npix;
    // the five masks and depths in one round of loads (a border pixel reads
    // itself in place of its missing neighbours; it is never valid), then
    // one store of the result
    const bool inner = u > 0 && v > 0 && u < c.W - 1 && v < c.H - 1;
    const int pl = inner ? p - 1 : p, pr = inner ? p + 1 : p;
    const int pu = inner ? p - c.W : p, pd = inner ? p + c.W : p;
    const bool m = (M[p] & M[pl] & M[pr] & M[pu] & M[pd]) != 0;   // masks are 0 / 1
    const float d = D[p], dl = D[pl], dr = D[pr], du = D[pu], dd = D[pd];
    float o[3] = {0.0f, 0.0f, 0.0f};
    uint8_t ok = 0;
    if (inner && m &&
        !(fabsf(dl - d) > disc || fabsf(dr - d) > disc || fabsf(du - d) > disc || fabsf(dd - d) > disc)) {
        float xl = ((float)(u - 1) + 0.5f - c.cx) * c.ifx, xr = ((float)(u + 1) + 0.5f - c.cx) * c.ifx;
        float x0 = ((float)u + 0.5f - c.cx) * c.ifx;
        float yu = ((float)(v - 1) + 0.5f - c.cy) * c.ify, yd = ((float)(v + 1) + 0.5f - c.cy) * c.ify;
        float y0 = ((float)v + 0.5f - c.cy) * c.ify;
        float a[3] = {dr * xr - dl * xl, dr * y0 - dl * y0, dr - dl};
        float b[3] = {dd * x0 - du * x0, dd * yd - du * yu, dd - du};
        float n[3];
        cross3(a, b, n);
        float len = sqrtf(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
        if (len > 0.0f) {
            float sgn = (n[0] * x0 + n[1] * y0 + n[2]) * d < 0.0f ? 1.0f : -1.0f;
            float il = sgn / len;
            o[0] = n[0] * il;
            o[1] = n[1] * il;
            o[2] = n[2] * il;
            ok = 1;
        }
    }
    float* N = normals + 3 * gid;
    N[0] = o[0];
    N[1] = o[1];
    N[2] = o[2];
    nmask[gid] = ok;
}

__global__ __launch_bounds__(256) void k_normals(CamC c, int n_frames, const float* __restrict__ depth,
                                                 const uint8_t* __restrict__ mask, float disc,
                                                 float* __restrict__ normals, uint8_t* __restrict__ nmask,
                                                 const int* __restrict__ counts, int ngroups,
                                                 int64_t* __restrict__ n_updated,
                                                 int64_t* __restrict__ n_updated_total) {
    normals_block(blockIdx.x, c, n_frames, depth, mask, disc, normals, nmask, counts, ngroups, n_updated,
                  n_updated_total);
}

__global__ __launch_bounds__(256) void k_normals_batch(BatchArgs b) {
    const int a = batch_agent(b, blockIdx.x);
    const AgentDesc& D = *b.d[a];
    normals_block(blockIdx.x - b.start[a], D.c, 1, D.a_depth, D.a_mask, D.normal_disc, D.a_normals, D.a_nmask,
                  D.aux.counts, D.upd_groups, &D.S->n_updated, &D.S->n_updated_total);
}

// ---------------------------------------------------------------------------
// render + P1 Jacobian + gated weighted normal equations
// ---------------------------------------------------------------------------
// workgroup blk (8x8 pixel tile) of frame `frame` at *pose; the
// workgroup's 29 sums go to partial_row
template <typename T, bool Pool>
__device__ __forceinline__ void render_jac_block(int blk, int frame, const GridC& g, const CamC& c, const GridD& gd,
                                                 const CamD& cd, const T* __restrict__ map,
                                                 const unsigned* __restrict__ gbits, const prism_pose* __restrict__ pose,
                                                 const float* __restrict__ obs_depth,
                                                 const float* __restrict__ obs_rgb, const WeightsC& wt,
                                                 float* __restrict__ depth, float* __restrict__ rgb,
                                                 uint8_t* __restrict__ mask, float* __restrict__ Jout,
                                                 float* __restrict__ resid, uint8_t* __restrict__ rowmask,
                                                 double* __restrict__ partial_row) {
    __shared__ BlockPose sp;
    __shared__ double lds[kRedLds];
    extern __shared__ __align__(16) unsigned lbits[];
    lds_u32* const fb = block_setup(g, gbits, lbits, pose, &sp);
    const BlockPose& P = sp;
    __shared__ int starts[4];
    const Tile tl = tile_of(c, blk);
    const int start = fb ? tile_start(g, c, P.f, tl, fb, starts) : 0;
    int u, v, s;
    quad_pixel(tl, u, v, s);
    // this lane's row in single precision, reduced over the workgroup by
    // block_reduce29f (single precision within 32 lanes, then double)
    float pacc[PRISM_NEQ];
#pragma unroll
    for (int q = 0; q < PRISM_NEQ; ++q) pacc[q] = 0.0f;
    if (u < c.W && v < c.H) {
        float dir[3];
        ray_dir32(c, P.f, u, v, dir);
        const RayCoef rc = ray_coef(g, c, P.f, dir);
        int k = march_quad<T, Pool>(g, c, rc, map, fb, s, start);
        long long pix = (long long)frame * c.W * c.H + (long long)v * c.W + u;
        float row[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        double r = 0.0;
        int rm = 0;
        bool valid = k >= 1;
        double value = 0.0;
        if (valid) {
            Cell c0 = sample_cell(rc, k - 1), c1 = sample_cell(rc, k);
            QuadShade q = shade_quad<T, Pool>(g, gd, cd, P.d, u, v, map, c0, c1, k, s);
            value = q.value;
            float D = obs_depth[pix];
            if (depth_ok(D)) {
                jac_row_quad(g, q, dir, s, row);
                r = s == 0 ? value - (double)D : value - (double)obs_rgb[3 * pix + s - 1];
                // colour gate on |r_r| + |r_g| + |r_b| (lanes 1-3), depth gate on lane 0
                double l1 = s == 0 ? 0.0 : fabs(r);
                l1 = quad_sum(l1);
                bool use_depth = fabs(quad_bcast0(r)) <= wt.gate_depth;
                bool use_rgb = l1 <= wt.gate_rgb;
                rm = (use_depth ? 1 : 0) | (use_rgb ? 2 : 0);
                if (s == 0 ? use_depth : use_rgb)
                    neq_add32(pacc, row, (float)r, row_weight(wt, s != 0, r));
                if (rm && s == 0) pacc[28] = 1.0f;
            }
            if (!rm) {
#pragma unroll
                for (int m = 0; m < 6; ++m) row[m] = 0.0f;
                r = 0.0;
            }
        }
        if (s == 0) {
            if (depth) depth[pix] = valid ? (float)value : 0.0f;
            if (mask) mask[pix] = valid ? 1 : 0;
            if (rowmask) rowmask[pix] = (uint8_t)rm;
        } else if (rgb) {
            rgb[3 * pix + s - 1] = valid ? (float)value : 0.0f;
        }
        if (Jout) {
            float* jo = Jout + 24 * pix + 6 * s;
#pragma unroll
            for (int m = 0; m < 6; ++m) jo[m] = row[m];
        }
        if (resid) resid[4 * pix + s] = (float)r;
    }
    block_reduce29f(pacc, lds, partial_row);
}

template <typename T, bool Pool>
// at least 5 waves per SIMD (96 VGPRs, no spills; 4 without the cap)
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void k_render_jac(GridC g, CamC c, GridD gd, CamD cd, const T* __restrict__ map,
                                                    const unsigned* __restrict__ gbits,
                                                    const prism_pose* __restrict__ poses,
                                                    const float* __restrict__ obs_depth,
                                                    const float* __restrict__ obs_rgb, WeightsC wt,
                                                    float* __restrict__ depth, float* __restrict__ rgb,
                                                    uint8_t* __restrict__ mask, float* __restrict__ Jout,
                                                    float* __restrict__ resid, uint8_t* __restrict__ rowmask,
                                                    double* __restrict__ partials) {
    render_jac_block<T, Pool>(blockIdx.x, blockIdx.y, g, c, gd, cd, map, gbits, poses + blockIdx.y, obs_depth, obs_rgb,
                              wt, depth, rgb, mask, Jout, resid, rowmask,
                              partials + ((long long)blockIdx.y * gridDim.x + blockIdx.x) * PRISM_NEQ);
}

// batched: the render-through objective of every filter at its current
// iterate with its slot's frame (one frame each)
template <typename T, bool Pool>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void k_render_jac_batch(BatchArgs b) {
    const int a = batch_agent(b, blockIdx.x);
    const AgentDesc& D = *b.d[a];
    const prism_frame& fr = D.slots[b.slot[a]];
    const int blk = blockIdx.x - b.start[a];
    render_jac_block<T, Pool>(blk, 0, D.g, D.c, D.gd, D.cd, (const T*)D.map, D.bits, &D.S->iter,
                              (const float*)fr.depth, (const float*)fr.rgb, b.irls ? D.w_irls : D.w, nullptr, nullptr,
                              nullptr, nullptr, nullptr, nullptr, D.partials + (long long)blk * PRISM_NEQ);
}

// ---------------------------------------------------------------------------
// scattering a tile's gradient into the map
// ---------------------------------------------------------------------------
// The 16 rays of a wavefront's 4x4 pixels reach some dozens of distinct voxels
// through 256 corners per plane, so a wavefront first sums its contributions
// in LDS of its own and then issues one global atomic per distinct (plane,
// voxel).  Rays that see one surface reach a small box of voxels: the sums
// live in a window over that box, addressed directly, and go out in window
// order, where neighbouring lanes hold neighbouring voxels of a brick row and
// their atomics share cache lines.  How many boxes a window holds depends on
// the ratio of pixel to voxel.  Boxes beyond 236 / 256 voxels (double / float
// windows), first views of two rooms of 6.4 m: 256^3 at 320x240 7-14 / 3-6 %, at
// 240x180 25-36 / 13-23 %, at 160x120 64-75 / 56-58 %, 384^3 at 320x240
// 41-49 / 24-37 %.  Beyond it the adjoint adds to global memory directly, which
// is still faster at all of these than hash tables per tile were (8 frames of
// 160x120 at 256^3: 167 -> 94 us, 4 at 384^3: 142 -> 113); the descent's dearer
// atomics first go sample by sample (see k_gd_grad).
//
// LDS float atomics would bound a scatter by corners (170 clocks per
// instruction measured, whether or not lanes meet in an address), so the
// window is summed with plain reads and writes, which needs the addresses of
// one instruction to differ.  A cell's eight corners lie in the eight parity
// classes of (x, y, z); in turn q ray r takes its corner of class q ^ r, so
// eight consecutive rays always hold eight different classes, hence voxels;
// the two eights of a wavefront have a copy of the window each or take turns,
// the four lanes of a ray have a plane each, and no other wavefront shares
// the window.  Measured at 256^3, 320x240 (hash tables per tile before): the
// adjoint of 8 frames 399 -> 113 us (67 without any scatter), the descent
// gradient 72 -> 40 us (23; 34 with five workgroups per CU, see Scatter, and 31
// with the samples of larger boxes taking turns).

template <typename V, int Copies>
struct Scatter {
    // voxels per plane; a box of as many spans fewer than 64 bricks.  Double
    // windows are what lets a fifth workgroup onto a CU (32000 bytes each, with
    // the free-space bits, done with by then, in the same LDS), which pays where
    // most boxes fit either way, and costs where more of them fit 256.  20 descent
    // steps with 256 / 236, us: 256^3 at 320x240 946 / 827, 384^3 at 640x480
    // 2056 / 1929, 128^3 at 320x240 742 / 696; 256^3 at 160x120 826 / 891, 384^3
    // at 320x240 1416 / 1539; 160x120 and 80x60 otherwise within 2 %.
    static constexpr int kWin = sizeof(V) == 8 ? 236 : 256;
    V win[4][Copies][kWin + 8];   // planes and copies shifted in the banks
};

// the wavefront's box of vol = dx dy dz voxels from (x0, y0, z0); vol 0: no
// lane has a corner, -1: larger than a window
struct Window {
    int x0, y0, z0, dx, dy, dz, vol;
};

// a workgroup's: its four wavefronts' windows
template <typename V, int Copies>
struct TileScatter {
    Scatter<V, Copies> wave[4];
    Window at[4];
    uint8_t mark[256];   // bricks of a box that goes out (of each window's 64, when they go out one by one)
};

// pixels of a scattering wavefront: 4x4, four wavefronts per 8x8 tile
__device__ __forceinline__ void scatter_pixel(const Tile& tl, int& u, int& v, int& s) {
    const int t = threadIdx.x, r = (t >> 2) & 15, wv = t >> 6;
    s = t & 3;
    u = tl.u0 + ((wv & 1) << 2) + (r & 3);
    v = tl.v0 + ((wv >> 1) << 2) + (r >> 2);
}

// every lane's two cells (live: the lane's ray contributes) -> the window,
// cleared; the whole wavefront
template <typename V, int Copies>
__device__ __forceinline__ Window scatter_window(const GridC& g, Scatter<V, Copies>& S, bool live, const Cell& c0,
                                                 const Cell& c1) {
    int lo[3], hi[3];
    bool any = live;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[a] = max(min(c0.i[a], c1.i[a]), 0);
        hi[a] = min(max(c0.i[a], c1.i[a]) + 1, g.n - 1);
        any &= lo[a] <= hi[a];
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        int l = any ? lo[a] : INT_MAX, h = any ? hi[a] : -1;
        // the four lanes of a ray agree: quads, then rows, then the wavefront
        l = min(l, __builtin_amdgcn_update_dpp(l, l, 0x141, 0xF, 0xF, false));
        h = max(h, __builtin_amdgcn_update_dpp(h, h, 0x141, 0xF, 0xF, false));
        l = min(l, __builtin_amdgcn_update_dpp(l, l, 0x140, 0xF, 0xF, false));
        h = max(h, __builtin_amdgcn_update_dpp(h, h, 0x140, 0xF, 0xF, false));
        l = min(l, __shfl_xor(l, 16, 64));
        h = max(h, __shfl_xor(h, 16, 64));
        lo[a] = __builtin_amdgcn_readfirstlane(min(l, __shfl_xor(l, 32, 64)));
        hi[a] = __builtin_amdgcn_readfirstlane(max(h, __shfl_xor(h, 32, 64)));
    }
    Window w{lo[0], lo[1], lo[2], 0, 0, 0, 0};
    if (hi[0] < 0) return w;
    w.dx = hi[0] - lo[0] + 1;
    w.dy = hi[1] - lo[1] + 1;
    w.dz = hi[2] - lo[2] + 1;
    w.vol = w.dx * w.dy * w.dz;   // at most 2^30
    if (w.vol > Scatter<V, Copies>::kWin) {
        w.vol = -1;
        return w;
    }
    for (int e = threadIdx.x & 63; e < w.vol; e += 64)
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int k = 0; k < Copies; ++k) S.win[p][k][e] = V(0);
    wave_lds_order();
    return w;
}

// no brick marks wanted
struct NoMarks {
    __device__ void operator()(int) const {}
};

__device__ __forceinline__ void grad_out(float* p, float v) { atomicAdd(p, v); }
__device__ __forceinline__ void grad_out(double* p, double v) { unsafeAtomicAdd(p, v); }

// coef * (trilinear weight) into plane s at the in-grid corners of the cell
// (add: this lane does).  The whole wavefront.
template <typename V, int Copies>
__device__ __forceinline__ void scatter_cell(const GridC& g, Scatter<V, Copies>& S, const Window& w, int s,
                                             const Cell& cl, const float wt[3], V coef, bool add,
                                             V* __restrict__ grad) {
    const int r = (threadIdx.x >> 2) & 15;   // ray of the wavefront
    int c[3][2];
    V hat[3][2];
    bool ok[3][2];
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int far = ((cl.i[a] ^ (r >> a)) & 1) ^ d;   // corner of the axis's parity class r ^ d
            c[a][d] = cl.i[a] + far;
            hat[a][d] = (V)(far ? wt[a] : 1.0f - wt[a]);
            ok[a][d] = (unsigned)c[a][d] < (unsigned)g.n;
        }
    if (w.vol <= 0) {
        if (!add || w.vol == 0) return;
#pragma unroll 1
        for (int q = 0; q < 8; ++q) {
            const bool fx = q & 1, fy = q & 2, fz = q & 4;
            if (!((fx ? ok[0][1] : ok[0][0]) && (fy ? ok[1][1] : ok[1][0]) && (fz ? ok[2][1] : ok[2][0]))) continue;
            const int id = (int)vidx(g, fx ? c[0][1] : c[0][0], fy ? c[1][1] : c[1][0], fz ? c[2][1] : c[2][0]);
            grad_out(grad + (long long)s * g.nvox + id,
                     coef * ((fx ? hat[0][1] : hat[0][0]) * (fy ? hat[1][1] : hat[1][0]) * (fz ? hat[2][1] : hat[2][0])));
        }
        return;
    }
    int off[3][2];
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        off[0][d] = c[0][d] - w.x0;
        off[1][d] = (c[1][d] - w.y0) * w.dx;
        off[2][d] = (c[2][d] - w.z0) * w.dx * w.dy;
    }
    V* const win = &S.win[s][Copies == 2 ? r >> 3 : 0][0];
#pragma unroll
    for (int turn = 0; turn < 2 / Copies; ++turn) {
        if (add && (Copies == 2 || (r >> 3) == turn)) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int dx = q & 1, dy = (q >> 1) & 1, dz = q >> 2;
                if (ok[0][dx] && ok[1][dy] && ok[2][dz])
                    win[off[0][dx] + off[1][dy] + off[2][dz]] += coef * (hat[0][dx] * hat[1][dy] * hat[2][dz]);
                wave_lds_order();
            }
        }
        wave_lds_order();
    }
}

// touched(b) for the bricks that a wavefront without a window added to: those
// of its rays' in-grid corners (add: some lane of the ray added to the cell).
// After the atomics, and about once per brick: the rays of a wavefront lie in
// few bricks, so each looks a brick up in a table (a slot per brick of 8x8x8
// neighbours, in LDS the window leaves unused) and only the first reports it.
// (Each corner looking at its brick's mark waited for the atomics before it,
// and in a run's first step many lanes found the mark unset and met in its
// atomic: 132 -> 190 us for the first step of a 320x240 frame of a 384^3 map.)
template <typename V, int Copies, typename Touched>
__device__ __forceinline__ void touch_cells(const GridC& g, Scatter<V, Copies>& S, int s, const Cell& cl, bool add,
                                            const Touched& touched) {
    constexpr int kSlots = 512;
    static_assert(sizeof(S.win) >= kSlots * sizeof(int), "the table lives in the windows");
    int* const seen = reinterpret_cast<int*>(&S.win);
    for (int e = threadIdx.x & 63; e < kSlots; e += 64) seen[e] = -1;
    wave_lds_order();
#pragma unroll
    for (int dz = 0; dz < 2; ++dz) {   // the four lanes of a ray take two of the eight corners each
        const int x = cl.i[0] + (s & 1), y = cl.i[1] + (s >> 1), z = cl.i[2] + dz;
        if (!add || max(max((unsigned)x, (unsigned)y), (unsigned)z) >= (unsigned)g.n) continue;
        const int bx = x >> 3, by = y >> 3, bz = z >> 3, b = (bz * g.nb + by) * g.nb + bx;
        if (atomicExch(&seen[((bz & 7) << 6) | ((by & 7) << 3) | (bx & 7)], b) != b) touched(b);
    }
    wave_lds_order();   // the LDS is the next window's
}

// the sums of voxel (x, y, z) in window w of wavefront wv, added to sum
template <typename V, int Copies>
__device__ __forceinline__ void window_add(const TileScatter<V, Copies>& T, int wv, const Window& w, int x, int y,
                                           int z, V sum[4]) {
    x -= w.x0;
    y -= w.y0;
    z -= w.z0;
    if (w.vol <= 0 || (unsigned)x >= (unsigned)w.dx || (unsigned)y >= (unsigned)w.dy || (unsigned)z >= (unsigned)w.dz)
        return;
    const int e = (z * w.dy + y) * w.dx + x;
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int k = 0; k < Copies; ++k) sum[p] += T.wave[wv].win[p][k][e];
}

// The sums over a box of voxels to global memory, one atomic per (plane, voxel)
// that is not zero, in brick order: lanes in eights hold a brick row's voxels.
// Threads first, first + step, ...; sums(x, y, z, out) gives a voxel's four;
// touched(b): each brick that received something, through mark (a byte per
// brick of the box; order() makes them visible among the threads).
template <typename V, typename Sums, typename Order, typename Touched>
__device__ __forceinline__ void box_out(const GridC& g, int first, int step, const int lo[3], const int hi[3],
                                        uint8_t* mark, const Sums& sums, const Order& order, V* __restrict__ grad,
                                        const Touched& touched) {
    const int gx0 = lo[0] >> 3, dy = hi[1] - lo[1] + 1, dz = hi[2] - lo[2] + 1;
    const int ngx = (hi[0] >> 3) - gx0 + 1, vol = ngx * 8 * dy * dz;
    constexpr bool marks = !std::is_same<Touched, NoMarks>::value;
    const int by0 = lo[1] >> 3, nby = (hi[1] >> 3) - by0 + 1, bz0 = lo[2] >> 3, nbz = (hi[2] >> 3) - bz0 + 1;
    if constexpr (marks) {
        for (int e = first; e < ngx * nby * nbz; e += step) mark[e] = 0;
        order();
    }
    // quotients of small integers by a reciprocal: (r + 1/2) / d is at
    // least 1/(2d) from an integer
    const float iy = __builtin_amdgcn_rcpf((float)dy), iz = __builtin_amdgcn_rcpf((float)dz);
    for (int e = first; e < vol; e += step) {
        const int r = e >> 3, ry = (int)(((float)r + 0.5f) * iy), gx = (int)(((float)ry + 0.5f) * iz);
        const int x = ((gx0 + gx) << 3) | (e & 7), y = lo[1] + r - ry * dy, z = lo[2] + ry - gx * dz;
        V sum[4] = {V(0), V(0), V(0), V(0)};
        sums(x, y, z, sum);
        const long long id = vidx(g, x, y, z);
#pragma unroll
        for (int p = 0; p < 4; ++p)
            if (sum[p] != V(0)) {
                grad_out(grad + (long long)p * g.nvox + id, sum[p]);
                if constexpr (marks) mark[(((z >> 3) - bz0) * nby + (y >> 3) - by0) * ngx + gx] = 1;
            }
    }
    // once per box: a look at a brick's mark waits for the atomics before it
    if constexpr (marks) {
        order();
        for (int e = first; e < ngx * nby * nbz; e += step)
            if (mark[e]) touched(((bz0 + e / (ngx * nby)) * g.nb + by0 + (e / ngx) % nby) * g.nb + gx0 + e % ngx);
    }
}

// a wavefront's own window
template <typename V, int Copies, typename Touched>
__device__ __forceinline__ void wave_out(const GridC& g, TileScatter<V, Copies>& T, const Window& w,
                                         V* __restrict__ grad, const Touched& touched) {
    const int wv = threadIdx.x >> 6;
    const int lo[3] = {w.x0, w.y0, w.z0}, hi[3] = {w.x0 + w.dx - 1, w.y0 + w.dy - 1, w.z0 + w.dz - 1};
    box_out(g, (int)(threadIdx.x & 63), 64, lo, hi, T.mark + 64 * wv,
            [&](int x, int y, int z, V sum[4]) { window_add(T, wv, w, x, y, z, sum); }, [] { wave_lds_order(); }, grad,
            touched);
    wave_lds_order();
}

// The tile's sums to global memory.  Global atomics bound the scatter once the
// window sums are cheap, so the four windows are summed on the way out (a voxel
// on their borders goes out once), over the box of all four.  Windows far apart
// (a box beyond kTileBox) go out one by one.  The whole workgroup.
constexpr int kTileBox = 2048;   // spans at most 256 bricks

template <typename V, int Copies, typename Touched>
__device__ __forceinline__ void scatter_flush(const GridC& g, TileScatter<V, Copies>& T, const Window& mine,
                                              V* __restrict__ grad, const Touched& touched) {
    if ((threadIdx.x & 63) == 0) T.at[threadIdx.x >> 6] = mine;
    __syncthreads();
    Window w[4];
    int lo[3] = {INT_MAX, INT_MAX, INT_MAX}, hi[3] = {-1, -1, -1};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        w[k] = T.at[k];
        if (w[k].vol <= 0) continue;
        lo[0] = min(lo[0], w[k].x0);
        lo[1] = min(lo[1], w[k].y0);
        lo[2] = min(lo[2], w[k].z0);
        hi[0] = max(hi[0], w[k].x0 + w[k].dx - 1);
        hi[1] = max(hi[1], w[k].y0 + w[k].dy - 1);
        hi[2] = max(hi[2], w[k].z0 + w[k].dz - 1);
    }
    if (hi[0] < 0) return;
    const long long vol = ((hi[0] >> 3) - (lo[0] >> 3) + 1) * 8LL * (hi[1] - lo[1] + 1) * (hi[2] - lo[2] + 1);
    if (vol <= kTileBox) {
        box_out(g, (int)threadIdx.x, 256, lo, hi, T.mark,
                [&](int x, int y, int z, V sum[4]) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) window_add(T, k, w[k], x, y, z, sum);
                },
                [] { __syncthreads(); }, grad, touched);
    } else if (mine.vol > 0) {
        wave_out(g, T, mine, grad, touched);
    }
}

// ---------------------------------------------------------------------------
// adjoint of render w.r.t. map means (atomic scatter) and pose
// ---------------------------------------------------------------------------
// Four lanes per ray, as in the render: lane s recomputes plane s of the
// forward pass at the ray's first crossing (the plane's corners at the two
// cells, the double-precision shading, its row of the Jacobian) and scatters
// its share of the upstream gradient to the plane's 16 corners.
using VjpScatter = TileScatter<float, 2>;    // 33 KB: four workgroups per CU, as many as the registers allow

// sum over the quad in single precision (every lane ends with (x0 + x1) + (x2 + x3))
__device__ __forceinline__ float quad_sumf(float x) {
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, false));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xF, 0xF, false));
    return x;
}

// partials: six pose sums per workgroup
__global__ __launch_bounds__(256) void k_render_vjp(GridC g, CamC c, GridD gd, CamD cd, const float* __restrict__ map,
                                                    const prism_pose* __restrict__ poses,
                                                    const int32_t* __restrict__ hit_k,
                                                    const float* __restrict__ g_depth,
                                                    const float* __restrict__ g_rgb,
                                                    float* __restrict__ grad_mean,
                                                    double* __restrict__ partials) {
    __shared__ BlockPose sp;
    __shared__ double wsum[4][6];
    __shared__ VjpScatter T;
    const BlockPose& P = block_pose(poses + blockIdx.y, &sp);   // synchronises the workgroup
    int u, v, s;
    scatter_pixel(tile_of(c, blockIdx.x), u, v, s);
    double acc[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    Cell c0{}, c1{};
    float w0[3] = {0.0f, 0.0f, 0.0f}, w1[3] = {0.0f, 0.0f, 0.0f}, k0 = 0.0f, k1 = 0.0f;
    bool live = false;
    if (u < c.W && v < c.H) {
        const long long pix = (long long)blockIdx.y * c.W * c.H + (long long)v * c.W + u;
        const int k = hit_k[pix];
        if (k >= 1 && k < c.K) {   // the same for the four lanes of a ray
            float dir[3];
            ray_dir32(c, P.f, u, v, dir);
            const RayCoef rc = ray_coef(g, c, P.f, dir);
            c0 = sample_cell(rc, k - 1);
            c1 = sample_cell(rc, k);
            const QuadShade q = shade_quad<float, false>(g, gd, cd, P.d, u, v, map, c0, c1, k, s);
            // the forward pass's crossing test on lane 0's occupancy corners
            const int crossing = trilerp(q.cv1, c1.w) > c.tau && !(trilerp(q.cv0, c0.w) > c.tau) ? 1 : 0;
            if (__builtin_amdgcn_update_dpp(0, crossing, 0x00, 0xF, 0xF, false)) {
                const float gs = s == 0 ? g_depth[pix] : g_rgb[3 * pix + s - 1];
                // pose: the upstream gradient times this output's Jacobian row
                float row[6];
                jac_row_quad(g, q, dir, s, row);
#pragma unroll
                for (int m = 0; m < 6; ++m) acc[m] = (double)(gs * row[m]);
                // means: every output depends on the two occupancies through
                // alpha; colour plane s also through its own blend
                const float ga = quad_sumf(gs * (s == 0 ? q.d1 - q.d0 : (float)q.v1 - (float)q.v0));
                const float al = (float)q.alpha;
                const float inv_den = (float)(1.0 / (q.f1 - q.f0));
                k0 = s == 0 ? -ga * (1.0f - al) * inv_den : gs * (1.0f - al);
                k1 = s == 0 ? -ga * al * inv_den : gs * al;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    w0[a] = q.w0[a];
                    w1[a] = q.w1[a];
                }
                live = true;
            }
        }
    }
    double sum[3];
    wave_sum6(acc, sum);
    if ((threadIdx.x & 31) == 0)
#pragma unroll
        for (int j = 0; j < 3; ++j) wsum[threadIdx.x >> 6][((threadIdx.x >> 5) & 1) * 3 + j] = sum[j];
    __syncthreads();
    if (threadIdx.x < 6)
        partials[((long long)blockIdx.y * gridDim.x + blockIdx.x) * 6 + threadIdx.x] =
            (wsum[0][threadIdx.x] + wsum[1][threadIdx.x]) + (wsum[2][threadIdx.x] + wsum[3][threadIdx.x]);
    Scatter<float, 2>& A = T.wave[threadIdx.x >> 6];
    const Window w = scatter_window(g, A, live, c0, c1);
    scatter_cell(g, A, w, s, c0, w0, k0, live, grad_mean);
    scatter_cell(g, A, w, s, c1, w1, k1, live, grad_mean);
    scatter_flush(g, T, w, grad_mean, NoMarks());
}

// ---------------------------------------------------------------------------
// gradient of the map-filter objective w.r.t. the map means (descent mapping)
// ---------------------------------------------------------------------------
// Sets the brick's bit; the caller that flips it appends the brick to the
// list of bricks the step has to visit.
__device__ __forceinline__ void mark_brick(unsigned* __restrict__ marks, int* __restrict__ list, int b) {
    const unsigned bit = 1u << (b & 31);
    if (marks[b >> 5] & bit) return;
    const unsigned old = atomicOr(marks + (b >> 5), bit);
    if (!(old & bit)) {
        const int at = atomicAdd(list, 1);
        list[1 + at] = b;
    }
}

using GdScatter = TileScatter<double, 1>;    // 31.6 KB

// One frame's rows of the map-filter objective at the current means: the
// render-through rows (same validity, gates and weights as the P1 objective)
// give the cost sum w r^2 (per-workgroup partial) and, through the adjoint of
// the emission with the first crossing held, dE/dmean = sum 2 w r d(out)/dmean
// accumulated in double precision into grad [4][n^3] (brick order).  Every
// brick that receives a contribution is marked, and appended to `list`
// (count first) the first time.
__global__ __launch_bounds__(256) void k_gd_grad(GridC g, CamC c, GridD gd, CamD cd, const float* __restrict__ map,
                                                 const unsigned* __restrict__ gbits,
                                                 const prism_pose* __restrict__ pose,
                                                 const float* __restrict__ obs_depth,
                                                 const float* __restrict__ obs_rgb, WeightsC wt,
                                                 double* __restrict__ grad, unsigned* __restrict__ marks,
                                                 int* __restrict__ list, double* __restrict__ partials,
                                                 const double* __restrict__ pp, int np,
                                                 double* __restrict__ last_cost) {
    __shared__ BlockPose sp;
    __shared__ double wsum[4];
    // the workgroup past the tiles totals the objective before the last step
    if (last_cost && blockIdx.x == gridDim.x - 1) {
        gd_cost_block(pp, np, last_cost, wsum);
        return;
    }
    extern __shared__ __align__(16) unsigned lbits[];   // the bits, then (every ray marched) the windows
    GdScatter& T = *reinterpret_cast<GdScatter*>(lbits);
    lds_u32* const fb = block_setup(g, gbits, lbits, pose, &sp);   // synchronises the workgroup
    const BlockPose& P = sp;
    __shared__ int starts[4];
    const Tile tl = tile_of(c, blockIdx.x);
    const int start = fb ? tile_start(g, c, P.f, tl, fb, starts) : 0;
    int u, v, s;
    scatter_pixel(tl, u, v, s);
    double cost = 0.0, k0 = 0.0, k1 = 0.0;   // k0, k1: coefficients of this lane's plane at samples k*-1, k*
    Cell c0{}, c1{};
    float w0[3] = {0.0f, 0.0f, 0.0f}, w1[3] = {0.0f, 0.0f, 0.0f};
    if (u < c.W && v < c.H) {
        // the observation is in flight during the march
        const int pix = v * c.W + u;
        const float D = obs_depth[pix], O = s == 0 ? D : obs_rgb[3 * pix + s - 1];
        float dir[3];
        ray_dir32(c, P.f, u, v, dir);
        const RayCoef rc = ray_coef(g, c, P.f, dir);
        const int k = march_quad<float, false>(g, c, rc, map, fb, s, start);
        if (k >= 1 && depth_ok(D)) {   // the same for the four lanes of a ray
            c0 = sample_cell(rc, k - 1);
            c1 = sample_cell(rc, k);
            const QuadShade q = shade_quad<float, false>(g, gd, cd, P.d, u, v, map, c0, c1, k, s);
            const double r = q.value - (double)O;
            double l1 = s == 0 ? 0.0 : fabs(r);
            l1 = quad_sum(l1);
            const bool use_depth = fabs(quad_bcast0(r)) <= wt.gate_depth;
            const bool use_rgb = l1 <= wt.gate_rgb;
            const bool keep = s == 0 ? use_depth : use_rgb;
            const double w = s == 0 ? wt.w_depth : wt.w_rgb;
            const double gout = keep ? 2.0 * w * r : 0.0;   // dE / d(this lane's output)
            if (keep) cost = w * r * r;
            // every output depends on the two occupancies through alpha
            const double d0 = cd.dn + (double)(k - 1) * cd.step, d1 = cd.dn + (double)k * cd.step;
            double ga = gout * (s == 0 ? d1 - d0 : q.v1 - q.v0);
            ga += __shfl_xor(ga, 1, 64);
            ga += __shfl_xor(ga, 2, 64);
            const double inv_den = 1.0 / (q.f1 - q.f0);
            if (s == 0) {
                k0 = -ga * (1.0 - q.alpha) * inv_den;
                k1 = -ga * q.alpha * inv_den;
            } else {
                k0 = gout * (1.0 - q.alpha);
                k1 = gout * q.alpha;
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                w0[a] = q.w0[a];
                w1[a] = q.w1[a];
            }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cost += __shfl_xor(cost, off, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = cost;
    // a ray contributes when one of its four lanes does
    const bool add0 = quad_min(k0 != 0.0 ? 0 : 1) == 0, add1 = quad_min(k1 != 0.0 ? 0 : 1) == 0;
    const bool live = add0 || add1;
    __syncthreads();
    if (threadIdx.x == 0) partials[blockIdx.x] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
    Scatter<double, 1>& A = T.wave[threadIdx.x >> 6];
    const Window w = scatter_window(g, A, live, c0, c1);
    auto touched = [&](int b) { mark_brick(marks, list, b); };
    if (w.vol >= 0) {
        scatter_cell(g, A, w, s, c0, w0, k0, k0 != 0.0, grad);
        scatter_cell(g, A, w, s, c1, w1, k1, k1 != 0.0, grad);
    } else {
        // The two samples of a ray lie a step apart (over two voxels at K = n / 2),
        // so the cells of one of them reach half the box of both (a median of 144
        // voxels, not 288, for 256^3 at 160x120): they take the window in turn,
        // and it goes out in between.  Beyond the window are then 1 % of the
        // wavefronts at 256^3 / 320x240 (7-14 % at once), 13-23 % at 160x120
        // (64-75 %) and 2-5 % at 384^3 / 320x240 (41-49 %).  20 steps at 256^3 /
        // 320x240 take 826 us instead of 1233, at 384^3 / 320x240 1539 instead of
        // 2553 (2486 before there were windows); 5 at 256^3 / 160x120 227 / 269.
#pragma unroll 1
        for (int k = 0; k < 2; ++k) {
            const Cell cl = k ? c1 : c0;
            const float wt[3] = {k ? w1[0] : w0[0], k ? w1[1] : w0[1], k ? w1[2] : w0[2]};
            const double coef = k ? k1 : k0;
            const bool add = k ? add1 : add0;
            const Window own = scatter_window(g, A, add, cl, cl);
            scatter_cell(g, A, own, s, cl, wt, coef, coef != 0.0, grad);
            if (own.vol > 0)
                wave_out(g, T, own, grad, touched);
            else if (own.vol < 0)
                touch_cells(g, A, s, cl, add, touched);
        }
    }
    scatter_flush(g, T, w, grad, touched);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
int render_blocks(const CamC& c) { return ((c.W + 7) >> 3) * ((c.H + 7) >> 3); }
int vjp_blocks(const CamC& c) { return render_blocks(c); }

static size_t bits_lds(const GridC& g, const unsigned* bits) {
    return bits ? (size_t)free_lds_words(free_words(g.nb)) * 4 : 0;
}

hipError_t launch_render(const GridC& g, const CamC& c, const GridD& gd, const CamD& cd, int dtype, const void* map,
                         const unsigned* bits, const prism_pose* poses, int n_frames, float* depth, float* rgb,
                         uint8_t* mask, int32_t* hit_k, hipStream_t st) {
    dim3 grid(render_blocks(c), n_frames);
    size_t lds = bits_lds(g, bits);
    const bool pool = g.table != nullptr;
    const uint16_t* mh = (const uint16_t*)map;
    const float* mf = (const float*)map;
    if (dtype == PRISM_BF16 && pool)
        k_render<uint16_t, true><<<grid, 256, lds, st>>>(g, c, gd, cd, mh, bits, poses, depth, rgb, mask, hit_k);
    else if (dtype == PRISM_BF16)
        k_render<uint16_t, false><<<grid, 256, lds, st>>>(g, c, gd, cd, mh, bits, poses, depth, rgb, mask, hit_k);
    else if (pool)
        k_render<float, true><<<grid, 256, lds, st>>>(g, c, gd, cd, mf, bits, poses, depth, rgb, mask, hit_k);
    else
        k_render<float, false><<<grid, 256, lds, st>>>(g, c, gd, cd, mf, bits, poses, depth, rgb, mask, hit_k);
    return hipGetLastError();
}

hipError_t launch_render_batch(const BatchArgs& b, int dtype, bool pool, int max_lds_words, hipStream_t st) {
    // every filter copies free_lds_words of its dilated bits to LDS (block_setup):
    // the allocation is the largest of these over the batch
    size_t lds = (size_t)max_lds_words * 4;
    if (dtype == PRISM_BF16 && pool)
        k_render_batch<uint16_t, true><<<b.start[b.n], 256, lds, st>>>(b);
    else if (dtype == PRISM_BF16)
        k_render_batch<uint16_t, false><<<b.start[b.n], 256, lds, st>>>(b);
    else if (pool)
        k_render_batch<float, true><<<b.start[b.n], 256, lds, st>>>(b);
    else
        k_render_batch<float, false><<<b.start[b.n], 256, lds, st>>>(b);
    return hipGetLastError();
}

hipError_t launch_render_jac_batch(const BatchArgs& b, int dtype, bool pool, int max_lds_words, hipStream_t st) {
    size_t lds = (size_t)max_lds_words * 4;
    if (dtype == PRISM_BF16 && pool)
        k_render_jac_batch<uint16_t, true><<<b.start[b.n], 256, lds, st>>>(b);
    else if (dtype == PRISM_BF16)
        k_render_jac_batch<uint16_t, false><<<b.start[b.n], 256, lds, st>>>(b);
    else if (pool)
        k_render_jac_batch<float, true><<<b.start[b.n], 256, lds, st>>>(b);
    else
        k_render_jac_batch<float, false><<<b.start[b.n], 256, lds, st>>>(b);
    return hipGetLastError();
}

hipError_t launch_normals_batch(const BatchArgs& b, hipStream_t st) {
    k_normals_batch<<<b.start[b.n], 256, 0, st>>>(b);
    return hipGetLastError();
}

hipError_t launch_normals(const CamC& c, int n_frames, const float* depth, const uint8_t* mask, float disc,
                          float* normals, uint8_t* nmask, const int* counts, int ngroups, int64_t* n_updated,
                          int64_t* n_updated_total, hipStream_t st) {
    long long n = (long long)c.W * c.H * n_frames;
    k_normals<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(c, n_frames, depth, mask, disc, normals, nmask, counts,
                                                           ngroups, n_updated, n_updated_total);
    return hipGetLastError();
}

hipError_t launch_render_jac(const GridC& g, const CamC& c, const GridD& gd, const CamD& cd, int dtype,
                             const void* map, const unsigned* bits, const prism_pose* poses, int n_frames,
                             const float* obs_depth, const float* obs_rgb, const WeightsC& w, float* depth,
                             float* rgb, uint8_t* mask, float* J, float* resid, uint8_t* rowmask, double* partials,
                             hipStream_t st) {
    dim3 grid(render_blocks(c), n_frames);
    size_t lds = bits_lds(g, bits);
    const bool pool = g.table != nullptr;
    const uint16_t* mh = (const uint16_t*)map;
    const float* mf = (const float*)map;
    if (dtype == PRISM_BF16 && pool)
        k_render_jac<uint16_t, true><<<grid, 256, lds, st>>>(g, c, gd, cd, mh, bits, poses, obs_depth, obs_rgb, w,
                                                             depth, rgb, mask, J, resid, rowmask, partials);
    else if (dtype == PRISM_BF16)
        k_render_jac<uint16_t, false><<<grid, 256, lds, st>>>(g, c, gd, cd, mh, bits, poses, obs_depth, obs_rgb, w,
                                                              depth, rgb, mask, J, resid, rowmask, partials);
    else if (pool)
        k_render_jac<float, true><<<grid, 256, lds, st>>>(g, c, gd, cd, mf, bits, poses, obs_depth, obs_rgb, w,
                                                          depth, rgb, mask, J, resid, rowmask, partials);
    else
        k_render_jac<float, false><<<grid, 256, lds, st>>>(g, c, gd, cd, mf, bits, poses, obs_depth, obs_rgb, w,
                                                           depth, rgb, mask, J, resid, rowmask, partials);
    return hipGetLastError();
}

hipError_t launch_gd_grad(const GridC& g, const CamC& c, const GridD& gd, const CamD& cd, const float* map,
                          const unsigned* bits, const prism_pose* pose, const float* obs_depth, const float* obs_rgb,
                          const WeightsC& w, double* grad, unsigned* marks, int* list, double* partials,
                          const double* pp, double* last_cost, hipStream_t st) {
    const size_t lds = std::max(bits_lds(g, bits), sizeof(GdScatter));
    k_gd_grad<<<render_blocks(c) + (last_cost ? 1 : 0), 256, lds, st>>>(g, c, gd, cd, map, bits, pose, obs_depth,
                                                                        obs_rgb, w, grad, marks, list, partials, pp,
                                                                        gd_update_groups(g), last_cost);
    return hipGetLastError();
}

hipError_t launch_render_vjp(const GridC& g, const CamC& c, const GridD& gd, const CamD& cd, const float* map,
                             const prism_pose* poses, int n_frames, const int32_t* hit_k, const float* g_depth,
                             const float* g_rgb, float* grad_mean, double* partials, hipStream_t st) {
    dim3 grid(vjp_blocks(c), n_frames);
    k_render_vjp<<<grid, 256, 0, st>>>(g, c, gd, cd, map, poses, hit_k, g_depth, g_rgb, grad_mean, partials);
    return hipGetLastError();
}

}  // namespace prism
