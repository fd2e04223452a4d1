// Voxel-map storage kernels and the closed-form map update (App. D).
//
// Storage: 8 planes (mean occ, R, G, B, var occ, R, G, B) of n^3 values in
// 8x8x8-brick order, brick-major, x fastest inside a brick, followed by the
// brick summary (one value per brick whose sign is exact: <= 0 exactly when
// every occupancy mean of the brick is <= 0, and then not necessarily the
// largest; the largest occupancy mean when that is > 0), a bit per brick
// telling whether the summary is <= 0, the same dilated (set when the 2x2x2
// bricks from this one are all free: what the renderer keeps in LDS to skip
// free space) and per-workgroup update counts.
//
// The map update runs in three kernels and uses no global atomics.
//   cull:   one thread per brick tests the brick's voxel-centre box against
//           the view frustum (conservatively, with margins far above
//           single-precision rounding); each workgroup compacts its survivors
//           into its own 256-entry segment of a brick list (ballot + prefix
//           sums) and stores the segment length.  Block 0 also stores the
//           pose in both precisions for the next kernel.
//   update: a fixed grid of workgroups scans the segment lengths in LDS and
//           walks the compacted list, one brick per wavefront at a time: each
//           lane decides its eight voxels (one column of the brick) with the
//           single-precision recipe and updates only those, so HBM traffic is
//           the updated voxels' 8 planes read and written once; the brick
//           summary is refreshed in the same pass (its free-space bit toggled
//           when its sign changes), reading the occupancy of voxels left alone
//           only in bricks that held a voxel above 0, and each workgroup stores
//           its update count.
//   The count of updated voxels is the sum of the per-workgroup counts, taken
//   by a one-wavefront kernel or by the next kernel of a filter step.
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"

namespace prism {

// value as it reads back after a store of type T
template <typename T>
__device__ __forceinline__ float stored(float v);
template <>
__device__ __forceinline__ float stored<float>(float v) { return v; }
template <>
__device__ __forceinline__ float stored<uint16_t>(float v) { return __uint_as_float(((uint32_t)f2bf(v)) << 16); }

template <typename T>
__global__ __launch_bounds__(256) void k_map_init(long long nvox, T* __restrict__ map, float occ0, float rgb0,
                                                  float var0, MapAux aux, int nbricks) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nbricks) aux.bmax[i] = stored<T>(occ0);
    if (i >= nvox) return;
    st(map, i, occ0);
    st(map, nvox + i, rgb0);
    st(map, 2 * nvox + i, rgb0);
    st(map, 3 * nvox + i, rgb0);
#pragma unroll
    for (int c = 4; c < 8; ++c) st(map, c * nvox + i, var0);
}

// brick-pool map: every brick without a slot, bricks summarised by the
// value their voxels read as, pool counters cleared, var0 kept
__global__ __launch_bounds__(256) void k_pool_init(int nbricks, float pocc, float var0, MapAux aux) {
    int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b == 0) {
        aux.pool[0] = 0;
        aux.pool[1] = 0;
        *aux.var0 = var0;
    }
    if (b >= nbricks) return;
    aux.table[b] = -1;
    aux.bmax[b] = pocc;
}

// ---------------------------------------------------------------------------
// dense <-> brick order
// ---------------------------------------------------------------------------
// A copy between two orders is bound by memory, so both sides are read and
// written in whole 128-byte lines by one wavefront: it takes one z-slice of
// four bricks along x (32 x 8 voxels), a lane four consecutive voxels.  The
// dense side is then eight rows of 128 bytes, the brick side four slices of 64
// consecutive values (256 bytes, BF16 128), and the planes' loads are all in
// flight before the first store.  (One voxel per lane in brick order made a
// wavefront touch eight 32-byte pieces of eight lines, whose other pieces
// belong to workgroups of other XCDs, each fetching the line again.)  Measured
// on a 384^3 BF16 map, loaded and exported: 2484 -> 1030 us through the caches,
// 983 past them (5.5 TB/s of the bytes both need; a large plain copy reaches
// 4.7).
typedef float float4v __attribute__((ext_vector_type(4)));
// four floats of a caller's dense array, which is only 4-byte aligned
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));
typedef uint16_t bf16x4 __attribute__((ext_vector_type(4)));

// (non-temporal: a map loaded whole is read again only after the caches have
// seen the rest of it)
__device__ __forceinline__ void st4(float* p, long long i, float4v v) {
    __builtin_nontemporal_store(v, reinterpret_cast<float4v*>(p + i));
}
__device__ __forceinline__ void st4(uint16_t* p, long long i, float4v v) {
    bf16x4 h;
#pragma unroll
    for (int q = 0; q < 4; ++q) h[q] = f2bf(v[q]);
    __builtin_nontemporal_store(h, reinterpret_cast<bf16x4*>(p + i));
}
__device__ __forceinline__ float4v ldu4(const float* p, long long i) {
    return *reinterpret_cast<const float4u*>(p + i);
}
__device__ __forceinline__ void stu4(float* p, long long i, float4v v) { *reinterpret_cast<float4u*>(p + i) = v; }

// The same past the caches (non-temporal), for passes over far more than they
// hold: a line that such a pass leaves behind only pushes out others, dirty ones
// among them.
__device__ __forceinline__ float4v ld4_stream(const float* p, long long i) {
    return __builtin_nontemporal_load(reinterpret_cast<const float4v*>(p + i));
}
__device__ __forceinline__ float4v ld4_stream(const uint16_t* p, long long i) {
    const bf16x4 h = __builtin_nontemporal_load(reinterpret_cast<const bf16x4*>(p + i));
    float4v v;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = __uint_as_float((uint32_t)h[q] << 16);
    return v;
}
__device__ __forceinline__ float4v ldu4_stream(const float* p, long long i) {
    return __builtin_nontemporal_load(reinterpret_cast<const float4u*>(p + i));
}
__device__ __forceinline__ void stu4_stream(float* p, long long i, float4v v) {
    __builtin_nontemporal_store((float4u)v, reinterpret_cast<float4u*>(p + i));
}

// a lane's four voxels of slice k of the four bricks from (4 xg, by): the
// brick of the lane, the offset within it, the dense index (in: x < n)
struct QuadAt {
    long long brick, dense;
    int loc;
    bool in;
};

__device__ __forceinline__ QuadAt quad_at(int n, int nb, int xg, int by, int k) {
    const int lane = threadIdx.x & 63, q = lane & 7, y = lane >> 3, x = (xg << 5) + (q << 2);
    QuadAt a;
    a.in = x < n;
    a.brick = ((long long)(k >> 3) * nb + by) * nb + (x >> 3);
    a.loc = ((k & 7) << 6) | (y << 3) | (x & 7);
    a.dense = ((long long)k * n + (by << 3) + y) * n + x;
    return a;
}

// wavefront w of a copy: slices in order of x group, brick row, z
__device__ __forceinline__ bool slice_of(int n, int nb, int& xg, int& by, int& k) {
    const int w = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    const int ngx = (nb + 3) >> 2;
    xg = w % ngx;
    by = (w / ngx) % nb;
    k = w / (ngx * nb);
    return k < n;
}
static unsigned slice_blocks(int n) {
    const int nb = n / 8, ngx = (nb + 3) / 4;
    return (unsigned)((ngx * nb * n + 3) / 4);
}

// maximum over a wavefront (every lane gets it): DPP steps within 16 lanes
// (lane ^ 1, lane ^ 2, half-row and row mirrors), then two exchanges
__device__ __forceinline__ float wave_max(float m) {
    auto dpp = [](float x, auto ctrl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), decltype(ctrl)::value, 0xF, 0xF, false));
    };
    m = fmaxf(m, dpp(m, std::integral_constant<int, 0xB1>()));
    m = fmaxf(m, dpp(m, std::integral_constant<int, 0x4E>()));
    m = fmaxf(m, dpp(m, std::integral_constant<int, 0x141>()));
    m = fmaxf(m, dpp(m, std::integral_constant<int, 0x140>()));
    m = fmaxf(m, __shfl_xor(m, 16, 64));
    return fmaxf(m, __shfl_xor(m, 32, 64));
}

// Dense planes -> map.  A workgroup takes four bricks along x (two slices per
// wavefront) and, when means come in, stores the bricks' occupancy maxima on
// the way: the means are not read again for the brick summary.
template <typename T>
__global__ __launch_bounds__(256) void k_from_dense(int n, int nb, T* __restrict__ map,
                                                    const float* __restrict__ mean4,
                                                    const float* __restrict__ var4, float* __restrict__ bmax) {
    __shared__ float wmax[4][4];
    const long long nvox = (long long)n * n * n;
    const int ngx = (nb + 3) >> 2;
    const int xg = blockIdx.x % ngx, by = (blockIdx.x / ngx) % nb, bz = blockIdx.x / (ngx * nb);
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const QuadAt a0 = quad_at(n, nb, xg, by, (bz << 3) | wv);
    const long long e0 = (a0.brick << 9) | a0.loc;
    const long long d4 = 4LL * n * n;   // four slices on: 256 elements in the brick
    float m = NAN;   // (fmaxf passes over it: a brick without a number keeps it, and is not free)
    if (a0.in) {
        float4v v[2][4], w[2][4];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (mean4) v[s][c] = ldu4_stream(mean4, c * nvox + a0.dense + s * d4);
                if (var4) w[s][c] = ldu4_stream(var4, c * nvox + a0.dense + s * d4);
            }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (mean4) st4(map, c * nvox + e0 + 256 * s, v[s][c]);
                if (var4) st4(map, (4 + c) * nvox + e0 + 256 * s, w[s][c]);
            }
        if (mean4)
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int q = 0; q < 4; ++q) m = fmaxf(m, stored<T>(v[s][0][q]));
    }
    if (!mean4) return;
    // lanes of one brick: those that agree in bits 1 and 2
    m = fmaxf(m, __shfl_xor(m, 1, 64));
    m = fmaxf(m, __shfl_xor(m, 8, 64));
    m = fmaxf(m, __shfl_xor(m, 16, 64));
    m = fmaxf(m, __shfl_xor(m, 32, 64));
    if (lane < 8 && !(lane & 1)) wmax[wv][lane >> 1] = m;
    __syncthreads();
    const int bx = (xg << 2) + (int)threadIdx.x;
    if (threadIdx.x < 4 && bx < nb)
        bmax[((long long)bz * nb + by) * nb + bx] = fmaxf(fmaxf(wmax[0][threadIdx.x], wmax[1][threadIdx.x]),
                                                         fmaxf(wmax[2][threadIdx.x], wmax[3][threadIdx.x]));
}

// Map -> dense planes; in a brick-pool map the voxels of bricks without a
// slot take the values they read as (and var0).
template <typename T, bool Pool>
__global__ __launch_bounds__(256) void k_to_dense(GridC g, const T* __restrict__ map, MapAux aux,
                                                  float* __restrict__ mean4, float* __restrict__ var4) {
    int xg, by, k;
    if (!slice_of(g.n, g.nb, xg, by, k)) return;
    const QuadAt a = quad_at(g.n, g.nb, xg, by, k);
    if (!a.in) return;
    const long long nvox = (long long)g.n * g.n * g.n;
    long long slot = a.brick;
    float v0 = 0.0f;
    if constexpr (Pool) {
        slot = g.table[a.brick];
        v0 = stored<T>(*aux.var0);
    }
    const long long e = (slot << 9) | a.loc;
    float4v m[4], w[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float prior = c == 0 ? g.pocc : g.prgb;
        if (mean4) m[c] = !Pool || slot >= 0 ? ld4_stream(map, c * g.nvox + e) : float4v(prior);
        if (var4) w[c] = !Pool || slot >= 0 ? ld4_stream(map, (4 + c) * g.nvox + e) : float4v(v0);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if (mean4) stu4_stream(mean4, c * nvox + a.dense, m[c]);
        if (var4) stu4_stream(var4, c * nvox + a.dense, w[c]);
    }
}

// single-precision planes between the two orders
template <bool ToDense>
__global__ __launch_bounds__(256) void k_planes(int n, int nb, int channels, const float* __restrict__ src,
                                                float* __restrict__ dst) {
    int xg, by, k;
    if (!slice_of(n, nb, xg, by, k)) return;
    const QuadAt a = quad_at(n, nb, xg, by, k);
    if (!a.in) return;
    const long long nvox = (long long)n * n * n, e = (a.brick << 9) | a.loc;
    const long long from = ToDense ? e : a.dense, to = ToDense ? a.dense : e;
    float4v v[8];
#pragma unroll
    for (int c = 0; c < 8; ++c)
        if (c < channels) v[c] = ldu4(src, c * nvox + from);
#pragma unroll
    for (int c = 0; c < 8; ++c)
        if (c < channels) stu4(dst, c * nvox + to, v[c]);
}

// Brick summary and free-space bits of every brick (after writes that bypass
// the map update).  Bound by the read of the occupancy plane: a workgroup
// takes the 32 bricks of one word of bits, eight per wavefront, whose loads
// (16 bytes per lane) are all issued before the first maximum is formed, and
// the word is packed here rather than by a pass of its own.  256^3 FP32: 25 us
// with cached loads (2.7 TB/s), 13.5 past the caches; the render that follows
// finds fewer of its lines there and takes 65 instead of 60.
template <typename T, bool Pool>
__global__ __launch_bounds__(256) void k_brick_summary(GridC g, const T* __restrict__ map, MapAux aux, int nbricks) {
    __shared__ unsigned wbits[4];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int b0 = (int)blockIdx.x * 32 + wv * 8;
    float4v v[8][2];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int b = b0 + j;
        v[j][0] = v[j][1] = float4v(g.pocc);
        if (b >= nbricks) continue;
        long long slot = b;
        if constexpr (Pool) {
            slot = g.table[b];
            if (slot < 0) continue;
        }
        const T* p = map + (slot << 9);
        // halves of the brick (FP32 1 KB, BF16 512 bytes each)
        v[j][0] = ld4_stream(p, 4 * lane);
        v[j][1] = ld4_stream(p, 256 + 4 * lane);
    }
    unsigned mine = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        float m = fmaxf(fmaxf(v[j][0][0], v[j][0][1]), fmaxf(v[j][0][2], v[j][0][3]));
        m = fmaxf(m, fmaxf(fmaxf(v[j][1][0], v[j][1][1]), fmaxf(v[j][1][2], v[j][1][3])));
        m = wave_max(m);
        if (b0 + j >= nbricks) continue;
        if (lane == 0) aux.bmax[b0 + j] = m;
        mine |= (m <= 0.0f ? 1u : 0u) << (wv * 8 + j);
    }
    if (lane == 0) wbits[wv] = mine;
    __syncthreads();
    if (threadIdx.x == 0) aux.bits[blockIdx.x] = (wbits[0] | wbits[1]) | (wbits[2] | wbits[3]);
}

// packs the free-space bits (brick maximum <= 0) from the brick summary
__global__ __launch_bounds__(256) void k_pack_bits(int nbricks, MapAux aux) {
    int w = blockIdx.x * blockDim.x + threadIdx.x;
    int nwords = (nbricks + 31) >> 5;
    if (w >= nwords) return;
    unsigned word = 0;
    if ((w << 5) + 32 <= nbricks) {
        // 32 contiguous floats: eight 16-byte loads issued together
        const float4* p4 = reinterpret_cast<const float4*>(aux.bmax + (w << 5));
        float4 v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = p4[i];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            word |= (v[i].x <= 0.0f ? 1u : 0u) << (4 * i);
            word |= (v[i].y <= 0.0f ? 1u : 0u) << (4 * i + 1);
            word |= (v[i].z <= 0.0f ? 1u : 0u) << (4 * i + 2);
            word |= (v[i].w <= 0.0f ? 1u : 0u) << (4 * i + 3);
        }
    } else {
        for (int i = 0; (w << 5) + i < nbricks; ++i)
            if (aux.bmax[(w << 5) + i] <= 0.0f) word |= 1u << i;
    }
    aux.bits[w] = word;
}

// The dilated free-space bits (second bitmap after the plain one): word w
// is the AND of the 32-bit windows of the plain bits that start at bricks
// 32 w + {0, 1} + {0, nb} + {0, nb^2}; words past the bitmap read as 0.  Every
// cell, whether it spans bricks or not, lies inside the 2x2x2 block of its base
// corner's brick, so this one bit proves it free.  Recomputed after every
// change of the plain bits.
__device__ __forceinline__ unsigned bits_window(const unsigned* __restrict__ bits, int nwords, int bit) {
    const int w = bit >> 5, sh = bit & 31;
    const unsigned lo = w < nwords ? bits[w] : 0u, hi = w + 1 < nwords ? bits[w + 1] : 0u;
    return sh ? (lo >> sh) | (hi << (32 - sh)) : lo;
}

__device__ __forceinline__ void dilate_block(int blk, int nb, unsigned* __restrict__ bits) {
    const int nwords = free_words(nb);
    const int w = blk * (int)blockDim.x + (int)threadIdx.x;
    if (w >= nwords) return;
    const int b = w << 5, sy = nb, sz = nb * nb;
    unsigned d = bits[w];
    d &= bits_window(bits, nwords, b + 1);
    d &= bits_window(bits, nwords, b + sy);
    d &= bits_window(bits, nwords, b + sy + 1);
    d &= bits_window(bits, nwords, b + sz);
    d &= bits_window(bits, nwords, b + sz + 1);
    d &= bits_window(bits, nwords, b + sz + sy);
    d &= bits_window(bits, nwords, b + sz + sy + 1);
    bits[nwords + w] = d;
}

__global__ __launch_bounds__(256) void k_dilate_bits(int nb, unsigned* __restrict__ bits) {
    dilate_block(blockIdx.x, nb, bits);
}

// the same, with workgroup 0 also totalling the update's per-workgroup
// voxel counts (the whole workgroup, before any thread leaves)
__global__ __launch_bounds__(256) void k_dilate_bits_sum(int nb, unsigned* __restrict__ bits,
                                                         const int* __restrict__ counts, int ngroups,
                                                         int64_t* __restrict__ n_updated) {
    __shared__ long long part[4];
    if (blockIdx.x == 0) sum_counts_block(counts, ngroups, n_updated, part);
    dilate_block(blockIdx.x, nb, bits);
}

// Conservative brick cull: true if no voxel centre of the brick can pass the
// per-voxel test.  Each test is a convex region (behind the camera, or beyond
// one side plane of the frustum) checked on the 8 corners of the brick's
// voxel-centre box.
__device__ inline bool brick_culled(const GridC& g, const CamC& c, const Pose32& P, int bx, int by, int bz) {
    const float mz = 1e-3f, mp = 0.5f;
    bool all_behind = true, all_l = true, all_r = true, all_t = true, all_b = true;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        float x[3] = {g.o[0] + g.s * ((float)((bx << 3) + ((q & 1) ? 7 : 0)) + 0.5f),
                      g.o[1] + g.s * ((float)((by << 3) + ((q & 2) ? 7 : 0)) + 0.5f),
                      g.o[2] + g.s * ((float)((bz << 3) + ((q & 4) ? 7 : 0)) + 0.5f)};
        float d[3] = {x[0] - P.t[0], x[1] - P.t[1], x[2] - P.t[2]};
        float X = P.R[0][0] * d[0] + P.R[1][0] * d[1] + P.R[2][0] * d[2];
        float Y = P.R[0][1] * d[0] + P.R[1][1] * d[1] + P.R[2][1] * d[2];
        float Z = P.R[0][2] * d[0] + P.R[1][2] * d[1] + P.R[2][2] * d[2];
        bool front = Z > mz;
        all_behind &= Z < -mz;
        all_l &= front && (c.fx * X + (c.cx + mp) * Z < 0.0f);
        all_r &= front && (c.fx * X + (c.cx - (float)c.W - mp) * Z > 0.0f);
        all_t &= front && (c.fy * Y + (c.cy + mp) * Z < 0.0f);
        all_b &= front && (c.fy * Y + (c.cy - (float)c.H - mp) * Z > 0.0f);
    }
    return all_behind || all_l || all_r || all_t || all_b;
}

struct PosePair {
    Pose32 f;
    Pose64 d;
};

// workgroup blk of the cull (bricks blk*256 .. blk*256+255)
__device__ __forceinline__ void cull_block(int blk, const GridC& g, const CamC& c, const prism_pose* __restrict__ pose,
                                           const MapAux& aux) {
    __shared__ PosePair sp;
    __shared__ int wcount[4];
    if (threadIdx.x == 0) {
        sp.d = load_pose64(pose);
        sp.f = to32(sp.d);
        if (blk == 0) *reinterpret_cast<PosePair*>(aux.pose) = sp;
    }
    __syncthreads();
    int nbricks = g.nb * g.nb * g.nb;
    int b = blk * blockDim.x + threadIdx.x;
    bool keep = false;
    if (b < nbricks) {
        int bx = b % g.nb, by = (b / g.nb) % g.nb, bz = b / (g.nb * g.nb);
        keep = !brick_culled(g, c, sp.f, bx, by, bz);
    }
    // compaction inside the workgroup: rank = survivors before this thread
    unsigned long long m = __ballot(keep);
    int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int rank = __popcll(m & ((1ull << lane) - 1ull));
    if (lane == 0) wcount[wv] = __popcll(m);
    __syncthreads();
    int base = 0;
    for (int w = 0; w < wv; ++w) base += wcount[w];
    if (keep) aux.list[blk * 256 + base + rank] = b;
    if (threadIdx.x == 0) aux.segcnt[blk] = wcount[0] + wcount[1] + wcount[2] + wcount[3];
}

__global__ __launch_bounds__(256) void k_cull(GridC g, CamC c, const prism_pose* __restrict__ pose, MapAux aux) {
    cull_block(blockIdx.x, g, c, pose, aux);
}



// plane p of a map as a global-space pointer (uniform, so it lives in
// scalar registers), and element loads / stores through it
template <typename T>
__device__ __forceinline__ gptr<T> plane_g(const T* map, const GridC& g, int p) {
    return as_global(map + (long long)p * g.nvox);
}
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T* plane_w(T* map, const GridC& g, int p) {
    return (__attribute__((address_space(1))) T*)(map + (long long)p * g.nvox);
}
// Element i of a plane through a 32-bit byte offset (a plane holds at most
// 2^30 elements of at most 4 bytes): the plane's base stays in scalar
// registers and one vector offset serves all eight planes (an element index
// scaled in 64 bits would take a 64-bit vector address per plane).
__device__ __forceinline__ float ldp(gptr<float> p, unsigned i) { return ldg(p, i * 4u); }
__device__ __forceinline__ float ldp(gptr<uint16_t> p, unsigned i) { return ldg(p, i * 2u); }
__device__ __forceinline__ void stp(__attribute__((address_space(1))) float* p, unsigned i, float v) {
    *(__attribute__((address_space(1))) float*)((__attribute__((address_space(1))) char*)p + i * 4u) = v;
}
__device__ __forceinline__ void stp(__attribute__((address_space(1))) uint16_t* p, unsigned i, float v) {
    *(__attribute__((address_space(1))) uint16_t*)((__attribute__((address_space(1))) char*)p + i * 2u) = f2bf(v);
}

// workgroup blk of ngroups of the update.  Bound by the latency of a brick's
// chain (list, projection, depth gather, planes, stores) at four wavefronts per
// SIMD (128 VGPRs, batched 114), warm also by the planes' bytes: 106 MB of a
// 256^3 FP32 map (1.65 M voxels) take 22 us at the rate of a large copy
// (4.7 TB/s), the kernel 27, of which 5 go before the first brick; 176 MB of a
// 384^3 BF16 map 37 and 50.  16-byte accesses with all of a brick in flight
// (27.7 / 62, 178 VGPRs) and a workgroup per brick (26.6 / 51) move them no
// faster, nor do loads or stores past the caches (27.7, 29.7).  All of these
// walk every brick in the frustum, about a third of which hold no voxel that the
// frame updates, and decide in the kernel that moves the values; a separate
// pass of decisions has not been tried.
template <typename T, bool Pool>
__device__ __forceinline__ void map_update_block(int blk, int ngroups, const GridC& g, const CamC& c, const GridD& gd,
                                                 T* __restrict__ map, const float* __restrict__ depth,
                                                 const float* __restrict__ rgb, const MapUpdC& mp, const MapAux& aux,
                                                 int nseg) {
    extern __shared__ int sstart[];    // [nseg + 1] exclusive prefix of the segment lengths
    __shared__ PosePair sp;
    __shared__ int lcnt[4];
    __shared__ int wsum[4];
    // segment lengths -> exclusive prefix sums: each thread sums one
    // contiguous chunk, the chunk sums are scanned across the workgroup
    // (shuffle scan per wavefront, then the four wavefront totals)
    int per = (nseg + 255) / 256;
    int lo = threadIdx.x * per, hi = min(lo + per, nseg);
    int s = 0;
    for (int i = lo; i < hi; ++i) {
        sstart[i] = s;
        s += aux.segcnt[i];
    }
    if (threadIdx.x == 0) sp = *reinterpret_cast<const PosePair*>(aux.pose);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int incl = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        int t = __shfl_up(incl, off, 64);
        if (lane >= off) incl += t;
    }
    if (lane == 63) wsum[wv] = incl;
    __syncthreads();
    int excl = incl - s;
    for (int w = 0; w < wv; ++w) excl += wsum[w];
    for (int i = lo; i < hi; ++i) sstart[i] += excl;
    if (threadIdx.x == 0) sstart[nseg] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
    const Pose32& P = sp.f;
    const Pose64& Q = sp.d;
    const int total = sstart[nseg];
    // one brick per wavefront at a time: lane `lane` owns voxel (lane & 7,
    // lane >> 3) of each of the brick's 8 z-slices, so every load and store
    // of a slice is 64 consecutive elements; no workgroup barrier per brick
    const int nwaves = ngroups * 4;
    int cnt = 0;
    // brick of list entry e: the segment holding e (binary search over the
    // prefix sums), then its list slot
    auto brick_of = [&](int e) {
        int a = 0, z = nseg;
        while (z - a > 1) {
            int mid = (a + z) >> 1;
            if (sstart[mid] <= e) a = mid; else z = mid;
        }
        return aux.list[a * 256 + (e - sstart[a])];
    };
    // the next brick's index is loaded while this one is processed, so the
    // list read is off each brick's chain of memory round trips
    int b_next = blk * 4 + wv < total ? brick_of(blk * 4 + wv) : 0;
    for (int e = blk * 4 + wv; e < total; e += nwaves) {
        const int b = b_next;
        if (e + nwaves < total) b_next = brick_of(e + nwaves);
        // the brick's summary, issued with the depth gathers below
        const float bm_old = aux.bmax[b];
        const int bx = b % g.nb, by = (b / g.nb) % g.nb, bz = b / (g.nb * g.nb);
        const int i = (bx << 3) | (lane & 7), j = (by << 3) | (lane >> 3);
        // decisions for the lane's 8 voxels in single precision
        int pix[8];
        float Dv[8];
        bool upd[8];
#pragma unroll
        for (int h = 0; h < 8; ++h) {
            const int k = (bz << 3) | h;
            float x[3] = {g.o[0] + g.s * ((float)i + 0.5f), g.o[1] + g.s * ((float)j + 0.5f),
                          g.o[2] + g.s * ((float)k + 0.5f)};
            float d[3] = {x[0] - P.t[0], x[1] - P.t[1], x[2] - P.t[2]};
            float X[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) X[q] = (P.R[0][q] * d[0] + P.R[1][q] * d[1]) + P.R[2][q] * d[2];
            upd[h] = false;
            pix[h] = 0;
            Dv[h] = 0.0f;
            if (X[2] > 0.0f) {
                float uu = c.fx * (X[0] / X[2]) + c.cx;
                float vv = c.fy * (X[1] / X[2]) + c.cy;
                if (uu >= 0.0f && uu < (float)c.W && vv >= 0.0f && vv < (float)c.H) {
                    pix[h] = (int)vv * c.W + (int)uu;
                    upd[h] = true;
                }
            }
        }
#pragma unroll
        for (int h = 0; h < 8; ++h)
            if (upd[h]) Dv[h] = ldg(as_global(depth), (unsigned)pix[h] * 4u);
#pragma unroll
        for (int h = 0; h < 8; ++h) {
            if (upd[h]) {
                const int k = (bz << 3) | h;
                float x[3] = {g.o[0] + g.s * ((float)i + 0.5f), g.o[1] + g.s * ((float)j + 0.5f),
                              g.o[2] + g.s * ((float)k + 0.5f)};
                float d[3] = {x[0] - P.t[0], x[1] - P.t[1], x[2] - P.t[2]};
                float X2 = (P.R[0][2] * d[0] + P.R[1][2] * d[1]) + P.R[2][2] * d[2];
                upd[h] = depth_ok(Dv[h]) && X2 <= Dv[h] + mp.trunc32;
            }
        }
        // a listed brick none of whose voxels this frame updates (in the
        // frustum but behind the observed surfaces) keeps its values and its
        // summary: nothing more to read or write
        {
            int any = 0;
#pragma unroll
            for (int h = 0; h < 8; ++h) any |= upd[h] ? 1 : 0;
            if (!__any(any)) continue;
        }
        // brick-pool map: the brick's slot, handed out the first time one of
        // its voxels is updated and filled with the values its voxels read as;
        // with the pool full the brick's update is dropped and counted
        long long slot = b;
        bool fresh = false;
        float pvar = 0.0f;
        if constexpr (Pool) {
            int sl = aux.table[b];
            if (sl < 0) {
                int got = -1;
                if (lane == 0) {
                    const int s2 = atomicAdd(&aux.pool[0], 1);
                    if (s2 < aux.capacity) {
                        aux.table[b] = s2;
                        got = s2;
                    } else {
                        // pool full: give the ticket back, count the drop
                        atomicSub(&aux.pool[0], 1);
                        atomicAdd(&aux.pool[1], 1);
                    }
                }
                sl = __shfl(got, 0, 64);
                fresh = sl >= 0;
                pvar = stored<T>(*aux.var0);
            }
            if (sl < 0) continue;
            slot = sl;
        }
        // occupancy of voxels this update leaves alone is read only where it
        // can decide the brick's free-space bit: in a brick holding a voxel
        // above 0 before the update (in a free brick every such voxel is <= 0)
        const bool need_occ = !fresh && !(bm_old <= 0.0f);
        float m = -INFINITY;
        // the lane's eight z-slices in groups of two: a group's plane and
        // colour loads are all issued before any of them is used (one memory
        // round trip per group, not per voxel; groups of four cost more in
        // registers, hence waves, than they save), through global-space
        // plane pointers with 32-bit element offsets (a plane holds at most
        // 2^30 elements)
        const unsigned base = (unsigned)((slot << 9) | lane);
#pragma unroll
        for (int h0 = 0; h0 < 8; h0 += 2) {
            float lv[2][8], lc[2][3];
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const int h = h0 + hh;
                const unsigned id = base | (unsigned)(h << 6);
                if (upd[h]) {
                    if (!fresh) {
#pragma unroll
                        for (int pl = 0; pl < 8; ++pl) lv[hh][pl] = ldp(plane_g(map, g, pl), id);
                    }
                    const int px = pix[h];
#pragma unroll
                    for (int ch = 0; ch < 3; ++ch) lc[hh][ch] = ldg(as_global(rgb), (unsigned)(3 * px + ch) * 4u);
                } else if (need_occ) {
                    lv[hh][0] = ldp(plane_g(map, g, 0), id);
                }
            }
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const int h = h0 + hh;
                const int k = (bz << 3) | h;
                const unsigned id = base | (unsigned)(h << 6);
                if (!upd[h]) {
                    if (fresh) {
#pragma unroll
                        for (int ch = 0; ch < 4; ++ch) {
                            stp(plane_w(map, g, ch), id, ch == 0 ? g.pocc : g.prgb);
                            stp(plane_w(map, g, 4 + ch), id, pvar);
                        }
                        m = fmaxf(m, g.pocc);
                    } else if (need_occ) {
                        m = fmaxf(m, lv[hh][0]);
                    }
                    continue;
                }
                // values in double precision: camera depth of the voxel centre,
                // truncated negative SDF, Gaussian product in precision form
                double dd0 = (gd.o[0] + gd.s * ((double)i + 0.5)) - Q.t[0];
                double dd1 = (gd.o[1] + gd.s * ((double)j + 0.5)) - Q.t[1];
                double dd2 = (gd.o[2] + gd.s * ((double)k + 0.5)) - Q.t[2];
                double zc = Q.R[0][2] * dd0 + Q.R[1][2] * dd1 + Q.R[2][2] * dd2;
                double f0 = zc - (double)Dv[h];
                if (f0 < -mp.trunc) f0 = -mp.trunc;
                // App. D: new precision = old + update precision; new mean =
                // inverse of the new precision times the precision-weighted sum.
                // The four channels of a voxel are always updated together with
                // one update precision, so their variances are normally equal bit
                // for bit: the precision algebra is then done once (same inputs,
                // same operations, same results as per channel).  Channels are
                // valued one after another (few double-precision registers live).
                const float vs0 = fresh ? pvar : lv[hh][4];
                const bool same = fresh || (lv[hh][4] == lv[hh][5] && lv[hh][5] == lv[hh][6] && lv[hh][6] == lv[hh][7]);
                double lam = 1.0 / (double)vs0;
                double var2 = 1.0 / (lam + mp.lam_u);
#pragma unroll
                for (int ch = 0; ch < 4; ++ch) {
                    if (ch > 0 && !same) {
                        lam = 1.0 / (double)lv[hh][4 + ch];
                        var2 = 1.0 / (lam + mp.lam_u);
                    }
                    const double mu = fresh ? (double)(ch == 0 ? g.pocc : g.prgb) : (double)lv[hh][ch];
                    const double fc = ch == 0 ? f0 : (double)lc[hh][ch - 1];
                    float nm = (float)(var2 * (lam * mu + mp.lam_u * fc));
                    stp(plane_w(map, g, ch), id, nm);
                    stp(plane_w(map, g, 4 + ch), id, (float)var2);
                    if (ch == 0) m = fmaxf(m, stored<T>(nm));
                }
                ++cnt;
            }
        }
        for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
        if (lane == 0) {
            // The summary keeps an exact sign: in a brick that held a voxel
            // above 0, every voxel was read and m is the largest occupancy;
            // in a free brick the voxels left alone are <= 0, so m > 0 is the
            // largest occupancy and m <= 0 (or no update) leaves the brick
            // free.  The free-space bit toggles when the sign changes (each
            // brick has one owner per launch, so toggles of one word touch
            // different bits).
            const bool was_free = bm_old <= 0.0f;
            const float bm_new = (was_free && !(m > 0.0f)) ? fmaxf(m, bm_old) : m;
            const bool now_free = bm_new <= 0.0f;
            aux.bmax[b] = bm_new;
            if (was_free != now_free) atomicXor(&aux.bits[b >> 5], 1u << (b & 31));
        }
    }
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, 64);
    if (lane == 0) lcnt[wv] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) aux.counts[blk] = lcnt[0] + lcnt[1] + lcnt[2] + lcnt[3];
}

template <typename T, bool Pool>
__global__ __launch_bounds__(256) void k_map_update(GridC g, CamC c, GridD gd, T* __restrict__ map,
                                                    const float* __restrict__ depth,
                                                    const float* __restrict__ rgb, MapUpdC mp, MapAux aux,
                                                    int nseg) {
    map_update_block<T, Pool>(blockIdx.x, gridDim.x, g, c, gd, map, depth, rgb, mp, aux, nseg);
}

// batched: every filter culls / updates its map at its posterior mean with
// its slot's frame
__global__ __launch_bounds__(256) void k_cull_batch(BatchArgs b) {
    const int a = batch_agent(b, blockIdx.x);
    const AgentDesc& D = *b.d[a];
    cull_block(blockIdx.x - b.start[a], D.g, D.c, &D.S->pose, D.aux);
}

__global__ __launch_bounds__(256) void k_dilate_bits_batch(BatchArgs b) {
    const int a = batch_agent(b, blockIdx.x);
    const AgentDesc& D = *b.d[a];
    dilate_block(blockIdx.x - b.start[a], D.g.nb, D.aux.bits);
}

template <typename T, bool Pool>
__global__ __launch_bounds__(256) void k_map_update_batch(BatchArgs b) {
    const int a = batch_agent(b, blockIdx.x);
    const AgentDesc& D = *b.d[a];
    const prism_frame& fr = D.slots[b.slot[a]];
    map_update_block<T, Pool>(blockIdx.x - b.start[a], D.upd_groups, D.g, D.c, D.gd, (T*)D.map, (const float*)fr.depth,
                        (const float*)fr.rgb, D.mp, D.aux, D.nseg);
}

// ---------------------------------------------------------------------------
// descent mapping: one gradient step on the marked bricks
// ---------------------------------------------------------------------------
// Every brick on the run's list (bricks some ray of some gradient pass
// touched; count first) takes the step mean <- mean - lr (grad + (mean -
// mean0) / var) per voxel and channel, with mean0 the brick's means before the
// run's first step (copied into `save` the first time the brick is visited,
// recorded in `saved`) and var the map's variance, which descent leaves
// unchanged.  One workgroup per brick, two voxels per thread, all four
// channels.  grad is cleared behind the step, the brick summary and
// free-space bit follow the new occupancy means, and each workgroup writes its
// share of the objective at the means before the step: of the previous-belief
// term 1/2 sum (mean - mean0)^2 / var, and of the gradient pass's data partials
// (pd[nd]).  Bricks off the list have zero gradient and means equal to mean0:
// the step leaves them as they are.
//
// The dilated bits stay good for the run's next pass without a launch over
// them: a brick that turns occupied clears the bits of the blocks it lies in,
// one that turns free leaves them (not proven free, which only skips less)
// until the run's end, where the whole bitmap is formed again.  (10 steps at
// 256^3, 320x240: 57 -> 47 us a step without the launch and its wait.)
__global__ __launch_bounds__(256) void k_gd_update(GridC g, float* __restrict__ map, MapAux aux,
                                                   float* __restrict__ save, double* __restrict__ grad,
                                                   const int* __restrict__ list, unsigned* __restrict__ saved,
                                                   double lr_occ, double lr_rgb, const double* __restrict__ pd, int nd,
                                                   double* __restrict__ partials) {
    __shared__ double wsum[4];
    __shared__ float wmax[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int count = list[0];
    double cost = 0.0;
    for (int e = blockIdx.x + gridDim.x * threadIdx.x; e < nd; e += 256 * gridDim.x) cost += pd[e];
    for (int e = blockIdx.x; e < count; e += gridDim.x) {
        const int b = list[1 + e];
        const bool first = !((saved[b >> 5] >> (b & 31)) & 1u);
        float mu[4][2], mu0[4][2], var[4][2];
        double gr[4][2];
        const long long id0 = ((long long)b << 9) | threadIdx.x;
#pragma unroll
        for (int ch = 0; ch < 4; ++ch)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const long long e2 = (long long)ch * g.nvox + id0 + 256 * h;
                mu[ch][h] = map[e2];
                var[ch][h] = map[(long long)(4 + ch) * g.nvox + id0 + 256 * h];
                gr[ch][h] = grad[e2];
                if (!first) mu0[ch][h] = save[e2];
            }
        float m = -INFINITY;
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) {
            const double lr = ch ? lr_rgb : lr_occ;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const long long e2 = (long long)ch * g.nvox + id0 + 256 * h;
                if (first) {
                    save[e2] = mu[ch][h];
                    mu0[ch][h] = mu[ch][h];
                }
                const double lam = 1.0 / (double)var[ch][h];
                const double diff = (double)mu[ch][h] - (double)mu0[ch][h];
                cost += 0.5 * lam * diff * diff;
                const float nm = (float)((double)mu[ch][h] - lr * (gr[ch][h] + lam * diff));
                map[e2] = nm;
                grad[e2] = 0.0;
                if (ch == 0) m = fmaxf(m, nm);
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
        if (lane == 0) wmax[wv] = m;
        __syncthreads();   // every thread has read `saved` and its values
        if (threadIdx.x == 0) {
            const float mb = fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]));
            bool was_free = aux.bmax[b] <= 0.0f, now_free = mb <= 0.0f;
            aux.bmax[b] = mb;
            if (was_free != now_free) atomicXor(&aux.bits[b >> 5], 1u << (b & 31));
            if (was_free && !now_free)
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int t = b - (q & 1) - ((q & 2) ? g.nb : 0) - ((q & 4) ? g.nb * g.nb : 0);
                    if (t >= 0) atomicAnd(&aux.bits[free_words(g.nb) + (t >> 5)], ~(1u << (t & 31)));
                }
            if (first) atomicOr(&saved[b >> 5], 1u << (b & 31));
        }
        __syncthreads();   // wmax is reused by the next brick
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cost += __shfl_xor(cost, off, 64);
    if (lane == 0) wsum[wv] = cost;
    __syncthreads();
    if (threadIdx.x == 0) partials[blockIdx.x] = (wsum[0] + wsum[1]) + (wsum[2] + wsum[3]);
}

// The dilated bits after a run's last step, with workgroup 0 also totalling
// the objective before that step.
__global__ __launch_bounds__(256) void k_dilate_bits_cost(int nb, unsigned* __restrict__ bits,
                                                          const double* __restrict__ pp, int np,
                                                          double* __restrict__ cost) {
    __shared__ double part[4];
    if (blockIdx.x > 0)
        dilate_block(blockIdx.x - 1, nb, bits);
    else
        gd_cost_block(pp, np, cost, part);
}

__global__ __launch_bounds__(256) void k_clear_words(unsigned* __restrict__ w, int n) {
    int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) w[i] = 0u;
}

int gd_update_groups(const GridC& g) {
    int nbricks = g.nb * g.nb * g.nb;
    return nbricks < kUpdateGrid ? nbricks : kUpdateGrid;
}

hipError_t launch_gd_clear(unsigned* words, int n, hipStream_t st) {
    k_clear_words<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(words, n);
    return hipGetLastError();
}

hipError_t launch_gd_update(const GridC& g, float* map, const MapAux& aux, float* save, double* grad,
                            const int* list, unsigned* saved, double lr_occ, double lr_rgb, const double* pd, int nd,
                            double* partials, hipStream_t st) {
    k_gd_update<<<gd_update_groups(g), 256, 0, st>>>(g, map, aux, save, grad, list, saved, lr_occ, lr_rgb, pd, nd,
                                                     partials);
    return hipGetLastError();
}

hipError_t launch_gd_end(const GridC& g, const MapAux& aux, const double* pp, double* cost, hipStream_t st) {
    if (!cost) return launch_dilate(g, aux, st);
    k_dilate_bits_cost<<<(unsigned)((free_words(g.nb) + 255) / 256) + 1, 256, 0, st>>>(g.nb, aux.bits, pp,
                                                                                      gd_update_groups(g), cost);
    return hipGetLastError();
}

static unsigned blocks_for(long long n) { return (unsigned)((n + 255) / 256); }

hipError_t launch_dilate(const GridC& g, const MapAux& aux, hipStream_t st) {
    k_dilate_bits<<<(unsigned)((free_words(g.nb) + 255) / 256), 256, 0, st>>>(g.nb, aux.bits);
    return hipGetLastError();
}

static hipError_t launch_pack(const GridC& g, const MapAux& aux, hipStream_t st) {
    int nbricks = g.nb * g.nb * g.nb;
    int nwords = (nbricks + 31) >> 5;
    k_pack_bits<<<(unsigned)((nwords + 255) / 256), 256, 0, st>>>(nbricks, aux);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_dilate(g, aux, st);
}


hipError_t launch_map_init(const GridC& g, int dtype, void* map, float occ0, float rgb0, float var0,
                           const MapAux& aux, hipStream_t st) {
    int nbricks = g.nb * g.nb * g.nb;
    if (aux.table) {
        k_pool_init<<<(unsigned)((nbricks + 255) / 256), 256, 0, st>>>(nbricks, g.pocc, var0, aux);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_pack(g, aux, st);
    }
    if (dtype == PRISM_BF16)
        k_map_init<uint16_t><<<blocks_for(g.nvox), 256, 0, st>>>(g.nvox, (uint16_t*)map, occ0, rgb0, var0, aux,
                                                                 nbricks);
    else
        k_map_init<float><<<blocks_for(g.nvox), 256, 0, st>>>(g.nvox, (float*)map, occ0, rgb0, var0, aux, nbricks);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_pack(g, aux, st);
}

hipError_t launch_brick_max(const GridC& g, int dtype, const void* map, const MapAux& aux, hipStream_t st) {
    const int nbricks = g.nb * g.nb * g.nb;
    const unsigned nw = (unsigned)free_words(g.nb);
    const uint16_t* mh = (const uint16_t*)map;
    const float* mf = (const float*)map;
    if (dtype == PRISM_BF16 && g.table)
        k_brick_summary<uint16_t, true><<<nw, 256, 0, st>>>(g, mh, aux, nbricks);
    else if (dtype == PRISM_BF16)
        k_brick_summary<uint16_t, false><<<nw, 256, 0, st>>>(g, mh, aux, nbricks);
    else if (g.table)
        k_brick_summary<float, true><<<nw, 256, 0, st>>>(g, mf, aux, nbricks);
    else
        k_brick_summary<float, false><<<nw, 256, 0, st>>>(g, mf, aux, nbricks);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_dilate(g, aux, st);
}

hipError_t launch_from_dense(const GridC& g, int dtype, void* map, const float* mean4, const float* var4,
                             const MapAux& aux, hipStream_t st) {
    const unsigned blocks = (unsigned)((g.nb + 3) / 4 * g.nb * g.nb);
    if (dtype == PRISM_BF16)
        k_from_dense<uint16_t><<<blocks, 256, 0, st>>>(g.n, g.nb, (uint16_t*)map, mean4, var4, aux.bmax);
    else
        k_from_dense<float><<<blocks, 256, 0, st>>>(g.n, g.nb, (float*)map, mean4, var4, aux.bmax);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    // without means the summary is that of the means the map holds
    return mean4 ? launch_pack(g, aux, st) : launch_brick_max(g, dtype, map, aux, st);
}

hipError_t launch_to_dense(const GridC& g, int dtype, const void* map, float* mean4, float* var4,
                           const MapAux& aux, hipStream_t st) {
    const unsigned blocks = slice_blocks(g.n);
    const uint16_t* mh = (const uint16_t*)map;
    const float* mf = (const float*)map;
    if (dtype == PRISM_BF16 && g.table)
        k_to_dense<uint16_t, true><<<blocks, 256, 0, st>>>(g, mh, aux, mean4, var4);
    else if (dtype == PRISM_BF16)
        k_to_dense<uint16_t, false><<<blocks, 256, 0, st>>>(g, mh, aux, mean4, var4);
    else if (g.table)
        k_to_dense<float, true><<<blocks, 256, 0, st>>>(g, mf, aux, mean4, var4);
    else
        k_to_dense<float, false><<<blocks, 256, 0, st>>>(g, mf, aux, mean4, var4);
    return hipGetLastError();
}

hipError_t launch_planes(int n, int channels, const float* src, float* dst, int to_dense, hipStream_t st) {
    if (to_dense)
        k_planes<true><<<slice_blocks(n), 256, 0, st>>>(n, n / 8, channels, src, dst);
    else
        k_planes<false><<<slice_blocks(n), 256, 0, st>>>(n, n / 8, channels, src, dst);
    return hipGetLastError();
}

// workgroups of the update kernel, sized to the work: a view frustum holds 12
// to 19 % of a room's bricks (four views of a 256^3 map: 4043-6240 of 32768),
// and a workgroup walks four bricks at a time, so nb^3 / 32 workgroups give each
// wavefront one or two (every workgroup first scans the segment lengths, a
// fixed cost that many idle workgroups would multiply); at least 64 (or every
// brick), at most kUpdateGrid
static int update_grid(const GridC& g) {
    int nbricks = g.nb * g.nb * g.nb;
    int ng = nbricks / 32;
    if (ng < 64) ng = nbricks < 64 ? nbricks : 64;
    return ng < kUpdateGrid ? ng : kUpdateGrid;
}

hipError_t launch_map_update(const GridC& g, const CamC& c, const GridD& gd, int dtype, void* map,
                             const prism_pose* pose, const float* depth, const float* rgb, double trunc, double lam_u,
                             const MapAux& aux, int64_t* n_updated, hipStream_t st, hipEvent_t t_begin,
                             hipEvent_t t_end) {
    int nbricks = g.nb * g.nb * g.nb;
    int nseg = (nbricks + 255) / 256;
    k_cull<<<nseg, 256, 0, st>>>(g, c, pose, aux);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    MapUpdC mp{(float)trunc, trunc, lam_u};
    int ng = update_grid(g);
    size_t lds = (size_t)(nseg + 1) * sizeof(int);
    if (t_begin && (e = hipEventRecord(t_begin, st)) != hipSuccess) return e;
    const bool pool = aux.table != nullptr;
    if (dtype == PRISM_BF16 && pool)
        k_map_update<uint16_t, true><<<ng, 256, lds, st>>>(g, c, gd, (uint16_t*)map, depth, rgb, mp, aux, nseg);
    else if (dtype == PRISM_BF16)
        k_map_update<uint16_t, false><<<ng, 256, lds, st>>>(g, c, gd, (uint16_t*)map, depth, rgb, mp, aux, nseg);
    else if (pool)
        k_map_update<float, true><<<ng, 256, lds, st>>>(g, c, gd, (float*)map, depth, rgb, mp, aux, nseg);
    else
        k_map_update<float, false><<<ng, 256, lds, st>>>(g, c, gd, (float*)map, depth, rgb, mp, aux, nseg);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (!n_updated) {
        if ((e = launch_dilate(g, aux, st)) != hipSuccess) return e;
        return t_end ? hipEventRecord(t_end, st) : hipSuccess;
    }
    k_dilate_bits_sum<<<(unsigned)((free_words(g.nb) + 255) / 256), 256, 0, st>>>(g.nb, aux.bits, aux.counts, ng,
                                                                                 n_updated);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return t_end ? hipEventRecord(t_end, st) : hipSuccess;
}

int map_update_groups(const GridC& g) { return update_grid(g); }

// A batched update launches the workgroups of every filter of the batch
// together, which fills the GPU with fewer per map: half of a lone map's
// grid (each wavefront walks about two bricks; on the 16-stream mix 198
// against 203 us per launch, while a lone 256^3 map's update takes 43
// against 40 us with half its grid)
int map_update_groups_batch(const GridC& g) {
    const int nbricks = g.nb * g.nb * g.nb;
    const int ng = update_grid(g) / 2;
    return ng >= 64 ? ng : (nbricks < 64 ? nbricks : 64);
}

hipError_t launch_cull_batch(const BatchArgs& b, hipStream_t st) {
    k_cull_batch<<<b.start[b.n], 256, 0, st>>>(b);
    return hipGetLastError();
}

hipError_t launch_dilate_batch(const BatchArgs& b, hipStream_t st) {
    k_dilate_bits_batch<<<b.start[b.n], 256, 0, st>>>(b);
    return hipGetLastError();
}

hipError_t launch_map_update_batch(const BatchArgs& b, int dtype, bool pool, int max_nseg, hipStream_t st) {
    size_t lds = (size_t)(max_nseg + 1) * sizeof(int);
    if (dtype == PRISM_BF16 && pool)
        k_map_update_batch<uint16_t, true><<<b.start[b.n], 256, lds, st>>>(b);
    else if (dtype == PRISM_BF16)
        k_map_update_batch<uint16_t, false><<<b.start[b.n], 256, lds, st>>>(b);
    else if (pool)
        k_map_update_batch<float, true><<<b.start[b.n], 256, lds, st>>>(b);
    else
        k_map_update_batch<float, false><<<b.start[b.n], 256, lds, st>>>(b);
    return hipGetLastError();
}

}  // namespace prism
