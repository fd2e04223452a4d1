// Prediction-to-observation tracking objective (App. E.3): point-to-plane
// against the nearest anchor pixel and photometric error against the
// bilinearly interpolated anchor colour, with the fused reduction of the
// gated, weighted normal equations.  One observed pixel per lane, pixels in
// row-major order so observation reads are coalesced; anchor reads are
// gathers around the reprojected location.  (Two or four pixels per lane,
// paying the 29-sum reduction once for them, measured slower: the running
// sums stay live across a pixel's work, which takes 100-170 VGPRs and halves
// the waves per SIMD.)
#include "common.hpp"
#include "launch.hpp"
#include "se3.hpp"

namespace prism {

// three floats at a 4-byte aligned address, one load
typedef float float3u __attribute__((ext_vector_type(3), aligned(4)));

// column and row of pixel p (< 2^26): the quotient by a single-precision
// reciprocal is off by at most one (rows are below 2^13) and is corrected; a
// division by a run-time width takes about three times the instructions
__device__ __forceinline__ void pixel_uv(int W, int p, int& u, int& v) {
    v = (int)((float)p * __builtin_amdgcn_rcpf((float)W));
    u = p - v * W;
    const int under = u < 0 ? 1 : 0, over = u >= W ? 1 : 0;
    u += (under - over) * W;
    v += over - under;
}

// anchor values at a pixel's two associations
struct AnchorTaps {
    float depth, n[3];     // nearest pixel
    float rgb[4][3];       // bilinear corners (0,0), (1,0), (0,1), (1,1)
};

// the bilinear corners from pixel q00, dx to the right and dy below, in elements
__device__ __forceinline__ void load_corners(const float* __restrict__ a_rgb, int q00, int dx, int dy,
                                             AnchorTaps& t) {
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const float3u v = *reinterpret_cast<const float3u*>(a_rgb + 3 * (q00 + r * dy + s * dx));
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) t.rgb[2 * r + s][ch] = v[ch];
        }
}

// Associations of an observed pixel in the fixed single-precision recipe:
// nearest anchor pixel q (geo) and bilinear base pixel q00 = biy W + bix (pho);
// without an association the indices are 0.
struct Assoc {
    bool geo, pho;
    int giu, giv, bix, biy, q, q00;
};

__device__ __forceinline__ Assoc p2_assoc(const CamC& c, const Rel32& rel, int u, int v, float D) {
    Assoc o{false, false, 0, 0, 0, 0, 0, 0};
    float rx = ((float)u + 0.5f - c.cx) * c.ifx;
    float ry = ((float)v + 0.5f - c.cy) * c.ify;
    float X[3] = {D * rx, D * ry, D};
    float Y[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) Y[a] = ((rel.R[a][0] * X[0] + rel.R[a][1] * X[1]) + rel.R[a][2] * X[2]) + rel.t[a];
    if (depth_ok(D) && Y[2] > 0.0f) {
        const float uu = c.fx * (Y[0] / Y[2]) + c.cx, vv = c.fy * (Y[1] / Y[2]) + c.cy;
        if (uu >= 0.0f && uu < (float)c.W && vv >= 0.0f && vv < (float)c.H) {
            o.giu = (int)uu;
            o.giv = (int)vv;
            o.geo = true;
        }
        const float bx = uu - 0.5f, by = vv - 0.5f;
        if (bx >= 0.0f && bx < (float)(c.W - 1) && by >= 0.0f && by < (float)(c.H - 1)) {
            o.bix = (int)bx;
            o.biy = (int)by;
            o.pho = true;
        }
    }
    o.q = o.giv * c.W + o.giu;
    o.q00 = o.biy * c.W + o.bix;
    return o;
}

// The value path may fuse multiplies and adds: the pixel decisions stay in the
// fixed single-precision recipe; the residual gates compare double-precision
// values, which differ from the oracle's by rounding either way.

// back-projected point in the anchor camera (double precision) and its
// derivative w.r.t. the pose perturbation (single precision)
struct Moved {
    double Y[3];
    float dY[3][6];
};

__device__ __forceinline__ Moved p2_moved(const CamD& cd, const Rel32& rel, int u, int v, float D) {
#pragma clang fp contract(fast)
    Moved o;
    const Pose64& Pc = rel.cur;
    const Pose64& Pp = rel.prev;
    double rc[3], Xd[3], RXd[3], dW[3];
    pixel_dir64(cd, u, v, rc);
#pragma unroll
    for (int a = 0; a < 3; ++a) Xd[a] = (double)D * rc[a];
#pragma unroll
    for (int a = 0; a < 3; ++a) RXd[a] = Pc.R[a][0] * Xd[0] + Pc.R[a][1] * Xd[1] + Pc.R[a][2] * Xd[2];
#pragma unroll
    for (int a = 0; a < 3; ++a) dW[a] = RXd[a] + Pc.t[a] - Pp.t[a];
#pragma unroll
    for (int a = 0; a < 3; ++a) o.Y[a] = Pp.R[0][a] * dW[0] + Pp.R[1][a] * dW[1] + Pp.R[2][a] * dW[2];
    // dY/ddelta = Rp^T [I | -[R X]x]
    float RX[3] = {(float)RXd[0], (float)RXd[1], (float)RXd[2]};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        float e0 = (float)Pp.R[0][a], e1 = (float)Pp.R[1][a], e2 = (float)Pp.R[2][a];
        o.dY[a][0] = e0;
        o.dY[a][1] = e1;
        o.dY[a][2] = e2;
        o.dY[a][3] = fmaf(RX[1], e2, -RX[2] * e1);
        o.dY[a][4] = fmaf(RX[2], e0, -RX[0] * e2);
        o.dY[a][5] = fmaf(RX[0], e1, -RX[1] * e0);
    }
    return o;
}

// geometric row: point-to-plane against the nearest anchor pixel
__device__ __forceinline__ void p2_geo_row(const CamD& cd, const Moved& m, const Assoc& as, const AnchorTaps& tap,
                                           float J[6], double& r) {
#pragma clang fp contract(fast)
    double ra[3];
    pixel_dir64(cd, as.giu, as.giv, ra);
    double da = (double)tap.depth;
    double n0 = tap.n[0], n1 = tap.n[1], n2 = tap.n[2];
    r = n0 * (da * ra[0] - m.Y[0]) + n1 * (da * ra[1] - m.Y[1]) + n2 * (da * ra[2] - m.Y[2]);
    float fn0 = (float)n0, fn1 = (float)n1, fn2 = (float)n2;
#pragma unroll
    for (int q = 0; q < 6; ++q) J[q] = -fmaf(fn2, m.dY[2][q], fmaf(fn1, m.dY[1][q], fn0 * m.dY[0][q]));
}

// colour rows: bilinear anchor colour minus the observation; returns
// |r_r| + |r_g| + |r_b|
__device__ __forceinline__ double p2_colour_rows(const CamC& c, const CamD& cd, const Moved& m, const Assoc& as,
                                                 const AnchorTaps& tap, const float orgb[3], float J[3][6],
                                                 double r[3]) {
#pragma clang fp contract(fast)
    const double izd = 1.0 / m.Y[2];
    double ud = cd.fx * m.Y[0] * izd + cd.cx;
    double vd = cd.fy * m.Y[1] * izd + cd.cy;
    double ax = (ud - 0.5) - (double)as.bix, ay = (vd - 0.5) - (double)as.biy;
    float Y2 = (float)m.Y[2];
    float iz = 1.0f / Y2;
    float du_[3] = {c.fx * iz, 0.0f, -c.fx * (float)m.Y[0] * iz * iz};
    float dv_[3] = {0.0f, c.fy * iz, -c.fy * (float)m.Y[1] * iz * iz};
    float dum[6], dvm[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        dum[q] = fmaf(du_[2], m.dY[2][q], du_[0] * m.dY[0][q]);
        dvm[q] = fmaf(dv_[2], m.dY[2][q], dv_[1] * m.dY[1][q]);
    }
    double l1 = 0.0;
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) {
        double I00 = tap.rgb[0][ch], I10 = tap.rgb[1][ch], I01 = tap.rgb[2][ch], I11 = tap.rgb[3][ch];
        // bilinear value and its image gradient as linear blends (fused
        // multiply-adds; the same interpolant as the hat-weight sum, to
        // rounding): rows blended along x, then the rows along y
        const double d0 = I10 - I00, d1 = I11 - I01;
        const double t0 = __builtin_fma(ax, d0, I00), t1 = __builtin_fma(ax, d1, I01);
        double Ii = __builtin_fma(ay, t1 - t0, t0);
        float gu = (float)__builtin_fma(ay, d1 - d0, d0);
        float gv = (float)(t1 - t0);
        double rp = Ii - (double)orgb[ch];
        r[ch] = rp;
        l1 += fabs(rp);
#pragma unroll
        for (int q = 0; q < 6; ++q) J[ch][q] = fmaf(gv, dvm[q], gu * dum[q]);
    }
    return l1;
}

// Every anchor value of a pixel loaded at once, before the masks are known and
// without a branch: one memory round trip, covered by the arithmetic that does
// not need the anchor (left inside branches the compiler sinks each load into
// the one that uses it).  Pixels without an association read pixel 0.
struct EagerTaps {
    AnchorTaps tap;
    int m[6];   // mask and normal mask of the nearest pixel, masks of the corners
};

__device__ __forceinline__ EagerTaps load_taps(const CamC& c, const Assoc& as, const float* __restrict__ a_depth,
                                               const float* __restrict__ a_rgb, const uint8_t* __restrict__ a_mask,
                                               const float* __restrict__ a_normals,
                                               const uint8_t* __restrict__ a_nmask) {
    EagerTaps o;
    const int dx = as.pho ? 1 : 0, dy = as.pho ? c.W : 0;
    o.m[0] = a_mask[as.q];
    o.m[1] = a_nmask[as.q];
    o.m[2] = a_mask[as.q00];
    o.m[3] = a_mask[as.q00 + dx];
    o.m[4] = a_mask[as.q00 + dy];
    o.m[5] = a_mask[as.q00 + dy + dx];
    o.tap.depth = a_depth[as.q];
    const float3u n = *reinterpret_cast<const float3u*>(a_normals + 3 * as.q);
#pragma unroll
    for (int a = 0; a < 3; ++a) o.tap.n[a] = n[a];
    load_corners(a_rgb, as.q00, dx, dy, o.tap);
    return o;
}

// The rows of an observed pixel (column u, row v): geometric row 0 and colour
// rows 1-3, residuals in double precision, Jacobians in single precision.
// rm: bit 0 the geometric row passed its gate, bit 1 the colour rows.
// D and orgb: the pixel's observed depth and colour (loaded by the caller).
// Eager: the anchor by load_taps, for launches that leave the GPU waiting;
// otherwise masks first, then the values they admit (fewest loads and
// registers), for a GPU full of wavefronts, which is bound by issue.
template <bool Eager>
__device__ __forceinline__ void p2_pixel(const CamC& c, const CamD& cd, const Rel32& rel, int u, int v, float D,
                                         const float orgb[3], const float* __restrict__ a_depth,
                                         const float* __restrict__ a_rgb, const uint8_t* __restrict__ a_mask,
                                         const float* __restrict__ a_normals, const uint8_t* __restrict__ a_nmask,
                                         const WeightsC& wt, float J[4][6], double r[4], int& rm) {
    rm = 0;
    const Assoc as = p2_assoc(c, rel, u, v, D);
    if constexpr (Eager) {
        const EagerTaps e = load_taps(c, as, a_depth, a_rgb, a_mask, a_normals, a_nmask);
        const Moved m = p2_moved(cd, rel, u, v, D);
        p2_geo_row(cd, m, as, e.tap, J[0], r[0]);
        const double l1 = p2_colour_rows(c, cd, m, as, e.tap, orgb, J + 1, r + 1);
        const bool geo = as.geo & (e.m[0] != 0) & (e.m[1] != 0);
        const bool pho = as.pho & (e.m[2] != 0) & (e.m[3] != 0) & (e.m[4] != 0) & (e.m[5] != 0);
        if (geo && fabs(r[0]) <= wt.gate_depth) rm |= 1;
        if (pho && l1 <= wt.gate_rgb) rm |= 2;
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const bool keep = a ? pho : geo;
            r[a] = keep ? r[a] : 0.0;
#pragma unroll
            for (int q = 0; q < 6; ++q) J[a][q] = keep ? J[a][q] : 0.0f;
        }
        return;
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        r[a] = 0.0;
#pragma unroll
        for (int m = 0; m < 6; ++m) J[a][m] = 0.0f;
    }
    const bool geo = as.geo && a_mask[as.q] && a_nmask[as.q];
    const bool pho = as.pho && a_mask[as.q00] && a_mask[as.q00 + 1] && a_mask[as.q00 + c.W] && a_mask[as.q00 + c.W + 1];
    if (!(geo || pho)) return;
    const Moved m = p2_moved(cd, rel, u, v, D);
    AnchorTaps tap;
    if (geo) {
        tap.depth = a_depth[as.q];
#pragma unroll
        for (int a = 0; a < 3; ++a) tap.n[a] = a_normals[3 * as.q + a];
        p2_geo_row(cd, m, as, tap, J[0], r[0]);
        if (fabs(r[0]) <= wt.gate_depth) rm |= 1;
    }
    if (pho) {
        load_corners(a_rgb, as.q00, 1, c.W, tap);
        if (p2_colour_rows(c, cd, m, as, tap, orgb, J + 1, r + 1) <= wt.gate_rgb) rm |= 2;
    }
}

// The pixel's share of the gradient sum w r J, added to g
__device__ __forceinline__ void p2_grad(const CamC& c, const CamD& cd, const Rel32& rel, int u, int v, float D,
                                        const float orgb[3], const float* __restrict__ a_depth,
                                        const float* __restrict__ a_rgb, const uint8_t* __restrict__ a_mask,
                                        const float* __restrict__ a_normals, const uint8_t* __restrict__ a_nmask,
                                        const WeightsC& wt, double g[6]) {
    float J[4][6];
    double r[4];
    const Assoc as = p2_assoc(c, rel, u, v, D);
    const EagerTaps e = load_taps(c, as, a_depth, a_rgb, a_mask, a_normals, a_nmask);
    const Moved m = p2_moved(cd, rel, u, v, D);
    p2_geo_row(cd, m, as, e.tap, J[0], r[0]);
    const double l1 = p2_colour_rows(c, cd, m, as, e.tap, orgb, J + 1, r + 1);
    const bool geo = as.geo & (e.m[0] != 0) & (e.m[1] != 0) & (fabs(r[0]) <= wt.gate_depth);
    const bool pho = as.pho & (e.m[2] != 0) & (e.m[3] != 0) & (e.m[4] != 0) & (e.m[5] != 0) & (l1 <= wt.gate_rgb);
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const double ag = wt.w_depth * r[0] * (double)J[0][q];
        double ac = wt.w_rgb * r[1] * (double)J[1][q];
        ac += wt.w_rgb * r[2] * (double)J[2][q];
        ac += wt.w_rgb * r[3] * (double)J[3][q];
        g[q] += (geo ? ag : 0.0) + (pho ? ac : 0.0);
    }
}

// one workgroup (blk: its index within this frame's grid) of the tracking
// objective; partials receives the workgroup's 29 sums at row blk
template <bool Eager>
__device__ __forceinline__ void track_p2_block(int blk, const CamC& c, const CamD& cd,
                                               const prism_pose* __restrict__ pose,
                                               const prism_pose* __restrict__ pose_prev,
                                               const float* __restrict__ obs_depth,
                                               const float* __restrict__ obs_rgb,
                                               const float* __restrict__ a_depth,
                                               const float* __restrict__ a_rgb,
                                               const uint8_t* __restrict__ a_mask,
                                               const float* __restrict__ a_normals,
                                               const uint8_t* __restrict__ a_nmask, const WeightsC& wt,
                                               float* __restrict__ Jout, float* __restrict__ resid,
                                               uint8_t* __restrict__ rowmask, double* __restrict__ partials,
                                               const Rel32* __restrict__ grel) {
    __shared__ Rel32 srel;
    __shared__ double lds[kRedLds];
    // the filter's relative pose when it keeps one (copied word by word),
    // else formed here by thread 0
    constexpr int kRelWords = (int)(sizeof(Rel32) / 4);
    static_assert(sizeof(Rel32) % 4 == 0 && kRelWords <= 256, "Rel32 is copied by one word per thread");
    if (grel) {
        if (threadIdx.x < kRelWords)
            reinterpret_cast<unsigned*>(&srel)[threadIdx.x] = reinterpret_cast<const unsigned*>(grel)[threadIdx.x];
    } else if (threadIdx.x == 0) {
        rel_of(pose, pose_prev, srel);
    }
    __syncthreads();
    const Rel32& rel = srel;
    // this pixel's rows summed in single precision (at most 4 rows of
    // single-precision Jacobians), reduced over the workgroup by
    // block_reduce29f (single precision within 32 lanes, then double)
    float pacc[PRISM_NEQ];
#pragma unroll
    for (int q = 0; q < PRISM_NEQ; ++q) pacc[q] = 0.0f;
    int p = blk * blockDim.x + threadIdx.x;
    if (p < c.W * c.H) {
        float J[4][6];
        double r[4];
        int rm;
        int u, v;
        pixel_uv(c.W, p, u, v);
        const float orgb[3] = {obs_rgb[3 * p], obs_rgb[3 * p + 1], obs_rgb[3 * p + 2]};
        p2_pixel<Eager>(c, cd, rel, u, v, obs_depth[p], orgb, a_depth, a_rgb, a_mask, a_normals, a_nmask, wt, J, r, rm);
        if (rm & 1) neq_add32(pacc, J[0], (float)r[0], row_weight(wt, false, r[0]));
        if (rm & 2)
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) neq_add32(pacc, J[1 + ch], (float)r[1 + ch], row_weight(wt, true, r[1 + ch]));
        if (rm) pacc[28] = 1.0f;
        if (Jout) {
            float4* jo = reinterpret_cast<float4*>(Jout + 24 * (long long)p);
#pragma unroll
            for (int q = 0; q < 6; ++q)
                jo[q] = make_float4(J[(4 * q) / 6][(4 * q) % 6], J[(4 * q + 1) / 6][(4 * q + 1) % 6],
                                    J[(4 * q + 2) / 6][(4 * q + 2) % 6], J[(4 * q + 3) / 6][(4 * q + 3) % 6]);
        }
        if (resid)
            reinterpret_cast<float4*>(resid)[p] = make_float4((float)r[0], (float)r[1], (float)r[2], (float)r[3]);
        if (rowmask) rowmask[p] = (uint8_t)rm;
    }
    block_reduce29f(pacc, lds, partials + (long long)blk * PRISM_NEQ);
}

template <bool Eager>
__global__ __launch_bounds__(256) void k_track_p2(CamC c, CamD cd, const prism_pose* __restrict__ pose,
                                                  const prism_pose* __restrict__ pose_prev,
                                                  const float* __restrict__ obs_depth,
                                                  const float* __restrict__ obs_rgb,
                                                  const float* __restrict__ a_depth,
                                                  const float* __restrict__ a_rgb,
                                                  const uint8_t* __restrict__ a_mask,
                                                  const float* __restrict__ a_normals,
                                                  const uint8_t* __restrict__ a_nmask, WeightsC wt,
                                                  float* __restrict__ Jout, float* __restrict__ resid,
                                                  uint8_t* __restrict__ rowmask,
                                                  double* __restrict__ partials, const Rel32* __restrict__ rel) {
    track_p2_block<Eager>(blockIdx.x, c, cd, pose, pose_prev, obs_depth, obs_rgb, a_depth, a_rgb, a_mask, a_normals, a_nmask,
                   wt, Jout, resid, rowmask, partials, rel);
}

// batched: every filter tracks its slot's frame from its current iterate
// against its anchor
__global__ __launch_bounds__(256) void k_track_p2_batch(BatchArgs b) {
    const int a = batch_agent(b, blockIdx.x);
    const AgentDesc& D = *b.d[a];
    const prism_frame& fr = D.slots[b.slot[a]];
    track_p2_block<false>(blockIdx.x - b.start[a], D.c, D.cd, &D.S->iter, &D.S->anchor, (const float*)fr.depth,
                   (const float*)fr.rgb, D.a_depth, D.a_rgb, D.a_mask, D.a_normals, D.a_nmask, b.irls ? D.w_irls : D.w,
                   nullptr, nullptr, nullptr, D.partials, D.rel);
}

// ---------------------------------------------------------------------------
// the paper's pose optimiser: Adam without momentum on sampled pixels
// ---------------------------------------------------------------------------
// One workgroup runs the whole optimisation: at each step 256 threads
// evaluate the objective's rows on that step's sampled pixels (row-major
// indices; an index outside the image is a pixel without rows; repeated
// indices count repeatedly) at the current iterate, the gradient
//   g = scale * sum 2 w r J + Lp e,   e = pose error of the iterate w.r.t. the prior,
// is reduced in a fixed order, and the step is taken: second moment
// v <- b2 v + (1 - b2) g^2 (first moment off: the step follows g itself),
// bias-corrected vhat = v / (1 - b2^k), delta = -lr g / (sqrt(vhat) + eps),
// iterate <- retract(iterate, delta).  scale = image pixels / sampled pixels
// makes each step's data term an unbiased estimate of the full-image sum.
//
// The steps are one dependent chain, so a step's latency is all that counts:
//  * a fifth wavefront forms the prior term Lp e while four evaluate pixels
//    (on one of their lanes it came after its pixel, in series);
//  * a pixel's anchor values are loaded at once and covered by the arithmetic
//    that does not need them; the next step's observations and the indices of
//    the step after it are requested once they have arrived;
//  * the six sums are reduced in registers, and every wavefront takes the
//    step redundantly on its own copy of the iterate (a rotation matrix,
//    converted back to a quaternion once, at the end), so a step has one
//    workgroup barrier and nothing is handed out through memory after it.
// 1000 steps of 200 pixels on a 320x240 frame: 5.6 -> 2.5 ms.  With the clock
// read between its parts, which lengthens a step to 6350 clocks, the pixel's
// chain takes 4100, the sums 720, the barrier 280 and the step 1250.  (Fetching
// the samples in the prior's wavefront took 3.1 ms: it then ends last.)
// Skipped when the prediction already fell back (improper prior).
constexpr int kAdamThreads = 320;   // four wavefronts of pixels, one for the prior

__device__ __forceinline__ double lane_value(double x, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                            __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// More: steps of more than 256 pixels
template <bool More>
__global__ __launch_bounds__(kAdamThreads) void k_pose_adam(
    prism_filter_state* __restrict__ S, CamC c, CamD cd, const float* __restrict__ obs_depth,
    const float* __restrict__ obs_rgb, const float* __restrict__ a_depth, const float* __restrict__ a_rgb,
    const uint8_t* __restrict__ a_mask, const float* __restrict__ a_normals, const uint8_t* __restrict__ a_nmask,
    WeightsC wt, const int32_t* __restrict__ pixels, AdamC ad) {
    __shared__ Rel32 srel;
    __shared__ double red[2][4][6], lpe[2][6];   // of even and odd steps
    __shared__ double sRp[9], stp[3];
    __shared__ int skip;
    if (threadIdx.x == 0) {
        const prism_pose it = S->iter, pr = S->prior, an = S->anchor;
        skip = (S->flags & PRISM_FLAG_CHOL_FALLBACK) != 0;
        rel_of(&it, &an, srel);
        quat_to_R9(pr.q, sRp);
        for (int i = 0; i < 3; ++i) stp[i] = pr.t[i];
    }
    __syncthreads();
    if (skip) return;
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int npix = c.W * c.H;
    Rel32 rel = srel;   // cur: the iterate (double R, t); prev: the anchor pose
    double Lrow[6];     // prior wavefront: row `lane` of Lp
#pragma unroll
    for (int k = 0; k < 6; ++k) Lrow[k] = S->Lp[(lane < 6 ? lane : 0) * 6 + k];
    double lr = ad.lr[lane < 6 ? lane : 0];
    // arrived before the loop: a wait for them inside it would also wait for
    // the loads a step requests ahead
    asm volatile("" : "+v"(lr), "+v"(Lrow[0]), "+v"(Lrow[1]), "+v"(Lrow[2]), "+v"(Lrow[3]), "+v"(Lrow[4]), "+v"(Lrow[5]));
    double v2 = 0.0, b2k = 1.0;   // second moment of component `lane`
    // The thread's first sampled pixel of a step: its index is requested two
    // steps ahead, its observation one step ahead (neither depends on the
    // pose).  Even and odd steps hold theirs in registers of their own: handed
    // on by copies, the values would be waited for when they are copied.
    struct Sample {
        int at;          // (row << 16 | column), or -1 for a pixel without rows
        float D, rgb[3];
    } sa, sb;
    int ia = 0, ib = 0;
    auto index_at = [&](int step, int j) {   // (a step or pixel past the last reads the last)
        return pixels[(long long)min(step, ad.n_steps - 1) * ad.n_pix + min(j, ad.n_pix - 1)];
    };
    auto observe = [&](int p, int j, Sample& o) {   // (no pixel: reads pixel 0)
        const bool any = j < ad.n_pix && (unsigned)p < (unsigned)npix;
        p = any ? p : 0;
        o.D = obs_depth[p];
        const float3u x = *reinterpret_cast<const float3u*>(obs_rgb + 3 * p);
        o.rgb[0] = x[0];
        o.rgb[1] = x[1];
        o.rgb[2] = x[2];
        int u, v;
        pixel_uv(c.W, p, u, v);
        o.at = any ? (v << 16) | u : -1;
    };
    if (wv < 4) {
        ia = index_at(0, threadIdx.x);
        ib = index_at(1, threadIdx.x);
        observe(ia, threadIdx.x, sa);
        // ahead of the prior wavefront, which shares a SIMD with one of these
        __builtin_amdgcn_s_setprio(2);
    }
    // step `step`: the sample in `cur`; `inext`, the index of the next step's
    // sample, becomes `next`, and the index of the step after it `iafter`
    auto do_step = [&](int step, int buf, const Sample& cur, Sample& next, const int& inext, int& iafter) {
        if (wv < 4) {
            double g[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
            if (cur.at >= 0)
                p2_grad(c, cd, rel, cur.at & 0xffff, cur.at >> 16, cur.D, cur.rgb, a_depth, a_rgb, a_mask, a_normals,
                        a_nmask, wt, g);
            if constexpr (More)
                for (int j = threadIdx.x + 256; j < ad.n_pix; j += 256) {
                    Sample o;
                    observe(index_at(step, j), j, o);
                    if (o.at >= 0)
                        p2_grad(c, cd, rel, o.at & 0xffff, o.at >> 16, o.D, o.rgb, a_depth, a_rgb, a_mask, a_normals,
                                a_nmask, wt, g);
                }
            // requested only now: a wait for the anchor covers all earlier loads
            __builtin_amdgcn_sched_barrier(0);
            observe(inext, threadIdx.x, next);
            iafter = index_at(step + 2, threadIdx.x);
            double s[3];
            wave_sum6(g, s);
            if ((lane & 31) == 0)
#pragma unroll
                for (int j = 0; j < 3; ++j) red[buf][wv][(lane >> 5) * 3 + j] = s[j];
        } else {
            // prior term at the current iterate: e = (t - tp, Log(R Rp^T))
            double M[9], e[6];
            for (int i = 0; i < 3; ++i)
                for (int k = 0; k < 3; ++k)
                    M[i * 3 + k] = rel.cur.R[i][0] * sRp[k * 3] + rel.cur.R[i][1] * sRp[k * 3 + 1] +
                                   rel.cur.R[i][2] * sRp[k * 3 + 2];
            for (int i = 0; i < 3; ++i) e[i] = rel.cur.t[i] - stp[i];
            so3_log(M, e + 3);
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < 6; ++k) s += Lrow[k] * e[k];
            if (lane < 6) lpe[buf][lane] = s;
        }
        // formed ahead of the barrier
        b2k *= ad.beta2;
        const double corr = 1.0 / (1.0 - b2k);
        __syncthreads();
        {
#pragma clang fp contract(fast)
            const int m6 = lane < 6 ? lane : 0;
            const double gi = 2.0 * ad.scale * ((red[buf][0][m6] + red[buf][1][m6]) +
                                                (red[buf][2][m6] + red[buf][3][m6])) + lpe[buf][m6];
            v2 = ad.beta2 * v2 + (1.0 - ad.beta2) * gi * gi;
            const double di = -lr * gi / (sqrt(v2 * corr) + ad.eps);
            double d[6], E[9], R2[3][3];
#pragma unroll
            for (int m = 0; m < 6; ++m) d[m] = lane_value(di, m);
            so3_exp_step(d + 3, E);
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    R2[i][k] = E[i * 3] * rel.cur.R[0][k] + E[i * 3 + 1] * rel.cur.R[1][k] + E[i * 3 + 2] * rel.cur.R[2][k];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                rel.cur.t[i] += d[i];
#pragma unroll
                for (int k = 0; k < 3; ++k) rel.cur.R[i][k] = R2[i][k];
            }
        }
        // outside the contracted block: the samples' pixels are decided with
        // it (the prior needs the iterate only)
        if (wv < 4) rel_of(rel.cur, rel.prev, rel);
    };
    for (int step = 0; step < ad.n_steps; step += 2) {
        do_step(step, 0, sa, sb, ib, ia);
        if (step + 1 == ad.n_steps) break;
        do_step(step + 1, 1, sb, sa, ia, ib);
    }
    if (threadIdx.x == 0) {
        double R[9];
        for (int i = 0; i < 3; ++i)
            for (int k = 0; k < 3; ++k) R[i * 3 + k] = rel.cur.R[i][k];
        prism_pose it;
        for (int i = 0; i < 3; ++i) it.t[i] = rel.cur.t[i];
        R9_to_quat(R, it.q);
        S->iter = it;
    }
}

hipError_t launch_pose_adam(prism_filter_state* S, const CamC& c, const CamD& cd, const float* obs_depth,
                            const float* obs_rgb, const float* a_depth, const float* a_rgb, const uint8_t* a_mask,
                            const float* a_normals, const uint8_t* a_nmask, const WeightsC& w, const int32_t* pixels,
                            const AdamC& ad, hipStream_t st) {
    auto* k = ad.n_pix > 256 ? k_pose_adam<true> : k_pose_adam<false>;
    k<<<1, kAdamThreads, 0, st>>>(S, c, cd, obs_depth, obs_rgb, a_depth, a_rgb, a_mask, a_normals, a_nmask, w, pixels, ad);
    return hipGetLastError();
}

int track_blocks(const CamC& c) { return (c.W * c.H + 255) / 256; }

hipError_t launch_track_p2_batch(const BatchArgs& b, hipStream_t st) {
    k_track_p2_batch<<<b.start[b.n], 256, 0, st>>>(b);
    return hipGetLastError();
}

hipError_t launch_track_p2(const CamC& c, const CamD& cd, const prism_pose* pose, const prism_pose* pose_prev,
                           const float* obs_depth, const float* obs_rgb, const float* a_depth,
                           const float* a_rgb, const uint8_t* a_mask, const float* a_normals,
                           const uint8_t* a_nmask, const WeightsC& w, float* J, float* resid,
                           uint8_t* rowmask, double* partials, const Rel32* rel, hipStream_t st) {
    // A lone frame leaves the GPU waiting on a chain of loads (320x240: 1.2
    // wavefronts per SIMD; 7.0 us masks first, 6.0 eager; 160x120 6.5 / 5.8;
    // 640x480, 4.7 per SIMD, 9.7 / 9.45); from six wavefronts per SIMD, as many
    // as the other variant's registers admit, loads wait for their masks.
    auto* k = track_blocks(c) <= 1536 ? k_track_p2<true> : k_track_p2<false>;
    k<<<track_blocks(c), 256, 0, st>>>(c, cd, pose, pose_prev, obs_depth, obs_rgb, a_depth, a_rgb, a_mask, a_normals,
                                       a_nmask, w, J, resid, rowmask, partials, rel);
    return hipGetLastError();
}

}  // namespace prism
