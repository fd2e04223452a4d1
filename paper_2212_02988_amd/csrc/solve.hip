// FP64 state-filter algebra on the device (App. E.1-E.3, Sec. 4.3.2):
// linearised transition + propagation + split into pose prior and velocity
// conditional; Gauss-Newton step of the MAP pose objective; Laplace
// covariance (squared-Jacobian Hessian, with the dynamics prior), its EMA,
// and the product with the velocity conditional; the same over the 15-D
// state with an accelerometer bias; predictive rollouts.
//
// Each kernel is one workgroup per filter (256 threads for the prediction;
// the Gauss-Newton and Laplace kernels reduce the block partial sums of the
// normal equations in a fixed order with 512, while a ninth wavefront forms
// what does not depend on them).  What remains is a chain of dependent double-
// precision operations, so it is kept short: small factorisations run in the
// registers of one wavefront with reciprocal roots, matrix products are
// spread over the threads with only their non-zero terms, and independent
// chains run in different wavefronts.  Everything stays on the device so a
// filter step can be captured in a HIP graph.
#include "common.hpp"
#include "launch.hpp"
#include "se3.hpp"

namespace prism {

// ---------------------------------------------------------------------------
// small helpers (row-major matrices in LDS)
// ---------------------------------------------------------------------------
// C[r x c] = A[r x k] * op(B);  op(B) = B [k x c] or B^T (B stored [c x k])
__device__ inline void mm(const double* A, const double* B, double* C, int r, int k, int c, bool bT) {
    for (int e = threadIdx.x; e < r * c; e += blockDim.x) {
        int i = e / c, j = e % c;
        double s = 0.0;
        for (int q = 0; q < k; ++q) s += A[i * k + q] * (bT ? B[j * k + q] : B[q * c + j]);
        C[e] = s;
    }
    __syncthreads();
}

__device__ inline void symmetrize(double* A, int n) {
    for (int e = threadIdx.x; e < n * n; e += blockDim.x) {
        int i = e / n, j = e % n;
        if (i < j) {
            double s = 0.5 * (A[i * n + j] + A[j * n + i]);
            A[i * n + j] = s;
            A[j * n + i] = s;
        }
    }
    __syncthreads();
}

// In-place lower Cholesky of an N x N matrix (single thread); false if not
// positive definite.  Sizes are compile-time constants and every loop is
// unrolled so the matrix stays in registers.
template <int N>
__device__ inline bool chol(double* A) {
    bool ok = true;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        double s = A[j * N + j];
#pragma unroll
        for (int k = 0; k < j; ++k) s -= A[j * N + k] * A[j * N + k];
        ok = ok && (s > 0.0);
        double d;
        const double id = rsqrt64(fmax(s, 1e-300), &d);
        A[j * N + j] = d;
#pragma unroll
        for (int i = j + 1; i < N; ++i) {
            double t = A[i * N + j];
#pragma unroll
            for (int k = 0; k < j; ++k) t -= A[i * N + k] * A[j * N + k];
            A[i * N + j] = t * id;
        }
#pragma unroll
        for (int i = 0; i < j; ++i) A[i * N + j] = 0.0;
    }
    return ok;
}

// Lower Cholesky factor of an N x N matrix in the registers of every lane of a
// wavefront (A: LDS or registers, row-major), with the reciprocals of its
// diagonal: a reciprocal root serves the diagonal and its inverse.  False if
// not positive definite (the same for all lanes).
template <int N>
struct Chol {
    double L[N][N], id[N];
};
template <int N>
__device__ __forceinline__ bool chol_regs(const double* A, Chol<N>& c) {
    bool ok = true;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        double s = A[j * N + j];
#pragma unroll
        for (int k = 0; k < j; ++k) s -= c.L[j][k] * c.L[j][k];
        ok = ok && (s > 0.0);
        double d;
        const double r = rsqrt64(fmax(s, 1e-300), &d);
        c.L[j][j] = d;
        c.id[j] = r;
#pragma unroll
        for (int i = j + 1; i < N; ++i) {
            double t = A[i * N + j];
#pragma unroll
            for (int k = 0; k < j; ++k) t -= c.L[i][k] * c.L[j][k];
            c.L[i][j] = t * r;
        }
    }
    return ok;
}

// solve L L^T x = b in place
template <int N>
__device__ __forceinline__ void chol_solve(const Chol<N>& c, double b[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        double s = b[i];
#pragma unroll
        for (int k = 0; k < i; ++k) s -= c.L[i][k] * b[k];
        b[i] = s * c.id[i];
    }
#pragma unroll
    for (int i = N - 1; i >= 0; --i) {
        double s = b[i];
#pragma unroll
        for (int k = i + 1; k < N; ++k) s -= c.L[k][i] * b[k];
        b[i] = s * c.id[i];
    }
}

// inverse of a symmetric positive definite matrix, symmetrised: A -> Ainv (both
// LDS, row-major), by one wavefront, a column per lane (N * N <= 64); false if
// not positive definite
template <int N>
__device__ __forceinline__ bool spd_inverse_wave(const double* A, double* Ainv) {
    const int lane = threadIdx.x & 63;
    Chol<N> c;
    const bool ok = chol_regs<N>(A, c);
    double x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = i == lane ? 1.0 : 0.0;
    chol_solve<N>(c, x);
    wave_lds_order();   // (Ainv may be A)
    if (lane < N)
#pragma unroll
        for (int i = 0; i < N; ++i) Ainv[i * N + lane] = x[i];
    wave_lds_order();
    double s = 0.0;
    if (lane < N * N) s = 0.5 * (Ainv[lane] + Ainv[(lane % N) * N + lane / N]);
    wave_lds_order();
    if (lane < N * N) Ainv[lane] = s;
    return ok;
}

// entry (i, j) of the symmetric 6x6 matrix packed by rows of its upper triangle
__device__ __forceinline__ int sym6(int i, int j) {
    const int a = i < j ? i : j, b = i < j ? j : i;
    return a * 6 - a * (a - 1) / 2 + b - a;
}

// Fixed-order block sum of partial sums (nblocks rows of NV = 29 doubles, the
// normal equations) into lds_out[NV], by the first kSumThreads threads of
// the workgroup (the others only meet the barriers).  The rows are read as one
// flat array with coalesced loads: thread t < NV G (G = row groups) reads
// elements t, t + NV G, ... which all belong to column t mod NV; the G sums of
// each column are then added in row-group order.  (Each thread reading whole
// rows made every load instruction touch 64 cache lines, which one workgroup's
// vector memory path takes serially.)  One workgroup reads at the latency of
// its rounds, so a round is 20 loads per thread, which covers a 320x240 frame's
// 300 rows, and the next round is requested before this one is added.
// lds_red: kSumThreads doubles.
// With sg given, the filter state is copied into ls on the way: its words
// are loaded together with the first partials (not one round trip before
// them) and stored to LDS before the sum's barrier.
constexpr int kSumThreads = 512;

__device__ inline void sum_partials(const double* __restrict__ partials, int nblocks, double* lds_red,
                                    double* lds_out, const prism_filter_state* __restrict__ sg = nullptr,
                                    prism_filter_state* ls = nullptr) {
    constexpr int kStateWords = (int)(sizeof(prism_filter_state) / 8);
    static_assert(sizeof(prism_filter_state) % 8 == 0 && kStateWords <= kSumThreads, "a state word per thread");
    constexpr int NV = PRISM_NEQ, G = kSumThreads / NV, span = G * NV, kRound = 20;
    const int t = threadIdx.x;
    unsigned long long sw = 0;
    if (sg && t < kStateWords) sw = reinterpret_cast<const unsigned long long*>(sg)[t];
    if (t < span) {
        const int total = nblocks * NV;   // at most 2^20 rows of 29
        double x[kRound], a[4] = {0.0, 0.0, 0.0, 0.0};
        auto load = [&](int e0) {
#pragma unroll
            for (int u = 0; u < kRound; ++u) {
                const int e = e0 + u * span;
                x[u] = e < total ? partials[e] : 0.0;
            }
        };
        load(t);
        for (int e0 = t; e0 < total; e0 += kRound * span) {
            double y[kRound];
#pragma unroll
            for (int u = 0; u < kRound; ++u) y[u] = x[u];
            if (e0 + kRound * span < total) load(e0 + kRound * span);
#pragma unroll
            for (int u = 0; u < kRound; ++u) a[u & 3] += y[u];
        }
        lds_red[t] = (a[0] + a[1]) + (a[2] + a[3]);
    }
    if (ls && t < kStateWords) reinterpret_cast<unsigned long long*>(ls)[t] = sw;
    __syncthreads();
    if (t < NV) {
        double r[G];
#pragma unroll
        for (int k = 0; k < G; ++k) r[k] = lds_red[k * NV + t];
        double sum = 0.0;
#pragma unroll
        for (int k = 0; k < G; ++k) sum += r[k];
        lds_out[t] = sum;
    }
    __syncthreads();
}

// The state lives in global memory; each kernel copies it into LDS once
// (one parallel round trip), works on the copy and writes it back, so the
// single-thread parts never wait on dependent global loads.
__device__ inline void state_in(const prism_filter_state* g, prism_filter_state* l) {
    const unsigned long long* s = reinterpret_cast<const unsigned long long*>(g);
    unsigned long long* d = reinterpret_cast<unsigned long long*>(l);
    for (int i = threadIdx.x; i < (int)(sizeof(prism_filter_state) / 8); i += blockDim.x) d[i] = s[i];
    __syncthreads();
}

__device__ inline void state_out(const prism_filter_state* l, prism_filter_state* g) {
    __syncthreads();
    const unsigned long long* s = reinterpret_cast<const unsigned long long*>(l);
    unsigned long long* d = reinterpret_cast<unsigned long long*>(g);
    for (int i = threadIdx.x; i < (int)(sizeof(prism_filter_state) / 8); i += blockDim.x) d[i] = s[i];
}

// ---------------------------------------------------------------------------
// predict + split
// ---------------------------------------------------------------------------
// Mean of the Euler transition (App. B, E.1) of one state, on one thread:
// new velocities (vnew = v', w' = v + u du, w + u_w du with du = dt, or dt^2
// as printed), E = Exp(w' dt) with its left Jacobian Jl, and the new pose
// (t + v' dt, E R).
__device__ inline void transition_mean_t0(const prism_pose& pose, const double* v0, const double* w0,
                                          const double* u, const TransC& tc, double* vnew, double* E, double* Jl,
                                          prism_pose& pr) {
    double v[3], w[3];
    for (int i = 0; i < 3; ++i) {
        v[i] = v0[i] + u[i] * tc.du;
        w[i] = w0[i] + u[3 + i] * tc.du;
        vnew[i] = v[i];
        vnew[3 + i] = w[i];
    }
    double phi[3] = {w[0] * tc.dt, w[1] * tc.dt, w[2] * tc.dt};
    double Ex[9], Jx[9], R[9], R2[9];
    so3_exp(phi, Ex, Jx);
    for (int e = 0; e < 9; ++e) { E[e] = Ex[e]; Jl[e] = Jx[e]; }
    quat_to_R9(pose.q, R);
    mat3mul(Ex, R, R2);
    for (int i = 0; i < 3; ++i) pr.t[i] = pose.t[i] + v[i] * tc.dt;
    R9_to_quat(R2, pr.q);
}

// Covariance of the linearised transition (App. E.2), whole workgroup:
// T2 = M P M^T + G Q G^T (symmetrised) in the error state (dt, dtheta, dv,
// dw), with E, Jl from transition_mean_t0; P, T1, T2: LDS [144].  M and G are
// mostly zeros and ones:
//   M = [I 0 dt I 0; 0 E 0 dt Jl; 0 0 I 0; 0 0 0 I],  G = M with E = I,
// so only their non-zero terms are summed, in the order of the full product.
__device__ __forceinline__ double cov_row(const double* E, const double* Jl, double dt, int i, const double* col,
                                          int step) {
    if (i < 3) return col[i * step] + dt * col[(6 + i) * step];
    if (i >= 6) return col[i * step];
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < 3; ++q) s += E[(i - 3) * 3 + q] * col[(3 + q) * step];
#pragma unroll
    for (int q = 0; q < 3; ++q) s += dt * Jl[(i - 3) * 3 + q] * col[(9 + q) * step];
    return s;
}
__device__ __forceinline__ double cov_noise(const double* Jl, const TransC& tc, int i, int j) {
    if (i > j) {
        const int k = i;
        i = j;
        j = k;
    }
    if (i < 3) return j == i ? tc.q[i] + tc.dt * tc.q[6 + i] * tc.dt : j == 6 + i ? tc.dt * tc.q[6 + i] : 0.0;
    if (i >= 6) return i == j ? tc.q[i] : 0.0;
    if (j >= 9) return tc.dt * Jl[(i - 3) * 3 + j - 9] * tc.q[j];
    if (j >= 6) return 0.0;
    double s = i == j ? tc.q[i] : 0.0;
#pragma unroll
    for (int q = 0; q < 3; ++q) s += tc.dt * Jl[(i - 3) * 3 + q] * tc.q[9 + q] * (tc.dt * Jl[(j - 3) * 3 + q]);
    return s;
}
__device__ inline void transition_cov(const double* E, const double* Jl, const TransC& tc, const double* P,
                                      double* T1, double* T2) {
    for (int e = threadIdx.x; e < 144; e += blockDim.x) T1[e] = cov_row(E, Jl, tc.dt, e / 12, P + e % 12, 12);   // M P
    __syncthreads();
    for (int e = threadIdx.x; e < 144; e += blockDim.x) {
        const int i = e / 12, j = e % 12;
        if (i > j) continue;
        const double q = cov_noise(Jl, tc, i, j);
        const double a = cov_row(E, Jl, tc.dt, j, T1 + i * 12, 1) + q;
        const double b = cov_row(E, Jl, tc.dt, i, T1 + j * 12, 1) + q;
        const double s = i == j ? a : 0.5 * (a + b);
        T2[i * 12 + j] = s;
        T2[j * 12 + i] = s;
    }
    __syncthreads();
}

// put(i, j) = D + sign X W^T, symmetrised, its pairs spread over the threads
// (X [n x 6]; W(j, q) and D(i, j) read an entry)
template <typename GetW, typename GetD, typename Put>
__device__ __forceinline__ void sym_plus_outer(int n, double sign, const double* X, const GetW& W, const GetD& D,
                                               const Put& put) {
    for (int e = threadIdx.x; e < n * n; e += blockDim.x) {
        const int i = e / n, j = e % n;
        if (i > j) continue;
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            a += X[i * 6 + q] * W(j, q);
            b += X[j * 6 + q] * W(i, q);
        }
        a = D(i, j) + sign * a;
        b = D(j, i) + sign * b;
        const double s = i == j ? a : 0.5 * (a + b);
        put(i, j, s);
        put(j, i, s);
    }
}

// 9.2 -> 6.0 us: the rotation's exponential comes first, and the new pose (its
// quaternion and its relation to the anchor) is formed in the second wavefront
// while the first inverts the pose block.
__device__ __forceinline__ void predict_block(prism_filter_state* __restrict__ Sg, const double* __restrict__ u,
                                              const TransC& tc, Rel32* __restrict__ rel) {
    __shared__ double T1[144], T2[144], Spp[36], Sinv[36], D[36];
    __shared__ double vnew[6], E[9], Jl[9];
    __shared__ int ok;
    __shared__ prism_filter_state Ls;
    state_in(Sg, &Ls);
    prism_filter_state* S = &Ls;
    const int wv = threadIdx.x >> 6;
    if (wv == 0) {
        double vn[6], Ex[9], Jx[9];
        for (int i = 0; i < 3; ++i) {
            vn[i] = S->v[i] + u[i] * tc.du;
            vn[3 + i] = S->w[i] + u[3 + i] * tc.du;
        }
        const double phi[3] = {vn[3] * tc.dt, vn[4] * tc.dt, vn[5] * tc.dt};
        so3_exp(phi, Ex, Jx);
        if (threadIdx.x == 0) {
            for (int i = 0; i < 6; ++i) vnew[i] = vn[i];
            for (int e = 0; e < 9; ++e) {
                E[e] = Ex[e];
                Jl[e] = Jx[e];
            }
        }
    }
    __syncthreads();
    transition_cov(E, Jl, tc, S->P, T1, T2);
    // split: Spp, D = Svp Spp^-1, Sv = Svv - D Svp^T
    if (wv == 0) {
        const int l = threadIdx.x;
        if (l < 36) Spp[l] = T2[(l / 6) * 12 + l % 6];
        wave_lds_order();
        const bool pd = spd_inverse_wave<6>(Spp, Sinv);
        if (l == 0) ok = pd;
    } else if (wv == 1) {
        double R[9], R2[9];
        prism_pose pr;
        quat_to_R9(S->pose.q, R);
        mat3mul(E, R, R2);
        for (int i = 0; i < 3; ++i) pr.t[i] = S->pose.t[i] + vnew[i] * tc.dt;
        R9_to_quat(R2, pr.q);
        if (threadIdx.x == 64) {
            if (rel) rel_of(&pr, &S->anchor, *rel);
            S->prior = pr;
            S->iter = pr;
            S->flags = 0;
        }
    } else if (wv == 2) {
        const int l = threadIdx.x & 63;
        if (l < 6) {
            S->u[l] = u[l];
            S->vel_prior[l] = vnew[l];
        }
    }
    __syncthreads();
    if (!ok) {
        // the predicted pose block is not positive definite: the step keeps
        // the predicted mean and joint covariance, and no pose objective is
        // solved (the Gauss-Newton and Laplace kernels see the flag)
        for (int e = threadIdx.x; e < 144; e += blockDim.x) S->P[e] = T2[e];
        if (threadIdx.x == 0) S->flags |= PRISM_FLAG_CHOL_FALLBACK | PRISM_FLAG_PRIOR_NOT_PD;
        state_out(S, Sg);
        return;
    }
    if (threadIdx.x < 36) {
        const int i = threadIdx.x / 6, j = threadIdx.x % 6;
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < 6; ++q) s += T2[(6 + i) * 12 + q] * Sinv[q * 6 + j];
        D[threadIdx.x] = s;
        S->D[threadIdx.x] = s;
        S->Lp[threadIdx.x] = Sinv[threadIdx.x];
    }
    __syncthreads();
    sym_plus_outer(6, -1.0, D, [&](int j, int q) { return T2[(6 + j) * 12 + q]; },
                   [&](int i, int j) { return T2[(6 + i) * 12 + 6 + j]; },
                   [&](int i, int j, double s) { S->Sv[i * 6 + j] = s; });
    state_out(S, Sg);
}

// The 15-D state (pose, velocities, accelerometer bias b): the linear
// control u[0..2] is the body-frame specific force f, the acceleration
// a = R (f - b) + g with the state's rotation R; then the mean transition
// above with a as the linear acceleration.  Ra = R (f - b) and R are kept
// for the linearisation.  One thread.
__device__ inline void transition_mean_bias_t0(const prism_pose& pose, const double* v0, const double* w0,
                                               const double* b, const double* u, const TransC& tc, double* vnew,
                                               double* E, double* Jl, double* Ra, double* R0, prism_pose& pr) {
    double R[9];
    quat_to_R9(pose.q, R);
    const double f[3] = {u[0] - b[0], u[1] - b[1], u[2] - b[2]};
    double a[6];
    for (int i = 0; i < 3; ++i) {
        Ra[i] = R[i * 3] * f[0] + R[i * 3 + 1] * f[1] + R[i * 3 + 2] * f[2];
        a[i] = Ra[i] + tc.g[i];
        a[3 + i] = u[3 + i];
    }
    for (int e = 0; e < 9; ++e) R0[e] = R[e];
    transition_mean_t0(pose, v0, w0, a, tc, vnew, E, Jl, pr);
}

// Covariance of the linearised 15-D transition, whole workgroup: the blocks
// of transition_cov plus the acceleration's dependence on the rotation and
// the bias at the start of the step, da = -[R (f - b)]x dtheta - R db,
// entering v' over du and t' through v' dt; the bias is a random walk.
// P, M, G, T1, T2: LDS [225].
__device__ inline void transition_cov_bias(const double* E, const double* Jl, const double* Ra, const double* R0,
                                           const TransC& tc, const double* P, double* M, double* G, double* T1,
                                           double* T2) {
    constexpr int N = 15;
    for (int e = threadIdx.x; e < N * N; e += blockDim.x) {
        M[e] = 0.0;
        G[e] = 0.0;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const double K[9] = {0.0, -Ra[2], Ra[1], Ra[2], 0.0, -Ra[0], -Ra[1], Ra[0], 0.0};
        for (int i = 0; i < 3; ++i) {
            M[i * N + i] = 1.0;
            M[i * N + 6 + i] = tc.dt;
            M[(6 + i) * N + 6 + i] = 1.0;
            M[(9 + i) * N + 9 + i] = 1.0;
            M[(12 + i) * N + 12 + i] = 1.0;
            G[i * N + i] = 1.0;
            G[i * N + 6 + i] = tc.dt;
            G[(3 + i) * N + 3 + i] = 1.0;
            G[(6 + i) * N + 6 + i] = 1.0;
            G[(9 + i) * N + 9 + i] = 1.0;
            G[(12 + i) * N + 12 + i] = 1.0;
            for (int j = 0; j < 3; ++j) {
                M[(3 + i) * N + 3 + j] = E[i * 3 + j];
                M[(3 + i) * N + 9 + j] = tc.dt * Jl[i * 3 + j];
                G[(3 + i) * N + 9 + j] = tc.dt * Jl[i * 3 + j];
                const double vth = -tc.du * K[i * 3 + j], vb = -tc.du * R0[i * 3 + j];
                M[(6 + i) * N + 3 + j] = vth;
                M[(6 + i) * N + 12 + j] = vb;
                M[i * N + 3 + j] = tc.dt * vth;
                M[i * N + 12 + j] = tc.dt * vb;
            }
        }
    }
    __syncthreads();
    mm(M, P, T1, N, N, N, false);       // M P
    mm(T1, M, T2, N, N, N, true);       // M P M^T
    for (int e = threadIdx.x; e < N * N; e += blockDim.x) {
        int i = e / N, j = e % N;
        double s = 0.0;
        for (int q = 0; q < N; ++q) s += G[i * N + q] * tc.q[q] * G[j * N + q];
        T2[e] += s;
    }
    __syncthreads();
    symmetrize(T2, N);
}

// predict + split of the 15-D state: the pose prior as for the 12-D state,
// the 9-D conditional of (v, w, b) given the pose into X
__device__ __forceinline__ void predict_block_bias(prism_filter_state* __restrict__ Sg,
                                                   prism_filter_bias_state* __restrict__ X,
                                                   const double* __restrict__ u, const TransC& tc,
                                                   Rel32* __restrict__ rel) {
    constexpr int N = 15, NR = 9;
    __shared__ double M[N * N], G[N * N], T1[N * N], T2[N * N], P[N * N], L[36], Sinv[36];
    __shared__ double vnew[6], E[9], Jl[9], Ra[3], R0[9], b[3];
    __shared__ int ok;
    __shared__ prism_filter_state Ls;
    state_in(Sg, &Ls);
    prism_filter_state* S = &Ls;
    for (int e = threadIdx.x; e < N * N; e += blockDim.x) P[e] = X->P[e];
    if (threadIdx.x < 3) b[threadIdx.x] = X->b[threadIdx.x];
    __syncthreads();
    if (threadIdx.x == 0) {
        S->flags = 0;
        for (int i = 0; i < 6; ++i) S->u[i] = u[i];
        prism_pose pr;
        transition_mean_bias_t0(S->pose, S->v, S->w, b, u, tc, vnew, E, Jl, Ra, R0, pr);
        S->prior = pr;
        S->iter = pr;
        if (rel) rel_of(&S->iter, &S->anchor, *rel);
        for (int i = 0; i < 6; ++i) S->vel_prior[i] = vnew[i];
    }
    __syncthreads();
    transition_cov_bias(E, Jl, Ra, R0, tc, P, M, G, T1, T2);
    for (int e = threadIdx.x; e < 36; e += blockDim.x) L[e] = T2[(e / 6) * N + e % 6];
    for (int e = threadIdx.x; e < N * N; e += blockDim.x) X->P[e] = T2[e];
    for (int e = threadIdx.x; e < 144; e += blockDim.x) S->P[e] = T2[(e / 12) * N + e % 12];
    if (threadIdx.x < 6) X->rest_prior[threadIdx.x] = vnew[threadIdx.x];
    else if (threadIdx.x < NR) X->rest_prior[threadIdx.x] = b[threadIdx.x - 6];
    __syncthreads();
    if (threadIdx.x < 64) {
        const bool pd = spd_inverse_wave<6>(L, Sinv);
        if (threadIdx.x == 0) ok = pd;
    }
    __syncthreads();
    if (!ok) {
        // no MAP problem: the step keeps the predicted mean and covariance
        if (threadIdx.x == 0) S->flags |= PRISM_FLAG_CHOL_FALLBACK | PRISM_FLAG_PRIOR_NOT_PD;
        state_out(S, Sg);
        return;
    }
    // D = P_rp Sinv [9 x 6], Sv = P_rr - D P_rp^T [9 x 9]
    for (int e = threadIdx.x; e < NR * 6; e += blockDim.x) {
        int i = e / 6, j = e % 6;
        double s = 0.0;
        for (int q = 0; q < 6; ++q) s += T2[(6 + i) * N + q] * Sinv[q * 6 + j];
        T1[e] = s;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < NR * NR; e += blockDim.x) {
        int i = e / NR, j = e % NR;
        double s = 0.0;
        for (int q = 0; q < 6; ++q) s += T1[i * 6 + q] * T2[(6 + j) * N + q];
        P[e] = T2[(6 + i) * N + 6 + j] - s;
    }
    __syncthreads();
    symmetrize(P, NR);
    for (int e = threadIdx.x; e < 36; e += blockDim.x) S->Lp[e] = Sinv[e];
    for (int e = threadIdx.x; e < NR * 6; e += blockDim.x) X->D[e] = T1[e];
    for (int e = threadIdx.x; e < NR * NR; e += blockDim.x) X->Sv[e] = P[e];
    state_out(S, Sg);
}

__global__ __launch_bounds__(256) void k_predict(prism_filter_state* __restrict__ Sg,
                                                 prism_filter_bias_state* __restrict__ X,
                                                 const double* __restrict__ u, TransC tc, Rel32* __restrict__ rel) {
    if (X)
        predict_block_bias(Sg, X, u, tc, rel);
    else
        predict_block(Sg, u, tc, rel);
}

// ---------------------------------------------------------------------------
// one Gauss-Newton step of the MAP pose objective
// ---------------------------------------------------------------------------
// What does not depend on the normal equations (the error of the iterate to the
// prior, its rotation, the anchor's) is formed by the ninth wavefront while the
// others sum them; the first then solves in registers.  8.1 -> 4.9 us at 300
// partial rows, 12.3 -> 8.3 at 1200 (0.4 of it for the relative pose from the
// quaternion, whose normalisation is the recipe's, root and divisions).
constexpr int kSolveThreads = kSumThreads + 64;

struct GnPrep {
    double le[6], Lp[36], R[9], t[3];   // Lp e; prior precision; the iterate
    Pose64 anchor;
    int flags;
};

__device__ __forceinline__ void gn_step_block(prism_filter_state* __restrict__ Sg,
                                              const double* __restrict__ partials, int nblocks,
                                              Rel32* __restrict__ rel) {
    __shared__ double red[kSumThreads], neq[PRISM_NEQ];
    __shared__ GnPrep pre;
    if (threadIdx.x >= kSumThreads) {
        const int l = threadIdx.x - kSumThreads;
        const double lp = Sg->Lp[l < 36 ? l : 0];
        const prism_pose it = Sg->iter, pr = Sg->prior, an = Sg->anchor;
        const int flags = Sg->flags;
        if (l < 36) pre.Lp[l] = lp;
        double e[6], R[9];
        pose_err(it, pr, e);
        quat_to_R9(it.q, R);
        const Pose64 Q = load_pose64(&an);
        if (l == 0) {
            for (int i = 0; i < 9; ++i) pre.R[i] = R[i];
            for (int i = 0; i < 3; ++i) pre.t[i] = it.t[i];
            pre.anchor = Q;
            pre.flags = flags;
        }
        wave_lds_order();
        if (l < 6) {
            double s = 0.0;
#pragma unroll
            for (int j = 0; j < 6; ++j) s += pre.Lp[l * 6 + j] * e[j];
            pre.le[l] = s;
        }
    }
    sum_partials(partials, nblocks, red, neq);
    if (threadIdx.x >= 64 || (pre.flags & PRISM_FLAG_CHOL_FALLBACK)) return;
    int flags = pre.flags;
    if (!(neq[28] > 0.0)) flags |= PRISM_FLAG_NO_VALID_PIXELS;
    double A[36], b[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
#pragma unroll
        for (int j = 0; j <= i; ++j) A[i * 6 + j] = 2.0 * neq[sym6(i, j)] + pre.Lp[i * 6 + j];
        b[i] = -(2.0 * neq[21 + i] + pre.le[i]);
    }
    Chol<6> c;
    if (!chol_regs<6>(A, c)) {
        if (threadIdx.x == 0) {
            const prism_pose pr = Sg->prior;
            Sg->iter = pr;
            Sg->flags = flags | PRISM_FLAG_CHOL_FALLBACK;
            if (rel) rel_of(load_pose64(&pr), pre.anchor, *rel);
        }
        return;
    }
    chol_solve<6>(c, b);
    // t <- t + dt, R <- Exp(dtheta) R
    double E[9], R2[9];
    so3_exp_step(b + 3, E);
    mat3mul(E, pre.R, R2);
    prism_pose it;
    for (int i = 0; i < 3; ++i) it.t[i] = pre.t[i] + b[i];
    R9_to_quat(R2, it.q);
    if (threadIdx.x == 0) {
        Sg->iter = it;
        Sg->flags = flags;
        // from the quaternion as it is stored, not from R2: a tracking call at
        // the stored pose takes the same decisions
        if (rel) rel_of(load_pose64(&it), pre.anchor, *rel);
    }
}

__global__ __launch_bounds__(kSolveThreads) void k_gn_step(prism_filter_state* __restrict__ Sg,
                                                           const double* __restrict__ partials, int nblocks,
                                                           Rel32* __restrict__ rel) {
    gn_step_block(Sg, partials, nblocks, rel);
}

// ---------------------------------------------------------------------------
// Laplace covariance, EMA, product with the velocity conditional
// ---------------------------------------------------------------------------
// The product with the 9-D conditional of (v, w, b) of the 15-D state:
// joint covariance [[Sb, Sb D^T], [D Sb, Sv + D Sb D^T]] over 15 dimensions,
// means rest_prior + D e; the leading 12x12 block also into S->P.
__device__ inline void combine_bias(prism_filter_state* S, prism_filter_bias_state* __restrict__ X,
                                    const double* Sb, const double* e) {
    constexpr int N = 15, NR = 9;
    __shared__ double D9[NR * 6], T9[NR * 6], P15[N * N];
    for (int i = threadIdx.x; i < NR * 6; i += blockDim.x) D9[i] = X->D[i];
    __syncthreads();
    mm(D9, Sb, T9, NR, 6, 6, false);   // D Sb
    for (int e2 = threadIdx.x; e2 < N * N; e2 += blockDim.x) {
        int i = e2 / N, j = e2 % N;
        double s;
        if (i < 6 && j < 6) s = Sb[i * 6 + j];
        else if (i < 6) s = T9[(j - 6) * 6 + i];
        else if (j < 6) s = T9[(i - 6) * 6 + j];
        else {
            s = X->Sv[(i - 6) * NR + (j - 6)];
            for (int q = 0; q < 6; ++q) s += T9[(i - 6) * 6 + q] * D9[(j - 6) * 6 + q];
        }
        P15[e2] = s;
    }
    __syncthreads();
    symmetrize(P15, N);
    for (int e2 = threadIdx.x; e2 < N * N; e2 += blockDim.x) X->P[e2] = P15[e2];
    for (int e2 = threadIdx.x; e2 < 144; e2 += blockDim.x) S->P[e2] = P15[(e2 / 12) * N + e2 % 12];
    if (threadIdx.x == 0) {
        double vm[NR];
        for (int i = 0; i < NR; ++i) {
            vm[i] = X->rest_prior[i];
            for (int j = 0; j < 6; ++j) vm[i] += D9[i * 6 + j] * e[j];
        }
        for (int i = 0; i < 3; ++i) {
            S->v[i] = vm[i];
            S->w[i] = vm[3 + i];
            X->b[i] = vm[6 + i];
        }
    }
}

// 7.9 -> 4.8 us at 300 partial rows, 12.7 -> 9.0 at 1200: the error of the
// iterate to the prior is formed by the ninth wavefront while the others sum the
// normal equations.
__device__ __forceinline__ void laplace_combine_block(prism_filter_state* __restrict__ Sg,
                                                      prism_filter_bias_state* __restrict__ X,
                                                      const double* __restrict__ partials, int nblocks, double ema,
                                                      double min_inliers, double lap_h) {
    __shared__ double red[kSumThreads], neq[PRISM_NEQ];
    __shared__ double A[36], Sl[36], Sb[36], T[36], e[6], eraw[6];
    __shared__ prism_filter_state Ls;
    prism_filter_state* S = &Ls;
    if (threadIdx.x >= kSumThreads) {
        double er[6];
        const prism_pose it = Sg->iter, pr = Sg->prior;
        pose_err(it, pr, er);
        if (threadIdx.x == kSumThreads)
            for (int i = 0; i < 6; ++i) eraw[i] = er[i];
    }
    sum_partials(partials, nblocks, red, neq, Sg, &Ls);
    if (threadIdx.x < PRISM_NEQ) S->neq[threadIdx.x] = neq[threadIdx.x];
    if (S->flags & PRISM_FLAG_PRIOR_NOT_PD) {
        // predicted mean and covariance as they are (the covariance was
        // written by the predict kernel); the Laplace EMA is left unchanged
        __syncthreads();   // every thread has read the flags
        if (threadIdx.x == 0) {
            if (!(neq[28] > 0.0)) S->flags |= PRISM_FLAG_NO_VALID_PIXELS;
            if (neq[28] < min_inliers) S->flags |= PRISM_FLAG_LOW_INLIERS;
            for (int i = 0; i < 3; ++i) { S->v[i] = S->vel_prior[i]; S->w[i] = S->vel_prior[3 + i]; }
            if (X)
                for (int i = 0; i < 3; ++i) X->b[i] = X->rest_prior[6 + i];
            S->iter = S->prior;
            S->pose = S->prior;
            S->anchor = S->prior;
            S->step += 1;
        }
        state_out(S, Sg);
        return;
    }
    if (threadIdx.x < 64) {
        const int l = threadIdx.x;
        int flags = S->flags;
        if (!(neq[28] > 0.0)) flags |= PRISM_FLAG_NO_VALID_PIXELS;
        // fewer contributing pixels at the final iterate than the filter asks for
        if (neq[28] < min_inliers) flags |= PRISM_FLAG_LOW_INLIERS;
        // Laplace precision lap_h H + Lp (Sec. 5.1 prints lap_h = 2)
        if (l < 36) A[l] = lap_h * neq[sym6(l / 6, l % 6)] + S->Lp[l];
        wave_lds_order();
        bool ok = !(flags & PRISM_FLAG_CHOL_FALLBACK) && spd_inverse_wave<6>(A, Sl);
        if (!ok) {
            // prior pose covariance = Lp^-1, and the iterate back to the prior
            flags |= PRISM_FLAG_CHOL_FALLBACK;
            (void)spd_inverse_wave<6>(S->Lp, Sl);
            if (l == 0) S->iter = S->prior;
        }
        if (l < 6) e[l] = ok ? eraw[l] : 0.0;
        wave_lds_order();
        if (l < 36) {
            S->S_lap[l] = Sl[l];
            const double sb = S->has_sbar ? ema * S->Sbar[l] + (1.0 - ema) * Sl[l] : Sl[l];
            Sb[l] = sb;
            S->Sbar[l] = sb;
        }
        if (l == 0) S->flags = flags;
    }
    __syncthreads();
    if (X) {
        combine_bias(S, X, Sb, e);
    } else {
        // joint covariance [[Sb, Sb D^T], [D Sb, Sv + D Sb D^T]], means vel_prior + D e
        if (threadIdx.x < 36) {
            const int i = threadIdx.x / 6, j = threadIdx.x % 6;
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < 6; ++q) s += S->D[i * 6 + q] * Sb[q * 6 + j];
            T[threadIdx.x] = s;   // D Sb
        } else if (threadIdx.x >= 64 && threadIdx.x < 70) {
            const int i = threadIdx.x - 64;
            double s = S->vel_prior[i];
#pragma unroll
            for (int j = 0; j < 6; ++j) s += S->D[i * 6 + j] * e[j];
            (i < 3 ? S->v[i] : S->w[i - 3]) = s;
        }
        __syncthreads();
        if (threadIdx.x >= 128 && threadIdx.x < 128 + 108) {
            // the pose rows: Sb and (D Sb)^T, and their mirror
            const int k = threadIdx.x - 128, i = k % 6, j = k / 6;   // j < 18: Sb, then T twice
            if (j < 6) S->P[i * 12 + j] = Sb[i * 6 + j];
            else if (j < 12) S->P[i * 12 + j] = T[(j - 6) * 6 + i];
            else S->P[(j - 6) * 12 + i] = T[(j - 12) * 6 + i];
        } else if (threadIdx.x < 36) {
            sym_plus_outer(6, 1.0, T, [&](int j, int q) { return S->D[j * 6 + q]; },
                           [&](int i, int j) { return S->Sv[i * 6 + j]; },
                           [&](int i, int j, double s) { S->P[(6 + i) * 12 + 6 + j] = s; });
        }
    }
    if (threadIdx.x == 0) {
        S->has_sbar = 1;
        S->pose = S->iter;
        S->anchor = S->iter;
        S->step += 1;
    }
    state_out(S, Sg);
}

__global__ __launch_bounds__(kSolveThreads) void k_laplace_combine(prism_filter_state* __restrict__ Sg,
                                                                   prism_filter_bias_state* __restrict__ X,
                                                                   const double* __restrict__ partials, int nblocks,
                                                                   double ema, double min_inliers, double lap_h) {
    laplace_combine_block(Sg, X, partials, nblocks, ema, min_inliers, lap_h);
}

// the left, world-frame retraction of n poses by n tangent increments
__global__ __launch_bounds__(256) void k_pose_retract(const prism_pose* __restrict__ poses,
                                                      const double* __restrict__ delta, int n,
                                                      prism_pose* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    prism_pose p = poses[i];
    double d[6];
    for (int a = 0; a < 6; ++a) d[a] = delta[6 * i + a];
    retract(p, d);
    out[i] = p;
}

__device__ __forceinline__ void first_frame_block(prism_filter_state* __restrict__ S) {
    if (threadIdx.x == 0) {
        S->anchor = S->pose;
        S->step = 1;
        S->flags = 0;
    }
}

__global__ void k_first_frame(prism_filter_state* __restrict__ S) { first_frame_block(S); }

// batched: one workgroup per filter
__global__ __launch_bounds__(256) void k_predict_batch(BatchArgs b) {
    const AgentDesc& D = *b.d[blockIdx.x];
    if (D.X)
        predict_block_bias(D.S, D.X, (const double*)D.slots[b.slot[blockIdx.x]].u, D.tc, D.rel);
    else
        predict_block(D.S, (const double*)D.slots[b.slot[blockIdx.x]].u, D.tc, D.rel);
}

__global__ __launch_bounds__(kSolveThreads) void k_gn_step_batch(BatchArgs b) {
    const AgentDesc& D = *b.d[blockIdx.x];
    gn_step_block(D.S, D.partials, D.obj_blocks, D.rel);
}

__global__ __launch_bounds__(kSolveThreads) void k_laplace_combine_batch(BatchArgs b) {
    const AgentDesc& D = *b.d[blockIdx.x];
    laplace_combine_block(D.S, D.X, D.partials, D.obj_blocks, D.ema, D.min_inliers, D.lap_h);
}

__global__ __launch_bounds__(64) void k_first_frame_batch(BatchArgs b) { first_frame_block(b.d[blockIdx.x]->S); }

// ---------------------------------------------------------------------------
// predictive rollouts from the state belief
// ---------------------------------------------------------------------------
// One workgroup per sample; its first thread draws the start state from the
// belief, x0 = x (+) L z0 with P = L L^T (tangent order t, theta, v, w; the
// pose part is the left retraction), then runs the generative transition
// with process noise n = sqrt(Q) z_j for each of the k controls:
//   v' = v + u_v du + n_v,  w' = w + u_w du + n_w,
//   t' = t + v' dt + n_t,   R' = Exp(n_theta) Exp(w' dt) R
// (du = dt, or dt^2 in the printed form).  The 15-D state (X non-NULL)
// draws 15 components per row (the bias last), takes the acceleration
// R (u_v - b) + g with the draw's rotation and bias, and walks the bias by
// n_b.  If P is not positive definite every sample starts at the mean and
// *flags gets PRISM_FLAG_CHOL_FALLBACK (else 0; written by the first
// workgroup).
//
// A sample is one chain of small dependent steps, run by one wavefront (its
// lanes hold the same values) at the latency of the arithmetic: the controls
// and the noise of kRolloutChunk steps are fetched at once.
constexpr int kRolloutChunk = 16;

__device__ __forceinline__ void rollout_sample_block(int sample, const prism_filter_state* __restrict__ S,
                                                     const prism_filter_bias_state* __restrict__ X,
                                                     const double* __restrict__ u, int k,
                                                     const double* __restrict__ noise, const TransC& tc,
                                                     prism_pose* __restrict__ poses, int32_t* __restrict__ flags) {
    __shared__ double A[225], sz[kRolloutChunk * 15], su[kRolloutChunk * 6];
    const int lane = threadIdx.x;
    if (lane >= 64) return;
    const int N = X ? 15 : 12;
    const double* z = noise + (long long)sample * (k + 1) * N;
    for (int e = lane; e < N * N; e += 64) A[e] = X ? X->P[e] : S->P[e];
    if (lane < N) sz[lane] = z[lane];
    prism_pose x = S->pose;
    double v[3], w[3], b[3], sq[15];
    for (int i = 0; i < 3; ++i) {
        v[i] = S->v[i];
        w[i] = S->w[i];
        b[i] = X ? X->b[i] : 0.0;
    }
    for (int i = 0; i < N; ++i) sq[i] = sqrt(tc.q[i]);
    wave_lds_order();
    bool ok = false;
    if (lane == 0) ok = X ? chol<15>(A) : chol<12>(A);
    ok = __builtin_amdgcn_readfirstlane((int)ok);
    wave_lds_order();
    if (lane == 0 && sample == 0 && flags) *flags = ok ? 0 : PRISM_FLAG_CHOL_FALLBACK;
    double e[15];
    for (int i = 0; i < N; ++i) {
        double acc = 0.0;
        if (ok)
            for (int j = 0; j <= i; ++j) acc += A[i * N + j] * sz[j];
        e[i] = acc;
    }
    retract(x, e);
    for (int i = 0; i < 3; ++i) {
        v[i] += e[6 + i];
        w[i] += e[9 + i];
        if (X) b[i] += e[12 + i];
    }
    for (int j0 = 0; j0 < k; j0 += kRolloutChunk) {
        const int steps = min(k - j0, kRolloutChunk);
        wave_lds_order();
        for (int i = lane; i < steps * N; i += 64) sz[i] = z[(long long)(j0 + 1) * N + i];
        for (int i = lane; i < steps * 6; i += 64) su[i] = u[6 * (long long)j0 + i];
        wave_lds_order();
        for (int j = 0; j < steps; ++j) {
            const double* zj = sz + j * N;
            const double* uj = su + 6 * j;
            double n[15], R[9];
            for (int i = 0; i < N; ++i) n[i] = sq[i] * zj[i];
            quat_to_R9(x.q, R);
            if (X) {
                const double f[3] = {uj[0] - b[0], uj[1] - b[1], uj[2] - b[2]};
                for (int i = 0; i < 3; ++i) {
                    const double a = R[i * 3] * f[0] + R[i * 3 + 1] * f[1] + R[i * 3 + 2] * f[2] + tc.g[i];
                    v[i] = v[i] + a * tc.du + n[6 + i];
                    w[i] = w[i] + uj[3 + i] * tc.du + n[9 + i];
                }
                for (int i = 0; i < 3; ++i) b[i] += n[12 + i];
            } else {
                for (int i = 0; i < 3; ++i) {
                    v[i] = v[i] + uj[i] * tc.du + n[6 + i];
                    w[i] = w[i] + uj[3 + i] * tc.du + n[9 + i];
                }
            }
            const double phi[3] = {w[0] * tc.dt, w[1] * tc.dt, w[2] * tc.dt};
            double E1[9], E2[9], T[9], R2[9];
            so3_exp_step(n + 3, E1);
            so3_exp_step(phi, E2);
            mat3mul(E2, R, T);
            mat3mul(E1, T, R2);
            for (int i = 0; i < 3; ++i) x.t[i] = x.t[i] + v[i] * tc.dt + n[i];
            R9_to_quat(R2, x.q);
            if (lane == 0) poses[(long long)sample * k + j0 + j] = x;
        }
    }
}

// Closed-form (linearised) prediction of the belief over the k controls:
// mean[j] = (t, q, v, w) after control j (13 doubles), cov[j] = its 12x12
// covariance; the same propagation as the filter's prediction step.
__device__ __forceinline__ void rollout_moments_block(const prism_filter_state* __restrict__ S,
                                                      const double* __restrict__ u, int k, const TransC& tc,
                                                      double* __restrict__ mean, double* __restrict__ cov) {
    __shared__ double T1[144], T2[144], P[144], su[kRolloutChunk * 6];
    __shared__ double vnew[6], E[9], Jl[9], v[3], w[3];
    __shared__ prism_pose pose;
    if (threadIdx.x == 0) {
        pose = S->pose;
        for (int i = 0; i < 3; ++i) {
            v[i] = S->v[i];
            w[i] = S->w[i];
        }
    }
    for (int e = threadIdx.x; e < 144; e += blockDim.x) P[e] = S->P[e];
    for (int j = 0; j < k; ++j) {
        if (j % kRolloutChunk == 0) {
            // (thread 0 has left the chunk before: a step ends with a barrier)
            if ((int)threadIdx.x < 6 * min(k - j, kRolloutChunk)) su[threadIdx.x] = u[6 * (long long)j + threadIdx.x];
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            prism_pose pr;
            transition_mean_t0(pose, v, w, su + 6 * (j % kRolloutChunk), tc, vnew, E, Jl, pr);
            pose = pr;
            for (int i = 0; i < 3; ++i) {
                v[i] = vnew[i];
                w[i] = vnew[3 + i];
            }
            if (mean) {
                double* m = mean + 13 * j;
                for (int i = 0; i < 3; ++i) m[i] = pr.t[i];
                for (int i = 0; i < 4; ++i) m[3 + i] = pr.q[i];
                for (int i = 0; i < 6; ++i) m[7 + i] = vnew[i];
            }
        }
        __syncthreads();
        transition_cov(E, Jl, tc, P, T1, T2);
        for (int e = threadIdx.x; e < 144; e += blockDim.x) {
            P[e] = T2[e];
            if (cov) cov[144 * j + e] = T2[e];
        }
        __syncthreads();
    }
}

// The same for the 15-D state: mean[j] = (t, q, v, w, b) (16 doubles),
// cov[j] its 15x15 covariance.
__device__ __forceinline__ void rollout_moments_bias_block(const prism_filter_state* __restrict__ S,
                                                           const prism_filter_bias_state* __restrict__ X,
                                                           const double* __restrict__ u, int k, const TransC& tc,
                                                           double* __restrict__ mean, double* __restrict__ cov) {
    constexpr int N = 15;
    __shared__ double M[N * N], G[N * N], T1[N * N], T2[N * N], P[N * N], su[kRolloutChunk * 6];
    __shared__ double vnew[6], E[9], Jl[9], Ra[3], R0[9], v[3], w[3], b[3];
    __shared__ prism_pose pose;
    if (threadIdx.x == 0) {
        pose = S->pose;
        for (int i = 0; i < 3; ++i) {
            v[i] = S->v[i];
            w[i] = S->w[i];
            b[i] = X->b[i];
        }
    }
    for (int e = threadIdx.x; e < N * N; e += blockDim.x) P[e] = X->P[e];
    for (int j = 0; j < k; ++j) {
        if (j % kRolloutChunk == 0) {
            if ((int)threadIdx.x < 6 * min(k - j, kRolloutChunk)) su[threadIdx.x] = u[6 * (long long)j + threadIdx.x];
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            prism_pose pr;
            transition_mean_bias_t0(pose, v, w, b, su + 6 * (j % kRolloutChunk), tc, vnew, E, Jl, Ra, R0, pr);
            pose = pr;
            for (int i = 0; i < 3; ++i) {
                v[i] = vnew[i];
                w[i] = vnew[3 + i];
            }
            if (mean) {
                double* m = mean + 16 * j;
                for (int i = 0; i < 3; ++i) m[i] = pr.t[i];
                for (int i = 0; i < 4; ++i) m[3 + i] = pr.q[i];
                for (int i = 0; i < 6; ++i) m[7 + i] = vnew[i];
                for (int i = 0; i < 3; ++i) m[13 + i] = b[i];
            }
        }
        __syncthreads();
        transition_cov_bias(E, Jl, Ra, R0, tc, P, M, G, T1, T2);
        for (int e = threadIdx.x; e < N * N; e += blockDim.x) {
            P[e] = T2[e];
            if (cov) cov[N * N * j + e] = T2[e];
        }
        __syncthreads();
    }
}

// The moments and the samples know nothing of each other and each is one chain:
// they run side by side, the moments in the first workgroup (when they are
// wanted).  16 samples of 10 controls: 29 and 37 us one after the other, 30
// together.
__global__ __launch_bounds__(256) void k_rollout(const prism_filter_state* __restrict__ S,
                                                 const prism_filter_bias_state* __restrict__ X,
                                                 const double* __restrict__ u, int k, TransC tc, int moments,
                                                 double* __restrict__ mean, double* __restrict__ cov,
                                                 const double* __restrict__ noise, prism_pose* __restrict__ poses,
                                                 int32_t* __restrict__ flags) {
    if ((int)blockIdx.x >= moments)
        rollout_sample_block(blockIdx.x - moments, S, X, u, k, noise, tc, poses, flags);
    else if (X)
        rollout_moments_bias_block(S, X, u, k, tc, mean, cov);
    else
        rollout_moments_block(S, u, k, tc, mean, cov);
}

hipError_t launch_rollout(const prism_filter_state* S, const prism_filter_bias_state* X, const double* u, int k,
                          int n_samples, const double* noise, const TransC& tc, prism_pose* poses, double* mean,
                          double* cov, int32_t* flags, hipStream_t st) {
    const int moments = mean || cov ? 1 : 0;
    if (moments + n_samples == 0) return hipSuccess;
    k_rollout<<<moments + n_samples, 256, 0, st>>>(S, X, u, k, tc, moments, mean, cov, noise, poses, flags);
    return hipGetLastError();
}

// Per-frame fixed-order sum of block partials (NV values each), eight columns
// per workgroup: one CU reads a frame's rows at its own rate (1200 rows of 29:
// 6.3 us by one workgroup, 4.7 by four), and 64 threads per column have a frame
// of 1280 rows in flight at once.
template <int NV>
__global__ __launch_bounds__(512) void k_finalize(const double* __restrict__ partials, int nblocks,
                                                  double* __restrict__ out) {
    __shared__ double red[8][8];
    constexpr int kRound = 20;
    const int col = (int)blockIdx.y * 8 + (threadIdx.x & 7);
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    if (col < NV) {
        const double* p = partials + (long long)blockIdx.x * nblocks * NV + col;
        for (int r0 = threadIdx.x >> 3; r0 < nblocks; r0 += 64 * kRound) {
            double x[kRound];
#pragma unroll
            for (int k = 0; k < kRound; ++k) x[k] = r0 + 64 * k < nblocks ? p[(long long)(r0 + 64 * k) * NV] : 0.0;
#pragma unroll
            for (int k = 0; k < kRound; ++k) a[k & 3] += x[k];
        }
    }
    double s = (a[0] + a[1]) + (a[2] + a[3]);
    // lanes that agree in their low three bits
    s = add_dpp<0x128>(s);   // row rotate by 8
    const unsigned lo = (unsigned)__double2loint(s), hi = (unsigned)__double2hiint(s);
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    s = __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
    const unsigned lo2 = (unsigned)__double2loint(s), hi2 = (unsigned)__double2hiint(s);
    const auto l2 = __builtin_amdgcn_permlane32_swap(lo2, lo2, false, false);
    const auto h2 = __builtin_amdgcn_permlane32_swap(hi2, hi2, false, false);
    s = __hiloint2double((int)h2[0], (int)l2[0]) + __hiloint2double((int)h2[1], (int)l2[1]);
    if ((threadIdx.x & 63) < 8) red[threadIdx.x >> 6][threadIdx.x & 7] = s;
    __syncthreads();
    if (threadIdx.x < 8 && col < NV) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < 8; ++w) t += red[w][threadIdx.x];
        out[(long long)blockIdx.x * NV + col] = t;
    }
}

hipError_t launch_predict(prism_filter_state* S, prism_filter_bias_state* X, const double* u, const TransC& tc,
                          Rel32* rel, hipStream_t st) {
    k_predict<<<1, 256, 0, st>>>(S, X, u, tc, rel);
    return hipGetLastError();
}

hipError_t launch_gn_step(prism_filter_state* S, const double* partials, int nblocks, Rel32* rel,
                          hipStream_t st) {
    k_gn_step<<<1, kSolveThreads, 0, st>>>(S, partials, nblocks, rel);
    return hipGetLastError();
}

hipError_t launch_laplace_combine(prism_filter_state* S, prism_filter_bias_state* X, const double* partials,
                                  int nblocks, double ema, double min_inliers, double lap_h, hipStream_t st) {
    k_laplace_combine<<<1, kSolveThreads, 0, st>>>(S, X, partials, nblocks, ema, min_inliers, lap_h);
    return hipGetLastError();
}

hipError_t launch_pose_retract(const prism_pose* poses, const double* delta, int n, prism_pose* out, hipStream_t st) {
    k_pose_retract<<<(n + 255) / 256, 256, 0, st>>>(poses, delta, n, out);
    return hipGetLastError();
}

hipError_t launch_first_frame(prism_filter_state* S, hipStream_t st) {
    k_first_frame<<<1, 1, 0, st>>>(S);
    return hipGetLastError();
}

hipError_t launch_predict_batch(const BatchArgs& b, hipStream_t st) {
    k_predict_batch<<<b.n, 256, 0, st>>>(b);
    return hipGetLastError();
}

hipError_t launch_gn_step_batch(const BatchArgs& b, hipStream_t st) {
    k_gn_step_batch<<<b.n, kSolveThreads, 0, st>>>(b);
    return hipGetLastError();
}

hipError_t launch_laplace_combine_batch(const BatchArgs& b, hipStream_t st) {
    k_laplace_combine_batch<<<b.n, kSolveThreads, 0, st>>>(b);
    return hipGetLastError();
}

hipError_t launch_first_frame_batch(const BatchArgs& b, hipStream_t st) {
    k_first_frame_batch<<<b.n, 64, 0, st>>>(b);
    return hipGetLastError();
}

hipError_t launch_finalize(const double* partials, int nblocks, int n_frames, double* out, hipStream_t st) {
    k_finalize<PRISM_NEQ><<<dim3(n_frames, (PRISM_NEQ + 7) / 8), 512, 0, st>>>(partials, nblocks, out);
    return hipGetLastError();
}

hipError_t launch_finalize6(const double* partials, int nblocks, int n_frames, double* out, hipStream_t st) {
    k_finalize<6><<<n_frames, 512, 0, st>>>(partials, nblocks, out);
    return hipGetLastError();
}

}  // namespace prism
