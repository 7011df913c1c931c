// Pieces of the scaled solves (streaming and on-chip): block geometry, the FP64 true residual, the transforms to and
// from the congruence basis, and the refinement loop around an inner PCG.
#pragma once

#include <math.h>

#include "ssp_device.h"
#include "ssp_fused.h"
#include "ssp_host.h"

namespace ssp {

namespace {

template <typename TM>
constexpr int vlen() { return 16 / (int)sizeof(TM); }
template <typename TM, int NX>
constexpr int bstride() { return (NX * NX + vlen<TM>() - 1) / vlen<TM>() * vlen<TM>(); }
template <typename TM, int NX>
constexpr int vstride() { return (NX + vlen<TM>() - 1) / vlen<TM>() * vlen<TM>(); }
template <int BLOCK, int NX>
constexpr int max_step() { return (BLOCK / 64) * (64 / NX); }

// Knots per step of residual_lean for an LDS budget: C + 1 knot slots of D
// (packed) and L in FP64 and a lambda window of C + 2 knots.
template <typename TM, int NX>
__host__ __device__ inline int residual3_knots(int lds_bytes) {
    constexpr int V = vlen<TM>();
    constexpr int SS = (NX * (NX + 1) / 2 + V - 1) / V * V + bstride<TM, NX>(), NXP = (NX + 1) & ~1;
    int C = (lds_bytes / 8 - NXP) / (SS + NXP) - 1;
    return C < 64 ? C : 64;
}

template <typename TI>
struct Vecs3 {
    TI *u, *w, *p, *s, *x, *r;
};

// Per-lane partial inner products of one pass: in the storage type, or (the
// FP64-accumulation option) the same storage-type products summed in FP64.
template <typename TI>
struct Dots3 {
    TI gam, del, rho;
    double g64 = 0.0, d64 = 0.0, r64 = 0.0;
};

// r = gamma - S lambda in FP64 with S read as D (packed) and L in the
// storage type plus their FP32 remainders (or FP64), in steps of C knots:
// the step's D, L (and L of the next knot) are converted to FP64 into LDS
// with 16-byte loads, lambda of knots k0 - 1 .. k1 into a window, then r is
// formed for knots [k0, k1).  No loads cross a step, so the pass needs few
// registers (it runs once per outer step).  Returns this thread's parts of
// ||r||^2 and ||gamma||^2, summed over the same rows in the same order.
template <typename TM, int BLOCK, int NX>
__device__ __forceinline__ ResNorms residual_lean(int N, int C, const TM *__restrict__ B3,
                                                  const float *__restrict__ Dlo, const float *__restrict__ Llo,
                                                  const double *__restrict__ lam, const double *__restrict__ gam,
                                                  double *__restrict__ r64, double *smem) {
    constexpr int V = vlen<TM>(), KW = 64 / NX, W = BLOCK / 64, NXP = (NX + 1) & ~1;
    constexpr int BS = bstride<TM, NX>(), BP = (NX * (NX + 1) / 2 + V - 1) / V * V, KS = 2 * BP + BS;
    constexpr int SS = BP + BS;  // FP64 slot: D packed, then L
    constexpr bool LO = sizeof(TM) == 4;
    double *ring = smem, *win = smem + (C + 1) * SS;  // C + 1 knot slots, C + 2 window slots
    const int lane = threadIdx.x & 63, kloc = lane / NX, i = lane - kloc * NX;
    const bool lane_ok = kloc < KW;
    const int kme = (threadIdx.x >> 6) * KW + kloc, group = W * KW;
    double rr = 0.0, gg = 0.0;
    __syncthreads();  // lambda rows were just written by other threads
    for (int k0 = 0; k0 < N; k0 += C) {
        const int k1 = min(k0 + C, N), kl = min(k1 + 1, N);  // blocks of knots [k0, kl)
        const int nv = (kl - k0) * (SS / V);
        for (int q = threadIdx.x; q < nv; q += BLOCK) {
            const int kk = q / (SS / V), e = (q - kk * (SS / V)) * V;
            const int64_t k = k0 + kk;
            const TM *src = B3 + k * KS + e;  // D packed then L: the first SS elements of the knot
            double *dst = ring + kk * SS + e;
            if constexpr (LO) {
                const f32x4 h = *(const f32x4 *)src;
                const f32x4 l = *(const f32x4 *)(e < BP ? Dlo + k * BP + e : Llo + k * BS + (e - BP));
                dst[0] = (double)h.x + (double)l.x;
                dst[1] = (double)h.y + (double)l.y;
                dst[2] = (double)h.z + (double)l.z;
                dst[3] = (double)h.w + (double)l.w;
            } else {
                const f64x2 h = *(const f64x2 *)src;
                dst[0] = h.x;
                dst[1] = h.y;
            }
        }
        const int lo = max(k0 - 1, 0), nl = (kl - lo) * NX;
        for (int q = threadIdx.x; q < nl; q += BLOCK) {
            const int kk = q / NX, j = q - kk * NX;
            win[kk * NXP + j] = lam[(int64_t)lo * NX + q];
        }
        __syncthreads();
        for (int kk = kme; kk < k1 - k0; kk += group) {
            if (!lane_ok) break;
            const int k = k0 + kk, wk = k - lo;  // window slot of knot k
            const double *Dk = ring + kk * SS;
            double y = lean_sym_dot<NX>(Dk, i, win + wk * NXP);
            if (k > 0) y += lean_dot<NX, false>(Dk + BP, i, win + (wk - 1) * NXP);
            if (k + 1 < N) y += lean_dot<NX, true>(ring + (kk + 1) * SS + BP, i, win + (wk + 1) * NXP);
            const double gv = gam[(int64_t)k * NX + i];
            const double r = gv - y;
            r64[(int64_t)k * NX + i] = r;
            rr += r * r;
            gg += gv * gv;
        }
        __syncthreads();
    }
    return ResNorms{rr, gg};
}

// rh = W r on every knot (W_k stored full, zero above the diagonal);
// returns this thread's part of ||rh||^2.
template <typename TM, int BLOCK, int NX>
__device__ __forceinline__ double zt_apply(int N, const TM *__restrict__ Z, const double *__restrict__ r,
                                           double *__restrict__ rh) {
    constexpr int KW = 64 / NX, BS = bstride<TM, NX>(), group = (BLOCK / 64) * KW;
    const int lane = threadIdx.x & 63, kloc = lane / NX, i = lane - kloc * NX;
    const int kme = (threadIdx.x >> 6) * KW + kloc;
    double acc = 0.0;
    __syncthreads();  // r rows come from other threads
    if (kloc < KW) {
        for (int k = kme; k < N; k += group) {
            const TM *zk = Z + (int64_t)k * BS;
            const double *rk = r + (int64_t)k * NX;
            double s0 = 0.0, s1 = 0.0;
#pragma unroll 4
            for (int l = 0; l < NX; l += 2) {
                s0 += (double)zk[i * NX + l] * rk[l];
                s1 += (double)zk[i * NX + l + 1] * rk[l + 1];
            }
            const double s = s0 + s1;
            rh[(int64_t)k * NX + i] = s;
            acc += s * s;
        }
    }
    return acc;
}

// lam += scale * W^T x on every knot.
template <typename TM, typename TI, int BLOCK, int NX>
__device__ __forceinline__ void z_apply_add(int N, const TM *__restrict__ Z, const TI *__restrict__ x, double scale,
                                            double *__restrict__ lam) {
    constexpr int KW = 64 / NX, BS = bstride<TM, NX>(), group = (BLOCK / 64) * KW;
    const int lane = threadIdx.x & 63, kloc = lane / NX, i = lane - kloc * NX;
    const int kme = (threadIdx.x >> 6) * KW + kloc;
    __syncthreads();  // x rows come from other threads
    if (kloc < KW) {
        for (int k = kme; k < N; k += group) {
            const TM *zk = Z + (int64_t)k * BS + i;
            const TI *xk = x + (int64_t)k * NX;
            double s0 = 0.0, s1 = 0.0;
#pragma unroll 4
            for (int l = 0; l < NX; l += 2) {
                s0 += (double)zk[l * NX] * (double)xk[l];
                s1 += (double)zk[(l + 1) * NX] * (double)xk[l + 1];
            }
            lam[(int64_t)k * NX + i] += scale * (s0 + s1);
        }
    }
    __syncthreads();  // lambda rows are read by other threads next
}

template <typename TI>
struct Prob3 {
    int N, max_iter;
    double gnorm;
    const TI *B3;  // D (packed), L, D^-1 (packed) per knot: the true residual reads D and L
    const float *SDlo, *SLlo;
    const TI *OH, *Z;
    double *lam, *r64, *rh64;
    const double *gam;
    Vecs3<TI> v;
};

struct Outcome3 {
    int st = kOk, total = 0, steps = 0;
    bool fallback = false, pc_fallback = false;
    double rnorm = 0.0;
};

// What an inner solve leaves: iterations and status (its solution is the Ops' own).
struct InnerEnd {
    int it, ist;
};

// The refinement loop.  Ops: residual() forms r = gamma - S lambda in FP64 (into q.r64) and returns this thread's
// parts of ||r||^2 and ||gamma||^2; to_scaled(r) forms rh = W r (into q.rh64) and returns its part of ||rh||^2;
// inner(m, hn, tau, budget) solves (I + Oh) d = rh / hn to tau with a polynomial of degree m in at most `budget`
// iterations; add_scaled(hn) adds hn W^T d to lambda.
template <typename TI, int BLOCK, int NX, typename Ops>
__device__ __forceinline__ Outcome3 refine_scaled(const SolveArgs &a, const Prob3<TI> &q, double *red64, Ops &&ops) {
    const int N = q.N, n = N * NX, tid = threadIdx.x;
    Outcome3 o;
    int pending = kOk, base = 0;
    int mcur = a.poly;  // block-Jacobi (m = 0) after a float breakdown of the polynomial
    bool broke = false;
    double prev = INFINITY, gsame = q.gnorm;
    const double *rsrc = q.r64;
    for (;;) {
        if (o.steps == 0 && a.use_lambda0 == 0) {
            rsrc = q.gam;
            o.rnorm = q.gnorm;
        } else {
            ResNorms nr = ops.residual();
            block_sum2<BLOCK>(nr.rr, nr.gg, red64);
            o.rnorm = uniform(sqrt(nr.rr));
            gsame = uniform(sqrt(nr.gg));
            rsrc = q.r64;
        }
        // a warm start is kept only if its residual is strictly below
        // ||gamma||, both norms summed in the same order
        if (o.steps == 0 && a.use_lambda0 == 2 && !(o.rnorm < gsame)) {
            for (int row = tid; row < n; row += BLOCK) q.lam[row] = 0.0;
            o.rnorm = q.gnorm;
            o.fallback = true;
            rsrc = q.gam;
            __syncthreads();
        }
        if (!isfinite(o.rnorm)) {
            o.st = kNonFinite;
            break;
        }
        if (pending != kOk) {
            o.st = pending;
            break;
        }
        if (o.rnorm <= a.tol * q.gnorm) break;
        if (o.steps > 0 && !a.refine) {
            o.st = kInaccurate;
            break;
        }
        if (broke && !(o.rnorm < prev)) {
            o.st = kBreakdown;
            break;
        }
        if (o.steps - base >= a.max_outer) {
            o.st = kMaxIter;
            break;
        }
        prev = o.rnorm;
        double tau = a.theta * a.tol * q.gnorm / o.rnorm;
        if (tau < a.tau_min) tau = a.tau_min;
        if (tau > 1.0) tau = 1.0;

        // the right-hand side in the scaled basis, rh = W r
        double hh = ops.to_scaled(rsrc);
        hh = block_sum<BLOCK>(hh, red64);
        const double hn = uniform(sqrt(hh));
        if (!(hn > 0.0) || !isfinite(hn)) {
            o.st = kNonFinite;
            break;
        }
        const InnerEnd e = ops.inner(mcur, hn, tau, q.max_iter - o.total);
        o.total += e.it;
        ++o.steps;
        ops.add_scaled(hn);
        // under refinement a float breakdown only ends the inner solve; with a
        // polynomial in Oh it also hands the rest of the solve to block-Jacobi
        broke = a.refine && e.ist == kBreakdown;
        if (broke && mcur != 0) {
            mcur = 0;
            o.pc_fallback = true;
            broke = false;
            base = o.steps;
        }
        if (e.ist != kOk && !broke && !(a.refine && e.ist == kBreakdown)) pending = e.ist;
    }
    return o;
}

// One problem from start to status, for state size NX; solve(q) runs the refinement loop.  Every path ends at
// the caller's workgroup barrier (no early return: a divergent-looking exit
// next to the queue's single-thread fetch lets the compiler thread it back
// to the loop head without that fetch).
// ||gamma|| is summed by the first SUM threads.
template <typename TI, int BLOCK, int SUM, int NX, typename F>
__device__ __forceinline__ void run_scaled(const SolveArgs &a, int p, int st_in, double *red64, F &&solve) {
    const int tid = threadIdx.x;
    const int N = a.N[p], n = N * NX;
    const int64_t ob = a.off_blk[p], ov = a.off_v[p];
    Prob3<TI> q;
    q.N = N;
    q.max_iter = a.max_iter > 0 ? a.max_iter : 10 * n;
    q.lam = a.lambda + ov;
    q.gam = a.gamma + ov;
    q.r64 = a.r64 + ov;
    q.rh64 = a.rh64 + ov;
    if (build_failed(st_in)) {
        for (int row = tid; row < n; row += BLOCK) q.lam[row] = 0.0;
        if (tid == 0) {
            a.iters[p] = 0;
            a.outer[p] = 0;
            a.relres[p] = NAN;
        }
    } else {
        q.B3 = (const TI *)a.B3 + a.off_b3[p];
        q.SDlo = a.SDlo ? a.SDlo + a.off_pk[p] : nullptr;
        q.SLlo = a.SLlo ? a.SLlo + ob : nullptr;
        q.OH = (const TI *)a.OH + ob;
        q.Z = (const TI *)a.Z + ob;
        TI *Wk = (TI *)a.work;
        q.v = Vecs3<TI>{Wk + 1 * a.tot_v + ov, Wk + 2 * a.tot_v + ov, Wk + 3 * a.tot_v + ov, Wk + 4 * a.tot_v + ov,
                        Wk + 5 * a.tot_v + ov, Wk + 0 * a.tot_v + ov};
        double gg = 0.0, bad = 0.0;
        if (SUM == BLOCK || tid < SUM)
            for (int row = tid; row < n; row += SUM) {
                const double gv = q.gam[row];
                gg += gv * gv;
                if (a.use_lambda0 == 1) {
                    if (!isfinite(q.lam[row])) bad = 1.0;
                } else if (a.use_lambda0 == 0) {
                    q.lam[row] = 0.0;
                }
            }
        block_sum2<BLOCK>(gg, bad, red64);
        gg = uniform(gg);
        bad = uniform(bad);
        q.gnorm = sqrt(gg);
        Outcome3 o;
        if (!isfinite(q.gnorm) || bad != 0.0) {
            o.st = kNonFinite;
            o.rnorm = NAN;
        } else if (gg == 0.0) {
            for (int row = tid; row < n; row += BLOCK) q.lam[row] = 0.0;
        } else {
            o = solve(q);
        }
        if (tid == 0) {
            a.iters[p] = o.total;
            a.outer[p] = o.steps;
            a.relres[p] = gg == 0.0 ? 0.0 : o.rnorm / q.gnorm;
            a.status[p] = o.st | (o.fallback ? kWarmFallback : 0) | (o.pc_fallback ? kPcFallback : 0);
        }
    }
}

}  // namespace

}  // namespace ssp
