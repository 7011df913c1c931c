// Batched PCG in the block-Jacobi congruence basis, one persistent grid.
//
// With D_k = C_k C_k^T (Cholesky) and W_k = C_k^-1, the congruence
// W S W^T = I + Oh (W = blockdiag(W_k)) has identity diagonal blocks and the
// off-diagonal blocks Oh_k = W_k L_k W_{k-1}^T (below) and Oh_k^T (above),
// with O = S - D and W O W^T = Oh; D^-1 = W^T W.  The preconditioners of the
// paper become polynomials in Oh:
//   block-Jacobi (Eq. (jacobi)):          D^-1                 = W^T W,
//   symmetric stair (Sec. IV):            D^-1 - D^-1 O D^-1   = W^T (I - Oh) W,
//   additive stair (Sec. III):            D^-1 - D^-1 O D^-1/2 = W^T (I - Oh/2) W,
//   Neumann polynomial of degree m (Eq. (polynomial_precon), Psi = D,
//   P = D - S = -O):  sum_{i<=m} (D^-1 P)^i D^-1 = W^T (sum_{i<=m} (-Oh)^i) W
// (the stair identities are those of Eq. (stair_inv) with S = Psi_l + Psi_r - D).
// PCG on S lambda = gamma with Phi^-1 = W^T q(Oh) W is therefore PCG on
// (I + Oh) lh = W gamma with the preconditioner q(Oh) and lambda = W^T lh:
// the same iterates in exact arithmetic, with residuals rh = W r.  Each PCG
// pass streams Oh_k only (nx^2 elements per knot instead of D_k, L_k and
// D_k^-1), and the float operator I + Oh is as well conditioned as
// block-Jacobi-preconditioned S, whatever the conditioning of the D_k.
//
// The refinement loop stays in the original basis: each outer step forms the
// true residual r = gamma - S lambda in FP64 from D, L (hi + lo), maps it to
// rh = W r, runs the float PCG on (I + Oh) d = rh / ||rh|| (stopping on the
// recurrence residual in the scaled basis) and adds ||rh|| W^T d to lambda in
// FP64.  FP64 storage runs the same loop in FP64 (further outer steps restart
// the FP64 iteration from the true residual).
//
// Per pass the single-reduction recurrences of the fused kernel are used:
//   p = u + beta p, s = w + beta s, x += alpha p, r -= alpha s,
//   u = q(Oh) r, w = (I + Oh) u, gamma = r.u, delta = w.u, rho = r.r,
// with u by Horner, h_0 = r, h_j = r - c Oh h_{j-1} (j = 1..m), u = h_m.  The
// pass walks the knots in steps of C: step c updates the lead knots [k0, k1)
// and writes r into window 0, computes h_j j knots behind the lead (Oh couples
// neighbours) and w m + 1 knots behind; the last step drains the tail.  The
// Oh blocks of a step arrive in registers (16-byte loads issued one step
// ahead) and are stored into an LDS ring.
//
// Scheduling: one launch for the whole ragged batch.  Workgroups take
// problems from a device queue ordered by decreasing work N nx^2, so the long
// problems start first and the short ones fill in at the end; each problem
// runs the code compiled for its state size.
#include <math.h>

#include "ssp_device.h"
#include "ssp_fused.h"
#include "ssp_host.h"
#include "ssp_scaled.h"
#include "ssp_sweep.h"

namespace ssp {

namespace {

// 16-byte prefetch registers per thread: one step of the largest step the
// wave mapping allows (capped; the LDS budget may shorten the step further)
template <typename TM, int BLOCK, int NX>
constexpr int pf3_slots() {
    constexpr int n = (max_step<BLOCK, NX>() * bstride<TM, NX>() / vlen<TM>() + BLOCK - 1) / BLOCK;
    constexpr int cap = sizeof(TM) == 4 ? 12 : 8;
    return n < cap ? n : cap;
}

// Knots per step for an LDS budget: the Oh ring and m + 1 vector windows
// (r, h_1 .. h_{m-1}, u) of R = C + m + 2 slots each, plus a 16-byte spot.
template <typename TM, int BLOCK, int NX>
__host__ __device__ inline int knots3(int lds_bytes, int m) {
    int C = max_step<BLOCK, NX>();
    const int Cp = pf3_slots<TM, BLOCK, NX>() * BLOCK * vlen<TM>() / bstride<TM, NX>();
    if (Cp < C) C = Cp;
    const int per = (bstride<TM, NX>() + (m + 1) * vstride<TM, NX>()) * (int)sizeof(TM);
    const int Cl = (lds_bytes - 16) / per - (m + 2);
    if (Cl < C) C = Cl;
    return C;
}

template <typename TM, int BLOCK, int NX>
__host__ __device__ inline int lds3_for(int C, int m) {
    return (C + m + 2) * (bstride<TM, NX>() + (m + 1) * vstride<TM, NX>()) * (int)sizeof(TM) + 16;
}

// The six recurrence vectors of a problem of N knots stay in the
// workgroup's LDS, behind the pass's ring, windows and spare spot, when
// they fit in the budget: the passes then stream only the Oh blocks from
// HBM.  Returns their byte offset in the dynamic LDS, or -1 if they do not
// fit.  Compiled for the small state sizes only (at nx 26 a budget that
// keeps three workgroups per CU holds no horizon of the workloads).
template <typename TM, int BLOCK, int NX>
__host__ __device__ inline int vectors3_offset(int N, int lds_bytes, int m) {
    if constexpr (NX > 14) {
        return -1;
    } else {
        const int C = knots3<TM, BLOCK, NX>(lds_bytes, m);
        if (C < 1) return -1;
        const int off = (lds3_for<TM, BLOCK, NX>(C, m) + 15) & ~15;
        return (int64_t)off + 6 * (int64_t)N * NX * (int64_t)sizeof(TM) <= lds_bytes ? off : -1;
    }
}

// Register prefetch of one step: the step's Oh blocks (one contiguous chunk,
// 16-byte loads, surplus slots re-read the first vector so that every load is
// unconditional) and the six recurrence vectors of this thread's lead row
// (the init pass: the FP64 right-hand side of that row instead).
template <typename TM, int BLOCK, int NX>
struct Prefetch3 {
    using VT = typename Vec16<TM>::T;
    static constexpr int V = Vec16<TM>::V;
    static constexpr int BS = bstride<TM, NX>();
    static constexpr int kPF = pf3_slots<TM, BLOCK, NX>();
    VT reg[kPF];
    TM vec[6];
    double res = 0;

    __device__ __forceinline__ void issue(const TM *OH, int k0, int kc, bool init, int lead_row, const double *rhs,
                                          const Vecs3<TM> vs) {
        const int nvec = kc * BS / V;
        const VT *src = (const VT *)(OH + (int64_t)k0 * BS);
        static_for<0, kPF>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            int q = threadIdx.x + m * BLOCK;
            if (q >= nvec) q = 0;
            reg[m] = src[q];
        });
        const int row = lead_row >= 0 ? lead_row : 0;
        if (init) {
            res = rhs[row];
        } else {
            vec[0] = vs.u[row];
            vec[1] = vs.w[row];
            vec[2] = vs.p[row];
            vec[3] = vs.s[row];
            vec[4] = vs.x[row];
            vec[5] = vs.r[row];
        }
    }

    // chunk -> ring slots sb, sb + 1, ... (mod R); surplus vectors (a
    // partial slot, or whole slots of a short step) go to the 16-byte spot
    // `dummy`.  Every register is stored on every path, so the next issue
    // finds no load still pending on them and need not wait for memory.
    __device__ __forceinline__ void store(TM *ring, int kc, int sb, int R, TM *dummy) const {
        const int nvec = kc * BS / V;
        const int wrap = R * BS, base = sb * BS;
        static_for<0, kPF>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            const int q = threadIdx.x + m * BLOCK;
            int off = base + q * V;
            if (off >= wrap) off -= wrap;
            *(VT *)(q < nvec ? ring + off : dummy) = reg[m];
        });
    }
};

// Row i (COL: column i) of a block of Oh as stored times x: even and odd terms apart, in order.
template <typename TM, int NX, bool COL>
__device__ __forceinline__ TM oh_dot(const TM *__restrict__ blk, int i, const TM *__restrict__ x) {
    if constexpr (!lane_major<TM, NX>()) {
        return lean_dot<NX, COL>(blk, i, x);
    } else {
        // The lane-major order, read as it lies in the ring.  A pass is bound by the latency of its steps and its LDS
        // accesses: with the rows put back in order at the store (two 8-byte writes for each 16-byte load) 256 problems of
        // 350 to 400 knots took 6.00 ms, so they take 5.18 (5.81 with blocks stored by rows); 1365 of 32 to 256 5.20,
        // 5.02 (5.05).
        constexpr int H = NX / 2, T = 4 * H;
        TM s0 = TM(0), s1 = TM(0);
        if constexpr (COL) {
            // entries (r, i) and (r + H, i), r < H: 4 r past these two
            const TM *top = blk + lane_major_place<NX>(0, i), *low = blk + lane_major_place<NX>(H, i);
#pragma unroll 3
            for (int j = 0; j + 2 < H; j += 2) {
                const f32x2 v = *(const f32x2 *)(x + j);
                s0 += top[4 * j] * v.x;
                s1 += top[4 * j + 4] * v.y;
            }
            {
                const f32x2 v = *(const f32x2 *)(x + H - 1);
                s0 += top[4 * H - 4] * v.x;
                s1 += low[0] * v.y;
            }
#pragma unroll 3
            for (int j = 1; j + 1 < H; j += 2) {
                const f32x2 v = *(const f32x2 *)(x + H + j);
                s0 += low[4 * j] * v.x;
                s1 += low[4 * j + 4] * v.y;
            }
        } else {
            // entries (i, 4 t), (i, 4 t + 1) and (i, 4 t + 2), (i, 4 t + 3): T t past these two
            const TM *a = blk + lane_major_place<NX>(i, 0), *b = blk + lane_major_place<NX>(i, 2);
#pragma unroll 2
            for (int t = 0; t < NX / 4; ++t) {
                const f32x2 v = *(const f32x2 *)(x + 4 * t), w = *(const f32x2 *)(x + 4 * t + 2);
                const f32x2 c = *(const f32x2 *)(a + T * t), d = *(const f32x2 *)(b + T * t);
                s0 += c.x * v.x;
                s1 += c.y * v.y;
                s0 += d.x * w.x;
                s1 += d.y * w.y;
            }
            static_assert(NX % 4 == 2, "one pair more");
            const f32x2 v = *(const f32x2 *)(x + NX - 2), c = *(const f32x2 *)(a + T * (NX / 4));
            s0 += c.x * v.x;
            s1 += c.y * v.y;
        }
        return s0 + s1;
    }
}

// Workgroup sums of a pass's partial inner products (fixed-order trees; in
// FP64 under the FP64-accumulation option, then rounded to the storage type).
template <typename TI, int BLOCK>
__device__ __forceinline__ Dots3<TI> reduce_dots(Dots3<TI> dt, bool acc64, double *red64, TI *redT) {
    if (acc64) {
        block_sum2<BLOCK>(dt.g64, dt.d64, red64);
        dt.r64 = block_sum<BLOCK>(dt.r64, red64 + 2 * (BLOCK / kWave));
        return Dots3<TI>{uniform((TI)dt.g64), uniform((TI)dt.d64), uniform((TI)dt.r64)};
    }
    block_sum2<BLOCK>(dt.gam, dt.del, redT);
    dt.rho = block_sum<BLOCK>(dt.rho, redT + 2 * (BLOCK / kWave));
    return Dots3<TI>{uniform(dt.gam), uniform(dt.del), uniform(dt.rho)};
}

struct Geo3 {
    int N, C, R, m;  // knots, knots per step, ring slots, Horner steps
    bool acc64;      // accumulate the inner products in FP64
};

// One pass over the knots (see the file comment).  init: the pass that starts
// an inner solve (r = rhs * inv_s, x = 0); first: the first update pass
// (p = u, s = w).
template <typename TI, int BLOCK, int NX>
__device__ __forceinline__ Dots3<TI> scaled_pass(const Geo3 &g, bool init, bool first, TI alpha, TI beta, TI cc,
                                                 double inv_s, const double *__restrict__ rhs,
                                                 const TI *__restrict__ OH, const Vecs3<TI> v, TI *smem) {
    constexpr int W = BLOCK / 64, KW = 64 / NX, BS = bstride<TI, NX>(), NXP = vstride<TI, NX>();
    const int N = g.N, C = g.C, R = g.R, m = g.m;
    TI *ring = smem;             // R slots of BS
    TI *win = ring + R * BS;     // window j (R slots of NXP) at win + j R NXP: 0 = r, m = u
    TI *dummy = win + (m + 1) * R * NXP;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int kloc = lane / NX, i = lane - kloc * NX;
    const bool lane_ok = kloc < KW;
    const int kme = wv * KW + kloc, group = W * KW;
    Dots3<TI> d{TI(0), TI(0), TI(0)};

    Prefetch3<TI, BLOCK, NX> pf;
    const int nsteps = (N + C - 1) / C;
    auto lead_row = [&](int k0, int kc) { return (lane_ok && kme < kc) ? (k0 + kme) * NX + i : -1; };
    pf.issue(OH, 0, min(C, N), init, lead_row(0, min(C, N)), rhs, v);
    int sb = 0;  // ring slot of knot k0
    for (int c = 0; c < nsteps; ++c) {
        const int k0 = c * C, kc = min(C, N - k0), k1 = k0 + kc;
        const bool last = k1 == N;
        __syncthreads();  // every reader of the slots refilled below is done
        pf.store(ring, kc, sb, R, dummy);
        TI cur[6];
#pragma unroll
        for (int e = 0; e < 6; ++e) cur[e] = pf.vec[e];
        const double res = pf.res;
        if (!last) pf.issue(OH, k1, min(C, N - k1), init, lead_row(k1, min(C, N - k1)), rhs, v);

        // A: recurrence updates on the lead rows, r into window 0
        if (lane_ok && kme < kc) {
            const int row = (k0 + kme) * NX + i;
            TI r;
            if (init) {
                r = (TI)(res * inv_s);
                v.x[row] = TI(0);
            } else {
                const TI pv = first ? cur[0] : cur[0] + beta * cur[2];
                const TI sv = first ? cur[1] : cur[1] + beta * cur[3];
                v.p[row] = pv;
                v.s[row] = sv;
                v.x[row] = cur[4] + alpha * pv;
                r = cur[5] - alpha * sv;
            }
            v.r[row] = r;
            win[slot_of(sb, kme, R) * NXP + i] = r;
            const TI rr = r * r;
            if (g.acc64)
                d.r64 += (double)rr;
            else
                d.rho += rr;
            if (m == 0) {  // block-Jacobi: u = r
                v.u[row] = r;
                if (g.acc64)
                    d.g64 += (double)rr;
                else
                    d.gam += rr;
            }
        }
        __syncthreads();  // ring blocks and window 0 come from every wave

        // H_j: h_j = r - c Oh h_{j-1}, j knots behind the lead
        for (int j = 1; j <= m; ++j) {
            const TI *hin = win + (j - 1) * R * NXP;
            TI *hout = win + j * R * NXP;
            const int lo = max(k0 - j, 0), hi = last ? N : k1 - j;
            for (int kk = kme; kk < hi - lo; kk += group) {
                if (!lane_ok) break;
                const int k = lo + kk, dk = k - k0;
                const int s = slot_of(sb, dk, R);
                TI t = TI(0);
                if (k > 0) t += oh_dot<TI, NX, false>(ring + s * BS, i, hin + slot_of(sb, dk - 1, R) * NXP);
                if (k + 1 < N) {
                    const int sp = slot_of(sb, dk + 1, R);
                    t += oh_dot<TI, NX, true>(ring + sp * BS, i, hin + sp * NXP);
                }
                const TI rk = win[s * NXP + i];
                const TI h = rk - cc * t;
                hout[s * NXP + i] = h;
                if (j == m) {
                    if (g.acc64)
                        d.g64 += (double)(rk * h);
                    else
                        d.gam += rk * h;
                    v.u[k * NX + i] = h;
                }
            }
            __syncthreads();
        }

        // W: w = u + Oh u, m + 1 knots behind the lead
        {
            const TI *u = win + m * R * NXP;
            const int lo = max(k0 - m - 1, 0), hi = last ? N : k1 - m - 1;
            for (int kk = kme; kk < hi - lo; kk += group) {
                if (!lane_ok) break;
                const int k = lo + kk, dk = k - k0;
                const int s = slot_of(sb, dk, R);
                const TI uk = u[s * NXP + i];
                TI w = uk;
                if (k > 0) w += oh_dot<TI, NX, false>(ring + s * BS, i, u + slot_of(sb, dk - 1, R) * NXP);
                if (k + 1 < N) {
                    const int sp = slot_of(sb, dk + 1, R);
                    w += oh_dot<TI, NX, true>(ring + sp * BS, i, u + sp * NXP);
                }
                if (g.acc64)
                    d.d64 += (double)(w * uk);
                else
                    d.del += w * uk;
                v.w[k * NX + i] = w;
            }
        }
        sb += C;
        if (sb >= R) sb -= R;
    }
    return d;
}

// The steps of the refinement loop.
template <typename TI, int BLOCK, int NX>
struct Ops3 {
    const SolveArgs &a;
    const Prob3<TI> &q;
    const Geo3 g;
    const Vecs3<TI> vv;
    unsigned char *smem_raw;
    double *red64;
    TI *redT;

    __device__ __forceinline__ ResNorms residual() const {
        return residual_lean<TI, BLOCK, NX>(g.N, residual3_knots<TI, NX>(a.lds_bytes), q.B3, q.SDlo, q.SLlo, q.lam,
                                            q.gam, q.r64, (double *)smem_raw);
    }
    __device__ __forceinline__ double to_scaled(const double *r) const {
        return zt_apply<TI, BLOCK, NX>(g.N, q.Z, r, q.rh64);
    }
    __device__ __forceinline__ void add_scaled(double hn) const {
        z_apply_add<TI, TI, BLOCK, NX>(g.N, q.Z, vv.x, hn, q.lam);
    }
    __device__ __forceinline__ InnerEnd inner(int mcur, double hn, double tau, int budget) const {
        const TI cc = (TI)a.pc_c;
        Geo3 gc = g;
        gc.m = mcur;
        gc.R = g.C + mcur + 2;
        int it = 0, ist = kOk;
        Dots3<TI> dt = scaled_pass<TI, BLOCK, NX>(gc, true, false, TI(0), TI(0), cc, 1.0 / hn, q.rh64, q.OH, vv,
                                                  (TI *)smem_raw);
        dt = reduce_dots<TI, BLOCK>(dt, gc.acc64, red64, redT);
        const TI bnorm = sqrt(dt.rho);
        const TI tauT = (TI)tau;
        TI gam_prev = TI(0), alpha = TI(0), beta = TI(0);
        for (;;) {
            const TI rn = sqrt(dt.rho);
            if (!isfinite(rn)) {
                ist = kNonFinite;
                break;
            }
            if (rn <= tauT * bnorm) break;
            if (it >= budget) {
                ist = kMaxIter;
                break;
            }
            TI den;
            if (it == 0) {
                den = dt.del;
                beta = TI(0);
            } else {
                beta = dt.gam / gam_prev;
                den = dt.del - beta * dt.gam / alpha;
            }
            if (!(den > TI(0)) || !(dt.gam > TI(0))) {
                ist = (isfinite(den) && isfinite(dt.gam)) ? kBreakdown : kNonFinite;
                break;
            }
            alpha = dt.gam / den;
            gam_prev = dt.gam;
            dt = scaled_pass<TI, BLOCK, NX>(gc, false, it == 0, alpha, beta, cc, 0.0, q.rh64, q.OH, vv,
                                            (TI *)smem_raw);
            dt = reduce_dots<TI, BLOCK>(dt, gc.acc64, red64, redT);
            ++it;
        }
        return InnerEnd{it, ist};
    }
};

// VL: the recurrence vectors live in LDS (vectors3_offset), a separate
// instantiation so that the compiler sees LDS pointers there and global
// pointers in the other (a pointer that may be either would turn every
// access into a flat one, whose waits also hold the LDS traffic).
template <typename TI, int BLOCK, int NX, bool ACC, bool VL>
__device__ __forceinline__ Outcome3 solve_scaled(const SolveArgs &a, const Prob3<TI> &q, unsigned char *smem_raw,
                                                 double *red64, TI *redT) {
    const int N = q.N, n = N * NX;
    Geo3 g;
    g.N = N;
    g.m = a.poly;
    g.acc64 = ACC;
    g.C = knots3<TI, BLOCK, NX>(a.lds_bytes, g.m);
    g.R = g.C + g.m + 2;
    Vecs3<TI> vv = q.v;
    if constexpr (VL) {
        TI *vb = (TI *)(smem_raw + vectors3_offset<TI, BLOCK, NX>(N, a.lds_bytes, g.m));
        vv = Vecs3<TI>{vb + 1 * n, vb + 2 * n, vb + 3 * n, vb + 4 * n, vb + 5 * n, vb};
    }
    const Ops3<TI, BLOCK, NX> ops{a, q, g, vv, smem_raw, red64, redT};
    return refine_scaled<TI, BLOCK, NX>(a, q, red64, ops);
}

// One problem from start to status, for state size NX.
template <typename TI, int BLOCK, int NX, bool ACC>
__device__ __forceinline__ void run_problem3(const SolveArgs &a, int p, int st_in, unsigned char *smem_raw,
                                             double *red64, TI *redT) {
    run_scaled<TI, BLOCK, BLOCK, NX>(a, p, st_in, red64, [&](const Prob3<TI> &q) {
        if (vectors3_offset<TI, BLOCK, NX>(q.N, a.lds_bytes, a.poly) >= 0)
            return solve_scaled<TI, BLOCK, NX, ACC, NX <= 14>(a, q, smem_raw, red64, redT);
        return solve_scaled<TI, BLOCK, NX, ACC, false>(a, q, smem_raw, red64, redT);
    });
}

}  // namespace

// Persistent solve of every problem: workgroups take queue positions from a
// device counter until the queue is empty (every workgroup reaches the exit
// test after each problem).
// The queue position, problem, state size and incoming status are read
// into scalar registers (readfirstlane), so every branch on them is uniform
// for the compiler too: each workgroup barrier is then reached the same
// number of times by every wave.
// One persistent grid for the problems of one compiled state size NX (a
// kernel instance per size keeps each size's register allocation to
// itself).  ACC: sum the inner products in FP64 (the option; FP32 storage
// only).
template <typename TI, int BLOCK, int NX, bool ACC>
__global__ __launch_bounds__(BLOCK, 3) void k_pcg3(SolveArgs a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double red64[3 * (BLOCK / kWave)];
    __shared__ TI redT[3 * (BLOCK / kWave)];
    __shared__ int s_next;
    if (threadIdx.x == 0) s_next = (int)atomicAdd(a.queue, 1u);
    __syncthreads();
    int qi = __builtin_amdgcn_readfirstlane(s_next);
    while (qi < a.nprob) {
        const int p = __builtin_amdgcn_readfirstlane(a.order[qi]);
        const int nx = __builtin_amdgcn_readfirstlane(a.nx[p]);
        const int st_in = __builtin_amdgcn_readfirstlane(a.status[p]);
        if (nx == NX) {
            run_problem3<TI, BLOCK, NX, ACC>(a, p, st_in, smem_raw, red64, redT);
        } else if (threadIdx.x == 0) {  // the host queues only problems of this size
            a.status[p] = kNonFinite;
            a.relres[p] = NAN;
            a.iters[p] = 0;
            a.outer[p] = 0;
        }
        __syncthreads();  // the problem is done: s_next, the LDS and the reduction scratch are free
        if (threadIdx.x == 0) s_next = (int)atomicAdd(a.queue, 1u);
        __syncthreads();
        qi = __builtin_amdgcn_readfirstlane(s_next);
    }
}

namespace {

template <typename TI>
int knots3_rt(int nx, int threads, int lds_bytes, int m) {
    switch (threads * 100 + nx) {
        case 25606: return knots3<TI, 256, 6>(lds_bytes, m);
        case 25614: return knots3<TI, 256, 14>(lds_bytes, m);
        case 25626: return knots3<TI, 256, 26>(lds_bytes, m);
        case 25636: return knots3<TI, 256, 36>(lds_bytes, m);
        case 12806: return knots3<TI, 128, 6>(lds_bytes, m);
        case 12814: return knots3<TI, 128, 14>(lds_bytes, m);
        case 12826: return knots3<TI, 128, 26>(lds_bytes, m);
        case 12836: return knots3<TI, 128, 36>(lds_bytes, m);
    }
    return 0;
}

template <typename TI>
int lds3_rt(int nx, int threads, int m) {
    int C = knots3_rt<TI>(nx, threads, 1 << 30, m);
    if (C < 1) return 0;
    switch (threads * 100 + nx) {
        case 25606: return lds3_for<TI, 256, 6>(C, m);
        case 25614: return lds3_for<TI, 256, 14>(C, m);
        case 25626: return lds3_for<TI, 256, 26>(C, m);
        case 25636: return lds3_for<TI, 256, 36>(C, m);
        case 12806: return lds3_for<TI, 128, 6>(C, m);
        case 12814: return lds3_for<TI, 128, 14>(C, m);
        case 12826: return lds3_for<TI, 128, 26>(C, m);
        case 12836: return lds3_for<TI, 128, 36>(C, m);
    }
    return 0;
}

template <typename TI, int BLOCK, bool ACC>
const void *pcg3_fn(int nx) {
    switch (nx) {
        case 6: return (const void *)k_pcg3<TI, BLOCK, 6, ACC>;
        case 14: return (const void *)k_pcg3<TI, BLOCK, 14, ACC>;
        case 26: return (const void *)k_pcg3<TI, BLOCK, 26, ACC>;
        case 36: return (const void *)k_pcg3<TI, BLOCK, 36, ACC>;
    }
    return nullptr;
}

const void *pcg3_kernel(bool fp32, int threads, bool acc, int nx) {
    if (fp32 && acc) return threads == 128 ? pcg3_fn<float, 128, true>(nx) : pcg3_fn<float, 256, true>(nx);
    if (fp32) return threads == 128 ? pcg3_fn<float, 128, false>(nx) : pcg3_fn<float, 256, false>(nx);
    return threads == 128 ? pcg3_fn<double, 128, false>(nx) : pcg3_fn<double, 256, false>(nx);
}

hipError_t allow_lds(const void *f) {
    hipFuncAttributes fa;
    hipError_t e = hipFuncGetAttributes(&fa, f);
    if (e != hipSuccess) return e;
    return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - (int)fa.sharedSizeBytes);
}

}  // namespace

int pcg3_residual_steps(int nx, bool fp32, int lds_bytes) {
    switch (nx) {
        case 6: return fp32 ? residual3_knots<float, 6>(lds_bytes) : residual3_knots<double, 6>(lds_bytes);
        case 14: return fp32 ? residual3_knots<float, 14>(lds_bytes) : residual3_knots<double, 14>(lds_bytes);
        case 26: return fp32 ? residual3_knots<float, 26>(lds_bytes) : residual3_knots<double, 26>(lds_bytes);
        case 36: return fp32 ? residual3_knots<float, 36>(lds_bytes) : residual3_knots<double, 36>(lds_bytes);
    }
    return 0;
}

template <typename TI>
int onchip3_rt(int nx, int threads, int lds_bytes, int m) {
    // the largest N whose vectors vectors3_offset keeps in LDS (0: none)
    int lo = 0;
    for (int N = 1; N <= 4096; ++N) {
        int off = -1;
        switch (threads * 100 + nx) {
            case 25606: off = vectors3_offset<TI, 256, 6>(N, lds_bytes, m); break;
            case 25614: off = vectors3_offset<TI, 256, 14>(N, lds_bytes, m); break;
            case 12806: off = vectors3_offset<TI, 128, 6>(N, lds_bytes, m); break;
            case 12814: off = vectors3_offset<TI, 128, 14>(N, lds_bytes, m); break;
        }
        if (off < 0) break;
        lo = N;
    }
    return lo;
}

int pcg3_onchip_horizon(int nx, bool fp32, int threads, int lds_bytes, int m) {
    return fp32 ? onchip3_rt<float>(nx, threads, lds_bytes, m) : onchip3_rt<double>(nx, threads, lds_bytes, m);
}

int pcg3_steps_for(int nx, bool fp32, int threads, int lds_bytes, int m) {
    return fp32 ? knots3_rt<float>(nx, threads, lds_bytes, m) : knots3_rt<double>(nx, threads, lds_bytes, m);
}

int pcg3_lds(int nx, bool fp32, int threads, int m) {
    int l = fp32 ? lds3_rt<float>(nx, threads, m) : lds3_rt<double>(nx, threads, m);
    if (l == 0) return 0;
    if (l > kFusedLdsCap) {
        // shrink to the cap
        l = kFusedLdsCap;
        if (pcg3_steps_for(nx, fp32, threads, l, m) < 1) return 0;
    }
    return l;
}

int pcg3_occupancy(bool fp32, int threads, int lds_bytes, int *cus, bool acc, int nx) {
    int dev = 0, n = 0;
    if (cus) *cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    const void *f = pcg3_kernel(fp32, threads, acc, nx);
    if (!f) return 0;
    if (allow_lds(f) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, threads, (size_t)lds_bytes) != hipSuccess) return 0;
    if (cus) {
        hipDeviceProp_t pr;
        if (hipGetDeviceProperties(&pr, dev) != hipSuccess) return 0;
        *cus = pr.multiProcessorCount;
    }
    return n;
}

hipError_t launch_pcg3(const SolveArgs &a, bool fp32, int threads, int nx, int grid, hipStream_t s) {
    if (a.nprob == 0) return hipSuccess;
    if (threads != 128 && threads != 256) return hipErrorInvalidValue;
    const bool acc = fp32 && a.acc64 != 0;
    const void *f = pcg3_kernel(fp32, threads, acc, nx);
    if (!f) return hipErrorInvalidValue;
    // per kernel instance: the LDS opt-in once, and the resident workgroups
    // for an LDS budget queried once per process (no runtime query inside a
    // graph capture after the first eager solve)
    struct Entry {
        const void *f;
        int lds, grid;
    };
    static Entry cache[64];
    static int used = 0, next = 0;
    int hit = -1;
    for (int c = 0; c < used; ++c)
        if (cache[c].f == f && cache[c].lds == a.lds_bytes) hit = c;
    if (hit < 0) {
        hipError_t e = allow_lds(f);
        if (e != hipSuccess) return e;
        int cus = 0;
        const int occ = pcg3_occupancy(fp32, threads, a.lds_bytes, &cus, acc, nx);
        if (occ < 1 || cus < 1) return hipErrorInvalidConfiguration;
        hit = used < 64 ? used++ : (next++ % 64);
        cache[hit] = Entry{f, a.lds_bytes, occ * cus};
    }
    if (grid <= 0) grid = cache[hit].grid;
    if (grid > a.nprob) grid = a.nprob;
    SolveArgs arg = a;
    void *args[] = {(void *)&arg};
    hipError_t e = hipLaunchKernel(f, dim3(grid), dim3(threads), args, (size_t)a.lds_bytes, s);
    return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace ssp
