// Scaled solve with the problem held on chip (FP32 storage, state sizes 6, 14, 26).
//
// The same iteration as the streaming solve of pcg3.hip (PCG on I + Oh, the preconditioner q(Oh) by Horner steps,
// single-reduction recurrences, FP64 refinement around it), organised so that a pass does not stream the Oh blocks
// and vectors through HBM.  One workgroup of eight waves owns a CU and a problem; the knots are dealt out in sets of
// four, each wave holds a contiguous range of sets, and the first RS sets of every wave stay in its registers for
// the whole inner solve.  The sets beyond those are read again at each product, forwards for the Horner products and
// backwards for w, so that the last ones read are the first ones needed.  (At nx 26 one in four of these reads hits L2:
// a CU's share of it is 128 KB, the blocks of 144 knots are 390 KB.  The others, 19 GB of the ragged 4096-problem batch's
// solve, come from past it.)  The vectors r, u and w (and p, s and x where they fit) live in LDS.
//
// A set puts knot 4 s + g on lanes 16 g .. 16 g + P - 1 of a wave; lane p holds rows p and (R = 2) p + P of Oh_k.
// The product with v needs, per block, a_k = Oh_k v_{k-1} (row i in one lane: every term is one multiply-add whose
// vector entry is read from the lane that holds it by a DPP row broadcast, no LDS traffic) and c_k = Oh_k^T v_k,
// which belongs to knot k - 1 and needs columns: state sizes 6 and 14 keep a second, column-wise copy of the block in
// registers, at 26 the rows are written to a wave-private LDS buffer and read back by columns, half the columns at a
// time.  (Oh v)_k = a_k + c_{k+1}; c crosses from lane group g + 1 to g by a shuffle, and from a wave's first set to
// the wave before it through LDS, completed after the barrier that ends a product.
//
// What bounds it: issue of the products' multiply-adds (a wave issues one every 8 cycles or so, and registers leave two
// waves per SIMD) and, at 26, the LDS transposition: 28 of 38 thousand cycles of a pass over 144 knots, updates, inner
// products and scalars share the rest; more sets in registers at 26 spill, and a second column-wise copy there gains
// nothing.  Measured, streaming and on chip, 1365 problems of 144 knots: nx 26 5.37 and 3.07 ms, nx 14 1.83 and 1.01
// ms; 16 problems of up to 256 knots 3.6 and 1.2 ms with their build.
//
// Rounding: the float arithmetic is that of the streaming solve, term by term.  A row's product sums its even and
// odd terms apart; the inner products are accumulated per lane in the order of the streaming solve's pipeline
// steps and summed by the same trees (dots4), so both solves return the same bits.
#include <math.h>

#include "ssp_device.h"
#include "ssp_fused.h"
#include "ssp_host.h"
#include "ssp_scaled.h"
#include "ssp_sweep.h"

namespace ssp {

namespace {

#pragma clang fp contract(off)

constexpr int kSet = 4;

// P lanes of a 16-lane group hold the rows of a knot, R rows per lane, RS sets per wave stay in registers; DUAL:
// with a column-wise copy.  S, G: row and knot stride of the transposing buffer, in floats (S odd and G = 16 mod 64
// put the writes by rows and the reads by columns of a wave on distinct banks).
template <int NX>
struct Geo4;
template <>
struct Geo4<26> {
    static constexpr int W = 8, P = 13, R = 2, RS = 1, S = 13, G = 400;
    static constexpr bool DUAL = false;
};
template <>
struct Geo4<14> {
    static constexpr int W = 8, P = 14, R = 1, RS = 4, S = 15, G = 272;
    static constexpr bool DUAL = true;
};
template <>
struct Geo4<6> {
    static constexpr int W = 8, P = 6, R = 1, RS = 5, S = 7, G = 80;
    static constexpr bool DUAL = true;
};

template <int NX>
constexpr int waves4() { return Geo4<NX>::W; }
template <int NX>
constexpr int block4() { return 64 * Geo4<NX>::W; }
template <int NX>
constexpr int scratch4() { return (3 * Geo4<NX>::G + NX * Geo4<NX>::S + 3) & ~3; }  // floats per wave

// LDS of a problem of N knots in floats: the transposing buffers, the waves' boundary products, nvec vectors of
// 4 ceil(N / 4) knots and the zero knot before the first one.
template <int NX>
__host__ __device__ inline int vec4_floats(int N) { return (((N + kSet - 1) / kSet * kSet + 1) * NX + 3) & ~3; }
template <int NX>
__host__ __device__ inline int64_t lds4_bytes(int N, int nvec) {
    return 4 * (int64_t)(waves4<NX>() * scratch4<NX>() + (waves4<NX>() + 1) * 32) + 4 * (int64_t)nvec * vec4_floats<NX>(N);
}

#define SSP_FMAC_B(s, x, a, l) "v_fmac_f32_dpp " s ", " x ", " a " row_newbcast:" l " row_mask:0xf bank_mask:0xf\n\t"

// s0 += sum of the even terms, s1 += sum of the odd terms of a[0 .. n) x(lane 0 .. n - 1 of the 16-lane group), in
// order (n = 13; O = 1: term 0 is odd).  The sums are written before the last inputs are read (early-clobber operands).
// The leading wait covers a VALU write of x just before (two wait states for a DPP read).
template <int O>
__device__ __forceinline__ void chain13(const float *a, float x, float &s0, float &s1) {
    float &e = O ? s1 : s0, &o = O ? s0 : s1;
    asm("s_nop 1\n\t" SSP_FMAC_B("%0", "%2", "%3", "0") SSP_FMAC_B("%1", "%2", "%4", "1")
            SSP_FMAC_B("%0", "%2", "%5", "2") SSP_FMAC_B("%1", "%2", "%6", "3") SSP_FMAC_B("%0", "%2", "%7", "4")
                SSP_FMAC_B("%1", "%2", "%8", "5") SSP_FMAC_B("%0", "%2", "%9", "6") SSP_FMAC_B("%1", "%2", "%10", "7")
                    SSP_FMAC_B("%0", "%2", "%11", "8") SSP_FMAC_B("%1", "%2", "%12", "9")
                        SSP_FMAC_B("%0", "%2", "%13", "10") SSP_FMAC_B("%1", "%2", "%14", "11")
                            SSP_FMAC_B("%0", "%2", "%15", "12") "s_nop 0"
        : "+&v"(e), "+&v"(o)
        : "v"(x), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]), "v"(a[8]),
          "v"(a[9]), "v"(a[10]), "v"(a[11]), "v"(a[12]));
}
__device__ __forceinline__ void chain14(const float *a, float x, float &s0, float &s1) {
    asm("s_nop 1\n\t" SSP_FMAC_B("%0", "%2", "%3", "0") SSP_FMAC_B("%1", "%2", "%4", "1")
            SSP_FMAC_B("%0", "%2", "%5", "2") SSP_FMAC_B("%1", "%2", "%6", "3") SSP_FMAC_B("%0", "%2", "%7", "4")
                SSP_FMAC_B("%1", "%2", "%8", "5") SSP_FMAC_B("%0", "%2", "%9", "6") SSP_FMAC_B("%1", "%2", "%10", "7")
                    SSP_FMAC_B("%0", "%2", "%11", "8") SSP_FMAC_B("%1", "%2", "%12", "9")
                        SSP_FMAC_B("%0", "%2", "%13", "10") SSP_FMAC_B("%1", "%2", "%14", "11")
                            SSP_FMAC_B("%0", "%2", "%15", "12") SSP_FMAC_B("%1", "%2", "%16", "13") "s_nop 0"
        : "+&v"(s0), "+&v"(s1)
        : "v"(x), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]), "v"(a[8]),
          "v"(a[9]), "v"(a[10]), "v"(a[11]), "v"(a[12]), "v"(a[13]));
}
__device__ __forceinline__ void chain6(const float *a, float x, float &s0, float &s1) {
    asm("s_nop 1\n\t" SSP_FMAC_B("%0", "%2", "%3", "0") SSP_FMAC_B("%1", "%2", "%4", "1")
            SSP_FMAC_B("%0", "%2", "%5", "2") SSP_FMAC_B("%1", "%2", "%6", "3") SSP_FMAC_B("%0", "%2", "%7", "4")
                SSP_FMAC_B("%1", "%2", "%8", "5") "s_nop 0"
        : "+&v"(s0), "+&v"(s1)
        : "v"(x), "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]));
}
#undef SSP_FMAC_B

// sum_j a[j] x_j with x spread over the lane group (x[q]: entries q P + lane), even and odd terms apart.
template <int NX>
__device__ __forceinline__ float dot_bcast(const float (&a)[NX], const float (&x)[Geo4<NX>::R]) {
    float s0 = 0.0f, s1 = 0.0f;
    if constexpr (NX == 26) {
        chain13<0>(a, x[0], s0, s1);
        chain13<1>(a + 13, x[1], s0, s1);
    } else if constexpr (NX == 14) {
        chain14(a, x[0], s0, s1);
    } else {
        chain6(a, x[0], s0, s1);
    }
    return s0 + s1;
}

__device__ __forceinline__ void pin(float v) { asm volatile("" ::"v"(v)); }

template <int NX>
using Rows4 = float[Geo4<NX>::R][NX];

// This lane's place: lane group g (knot 4 s + g of a set), lane p of it, the wave's sets [s0, s1).
struct Place4 {
    int g, p, pc, s0, s1;  // pc: p clamped to a lane that holds rows
    bool on;               // the lane holds rows
};
template <int NX>
__device__ __forceinline__ Place4 place4(int N) {
    constexpr int P = Geo4<NX>::P;
    Place4 z;
    const int lane = threadIdx.x & 63, wv = uniform((int)(threadIdx.x >> 6));
    z.g = lane >> 4;
    z.p = lane & 15;
    z.on = z.p < P;
    z.pc = z.on ? z.p : P - 1;
    const int ns = (N + kSet - 1) / kSet, q = ns / waves4<NX>(), rem = ns - q * waves4<NX>();
    z.s0 = wv * q + min(wv, rem);
    z.s1 = z.s0 + q + (wv < rem ? 1 : 0);
    return z;
}

using ssp::fresh;
__device__ __forceinline__ Place4 fresh(Place4 z) {
    z.g = fresh(z.g);
    z.p = fresh(z.p);
    z.pc = fresh(z.pc);
    return z;
}

// Rows of knot 4 s + g: zero from knot N on, so that its products are zero.
template <int NX>
__device__ __forceinline__ void load_rows4(const float *__restrict__ OH, int s, int N, const Place4 &z, Rows4<NX> &a) {
    constexpr int P = Geo4<NX>::P, R = Geo4<NX>::R, BS = bstride<float, NX>();
    const int k = min(kSet * s + z.g, N - 1);
    const float *blk = OH + (int64_t)k * BS;
    if constexpr (NX == kLaneMajorNx) {  // lane p's rows p and p + P are its 16-byte vectors p, p + P, p + 2 P ...
        float *f = &a[0][0];
        static_for<0, R * NX / 4>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            const f32x4 v = *(const f32x4 *)(blk + 4 * (t * P + z.pc));
            f[4 * t] = v.x;
            f[4 * t + 1] = v.y;
            f[4 * t + 2] = v.z;
            f[4 * t + 3] = v.w;
        });
    } else {
        static_for<0, R>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            static_for<0, NX / 2>([&](auto hc) {
                constexpr int j = 2 * decltype(hc)::value;
                const f32x2 v = *(const f32x2 *)(blk + (z.pc + r * P) * NX + j);
                a[r][j] = v.x;
                a[r][j + 1] = v.y;
            });
        });
    }
    if (kSet * s + kSet > N && kSet * s + z.g >= N) {
        static_for<0, R>([&](auto rc) {
            static_for<0, NX>([&](auto jc) { a[decltype(rc)::value][decltype(jc)::value] = 0.0f; });
        });
    }
}

// Column h P + p of the lane group's block: the rows' entries of columns [h P, h P + P) through the wave's buffer.
template <int NX>
__device__ __forceinline__ void put_cols4(const Rows4<NX> &a, int h, const Place4 &z, float *buf) {
    constexpr int P = Geo4<NX>::P, R = Geo4<NX>::R, S = Geo4<NX>::S, G = Geo4<NX>::G;
    wave_sync();
    static_for<0, R>([&](auto rc) {  // lanes past P write what lane P - 1 writes
        constexpr int r = decltype(rc)::value;
        float *dst = buf + z.g * G + (z.pc + r * P) * S;
        static_for<0, P>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            dst[q] = h == 0 ? a[r][q] : a[r][NX - P + q];
        });
    });
    wave_sync();
}
template <int NX>
__device__ __forceinline__ void get_cols4(float (&c)[NX], const Place4 &z, const float *buf) {
    constexpr int S = Geo4<NX>::S, G = Geo4<NX>::G;
    const float *src = buf + z.g * G + z.pc;
    static_for<0, NX>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        c[j] = src[j * S];
    });
}

// The whole inner solve's state of a wave.
template <int NX>
struct Inner4 {
    static constexpr int P = Geo4<NX>::P, R = Geo4<NX>::R, RS = Geo4<NX>::RS;
    static constexpr bool DUAL = Geo4<NX>::DUAL;
    Rows4<NX> row[RS > 0 ? RS : 1];
    Rows4<NX> col[DUAL && RS > 0 ? RS : 1];
    float p[RS + 1][R], s[RS + 1][R], x[RS + 1][R], r[RS + 1][R];  // recurrence vectors on the held sets' rows
    float un[RS + 1][R], wn[RS + 1][R];                            // u and w there, read ahead of the update
    Place4 z;
    int N;
    const float *OH;
    float *buf;    // this wave's transposing buffer
    float *bound;  // 32 floats per wave: c of the wave's first knot (zero where there is none)
    float cc;

    __device__ __forceinline__ void load() {
        static_for<0, RS>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            if (z.s0 + r < z.s1) {
                load_rows4<NX>(OH, z.s0 + r, N, z, row[r]);
                if constexpr (DUAL) {
                    static_for<0, R>([&](auto hc) {
                        put_cols4<NX>(row[r], decltype(hc)::value, z, buf);
                        get_cols4<NX>(col[r][decltype(hc)::value], z, buf);
                    });
                }
            }
        });
    }

    // v of knot k - 1 and k on this lane's rows, k the lane's knot of set s.
    __device__ __forceinline__ void vectors(const float *v, int s, float (&xm)[R], float (&xk)[R]) const {
        const float *vk = v + (kSet * s + z.g) * NX + z.pc;
        static_for<0, R>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            xm[r] = vk[r * P - NX];
            xk[r] = vk[r * P];
        });
    }
    // a = Oh_k v_{k-1} and c = Oh_k^T v_k from the rows of Oh_k.  BOTH: the columns of both halves are fetched before
    // the row products, which cover the buffer's latency (52 more registers).
    template <bool BOTH>
    __device__ __forceinline__ void products(const Rows4<NX> &a, const float (&xm)[R], const float (&xk)[R],
                                             float (&av)[R], float (&cv)[R]) const {
        if constexpr (R == 1 || BOTH) {
            float c[R][NX];
            static_for<0, R>([&](auto hc) {
                put_cols4<NX>(a, decltype(hc)::value, z, buf);
                get_cols4<NX>(c[decltype(hc)::value], z, buf);
            });
            static_for<0, R>([&](auto rc) { av[decltype(rc)::value] = dot_bcast<NX>(a[decltype(rc)::value], xm); });
            static_for<0, R>([&](auto rc) { cv[decltype(rc)::value] = dot_bcast<NX>(c[decltype(rc)::value], xk); });
        } else {
            static_assert(R <= 2, "two halves");
            float c[NX];
            put_cols4<NX>(a, 0, z, buf);
            get_cols4<NX>(c, z, buf);
            static_for<0, R>([&](auto rc) { av[decltype(rc)::value] = dot_bcast<NX>(a[decltype(rc)::value], xm); });
            cv[0] = dot_bcast<NX>(c, xk);
            put_cols4<NX>(a, 1, z, buf);
            get_cols4<NX>(c, z, buf);
            cv[1] = dot_bcast<NX>(c, xk);
        }
    }

    // A row of the product, written at o: H: h = r - cc t, else w = u + t, t = a + c (c: Oh_{k+1}^T v_{k+1}), b the row
    // of r or u.  Lanes past P repeat lane P - 1; the knots from N on, and c past the last knot, are zero.
    template <bool H>
    __device__ __forceinline__ void finish(float *o, const float (&b)[R], const float (&av)[R],
                                           const float (&cv)[R]) const {
        static_for<0, R>([&](auto rc) {
            constexpr int r = decltype(rc)::value;
            o[r * P] = H ? __builtin_fmaf(-cc, av[r] + cv[r], b[r]) : (b[r] + av[r]) + cv[r];
        });
    }
    __device__ __forceinline__ void put_bound(const float (&cv)[R]) const {
        if (z.g == 0)
            static_for<0, R>([&](auto rc) { bound[(threadIdx.x >> 6) * 32 + decltype(rc)::value * P + z.pc] = cv[decltype(rc)::value]; });
    }

    // out = r - cc Oh v (H) or v + Oh v on the wave's knots, its last one left open: the product of set s gives c of
    // its knots' predecessors, so knot 4 s + 3 (lane group 3) is finished with set s + 1.  H walks the sets forwards,
    // w backwards.  SAME: the row of r is that of v.  open, openb: a and the base row of the wave's last knot, in
    // lane group 3.
    template <bool H, bool SAME>
    __device__ __forceinline__ void product(const float *v, const float *base, float *out, float (&open)[R],
                                            float (&openb)[R]) {
        z = fresh(z);
        const int src = (int)((threadIdx.x + 16) & 63);
        const bool g3 = z.g == 3;
        float *const mine = out + (H && g3 ? -1 : z.g) * NX + z.pc;
        float carry[R], carryb[R];  // H: a and base of the set before (lane group 3); w: c of the set behind
        auto step = [&](int s, const float (&b)[R], const float (&av)[R], const float (&cv)[R]) {
            float sh[R], bm[R], am[R], cm[R];
            // the products stay in wave-uniform code: their broadcasts read lanes that a branch would mask off
            static_for<0, R>([&](auto rc) { pin(av[decltype(rc)::value]), pin(cv[decltype(rc)::value]); });
            static_for<0, R>([&](auto rc) { sh[decltype(rc)::value] = __shfl(cv[decltype(rc)::value], src, 64); });
            if (s == z.s0) put_bound(cv);
            static_for<0, R>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                am[r] = H && g3 ? carry[r] : av[r];
                bm[r] = H && g3 ? carryb[r] : b[r];
                cm[r] = !H && g3 ? carry[r] : sh[r];
                carry[r] = H ? av[r] : sh[r];
                carryb[r] = b[r];
            });
            if (s == (H ? z.s0 : z.s1 - 1)) {
                if (!H)
                    static_for<0, R>([&](auto rc) {
                        open[decltype(rc)::value] = av[decltype(rc)::value];
                        openb[decltype(rc)::value] = b[decltype(rc)::value];
                    });
                if (!g3) finish<H>(mine + s * (kSet * NX), bm, am, cm);
            } else {
                finish<H>(mine + s * (kSet * NX), bm, am, cm);
            }
        };
        static_for<0, R>([&](auto rc) { carry[decltype(rc)::value] = carryb[decltype(rc)::value] = 0.0f; });
        auto base_row = [&](int s, const float (&xk)[R], float (&b)[R]) {
            static_for<0, R>([&](auto rc) {
                constexpr int r = decltype(rc)::value;
                b[r] = SAME ? xk[r] : base[(kSet * s + z.g) * NX + z.pc + r * P];
            });
        };
        auto held = [&]() {
            float xm[RS + 1][R], xk[RS + 1][R], b[RS + 1][R];
            static_for<0, RS>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                if (z.s0 + q < z.s1) {
                    vectors(v, z.s0 + q, xm[q], xk[q]);
                    base_row(z.s0 + q, xk[q], b[q]);
                }
            });
            static_for<0, RS>([&](auto qc) {
                constexpr int q = H ? decltype(qc)::value : RS - 1 - decltype(qc)::value;
                if (z.s0 + q < z.s1) {
                    float av[R], cv[R];
                    if constexpr (DUAL) {
                        static_for<0, R>([&](auto rc) {
                            av[decltype(rc)::value] = dot_bcast<NX>(row[q][decltype(rc)::value], xm[q]);
                            cv[decltype(rc)::value] = dot_bcast<NX>(col[q][decltype(rc)::value], xk[q]);
                        });
                    } else {
                        products<true>(row[q], xm[q], xk[q], av, cv);
                    }
                    step(z.s0 + q, b[q], av, cv);
                }
            });
        };
        auto streamed = [&](int s) {
            Rows4<NX> a;
            load_rows4<NX>(OH, s, N, z, a);
            float xm[R], xk[R], b[R], av[R], cv[R];
            vectors(v, s, xm, xk);
            base_row(s, xk, b);
            products<false>(a, xm, xk, av, cv);
            step(s, b, av, cv);
        };
        if constexpr (H) {
            held();
            for (int s = z.s0 + RS; s < z.s1; ++s) streamed(s);
            static_for<0, R>([&](auto rc) {
                open[decltype(rc)::value] = carry[decltype(rc)::value];
                openb[decltype(rc)::value] = carryb[decltype(rc)::value];
            });
        } else {
            for (int s = z.s1 - 1; s >= z.s0 + RS; --s) streamed(s);
            held();
        }
    }
    // The wave's last knot, once the next wave has left its c (after a barrier).
    template <bool H>
    __device__ __forceinline__ void close(float *out, const float (&open)[R], const float (&openb)[R]) const {
        if (z.s1 == z.s0 || z.g != 3) return;
        float cv[R];
        static_for<0, R>([&](auto rc) { cv[decltype(rc)::value] = bound[((threadIdx.x >> 6) + 1) * 32 + decltype(rc)::value * P + z.pc]; });
        finish<H>(out + (kSet * z.s1 - 1) * NX + z.pc, openb, open, cv);
    }

    __device__ __forceinline__ void fetch(const float *u, const float *w) {
        const Place4 y = fresh(z);
        static_for<0, RS>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            if (z.s0 + q < z.s1) {
                const int k = kSet * (z.s0 + q) + y.g;
                static_for<0, R>([&](auto rc) {
                    constexpr int r_ = decltype(rc)::value;
                    un[q][r_] = u[k * NX + y.pc + r_ * P];
                    wn[q][r_] = w[k * NX + y.pc + r_ * P];
                });
            }
        });
    }

    // The recurrences on this wave's rows (pass 0: the start of the solve, 1: the first update); streamed sets keep
    // p, s, x at pv, sv, xv.  Every load of a set precedes its stores.
    __device__ __forceinline__ void update(int pass, int m, float alpha, float beta, double inv_s, const double *rh,
                                           float *rl, float *u, const float *w, float *pv, float *sv, float *xv) {
        const Place4 y = fresh(z);
        auto rows = [&](int s, const float (&rn)[R]) {
            const int o = (kSet * s + y.g) * NX + y.pc;
            static_for<0, R>([&](auto rc) {
                rl[o + decltype(rc)::value * P] = rn[decltype(rc)::value];
                if (m == 0) u[o + decltype(rc)::value * P] = rn[decltype(rc)::value];
            });
        };
        if (pass == 0) {
            static_for<0, RS>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                if (z.s0 + q < z.s1) {
                    const int k = min(kSet * (z.s0 + q) + y.g, N - 1);
                    static_for<0, R>([&](auto rc) {
                        constexpr int r_ = decltype(rc)::value;
                        const float v = (float)(rh[k * NX + y.pc + r_ * P] * inv_s);
                        r[q][r_] = kSet * (z.s0 + q) + y.g < N ? v : 0.0f;
                        x[q][r_] = p[q][r_] = s[q][r_] = 0.0f;
                    });
                    rows(z.s0 + q, r[q]);
                }
            });
            for (int t = z.s0 + RS; t < z.s1; ++t) {
                const int k = min(kSet * t + y.g, N - 1);
                float rn[R];
                static_for<0, R>([&](auto rc) {
                    constexpr int r_ = decltype(rc)::value;
                    const float v = (float)(rh[k * NX + y.pc + r_ * P] * inv_s);
                    rn[r_] = kSet * t + y.g < N ? v : 0.0f;
                    if (y.on && kSet * t + y.g < N) xv[k * NX + y.pc + r_ * P] = 0.0f;
                });
                rows(t, rn);
            }
            return;
        }
        static_for<0, RS>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            if (z.s0 + q < z.s1) {
                static_for<0, R>([&](auto rc) {
                    constexpr int r_ = decltype(rc)::value;
                    p[q][r_] = pass == 1 ? un[q][r_] : __builtin_fmaf(beta, p[q][r_], un[q][r_]);
                    s[q][r_] = pass == 1 ? wn[q][r_] : __builtin_fmaf(beta, s[q][r_], wn[q][r_]);
                    x[q][r_] = __builtin_fmaf(alpha, p[q][r_], x[q][r_]);
                    r[q][r_] = __builtin_fmaf(-alpha, s[q][r_], r[q][r_]);
                });
                rows(z.s0 + q, r[q]);
            }
        });
        float v[6][R], nx[6][R];
        auto fetch6 = [&](int t, float (&d)[6][R]) {
            const int o = min(kSet * t + y.g, N - 1) * NX + y.pc;
            static_for<0, R>([&](auto rc) {
                constexpr int r_ = decltype(rc)::value;
                d[0][r_] = u[o + r_ * P];
                d[1][r_] = w[o + r_ * P];
                d[2][r_] = pv[o + r_ * P];
                d[3][r_] = sv[o + r_ * P];
                d[4][r_] = xv[o + r_ * P];
                d[5][r_] = rl[o + r_ * P];
            });
        };
        if (z.s0 + RS < z.s1) fetch6(z.s0 + RS, v);
        for (int t = z.s0 + RS; t < z.s1; ++t) {
            if (t + 1 < z.s1) fetch6(t + 1, nx);
            const int o = (kSet * t + y.g) * NX + y.pc;
            const bool real = kSet * t + y.g < N;
            float rr[R];
            static_for<0, R>([&](auto rc) {
                constexpr int r_ = decltype(rc)::value;
                const float pn = pass == 1 ? v[0][r_] : __builtin_fmaf(beta, v[2][r_], v[0][r_]);
                const float sn = pass == 1 ? v[1][r_] : __builtin_fmaf(beta, v[3][r_], v[1][r_]);
                rr[r_] = real ? __builtin_fmaf(-alpha, sn, v[5][r_]) : 0.0f;
                if (y.on && real) {
                    pv[o + r_ * P] = pn;
                    sv[o + r_ * P] = sn;
                    xv[o + r_ * P] = __builtin_fmaf(alpha, pn, v[4][r_]);
                }
            });
            rows(t, rr);
            static_for<0, 6>([&](auto ec) {
                static_for<0, R>([&](auto rc) { v[decltype(ec)::value][decltype(rc)::value] = nx[decltype(ec)::value][decltype(rc)::value]; });
            });
        }
    }
    // x of the wave's knots to global memory (the LDS is needed next).
    __device__ __forceinline__ void put_x(const float *xv, float *out) const {
        static_for<0, RS>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            const int k = kSet * (z.s0 + q) + z.g;
            if (z.s0 + q < z.s1 && z.on && k < N)
                static_for<0, R>([&](auto rc) { out[k * NX + z.p + decltype(rc)::value * P] = x[q][decltype(rc)::value]; });
        });
        if (xv != out)
            for (int t = z.s0 + RS; t < z.s1; ++t) {
                const int k = kSet * t + z.g;
                if (z.on && k < N)
                    static_for<0, R>([&](auto rc) {
                        const int o = k * NX + z.p + decltype(rc)::value * P;
                        out[o] = xv[o];
                    });
            }
    }
};

// The inner products of a pass in the order of the streaming solve: its thread t (256 of them) holds row i of knot
// kme of a step of C knots and adds its knots' terms in order; r.u runs m knots and w.u m + 1 knots behind the
// step.  Threads 0 .. 255 form r.u and r.r, 256 .. 511 w.u; the sums go through the same butterflies and trees.
// Walk4: the places of this thread's terms, `lag` knots behind the steps (a term it does not have is read from the
// zero knot before knot 0: it adds nothing).
template <int NX>
struct Walk4 {
    int first, mid, stride, cnt, last, extra;
    bool in;  // it has terms of the steps between the first and the last
    __device__ __forceinline__ Walk4(int N, int C, int nsteps, int lag, int vt) {
        constexpr int KW = 64 / NX, group = 4 * KW;
        const int lane = vt & 63, kloc = lane / NX, i = lane - kloc * NX, kme = (vt >> 6) * KW + kloc;
        const bool ok = kloc < KW;
        const int lo = nsteps > 1 ? (nsteps - 1) * C - lag : 0, none = i - NX;
        first = ok && kme < (nsteps > 1 ? C - lag : N) ? kme * NX + i : none;
        in = ok && kme < C;
        mid = (C - lag + min(kme, C - 1)) * NX + i;
        stride = C * NX;
        cnt = nsteps - 2;
        last = ok && nsteps > 1 && lo + kme < N ? (lo + kme) * NX + i : none;
        extra = ok && lo + kme + group < N ? (lo + kme + group) * NX + i : none;
    }
    // f(acc, x, y) over the terms, the loads of up to eight terms in flight
    template <typename F>
    __device__ __forceinline__ float sum(const float *x, const float *y, F &&f) const {
        const float x0 = x[first], y0 = y[first], x1 = x[last], y1 = y[last], x2 = x[extra], y2 = y[extra];
        float acc = f(0.0f, x0, y0);
        const float *xm = x + mid, *ym = y + mid;
        for (int c = 0; c < cnt; c += 8) {
            float xv[8], yv[8];
            static_for<0, 8>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                const int o = min(c + q, cnt - 1) * stride;  // uniform
                xv[q] = xm[o];
                yv[q] = ym[o];
            });
            static_for<0, 8>([&](auto qc) {
                constexpr int q = decltype(qc)::value;
                if (c + q < cnt) acc = f(acc, xv[q], yv[q]);
            });
        }
        if (!in) acc = f(0.0f, x0, y0);
        acc = f(acc, x1, y1);
        return f(acc, x2, y2);
    }
};

template <int NX>
__device__ __forceinline__ Dots3<float> dots4(int N, int C, int nsteps, int m, const float *r, const float *u, const float *w,
                                              float *red) {
    const int vt = fresh(threadIdx.x) & 255;
    auto fma3 = [](float acc, float x, float y) { return __builtin_fmaf(x, y, acc); };
    if (threadIdx.x < 256) {
        const Walk4<NX> own(N, C, nsteps, 0, vt);
        float rho = own.sum(r, r, fma3), gam;
        if (m == 0) {  // r.r again, there without a fused multiply-add
            gam = own.sum(r, r, [](float acc, float x, float) {
                const float xx = x * x;
                return acc + xx;
            });
        } else {
            gam = Walk4<NX>(N, C, nsteps, m, vt).sum(r, u, fma3);
        }
        gam = wave_sum(gam);
        rho = wave_sum(rho);
        if ((vt & 63) == 0) {
            red[vt >> 6] = gam;
            red[4 + (vt >> 6)] = rho;
        }
    }
    if (block4<NX>() == 256 || threadIdx.x >= 256) {
        const float del = wave_sum(Walk4<NX>(N, C, nsteps, m + 1, vt).sum(w, u, fma3));
        if ((vt & 63) == 0) red[8 + (vt >> 6)] = del;
    }
    __syncthreads();
    Dots3<float> d{red[0], red[8], red[4]};
#pragma unroll
    for (int q = 1; q < 4; ++q) {
        d.gam += red[q];
        d.del += red[8 + q];
        d.rho += red[4 + q];
    }
    return Dots3<float>{uniform(d.gam), uniform(d.del), uniform(d.rho)};
}

// One inner PCG solve of (I + Oh) d = rh / ||rh|| (hn) to tau; leaves d in q.v.x.  PL: p, s and x in LDS.
template <int NX, bool PL>
__device__ __forceinline__ InnerEnd inner4(const Prob3<float> &q, int m, int C, float cc, double hn, double tau,
                                               int budget, float *smem, float *red) {
    constexpr int R = Geo4<NX>::R;
    const int N = q.N, nv = vec4_floats<NX>(N), nsteps = (N + C - 1) / C;
    Inner4<NX> in;
    in.z = place4<NX>(N);
    in.N = N;
    in.OH = q.OH;
    in.buf = smem + (threadIdx.x >> 6) * scratch4<NX>();
    in.bound = smem + waves4<NX>() * scratch4<NX>();
    in.cc = cc;
    float *vb = in.bound + (waves4<NX>() + 1) * 32;
    // the zero knot before knot 0, and zeros behind the last one
    for (int e = threadIdx.x; e < (waves4<NX>() + 1) * 32 + 3 * nv; e += block4<NX>()) in.bound[e] = 0.0f;
    float *r = vb + NX, *u = vb + nv + NX, *w = vb + 2 * nv + NX;
    float *pv = PL ? vb + 3 * nv + NX : q.v.p, *sv = PL ? vb + 4 * nv + NX : q.v.s, *xv = PL ? vb + 5 * nv + NX : q.v.x;
    in.load();
    const double inv_s = 1.0 / hn;
    __syncthreads();
    float alpha = 0.0f, beta = 0.0f, gam_prev = 0.0f, bnorm = 0.0f;
    const float tauT = (float)tau;
    InnerEnd o{0, kOk};
    for (int pass = 0;; ++pass) {
        in.update(pass, m, alpha, beta, inv_s, q.rh64, r, u, w, pv, sv, xv);
        __syncthreads();
        float open[R], openb[R];
        for (int j = 1; j <= m; ++j) {
            // h_j lands in u for j = m and in w and u in turn before
            float *hout = ((m - j) & 1) ? w : u;
            if (j == 1)
                in.template product<true, true>(r, r, hout, open, openb);
            else
                in.template product<true, false>(((m - j) & 1) ? u : w, r, hout, open, openb);
            __syncthreads();
            in.template close<true>(hout, open, openb);
            __syncthreads();
        }
        in.template product<false, true>(u, u, w, open, openb);
        __syncthreads();
        in.template close<false>(w, open, openb);
        __syncthreads();
        in.fetch(u, w);
        const Dots3<float> dt = dots4<NX>(N, C, nsteps, m, r, u, w, red);
        if (pass == 0)
            bnorm = sqrtf(dt.rho);
        else
            ++o.it;
        const float rn = sqrtf(dt.rho);
        if (!isfinite(rn)) {
            o.ist = kNonFinite;
            break;
        }
        if (rn <= tauT * bnorm) break;
        if (o.it >= budget) {
            o.ist = kMaxIter;
            break;
        }
        float den;
        if (o.it == 0) {
            den = dt.del;
            beta = 0.0f;
        } else {
            beta = dt.gam / gam_prev;
            const float t = beta * dt.gam / alpha;
            den = dt.del - t;
        }
        if (!(den > 0.0f) || !(dt.gam > 0.0f)) {
            o.ist = (isfinite(den) && isfinite(dt.gam)) ? kBreakdown : kNonFinite;
            break;
        }
        alpha = dt.gam / den;
        gam_prev = dt.gam;
    }
    if constexpr (PL) in.put_x(xv, q.v.x);
    else in.put_x(q.v.x, q.v.x);
    return o;
}

// ---- the refinement loop's FP64 steps: each wave streams a few knots' blocks at a time through its share of the
// LDS, the next knots' loads in flight while it computes (one latency per item otherwise bounds these steps).

// A contiguous chunk of nvec 16-byte vectors by one wave; surplus slots read the first vector again.
template <int NV>
__device__ __forceinline__ void wave_load(const float *src, int nvec, f32x4 (&v)[NV]) {
    const int lane = threadIdx.x & 63;
    static_for<0, NV>([&](auto mc) {
        const int e = lane + 64 * decltype(mc)::value;
        v[decltype(mc)::value] = *(const f32x4 *)(src + 4 * (e < nvec ? e : 0));
    });
}

template <int NX>
constexpr int block_floats4() { return kSet * bstride<float, NX>(); }
template <int NX>
constexpr int kw4() { return 64 / NX; }  // knots per wave of the residual
template <int NX>
constexpr int dl4() {  // floats of D (packed) and L of a knot
    return (NX * (NX + 1) / 2 + 3) / 4 * 4 + bstride<float, NX>();
}
template <int NX>
__host__ __device__ constexpr int wave_bytes4() {  // LDS share of a wave
    constexpr int t = 4 * block_floats4<NX>() + 8 * kSet * NX;
    constexpr int r = 8 * kw4<NX>() * dl4<NX>() + 8 * ((kw4<NX>() + 1) * NX + 1);
    return ((t > r ? t : r) + 15) & ~15;
}

// The blocks of a set of W_k in flight: walks sets wave, wave + waves4<NX>(), ...
template <int NX>
struct SetStream4 {
    static constexpr int BS = bstride<float, NX>(), NV = (kSet * BS / 4 + 63) / 64;
    f32x4 v[NV];
    const float *Z;
    int N, nvec;
    __device__ __forceinline__ void load(int s) {
        nvec = min(kSet, N - kSet * s) * (BS / 4);
        wave_load<NV>(Z + (int64_t)kSet * s * BS, nvec, v);
    }
    __device__ __forceinline__ void store(float *buf) const {
        static_for<0, NV>([&](auto mc) {
            const int e = (threadIdx.x & 63) + 64 * decltype(mc)::value;
            if (e < nvec) *(f32x4 *)(buf + 4 * e) = v[decltype(mc)::value];
        });
    }
};

// Sums of f64 rows in the streaming solve's order: its thread t (256 of them; the others add nothing) adds rows
// next() one after another, up to eight loads in flight.
template <typename G, typename F>
__device__ __forceinline__ void ordered_rows(G &&next, F &&add) {
    if (threadIdx.x >= 256) return;
    for (;;) {
        int o[8];
        static_for<0, 8>([&](auto ec) { o[decltype(ec)::value] = next(); });
        add(o);
        if (o[7] < 0) return;
    }
}

template <int NX>
struct Ops4 {
    static constexpr int P = Geo4<NX>::P, R = Geo4<NX>::R, BS = bstride<float, NX>();
    const SolveArgs &a;
    const Prob3<float> &q;
    float *smem, *red;

    __device__ __forceinline__ Place4 place() const {
        Place4 z;
        const int lane = threadIdx.x & 63;
        z.g = lane >> 4;
        z.p = lane & 15;
        z.on = z.p < P;
        z.pc = z.on ? z.p : P - 1;
        z.s0 = uniform((int)(threadIdx.x >> 6));
        z.s1 = (q.N + kSet - 1) / kSet;
        return z;
    }
    __device__ __forceinline__ float *share() const {
        return smem + uniform((int)(threadIdx.x >> 6)) * (wave_bytes4<NX>() / 4);
    }

    // ||x||^2's part of this thread: row i of every 4 KW-th knot
    __device__ __forceinline__ double norm_part(const double *x) const {
        constexpr int KW = 64 / NX;
        const int lane = threadIdx.x & 63, kloc = lane / NX, i = lane - kloc * NX;
        int k = (threadIdx.x >> 6) * KW + kloc;
        if (kloc >= KW) k = q.N;
        double acc = 0.0;
        ordered_rows([&] { const int o = k < q.N ? k * NX + i : -1; k += 4 * KW; return o; }, [&](const int (&o)[8]) {
            double v[8];
            static_for<0, 8>([&](auto ec) { v[decltype(ec)::value] = x[o[decltype(ec)::value] < 0 ? 0 : o[decltype(ec)::value]]; });
            static_for<0, 8>([&](auto ec) {
                constexpr int e = decltype(ec)::value;
                if (o[e] >= 0) acc = __builtin_fma(v[e], v[e], acc);
            });
        });
        return acc;
    }

    // rh = W r (W_k full, zero above the diagonal)
    __device__ __forceinline__ double to_scaled(const double *r) const {
        const Place4 z = place();
        float *buf = share();
        double *rb = (double *)(buf + block_floats4<NX>());
        const int N = q.N;
        double rv[R];
        SetStream4<NX> st;
        st.Z = q.Z;
        st.N = N;
        auto fetch = [&](int s) {
            st.load(s);
            const double *src = r + (int64_t)min(kSet * s + z.g, N - 1) * NX + z.pc;
            static_for<0, R>([&](auto rc) { rv[decltype(rc)::value] = src[decltype(rc)::value * P]; });
        };
        __syncthreads();  // r comes from other threads
        if (z.s0 < z.s1) fetch(z.s0);
        for (int s = z.s0; s < z.s1; s += waves4<NX>()) {
            wave_sync();
            st.store(buf);
            if (z.on) static_for<0, R>([&](auto rc) { rb[z.g * NX + z.p + decltype(rc)::value * P] = rv[decltype(rc)::value]; });
            wave_sync();
            if (s + waves4<NX>() < z.s1) fetch(s + waves4<NX>());
            const int k = kSet * s + z.g;
            static_for<0, R>([&](auto rc) {
                constexpr int r_ = decltype(rc)::value;
                const float *w = buf + z.g * BS + (z.pc + r_ * P) * NX;
                double s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int j = 0; j < NX; j += 2) {
                    const f32x2 wv = *(const f32x2 *)(w + j);
                    const f64x2 x = *(const f64x2 *)(rb + z.g * NX + j);
                    s0 = __builtin_fma((double)wv.x, x.x, s0);
                    s1 = __builtin_fma((double)wv.y, x.y, s1);
                }
                const double t = s0 + s1;
                if (z.on && k < N) q.rh64[(int64_t)k * NX + z.p + r_ * P] = t;
            });
        }
        __syncthreads();
        return norm_part(q.rh64);
    }

    // lambda += hn W^T x
    __device__ __forceinline__ void add_scaled(double hn) const {
        const Place4 z = place();
        float *buf = share(), *xb = buf + block_floats4<NX>();
        const int N = q.N;
        float xv[R];
        double lv[R];
        SetStream4<NX> st;
        st.Z = q.Z;
        st.N = N;
        auto fetch = [&](int s) {
            st.load(s);
            const int64_t o = (int64_t)min(kSet * s + z.g, N - 1) * NX + z.pc;
            static_for<0, R>([&](auto rc) {
                xv[decltype(rc)::value] = q.v.x[o + decltype(rc)::value * P];
                lv[decltype(rc)::value] = q.lam[o + decltype(rc)::value * P];
            });
        };
        __syncthreads();  // x comes from other threads
        if (z.s0 < z.s1) fetch(z.s0);
        for (int s = z.s0; s < z.s1; s += waves4<NX>()) {
            wave_sync();
            st.store(buf);
            double lam[R];
            static_for<0, R>([&](auto rc) {
                lam[decltype(rc)::value] = lv[decltype(rc)::value];
                if (z.on) xb[z.g * NX + z.p + decltype(rc)::value * P] = xv[decltype(rc)::value];
            });
            wave_sync();
            if (s + waves4<NX>() < z.s1) fetch(s + waves4<NX>());
            const int k = kSet * s + z.g;
            static_for<0, R>([&](auto rc) {
                constexpr int r_ = decltype(rc)::value;
                const float *w = buf + z.g * BS + z.pc + r_ * P;
                double s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int j = 0; j < NX; j += 2) {
                    const f32x2 x = *(const f32x2 *)(xb + z.g * NX + j);
                    s0 = __builtin_fma((double)w[j * NX], (double)x.x, s0);
                    s1 = __builtin_fma((double)w[(j + 1) * NX], (double)x.y, s1);
                }
                if (z.on && k < N) q.lam[(int64_t)k * NX + z.p + r_ * P] = __builtin_fma(hn, s0 + s1, lam[r_]);
            });
        }
        __syncthreads();  // lambda rows are read by other threads next
    }

    // r = gamma - S lambda, S from D (packed), L and their FP32 remainders.  First y_k = D_k lambda_k +
    // L_k lambda_{k-1} and c_k = L_k^T lambda_k (for row k - 1) knot by knot, then the rows of r.
    __device__ __forceinline__ ResNorms residual() const {
        constexpr int KW = kw4<NX>(), DL = dl4<NX>(), VH = DL / 4, NV = (KW * VH + 63) / 64, BP = DL - BS;
        constexpr int KS = 2 * BP + BS;
        const int lane = threadIdx.x & 63, kloc = lane / NX, i = lane - kloc * NX, wv = uniform((int)(threadIdx.x >> 6));
        float *buf = share();  // hi and remainder of an entry side by side
        double *win = (double *)(buf + 2 * KW * DL);  // lambda of knots k0 - 1 .. k0 + KW - 1
        const int N = q.N, ng = (N + KW - 1) / KW, n = N * NX;
        double *y = q.r64, *cb = q.rh64;
        f32x4 hi[NV], lo[NV];
        double lv[2];
        auto fetch = [&](int gi) {
            const int k0 = gi * KW, nvec = min(KW, N - k0) * VH;
            static_for<0, NV>([&](auto mc) {
                constexpr int m = decltype(mc)::value;
                int v = lane + 64 * m;
                if (v >= nvec) v = 0;
                const int kk = v / VH, e = 4 * (v - kk * VH);
                const int64_t k = k0 + kk;
                hi[m] = *(const f32x4 *)(q.B3 + k * KS + e);
                lo[m] = *(const f32x4 *)(e < BP ? q.SDlo + k * BP + e : q.SLlo + k * BS + (e - BP));
            });
            static_for<0, 2>([&](auto mc) {
                const int o = (k0 - 1) * NX + lane + 64 * decltype(mc)::value;
                lv[decltype(mc)::value] = q.lam[o < 0 ? 0 : o < n ? o : n - 1];
            });
        };
        __syncthreads();  // lambda rows were just written by other threads
        if (wv < ng) fetch(wv);
        for (int gi = wv; gi < ng; gi += waves4<NX>()) {
            wave_sync();
            static_for<0, NV>([&](auto mc) {
                constexpr int m = decltype(mc)::value;
                const int v = lane + 64 * m;
                if (v < KW * VH) {
                    *(f32x4 *)(buf + 8 * v) = f32x4{hi[m].x, lo[m].x, hi[m].y, lo[m].y};
                    *(f32x4 *)(buf + 8 * v + 4) = f32x4{hi[m].z, lo[m].z, hi[m].w, lo[m].w};
                }
            });
            static_for<0, 2>([&](auto mc) {
                const int o = lane + 64 * decltype(mc)::value;
                if (o < (KW + 1) * NX) win[o] = lv[decltype(mc)::value];
            });
            wave_sync();
            if (gi + waves4<NX>() < ng) fetch(gi + waves4<NX>());
            const int k = gi * KW + kloc;
            if (kloc < KW && k < N) {
                const float *D = buf + 2 * kloc * DL, *L = D + 2 * BP;
                const double *lk = win + (kloc + 1) * NX, *lm = win + kloc * NX;
                const int ri = packed_row(i, NX);
                double d0 = 0.0, d1 = 0.0, a0 = 0.0, a1 = 0.0, c0 = 0.0, c1 = 0.0;
                auto sum2 = [](f32x2 v) { return (double)v.x + (double)v.y; };
#pragma unroll 4
                for (int j = 0; j < NX; j += 2) {
                    const double x0 = lk[j], x1 = lk[j + 1];
                    // the column part of the row (j < i) and the row part apart
                    const double v0 = sum2(*(const f32x2 *)(D + 2 * (j < i ? packed_row(j, NX) + i : ri + j)));
                    const double v1 = sum2(*(const f32x2 *)(D + 2 * (j + 1 < i ? packed_row(j + 1, NX) + i : ri + j + 1)));
                    d0 = __builtin_fma(v0, j < i ? x0 : 0.0, d0);
                    d1 = __builtin_fma(v0, j < i ? 0.0 : x0, d1);
                    d0 = __builtin_fma(v1, j + 1 < i ? x1 : 0.0, d0);
                    d1 = __builtin_fma(v1, j + 1 < i ? 0.0 : x1, d1);
                    const f32x4 l = *(const f32x4 *)(L + 2 * (i * NX + j));
                    a0 = __builtin_fma((double)l.x + (double)l.y, lm[j], a0);
                    a1 = __builtin_fma((double)l.z + (double)l.w, lm[j + 1], a1);
                    c0 = __builtin_fma(sum2(*(const f32x2 *)(L + 2 * (j * NX + i))), x0, c0);
                    c1 = __builtin_fma(sum2(*(const f32x2 *)(L + 2 * ((j + 1) * NX + i))), x1, c1);
                }
                const int64_t o = (int64_t)k * NX + i;
                y[o] = k > 0 ? (d0 + d1) + (a0 + a1) : d0 + d1;
                if (k > 0) cb[o - NX] = c0 + c1;
            }
        }
        __syncthreads();  // the products come from every wave
        constexpr int B = 4;
        for (int row = threadIdx.x; row < n; row += B * block4<NX>()) {
            double yv[B], cv[B], gv[B];
            static_for<0, B>([&](auto bc) {
                constexpr int b = decltype(bc)::value;
                const int o = min(row + b * block4<NX>(), n - 1);
                yv[b] = y[o];
                cv[b] = cb[min(o, max(n - NX - 1, 0))];
                gv[b] = q.gam[o];
            });
            static_for<0, B>([&](auto bc) {
                constexpr int b = decltype(bc)::value;
                const int o = row + b * block4<NX>();
                if (o < n) y[o] = gv[b] - (o < n - NX ? yv[b] + cv[b] : yv[b]);
            });
        }
        __syncthreads();
        // both norms over the rows of the streaming solve's steps of a.res_knots knots
        ResNorms nr{0.0, 0.0};
        constexpr int group = 4 * KW;
        const int kme = wv * KW + kloc, C = a.res_knots;
        int k0 = kloc < KW ? 0 : N, kk = kme;
        ordered_rows(
            [&] {
                while (k0 < N && kk >= min(C, N - k0)) {
                    k0 += C;
                    kk = kme;
                    if (kme >= C) k0 = N;
                }
                const int o = k0 < N ? (k0 + kk) * NX + i : -1;
                kk += group;
                return o;
            },
            [&](const int (&o)[8]) {
                double rv[8], gv[8];
                static_for<0, 8>([&](auto ec) {
                    constexpr int e = decltype(ec)::value;
                    rv[e] = y[o[e] < 0 ? 0 : o[e]];
                    gv[e] = q.gam[o[e] < 0 ? 0 : o[e]];
                });
                static_for<0, 8>([&](auto ec) {
                    constexpr int e = decltype(ec)::value;
                    if (o[e] >= 0) {
                        nr.rr = __builtin_fma(rv[e], rv[e], nr.rr);
                        nr.gg = __builtin_fma(gv[e], gv[e], nr.gg);
                    }
                });
            });
        return nr;
    }

    __device__ __forceinline__ InnerEnd inner(int m, double hn, double tau, int budget) const {
        const float cc = (float)a.pc_c;
        if (lds4_bytes<NX>(q.N, 6) <= a.lds_bytes)
            return inner4<NX, true>(q, m, a.step_knots, cc, hn, tau, budget, smem, red);
        return inner4<NX, false>(q, m, a.step_knots, cc, hn, tau, budget, smem, red);
    }
};

}  // namespace

// Persistent grid over the problems order[0 .. nprob) of state size NX: workgroups take them from the device queue
// until it is empty (see k_pcg3 for the scalar reads).
template <int NX>
__global__ __launch_bounds__(block4<NX>(), 2) void k_pcg4(SolveArgs a) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double red64[2 * waves4<NX>()];
    __shared__ float red[12];
    __shared__ int s_next;
    if (threadIdx.x == 0) s_next = (int)atomicAdd(a.queue, 1u);
    __syncthreads();
    int qi = __builtin_amdgcn_readfirstlane(s_next);
    while (qi < a.nprob) {
        const int p = __builtin_amdgcn_readfirstlane(a.order[qi]);
        const int nx = __builtin_amdgcn_readfirstlane(a.nx[p]);
        const int st_in = __builtin_amdgcn_readfirstlane(a.status[p]);
        const int N = __builtin_amdgcn_readfirstlane(a.N[p]);
        if (nx == NX && lds4_bytes<NX>(N, 3) <= a.lds_bytes && waves4<NX>() * wave_bytes4<NX>() <= a.lds_bytes) {
            run_scaled<float, block4<NX>(), 256, NX>(a, p, st_in, red64, [&](const Prob3<float> &q) {
                const Ops4<NX> ops{a, q, (float *)smem_raw, red};
                return refine_scaled<float, block4<NX>(), NX>(a, q, red64, ops);
            });
        } else if (threadIdx.x == 0) {  // the host queues only problems that fit
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

const void *pcg4_kernel(int nx) {
    switch (nx) {
        case 6: return (const void *)k_pcg4<6>;
        case 14: return (const void *)k_pcg4<14>;
        case 26: return (const void *)k_pcg4<26>;
    }
    return nullptr;
}

}  // namespace

template <int NX>
static int64_t need4(int N, int nvec) {
    if (N > 1 << 20) return INT64_MAX;  // far past any LDS, and vec4_floats overflows further on
    const int64_t v = lds4_bytes<NX>(N, nvec);
    constexpr int o = waves4<NX>() * wave_bytes4<NX>();
    return v > o ? v : o;
}

int64_t pcg4_lds(int nx, int N, bool all_vectors) {
    const int nvec = all_vectors ? 6 : 3;
    switch (nx) {
        case 6: return need4<6>(N, nvec);
        case 14: return need4<14>(N, nvec);
        case 26: return need4<26>(N, nvec);
    }
    return -1;
}

hipError_t launch_pcg4(const SolveArgs &a, int nx, hipStream_t s) {
    if (a.nprob == 0) return hipSuccess;
    const void *f = pcg4_kernel(nx);
    if (!f) return hipErrorInvalidValue;
    const int block = nx == 6 ? block4<6>() : nx == 14 ? block4<14>() : block4<26>();
    // the LDS opt-in and the CU count once per kernel and device (no runtime query of either inside a graph capture after
    // the first eager solve)
    static PerDevice cus[3];
    PerDevice &known = cus[nx == 6 ? 0 : nx == 14 ? 1 : 2];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    int n = known.get(dev);
    if (n == 0) {
        if ((e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kLds4Cap)) != hipSuccess) return e;
        if ((e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
        known.set(dev, n);
    }
    // workgroups that fit a CU together: by registers (two waves per SIMD) and LDS
    const int by_lds = 160 * 1024 / (a.lds_bytes + 256), by_reg = 512 / block;
    n *= by_lds < by_reg ? by_lds : by_reg;
    SolveArgs arg = a;
    void *args[] = {(void *)&arg};
    e = hipLaunchKernel(f, dim3(n < a.nprob ? n : a.nprob), dim3(block), args, (size_t)a.lds_bytes, s);
    return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace ssp
