// Learned per-knot warm start: a network with two GELU hidden layers maps
// each knot's stored blocks D_k, L_k (Sec. II-A, Eq. (schur)) and its slice of
// gamma to a guess of that knot's part of lambda.  Inference and training
// (forward, residual loss, backward, Adam) run in these kernels.
//
// Every product is an FP32 GEMM on the matrix cores
// (v_mfma_f32_16x16x4_f32): 32 x 32 output tiles per 256-thread workgroup
// (32 x 64 for the first layer's weight gradient from 256 inputs on), each wave
// one MFMA tile (two), K staged through two LDS buffers 32 at a time.  Operand
// loaders read the network inputs straight from the stored blocks (no feature
// matrix is materialised) and the epilogues fuse bias,
// GELU and its derivative.  Weight gradients reduce over the knots with a
// fixed K split and a fixed-order sum, so training steps are reproducible.
#include <math.h>

#include "ssp_device.h"
#include "ssp_mlp.h"
#include "ssp_sweep.h"

namespace ssp {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int T = 32, BK = 32, GT = 256, PADL = 4;
constexpr int kWideIn = 256;     // inputs from which their weight gradient takes 64 columns per tile
constexpr int kSplitStep = 16;  // K ranges are multiples of this

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }

__device__ __forceinline__ float gelu_grad(float z) {
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * 0.39894228040143268f * expf(-0.5f * z * z);
}

// ---------------------------------------------------------------- loaders ---
// A loader returns element (m, k) of op(A) (0 outside M x K); kFast tells the
// tile loop to walk k fastest (row-major A) or m fastest (column access).

struct RowA {  // A(m, k) = p[m * ld + k]
    static constexpr bool kFast = true;
    const float *p;
    int ld, M, K;
    __device__ float operator()(int m, int k) const { return (m < M && k < K) ? p[(int64_t)m * ld + k] : 0.f; }
};

struct ColA {  // A(m, k) = p[k * ld + m]
    static constexpr bool kFast = false;
    const float *p;
    int ld, M, K;
    __device__ float operator()(int m, int k) const { return (m < M && k < K) ? p[(int64_t)k * ld + m] : 0.f; }
};

struct RowB {  // B(k, n) = p[k * ld + n]
    static constexpr bool kFast = false;
    const float *p;
    int ld, K, N;
    __device__ float operator()(int k, int n) const { return (k < K && n < N) ? p[(int64_t)k * ld + n] : 0.f; }
};

struct ColB {  // B(k, n) = p[n * ld + k]
    static constexpr bool kFast = true;
    const float *p;
    int ld, K, N;
    __device__ float operator()(int k, int n) const { return (k < K && n < N) ? p[(int64_t)n * ld + k] : 0.f; }
};

// Raw input f of knot m: vec D_k (row-major, read from the packed upper
// triangle), then vec L_k (zero at the first knot), then gamma_k.
template <typename TM>
__device__ __forceinline__ float raw_feature(const FeatSrc &s, const KnotInfo &q, int f) {
    const int nn = s.nx * s.nx;
    const TM *B3 = (const TM *)s.B3;
    if (f < nn) {
        const int r = f / s.nx, c = f - r * s.nx;
        return (float)B3[q.blk + packed_index(r, c, s.nx)];
    }
    if (f < 2 * nn) return q.first ? 0.f : (float)B3[q.blk + s.lofs + (f - nn)];
    return (float)s.gamma[q.vec + (f - 2 * nn)];
}

template <typename TM>
struct FeatA {  // A(m, f) = standardised input f of knot m
    static constexpr bool kFast = true;
    FeatSrc s;
    const float *mu, *isd;
    int K;
    __device__ float operator()(int m, int f) const {
        if (m >= s.M || f >= K) return 0.f;
        return (raw_feature<TM>(s, s.ki[m], f) - mu[f]) * isd[f];
    }
};

template <typename TM>
struct FeatAT {  // A(f, m) = standardised input f of knot m (transposed features)
    static constexpr bool kFast = false;
    FeatA<TM> a;
    __device__ float operator()(int f, int m) const { return a(m, f); }
};

// -------------------------------------------------------------- epilogues ---

struct EpStore {  // C[z][m][n] = v  (z: K-split index)
    float *c;
    int ld;
    int64_t zstride;
    __device__ void operator()(int m, int n, int z, float v) const { c[z * zstride + (int64_t)m * ld + n] = v; }
};

struct EpBiasGelu {
    const float *b;
    float *z, *h;
    int ld;
    __device__ void operator()(int m, int n, int, float v) const {
        const float zz = v + b[n];
        if (z) z[(int64_t)m * ld + n] = zz;
        h[(int64_t)m * ld + n] = gelu(zz);
    }
};

struct EpOut {  // network output (+ lambda0 = y_scale * o at the knot's rows)
    const float *b;
    float *o;
    int ld;
    const KnotInfo *ki;
    double *lam;
    float ys;
    __device__ void operator()(int m, int n, int, float v) const {
        const float oo = v + b[n];
        if (o) o[(int64_t)m * ld + n] = oo;
        if (lam) lam[ki[m].vec + n] = (double)(ys * oo);
    }
};

struct EpGeluBack {  // dZ = v * gelu'(Z)
    const float *z;
    float *dz;
    int ld;
    __device__ void operator()(int m, int n, int, float v) const {
        dz[(int64_t)m * ld + n] = v * gelu_grad(z[(int64_t)m * ld + n]);
    }
};

// ------------------------------------------------------------------- GEMM ---
// C = op(A) op(B) over k in [z * kspl, min(K, (z + 1) * kspl)), z = blockIdx.z,
// for a T x TN tile of C per workgroup, each wave a 16 x TN / 2 quarter of it.
// Bound by the latency of its loads (short K ranges, operands gathered an
// element at a time): 32 x 32 tiles, 8 workgroups per CU, beat 64 x 64 ones at
// every size from 2304 to 57600 knots (a step's loss and gradient, nx 14, 2304
// knots: 180 us with 64 x 64 tiles, 131 us; nx 26, 57600 knots: 3.95 and 3.66
// ms).
template <int TN, class AL, class BL, class EP>
__global__ __launch_bounds__(GT) void k_gemm(int M, int N, int K, int kspl, AL al, BL bl, EP ep) {
    __shared__ float As[2][BK][T + PADL];
    __shared__ float Bs[2][BK][TN + PADL];
    constexpr int EA = T * BK / GT, EB = TN * BK / GT, NT = TN / 32;  // elements per thread, MFMA tiles per wave
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int m0 = blockIdx.x * T, n0 = blockIdx.y * TN, z = blockIdx.z;
    const int wm = (w >> 1) * (T / 2), wn = (w & 1) * (TN / 2);
    const int kb = z * kspl, ke = min(K, kb + kspl);
    f32x4 acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // this thread's element e of a tile
    auto at_a = [&](int e, int &mm, int &kk) {
        const int idx = t + GT * e;
        mm = AL::kFast ? idx / BK : idx % T;
        kk = AL::kFast ? idx % BK : idx / T;
    };
    auto at_b = [&](int e, int &nn, int &kk) {
        const int idx = t + GT * e;
        nn = BL::kFast ? idx / BK : idx % TN;
        kk = BL::kFast ? idx % BK : idx / TN;
    };
    // the next tile's elements are fetched before this tile's products and go to the other LDS buffer, one barrier a
    // step: the short K ranges of a training step's products are bound by this latency
    float ra[EA], rb[EB];
    auto load = [&](int k0) {
#pragma unroll
        for (int e = 0; e < EA; ++e) {
            int mm, kk;
            at_a(e, mm, kk);
            ra[e] = (k0 + kk < ke) ? al(m0 + mm, k0 + kk) : 0.f;
        }
#pragma unroll
        for (int e = 0; e < EB; ++e) {
            int nn, kk;
            at_b(e, nn, kk);
            rb[e] = (k0 + kk < ke) ? bl(k0 + kk, n0 + nn) : 0.f;
        }
    };
    load(kb);
    for (int k0 = kb, buf = 0; k0 < ke; k0 += BK, buf ^= 1) {
#pragma unroll
        for (int e = 0; e < EA; ++e) {
            int mm, kk;
            at_a(e, mm, kk);
            As[buf][kk][mm] = ra[e];
        }
#pragma unroll
        for (int e = 0; e < EB; ++e) {
            int nn, kk;
            at_b(e, nn, kk);
            Bs[buf][kk][nn] = rb[e];
        }
        __syncthreads();  // this buffer is full; the other one's readers passed this barrier a step ago
        if (k0 + BK < ke) load(k0 + BK);
#pragma unroll
        for (int sub = 0; sub < BK / 4; ++sub) {
            const int kr = 4 * sub + (lane >> 4), c = lane & 15;
            const float a = As[buf][kr][wm + c];
#pragma unroll
            for (int j = 0; j < NT; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, Bs[buf][kr][wn + 16 * j + c], acc[j], 0, 0, 0);
        }
    }
    // lane l holds rows 4 (l / 16) + r, column l % 16 of each 16 x 16 tile
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = m0 + wm + 4 * (lane >> 4) + r, n = n0 + wn + 16 * j + (lane & 15);
            if (m < M && n < N) ep(m, n, z, acc[j][r]);
        }
}

// K range of each of about `splits` parts, and their number
int split_length(int K, int splits) {
    const int kspl = (K + splits - 1) / splits;
    return kspl > kSplitStep ? (kspl + kSplitStep - 1) / kSplitStep * kSplitStep : kSplitStep;
}
int split_count(int K, int splits) {
    const int kspl = split_length(K, splits);
    return K > 0 ? (K + kspl - 1) / kspl : 1;
}

template <int TN = 32, class AL, class BL, class EP>
hipError_t gemm(int M, int N, int K, int splits, const AL &al, const BL &bl, const EP &ep, hipStream_t s) {
    if (M <= 0 || N <= 0) return hipSuccess;
    const int nz = split_count(K, splits), kspl = split_length(K, splits);
    hipLaunchKernelGGL((k_gemm<TN, AL, BL, EP>), dim3((M + T - 1) / T, (N + TN - 1) / TN, nz), dim3(GT), 0, s, M, N, K,
                       kspl, al, bl, ep);
    return hipGetLastError();
}

// First layer, z = standardised inputs x W1 + b1, h = gelu(z), for MT knots
// by up to 128 hidden units per workgroup (MT = 64: 4 waves, each 16 knots x
// 128 units as 8 MFMA tiles; MT = 16, for few knots: each wave 16 knots x 32
// units), K in steps of 32 through two LDS buffers.  A
// row's threads gather its raw inputs in turn (a load's lanes on few cache
// lines: these gathers, not the products, bound the kernel), gamma only in
// the last steps, which hold it, through a
// table of input offsets built in LDS at the start (D_k from its packed upper
// triangle, L_k, gamma_k); the step's 32 means and inverse deviations go to
// LDS beside the tile and standardise each A operand as it is read (features
// past nin get inverse deviation 0, so they add nothing; rows past M only
// feed outputs that are not stored).  The next step's loads are issued
// before this step's products, at clamped addresses and without branches,
// so that no wait separates them.
constexpr int kL1N = 128, kL1K = 32;
// Knots up to which MT is 16: 64-knot workgroups give 8192 knots 128 of 256 CUs.  Measured with either, one nx 26
// inference: 2048 knots 167 (MT = 64) and 87 us (16), 8192 knots 190 and 131, 12288 knots 190 and 201; with a row's
// inputs dealt out in turn 4608 knots 86 us (16), 9216 knots 140 (64), and 57600 knots 479 where they took 659.
constexpr int kL1Few = 8192;
constexpr int kFeatL = 1, kFeatG = 2;  // input kinds in the table's top bits (0: D_k)
constexpr int kL1MaxIn = 3136;         // table entries (the static tiles leave room for these)

template <typename TM, int MT>
__global__ __launch_bounds__(GT) void k_layer1(FeatSrc s, const float *__restrict__ W1, const float *__restrict__ b1,
                                               const float *__restrict__ mu, const float *__restrict__ isd, int nin,
                                               int H, float *__restrict__ Z, float *__restrict__ Hout) {
    constexpr int EA = MT / 8, NT = MT / 8;  // inputs per thread and step, tiles per wave
    __shared__ float As[2][kL1K][MT + PADL];
    __shared__ __align__(16) float Bs[2][kL1K][kL1N + PADL];
    __shared__ float Ms[2][2][kL1K];  // mean, inverse deviation of the step's inputs
    __shared__ int foff[kL1MaxIn];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int m0 = blockIdx.x * MT, n0 = blockIdx.y * kL1N;
    const int wr = MT == 64 ? 16 * w : 0, wc = MT == 64 ? 0 : 32 * w;  // this wave's rows and columns of the tile
    const int nx = s.nx, nn = nx * nx;
    for (int f = t; f < nin; f += GT) {
        int v;
        if (f < nn) {
            const int r = f / nx, c = f - r * nx;
            v = packed_index(r, c, nx);
        } else if (f < 2 * nn) {
            v = (kFeatL << 30) | (s.lofs + f - nn);
        } else {
            v = (kFeatG << 30) | (f - 2 * nn);
        }
        foff[f] = v;
    }
    // this thread's A row and its inputs of each step
    constexpr int TR = kL1K / EA;  // threads per row, which take its inputs in turn: a row's loads share cache lines
    const int am = t / TR, aq = t % TR;
    const KnotInfo q = s.ki[min(m0 + am, s.M - 1)];  // rows past M: a valid knot (outputs not stored)
    const TM *src = (const TM *)s.B3 + q.blk;
    const double *gsrc = s.gamma + q.vec;
    // B tile: row t / 8 of the step, columns 4 (t % 8) + 32 c .. + 3; the
    // first 64 threads also fetch the step's scaling (t < 32 means, else
    // inverse deviations)
    const int bk = t >> 3, bn = (t & 7) * 4;
    const int nlast = nin - 1;
    f32x4 acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // the next step's raw loads and their 0/1 weights: combined only when
    // they are stored, so that the loads stay in flight over this step's
    // products.  Both input loads are kept (weighted rather than selected) so
    // that the compiler issues them unconditionally; they read finite inputs
    // at valid addresses.
    TM rd[EA];
    double rg[EA];
    float wd[EA], wg[EA], wb[4], rs, ws;
    f32x4 rb[4];
    auto load = [&](int k0) {
#pragma unroll
        for (int j = 0; j < EA; ++j) {
            const int fc = min(k0 + aq + TR * j, nlast);
            const int e = foff[fc], kind = (int)((unsigned)e >> 30), o = e & 0x3fffffff;
            rd[j] = src[kind == kFeatG ? 0 : o];
            wd[j] = (kind == kFeatG || (kind == kFeatL && q.first)) ? 0.f : 1.f;
            wg[j] = kind == kFeatG ? 1.f : 0.f;
            rg[j] = 0.0;
        }
        if (k0 + kL1K > 2 * nn) {  // only the last steps hold parts of gamma
#pragma unroll
            for (int j = 0; j < EA; ++j) {
                const int e = foff[min(k0 + aq + TR * j, nlast)];
                rg[j] = gsrc[(int)((unsigned)e >> 30) == kFeatG ? e & 0x3fffffff : 0];
            }
        }
        const int kr = k0 + bk;
        const float *wrow = W1 + (int64_t)min(kr, nlast) * H;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int n = n0 + bn + 32 * c;
            rb[c] = *(const f32x4 *)(wrow + min(n, H - 4));
            wb[c] = (kr < nin && n < H) ? 1.f : 0.f;
        }
        const int fs = k0 + (t & 31);
        rs = (t < 32 ? mu : isd)[min(fs, nlast)];
        ws = (t < 32 || fs < nin) ? 1.f : 0.f;
    };
    __syncthreads();  // the input table is complete
    load(0);
    for (int k0 = 0, buf = 0; k0 < nin; k0 += kL1K, buf ^= 1) {
#pragma unroll
        for (int j = 0; j < EA; ++j) As[buf][aq + TR * j][am] = (float)rd[j] * wd[j] + (float)rg[j] * wg[j];
#pragma unroll
        for (int c = 0; c < 4; ++c) *(f32x4 *)&Bs[buf][bk][bn + 32 * c] = rb[c] * wb[c];
        if (t < 64) Ms[buf][t >> 5][t & 31] = rs * ws;
        __syncthreads();  // this buffer is full; the other one's readers are done (they passed this barrier)
        load(k0 + kL1K);  // past nin: clamped addresses, zero scaling
#pragma unroll
        for (int sub = 0; sub < kL1K / 4; ++sub) {
            const int kr = 4 * sub + (lane >> 4), c = lane & 15;
            const float a = (As[buf][kr][wr + c] - Ms[buf][0][kr]) * Ms[buf][1][kr];
#pragma unroll
            for (int j = 0; j < NT; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, Bs[buf][kr][wc + 16 * j + c], acc[j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = m0 + wr + 4 * (lane >> 4) + r, n = n0 + wc + 16 * j + (lane & 15);
            if (m < s.M && n < H) {
                const float z = acc[j][r] + b1[n];
                if (Z) Z[(int64_t)m * H + n] = z;
                Hout[(int64_t)m * H + n] = gelu(z);
            }
        }
}

// ------------------------------------------------------------ small kernels ---

__global__ void k_knot_info(const int32_t *knot_prob, const int64_t *koff, const int32_t *N, const int64_t *off_b3,
                            const int64_t *off_v, const int32_t *list, int64_t g0, int M, int nx, int ks,
                            KnotInfo *out) {
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= M) return;
    const int64_t g = list ? (int64_t)list[m] : g0 + m;
    const int p = knot_prob[g];
    const int k = (int)(g - koff[p]);
    KnotInfo q;
    q.blk = off_b3[p] + (int64_t)k * ks;
    q.vec = off_v[p] + (int64_t)k * nx;
    q.first = k == 0;
    q.last = k == N[p] - 1;
    out[m] = q;
}

// The end of a backward pass: the weight gradients' partial sums over the K ranges (out = sum_z part[z]) and the bias
// gradients, which are the column sums of the three row-major M x n output gradients, all in a fixed order.  The first
// workgroups take the column sums, one wave to 16 columns (lane = column + 16 (row mod 4)), each a serial chain over
// the rows that is bound by the latency of its loads: 128 rows' loads are in flight while the previous 128 are added.
// (2300 rows: 108 us for each of the three with one load in flight, now 12 us for all of this kernel.)
struct GradEnd {
    const float *x[3];  // M x n
    float *sum[3];
    int n[3], first[4];  // columns; first 16-column group of each matrix
    const float *part[3];
    float *out[3];
    int64_t cnt[3];
    int M, nz, sums;  // sums: workgroups of column sums
};

constexpr int kSumRows = 32;  // loads of one lane per batch

// a[q] as a selection: an index would read the kernel's arguments through the vector memory path, from the host
template <typename T>
__device__ __forceinline__ T pick(const T (&a)[3], int q) {
    return q == 2 ? a[2] : q == 1 ? a[1] : a[0];
}

__global__ __launch_bounds__(256) void k_grad_end(GradEnd a) {
    if ((int)blockIdx.x < a.sums) {
        const int g = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)), lane = threadIdx.x & 63;
        if (g >= a.first[3]) return;
        const int q = g >= a.first[2] ? 2 : g >= a.first[1] ? 1 : 0, n = pick(a.n, q);
        const int first = q == 2 ? a.first[2] : q == 1 ? a.first[1] : 0;
        const int col = (g - first) * 16 + (lane & 15), M = a.M;
        const float *x = pick(a.x, q);
        const int ofs = 4 * ((lane >> 4) * n + min(col, n - 1));
        float v[2][kSumRows], s = 0.f;
        // batch b: rows 4 (kSumRows b + e) + lane / 16; buffer loads give zeros for rows past M
        auto load = [&](float(&d)[kSumRows], int b) {
            const int64_t m0 = min((int64_t)4 * kSumRows * b, (int64_t)M);
            const int rows = (int)min((int64_t)4 * kSumRows, M - m0);
            const auto src = __builtin_amdgcn_make_buffer_rsrc((void *)(x + m0 * n), 0, 4 * rows * n, 0x00020000);
#pragma unroll
            for (int e = 0; e < kSumRows; ++e)
                d[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(src, ofs + 16 * e * n, 0, 0));
            __builtin_amdgcn_sched_barrier(0);  // else each load sinks to the add that uses it
        };
        auto add = [&](const float(&d)[kSumRows]) {
#pragma unroll
            for (int e = 0; e < kSumRows; ++e) s += d[e];
        };
        const int batches = (M + 4 * kSumRows - 1) / (4 * kSumRows);
        load(v[0], 0);
        for (int b = 0; b < batches; b += 2) {
            load(v[1], b + 1);
            add(v[0]);
            load(v[0], b + 2);
            add(v[1]);
        }
        const float s1 = __shfl(s, (lane & 15) + 16), s2 = __shfl(s, (lane & 15) + 32),
                    s3 = __shfl(s, (lane & 15) + 48);
        if (lane < 16 && col < n) pick(a.sum, q)[col] = (s + s1) + (s2 + s3);
        return;
    }
    const int64_t c0 = a.cnt[0], c1 = c0 + a.cnt[1], c2 = c1 + a.cnt[2];
    for (int64_t i = (int64_t)(blockIdx.x - a.sums) * 256 + threadIdx.x; i < c2;
         i += (int64_t)(gridDim.x - a.sums) * 256) {
        const int q = i >= c1 ? 2 : i >= c0 ? 1 : 0;
        const int64_t o = i - (q == 2 ? c1 : q == 1 ? c0 : 0);
        const float *part = pick(a.part, q) + o;
        const int64_t cnt = pick(a.cnt, q);
        float s = 0.f;
#pragma unroll 8
        for (int z = 0; z < a.nz; ++z) s += part[z * cnt];
        pick(a.out, q)[o] = s;
    }
}

// Partial sums (x - shift) and (x - shift)^2 over knots for 64 features per
// block column; blockIdx.y strides the knots.  Features f < nin are network
// inputs, f >= nin are label entries lam[vec + f - nin].
template <typename TM>
__global__ __launch_bounds__(256) void k_stats_part(FeatSrc s, const double *lam, int nin, int nf, double *part) {
    __shared__ double r1[4][64], r2[4][64];
    const int c = threadIdx.x & 63, r = threadIdx.x >> 6, f = blockIdx.x * 64 + c;
    double a = 0.0, b = 0.0;
    if (f < nf) {
        auto val = [&](int m) -> double {
            const KnotInfo q = s.ki[m];
            return f < nin ? (double)raw_feature<TM>(s, q, f) : lam[q.vec + (f - nin)];
        };
        const double shift = val(0);
        for (int m = blockIdx.y * 4 + r; m < s.M; m += 4 * gridDim.y) {
            const double d = val(m) - shift;
            a += d;
            b += d * d;
        }
    }
    r1[r][c] = a;
    r2[r][c] = b;
    __syncthreads();
    if (r == 0 && f < nf) {
        part[(int64_t)blockIdx.y * 2 * nf + f] = (r1[0][c] + r1[1][c]) + (r1[2][c] + r1[3][c]);
        part[(int64_t)blockIdx.y * 2 * nf + nf + f] = (r2[0][c] + r2[1][c]) + (r2[2][c] + r2[3][c]);
    }
}

template <typename TM>
__global__ __launch_bounds__(256) void k_stats_final(FeatSrc s, const double *lam, int nin, int nf, int ny,
                                                     const double *part, float *mu, float *isd, float *ys) {
    __shared__ double red[256];
    double lab = 0.0;  // this thread's share of sum over label features of E[x^2]
    for (int f = threadIdx.x; f < nf; f += blockDim.x) {
        double a = 0.0, b = 0.0;
        for (int y = 0; y < ny; ++y) {
            a += part[(int64_t)y * 2 * nf + f];
            b += part[(int64_t)y * 2 * nf + nf + f];
        }
        const KnotInfo q = s.ki[0];
        const double shift = f < nin ? (double)raw_feature<TM>(s, q, f) : lam[q.vec + (f - nin)];
        const double mean_d = a / s.M;
        double var = b / s.M - mean_d * mean_d;
        if (var < 0.0) var = 0.0;
        const double mean = shift + mean_d;
        if (f < nin) {
            mu[f] = (float)mean;
            const double sd = sqrt(var);
            isd[f] = (float)(1.0 / (sd > 1e-6 ? sd : 1e-6));
        } else {
            lab += var + mean * mean;
        }
    }
    red[threadIdx.x] = lab;
    __syncthreads();
    if (threadIdx.x == 0 && nf > nin) {
        double t = 0.0;
        for (int i = 0; i < (int)blockDim.x; ++i) t += red[i];
        *ys = (float)sqrt(t / (nf - nin));
    }
}

// E = ys * O - lam*
__global__ void k_err(const KnotInfo *ki, int M, int nx, const float *O, float ys, const double *lam, float *E) {
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (e >= (int64_t)M * nx) return;
    const int m = (int)(e / nx), i = (int)(e - (int64_t)m * nx);
    E[e] = ys * O[e] - (float)lam[ki[m].vec + i];
}

// Y = scale * S X over whole problems (rows of knot m in X, Y at m * nx);
// part[block] = sum of Y^2 over the block (when part != null).  Bound by the
// latency of its loads: with the state size compiled in (NX > 0) the loads of
// a row go out together (2300 knots of nx 14: 10.9 us a product, now 4.3;
// a step's loss and gradient at 18432 knots of nx 26: 951 and 731 us).
template <typename TM, int NX>
__global__ __launch_bounds__(256) void k_smul(FeatSrc s, const float *X, float scale, float *Y, double *part) {
    __shared__ double red[4];
    const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int nx = NX > 0 ? NX : s.nx;
    double sq = 0.0;
    if (e < (int64_t)s.M * nx) {
        const int m = (int)(e / nx), i = (int)(e - (int64_t)m * nx);
        const KnotInfo q = s.ki[m];
        const TM *B3 = (const TM *)s.B3;
        const TM *Dp = B3 + q.blk;  // D_k packed
        const float *x = X + (int64_t)m * nx;
        float y = 0.f;
#pragma unroll
        for (int j = 0; j < nx; ++j) y += (float)Dp[packed_index(i, j, nx)] * x[j];
        if (!q.first) {
            const TM *Lr = B3 + q.blk + s.lofs + i * nx;  // row i of L_k
#pragma unroll
            for (int j = 0; j < nx; ++j) y += (float)Lr[j] * x[j - nx];
        }
        if (!q.last) {
            const TM *Ln = B3 + s.ki[m + 1].blk + s.lofs;  // column i of L_{k+1}
#pragma unroll
            for (int j = 0; j < nx; ++j) y += (float)Ln[j * nx + i] * x[nx + j];
        }
        y *= scale;
        Y[e] = y;
        sq = (double)y * y;
    }
    if (part) {
        sq = wave_sum(sq);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sq;
        __syncthreads();
        if (threadIdx.x == 0) part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
    }
}

__global__ __launch_bounds__(256) void k_loss_final(const double *part, int n, double scale, double *loss) {
    __shared__ double red[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int i = 0; i < 256; ++i) t += red[i];
        *loss = t * scale;
    }
}

__global__ void k_adam(float *theta, const float *grad, float *m, float *v, int64_t n, float lr, float b1, float b2,
                       float eps, float bc1, float bc2) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float g = grad[i];
        const float mi = b1 * m[i] + (1.f - b1) * g;
        const float vi = b2 * v[i] + (1.f - b2) * g * g;
        m[i] = mi;
        v[i] = vi;
        theta[i] -= lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
    }
}

int grid_for(int64_t n, int block) {
    const int64_t g = (n + block - 1) / block;
    return (int)(g < 65535 ? (g > 0 ? g : 1) : 65535);
}

template <typename TM>
void smul(const FeatSrc &f, const float *X, float scale, float *Y, double *part, int grid, hipStream_t s) {
    switch (f.nx) {
        case 6: hipLaunchKernelGGL((k_smul<TM, 6>), dim3(grid), dim3(256), 0, s, f, X, scale, Y, part); break;
        case 14: hipLaunchKernelGGL((k_smul<TM, 14>), dim3(grid), dim3(256), 0, s, f, X, scale, Y, part); break;
        case 26: hipLaunchKernelGGL((k_smul<TM, 26>), dim3(grid), dim3(256), 0, s, f, X, scale, Y, part); break;
        default: hipLaunchKernelGGL((k_smul<TM, 0>), dim3(grid), dim3(256), 0, s, f, X, scale, Y, part);
    }
}

template <typename TM>
hipError_t forward_t(const FeatSrc &f, const NetView &w, const float *mu, const float *isd, float ys, float *Z1,
                     float *H1, float *Z2, float *H2, float *O, double *lam, hipStream_t s) {
    hipError_t e;
    if (w.nin <= kL1MaxIn && w.H % 4 == 0) {
        const int cols = (w.H + kL1N - 1) / kL1N;
        if (f.M <= kL1Few)
            hipLaunchKernelGGL((k_layer1<TM, 16>), dim3((f.M + 15) / 16, cols), dim3(GT), 0, s, f, w.W1, w.b1, mu,
                               isd, w.nin, w.H, Z1, H1);
        else
            hipLaunchKernelGGL((k_layer1<TM, 64>), dim3((f.M + 63) / 64, cols), dim3(GT), 0, s, f, w.W1, w.b1, mu,
                               isd, w.nin, w.H, Z1, H1);
        if ((e = hipGetLastError())) return e;
    } else {
        FeatA<TM> fa{f, mu, isd, w.nin};
        if ((e = gemm(f.M, w.H, w.nin, 1, fa, RowB{w.W1, w.H, w.nin, w.H}, EpBiasGelu{w.b1, Z1, H1, w.H}, s)))
            return e;
    }
    if ((e = gemm(f.M, w.H, w.H, 1, RowA{H1, w.H, f.M, w.H}, RowB{w.W2, w.H, w.H, w.H}, EpBiasGelu{w.b2, Z2, H2, w.H},
                  s)))
        return e;
    return gemm(f.M, w.nx, w.H, 1, RowA{H2, w.H, f.M, w.H}, RowB{w.W3, w.nx, w.H, w.nx},
                EpOut{w.b3, O, w.nx, f.ki, lam, ys}, s);
}

template <typename TM>
hipError_t backward_t(const FeatSrc &f, const NetView &w, const float *mu, const float *isd, const float *Z1,
                      const float *H1, const float *Z2, const float *H2, const float *dO, float *dZ2, float *dZ1,
                      float *grad, float *split, hipStream_t s) {
    const int M = f.M, H = w.H, nx = w.nx, nin = w.nin;
    float *gW1 = grad, *gb1 = gW1 + (int64_t)nin * H, *gW2 = gb1 + H, *gb2 = gW2 + (int64_t)H * H, *gW3 = gb2 + H,
          *gb3 = gW3 + (int64_t)H * nx;
    // weight gradients over kSplits ranges of the knots, summed at the end with the bias gradients
    GradEnd end{{dZ1, dZ2, dO}, {gb1, gb2, gb3}, {H, H, nx}, {}, {}, {gW1, gW2, gW3},
                {(int64_t)nin * H, (int64_t)H * H, (int64_t)H * nx}, M, split_count(M, kSplits), 0};
    for (int q = 0; q < 3; ++q) {
        end.first[q + 1] = end.first[q] + (end.n[q] + 15) / 16;
        end.part[q] = split;
        split += kSplits * end.cnt[q];
    }
    end.sums = (end.first[3] + 3) / 4;
    auto part = [&](int q, int ld) { return EpStore{(float *)end.part[q], ld, end.cnt[q]}; };
    hipError_t e;
    // layer 3: dW3 = H2^T dO, db3 = colsum dO, dZ2 = (dO W3^T) * gelu'(Z2)
    if ((e = gemm(H, nx, M, kSplits, ColA{H2, H, H, M}, RowB{dO, nx, M, nx}, part(2, nx), s))) return e;
    if ((e = gemm(M, H, nx, 1, RowA{dO, nx, M, nx}, ColB{w.W3, nx, nx, H}, EpGeluBack{Z2, dZ2, H}, s))) return e;
    // layer 2
    if ((e = gemm(H, H, M, kSplits, ColA{H1, H, H, M}, RowB{dZ2, H, M, H}, part(1, H), s))) return e;
    if ((e = gemm(M, H, H, 1, RowA{dZ2, H, M, H}, ColB{w.W2, H, H, H}, EpGeluBack{Z1, dZ1, H}, s))) return e;
    // layer 1 (inputs re-read from the stored blocks)
    FeatAT<TM> ft{FeatA<TM>{f, mu, isd, nin}};
    // 64 columns per tile gather each input half as often; with few inputs (nx 6: 78) that leaves too few workgroups.
    // A step's loss and gradient, 32 and 64 columns, 18432 knots: nx 6 394 and 409 us, nx 14 547 and 536, nx 26 1057
    // and 956.
    const EpStore p0 = part(0, H);
    const RowB z1{dZ1, H, M, H};
    if ((e = nin >= kWideIn ? gemm<64>(nin, H, M, kSplits, ft, z1, p0, s) : gemm(nin, H, M, kSplits, ft, z1, p0, s)))
        return e;
    hipLaunchKernelGGL(k_grad_end, dim3(end.sums + grid_for(end.cnt[0] + end.cnt[1] + end.cnt[2], 256)), dim3(256),
                       0, s, end);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_knot_info(const int32_t *knot_prob, const int64_t *koff, const int32_t *N, const int64_t *off_b3,
                            const int64_t *off_v, const int32_t *list, int64_t g0, int M, int nx, int ks,
                            KnotInfo *out, hipStream_t s) {
    if (M <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_knot_info, dim3((M + 255) / 256), dim3(256), 0, s, knot_prob, koff, N, off_b3, off_v, list,
                       g0, M, nx, ks, out);
    return hipGetLastError();
}

hipError_t launch_feature_stats(const FeatSrc &f, const double *lam, float *mu, float *inv_sd, float *y_scale,
                                double *part, hipStream_t s) {
    if (f.M <= 0) return hipErrorInvalidValue;
    const int nin = 2 * f.nx * f.nx + f.nx, nf = nin + (lam ? f.nx : 0), ny = 64;
    const dim3 g1((nf + 63) / 64, ny);
    if (f.fp32) {
        hipLaunchKernelGGL(k_stats_part<float>, g1, dim3(256), 0, s, f, lam, nin, nf, part);
        hipLaunchKernelGGL(k_stats_final<float>, dim3(1), dim3(256), 0, s, f, lam, nin, nf, ny, part, mu, inv_sd,
                           y_scale);
    } else {
        hipLaunchKernelGGL(k_stats_part<double>, g1, dim3(256), 0, s, f, lam, nin, nf, part);
        hipLaunchKernelGGL(k_stats_final<double>, dim3(1), dim3(256), 0, s, f, lam, nin, nf, ny, part, mu, inv_sd,
                           y_scale);
    }
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const FeatSrc &f, const NetView &w, const float *mu, const float *inv_sd, float y_scale,
                              float *Z1, float *H1, float *Z2, float *H2, float *O, double *lambda, hipStream_t s) {
    if (f.M <= 0) return hipSuccess;
    return f.fp32 ? forward_t<float>(f, w, mu, inv_sd, y_scale, Z1, H1, Z2, H2, O, lambda, s)
                  : forward_t<double>(f, w, mu, inv_sd, y_scale, Z1, H1, Z2, H2, O, lambda, s);
}

hipError_t launch_mlp_loss(const FeatSrc &f, const float *O, float y_scale, const double *lam_star, int nprob,
                           float *E, float *R, float *dO, double *part, double *loss, hipStream_t s) {
    if (f.M <= 0 || nprob <= 0) return hipErrorInvalidValue;
    const int64_t n = (int64_t)f.M * f.nx;
    const int g = (int)((n + 255) / 256);
    hipLaunchKernelGGL(k_err, dim3(g), dim3(256), 0, s, f.ki, f.M, f.nx, O, y_scale, lam_star, E);
    const float back = y_scale * 2.0f / nprob;
    if (f.fp32) {
        smul<float>(f, E, 1.0f, R, part, g, s);
        smul<float>(f, R, back, dO, nullptr, g, s);
    } else {
        smul<double>(f, E, 1.0f, R, part, g, s);
        smul<double>(f, R, back, dO, nullptr, g, s);
    }
    hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(256), 0, s, part, g, 1.0 / nprob, loss);
    return hipGetLastError();
}

hipError_t launch_mlp_backward(const FeatSrc &f, const NetView &w, const float *mu, const float *inv_sd,
                               const float *Z1, const float *H1, const float *Z2, const float *H2, const float *dO,
                               float *dZ2, float *dZ1, float *grad, float *split, hipStream_t s) {
    if (f.M <= 0) return hipErrorInvalidValue;
    return f.fp32 ? backward_t<float>(f, w, mu, inv_sd, Z1, H1, Z2, H2, dO, dZ2, dZ1, grad, split, s)
                  : backward_t<double>(f, w, mu, inv_sd, Z1, H1, Z2, H2, dO, dZ2, dZ1, grad, split, s);
}

hipError_t launch_adam(float *theta, const float *grad, float *m, float *v, int64_t n, float lr, float beta1,
                       float beta2, float eps, float bc1, float bc2, hipStream_t s) {
    hipLaunchKernelGGL(k_adam, dim3(grid_for(n, 256)), dim3(256), 0, s, theta, grad, m, v, n, lr, beta1, beta2, eps,
                       bc1, bc2);
    return hipGetLastError();
}

hipError_t launch_gemm_f32(int M, int N, int K, const float *A, int lda, bool ta, const float *B, int ldb, bool tb,
                           float *C, int ldc, hipStream_t s) {
    const EpStore ep{C, ldc, 0};
    if (!ta && !tb) return gemm(M, N, K, 1, RowA{A, lda, M, K}, RowB{B, ldb, K, N}, ep, s);
    if (!ta && tb) return gemm(M, N, K, 1, RowA{A, lda, M, K}, ColB{B, ldb, K, N}, ep, s);
    if (ta && !tb) return gemm(M, N, K, 1, ColA{A, lda, M, K}, RowB{B, ldb, K, N}, ep, s);
    return gemm(M, N, K, 1, ColA{A, lda, M, K}, ColB{B, ldb, K, N}, ep, s);
}

}  // namespace ssp
