// Complex FP64 contractions on the matrix cores (v_mfma_f64_16x16x4f64).
//
// Two shapes cover the nonlocal pseudopotential term and the projector onto
// the empty manifold of every (side, k) block:
//   k_gemm_cn:     C[m][n] = sum_k conj(A[m][k]) B[n][k]   (small C, long K;
//                  split over K, partials summed by k_reduce_pair)
//   k_gemm_update: Y[n][k] = os * (Y[n][k] + cs * sum_m C[m][n] A[m][k])
//                  (long output rows, short inner dimension)
// Nonlocal term (Eq. H0_k_plus_q, V_NL with the 2x2 spin D matrix):
//   B = beta^dag x,  W_i = sum_j D_ij B_j,  phi += beta W.
// Projector (Eqs. P_minus_q2 / P_plus_q2):
//   S = O^dag phi,  phi <- sg (phi - O S), sg = -1 on the lower row of L.
// Complex products use four real MFMAs (re*re, im*im, re*im, im*re).
//
// Lane layout of the 16x16x4 MFMAs for wave lane l (measured on gfx950):
// A[l%16][l/16], B[l/16][l%16]; accumulator element v holds
//   FP64 (v_mfma_f64_16x16x4f64): D[4*v + l/16][l%16]
//   FP32 (v_mfma_f32_16x16x4f32): D[4*(l/16) + v][l%16]
// The FP32 variants (single-precision bulk path) round the FP64 operands to
// FP32 on load and accumulate in FP32; partial sums and outputs stay FP64.
#include "tm_internal.h"

namespace tml {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ inline v4d mfma(double a, double b, v4d c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ inline v4f mfma(float a, float b, v4f c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <class R>
struct MF;
template <>
struct MF<double> {
    using V = v4d;
    // output row of accumulator element v for lane group kk = l / 16
    __device__ static int row(int v, int kk) { return 4 * v + kk; }
};
template <>
struct MF<float> {
    using V = v4f;
    __device__ static int row(int v, int kk) { return 4 * kk + v; }
};

// Batches of several right-hand sides: batch b uses the A of b % amod (its
// side and k point); B, C, Y and the partials are per b.
struct GemmCN {
    const double2* const* A_tab;  // per batch b % amod (or null -> A_base + b*a_bstride)
    int amod;
    const double2* A_base;
    long long a_bstride;
    int lda;
    const double2* B_base;        // per batch B_base + b*b_bstride
    long long b_bstride;
    int ldb;
    int M, Nn, K, kchunk, ksplit, nt;
    double2* part;                // [b][ks][M][Nn]
};

__device__ double2 g_zero2;  // zero-initialised, never written
// a complex value as a native vector, and a pointer to one in global memory
// (operands reached through pointer tables would otherwise be read with flat
// loads, which make every wait a wait for all loads, LDS included)
typedef double __attribute__((ext_vector_type(2))) DVec2;
typedef const DVec2 __attribute__((address_space(1))) GlobalD2;

// *p as a global-memory load
__device__ __forceinline__ double2 gload(const double2* p) {
    const DVec2 v = *(const GlobalD2*)p;
    return cmk(v.x, v.y);
}

template <class R>
__global__ void __launch_bounds__(64) k_gemm_cn(GemmCN g) {
    const int b = blockIdx.z, ks = blockIdx.y;
    const int tile = blockIdx.x;
    const int m0 = (tile / g.nt) * 16, n0 = (tile % g.nt) * 16;
    const int l = threadIdx.x, i = l & 15, kk = l >> 4;
    const double2* A = g.A_tab ? g.A_tab[b % g.amod] : g.A_base + (long long)b * g.a_bstride;
    const double2* B = g.B_base + (long long)b * g.b_bstride;
    const int kbeg = ks * g.kchunk;
    const int kend = min(g.K, kbeg + g.kchunk);
    typename MF<R>::V cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
    const bool arow = (m0 + i) < g.M, brow = (n0 + i) < g.Nn;
    const double2* Ap = A + (long long)(m0 + i) * g.lda;
    const double2* Bp = B + (long long)(n0 + i) * g.ldb;
    // KU steps' loads in flight together (global loads, an element outside
    // the operands read from a zero); the products run in step order
    constexpr int KU = 4;
    for (int k = kbeg; k < kend; k += 4 * KU) {
        double2 a[KU], bv[KU];
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const int kx = k + 4 * u + kk;
            a[u] = gload((arow && kx < kend) ? Ap + kx : &g_zero2);
            bv[u] = gload((brow && kx < kend) ? Bp + kx : &g_zero2);
        }
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            if (k + 4 * u < kend) {
                const R ax = (R)a[u].x, ay = (R)a[u].y, bx = (R)bv[u].x, by = (R)bv[u].y;
                cr = mfma(ax, bx, cr);
                cr = mfma(ay, by, cr);
                ci = mfma(ax, by, ci);
                ci = mfma(-ay, bx, ci);
            }
        }
    }
    double2* out = g.part + ((long long)b * g.ksplit + ks) * g.M * g.Nn;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        int m = m0 + MF<R>::row(v, kk), n = n0 + i;
        if (m < g.M && n < g.Nn) out[(long long)m * g.Nn + n] = cmk((double)cr[v], (double)ci[v]);
    }
}

// Small contractions (a few output tiles, K of at most kSmallK): one block
// per (tile, batch); its waves take interleaved K slices of 4 and their
// 16 x 16 accumulators are added in wave order through LDS, so the result
// goes straight to `out` with no partial buffer and no second launch.
constexpr int kSmallWaves = 16;
constexpr int kSmallK = 4096;

template <class R>
__global__ void __launch_bounds__(64 * kSmallWaves) k_gemm_cn_small(GemmCN g, double2* out) {
    __shared__ double2 red[kSmallWaves][256];
    const int b = blockIdx.y, tile = blockIdx.x;
    const int m0 = (tile / g.nt) * 16, n0 = (tile % g.nt) * 16;
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, i = l & 15, kk = l >> 4;
    const double2* A = g.A_tab ? g.A_tab[b % g.amod] : g.A_base + (long long)b * g.a_bstride;
    const double2* B = g.B_base + (long long)b * g.b_bstride;
    typename MF<R>::V cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
    const bool arow = (m0 + i) < g.M, brow = (n0 + i) < g.Nn;
    const double2* Ap = A + (long long)(m0 + i) * g.lda;
    const double2* Bp = B + (long long)(n0 + i) * g.ldb;
    // KU slices a wave's loads are in flight together
    constexpr int KU = 4, KS = 4 * kSmallWaves;
    for (int k0 = 4 * w; k0 < g.K; k0 += KU * KS) {
        double2 a[KU], bv[KU];
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const int kx = k0 + u * KS + kk;
            a[u] = gload((arow && kx < g.K) ? Ap + kx : &g_zero2);
            bv[u] = gload((brow && kx < g.K) ? Bp + kx : &g_zero2);
        }
#pragma unroll
        for (int u = 0; u < KU; ++u) {
            const R ax = (R)a[u].x, ay = (R)a[u].y, bx = (R)bv[u].x, by = (R)bv[u].y;
            cr = mfma(ax, bx, cr);
            cr = mfma(ay, by, cr);
            ci = mfma(ax, by, ci);
            ci = mfma(-ay, bx, ci);
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) red[w][MF<R>::row(v, kk) * 16 + i] = cmk((double)cr[v], (double)ci[v]);
    __syncthreads();
    if (threadIdx.x < 256) {
        const int m = m0 + threadIdx.x / 16, n = n0 + (threadIdx.x & 15);
        double2 sum = red[0][threadIdx.x];
#pragma unroll
        for (int v = 1; v < kSmallWaves; ++v) sum = cadd(sum, red[v][threadIdx.x]);
        if (m < g.M && n < g.Nn) out[((long long)b * g.M + m) * g.Nn + n] = sum;
    }
}

// The same contraction with both operands of a K-chunk staged in LDS: one
// block per (batch, K split) computes every 16x16 output tile from LDS (waves
// take tiles in turn), so each operand element is read from memory once
// instead of once per output tile.  The next chunk's loads are issued before
// the current chunk's products, so memory latency hides behind the MFMAs.
// Needs M, Nn <= 16 * kMaxTiles1D.
constexpr int kCnThreads = 512;
constexpr int kCnChunk = 16;          // K values per LDS chunk
constexpr int kMaxTiles1D = 14;       // M, Nn up to 224
constexpr int kCnTilesPerWave = 7;    // (mt * nt) / 8 waves, at most
constexpr int kCnMaxTilesSum = 16;   // mt + nt, at most
constexpr int kCnStage = kCnMaxTilesSum * 16 * kCnChunk / kCnThreads;  // staged elements per thread

template <class R>
struct LdsC {
    R re, im;
};

template <class R>
__global__ void __launch_bounds__(kCnThreads) k_gemm_cn_lds(GemmCN g, int mt) {
    extern __shared__ double lds_raw[];
    constexpr int LS = kCnChunk + 1;  // padded row
    const int Mp = mt * 16, Np = g.nt * 16;
    LdsC<R>* As = reinterpret_cast<LdsC<R>*>(lds_raw);
    LdsC<R>* Bs = As + Mp * LS;
    const int b = blockIdx.y, ks = blockIdx.x;
    const double2* A = g.A_tab ? g.A_tab[b % g.amod] : g.A_base + (long long)b * g.a_bstride;
    const double2* B = g.B_base + (long long)b * g.b_bstride;
    const int kbeg = ks * g.kchunk;
    const int kend = min(g.K, kbeg + g.kchunk);
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6, i = l & 15, kk = l >> 4;
    const int ntiles = mt * g.nt;
    typename MF<R>::V cr[kCnTilesPerWave], ci[kCnTilesPerWave];
#pragma unroll
    for (int t = 0; t < kCnTilesPerWave; ++t) {
        cr[t] = typename MF<R>::V{0, 0, 0, 0};
        ci[t] = typename MF<R>::V{0, 0, 0, 0};
    }
    // A[0..Mp)[k0..k0+16) and B[0..Np)[k0..k0+16) of one chunk, kCnStage
    // elements per thread; rows past M / Nn and k past the range read as zero
    const int nst = (Mp + Np) * kCnChunk;
    double2 stage[kCnStage];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int j = 0; j < kCnStage; ++j) {
            const int e = threadIdx.x + j * kCnThreads;
            const int row = e / kCnChunk, kx = k0 + (e - row * kCnChunk);
            const bool isA = row < Mp;
            const int r = isA ? row : row - Mp;
            // unconditional global loads (an element outside the operands is
            // read from a zero in device memory): no branch around a load, and
            // no flat load, whose pending count would also hold up the LDS reads
            // of the products below
            const bool in = e < nst && kx < kend && (isA ? r < g.M : r < g.Nn);
            stage[j] = gload(!in ? &g_zero2 : isA ? A + (long long)r * g.lda + kx : B + (long long)r * g.ldb + kx);
        }
    };
    fetch(kbeg);
    for (int k0 = kbeg; k0 < kend; k0 += kCnChunk) {
#pragma unroll
        for (int j = 0; j < kCnStage; ++j) {
            const int e = threadIdx.x + j * kCnThreads;
            if (e < nst) {
                const int row = e / kCnChunk;
                const bool isA = row < Mp;
                const int r = isA ? row : row - Mp;
                LdsC<R>* dst = isA ? As : Bs;
                dst[r * LS + (e - row * kCnChunk)] = LdsC<R>{(R)stage[j].x, (R)stage[j].y};
            }
        }
        __syncthreads();
        if (k0 + kCnChunk < kend) fetch(k0 + kCnChunk);  // in flight during the products below
#pragma unroll
        for (int t = 0; t < kCnTilesPerWave; ++t) {
            const int tile = w + 8 * t;
            if (tile < ntiles) {
                const int m0 = (tile / g.nt) * 16, n0 = (tile % g.nt) * 16;
#pragma unroll
                for (int k4 = 0; k4 < kCnChunk; k4 += 4) {
                    const LdsC<R> a = As[(m0 + i) * LS + k4 + kk];
                    const LdsC<R> bv = Bs[(n0 + i) * LS + k4 + kk];
                    cr[t] = mfma(a.re, bv.re, cr[t]);
                    cr[t] = mfma(a.im, bv.im, cr[t]);
                    ci[t] = mfma(a.re, bv.im, ci[t]);
                    ci[t] = mfma(-a.im, bv.re, ci[t]);
                }
            }
        }
        __syncthreads();
    }
    double2* out = g.part + ((long long)b * g.ksplit + ks) * g.M * g.Nn;
#pragma unroll
    for (int t = 0; t < kCnTilesPerWave; ++t) {
        const int tile = w + 8 * t;
        if (tile < ntiles) {
            const int m0 = (tile / g.nt) * 16, n0 = (tile % g.nt) * 16;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = m0 + MF<R>::row(v, kk), n = n0 + i;
                if (m < g.M && n < g.Nn) out[(long long)m * g.Nn + n] = cmk((double)cr[t][v], (double)ci[t][v]);
            }
        }
    }
}

struct GemmUpd {
    double2* Y_base;
    long long y_bstride;
    int ldy;
    const double2* C_base;        // per batch C_base + b*c_bstride, [Minner][Nout]
    long long c_bstride;
    int ldc;
    const double2* const* A_tab;  // per batch b % tmod
    int tmod;
    int lda;
    int Nout, K, Minner;
    double cs;
    double os_x, os_y;            // output sign of side 0 / side 1 batches
    int nk;
};

// One block per 16 rows k of A and batch; its waves take the 16-wide tiles of
// n, so that the A rows are fetched once (into one XCD's L2 and the CU's L1)
// for all of them.  U = 0: one step of 4 at a time (loads, then products);
// U > 0: the inner dimension goes in groups of U steps, two register groups
// in turn, the loads of the next group issued before the products of the
// current one and the outputs' current values read at the start, so that a
// wave does not wait a full memory latency per step (more registers, fewer
// waves per CU).  The products run in the same order in every variant, so the
// results are identical; the autotuner picks per shape.
template <class R, int U>
__global__ void __launch_bounds__(1024) k_gemm_update(GemmUpd g) {
    const int b = blockIdx.z;
    const int n0 = (threadIdx.x >> 6) * 16, k0 = blockIdx.y * 16;
    const int l = threadIdx.x & 63, i = l & 15, kk = l >> 4;
    const int bt = b % (2 * g.nk);  // side and k point (the output sign)
    const double2* A = g.A_tab[b % g.tmod];
    const double2* C = g.C_base + (long long)b * g.c_bstride;
    double2* Y = g.Y_base + (long long)b * g.y_bstride;
    typename MF<R>::V dr = {0, 0, 0, 0}, di = {0, 0, 0, 0};
    const bool ncol = (n0 + i) < g.Nout, kcol = (k0 + i) < g.K;
    const double os = bt < g.nk ? g.os_x : g.os_y;
    if constexpr (U == 0) {
        for (int m = 0; m < g.Minner; m += 4) {
            int mm = m + kk;
            double2 c = (mm < g.Minner && ncol) ? C[(long long)mm * g.ldc + n0 + i] : cmk(0.0, 0.0);
            double2 a = (mm < g.Minner && kcol) ? A[(long long)mm * g.lda + k0 + i] : cmk(0.0, 0.0);
            const R cx = (R)c.x, cy = (R)c.y, ax = (R)a.x, ay = (R)a.y;
            dr = mfma(cx, ax, dr);
            dr = mfma(-cy, ay, dr);
            di = mfma(cx, ay, di);
            di = mfma(cy, ax, di);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            int n = n0 + MF<R>::row(v, kk), k = k0 + i;
            if (n < g.Nout && k < g.K) {
                double2* y = Y + (long long)n * g.ldy + k;
                double2 cur = *y;
                *y = cmk(os * (cur.x + g.cs * (double)dr[v]), os * (cur.y + g.cs * (double)di[v]));
            }
        }
    } else {
        // every load is issued unconditionally (an element outside the
        // operands is read from a zero in device memory), so that no branch
        // separates the loads from their uses and a group's products wait only
        // for that group's loads
        auto load = [&](int m, double2* c, double2* a) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int mm = m + 4 * u + kk;
                const double2* pc = (mm < g.Minner && ncol) ? C + (long long)mm * g.ldc + n0 + i : &g_zero2;
                const double2* pa = (mm < g.Minner && kcol) ? A + (long long)mm * g.lda + k0 + i : &g_zero2;
                c[u] = gload(pc);
                a[u] = gload(pa);
            }
        };
        auto products = [&](int m, const double2* c, const double2* a) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (m + 4 * u < g.Minner) {
                    const R cx = (R)c[u].x, cy = (R)c[u].y, ax = (R)a[u].x, ay = (R)a[u].y;
                    dr = mfma(cx, ax, dr);
                    dr = mfma(-cy, ay, dr);
                    di = mfma(cx, ay, di);
                    di = mfma(cy, ax, di);
                }
            }
        };
        DVec2 ycur[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int n = n0 + MF<R>::row(v, kk), k = k0 + i;
            const double2* py = (n < g.Nout && k < g.K) ? Y + (long long)n * g.ldy + k : &g_zero2;
            ycur[v] = *(const GlobalD2*)py;
        }
        // two register groups in turn (no copies, which would wait for the loads)
        double2 c0[U], a0[U], c1[U], a1[U];
        load(0, c0, a0);
        for (int m = 0; m < g.Minner; m += 8 * U) {
            load(m + 4 * U, c1, a1);  // in flight during the products below (past the end: zeros, unused)
            products(m, c0, a0);
            load(m + 8 * U, c0, a0);
            products(m + 4 * U, c1, a1);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            int n = n0 + MF<R>::row(v, kk), k = k0 + i;
            if (n < g.Nout && k < g.K)
                Y[(long long)n * g.ldy + k] =
                    cmk(os * (ycur[v].x + g.cs * (double)dr[v]), os * (ycur[v].y + g.cs * (double)di[v]));
        }
    }
}

// ---- the nonlocal term and the projector of an apply together (FP64)
// With G = O^dag beta (per q set, laid out once), S = O^dag (phi + beta W) =
// O^dag phi + G W: both contractions read the apply's x and phi as they are, and
// one update adds beta W - O S.  phi is read twice and written once instead of
// four times and twice, in 3 to 5 launches instead of 5 to 7.  us of the stage,
// before -> after: 20^3, 8 bands 31 -> 13; 24^3, 16 bands, 4 k 56 -> 21; 45 x 40 x 50, 12
// bands 103 -> 24; 48 x 48 x 96, 64 bands 143 -> 101.  48 x 48 x 180, 104 bands, 4 k: 794 ->
// 749, where the contractions and the update run at 60 to 72 TFLOP/s of the 72.6
// of a large matrix product and what is saved is the summing in between.

// Contractions of up to two pairs of operands, few output tiles each: a block
// per (tile of either, K split, batch), whose four waves take groups of KU
// steps in turn (as many loads in flight) and add up in LDS.  A split of 64 is
// one group a wave, and at most 32 splits bound the summing that follows.
constexpr int kPairWaves = 4, kPairKU = 4, kPairK = 16 * kPairWaves, kPairSplits = 32;

__global__ void __launch_bounds__(64 * kPairWaves) k_cn_pair(GemmCN g0, GemmCN g1, int tiles0) {
    __shared__ double2 red[kPairWaves][256];
    const bool second = (int)blockIdx.x >= tiles0;
    const GemmCN& g = second ? g1 : g0;
    const int tile = second ? blockIdx.x - tiles0 : blockIdx.x;
    const int b = blockIdx.z, ks = blockIdx.y;
    if (ks >= g.ksplit) return;
    const int m0 = (tile / g.nt) * 16, n0 = (tile % g.nt) * 16;
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, i = l & 15, kk = l >> 4;
    const double2* A = g.A_tab[b % g.amod];
    const double2* B = g.B_base + (long long)b * g.b_bstride;
    const int kbeg = ks * g.kchunk, kend = min(g.K, kbeg + g.kchunk);
    v4d cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
    const bool arow = (m0 + i) < g.M, brow = (n0 + i) < g.Nn;
    const double2* Ap = A + (long long)(m0 + i) * g.lda;
    const double2* Bp = B + (long long)(n0 + i) * g.ldb;
    for (int k = kbeg + 4 * kPairKU * w; k < kend; k += kPairK) {
        double2 a[kPairKU], bv[kPairKU];
#pragma unroll
        for (int u = 0; u < kPairKU; ++u) {
            const int kx = k + 4 * u + kk;
            a[u] = gload((arow && kx < kend) ? Ap + kx : &g_zero2);
            bv[u] = gload((brow && kx < kend) ? Bp + kx : &g_zero2);
        }
#pragma unroll
        for (int u = 0; u < kPairKU; ++u) {
            cr = mfma(a[u].x, bv[u].x, cr);
            cr = mfma(a[u].y, bv[u].y, cr);
            ci = mfma(a[u].x, bv[u].y, ci);
            ci = mfma(-a[u].y, bv[u].x, ci);
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) red[w][(4 * v + kk) * 16 + i] = cmk(cr[v], ci[v]);
    __syncthreads();
    const int m = m0 + threadIdx.x / 16, n = n0 + (threadIdx.x & 15);
    if (m < g.M && n < g.Nn) {
        double2 sum = red[0][threadIdx.x];
#pragma unroll
        for (int v = 1; v < kPairWaves; ++v) sum = cadd(sum, red[v][threadIdx.x]);
        g.part[(((long long)b * g.ksplit + ks) * g.M + m) * g.Nn + n] = sum;
    }
}

// G[(s, i)][m] = sum_k conj(occ[m][s][k]) vkb[i][k] of batch blockIdx.z; a block
// per 16 x 16 tile and spin, its waves take interleaved slices of K
__global__ void __launch_bounds__(64 * kSmallWaves) k_gram(const double2* const* occ, const double2* const* vkb,
                                                           double2* const* gram, int nb, int nproj, int P) {
    __shared__ double2 red[kSmallWaves][256];
    const int b = blockIdx.z, sp = blockIdx.y, nt = (nproj + 15) / 16;
    const int m0 = blockIdx.x / nt * 16, n0 = blockIdx.x % nt * 16;
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, i = l & 15, kk = l >> 4;
    v4d cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
    const bool arow = (m0 + i) < nb, brow = (n0 + i) < nproj;
    const double2* Ap = occ[b] + ((long long)(m0 + i) * 2 + sp) * P;
    const double2* Bp = vkb[b] + (long long)(n0 + i) * P;
    for (int k = 4 * w; k < P; k += 4 * kSmallWaves) {
        const int kx = k + kk;
        const double2 a = gload(arow && kx < P ? Ap + kx : &g_zero2), v = gload(brow && kx < P ? Bp + kx : &g_zero2);
        cr = mfma(a.x, v.x, cr);
        cr = mfma(a.y, v.y, cr);
        ci = mfma(a.x, v.y, ci);
        ci = mfma(-a.y, v.x, ci);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) red[w][(4 * v + kk) * 16 + i] = cmk(cr[v], ci[v]);
    __syncthreads();
    if (threadIdx.x < 256) {
        const int m = m0 + threadIdx.x / 16, n = n0 + (threadIdx.x & 15);
        double2 sum = red[0][threadIdx.x];
        for (int v = 1; v < kSmallWaves; ++v) sum = cadd(sum, red[v][threadIdx.x]);
        if (m < nb && n < nproj) gram[b][((long long)sp * nproj + n) * nb + m] = sum;
    }
}

// Sums of the partials of up to two contractions; 32 elements of 8 slices of the
// splits a block, added up in slice order.  (A thread an element, as before,
// waited on one load after the other: 64 x 64 outputs of 512 splits 34 -> 6 us.)
__global__ void __launch_bounds__(256) k_reduce_pair(const double2* p0, double2* o0, int ks0, long long mn0, const double2* p1,
                                                     double2* o1, int ks1, long long mn1, int blocks0) {
    __shared__ double2 red[8][32];
    const bool second = (int)blockIdx.x >= blocks0;
    const long long mn = second ? mn1 : mn0;
    const int ks = second ? ks1 : ks0, b = blockIdx.y, e = threadIdx.x & 31, sl = threadIdx.x >> 5;
    const long long el = (long long)(second ? blockIdx.x - blocks0 : blockIdx.x) * 32 + e;
    const double2* p = (second ? p1 : p0) + (long long)b * ks * mn + el;
    double2 sum = cmk(0.0, 0.0);
    if (el < mn) {
#pragma unroll 4
        for (int k = sl; k < ks; k += 8) sum = cadd(sum, p[k * mn]);
    }
    red[sl][e] = sum;
    __syncthreads();
    if (sl == 0 && el < mn) {
#pragma unroll
        for (int v = 1; v < 8; ++v) sum = cadd(sum, red[v][e]);
        ((second ? o1 : o0) + (long long)b * mn)[el] = sum;
    }
}

// The coefficients of the update, for columns n of 8 bands of batch blockIdx.y:
//   W[i][(n,s)] = sum_j sum_t D[i][j][s][t] B[j][(n,t)],
//   T[m][n] = -(S[m][n] + sum_s sum_i G[(s,i)][m] W[i][(n,s)]),
// B and S being sums of ksb and kss partials (added up here: slices of them by
// threads that the elements leave over, then the slices in order).  No
// projectors: T = -S.
constexpr int kCoefCols = 8, kCoefThreads = 512;
struct Coef {
    const double2 *Bp, *Sp;   // partials [b][ks][nproj][2 nb], [b][ks][nb][nb]
    int ksb, kss;
    const double2* D;
    const double2* const* G;  // of batch b % tmod
    int tmod, nproj, nb;
    double2 *W, *T;
};

__global__ void __launch_bounds__(kCoefThreads) k_coefficients(Coef c) {
    extern __shared__ double2 lds[];
    const int nb = c.nb, np = c.nproj, b = blockIdx.y, n0 = blockIdx.x * kCoefCols;
    const int eb = np * 2 * kCoefCols, es = nb * kCoefCols, E = eb + es;
    const int slices = E < kCoefThreads ? kCoefThreads / E : 1;
    double2* B = lds;            // [j][(n,t)]
    double2* S = lds + eb;       // [m][n]
    double2* Ws = lds + E;       // [i][(n,s)]
    double2* red = Ws + eb;      // slices > 1: [slice][E]
    const double2* bp = c.Bp + (long long)b * c.ksb * np * 2 * nb;
    const double2* sp = c.Sp + (long long)b * c.kss * nb * nb;
    for (int t = threadIdx.x; t < slices * E; t += kCoefThreads) {
        const int sl = t / E, e = t - sl * E;
        const bool isB = e < eb;
        const int r = isB ? e / (2 * kCoefCols) : (e - eb) / kCoefCols;
        const int col = isB ? e - r * 2 * kCoefCols : e - eb - r * kCoefCols;
        const bool in = isB ? 2 * n0 + col < 2 * nb : n0 + col < nb;
        double2 sum = cmk(0.0, 0.0);
        if (in) {
            const double2* p = isB ? bp + (long long)r * 2 * nb + 2 * n0 + col : sp + (long long)r * nb + n0 + col;
            const long long st = isB ? (long long)np * 2 * nb : (long long)nb * nb;
            const int ks = isB ? c.ksb : c.kss;
#pragma unroll 4
            for (int k = sl; k < ks; k += slices) sum = cadd(sum, p[k * st]);
        }
        if (slices > 1) red[t] = sum;
        else lds[e] = sum;
    }
    __syncthreads();
    if (slices > 1) {
        for (int e = threadIdx.x; e < E; e += kCoefThreads) {
            double2 sum = red[e];
            for (int v = 1; v < slices; ++v) sum = cadd(sum, red[v * E + e]);
            lds[e] = sum;
        }
        __syncthreads();
    }
    for (int e = threadIdx.x; e < eb; e += kCoefThreads) {
        const int i = e / (2 * kCoefCols), col = e - i * 2 * kCoefCols, s = col & 1;
        const double2* D = c.D + ((long long)i * np * 2 + s) * 2;
        double2 w = cmk(0.0, 0.0);
        for (int j = 0; j < np; ++j)
#pragma unroll
            for (int t = 0; t < 2; ++t) w = cadd(w, cmul(D[j * 4 + t], B[j * 2 * kCoefCols + col - s + t]));
        Ws[e] = w;
        if (2 * n0 + col < 2 * nb) c.W[((long long)b * np + i) * 2 * nb + 2 * n0 + col] = w;
    }
    __syncthreads();
    const double2* G = np > 0 ? c.G[b % c.tmod] : nullptr;
    for (int e = threadIdx.x; e < es; e += kCoefThreads) {
        const int m = e / kCoefCols, n = e - m * kCoefCols;
        double2 t = S[e];
        for (int s = 0; s < 2; ++s)
#pragma unroll 4
            for (int i = 0; i < np; ++i) t = cadd(t, cmul(G[((long long)s * np + i) * nb + m], Ws[i * 2 * kCoefCols + 2 * n + s]));
        if (n0 + n < nb) c.T[((long long)b * nb + m) * nb + n0 + n] = cmk(-t.x, -t.y);
    }
}

// Y[n][(s,k)] = os (Y + sum_i W[i][(n,s)] vkb[i][k] + sum_m T[m][n] occ[m][(s,k)]):
// the steps of both sums one after the other, grouped as in k_gemm_update<U>.
struct UpdPair {
    double2* Y;
    const double2 *W, *T;
    const double2 *const *vkb, *const *occ;  // of batch b % tmod
    int tmod, nproj, nb, P, nk;
    double os_x, os_y;
};

template <int U>
__global__ void __launch_bounds__(1024) k_update_pair(UpdPair g) {
    const int b = blockIdx.z, sp = blockIdx.x, nb = g.nb, P = g.P;
    const int n0 = (threadIdx.x >> 6) * 16, k0 = blockIdx.y * 16;
    const int l = threadIdx.x & 63, i = l & 15, kk = l >> 4;
    const bool ncol = n0 + i < nb, kcol = k0 + i < P;
    const double os = b % (2 * g.nk) < g.nk ? g.os_x : g.os_y;
    const double2* A0 = g.nproj > 0 ? g.vkb[b % g.tmod] + k0 + i : nullptr;
    const double2* A1 = g.occ[b % g.tmod] + (long long)sp * P + k0 + i;
    const double2* C0 = g.W + (long long)b * g.nproj * 2 * nb + 2 * (n0 + i) + sp;
    const double2* C1 = g.T + (long long)b * nb * nb + n0 + i;
    double2* Y = g.Y + (long long)b * nb * 2 * P + (long long)sp * P + k0 + i;
    const int t0 = (g.nproj + 3) / 4, t1 = t0 + (nb + 3) / 4;
    v4d dr = {0, 0, 0, 0}, di = {0, 0, 0, 0};
    auto load = [&](int t, double2* c, double2* a) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int st = t + u;
            const bool first = st < t0;
            const int m = 4 * (first ? st : st - t0) + kk;
            const bool in = m < (first ? g.nproj : nb);
            c[u] = gload(in && ncol ? (first ? C0 + m * 2 * nb : C1 + m * nb) : &g_zero2);
            a[u] = gload(in && kcol ? (first ? A0 + (long long)m * P : A1 + (long long)m * 2 * P) : &g_zero2);
        }
    };
    auto products = [&](int t, const double2* c, const double2* a) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (t + u < t1) {
                dr = mfma(c[u].x, a[u].x, dr);
                dr = mfma(-c[u].y, a[u].y, dr);
                di = mfma(c[u].x, a[u].y, di);
                di = mfma(c[u].y, a[u].x, di);
            }
        }
    };
    DVec2 ycur[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int n = n0 + 4 * v + kk;
        const double2* py = (n < nb && kcol) ? Y + (long long)n * 2 * P : &g_zero2;
        ycur[v] = *(const GlobalD2*)py;
    }
    double2 c0[U], a0[U], c1[U], a1[U];
    load(0, c0, a0);
    for (int t = 0; t < t1; t += 2 * U) {
        load(t + U, c1, a1);
        products(t, c0, a0);
        load(t + 2 * U, c0, a0);
        products(t + U, c1, a1);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int n = n0 + 4 * v + kk;
        if (n < nb && kcol) Y[(long long)n * 2 * P] = cmk(os * (ycur[v].x + dr[v]), os * (ycur[v].y + di[v]));
    }
}

// W[b][i][(n,s)] = sum_j sum_t D[i][j][s][t] Bm[b][j][(n,t)]
__global__ void k_dmat(const double2* Bm, const double2* D, double2* Wm, int nproj, int nb, int nbatch) {
    long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long per = (long long)nproj * 2 * nb;
    if (idx >= per * nbatch) return;
    long long b = idx / per;
    int r = (int)(idx - b * per);
    int i = r / (2 * nb), ns = r % (2 * nb);
    int n = ns >> 1, s = ns & 1;
    const double2* Bb = Bm + b * per;
    double2 acc = cmk(0.0, 0.0);
    for (int j = 0; j < nproj; ++j)
        for (int t = 0; t < 2; ++t)
            acc = cadd(acc, cmul(D[((i * nproj + j) * 2 + s) * 2 + t], Bb[(long long)j * 2 * nb + 2 * n + t]));
    Wm[idx] = acc;
}

// the LDS-staged kernel needs its tiles to fit the waves, and enough tiles to
// keep its 8 waves busy (single-tile products stay on k_gemm_cn)
bool cn_lds_fits(int M, int Nn) {
    const int mt = (M + 15) / 16, nt = (Nn + 15) / 16;
    return mt <= kMaxTiles1D && nt <= kMaxTiles1D && mt + nt <= kCnMaxTilesSum && mt * nt <= 8 * kCnTilesPerWave &&
           mt * nt >= 8;
}

// K range per block: about 4 blocks per CU over all batches, a multiple of the LDS chunk
// K chunk per block: about `target` blocks over the batches of one right-hand
// side (the autotuner times 1024, 512 and 2048)
int cn_lds_kchunk(int K, int nbatch, int target = 1024) {
    const int ks = std::max(1, target / std::max(1, nbatch));
    int kc = (K + ks - 1) / ks;
    kc = std::max(kCnChunk * 4, (kc + kCnChunk - 1) / kCnChunk * kCnChunk);
    return kc;
}

int choose_kchunk(int K, long long tiles_times_batch, long long target = 8192) {
    // enough waves to fill the chip, but chunks of at least 64
    int ks = (int)std::max<long long>(1, target / std::max<long long>(1, tiles_times_batch));
    int kc = (K + ks - 1) / ks;
    kc = std::max(64, (kc + 3) / 4 * 4);
    return kc;
}

// the two products in the autotuner's report
constexpr const char* kNonlocal = "nonlocal term";
constexpr const char* kProjector = "projector";

// nbatch batches per right-hand side, nrhs right-hand sides (the K chunking
// depends on nbatch only, so each right-hand side is summed as when alone);
// batch b takes A_tab[b % amod]
void run_gemm_cn(const System& s, const double2* const* A_tab, int amod, int lda, const double2* B_base,
                 long long b_bstride, int ldb, int M, int Nn, int K, int nbatch, int nrhs, double2* out,
                 hipStream_t st, bool f32, const char* what) {
    GemmCN g;
    g.A_tab = A_tab;
    g.amod = amod;
    g.A_base = nullptr;
    g.a_bstride = 0;
    g.lda = lda;
    g.B_base = B_base;
    g.b_bstride = b_bstride;
    g.ldb = ldb;
    g.M = M;
    g.Nn = Nn;
    g.K = K;
    int mt = (M + 15) / 16;
    g.nt = (Nn + 15) / 16;
    g.part = s.ws.gpart;
    if (!cn_lds_fits(M, Nn) && K <= kSmallK) {
        dim3 grid(mt * g.nt, nrhs * nbatch);
        if (f32) {
            TM_LAUNCH(k_gemm_cn_small<float>, grid, dim3(64 * kSmallWaves), 0, st, g, out);
        } else {
            TM_LAUNCH(k_gemm_cn_small<double>, grid, dim3(64 * kSmallWaves), 0, st, g, out);
        }
        return;
    }
    // the K split the autotuner picked for this contraction (per right-hand side,
    // so that every right-hand side is summed as when alone); FP64 only.  The
    // key is the output shape and the batch count, not K: the q sets of a
    // system differ only in K, so all of them take the choice made at the
    // system's first apply, and a chain's arithmetic does not depend on which
    // q set happened to be applied first.
    constexpr int kTargets[3] = {1024, 512, 2048};
    const int tv = f32 ? 0 : tune_pick(kTuneGemm, tune_key(M, Nn, nbatch), 3, what);
    if (cn_lds_fits(M, Nn)) {
        g.kchunk = cn_lds_kchunk(K, nbatch, kTargets[tv]);
        g.ksplit = (K + g.kchunk - 1) / g.kchunk;
        TM_CHECK((size_t)nrhs * nbatch * g.ksplit * M * Nn <= s.ws.cap_gpart, TM_EINVAL,
                 "GEMM partial buffer too small");
        const size_t shm = (size_t)(mt + g.nt) * 16 * (kCnChunk + 1) * (f32 ? 8 : 16);
        dim3 grid(g.ksplit, nrhs * nbatch);
        const void* fn = f32 ? (const void*)k_gemm_cn_lds<float> : (const void*)k_gemm_cn_lds<double>;
        TM_CHECK(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm) == hipSuccess,
                 TM_EDEVICE, "cannot raise the LDS limit of k_gemm_cn_lds");
        if (f32) {
            TM_LAUNCH(k_gemm_cn_lds<float>, grid, dim3(kCnThreads), shm, st, g, mt);
        } else {
            TM_LAUNCH(k_gemm_cn_lds<double>, grid, dim3(kCnThreads), shm, st, g, mt);
        }
    } else {
        g.kchunk = choose_kchunk(K, (long long)mt * g.nt * nbatch, 8LL * kTargets[tv]);
        g.ksplit = (K + g.kchunk - 1) / g.kchunk;
        TM_CHECK((size_t)nrhs * nbatch * g.ksplit * M * Nn <= s.ws.cap_gpart, TM_EINVAL,
                 "GEMM partial buffer too small");
        dim3 grid(mt * g.nt, g.ksplit, nrhs * nbatch);
        if (f32) {
            TM_LAUNCH(k_gemm_cn<float>, grid, dim3(64), 0, st, g);
        } else {
            TM_LAUNCH(k_gemm_cn<double>, grid, dim3(64), 0, st, g);
        }
    }
    long long mn = (long long)M * Nn;
    const int blocks = (int)((mn + 31) / 32);
    TM_LAUNCH(k_reduce_pair, dim3(blocks, nrhs * nbatch), dim3(256), 0, st, s.ws.gpart, out, g.ksplit, mn, nullptr, nullptr, 0,
              0, blocks);
}

// one contraction of the pair: operands and K split (cap: partials of a right-hand side)
GemmCN pair_side(const System& s, const double2* const* A_tab, int amod, const double2* B_base, long long b_bstride, int ld,
                 int M, int Nn, int nbatch, long long cap, const char* what, bool& staged) {
    GemmCN g{};
    g.A_tab = A_tab;
    g.amod = amod;
    g.lda = g.ldb = g.K = ld;
    g.B_base = B_base;
    g.b_bstride = b_bstride;
    g.M = M;
    g.Nn = Nn;
    g.nt = (Nn + 15) / 16;
    staged = cn_lds_fits(M, Nn);
    if (staged) {
        constexpr int kTargets[3] = {1024, 512, 2048};  // as in run_gemm_cn
        g.kchunk = cn_lds_kchunk(ld, nbatch, kTargets[tune_pick(kTuneGemm, tune_key(M, Nn, nbatch), 3, what)]);
    } else {
        const int splits = (int)std::max<long long>(1, std::min<long long>(kPairSplits, cap / ((long long)nbatch * M * Nn)));
        g.kchunk = std::max(kPairK, ((ld + splits - 1) / splits + kPairK - 1) / kPairK * kPairK);
    }
    g.ksplit = (ld + g.kchunk - 1) / g.kchunk;
    return g;
}

void launch_staged(const GemmCN& g, int nbatch, hipStream_t st) {
    const int mt = (g.M + 15) / 16;
    const size_t shm = (size_t)(mt + g.nt) * 16 * (kCnChunk + 1) * 16;
    TM_CHECK(hipFuncSetAttribute((const void*)k_gemm_cn_lds<double>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm) ==
                 hipSuccess,
             TM_EDEVICE, "cannot raise the LDS limit of k_gemm_cn_lds");
    TM_LAUNCH(k_gemm_cn_lds<double>, dim3(g.ksplit, nbatch), dim3(kCnThreads), shm, st, g, mt);
}

size_t coef_lds(int nproj, int nb) {
    const int eb = nproj * 2 * kCoefCols, E = eb + nb * kCoefCols;
    return (size_t)(E + eb + (E < kCoefThreads ? kCoefThreads / E * E : 0)) * sizeof(double2);
}

// phi <- os (phi + beta D beta^dag x - O O^dag (phi + beta D beta^dag x)), FP64;
// x null: the projector alone.  The columns of the plane kernels are free here
// and hold the partials of B and T.  False where they are too small for them:
// the terms go one after the other then.  (The K splits and the choice depend on
// the shape of one right-hand side, so that each is summed as when alone.)
bool run_pair(const System& s, const QSet& q, const double2* x, double2* phi, double osx, double osy, int nrhs,
              hipStream_t st) {
    const int nb = s.nbnd, P = q.npw_pad, nbatch = 2 * q.nk, all = nbatch * nrhs, np = x ? s.nproj : 0;
    const long long bstride = (long long)nb * 2 * P;
    // k_update_pair holds 256 bands, but the sequence's update takes both spins of
    // a band as columns of its own: where one is refused the other is too
    TM_CHECK((np > 0 ? 2 : 1) * nb <= 256, TM_EUNSUPPORTED, "more than 256 output columns per batch");
    if (coef_lds(np, nb) > 150 * 1024) return false;
    bool sb = false, ss = false;
    const long long mns = (long long)nb * nb, mnb = (long long)np * 2 * nb;
    const long long T = nbatch * mns, room = (long long)(s.ws.cap_xcols / s.ws.width) - T - nbatch * mnb;
    GemmCN gs = pair_side(s, (const double2* const*)q.d_occ, q.tmod, phi, bstride, 2 * P, nb, nb, nbatch,
                          (long long)(s.ws.cap_gpart / s.ws.width), kProjector, ss);
    GemmCN gb{};
    if (np > 0) gb = pair_side(s, q.d_vkb, q.tmod, x, bstride, P, np, 2 * nb, nbatch, room, kNonlocal, sb);
    const long long parts = nbatch * gb.ksplit * mnb;
    if (parts > room) return false;
    // more elements than a block has threads: their sums in a launch of their own
    const bool sums = (gs.ksplit > 1 || gb.ksplit > 1) && (np * 2 + nb) * kCoefCols > kCoefThreads;
    TM_CHECK((size_t)all * gs.ksplit * mns <= s.ws.cap_gpart, TM_EINVAL, "GEMM partial buffer too small");
    double2* t = s.ws.xcols;
    gb.part = t + nrhs * T;
    gs.part = s.ws.gpart;
    double2* bred = gb.part + nrhs * parts;
    const int tiles_b = np > 0 ? (np + 15) / 16 * gb.nt : 0, tiles_s = (nb + 15) / 16 * gs.nt;
    if (ss) launch_staged(gs, all, st);
    if (sb) launch_staged(gb, all, st);
    if (!ss || (np > 0 && !sb)) {
        const int tb = sb ? 0 : tiles_b, ts = ss ? 0 : tiles_s;
        const int ks = std::max(tb > 0 ? gb.ksplit : 0, ts > 0 ? gs.ksplit : 0);
        TM_LAUNCH(k_cn_pair, dim3(tb + ts, ks, all), dim3(64 * kPairWaves), 0, st, gb, gs, tb);
    }
    Coef c{gb.part, gs.part, gb.ksplit, gs.ksplit, s.dvan, q.d_gram, q.tmod, np, nb, s.ws.gsmall, t};
    if (sums) {
        const int blocks_s = (int)((mns + 31) / 32), blocks_b = (int)((mnb + 31) / 32);
        TM_LAUNCH(k_reduce_pair, dim3(blocks_s + blocks_b, all), dim3(256), 0, st, gs.part, t, gs.ksplit, mns, gb.part, bred,
                  gb.ksplit, mnb, blocks_s);
        c.Bp = bred;
        c.Sp = t;
        c.ksb = c.kss = 1;
    }
    const size_t shm = coef_lds(np, nb);
    TM_CHECK(hipFuncSetAttribute((const void*)k_coefficients, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm) ==
                 hipSuccess,
             TM_EDEVICE, "cannot raise the LDS limit of k_coefficients");
    TM_LAUNCH(k_coefficients, dim3((nb + kCoefCols - 1) / kCoefCols, all), dim3(kCoefThreads), shm, st, c);
    UpdPair u{phi, c.W, t, q.d_vkb, (const double2* const*)q.d_occ, q.tmod, np, nb, P, q.nk, osx, osy};
    const int ntile = (nb + 15) / 16;
    const dim3 grid(2, (P + 15) / 16, all);
    if (tune_pick(kTuneUpdPair, tune_key(nb, np, nbatch), 2) == 0) {
        TM_LAUNCH(k_update_pair<3>, grid, dim3(64 * ntile), 0, st, u);
    } else {
        TM_LAUNCH(k_update_pair<2>, grid, dim3(64 * ntile), 0, st, u);
    }
    return true;
}

void run_gemm_update(double2* Y, long long y_bstride, int ldy, const double2* C, long long c_bstride, int ldc,
                     const double2* const* A_tab, int tmod, int lda, int Nout, int K, int Minner, double cs,
                     double osx, double osy, int nk, int nrhs, hipStream_t st, bool f32, const char* what) {
    GemmUpd g;
    g.tmod = tmod;
    g.Y_base = Y;
    g.y_bstride = y_bstride;
    g.ldy = ldy;
    g.C_base = C;
    g.c_bstride = c_bstride;
    g.ldc = ldc;
    g.A_tab = A_tab;
    g.lda = lda;
    g.Nout = Nout;
    g.K = K;
    g.Minner = Minner;
    g.cs = cs;
    g.os_x = osx;
    g.os_y = osy;
    g.nk = nk;
    const int ntile = (Nout + 15) / 16;
    TM_CHECK(ntile <= 16, TM_EUNSUPPORTED, "more than 256 output columns per batch");
    dim3 grid(1, (K + 15) / 16, 2 * nk * nrhs);
    if (f32) {
        TM_LAUNCH((k_gemm_update<float, 3>), grid, dim3(64 * ntile), 0, st, g);
        return;
    }
    // the variant the autotuner picked for this shape (tuned with one
    // right-hand side; every variant gives the same result)
    switch (tune_pick(kTuneUpd, tune_key(Nout, Minner, 2 * nk), 3, what)) {
        case 0: TM_LAUNCH((k_gemm_update<double, 0>), grid, dim3(64 * ntile), 0, st, g); break;
        case 1: TM_LAUNCH((k_gemm_update<double, 2>), grid, dim3(64 * ntile), 0, st, g); break;
        default: TM_LAUNCH((k_gemm_update<double, 3>), grid, dim3(64 * ntile), 0, st, g); break;
    }
}

}  // namespace

// partial sums of the finest K split any variant uses
size_t gemm_partial_elems(int nbatch, int M, int Nn, int K) {
    int mt = (M + 15) / 16, nt = (Nn + 15) / 16;
    int kc = cn_lds_fits(M, Nn) ? cn_lds_kchunk(K, nbatch, 2048) : choose_kchunk(K, (long long)mt * nt * nbatch, 16384);
    int ks = (K + kc - 1) / kc;
    return (size_t)nbatch * ks * M * Nn;
}

// G of k_coefficients, for the batches of a q set
void launch_gram(const System& s, const QSet& q, hipStream_t st) {
    const int tiles = (s.nbnd + 15) / 16 * ((s.nproj + 15) / 16);
    TM_LAUNCH(k_gram, dim3(tiles, 2, 2 * q.nk), dim3(64 * kSmallWaves), 0, st, (const double2* const*)q.d_occ,
              (const double2* const*)q.d_vkb, q.d_gram, s.nbnd, s.nproj, q.npw_pad);
}

// x and out hold nrhs BR vectors back to back
void launch_nonlocal_project(const System& s, const QSet& q, const double2* x, double2* out, hipStream_t st, bool f32,
                             int nrhs) {
    if (!f32 && run_pair(s, q, x, out, 1.0, -1.0, nrhs, st)) return;
    launch_nonlocal(s, q, x, out, st, f32, nrhs);
    launch_project(s, q, out, st, f32, nrhs);
}

void launch_nonlocal(const System& s, const QSet& q, const double2* x, double2* out, hipStream_t st, bool f32,
                     int nrhs) {
    if (s.nproj == 0) return;
    const int nb = s.nbnd, P = q.npw_pad, nbatch = 2 * q.nk;
    const long long bstride = (long long)nb * 2 * P;
    double2* Bm = s.ws.gsmall;
    double2* Wm = s.ws.gsmall + (size_t)nrhs * nbatch * s.nproj * 2 * nb;
    run_gemm_cn(s, q.d_vkb, q.tmod, P, x, bstride, P, s.nproj, 2 * nb, P, nbatch, nrhs, Bm, st, f32,
                kNonlocal);
    long long tot = (long long)nrhs * nbatch * s.nproj * 2 * nb;
    TM_LAUNCH(k_dmat, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, st, Bm, s.dvan, Wm, s.nproj, nb,
                       nrhs * nbatch);
    run_gemm_update(out, bstride, P, Wm, (long long)s.nproj * 2 * nb, 2 * nb, q.d_vkb, q.tmod, P, 2 * nb, P,
                    s.nproj, 1.0, 1.0, 1.0, q.nk, nrhs, st, f32, kNonlocal);
}

void launch_project_signed(const System& s, const QSet& q, double2* phi, double osx, double osy, hipStream_t st,
                           bool f32, int nrhs) {
    const int nb = s.nbnd, P = q.npw_pad, nbatch = 2 * q.nk;
    const long long bstride = (long long)nb * 2 * P;
    if (!f32 && !cn_lds_fits(nb, nb) && run_pair(s, q, nullptr, phi, osx, osy, nrhs, st)) return;
    double2* S = s.ws.gsmall;
    run_gemm_cn(s, (const double2* const*)q.d_occ, q.tmod, 2 * P, phi, bstride, 2 * P, nb, nb, 2 * P, nbatch, nrhs,
                S, st, f32, kProjector);
    run_gemm_update(phi, bstride, 2 * P, S, (long long)nb * nb, nb, (const double2* const*)q.d_occ, q.tmod, 2 * P,
                    nb, 2 * P, nb, -1.0, osx, osy, q.nk, nrhs, st, f32, kProjector);
}

void launch_project(const System& s, const QSet& q, double2* out, hipStream_t st, bool f32, int nrhs) {
    launch_project_signed(s, q, out, 1.0, -1.0, st, f32, nrhs);
}

}  // namespace tml
