// Susceptibility from the Lanczos tridiagonal matrix (Eqs.
// resolvent_Liouvillian_Lanczos_q and post_processing):
//   chi_l(w) = n1 sum_i z_l[i] eta_i,   ((w + i eta) I - T) eta = e_1.
//
// With A = (w + i eta) I - T this is chi_l = n1 y_1, A^T y = z_l: only the
// first component is wanted, so A^T is eliminated from its last row upward
// with the rows z_l carried along, and y_1 is the quotient that is left.  One
// sweep, a state of one row (two coefficients and the z_l) in registers, no
// work arrays.  Each step takes the larger of the two candidate pivots (row
// interchange), as Gaussian elimination with partial pivoting does.
//
// Bounded by the dependent steps of one thread: M of them, and at one wave per
// SIMD what a step costs is its instruction count.  So a thread takes one
// frequency and one row l (the pivots are recomputed by the four threads of a
// frequency: waves are free, instructions are not), the reciprocal is two
// Newton steps on the hardware's estimate, and the chain coefficients, the same
// for every frequency, are staged in LDS a chunk ahead and read a group of
// steps at a time.
// M = 3000, 400 frequencies, 4 rows: 10.57 ms for the elimination from the top
// with its rows in global memory and a back substitution; from the bottom 0.95
// ms with the four rows in one thread, 0.72 with one row a thread, 0.57 with
// both candidate eliminations formed before the pivot is known, 0.49 with the
// group reads, 0.50 with the range of the pivots kept (the call 587 -> 557 us: the
// host no longer scales the coefficients).
//
// k_chi squares its pivots, and the other order of elimination can meet a
// rounding error where the one from the top meets a zero.  So it answers for
// the frequencies whose pivots lie in 2^+-300 and within a factor 2^40 of each
// other, with finite results; it marks the others (a frequency far from the
// spectrum or infinite, coefficients far apart, a pole of the undamped chain),
// and k_chi_pivoted solves those from the top, each with Smith's quotients and
// work arrays of its own: frequencies do not affect each other, and whether a
// chain counts as singular is decided there alone.
#include "tm_internal.h"

namespace tml {

namespace {

__device__ inline double2 cdiv(double2 a, double2 b) {
    // Smith's algorithm for a / b
    if (fabs(b.x) >= fabs(b.y)) {
        double r = b.y / b.x, d = b.x + b.y * r;
        return cmk((a.x + a.y * r) / d, (a.y - a.x * r) / d);
    }
    double r = b.x / b.y, d = b.x * r + b.y;
    return cmk((a.x * r + a.y) / d, (a.y * r - a.x) / d);
}

__device__ inline double cabs1(double2 a) { return fabs(a.x) + fabs(a.y); }

// 1 / d for d well inside the exponent range: the hardware's estimate and two
// Newton steps
__device__ __forceinline__ double recip(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
    return __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
}

// c - a b
__device__ __forceinline__ double2 cnma(double2 a, double2 b, double2 c) {
    return cmk(__builtin_fma(-a.x, b.x, __builtin_fma(a.y, b.y, c.x)),
               __builtin_fma(-a.x, b.y, __builtin_fma(-a.y, b.x, c.y)));
}

// One thread per frequency: Gaussian elimination from the first row down with
// partial pivoting (row interchanges create a second superdiagonal), back
// substitution, and the contraction with z.  Work arrays [i][frequency] in
// global memory; 3.5 us a row, all of it memory latency.
__global__ void k_chi_pivoted(const double2* alpha, const double* beta, const double2* gamma, const double2* z, int nz,
                              int cap, int M, double n1, const double* omega, int nw, double eta, double2* wd,
                              double2* wdu, double2* wdu2, double2* wb, double2* chi, int* status) {
    int w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= nw) return;
    auto D = [&](int i) -> double2& { return wd[(long long)i * nw + w]; };
    auto DU = [&](int i) -> double2& { return wdu[(long long)i * nw + w]; };
    auto DU2 = [&](int i) -> double2& { return wdu2[(long long)i * nw + w]; };
    auto Bv = [&](int i) -> double2& { return wb[(long long)i * nw + w]; };
    const double2 wc = cmk(omega[w], eta);
    for (int i = 0; i < M; ++i) {
        D(i) = csub(wc, alpha[i]);
        DU(i) = i + 1 < M ? cmk(-gamma[i].x, -gamma[i].y) : cmk(0.0, 0.0);
        DU2(i) = cmk(0.0, 0.0);
        Bv(i) = i == 0 ? cmk(1.0, 0.0) : cmk(0.0, 0.0);
    }
    int bad = 0;
    for (int i = 0; i + 1 < M; ++i) {
        double2 dl = cmk(-beta[i], 0.0);  // A[i+1][i]
        double2 di = D(i);
        if (cabs1(di) >= cabs1(dl)) {
            if (cabs1(di) == 0.0) { bad = 1; break; }
            double2 f = cdiv(dl, di);
            D(i + 1) = csub(D(i + 1), cmul(f, DU(i)));
            Bv(i + 1) = csub(Bv(i + 1), cmul(f, Bv(i)));
        } else {
            double2 f = cdiv(di, dl);
            D(i) = dl;
            double2 tmp = D(i + 1);
            D(i + 1) = csub(DU(i), cmul(f, tmp));
            if (i + 2 < M) {
                DU2(i) = DU(i + 1);
                DU(i + 1) = cmk(-(f.x * DU2(i).x - f.y * DU2(i).y), -(f.x * DU2(i).y + f.y * DU2(i).x));
            }
            DU(i) = tmp;
            double2 bi = Bv(i);
            Bv(i) = Bv(i + 1);
            Bv(i + 1) = csub(bi, cmul(f, Bv(i + 1)));
        }
    }
    if (!bad && cabs1(D(M - 1)) == 0.0) bad = 1;
    double2 acc[4] = {cmk(0, 0), cmk(0, 0), cmk(0, 0), cmk(0, 0)};
    if (!bad) {
        double2 x1 = cmk(0, 0), x2 = cmk(0, 0);  // x[i+1], x[i+2]
        for (int i = M - 1; i >= 0; --i) {
            double2 r = Bv(i);
            if (i + 1 < M) r = csub(r, cmul(DU(i), x1));
            if (i + 2 < M) r = csub(r, cmul(DU2(i), x2));
            double2 xi = cdiv(r, D(i));
            for (int l = 0; l < 4; ++l)
                if (l < nz) acc[l] = cadd(acc[l], cmul(z[(long long)l * cap + i], xi));
            x2 = x1;
            x1 = xi;
        }
    } else {
        atomicOr(status, 1);
    }
    for (int l = 0; l < nz; ++l) chi[(long long)l * nw + w] = cscale(acc[l], n1);
}

constexpr int kChiThreads = 64;
constexpr int kChiRows = 4;                       // rows l a block works on (the fourth idle for three)
constexpr int kChiFreqs = kChiThreads / kChiRows; // frequencies of a block
constexpr int kChiChunk = 64;                     // chain steps staged together
constexpr int kChiGroup = 4;                      // of them read together
constexpr int kChiVals = 6;                       // alpha, gamma of the row above, beta, 1 / beta
// The pivots (|re| + |im|) that k_chi answers for: their squares, reciprocals and
// products with the couplings are normal numbers, and none is so far below the
// others that it could be a zero but for rounding (a chain of 3000 steps rounds by
// some 2^-45 of them).
constexpr double kChiPivotMin = 0x1p-300, kChiPivotMax = 0x1p300, kChiPivotRatio = 0x1p-40;

__global__ void __launch_bounds__(kChiThreads) k_chi(const double2* __restrict__ alpha,
                                                     const double* __restrict__ beta,
                                                     const double2* __restrict__ gamma,
                                                     const double2* __restrict__ z, int nz, int cap, int M, double n1,
                                                     const double* __restrict__ omega, int nw, double eta,
                                                     double2* __restrict__ chi, int* __restrict__ general) {
    __shared__ double sh[2][kChiChunk][kChiVals];
    __shared__ double2 shz[2][kChiChunk][kChiRows];
    const int row = threadIdx.x / kChiFreqs;
    const int w = blockIdx.x * kChiFreqs + threadIdx.x % kChiFreqs;
    const double2 wc = cmk(omega[min(w, nw - 1)], eta);
    // thread t's row of the chunk whose first (highest) row is `top`
    double st[kChiVals];
    double2 stz[kChiRows];
    auto fetch = [&](int top) {
        const int i = max(top - (int)threadIdx.x, 0);
        const double2 a = alpha[i], g = i > 0 ? gamma[i - 1] : cmk(0.0, 0.0);
        st[0] = a.x;
        st[1] = a.y;
        st[2] = g.x;
        st[3] = g.y;
        st[4] = beta[i];
        st[5] = 1.0 / beta[i];
#pragma unroll
        for (int l = 0; l < kChiRows; ++l) stz[l] = z[(long long)min(l, nz - 1) * cap + i];
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int v = 0; v < kChiVals; ++v) sh[buf][threadIdx.x][v] = st[v];
#pragma unroll
        for (int l = 0; l < kChiRows; ++l) shz[buf][threadIdx.x][l] = stz[l];
    };
    fetch(M - 1);
    stage(0);
    __syncthreads();
    // the row in hand: p y_{i+1} + q y_i = zc
    double2 p = cmk(wc.x - sh[0][0][0], wc.y - sh[0][0][1]), q = cmk(-sh[0][0][2], -sh[0][0][3]);
    double2 zc = shz[0][0][row];
    double pmin = kChiPivotMax, pmax = kChiPivotMin;  // of the pivots
    int buf = 0;
    for (int top = M - 1; top >= 0; top -= kChiChunk) {
        const int rows = min(kChiChunk, top + 1);
        if (top - kChiChunk >= 0) fetch(top - kChiChunk);  // in flight during this chunk
        const int first = top == M - 1 ? 1 : 0;            // the last row is already in hand
        // kChiGroup steps' values are read together, ahead of the steps
        for (int k0 = first; k0 < rows; k0 += kChiGroup) {
            double v[kChiGroup][kChiVals];
            double2 zv[kChiGroup];
#pragma unroll
            for (int u = 0; u < kChiGroup; ++u) {
                const int k = min(k0 + u, rows - 1);
                zv[u] = shz[buf][k][row];
#pragma unroll
                for (int j = 0; j < kChiVals; ++j) v[u][j] = sh[buf][k][j];
            }
#pragma unroll
            for (int u = 0; u < kChiGroup; ++u) {
                if (k0 + u >= rows) break;
                // row i = top - k: -beta_i y_{i+1} + d y_i - gamma_{i-1} y_{i-1} = z_i
                const double2 d = cmk(wc.x - v[u][0], wc.y - v[u][1]), g = cmk(-v[u][2], -v[u][3]), zr = zv[u];
                const double e = -v[u][4], ie = -v[u][5];
                // both eliminations, the pivot p (keep) or e, and the one the rule
                // takes: the reciprocal of p then does not wait for the comparison
                const double mag = cabs1(p);
                const bool keep = mag >= fabs(e);
                const double piv = keep ? mag : fabs(e);
                pmin = fmin(pmin, piv);
                pmax = fmax(pmax, piv);
                const double s = recip(__builtin_fma(p.x, p.x, p.y * p.y));
                const double2 fk = cmk(e * p.x * s, -(e * p.y) * s), fs = cscale(p, ie);
                const double2 pk = cnma(fk, q, d), ps = cnma(fs, d, q);
                const double2 zk = cnma(fk, zc, zr), zs = cnma(fs, zr, zc);
                const double2 qs = cmul(fs, g);
                p = keep ? pk : ps;
                q = keep ? g : cmk(-qs.x, -qs.y);
                zc = keep ? zk : zs;
            }
        }
        buf ^= 1;
        if (top - kChiChunk >= 0) stage(buf);
        __syncthreads();
    }
    if (w >= nw || row >= nz) return;
    const double mag = cabs1(p);
    pmin = fmin(pmin, mag);
    pmax = fmax(pmax, mag);
    const double2 x = cscale(cdiv(zc, p), n1);
    chi[(long long)row * nw + w] = x;
    // (a NaN that came up on the way stays in p, or in zc, to the end)
    const bool in = pmin >= kChiPivotMin && pmax <= kChiPivotMax && pmin >= kChiPivotRatio * pmax &&
                    isfinite(mag) && isfinite(x.x) && isfinite(x.y);
    if (!in) general[w] = 1;  // all rows of a frequency write the same
}

}  // namespace

// chi of every frequency; general[w] (zero before): 1 where launch_chi_pivoted has to solve instead
void launch_chi(const double2* alpha, const double* beta, const double2* gamma, const double2* z, int nz, int cap,
                int M, double n1, const double* omega, int nw, double eta, double2* chi, int* general,
                hipStream_t st) {
    TM_CHECK(nz >= 1 && nz <= 4, TM_EINVAL, "1 to 4 measure rows");
    TM_LAUNCH(k_chi, dim3((nw + kChiFreqs - 1) / kChiFreqs), dim3(kChiThreads), 0, st, alpha, beta, gamma, z, nz,
              cap, M, n1, omega, nw, eta, chi, general);
}

// work: 4 M nw elements; status: set to 1 if a frequency's system is singular
void launch_chi_pivoted(const double2* alpha, const double* beta, const double2* gamma, const double2* z, int nz,
                        int cap, int M, double n1, const double* omega, int nw, double eta, double2* work,
                        double2* chi, int* status, hipStream_t st) {
    TM_CHECK(nz >= 1 && nz <= 4, TM_EINVAL, "1 to 4 measure rows");
    const long long per = (long long)M * nw;
    TM_LAUNCH(k_chi_pivoted, dim3((nw + 63) / 64), dim3(64), 0, st, alpha, beta, gamma, z, nz, cap, M, n1, omega, nw,
              eta, work, work + per, work + 2 * per, work + 3 * per, chi, status);
}

}  // namespace tml
