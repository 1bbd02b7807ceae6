// Response density and potential of an apply, one plane or one column tile per
// block: the partial densities of the plane kernels are added up plane by plane
// and the charge component goes to G space in the plane while it is in LDS;
// columns along i3 are transformed, multiplied by the Coulomb kernel (Eq.
// v_H_q, normalisation included) and transformed back in one pass; then each
// plane goes back to real space in LDS and meets the exchange-correlation
// kernel (Eqs. v_XC_q, b_XC_q), whose result leaves as W, or directly as the
// field table of the matrix-core plane kernels.
//
// Three launches and 1.5 passes over each array in place of ten launches (sum,
// copy, three axes forward, multiply, three axes back, W, fields), which were
// bound by their own latency of 5 to 15 us each.  us for the whole stage, before
// -> after: 24^3, 16 bands, 4 k: 90 -> 20; 48 x 48 x 96, 64 bands: 127 -> 61 (the
// partials' bytes at the rate of a copy 24 of them); 20^3, where one block had the
// grid in LDS: 40 -> 14.  Grids of more than kPotLdsMax points: below, that one
// launch is as fast (8^3: 43 us an apply either way).
#include <algorithm>

#include "fft_lds.h"
#include "plane.h"

namespace tml {

namespace {

constexpr int kPotNT = 512;  // threads of the generic plane kernels
constexpr int kZNT = 256;    // of the column kernel

template <int N>
constexpr int plane_threads_ct() { return N == 20 ? 448 : N == 24 ? 576 : kPotNT; }

// The plane in LDS: rows i1 an odd pitch apart (both axes free of bank
// conflicts), the twiddles of both axes behind it.  N > 0: N x N, known at
// compile time.
template <int N>
struct PotPlane {
    static constexpr int NT = plane_threads_ct<N>();
    double2 *g, *tw1, *tw2;
    int n1, n2, pitch;
    __device__ PotPlane(double2* lds, int m1, int m2, const FFTPlan& p1, const FFTPlan& p2) {
        n1 = N > 0 ? N : m1;
        n2 = N > 0 ? N : m2;
        pitch = n2 | 1;
        g = lds;
        tw1 = lds + n1 * pitch;
        tw2 = tw1 + n1;
        for (int i = threadIdx.x; i < n1; i += NT) tw1[i] = p1.tw[i];
        for (int i = threadIdx.x; i < n2; i += NT) tw2[i] = p2.tw[i];
    }
    __device__ double2& at(int i1, int i2) const { return g[i1 * pitch + i2]; }
    __device__ double2& flat(int p) const {
        const int i1 = index_div(p, n2);
        return at(i1, p - i1 * n2);
    }
    // after a barrier; ends with one
    __device__ void transform(const FFTPlan& p1, const FFTPlan& p2, int sign) const {
        if constexpr (N > 0) {
            ct_fft<N, N, NT>(g, StrideLines{N | 1}, 1, tw2, sign);
            ct_fft<N, N, NT>(g, StrideLines{1}, N | 1, tw1, sign);
        } else {
            lds_fft_lines(g, n1, StrideLines{pitch}, 1, p2, tw2, sign);
            lds_fft_lines(g, n2, StrideLines{1}, pitch, p1, tw1, sign);
        }
    }
};
size_t plane_lds(int n1, int n2) { return ((size_t)n1 * (n2 | 1) + n1 + n2) * sizeof(double2); }

// Plane blockIdx.x of component blockIdx.y of right-hand side blockIdx.z: the
// sum of the partials to rho, and of the charge its transform in the plane to
// work.  TURNED: the partials' planes are [i2][i1] (the matrix-core kernels'),
// a batch's parts summed by themselves as those kernels add them up; else
// [i1][i2] and all parts of a side in one sum.
template <class T2, bool TURNED, int N>
__global__ void __launch_bounds__(plane_threads_ct<N>()) k_rho_planes(const T2* part, double2* rho, double2* work,
                                                                     int m1, int m2, int n3, FFTPlan p1, FFTPlan p2,
                                                                     int nk, int nparts, double scale) {
    extern __shared__ double2 lds[];
    const PotPlane<N> pl(lds, m1, m2, p1, p2);
    constexpr int NT = PotPlane<N>::NT;
    const int n1 = pl.n1, n2 = pl.n2, NP = n1 * n2;
    const int i3 = blockIdx.x, comp = blockIdx.y, rhs = blockIdx.z;
    const long long N3 = (long long)NP * n3, stride = 4 * N3;
    part += rhs * 2LL * nk * nparts * stride + comp * N3 + (long long)i3 * NP;
    rho += (rhs * 4LL + comp) * N3 + (long long)i3 * NP;
    const double sgn = comp == 0 ? 1.0 : -1.0;
    for (int p = threadIdx.x; p < NP; p += NT) {
        const T2* x = part + p;
        const T2* y = x + (long long)nk * nparts * stride;
        double2 sx = cmk(0.0, 0.0), sy = cmk(0.0, 0.0);
        if constexpr (TURNED) {
            double2 bx = cmk(0.0, 0.0), by = cmk(0.0, 0.0);
            int left = nparts;
#pragma unroll 8
            for (int c = 0; c < nk * nparts; ++c) {  // both sides' loads in flight together
                bx = cadd(bx, Cx<double2>::from(x[c * stride]));
                by = cadd(by, Cx<double2>::from(y[c * stride]));
                if (--left == 0) {  // a batch's sum is whole
                    sx = cadd(sx, bx);
                    sy = cadd(sy, by);
                    bx = by = cmk(0.0, 0.0);
                    left = nparts;
                }
            }
        } else {
#pragma unroll 8
            for (int c = 0; c < nk * nparts; ++c) sx = cadd(sx, Cx<double2>::from(x[c * stride]));
#pragma unroll 8
            for (int c = 0; c < nk * nparts; ++c) sy = cadd(sy, Cx<double2>::from(y[c * stride]));
        }
        const double2 r = cscale(cmk(sx.x + sgn * sy.x, sx.y + sgn * sy.y), scale);
        if (TURNED) {
            pl.at(p - index_div(p, n1) * n1, index_div(p, n1)) = r;
        } else {
            rho[p] = r;
            if (comp == 0) pl.flat(p) = r;
        }
    }
    if (!TURNED && comp > 0) return;
    __syncthreads();
    if (TURNED)
        for (int p = threadIdx.x; p < NP; p += NT) rho[p] = pl.flat(p);
    if (comp > 0) return;
    if (TURNED) __syncthreads();
    pl.transform(p1, p2, -1);
    work += rhs * N3 + (long long)i3 * NP;
    for (int p = threadIdx.x; p < NP; p += NT) work[p] = pl.flat(p);
}

// L columns along i3 of right-hand side blockIdx.y: forward, times the Coulomb
// multiplier, back.  N3 > 0: known at compile time.
template <int N3, int L>
__global__ void __launch_bounds__(kZNT) k_pot_columns(double2* work, const double* const* hqt, int hmod, int NP,
                                                      int m3, FFTPlan p3) {
    extern __shared__ double2 lds[];
    const int n3 = N3 > 0 ? N3 : m3;
    constexpr int pitch = L + 1;
    double2* tw = lds + n3 * pitch;
    const int c0 = blockIdx.x * L;
    work += (long long)blockIdx.y * NP * n3;
    const double* h = hqt[blockIdx.y % hmod];
    for (int i = threadIdx.x; i < n3; i += kZNT) tw[i] = p3.tw[i];
    for (int i = threadIdx.x; i < n3 * L; i += kZNT) {
        const int t = i / L, l = i - t * L;
        lds[t * pitch + l] = c0 + l < NP ? work[(long long)t * NP + c0 + l] : cmk(0.0, 0.0);
    }
    __syncthreads();
    auto transform = [&](int sign) {
        if constexpr (N3 > 0) ct_fft<N3, L, kZNT>(lds, StrideLines{1}, pitch, tw, sign);
        else lds_fft_lines(lds, L, StrideLines{1}, pitch, p3, tw, sign);
    };
    transform(-1);
    for (int i = threadIdx.x; i < n3 * L; i += kZNT) {
        const int t = i / L, l = i - t * L;
        if (c0 + l < NP) lds[t * pitch + l] = cscale(lds[t * pitch + l], h[(long long)t * NP + c0 + l]);
    }
    __syncthreads();
    transform(+1);
    for (int i = threadIdx.x; i < n3 * L; i += kZNT) {
        const int t = i / L, l = i - t * L;
        if (c0 + l < NP) work[(long long)t * NP + c0 + l] = lds[t * pitch + l];
    }
}

// Plane blockIdx.x of right-hand side blockIdx.z: W_a = delta_a0 vH + sum_b f_ab
// rho_b (f stored as 00,01,02,03,11,12,13,22,23,33) as W, or (FIELDS) as the
// field table of the matrix-core kernels (k_fields_mx).  Blocks with blockIdx.y
// < 2 transform vH back (both) and form what contains it for half of the points;
// the other two form the rest.  (48 x 48 x 96: 23.3 us, as two blocks a
// plane 25.4; 48 x 48 x 180: 36.3 and 42.2.)
template <bool FIELDS, int N>
__global__ void __launch_bounds__(plane_threads_ct<N>()) k_pot_planes(const double2* work, const double2* rho,
                                                                     const double* fxc, const double* vrs, double2* W,
                                                                     double2* F, int m1, int m2, int n3, FFTPlan p1,
                                                                     FFTPlan p2, long long fstride) {
    extern __shared__ double2 lds[];
    const PotPlane<N> pl(lds, m1, m2, p1, p2);
    constexpr int NT = PotPlane<N>::NT;
    const int n1 = pl.n1, n2 = pl.n2, NP = n1 * n2;
    const int i3 = blockIdx.x, rhs = blockIdx.z;
    const bool first = blockIdx.y < 2;
    const int half = blockIdx.y & 1;
    const long long NN = (long long)NP * n3, off = (long long)i3 * NP;
    rho += rhs * 4 * NN + off;
    fxc += off;
    if (first) {
        work += rhs * NN + off;
        for (int p = threadIdx.x; p < NP; p += NT) pl.flat(p) = work[p];
        __syncthreads();
        pl.transform(p1, p2, +1);
    }
    auto comb = [&](const double2 (&r)[4], double a0, double a1, double a2, double a3) {
        return cmk(a0 * r[0].x + a1 * r[1].x + a2 * r[2].x + a3 * r[3].x,
                   a0 * r[0].y + a1 * r[1].y + a2 * r[2].y + a3 * r[3].y);
    };
    if constexpr (FIELDS) {
        // tiles of 16 x 16 points, so that both sides of the transposition go in whole lines
        vrs += off;
        double2* f = F + rhs * fstride + (long long)i3 * 6 * NP;
        const int t1 = (n1 + 15) / 16, t2 = (n2 + 15) / 16;
        const int all = t1 * t2 * 256, per = (t1 * t2 + 1) / 2 * 256;
        for (int i = half * per + threadIdx.x; i < min(all, (half + 1) * per); i += NT) {
            const int tile = i >> 8, i2 = tile / t1 * 16 + (i >> 4 & 15), i1 = tile % t1 * 16 + (i & 15);
            if (i1 >= n1 || i2 >= n2) continue;
            const int p = i1 * n2 + i2, up = i2 * 2 * n1 + i1, dn = up + n1;  // [i2][spin][i1]
            double2 r[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) r[c] = rho[c * NN + p];
            if (first) {
                const double f03 = fxc[3 * NN + p];
                const double2 w0 = cadd(pl.at(i1, i2), comb(r, fxc[p], fxc[NN + p], fxc[2 * NN + p], f03));
                const double2 wz = comb(r, f03, fxc[6 * NN + p], fxc[8 * NN + p], fxc[9 * NN + p]);
                f[2 * NP + up] = cadd(w0, wz);
                f[2 * NP + dn] = csub(w0, wz);
            } else {
                const double v = vrs[p], bx = vrs[NN + p], by = vrs[2 * NN + p], bz = vrs[3 * NN + p];
                const double f12 = fxc[5 * NN + p];
                const double2 wx = comb(r, fxc[NN + p], fxc[4 * NN + p], f12, fxc[6 * NN + p]);
                const double2 wy = comb(r, fxc[2 * NN + p], f12, fxc[7 * NN + p], fxc[8 * NN + p]);
                double* d = reinterpret_cast<double*>(f);
                d[up] = v + bz;
                d[dn] = v - bz;
                f[NP + i2 * n1 + i1] = cmk(bx, by);
                f[4 * NP + up] = cadd(wx, cmuli(wy));
                f[4 * NP + dn] = csub(wx, cmuli(wy));
            }
        }
    } else {
        W += rhs * 4 * NN + off;
        const int per = (NP + 1) / 2;
        for (int p = half * per + threadIdx.x; p < min(NP, (half + 1) * per); p += NT) {
            double2 r[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) r[c] = rho[c * NN + p];
            auto f = [&](int t) { return fxc[t * NN + p]; };
            if (first) {
                W[p] = cadd(pl.flat(p), comb(r, f(0), f(1), f(2), f(3)));
            } else {
                W[NN + p] = comb(r, f(1), f(4), f(5), f(6));
                W[2 * NN + p] = comb(r, f(2), f(5), f(7), f(8));
                W[3 * NN + p] = comb(r, f(3), f(6), f(8), f(9));
            }
        }
    }
}

template <class... A, class... B>
void launch_pot(const char* name, void (*kernel)(A...), dim3 grid, int nt, size_t shm, hipStream_t st, B... args) {
    TM_CHECK(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm) ==
                 hipSuccess,
             TM_EDEVICE, std::string("cannot raise the LDS limit of ") + name);
    ProfScope ps(name, st);
    hipLaunchKernelGGL(kernel, grid, dim3(nt), shm, st, static_cast<A>(args)...);
    check_launch(name);
}

int smallest_radix(const FFTPlan& p) {
    int m = p.n;
    for (int r = 0; r < p.nrad; ++r) m = std::min(m, p.rad[r]);
    return m;
}

// f(std::integral_constant<int, N>) for the square planes known at compile time, N = 0 for the others
template <class F>
void with_plane(const System& s, F f) {
    const int n = s.n1 == s.n2 ? s.n1 : 0;
    if (n == 20) f(std::integral_constant<int, 20>());
    else if (n == 24) f(std::integral_constant<int, 24>());
    else if (n == 32) f(std::integral_constant<int, 32>());
    else if (n == 48) f(std::integral_constant<int, 48>());
    else f(std::integral_constant<int, 0>());
}

// columns a block: 16, or 8 where that leaves less than a block a CU or does not fit
int pot_columns(const System& s) {
    const int NP = s.n1 * s.n2;
    const long long fly = s.n3 / smallest_radix(s.plan[2]);
    if (NP / 16 >= 256 && 16 * fly <= kMaxBfly * kZNT && (size_t)s.n3 * 18 * sizeof(double2) <= 64 * 1024) return 16;
    return 8;
}

}  // namespace

// Grids with columns that 8 of fit a block (butterflies a thread, LDS; up to 256
// points at radix 2); planes of 4096 points, the most that the plane kernels
// take, always do.  Longer columns keep the line transforms over the whole grid.
bool pot_planes_supported(const System& s) {
    if ((long long)s.n1 * s.n2 * s.n3 <= kPotLdsMax) return false;
    const long long NP = (long long)s.n1 * s.n2;
    const int r = std::min(smallest_radix(s.plan[0]), smallest_radix(s.plan[1]));
    return plane_lds(s.n1, s.n2) <= 150 * 1024 && NP / r <= (long long)kMaxBfly * kPotNT &&
           8LL * (s.n3 / smallest_radix(s.plan[2])) <= (long long)kMaxBfly * kZNT &&
           (size_t)s.n3 * 10 * sizeof(double2) <= 150 * 1024;
}

void launch_rho_planes(const System& s, const void* part, bool single, int nk, int nparts, bool turned, double scale,
                       int nrhs, hipStream_t st) {
    const dim3 grid(s.n3, 4, nrhs);
    with_plane(s, [&](auto nn) {
        constexpr int N = decltype(nn)::value;
        auto launch = [&](auto kernel, auto* p) {
            launch_pot("k_rho_planes", kernel, grid, plane_threads_ct<N>(), plane_lds(s.n1, s.n2), st, p, s.ws.rho, s.ws.work,
                       s.n1, s.n2, s.n3, s.plan[0], s.plan[1], nk, nparts, scale);
        };
        if (single) launch(k_rho_planes<float2, false, N>, (const float2*)part);
        else if (turned) launch(k_rho_planes<double2, true, N>, (const double2*)part);
        else launch(k_rho_planes<double2, false, N>, (const double2*)part);
    });
}

void launch_pot_planes(const System& s, const QSet& q, double2* fields, long long fstride, int nrhs, hipStream_t st) {
    const int NP = s.n1 * s.n2;
    auto columns = [&](auto kernel, int L) {
        launch_pot("k_pot_columns", kernel, dim3((NP + L - 1) / L, nrhs), kZNT,
                   (size_t)s.n3 * (L + 2) * sizeof(double2), st, s.ws.work, (const double* const*)q.d_hqt, q.hmod, NP, s.n3,
                   s.plan[2]);
    };
    const bool wide = pot_columns(s) == 16;
    switch (s.n3) {
        case 20: columns(k_pot_columns<20, 8>, 8); break;
        case 24: columns(k_pot_columns<24, 8>, 8); break;
        case 32: columns(k_pot_columns<32, 8>, 8); break;
        case 48: columns(k_pot_columns<48, 8>, 8); break;
        case 96: columns(k_pot_columns<96, 8>, 8); break;
        case 180: columns(k_pot_columns<180, 8>, 8); break;
        default:
            if (wide) columns(k_pot_columns<0, 16>, 16);
            else columns(k_pot_columns<0, 8>, 8);
    }
    const dim3 grid(s.n3, 4, nrhs);
    with_plane(s, [&](auto nn) {
        constexpr int N = decltype(nn)::value;
        auto kernel = fields ? k_pot_planes<true, N> : k_pot_planes<false, N>;
        launch_pot("k_pot_planes", kernel, grid, plane_threads_ct<N>(), plane_lds(s.n1, s.n2), st, s.ws.work, s.ws.rho, s.fxc,
                   s.vrs, s.ws.W, fields, s.n1, s.n2, s.n3, s.plan[0], s.plan[1], fstride);
    });
}

}  // namespace tml
