// Arguments of the plane kernels (generic ones in apply.hip, fixed-size ones in plane.hip).
#pragma once

#include "tm_internal.h"

namespace tml {

// Several right-hand sides run as one batch: batch b of the grid is side and
// k point b % nb2 of right-hand side b / nb2.  Sphere tables are per b % tmod
// (tmod = nb2 when every right-hand side has the same q set; nb2 times the
// right-hand sides when each has its own); columns, densities, fields and W
// are per b (or per right-hand side).
struct PlaneArgs {
    int n1, n2, n3, NP;
    int nk, nb, nitems, bpc, nchunk;
    int cpb;            // chunks of bands per block of the wave kernels (grid.y = nchunk / cpb, rounded up)
    int nb2;            // 2 nk: batches of one right-hand side
    int tmod;           // sphere and slot tables are per b % tmod
    long long wstride;  // elements between the W (and rho) of consecutive right-hand sides (4 N)
    long long fstride;  // elements between the local field tables of consecutive right-hand sides (6 N)
    double2* xcols;
    int ncol_max;
    const double2* ucols;
    int ncol_u_max;
    const int* const* colpos_kq;
    const int* ncol_kq;
    const int* const* colpos_u;
    const int* ncol_u;
    double2* rho_part;
    const double* vrs;
    const double2* W;
    // resident real-space ground state (fixed-size kernels only; null = use
    // ucols): [slot][nb][n3][spin][p2][i1], p2 the digit-reversed position of
    // i2, time reversal applied on the y side
    double2* ureal;
    const int* uslot;  // [2nk] slot of each batch
    double2* fields;   // [n3][n1*n2][6] local fields (k_fields_w)
    // single-precision views of xcols, rho_part and fields (FP32 bulk path)
    float2* xcols32;
    float2* rho_part32;
    float2* fields32;
};

// rows of the (i1, i2) plane occupied by each sphere, per batch b
struct PlaneTabs {
    const int* nrows_kq;
    const int* nrows_u;
    const unsigned long long* rmask_kq;
    const unsigned long long* rmask_u;
    const int* const* rows_kq;
    const int* const* rows_u;
    const double2* tw1;  // exp(-2 pi i j / n1)
    const double2* tw2;  // exp(-2 pi i j / n2)
    const int* perm1;    // mixed-radix digit reversal of the in-place transforms along i1
    const int* perm2;    // and along i2
    const short* const* colidx_kq;  // [n1*n2] column of the k+q sphere at each plane position, or -1
    const float2* tw1f;  // single-precision twiddles (FP32 bulk path)
    const float2* tw2f;
};

// position p of an in-place decimation-in-frequency transform of length n holds
// output index perm[p] (radices 4, 5, 3, 2 in that order)
std::vector<int> digit_reversal(int n);

// arguments of the fixed-size z passes (sphere <-> columns along i3)
struct ZPassArgs {
    int nb2;                           // the table period: sphere and per-batch tables are per b % nb2
                                       // (2 nk, or 2 nk times the right-hand sides when each has its own q set)
    const double2* const* coef_table;  // inverse: per-batch coefficient base, or null
    const double2* coef_base;          //          else coef_base + b * coef_bstride
    long long coef_bstride;
    long long istride;                 // complex elements between items
    const int* istride_tab;            // per-batch item stride (overrides when non-null)
    const int* const* colptr;
    const int* const* entg;
    const int* const* enti3;
    const int* ncol;
    double2* cols;                     // [b][item][n3][ncol_stride]
    float2* cols32;                    // the same in single precision (FP32 bulk path)
    int ncol_stride;
    int nitems;
    const double2* tw;                 // exp(-2 pi i j / n3)
    const float2* tw32;
    const int* perm;                   // digit reversal along i3
    // forward only
    const int* npw;
    const double* const* kin;
    const double* const* eps;
    const double2* xin;
    double2* out;
    int npw_pad;
    double inv_n;
};

bool zpass_fixed_supported(int n3);
void launch_zpass_fixed(bool inverse, const ZPassArgs& a, int ncolmax, int nbatch, int n3, hipStream_t st,
                        bool fp32 = false);

// radix plan of the fixed plane sizes; position p of a digit-reversed line holds
// element sum_s d_s pre[s], p = sum_s d_s n / (pre[s] rad[s])
struct CPlan {
    int nrad;
    int rad[8];
    int pre[8];  // product of the radices before stage s
};

constexpr CPlan cplan(int n) {
    CPlan p{};
    p.nrad = 0;
    int m = n, pre = 1;
    const int order[4] = {4, 5, 3, 2};
    for (int oi = 0; oi < 4; ++oi) {
        int r = order[oi];
        while (m % r == 0) {
            p.rad[p.nrad] = r;
            p.pre[p.nrad] = pre;
            pre *= r;
            ++p.nrad;
            m /= r;
        }
    }
    return p;
}

// arguments of the matrix-core plane kernels (planemx.hip)
struct MxArgs {
    int n1, n2, n3, nk, nb, nitems;
    int nb2, tmod;               // see PlaneArgs
    int m1, m2;                  // |m1|, |m2| of every sphere of the system, at most
    int pitch, sp;               // row buffer: elements between rows, and between the spins
    int ncol_max, ncol_u_max;
    int nchunk, bpc;             // chunks of bands of the density partials, and bands in one
    int cpb;                     // of them in a block (density)
    int bb, bpb;                 // bands in a group, in a block (apply)
    int rtiles;                  // row tiles of a group
    int cwaves, rwaves;          // column and row waves of a block (density)
    int nbatch, ny;              // batches, and blocks of one batch and plane
    int cgroups;                 // blocks the columns are split over (density)
    bool dbuf;                   // two row buffers (density)
    long long fstride;           // elements between the field tables of right-hand sides
    double2* xcols;              // [batch][item][n3][ncol_max]
    const double2* ucols;        // column path: [2 nk][item][n3][ncol_u_max]
    const short* const* colidx_x;  // [n1 n2] column of the k+q sphere at a plane position, or -1
    const short* const* colidx_u;  // the same for the ground-state sphere
    double2* rho_part;           // [batch][chunk][4][N]
    double2* fields;             // laid out by launch_fields_mx
    const double2* ureal;        // [slot][nb][n3][spin][digit-reversed row][column], or null: column path
    const int* uslot;
    const double2 *ctab1, *ctab2;    // mx_constants of both axes
    const double2 *twist1, *twist2;  // mx_twists of both axes
};
// row buffer: an odd pitch (a column's rows fall into distinct LDS banks), the
// two spins of a column tile's rows 8 banks of 16 bytes apart
__host__ __device__ constexpr int mx_pitch(int n2) { return n2 | 1; }
__host__ __device__ constexpr int mx_spin_stride(int n2, int m1) {
    return ((2 * m1 + 1) * mx_pitch(n2) + 7) / 16 * 16 + 8;
}
constexpr int kMxSide = 64;  // longest side of a plane they take
bool mx_supported(int n1, int n2, int m1, int m2);
// The reach up to which they take the resident ground state's planes.  At 48 x
// 48 a sphere that reaches 23 has 6 K steps, twice the products of the
// half-filled one, and spills: 907 us an apply (48^3, 16 bands) against 756 us of
// the wave kernels; reach 12 still 430 against 472.  The smaller planes stay
// ahead up to the fullest sphere (20^3, reach 9: 132 both; 24^3, 11: 272 against
// 318; 32^3, 15: 321 against 328).
constexpr int mx_resident_reach(int n1) { return n1 == 48 ? 13 : n1 / 2 - 1; }
// The same for the column path of those planes, where the ground state is
// transformed too: half-filled spheres are ahead (24^3, reach 6: 236 us against
// 267; 48^3, 11: 404 against 452), full ones are not (24^3, 9: 348 against 322;
// 48^3, 18: 1277 against 817).  Other planes have no kernels with compile-time
// sizes, and there the fullest is still ahead of the generic ones (45 x 40 x 40,
// reach 19: 1010 against 1536; 60^3, 18: 1054 against 2320).
constexpr int mx_column_reach(int n1) { return n1 == 8 ? 3 : 7 * n1 / 24; }
// Rows j of the pairs, their number rounded up to K steps of 4, and the elements
// between the rows of an axis' constants (odd)
__host__ __device__ constexpr int mx_pairs(int n) { return (n + 1) / 2; }
__host__ __device__ constexpr int mx_steps(int n) { return (mx_pairs(n) + 3) / 4; }
__host__ __device__ constexpr int mx_stride(int n) { return 4 * mx_steps(n) + 1; }
// partner of row j
__host__ __device__ constexpr int mx_partner(int n, int j) { return n % 2 == 0 ? n - 1 - j : j == 0 ? 0 : n - j; }
// the row that the partners of rows j0 + k (j0 a multiple of 4, k = 0 .. 3) are
// counted from: 3 - k rows on (the first ones of odd n: n - k, row 0 its own)
__host__ __device__ constexpr int mx_partner_base(int n, int j0) {
    return n % 2 == 0 ? n - 4 - j0 : j0 == 0 ? 0 : n - 3 - j0;
}
// row of the resident ground state that holds row j0 (a multiple of 4) of a plane
// of n: the digits of j0 / 4 reversed (rows j0 + k are k n / 4 further, every
// resident size having 4 as its first radix)
__host__ __device__ constexpr int mx_resident_row(int n, int j0) {
    const CPlan p = cplan(n);
    int d = j0 / 4, w = n / 4, r = 0;
    for (int s = 1; s < p.nrad; ++s) {
        w /= p.rad[s];
        r += d % p.rad[s] * w;
        d /= p.rad[s];
    }
    return r;
}
// constants of the transforms of length n: rows m = 0 .. 23 of (cos, sin), see
// planemx.hip, and the twists exp(-i pi m / n) (1 for odd n)
std::vector<double2> mx_constants(int n);
std::vector<double2> mx_twists(int n);
constexpr int kMxVariants = 3;  // of the apply: bands in a group 1, 2, 4 at most
// density: returns the partial sums of a batch that it wrote, a.nchunk at most
int launch_plane_mx(bool density, const MxArgs& a, int nbatch, int variant, hipStream_t st);
void launch_fields_mx(const double* vrs, const double2* W, double2* fields, int n1, int n2, int n3, long long wstride,
                      long long fstride, int nrhs, hipStream_t st);

// response density and potential by planes and columns (potential.hip)
constexpr long long kPotLdsMax = 1024;  // grids up to here: k_potential_lds
bool pot_planes_supported(const System& s);
// partials -> ws.rho, and the charge transformed in its planes -> ws.work
void launch_rho_planes(const System& s, const void* part, bool single, int nk, int nparts, bool turned, double scale,
                       int nrhs, hipStream_t st);
// ws.work, ws.rho -> W, or the field tables if fields is given
void launch_pot_planes(const System& s, const QSet& q, double2* fields, long long fstride, int nrhs, hipStream_t st);

bool plane_fixed_supported(int n1, int n2);
void launch_plane_fixed(bool density, const PlaneArgs& a, const PlaneTabs& t, dim3 grid, int n1, int n2,
                        hipStream_t st, bool fp32 = false);
// fills a.ureal for the batches of the grid from a.ucols
void launch_ureal_fixed(const PlaneArgs& a, const PlaneTabs& t, dim3 grid, int n1, int n2, hipStream_t st);

}  // namespace tml
