// Plane kernels of the Liouvillian on the matrix cores.
//
// A band's spinor arrives at a plane i3 as its z-transformed columns: the few
// (m1, m2) of the plane-wave sphere, |m1| <= M1, |m2| <= M2, out of n1 x n2.
// The in-plane transforms are products with the pruned DFT matrices instead of
// radix passes over LDS lines.  For even n, grid rows come in pairs j and
// -1 - j about -1/2: with the input twisted by exp(-i pi m / n),
//     s_m = x_m + x_-m,   d_m = x_m - x_-m,
//     C(j) = sum_m s_m cos(2 pi (j + 1/2) m / n),   S(j) = sum_m d_m sin(2 pi (j + 1/2) m / n),
//     X(j) = C(j) + i S(j),   X(-1 - j) = C(j) - i S(j),   0 <= j < n/2,
// so a length-n inverse transform is two real (n/2) x (M+1) matrices applied to
// complex vectors, and no row is its own partner.  (Odd n: pairs j and -j, no
// twist, 2 pi j m / n.)  The forward one is the same with j and m exchanged
// (F(+-m) = C'(m) -+ i S'(m), s_j and d_j from the products), its result
// twisted back.  At half-filled spheres that is about the multiply count of a
// mixed-radix FFT, all of it v_mfma_f64_16x16x4.
//
// The accumulator layout of these instructions (element v of lane l: row
// 4 v + l / 16, column l % 16) is the operand layout of their second factor at
// K step v, so along axis 1 the inverse transform, the point-wise products and the
// forward transform follow each other in registers: of a plane only the
// occupied rows pass through LDS, once in each direction, to turn the row
// transforms (along axis 2) into the column transforms (along axis 1).
//
// A column tile is 8 columns of both spins (lane % 16 = 8 spin + column): the
// two spins of a point sit 8 lanes apart, and the spin-mixing terms cross by
// one DPP rotation of a complex value.
//
// Axis 1 (rows, the columns' K axis) is the plane's i2 and axis 2 its i1: the
// resident ground state is kept as columns of i1 (which the wave kernels of
// plane.hip read one after the other), so that the 8 columns of a tile are one
// 128-byte line of it.
//
// Against the radix kernels these replace (FP64, us a launch, before -> after):
//   48 x 48 x 180, 104 bands, 4 k, resident: density 3028 -> 2470, apply 6206 -> 4583
//   48 x 48 x 96, 64 bands, 1 k, resident:   density  367 -> 204,  apply  524 -> 413
//   24 x 24 x 24, 16 bands, 4 k, resident:   density 47.3 -> 24.8, apply 63.1 -> 31.4
//   45 x 40 x 50, 12 bands, column path:     density  606 -> 60,   apply  765 -> 87
//   24 x 20 x 18, 5 bands, column path:      density  132 -> 11.6, apply  189 -> 11.7
// FP64 only: in FP32 (v_mfma_f32_16x16x4) the 48 x 48 x 180 apply takes 3751 us
// against the wave kernel's 4903, but results would round in another order.
#include <type_traits>

#include "plane.h"

namespace tml {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4d mfma(double a, double b, v4d c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// the value 8 lanes away in the row of 16
__device__ __forceinline__ double swap(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x128, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x128, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double2 swap(double2 x) { return cmk(swap(x.x), swap(x.y)); }

// Shape of a plane: N > 0, square planes of that size whose spheres reach
// |m| <= M at most (everything folds to constants; the resident ground state);
// N = 0, any plane and reach up to 4 KS - 1, from the arguments (the column path).
template <int N, int M>
struct Shape {
    static constexpr bool fixed = N > 0;
    __device__ static int n1(const MxArgs& a) { return fixed ? N : a.n1; }
    __device__ static int n2(const MxArgs& a) { return fixed ? N : a.n2; }
    __device__ static int m1(const MxArgs& a) { return fixed ? M : a.m1; }
    __device__ static int m2(const MxArgs& a) { return fixed ? M : a.m2; }
    __device__ static int pitch(const MxArgs& a) { return fixed ? mx_pitch(N) : a.pitch; }
    __device__ static int sp(const MxArgs& a) { return fixed ? mx_spin_stride(N, M) : a.sp; }
};

// The constants of one axis: (cos, sin) of row m = 0 .. 4 KS - 1 and column j
// (zero past the last pair), rows an odd number of elements apart.  Both
// transforms read their first factor there: the inverse one rows j of column
// block m (16 neighbours), the forward one rows m at column j (an odd stride),
// neither with LDS bank conflicts.  (Reads past the table's last rows meet the
// row buffer behind it and only make results that are not used.)
template <int KS>
__host__ __device__ constexpr int mx_table(int n) {
    return 4 * KS * mx_stride(n);
}
// planes whose last row tile is at most half full: a density wave takes it for two column tiles
__host__ __device__ constexpr bool mx_paired(int n) { return n > 32 && mx_pairs(n) % 16 > 0 && mx_pairs(n) % 16 <= 8; }

// Inverse transform of 16 columns: C and S of a row tile.
template <int KS>
struct Inverse {
    v4d cr, ci, ssr, ssi;
    __device__ __forceinline__ void clear() { cr = ci = ssr = ssi = v4d{0, 0, 0, 0}; }
    // K step st: p = x_m, q = x_-m (zero for m = 0 and past M); tab: the axis'
    // constants at row tile t of the lane
    __device__ __forceinline__ void step(const double2* tab, int st, int stride, double2 p, double2 q) {
        const double2 c = tab[4 * st * stride];
        cr = mfma(c.x, p.x + q.x, cr);
        ci = mfma(c.x, p.y + q.y, ci);
        ssr = mfma(c.y, p.x - q.x, ssr);
        ssi = mfma(c.y, p.y - q.y, ssi);
    }
    // of the column whose row m = 0 is y: operands read from the row buffer step
    // by step (holding them all costs the registers that the loads in flight need)
    template <class S>
    __device__ __forceinline__ void run_column(const MxArgs& a, const double2* y, int k, const double2* tab, int ks) {
        const int pitch = S::pitch(a), m1 = S::m1(a), stride = mx_stride(S::n1(a));
        clear();
#pragma unroll
        for (int st = 0; st < KS; ++st)
            if (st < ks) {
                const int m = 4 * st + k;
                const bool all = 4 * st + 3 <= m1;  // no lane past M
                const int mc = all || m <= m1 ? m : 0;
                double2 p = y[mc * pitch], q = y[-mc * pitch];
                if (!all && m > m1) p = cmk(0.0, 0.0);
                if ((!all && m > m1) || (st == 0 && m == 0)) q = cmk(0.0, 0.0);
                step(tab, st, stride, p, q);
                __builtin_amdgcn_sched_barrier(0);
            }
    }
    // X at row 4 v + l / 16 of the tile and at its partner
    __device__ __forceinline__ double2 plus(int v) const { return cmk(cr[v] - ssi[v], ci[v] + ssr[v]); }
    __device__ __forceinline__ double2 minus(int v) const { return cmk(cr[v] + ssi[v], ci[v] - ssr[v]); }
};

// Forward transform: accumulates K steps, result F(+-m) at m = 4 i + l / 16.
template <int KS>
struct Forward {
    static constexpr int MT = (KS + 3) / 4;
    v4d cr[MT], ci[MT], ssr[MT], ssi[MT];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int i = 0; i < MT; ++i) cr[i] = ci[i] = ssr[i] = ssi[i] = v4d{0, 0, 0, 0};
    }
    // K step s: p at row j, q at its partner (zero where that is j itself);
    // tab: the axis' constants at the lane
    __device__ __forceinline__ void step(const double2* tab, int s, int stride, double2 p, double2 q) {
        const double sr = p.x + q.x, si = p.y + q.y, dr = p.x - q.x, di = p.y - q.y;
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            const double2 c = tab[16 * i * stride + 4 * s];
            cr[i] = mfma(c.x, sr, cr[i]);
            ci[i] = mfma(c.x, si, ci[i]);
            ssr[i] = mfma(c.y, dr, ssr[i]);
            ssi[i] = mfma(c.y, di, ssi[i]);
        }
    }
    __device__ __forceinline__ double2 plus(int i) const {
        return cmk(cr[i / 4][i % 4] + ssi[i / 4][i % 4], ci[i / 4][i % 4] - ssr[i / 4][i % 4]);
    }
    __device__ __forceinline__ double2 minus(int i) const {
        return cmk(cr[i / 4][i % 4] - ssi[i / 4][i % 4], ci[i / 4][i % 4] + ssr[i / 4][i % 4]);
    }
};

// Loads from a wave-uniform base, a uniform and a lane byte offset (buffer
// loads: the lane holds 32 bits of address per access pattern and no sums of
// them; an element past the buffer reads as zero).
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));
struct Buf {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Buf(const void* p, unsigned bytes)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000)) {}
    // AUX: cache policy (2: streamed, not kept in L2)
    template <class E, int AUX = 0>
    __device__ __forceinline__ E at(unsigned lane_off, unsigned off) const {
        if constexpr (sizeof(E) == 16) {
            const v4u x = __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)off, AUX);
            return __builtin_bit_cast(E, x);
        } else if constexpr (sizeof(E) == 8) {
            const v2u x = __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane_off, (int)off, AUX);
            return __builtin_bit_cast(E, x);
        } else {
            const unsigned x = __builtin_amdgcn_raw_buffer_load_b32(r, (int)lane_off, (int)off, AUX);
            return __builtin_bit_cast(E, x);
        }
    }
};

// Blocks go to the 8 XCDs in turn: give each XCD a contiguous run of the work
// list (batch fastest, then band groups, then planes), so that the blocks
// sharing an L2 work on the same few planes and their field tables stay in it.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_order(int id, int total) {
    const int per = total / kXcds, rem = total % kXcds;
    const int x = id % kXcds, i = id / kXcds;
    return x * per + min(x, rem) + i;
}

// Lane coordinates, LDS pieces and the constants of a block.
template <int KS, int N, int M>
struct MxBlock {
    using S = Shape<N, M>;
    int k, n;                 // lane / 16, lane % 16
    // constants along axes 1 and 2 at the lane: first factor of the inverse
    // transform (row j of tile 0) and of the forward one (row m of tile 0)
    const double2 *inv1, *inv2, *fwd1, *fwd2;
    double2* Y;                    // row buffer(s)

    __device__ __forceinline__ void init(const MxArgs& a, double2* lds, int nt) {
        const int n1 = S::n1(a), n2 = S::n2(a);
        const int lane = threadIdx.x & 63;
        k = lane >> 4;
        n = lane & 15;
        const int e1 = mx_table<KS>(n1);
        const double2* g1 = a.ctab1;
        for (int i = threadIdx.x; i < e1; i += nt) lds[i] = g1[i];
        double2* t2 = lds;
        Y = lds + e1;
        if (!S::fixed && n1 != n2) {
            const int e2 = mx_table<KS>(n2);
            const double2* g2 = a.ctab2;
            t2 = Y;
            for (int i = threadIdx.x; i < e2; i += nt) t2[i] = g2[i];
            Y = t2 + e2;
        }
        inv1 = lds + k * mx_stride(n1) + n;
        inv2 = t2 + k * mx_stride(n2) + n;
        fwd1 = lds + n * mx_stride(n1) + k;
        fwd2 = t2 + n * mx_stride(n2) + k;
    }
};

// A tile of 16 lines of a band group: line = (x or ground state, band of the
// group, spin, row m1).  The lane's line is column lane % 16 of its operands.
template <int KS, bool RES, int N, int M>
struct RowTile {
    using S = Shape<N, M>;
    using B = MxBlock<KS, N, M>;
    static constexpr unsigned kNone = 0xffff;
    bool live;                // the lane has a line
    int kind, bl;             // 0 x, 1 u (column path); band within the group
    int yb;                   // LDS offset of the line
    unsigned cc[KS];          // columns of m2 (low half) and -m2, kNone outside the sphere
    const double2* src;            // the line's columns of band 0 of the group at this plane
    double2 ph;                    // twist of the line's row m1
    const double2* tw2;            // twists along axis 2 at m2 = lane / 16

    // elements between bands in src
    __device__ __forceinline__ long long band(const MxArgs& a) const {
        return 2LL * a.n3 * (RES || kind == 0 ? a.ncol_max : a.ncol_u_max);
    }
    __device__ __forceinline__ unsigned colp(int st) const { return cc[st] & 0xffff; }
    __device__ __forceinline__ unsigned colm(int st) const { return cc[st] >> 16; }

    __device__ __forceinline__ void init(const MxArgs& a, const B& blk, int b, int bt, int tb, int i3, int rt) {
        const int n1 = S::n1(a), n2 = S::n2(a), m1 = S::m1(a), m2 = S::m2(a);
        const int R1 = 2 * m1 + 1;
        const int NL = a.bb * 2 * R1;  // lines of one kind
        const int L = rt * 16 + blk.n;
        kind = RES ? 0 : L / NL;
        live = L < (RES ? 1 : 2) * NL;
        const int L1 = live ? L - kind * NL : 0;
        if (!live) kind = 0;
        bl = L1 / (2 * R1);
        const int rem = L1 - bl * 2 * R1;
        const int s = rem / R1, r = rem - s * R1;
        const int q1 = r - m1, i1 = q1 < 0 ? q1 + n1 : q1;
        yb = kind * a.bb * 2 * S::sp(a) + (bl * 2 + s) * S::sp(a) + r * S::pitch(a);
        const short* ci = (kind == 0 ? a.colidx_x[tb] : a.colidx_u[bt]) + i1;
        const int ncs = kind == 0 ? a.ncol_max : a.ncol_u_max;
        const long long cs = (long long)a.n3 * ncs;
        src = (kind == 0 ? a.xcols + (long long)b * a.nitems * cs
                         : a.ucols + (long long)bt * a.nitems * cs) +
              (long long)i3 * ncs + (2 * bl + s) * cs;
#pragma unroll
        for (int st = 0; st < KS; ++st) {
            const int m = 4 * st + blk.k;
            const bool in = live && m <= m2;
            const int cp = in ? ci[m * n1] : -1;
            const int cm = in && m > 0 ? ci[(n2 - m) * n1] : -1;
            cc[st] = (unsigned)(cp & 0xffff) | ((unsigned)cm << 16);
        }
        const double2* w1 = a.twist1;
        ph = w1[q1 < 0 ? -q1 : q1];
        if (q1 < 0) ph.y = -ph.y;
        tw2 = a.twist2 + blk.k;
    }
    // twists of columns m2 and -m2 of K step st
    __device__ __forceinline__ void twists(int st, double2& p, double2& m) const {
        const double2 w = tw2[4 * st];
        p = cmul(ph, w);
        m = cmulc(w, ph);
    }
    // the lane's row elements of the band group starting at band g
    __device__ __forceinline__ void load(const MxArgs& a, int g, int gend, double2 (&xp)[KS], double2 (&xm)[KS]) const {
        // unconditional loads (past the sphere or the bands: some element of the
        // line's columns, taken as zero by inverse or never used)
        const double2* c = src + (long long)(g + bl < gend ? g : -bl) * band(a);
#pragma unroll
        for (int st = 0; st < KS; ++st) {
            const unsigned p = colp(st), m = colm(st);
            xp[st] = c[p == kNone ? 0 : p];
            xm[st] = c[m == kNone ? 0 : m];
        }
    }
    // inverse transform along axis 2, row tiles t0 .. t1 - 1, into the row buffer Y
    __device__ __forceinline__ void inverse(const MxArgs& a, const B& blk, double2 (&xp)[KS], double2 (&xm)[KS], double2* Y, int t0,
                                            int t1) const {
        Inverse<KS> iv;
        const int n2 = S::n2(a), H = mx_pairs(n2), ks = S::m2(a) / 4 + 1;
#pragma unroll
        for (int st = 0; st < KS; ++st) {
            double2 wp, wm;
            twists(st, wp, wm);
            xp[st] = colp(st) == kNone ? cmk(0.0, 0.0) : cmul(xp[st], wp);
            xm[st] = colm(st) == kNone ? cmk(0.0, 0.0) : cmul(xm[st], wm);
        }
        double2* y = Y + yb;
#pragma unroll 1
        for (int t = t0; t < t1; ++t) {
            iv.clear();
#pragma unroll
            for (int st = 0; st < KS; ++st)
                if (st < ks) iv.step(blk.inv2 + 16 * t, st, mx_stride(n2), xp[st], xm[st]);
            __builtin_amdgcn_sched_barrier(0);
            if (live) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int j = 16 * t + 4 * v + blk.k;
                    if (j < H) {
                        y[j] = iv.plus(v);
                        if (n2 % 2 == 0 || j > 0) y[mx_partner(n2, j)] = iv.minus(v);
                    }
                }
            }
        }
    }
    // forward transform along axis 2 of the x lines of the row buffer, to their columns
    __device__ __forceinline__ void forward(const MxArgs& a, const B& blk, const double2* Y, int g, int gend) const {
        const int n2 = S::n2(a), H = mx_pairs(n2);
        Forward<KS> fw;
        fw.clear();
        const double2* y = Y + (live && kind == 0 ? yb : 0);
#pragma unroll 1
        for (int s = 0; s < mx_steps(n2); ++s) {
            const int j = 4 * s + blk.k;
            const bool in = H % 4 == 0 || j < H;
            double2 p = y[in ? j : 0], q = y[in ? mx_partner(n2, j) : 0];
            if (!in) p = cmk(0.0, 0.0);
            if (!in || (n2 % 2 == 1 && j == 0)) q = cmk(0.0, 0.0);
            fw.step(blk.fwd2, s, mx_stride(n2), p, q);
        }
        if (live && kind == 0 && g + bl < gend) {
            double2* o = const_cast<double2*>(src) + (long long)g * band(a);
#pragma unroll
            for (int i = 0; i < KS; ++i) {
                double2 wp, wm;
                twists(i, wp, wm);
                if (colp(i) != kNone) o[colp(i)] = cmulc(wp, fw.plus(i));
                if (colm(i) != kNone) o[colm(i)] = cmulc(wm, fw.minus(i));
            }
        }
    }
};

// time reversal of the spinor held 8 lanes apart: (up, dn) -> (conj dn, -conj up)
__device__ __forceinline__ double2 time_reversed(double2 u, int spin) {
    const double x = swap(u.x), y = swap(u.y);
    return spin == 0 ? cmk(x, -y) : cmk(-x, y);
}

// phi of the lane's spin at one point: d x + Wd u, plus what the other spin's
// lane adds, b x + Wo u of its own x and u (bsg: the sign of By for this spin,
// sg: of the side).  Every operation spelled out, so that each kernel that
// inlines it rounds alike.
__device__ __forceinline__ double2 local_product(double d, double2 b, double2 wd,
                                                            double2 wo, double2 x,
                                                            double2 u, double bsg, double sg) {
    const double by = b.y * bsg;
    const double cx = fma(-wo.y, u.y, fma(wo.x, u.x, fma(-by, x.y, b.x * x.x)));
    const double cy = fma(wo.y, u.x, fma(wo.x, u.y, fma(by, x.x, b.x * x.y)));
    const double px = fma(-wd.y, u.y, fma(wd.x, u.x, d * x.x));
    const double py = fma(wd.y, u.x, fma(wd.x, u.y, d * x.y));
    return cmk(fma(sg, swap(cx), px), fma(sg, swap(cy), py));
}

// Byte offsets of a lane's points in an array of rows of `stride` bytes: the
// rows j = j0 + k of a K step j0 from the base of row j0, and their partners
// from the base of mx_partner_base(j0) (both bases wave-uniform).
struct RowOff {
    unsigned p, m, m0;  // m0: the partners of the first step (odd n: row 0 is its own)
    __device__ __forceinline__ RowOff(int k, int n, unsigned stride, unsigned lane_off) {
        p = k * stride + lane_off;
        m = (3 - k) * stride + lane_off;
        m0 = n % 2 == 0 ? m : (k == 0 ? 0 : n - k) * stride + lane_off;
    }
};

// Response density.  The waves of a block have two roles: column waves own
// column tiles (kind A: one row tile t of a column tile; kind B, where the last
// row tile is at most half full: that tile of two column tiles) and keep
// u^dag S_a x of their points in registers over the bands of the chunk; row
// waves transform the next band's rows into the other half of the row buffer
// meanwhile.  One barrier a band.  With the roles apart neither holds the
// other's registers, which leaves room for a whole band's ground state in
// flight per column wave.
//
// Bounded by the resident ground state's bytes at 48 x 48 (each point of each
// band is read once: 48 x 48 x 180, 104 bands, 4 k 11.0 GB in 2470 us, 4.5 TB/s;
// 36 k 99.4 GB in 20.7 ms, 4.8, and by the counters 112.8 GB with the columns
// and partials, 5.4 TB/s, more than a device copy's 4.7, with the matrix cores
// 45 % busy); the radix kernel took 3028 us at 4 k, with more of the time in its
// LDS passes than in the loads.  Small planes: by the latency of a band's chain (row transform,
// barrier, column transform, products).
//
// One buffer (two barriers a band) where two do not fit.  TOT: the block has all
// chunks of its batch, and adds their sums up in registers, in the order in which
// the reduction adds partials, to write one.
template <int KS, int JT, bool RES, int N, int M, int NW, int MINW, int RTW, bool TOT>
__global__ void __launch_bounds__(64 * NW, MINW) k_density_mx(MxArgs a) {
    using S = Shape<N, M>;
    extern __shared__ double2 lds_raw[];
    const int n1 = S::n1(a), n2 = S::n2(a), m1 = S::m1(a), sp = S::sp(a), pitch = S::pitch(a);
    const int nt = blockDim.x;
    const int id = xcd_order(blockIdx.x, gridDim.x), by = id / a.nbatch;
    const int b = id - by * a.nbatch, i3 = by / a.ny, yy = by - i3 * a.ny;
    const int bt = b % a.nb2, tb = b % a.tmod;
    const int cg = yy % a.cgroups, ch0 = yy / a.cgroups * a.cpb;
    const int H1 = mx_pairs(n1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n0 = ch0 * a.bpc, n1e = min(a.nb, n0 + a.cpb * a.bpc);
    const int half = (RES ? 1 : 2) * 2 * sp;  // elements of one row buffer (one band)
    MxBlock<KS, N, M> k;
    k.init(a, lds_raw, nt);
    __syncthreads();  // the constant tables
    if (w >= a.cwaves) {
        // row wave: tiles w - cwaves, + rwaves, ...
        const int rw = w - a.cwaves, jt2 = (mx_pairs(n2) + 15) / 16;
        RowTile<KS, RES, N, M> tile[RTW];
        double2 xp[RTW][KS], xm[RTW][KS];
        auto load = [&](int n) {
#pragma unroll
            for (int r = 0; r < RTW; ++r)
                if (rw + r * a.rwaves < a.rtiles) tile[r].load(a, n, n1e, xp[r], xm[r]);
        };
        auto rows = [&](double2* Y) {
#pragma unroll
            for (int r = 0; r < RTW; ++r)
                if (rw + r * a.rwaves < a.rtiles) tile[r].inverse(a, k, xp[r], xm[r], Y, 0, jt2);
        };
#pragma unroll
        for (int r = 0; r < RTW; ++r) tile[r].init(a, k, b, bt, tb, i3, rw + r * a.rwaves);
        load(n0);
        rows(k.Y);
        if (n0 + 1 < n1e) load(n0 + 1);
        __syncthreads();
        int buf = 0;
        for (int n = n0; n < n1e; ++n) {
            if (!a.dbuf) __syncthreads();  // the band's columns have been read
            if (n + 1 < n1e) {
                rows(k.Y + (a.dbuf ? buf ^ 1 : 0) * half);
                if (n + 2 < n1e) load(n + 2);
            }
            buf = a.dbuf ? buf ^ 1 : 0;
            __syncthreads();
        }
        return;
    }
    // column wave: kind A (ct, t), all 8 slots (row 4 v + k and partner, v < 4) on
    // one column tile; kind B (ct and ct + 1, t = JT - 1), 4 slots (v < 2) on each
    constexpr bool kPair = mx_paired(N);
    const int ctiles = (n2 + 7) / 8, cper = (ctiles + a.cgroups - 1) / a.cgroups;
    const int cend = min(ctiles, (cg + 1) * cper);
    const int jt1 = (H1 + 15) / 16;
    const int full = kPair ? jt1 - 1 : jt1;       // row tiles with waves of kind A
    const bool kindB = kPair && w >= cper * full;
    const int t = kindB ? jt1 - 1 : w / cper;
    const int ct = cg * cper + (kindB ? 2 * (w - cper * full) : w - t * cper);
    const int spin = k.n >> 3;
    int col[2], cc[2];
    bool live[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        col[q] = (ct + q) * 8 + (k.n & 7);
        live[q] = (q == 0 || kindB) && ct + q < cend && col[q] < n2;
        cc[q] = live[q] ? col[q] : 0;
    }
    const bool yside = bt >= a.nk;
    const int ks1 = m1 / 4 + 1;
    const int NP = n1 * n2;
    const unsigned urow = n2 * sizeof(double2);
    const double2* ub = nullptr;
    if (RES) ub = a.ureal + ((long long)a.uslot[tb] * a.nb * a.n3 + i3) * 2 * NP;
    const RowOff uoff(k.k, n1, n1 / 4 * urow, (spin * NP + cc[0]) * (unsigned)sizeof(double2));
    const RowOff uoff1(k.k, n1, n1 / 4 * urow, (spin * NP + cc[1]) * (unsigned)sizeof(double2));
    const long long NN = (long long)NP * a.n3;
    double2* out = a.rho_part + ((long long)b * (TOT ? 1 : a.nchunk) + ch0) * 4 * NN + (long long)i3 * NP;
    const double2* y0 = k.Y + spin * sp + m1 * pitch;
    const double2* inv = k.inv1 + 16 * t;
    auto work = [&](auto kind) {
        constexpr bool kB = decltype(kind)::value;
        // slot i: column tile sq(i), K step sv(i)
        auto sq = [](int i) { return kB ? i / 2 : 0; };
        auto sv = [](int i) { return kB ? i % 2 : i; };
        // A = u_s^* x_s, Bm = u_s'^* x_s (s' the other spin), rows and partners
        // a band's ground state at the lane's points, loaded when the products of
        // the band before have used theirs
        double2 ur[8];
        auto load_u = [&](int n) {
            const Buf u(ub + (long long)n * a.n3 * 2 * NP, 2 * NP * sizeof(double2));
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int j0 = 16 * t + 4 * sv(i);
                if (j0 >= H1) break;
                ur[2 * i] = u.at<double2, 2>(sq(i) ? uoff1.p : uoff.p, mx_resident_row(N, j0) * urow);
                ur[2 * i + 1] = u.at<double2, 2>(sq(i) ? uoff1.m : uoff.m, mx_resident_row(N, mx_partner_base(N, j0)) * urow);
            }
        };
        if (RES) load_u(n0);
        __syncthreads();
        int buf = 0;
        // (A_up, B_up) and (A_dn, B_dn) -> the four components:
        // rho_0 = A_up + A_dn, rho_x = B_up + B_dn, rho_y = i (B_up - B_dn), rho_z = A_up - A_dn;
        // the up lane has 0 and x, the down lane y and z
        auto component = [&](double2 A, double2 B, double2& f, double2& g) {
            const double2 Ao = swap(A), Bo = swap(B);
            f = spin == 0 ? cadd(A, Ao) : cmuli(csub(Bo, B));
            g = spin == 0 ? cadd(B, Bo) : csub(Ao, A);
        };
        auto store = [&](auto value) {
            int kk = k.k;
            asm volatile("" : "+v"(kk));  // the addresses are not held through the bands
            double2* o = out + (spin == 0 ? 0 : 2 * NN);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int j = 16 * t + 4 * sv(i / 2) + kk;
                double2 f, g;
                value(i, f, g);
                if (live[sq(i / 2)] && j < H1 && (i % 2 == 0 || n1 % 2 == 0 || j > 0)) {
                    const int p = (i % 2 == 0 ? j : mx_partner(n1, j)) * n2 + cc[sq(i / 2)];
                    o[p] = f;
                    o[NN + p] = g;
                }
            }
            out += 4 * NN;
        };
        double2 tf[8], tg[8];  // TOT
#pragma unroll
        for (int i = 0; i < 8; ++i) tf[i] = tg[i] = cmk(0.0, 0.0);
        for (int c0 = n0; c0 < n1e; c0 += a.bpc) {
            const int c1 = min(n1e, c0 + a.bpc);
            double2 A[8], Bm[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) A[i] = Bm[i] = cmk(0.0, 0.0);
            for (int n = c0; n < c1; ++n) {
                Inverse<KS> iv;
                double2 us[8];
                if (!RES) {
                    iv.template run_column<S>(a, y0 + buf * half + cc[0] + 2 * sp, k.k, inv, ks1);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        us[2 * v] = iv.plus(v);
                        us[2 * v + 1] = iv.minus(v);
                        if (yside) {
                            us[2 * v] = time_reversed(us[2 * v], spin);
                            us[2 * v + 1] = time_reversed(us[2 * v + 1], spin);
                        }
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (16 * t + 4 * sv(i) >= H1) break;
                    if (sv(i) == 0) iv.template run_column<S>(a, y0 + buf * half + cc[sq(i)], k.k, inv, ks1);
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const double2 x = e == 0 ? iv.plus(sv(i)) : iv.minus(sv(i));
                        const double2 uu = RES ? ur[2 * i + e] : us[2 * i + e];
                        const double2 uo = swap(uu);
                        A[2 * i + e] = cadd(A[2 * i + e], cmulc(uu, x));
                        Bm[2 * i + e] = cadd(Bm[2 * i + e], cmulc(uo, x));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (RES && n + 1 < n1e) load_u(n + 1);
                if (!a.dbuf) __syncthreads();
                buf = a.dbuf ? buf ^ 1 : 0;
                __syncthreads();
            }
            if (TOT) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    double2 f, g;
                    component(A[i], Bm[i], f, g);
                    tf[i] = cadd(tf[i], f);
                    tg[i] = cadd(tg[i], g);
                }
            } else {
                store([&](int i, double2& f, double2& g) { component(A[i], Bm[i], f, g); });
            }
        }
        if (TOT) store([&](int i, double2& f, double2& g) {
            f = tf[i];
            g = tg[i];
        });
    };
    if constexpr (kPair) {
        if (kindB) return work(std::true_type{});
    }
    work(std::false_type{});
}

// Local fields of a plane, in pieces of NP = n1 n2 complex elements:
//   reals v + Bz, v - Bz as [row][spin][column]; (Bx, By) as [row][column];
//   W0 + Wz, W0 - Wz as [row][spin][column] (two pieces); Wx + i Wy, Wx - i Wy (two)
// (x side; the y side takes B -> -B and W -> (W0, -W)).
__global__ void k_fields_mx(const double* __restrict__ vrs, const double2* __restrict__ W,
                            double2* __restrict__ F, int n1, int n2, int n3, long long wstride,
                            long long fstride) {
    const int NP = n1 * n2;
    // tiles of 16 x 16 points: both sides of the transposition in whole lines
    const int t2 = (n2 + 15) / 16, tr = blockIdx.x / t2, tc = blockIdx.x - tr * t2, i3 = blockIdx.y;
    const int row = 16 * tr + threadIdx.y, c = 16 * tc + threadIdx.x;
    if (row >= n1 || c >= n2) return;
    W += blockIdx.z * wstride;
    double2* f = F + blockIdx.z * fstride + (long long)i3 * 6 * NP;
    const long long N = (long long)NP * n3, g = (long long)i3 * NP + c * n1 + row;
    const double v = vrs[g], bx = vrs[N + g], by = vrs[2 * N + g], bz = vrs[3 * N + g];
    const double2 w0 = W[g], wx = W[N + g], wy = W[2 * N + g], wz = W[3 * N + g];
    const int up = row * 2 * n2 + c, dn = up + n2;  // [row][spin][column]
    double* d = reinterpret_cast<double*>(f);
    d[up] = v + bz;
    d[dn] = v - bz;
    f[NP + row * n2 + c] = cmk(bx, by);
    f[2 * NP + up] = cadd(w0, wz);
    f[2 * NP + dn] = csub(w0, wz);
    f[4 * NP + up] = cadd(wx, cmuli(wy));
    f[4 * NP + dn] = csub(wx, cmuli(wy));
}

// phi = V0 x + V' u of every band, back to its columns: row transforms of a
// group of bb bands into the row buffer, then per column tile inverse along
// axis 1, products, forward along axis 1 (in place in the row buffer), then the rows'
// forward transforms.
// RTW: row tiles of a wave, at most
//
// Bound: at 48 x 48 x 180, 104 bands, 36 k (41.1 ms) the counters show the matrix
// cores busy 38 % of the time and 128 GB moved, 3.1 TB/s, of which the ground
// state is 99 (2.4 TB/s); what is left is latency inside a wave (a band's row
// transforms, columns and row transforms are separated by barriers, and the
// fields of a half step come from L2), with two blocks a CU to hide it.
// Four-wave blocks with 256 registers a wave (two a SIMD) hold a column tile's
// ground state in flight; tried and slower at 48 x 48 x 180: fields 4 half
// steps ahead (spills, 6.1 ms), eight-wave blocks with role-specialised waves
// and one barrier a band (5.4 ms, one block a CU).
template <int KS, int JT, bool RES, int N, int M, int NW, int MINW, int RTW>
__global__ void __launch_bounds__(64 * NW, MINW) k_apply_mx(MxArgs a) {
    using S = Shape<N, M>;
    extern __shared__ double2 lds_raw[];
    const int n1 = S::n1(a), n2 = S::n2(a), m1 = S::m1(a), sp = S::sp(a), pitch = S::pitch(a);
    const int nt = blockDim.x, nw = nt >> 6;
    const int id = xcd_order(blockIdx.x, gridDim.x), by = id / a.nbatch;
    const int b = id - by * a.nbatch, i3 = by / a.ny, yy = by - i3 * a.ny;
    const int bt = b % a.nb2, tb = b % a.tmod;
    const int H1 = mx_pairs(n1);
    const int ks1 = m1 / 4 + 1;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    MxBlock<KS, N, M> k;
    k.init(a, lds_raw, nt);
    RowTile<KS, RES, N, M> tile[RTW];  // those of w, w + nw, ... the block has
#pragma unroll
    for (int r = 0; r < RTW; ++r) tile[r].init(a, k, b, bt, tb, i3, w + r * nw);
    const int spin = k.n >> 3;
    const bool yside = bt >= a.nk;
    const double sg = yside ? -1.0 : 1.0;
    const double bsg = spin == 0 ? 1.0 : -1.0;
    const int NP = n1 * n2;
    const double2* ub = nullptr;
    if (RES) ub = a.ureal + ((long long)a.uslot[tb] * a.nb * a.n3 + i3) * 2 * NP;
    // field tables of the plane; a lane takes v +- Bz and W0 +- Wz of its spin
    // (the other one's on the y side), and what it adds to the other spin
    const Buf f(a.fields + (long long)(b / a.nb2) * a.fstride + (long long)i3 * 6 * NP,
                6 * NP * sizeof(double2));
    const int sy = spin ^ (yside ? 1 : 0);
    const int n0 = yy * a.bpb, n1e = min(a.nb, n0 + a.bpb);
    const unsigned uband = (unsigned)a.n3 * 2 * NP * sizeof(double2);
    double2 xp[RTW][KS], xm[RTW][KS];
    auto load_rows = [&](int g) {
#pragma unroll
        for (int r = 0; r < RTW; ++r)
            if (w + r * nw < a.rtiles) tile[r].load(a, g, n1e, xp[r], xm[r]);
    };
    load_rows(n0);
    __syncthreads();  // the constant tables
    for (int g = n0; g < n1e; g += a.bb) {
#pragma unroll
        for (int r = 0; r < RTW; ++r)
            if (w + r * nw < a.rtiles) tile[r].inverse(a, k, xp[r], xm[r], k.Y, 0, (mx_pairs(n2) + 15) / 16);
        __syncthreads();
        const int nbg = min(a.bb, n1e - g);  // bands of the group
        const int ctiles = (nbg * n2 + 7) / 8;
        const Buf ug(RES ? ub + (long long)g * a.n3 * 2 * NP : nullptr, (nbg - 1) * uband + 2 * NP * (unsigned)sizeof(double2));
        for (int ct = w; ct < ctiles; ct += nw) {
            const int q = ct * 8 + (k.n & 7);
            const bool clive = q < nbg * n2;
            const int qc = clive ? q : 0;
            const int bl = qc / n2, col = qc - bl * n2;
            double2* y = k.Y + (bl * 2 + spin) * sp + m1 * pitch + col;
            const RowOff uoff(k.k, n1, n1 / 4 * n2 * sizeof(double2), bl * uband + (spin * NP + col) * (unsigned)sizeof(double2));
            // rows of the spin-resolved tables (the lane's spin, its spin or the other
            // one by side) and of (Bx, By)
            const RowOff ooff(k.k, n1, 2 * n2 * sizeof(double2), (spin * n2 + col) * (unsigned)sizeof(double2));
            const RowOff doff(k.k, n1, 2 * n2 * sizeof(double2), (sy * n2 + col) * (unsigned)sizeof(double2));
            const RowOff boff(k.k, n1, n2 * sizeof(double2), col * (unsigned)sizeof(double2));
            Inverse<KS> iv;
            Forward<KS> fw;
            fw.clear();
#pragma unroll 1
            for (int t = 0; t < JT; ++t) {
                if (16 * t >= H1) break;
                // half steps hs = 2 v + e: rows j (e = 0) and partners of K step v.  The
                // fields (L2) are loaded FD - 1 half steps ahead, the ground state (HBM) all
                // before them: loads complete in order, so a later one would hold the
                // fields up
                auto live_step = [&](int hs) { return 16 * t + 4 * (hs / 2) < H1; };
                auto row_base = [&](int hs) {
                    const int j0 = 16 * t + 4 * (hs / 2);
                    return hs % 2 == 0 ? j0 : mx_partner_base(n1, j0);
                };
                auto row_off = [&](int hs, const RowOff& o) {
                    return hs % 2 == 0 ? o.p : hs == 1 && t == 0 ? o.m0 : o.m;
                };
                double2 ur[8];
                constexpr int FD = 2;  // field half steps held
                double fdv[FD];
                double2 fbv[FD], fwd[FD], fwo[FD];
                auto load_u = [&](int hs) {
                    if (RES && live_step(hs))
                        ur[hs] = ug.at<double2, 2>(hs % 2 == 0 ? uoff.p : uoff.m, mx_resident_row(N, row_base(hs)) * (n2 * sizeof(double2)));
                };
                auto load_f = [&](int hs) {
                    if (!live_step(hs)) return;
                    const unsigned r2 = row_base(hs) * (2 * n2 * sizeof(double2)), piece = NP * sizeof(double2);
                    const unsigned od = row_off(hs, doff);
                    fdv[hs % FD] = f.at<double>(od >> 1, r2 >> 1);
                    fbv[hs % FD] = f.at<double2>(row_off(hs, boff), piece + (r2 >> 1));
                    fwd[hs % FD] = f.at<double2>(od, 2 * piece + r2);
                    fwo[hs % FD] = f.at<double2>(row_off(hs, ooff), 4 * piece + r2);
                };
#pragma unroll
                for (int hs = 0; hs < 8; ++hs) load_u(hs);
#pragma unroll
                for (int hs = 0; hs < FD - 1; ++hs) load_f(hs);
                double2 us[8];
                if (!RES) {
                    iv.template run_column<S>(a, y + a.bb * 2 * sp, k.k, k.inv1 + 16 * t, ks1);
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        us[2 * v] = iv.plus(v);
                        us[2 * v + 1] = iv.minus(v);
                        if (yside) {
                            us[2 * v] = time_reversed(us[2 * v], spin);
                            us[2 * v + 1] = time_reversed(us[2 * v + 1], spin);
                        }
                    }
                }
                iv.template run_column<S>(a, y, k.k, k.inv1 + 16 * t, ks1);
                double2 ph0 = cmk(0.0, 0.0);
#pragma unroll
                for (int hs = 0; hs < 8; ++hs) {
                    const int v = hs / 2, e = hs % 2;
                    if (!live_step(hs)) break;
                    if (hs + FD - 1 < 8) load_f(hs + FD - 1);
                    const int fs = hs % FD;
                    const double2 x = e == 0 ? iv.plus(v) : iv.minus(v);
                    const double2 uu = RES ? ur[hs] : us[hs];
                    double2 p = local_product(fdv[fs], fbv[fs], fwd[fs], fwo[fs], x, uu, bsg, sg);
                    if (e == 0) {
                        ph0 = p;
                    } else {
                        if (n1 % 2 == 1 && 16 * t + 4 * v + k.k == 0) p = cmk(0.0, 0.0);  // row 0 is its own partner
                        fw.step(k.fwd1, 4 * t + v, mx_stride(n1), ph0, p);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            if (clive) {
#pragma unroll
                for (int i = 0; i < KS; ++i) {
                    const int m = 4 * i + k.k;
                    if (4 * i + 3 <= m1 || m <= m1) {
                        y[m * pitch] = fw.plus(i);
                        if (i > 0 || m > 0) y[-m * pitch] = fw.minus(i);
                    }
                }
            }
        }
        // the next group's row elements, in flight during the rows' forward transforms
        if (g + a.bb < n1e) load_rows(g + a.bb);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RTW; ++r)
            if (w + r * nw < a.rtiles) tile[r].forward(a, k, k.Y, g, n1e);
    }
}

int cdiv_i(long long a, long long b) { return (int)((a + b - 1) / b); }

// LDS of a block: the constants of both axes and `halves` row buffers of bb bands
// (and room for the forward transforms' reads of whole row tiles of constants)
template <int KS>
size_t mx_lds(const MxArgs& a, int halves) {
    const size_t t1 = mx_table<KS>(a.n1), t = t1 + (a.n1 != a.n2 ? mx_table<KS>(a.n2) : 0);
    constexpr size_t rows = 16 * ((KS + 3) / 4);
    const size_t reach = std::max(rows * mx_stride(a.n1), (t - (a.n1 != a.n2 ? t - t1 : t1)) + rows * mx_stride(a.n2)) + 32;
    return std::max(t + (size_t)halves * a.bb * 2 * a.sp, reach) * sizeof(double2);
}

constexpr size_t kMxLds = 160 * 1024;

template <class F>
void launch_mx(F kernel, const char* name, size_t shm, dim3 grid, int nt, hipStream_t st, MxArgs a) {
    TM_CHECK(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm) ==
                 hipSuccess,
             TM_EDEVICE, std::string("cannot raise the LDS limit of ") + name);
    ProfScope ps(name, st);
    void* args[] = {&a};
    TM_CHECK(hipLaunchKernel((const void*)kernel, grid, dim3(nt), args, shm, st) == hipSuccess, TM_EDEVICE,
             std::string("launch of ") + name + " failed");
    check_launch(name);
}

// The waves of a block, at most.
constexpr int kDensityW = 12, kApplyW = 8;

// (density: returns the partial sums of a batch)
template <int KS, int JT, bool RES, int N, int M>
int launch_shape(bool density, MxArgs a, int nbatch, int variant, hipStream_t st) {
    if (N > 0) {  // rows up to the kernel's reach, zero past the spheres'
        a.m1 = a.m2 = M;
        a.sp = mx_spin_stride(N, M);
    }
    const int kinds = RES ? 1 : 2, R1 = 2 * a.m1 + 1;
    const int want = 1 << variant;  // bands a group
    const int jt1 = cdiv_i(mx_pairs(a.n1), 16), ctiles = (a.n2 + 7) / 8;
    auto rtiles = [&](int bb) { return cdiv_i((long long)kinds * bb * 2 * R1, 16); };
    if (density) {
        // at most 12 waves (three a SIMD): the column waves of a plane or of a share
        // of its columns, and row waves to fill up to a multiple of four (a SIMD each)
        constexpr bool pair = N > 0 && mx_paired(N);
        auto colwaves = [&](int groups) {
            const int cper = cdiv_i(ctiles, groups);
            return pair ? cper * (jt1 - 1) + cdiv_i(cper, 2) : cper * jt1;
        };
        a.bb = 1;
        a.rtiles = rtiles(1);
        constexpr int RTW = N == 48 && M <= 11 ? 1 : 2;
        const int minrow = cdiv_i(a.rtiles, RTW);
        a.cgroups = 1;
        while (colwaves(a.cgroups) + minrow > kDensityW) ++a.cgroups;
        a.cwaves = colwaves(a.cgroups);
        a.rwaves = std::min(a.rtiles, std::max(minrow, cdiv_i(a.cwaves + minrow, 4) * 4 - a.cwaves));
        a.dbuf = mx_lds<KS>(a, 2 * kinds) <= kMxLds;
        const size_t shm = mx_lds<KS>(a, (a.dbuf ? 2 : 1) * kinds);
        const int nw = a.cwaves + a.rwaves;
        TM_CHECK(shm <= kMxLds && nw <= kDensityW, TM_EUNSUPPORTED, "plane too large for the matrix-core kernels");
        constexpr int NW = N == 48 || N == 0 ? kDensityW : 8, MINW = N == 20 ? 2 : 3;
        TM_CHECK(nw <= NW, TM_EUNSUPPORTED, "plane too large for the matrix-core kernels");
        // Chunks: as few rounds of blocks as possible, weighing what a chunk costs
        // besides its bands: about two of set-up, and its partial sums, written and
        // read again, about four (8 values a point against a band's 2).  By the shape
        // of one right-hand side, so that the sums do not depend on their number.
        const int percu = std::max(1, std::min(4 * MINW / nw, (int)(kMxLds / shm)));
        const long long per = (long long)a.nb2 * a.n3 * a.cgroups, slots = 256LL * percu;
        long long best = 0;
        int chunks = 1;
        for (int c = 1; c <= a.nchunk; ++c) {
            const int bpc = cdiv_i(a.nb, c);
            const long long cost = (per * cdiv_i(a.nb, bpc) + slots - 1) / slots * (bpc + 6);
            if (c == 1 || cost < best) {
                best = cost;
                chunks = cdiv_i(a.nb, bpc);
            }
        }
        a.nchunk = chunks;
        a.bpc = cdiv_i(a.nb, chunks);
        a.nbatch = nbatch;
        // several chunks a block while about four rounds of blocks remain: its set-up is
        // shared and the next chunk's loads are in flight.  Right-hand sides enough for a
        // round of blocks with all chunks each: only their total is written (added up in
        // the reduction's order)
        const long long all = (long long)nbatch * a.n3 * a.cgroups;
        const bool total = RES && N < 48 && chunks > 1 && all >= slots;
        a.cpb = total ? chunks : (int)std::max<long long>(1, std::min<long long>(chunks, all * chunks / slots / 4));
        a.ny = cdiv_i(chunks, a.cpb) * a.cgroups;
        const dim3 grid(nbatch * a.ny * a.n3);
        if constexpr (RES && N < 48) {
            if (total) {
                launch_mx(k_density_mx<KS, JT, RES, N, M, NW, 2, RTW, true>, "k_density_mx", shm, grid, 64 * nw, st, a);
                return 1;
            }
        }
        launch_mx(k_density_mx<KS, JT, RES, N, M, NW, MINW, RTW, false>, "k_density_mx", shm, grid, 64 * nw, st, a);
        return chunks;
    } else {
        // four waves (one a SIMD); planes of two row tiles with 256 registers, the
        // others with 168
        constexpr bool wide = JT == 2 && RES;
        constexpr int RTW = (RES && JT == 2) || KS > 4 ? 2 : 1, NW = RES ? 4 : kApplyW;
        const int waves = RES ? 4 : 6;
        a.bb = std::max(1, std::min(want, a.nb));
        while (a.bb > 1 && (rtiles(a.bb) > std::max(RTW * waves, rtiles(1)) || mx_lds<KS>(a, kinds) > kMxLds / 2))
            --a.bb;
        a.rtiles = rtiles(a.bb);
        const int nw = std::min(NW, std::max(cdiv_i(a.rtiles, RTW), std::min(waves, cdiv_i((long long)a.bb * a.n2, 8))));
        const size_t shm = mx_lds<KS>(a, kinds);
        TM_CHECK(shm <= kMxLds && a.rtiles <= RTW * nw, TM_EUNSUPPORTED, "plane too large for the matrix-core kernels");
        // bands of a block: whole groups, about 4096 blocks
        const long long per = (long long)nbatch * a.n3;
        const int groups = cdiv_i(a.nb, a.bb);
        const int gpb = (int)std::max<long long>(1, std::min<long long>(groups, per * groups / 4096));
        a.bpb = gpb * a.bb;
        constexpr int MINW = wide || !RES || N == 32 ? 2 : 3;
        a.nbatch = nbatch;
        a.ny = cdiv_i(a.nb, a.bpb);
        launch_mx(k_apply_mx<KS, JT, RES, N, M, NW, MINW, RTW>, "k_apply_mx", shm, dim3(nbatch * a.ny * a.n3),
                  64 * nw, st, a);
        return 0;
    }
}

// the resident ground state's plane sizes, by the spheres' reach
template <int N, int M0, int... Ms>
int launch_fixed(bool density, const MxArgs& a, int nbatch, int variant, hipStream_t st) {
    if (std::max(a.m1, a.m2) <= M0)
        return launch_shape<M0 / 4 + 1, (mx_pairs(N) + 15) / 16, true, N, M0>(density, a, nbatch, variant, st);
    if constexpr (sizeof...(Ms) > 0) return launch_fixed<N, Ms...>(density, a, nbatch, variant, st);
    throw Error{TM_EINVAL, "sphere larger than the plane"};
}

// Reaches (mx_resident_reach at most): half-filled spheres (the density cutoff four times the
// wavefunctions') with k and q inside the first zone take the first of each
// size; the others are for fuller spheres, up to the largest that fits.
int launch_resident(bool density, const MxArgs& a, int nbatch, int variant, hipStream_t st) {
    switch (a.n1) {
        case 8: return launch_fixed<8, 3>(density, a, nbatch, variant, st);
        case 20: return launch_fixed<20, 5, 9>(density, a, nbatch, variant, st);
        case 24: return launch_fixed<24, 7, 11>(density, a, nbatch, variant, st);
        case 32: return launch_fixed<32, 8, 15>(density, a, nbatch, variant, st);
        case 48: return launch_fixed<48, 11, 13>(density, a, nbatch, variant, st);
        default: throw Error{TM_EUNSUPPORTED, "no resident plane kernel for this grid"};
    }
}

int launch_columns(bool density, const MxArgs& a, int nbatch, int variant, hipStream_t st) {
    const int ks = std::max(a.m1, a.m2) / 4 + 1, jt = cdiv_i(mx_pairs(std::max(a.n1, a.n2)), 16);
    if (jt == 1) {
        if (ks <= 1) return launch_shape<1, 1, false, 0, 0>(density, a, nbatch, variant, st);
        if (ks <= 2) return launch_shape<2, 1, false, 0, 0>(density, a, nbatch, variant, st);
        if (ks <= 3) return launch_shape<3, 1, false, 0, 0>(density, a, nbatch, variant, st);
        return launch_shape<4, 1, false, 0, 0>(density, a, nbatch, variant, st);
    }
    if (ks <= 2) return launch_shape<2, 2, false, 0, 0>(density, a, nbatch, variant, st);
    if (ks <= 3) return launch_shape<3, 2, false, 0, 0>(density, a, nbatch, variant, st);
    if (ks <= 4) return launch_shape<4, 2, false, 0, 0>(density, a, nbatch, variant, st);
    return launch_shape<6, 2, false, 0, 0>(density, a, nbatch, variant, st);
}

}  // namespace

// whether the matrix-core plane kernels take planes of n1 x n2 whose spheres
// reach |m1|, |m2|: up to two row tiles (n <= 64) and six K steps (|m| <= 23),
// a first K step of rows inside the plane (n >= 4), and one band's row buffers (x
// and ground state) in LDS
bool mx_supported(int n1, int n2, int m1, int m2) {
    if (std::min(n1, n2) < 4 || std::max(n1, n2) > kMxSide || std::max(m1, m2) > 23) return false;
    const size_t tabs = (size_t)(mx_table<6>(n1) + (n1 != n2 ? mx_table<6>(n2) : 0)) * sizeof(double2);
    return tabs + (size_t)2 * 2 * mx_spin_stride(n2, m1) * sizeof(double2) <= kMxLds;
}

std::vector<double2> mx_constants(int n) {
    const int st = mx_stride(n);
    std::vector<double2> t(24 * (size_t)st, cmk(0.0, 0.0));
    for (int m = 0; m < 24; ++m)
        for (int j = 0; j < mx_pairs(n); ++j) {
            // 2 pi (j + 1/2) m / n, or 2 pi j m / n for odd n, reduced to a turn
            const int num = n % 2 == 0 ? (2 * j + 1) * m % (2 * n) : 2 * j * m % (2 * n);
            const double ang = M_PI * (double)num / (double)n;
            t[m * (size_t)st + j] = cmk(std::cos(ang), std::sin(ang));
        }
    return t;
}

std::vector<double2> mx_twists(int n) {
    std::vector<double2> t(24, cmk(1.0, 0.0));
    for (int m = 0; m < 24 && n % 2 == 0; ++m) t[m] = cmk(std::cos(M_PI * m / n), -std::sin(M_PI * m / n));
    return t;
}

int launch_plane_mx(bool density, const MxArgs& a, int nbatch, int variant, hipStream_t st) {
    if (a.ureal) return launch_resident(density, a, nbatch, variant, st);
    return launch_columns(density, a, nbatch, variant, st);
}

void launch_fields_mx(const double* vrs, const double2* W, double2* fields, int n1, int n2, int n3, long long wstride,
                      long long fstride, int nrhs, hipStream_t st) {
    const dim3 grid(((n1 + 15) / 16) * ((n2 + 15) / 16), n3, nrhs);
    TM_LAUNCH(k_fields_mx, grid, dim3(16, 16), 0, st, vrs, W, fields, n1, n2, n3, wstride, fstride);
}

}  // namespace tml
