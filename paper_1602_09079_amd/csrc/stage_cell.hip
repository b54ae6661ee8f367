// Stage kernel of k = 1 and k = 2 in FP64 and FP32: one cell per lane, sum factorisation on the
// vector units (the modal DG operator of Bauer et al., arXiv 1602.09079, Sec. 2.3).
//
// What bounds it: vector issue.  At k = 2 an operator evaluation is about 30 HLLC solves and 27
// volume points per cell; on 16x16 matrix-core tiles the 9 face points fill 9 of 16 rows (4 of 16 at
// k = 1) and the padding rows are solved as well, so the matrix form issues about twice the vector
// instructions and waits for its exchanges besides.  Here every lane works on a cell of its own and
// no row is padding.
//
// Measured, one driven stage repeated on the same input, us, matrix form -> this one: 64^3 k = 1 FP32
// 161 -> 31, FP64 217 -> 60; k = 2 FP32 230 -> 88, FP64 452 -> 233; a 90 x 77 x 51 mesh at k = 2 FP32
// 701 -> 134 (14-cell blocks by groups of 8 rows leave more of a ragged mesh idle than tiles).  In whole
// steps, with inputs from memory, the average launch takes 36 (k = 1 FP32), 104 and 259 (k = 2 FP32, FP64)
// and 157 us (ragged).  k = 2 FP32 at 64^3 issues vector instructions about three quarters of the time with
// two waves per SIMD; the rest is memory and LDS latency.
//
// A wave owns a tile of 16 x 4 cells in x and y and sweeps a chunk of z.  Waves are independent:
// nothing is shared between them, so there is no barrier, and a small mesh is cut into as many work
// items as it has tiles and chunks.  Four waves on consecutive tiles along x form a workgroup, so the
// 64-byte runs of a row that they read come from the same cache lines of one compute unit (k = 2 FP32
// at 64^3, by 8 x 8 tiles: 133 -> 124 us against one wave per workgroup).  Tiles of 8 x 8 read 32-byte
// runs and have twice the cells past their x edges, each of whose values costs a cache line (k = 2 FP32,
// 8 x 8 -> 16 x 4: 64^3 121 -> 113 us, 128^3 984 -> 885; 12 x 5 or 32 x 2 leave lanes idle or have
// more edge faces).
//
// Meshes of few tiles and planes (cell_split_kernel): with a few waves in flight the time of a launch is
// one wave's chain of dependent instructions and memory round trips.  There a workgroup takes one tile and
// one plane and its waves one task each - x faces, y faces, the two z faces, the volume integral - and
// their shares of R are added through LDS in a fixed order (driven 16^3, one wave per tile -> this: k = 1
// FP64 18.5 -> 9.3 us, k = 2 FP32 32 -> 15, FP64 51 -> 20; the waves of the x and the y faces each solve only
// the tile's low-edge faces of their own axis, 9.8 -> 8.4 us at k = 1 FP64 against all 20 in both).
//
// Volume integral.  The integral of F_a against the gradient of the basis needs the moments of F_a
// with the polynomials of degree k - 1 only: 1 moment at k = 1, 4 at k = 2, of the 9 distinct
// components of the momentum and energy fluxes (the mass flux is the momentum itself, whose moments
// are its modes).  They are collected point by point, and the derivative matrices, which are sparse
// in this basis, are applied to them once per cell.
//
// Faces.  A face is described by its 2D trace modes (p, q), p + q <= k, of each field: 15 values at
// k = 1, 30 at k = 2 instead of 20 or 45 point values.  Neighbours exchange trace modes and flux
// moments in LDS.  Each lane solves its +x, +y and +z faces; the faces on the tile's low x and y
// edges (20 of them) are solved point by point, spread over all 64 lanes.  The +z flux moments are
// carried to the next plane.  Every solve takes the same arithmetic on the same modes, so a face on
// a tile edge, which two waves solve, gets the same flux in both.
//
// Deviation form: the flux of the cell mean is subtracted from every volume and face flux before the
// moments are formed.  The subtracted terms are the same numbers everywhere, so they cancel exactly, and the
// sums run over the variation inside the cell.  Point values are interpolated the same way: the variation
// first, the cell mean last.  The rounding of R is then that of one rounding per point (48^3, Mach number
// 0.3, FP32: 5.3e-6 of R at k = 1, 7.5e-6 at k = 2).  With the mean inside mode (0, 0) of a face's trace,
// every point of the face shares its rounding, and R's error is 7.6e-6 and 15.3e-6, in FP64 likewise; the
// additions cost 5..10 % of a k = 1 launch in FP32.

#include <type_traits>

#include "dg_device.h"

namespace dgmi {

// ------------------------------------------------------------------ 1D Gauss and Legendre tables
//
// P[u][a]: scaled Legendre polynomial sqrt(2u+1) P_u at Gauss node a; W[a]: Gauss weight / 2; E[u] =
// sqrt(2u+1), the value at +1 (that at -1 has the sign (-1)^u).
template <int K>
struct Leg;
template <>
struct Leg<1> {
    static constexpr double P[2][2] = {{1.0, 1.0}, {-1.0, 1.0}};
    static constexpr double W[2] = {0.5, 0.5};
    static constexpr double E[2] = {1.0, 1.7320508075688772935};
};
template <>
struct Leg<2> {
    // sqrt(3) x and sqrt(5) (3 x^2 - 1) / 2 at x = -sqrt(3/5), 0, sqrt(3/5)
    static constexpr double P[3][3] = {{1.0, 1.0, 1.0},
                                       {-1.3416407864998738178, 0.0, 1.3416407864998738178},
                                       {0.8944271909999158786, -1.1180339887498948482, 0.8944271909999158786}};
    static constexpr double W[3] = {0.27777777777777777778, 0.44444444444444444444, 0.27777777777777777778};
    static constexpr double E[3] = {1.0, 1.7320508075688772935, 2.2360679774997896964};
};

// P_u at node b, b an index the compiler need not know
template <int K, class C>
__device__ inline C leg_at(int u, int b) {
    C r = (C)Leg<K>::P[u][0];
#pragma unroll
    for (int a = 1; a <= K; a++) r = b == a ? (C)Leg<K>::P[u][a] : r;
    return r;
}

// degrees of the modes in the graded order
template <int K>
struct ModeTab {
    int u[Dims<K>::N], v[Dims<K>::N], w[Dims<K>::N];
    constexpr ModeTab() : u(), v(), w() {
        int l = 0;
        for (int d = 0; d <= K; d++)
            for (int a = d; a >= 0; a--)
                for (int b = d - a; b >= 0; b--) {
                    u[l] = a;
                    v[l] = b;
                    w[l] = d - a - b;
                    l++;
                }
    }
};

// index of the 2D mode (p, q), p + q <= K
template <int K>
constexpr int t2(int p, int q) {
    return p * (K + 1) - p * (p - 1) / 2 + q;
}
// the volume mode with degree r along the axis and (p, q) along the other two, lower axis first
template <int K, int AX>
constexpr int face_mode(int r, int p, int q) {
    return AX == 0 ? mode_of<K>(r, p, q) : AX == 1 ? mode_of<K>(p, r, q) : mode_of<K>(p, q, r);
}
// fields seen from a face: density, normal momentum, the other two momenta, energy
template <int AX>
constexpr int face_field(int f) {
    return f == 0 || f == 4 ? f : f == 1 ? 1 + AX : f == 2 ? (AX == 0 ? 2 : 1) : (AX == 2 ? 2 : 3);
}

__device__ inline float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

// ------------------------------------------------------------------ LDS of a wave
//
// Exchange planes, one per (field, 2D mode): 64 slots of the tile's cells (slot = lane), then the trace
// modes past the high x edge (4) and below the low x edge's flux moments (4), and the same of the y
// edges (16 and 16).  Then one region that first holds the trace modes of the 20 low-edge faces from
// both sides and after them the cells' own trace modes on the face being solved.  The low-edge faces'
// point fluxes pass through the cells' slots of the planes, which are free at that time.
constexpr int CTX = CELL_TX, CTY = CELL_TY;  // the tile
constexpr int EF = CTX + CTY;                // its low-edge faces: CTY in x, then CTX in y
constexpr int SL_XHI = 64, SL_XLO = SL_XHI + CTY, SL_YHI = SL_XLO + CTY, SL_YLO = SL_YHI + CTX;
constexpr int CX_PLANE = SL_YLO + CTX;
template <int K>
struct CellLds {
    static constexpr int NT = (K + 1) * (K + 2) / 2, NV = NF * NT, P = Dims<K>::P, N = Dims<K>::N;
    static constexpr int X = NV * CX_PLANE;         // exchange planes
    // low-edge trace modes [side][value][face], cell means [side][field][face], the tile's cells' mean
    // fluxes [field][face]
    static constexpr int E = (2 * NV + 3 * NF) * EF;
    static constexpr int S = NV * 64;               // this tile's trace modes on the face being solved
    // during the volume integral: the weights but the means (k = 2, to free their registers), and the weights
    // of the 40 cells across the tile's edges on their way in from memory: 32 past the y edges
    // (two lanes a cell, half of the modes each), then 8 past the x edges (eight values a load)
    static constexpr int STASHED = K >= 2 ? NF * (N - 1) : 0, W = STASHED * 64, H = N / 2;
    static constexpr int RAW = W, RAWN = NF * H * 64 + (NF * N + 7) / 8 * 64;
    static constexpr int ELEMS0 = X + (E > S ? E : S), ELEMS = ELEMS0 > RAW + RAWN ? ELEMS0 : RAW + RAWN;
    static_assert(NF * EF * P <= 64 * NV, "the point fluxes fit the cells' slots");
};
// point flux number j of the low-edge faces among the cells' slots
__device__ inline int flux_slot(int j) { return (j >> 6) * CX_PLANE + (j & 63); }

// a wave-uniform value, in scalar registers
__device__ inline float uniform(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }
__device__ inline double uniform(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(b & 0xffffffffll));
    const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | lo);
}

// Values computed up to here stay here: the compiler otherwise sinks whole phases of arithmetic past
// the memory operations of the following ones, with their inputs live (and spilled) in between.
template <class T, int A, int B>
__device__ inline void pin(T (&v)[A][B]) {
#pragma unroll
    for (int i = 0; i < A; i++)
#pragma unroll
        for (int j = 0; j < B; j++) asm volatile("" : "+v"(v[i][j]));
}

// orders this wave's LDS accesses for the compiler; the LDS unit serves a wave in order
__device__ inline void lds_order() { asm volatile("" ::: "memory"); }

// a value that to_lds put down: d points at its low word
__device__ inline float from_lds(const int *d, float) { return __int_as_float(d[0]); }
__device__ inline double from_lds(const int *d, double) {
    return __longlong_as_double(((long long)d[64] << 32) | (unsigned)d[0]);
}

// lane's value of v
__device__ inline float lane_value(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(lane << 2, __float_as_int(v)));
}
__device__ inline double lane_value(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_ds_bpermute(lane << 2, (int)(b & 0xffffffffll));
    const int hi = __builtin_amdgcn_ds_bpermute(lane << 2, (int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | lo);
}

template <int K, class C>
constexpr int cell_waves() { return K == 1 ? (sizeof(C) == 8 ? 2 : 3) : (sizeof(C) == 8 ? 1 : 2); }

// Waves of a workgroup that splits one tile and plane by task (small meshes): the x faces, the y
// faces, the two z faces, and the volume integral; at k = 2 in FP32 one Gauss plane of it each (in
// FP64 a fifth wave would halve the registers of all).
template <int K, class C>
struct CellSplit {
    static constexpr int VOL = 3, NVOL = K == 1 || sizeof(C) == 8 ? 1 : 3, WAVES = VOL + NVOL;
    using LD = CellLds<K>;
    static constexpr int ZS = 2 * LD::S, RS = NF * Dims<K>::N * 64;  // z-face modes, a wave's share of R
    static_assert(ZS >= RS && LD::ELEMS >= RS, "the shares of R fit the regions of their waves");
    // element offset of a wave's region; the first volume wave keeps its share in registers
    static __device__ int base(int w) {
        return w < 2 ? w * LD::ELEMS : w <= VOL ? 2 * LD::ELEMS : 2 * LD::ELEMS + ZS + (w - VOL - 1) * RS;
    }
    static constexpr int ELEMS = 2 * LD::ELEMS + ZS + (NVOL - 1) * RS;
};

template <int K, class C, bool FORCE, int RS, bool BIG, bool SPLIT>
__device__ __forceinline__ void cell_stage(const StageArgs &a) {
    using L = Leg<K>;
    using PR = Prec<sizeof(C) == 8 ? DG_FP64 : DG_FP32>;
    using LD = CellLds<K>;
    constexpr int N = Dims<K>::N, n = K + 1, P = Dims<K>::P, NT = LD::NT, NV = LD::NV;
    constexpr int NL = K * (K + 1) * (K + 2) / 6;  // modes of degree <= k - 1
    constexpr ModeTab<K> T;
    extern __shared__ __attribute__((aligned(16))) char lds_all[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    C *const lds0 = reinterpret_cast<C *>(lds_all);
    C *const lds = lds0 + (SPLIT ? CellSplit<K, C>::base(wave) : wave * LD::ELEMS);
    C *const lx = lds, *const le = lds + LD::X;

    const int lane = threadIdx.x & 63, cx = lane & (CTX - 1), cy = lane / CTX;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const unsigned unx = (unsigned)nx;
    // items in 8 contiguous ranges by workgroup id modulo 8 (one per XCD), so neighbouring tiles share
    // the L2 their edge cells are read through
    long long item;
    {
        const int per = SPLIT ? 1 : a.wgw;  // items per workgroup
        const long long bid = blockIdx.x, nwg = (a.nitems + per - 1) / per;
        const long long lo = nwg / 8, extra = nwg % 8;
        const int xcd = (int)(bid & 7);
        item = ((bid >> 3) + xcd * lo + (xcd < extra ? xcd : extra)) * per + (SPLIT ? 0 : wave);
    }
    if (item >= a.nitems) return;
    const int ntx = a.nbx, nty = (ny + CTY - 1) / CTY;
    const int bx = (int)(item % ntx);
    const long long rest = item / ntx;
    const int by = (int)(rest % nty), zc = (int)(rest / nty);
    const int x0 = bx * CTX, y0t = by * CTY;
    const int zlen = SPLIT ? 1 : a.zlen;
    const int z0 = zc * zlen, z1 = z0 + zlen < nz ? z0 + zlen : nz;
    // lanes past the end of a ragged tile take the cells the periodic mesh continues with
    const int ix = (x0 + cx) % nx, iy = (y0t + cy) % ny;
    const bool keep = x0 + cx < nx && y0t + cy < ny;
    const long long plane = (long long)NF * N * nx * ny;
    const long long cell = (long long)iy * NF * N * nx + ix;
    // the cells across the edges: past the y edges lanes 0..15 low, 16..31 high (32..63 again), past the
    // x edges lanes 0..3 low, 4..7 high (8..63 again)
    long long ycell, xcell;
    {
        const int ex = (x0 + cx) % nx, ey = (lane & CTX) ? (y0t + CTY) % ny : (y0t + ny - 1) % ny;
        ycell = (long long)ey * NF * N * nx + ex;
        const int fx = (lane & CTY) ? (x0 + CTX) % nx : (x0 + nx - 1) % nx, fy = (y0t + (lane & (CTY - 1))) % ny;
        xcell = (long long)fy * NF * N * nx + fx;
    }
    const C *yin = static_cast<const C *>(a.yin);
    // z plane zz of the input, across the ends from the halo planes or periodic
    auto in_plane = [&](int zz, long long &zi) -> const C * {
        zi = 0;
        if (a.halo_lo && zz < 0) return static_cast<const C *>(a.halo_lo);
        if (a.halo_hi && zz >= nz) return static_cast<const C *>(a.halo_hi);
        zi = zz < 0 ? zz + nz : (zz >= nz ? zz - nz : zz);
        return yin;
    };
    const C gam = uniform((C)a.gamma), g1 = uniform(gam - C(1));
    double dtd = a.dt;
    if (a.rate) dtd = a.dtfac / a.rate[0];
    const C dt = uniform((C)dtd);
    if (a.tacc && blockIdx.x == 0 && threadIdx.x == 0) a.tacc[0] += dtd;
    if (SPLIT && a.zero_rate && blockIdx.x == 0 && threadIdx.x == 0) a.zero_rate[0] = 0.0;
    const C ih[3] = {uniform((C)a.ih[0]), uniform((C)a.ih[1]), uniform((C)a.ih[2])};

    C w[NF][N], R[NF][N], mz[NF][NT];  // weights, operator, flux moments of the face below

    auto load_cells = [&](int zz) {
        long long zi;
        const C *b = in_plane(zz, zi);
        const PlaneView<C, BIG> pv(b, plane, zi, cell);
#pragma unroll
        for (int i = 0; i < NF; i++)
#pragma unroll
            for (int l = 0; l < N; l++) w[i][l] = pv.get(i * N + l, unx);
    };
    // trace modes of this lane's cell on a face (sgn = -1, +1), fields as seen from the face; mode (0, 0)
    // without the cell mean
    auto trace = [&](auto ax_c, auto sgn_c, C t[NF][NT]) {
        constexpr int AX = decltype(ax_c)::value, SG = decltype(sgn_c)::value;
#pragma unroll
        for (int f = 0; f < NF; f++)
#pragma unroll
            for (int p = 0; p <= K; p++)
#pragma unroll
                for (int q = 0; q <= K - p; q++) {
                    auto term = [&](int r) { return (C)((SG < 0 && (r & 1)) ? -L::E[r] : L::E[r]); };
                    const C *const wf = w[face_field<AX>(f)];
                    const bool dev = p + q == 0;
                    C s = dev ? term(1) * wf[face_mode<K, AX>(1, 0, 0)] : wf[face_mode<K, AX>(0, p, q)];
#pragma unroll
                    for (int r = dev ? 2 : 1; r <= K - p - q; r++)
                        s = fma_(term(r), wf[face_mode<K, AX>(r, p, q)], s);
                    t[f][t2<K>(p, q)] = s;
                }
    };
    // fluxes of a state: xx xy xz yy yz zz of the momentum, x y z of the energy (the mass flux is the momentum)
    auto fluxes = [&](const C q[NF], C f[9]) __attribute__((always_inline)) {
        const C inv = PR::rcp(q[0]);
        const C u = q[1] * inv, v = q[2] * inv, ww = q[3] * inv;
        const C p = g1 * (q[4] - C(0.5) * (q[1] * u + q[2] * v + q[3] * ww));
        const C ep = q[4] + p;
        f[0] = q[1] * u + p;
        f[1] = q[1] * v;
        f[2] = q[1] * ww;
        f[3] = q[2] * v + p;
        f[4] = q[2] * ww;
        f[5] = q[3] * ww + p;
        f[6] = ep * u;
        f[7] = ep * v;
        f[8] = ep * ww;
    };
    // this lane's cell means
    auto means = [&](C q[NF]) {
#pragma unroll
        for (int i = 0; i < NF; i++) q[i] = w[i][0];
    };
    // the flux of the cell means q along an axis, fields as seen from the face: the numbers that the volume
    // integral subtracts, so that they cancel to the last bit
    auto mean_flux = [&](auto ax_c, const C q[NF], C F[NF]) {
        constexpr int AX = decltype(ax_c)::value, TENS[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
        C f[9];
        fluxes(q, f);
        F[0] = q[1 + AX];
#pragma unroll
        for (int j = 1; j < 4; j++) F[j] = f[TENS[AX][face_field<AX>(j) - 1]];
        F[4] = f[6 + AX];
    };
    auto solve = [&](const C qL[NF], const C qR[NF], C F[NF]) {
        if constexpr (RS == 1)
            exact_rs<PR, 0>(qL, qR, gam, F);
        else
            hllc<PR, 0>(qL, qR, gam, F);
    };
    // one row (second-axis node b) of a face's modes: coefficients along the last axis
    auto row_of = [&](const C *tp, int stride, const C pb[n], C o[n]) {
#pragma unroll
        for (int q = 0; q <= K; q++) {
            C s = tp[t2<K>(0, q) * stride];
#pragma unroll
            for (int p = 1; p <= K - q; p++) s = fma_(pb[p], tp[t2<K>(p, q) * stride], s);
            o[q] = s;
        }
    };
    // a point value: the row's variation first, the cell mean last, so that each point's value is rounded
    // by itself and the points of a face share no rounding of the mean
    auto point_of = [&](const C o[n], const C pc[n], C mean) -> C {
        C s = o[0];
#pragma unroll
        for (int q = K; q >= 1; q--) s = fma_(pc[q], o[q], s);
        return s + mean;
    };
    // the same at node c, known at compile time: terms whose coefficient is zero drop out
    auto point_at = [&](const C o[n], int c, C mean) -> C {
        C s = o[0];
#pragma unroll
        for (int q = K; q >= 1; q--)  // nodes 0 and 2 share the even part
            if (L::P[q][c] != 0.0) s = fma_((C)L::P[q][c], o[q], s);
        return s + mean;
    };
    // moments of a face's point fluxes: row b's contribution, from its moments s along the last axis
    auto add_row = [&](C m[NT], const C s[n], C wb, const C pb[n]) {
#pragma unroll
        for (int q = 0; q <= K; q++) {
            const C t = wb * s[q];
            m[t2<K>(0, q)] += t;
#pragma unroll
            for (int p = 1; p <= K - q; p++) m[t2<K>(p, q)] = fma_(pb[p], t, m[t2<K>(p, q)]);
        }
    };
    // (The lambdas that solve faces are inlined by attribute: with the FP64 exact solver they pass the
    // inliner's limit, and as calls they cost half of the kernel's speed or do not compile.)
    // the face between this lane's cell (trace modes at lp, means lm) and the cell above (modes at rp,
    // value stride rs, means rm), the modes in LDS: flux moments, the flux F0 subtracted at the points
    auto face = [&](auto ax_c, const C *lp, const C lm[NF], const C *rp, auto rs_c, const C rm[NF], const C F0[NF],
                    C m[NF][NT]) __attribute__((always_inline)) {
        constexpr int AX = decltype(ax_c)::value, RSTR = decltype(rs_c)::value;
        // One point after the other: the compiler otherwise interpolates a row's points ahead of their solves
        // and spills about 100 registers at k = 2 (128^3 undriven, us: FP32 894 -> 547, FP64 1611 -> 1259).  At
        // k = 1 in FP64 it leaves 256 registers, two waves per SIMD (466 -> 387).  k = 1 in FP32 has the
        // registers (181, 183 with it); in the split form the chain's latency counts (16^3 k = 2 FP32 14.5,
        // 14.9 with it).
        constexpr bool PIN = !SPLIT && (K == 2 || sizeof(C) == 8);
#pragma unroll
        for (int f = 0; f < NF; f++)
#pragma unroll
            for (int t = 0; t < NT; t++) m[f][t] = C(0);
#pragma unroll (K == 1 ? 2 : 1)
        for (int b = 0; b < n; b++) {
            C pb[n], ol[NF][n], orr[NF][n], s[NF][n];
            pb[0] = C(1);
#pragma unroll
            for (int p = 1; p <= K; p++) pb[p] = leg_at<K, C>(p, b);
            C wb = (C)L::W[0];
            if (K == 2) wb = b == 1 ? (C)L::W[1] : wb;
#pragma unroll
            for (int f = 0; f < NF; f++) {
                row_of(lp + f * NT * 64, 64, pb, ol[f]);
                row_of(rp + f * NT * RSTR, RSTR, pb, orr[f]);
#pragma unroll
                for (int q = 0; q <= K; q++) s[f][q] = C(0);
            }
#pragma unroll
            for (int c = 0; c < n; c++) {
                C qL[NF], qR[NF], F[NF];
#pragma unroll
                for (int f = 0; f < NF; f++) {
                    qL[f] = point_at(ol[f], c, lm[face_field<AX>(f)]);
                    qR[f] = point_at(orr[f], c, rm[face_field<AX>(f)]);
                }
                solve(qL, qR, F);
#pragma unroll
                for (int f = 0; f < NF; f++) {
                    const C d = F[f] - F0[f];
#pragma unroll
                    for (int q = 0; q <= K; q++)
                        if (L::P[q][c] != 0.0) s[f][q] = fma_((C)(L::W[c] * L::P[q][c]), d, s[f][q]);
                }
                if constexpr (PIN) pin(s);
            }
#pragma unroll
            for (int f = 0; f < NF; f++) add_row(m[f], s[f], wb, pb);
        }
    };
    // the flux moments m of one face into R (side: +1 high face, -1 low face)
    auto lift = [&](auto ax_c, auto sgn_c, const C m[NF][NT]) {
        constexpr int AX = decltype(ax_c)::value, SG = decltype(sgn_c)::value;
#pragma unroll
        for (int f = 0; f < NF; f++)
#pragma unroll
            for (int p = 0; p <= K; p++)
#pragma unroll
                for (int q = 0; q <= K - p; q++) {
                    const C v = (SG > 0 ? ih[AX] : -ih[AX]) * m[f][t2<K>(p, q)];
#pragma unroll
                    for (int r = 0; r <= K - p - q; r++) {
                        C &o = R[face_field<AX>(f)][face_mode<K, AX>(r, p, q)];
                        if (r == 0)
                            o += v;
                        else
                            o = fma_((C)((SG < 0 && (r & 1)) ? -L::E[r] : L::E[r]), v, o);
                    }
                }
    };
    auto put_modes = [&](C *dst, int stride, const C t[NF][NT]) {
#pragma unroll
        for (int f = 0; f < NF; f++)
#pragma unroll
            for (int j = 0; j < NT; j++) dst[(f * NT + j) * stride] = t[f][j];
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using PLUS = std::integral_constant<int, 1>;
    using MINUS = std::integral_constant<int, -1>;
    using YES = std::true_type;
    using NO = std::false_type;

    // the weights of the 40 cells across the tile's edges, requested before the volume integral
    // (DX, DY: those of the x, the y faces)
    auto request_edges = [&](int z, auto dx_c, auto dy_c) {
        constexpr bool DX = decltype(dx_c)::value, DY = decltype(dy_c)::value;
        const int el = opaque(lane);
        const PlaneView<C, BIG> py(yin, plane, z, ycell + (long long)(el >> 5) * LD::H * nx);
        C *dst = lds + LD::RAW;
        asm volatile("" : "+s"(dst));
#pragma unroll
        for (int i = 0; DY && i < NF; i++)
#pragma unroll
            for (int l = 0; l < LD::H; l++) py.to_lds(i * N + l, unx, dst + (i * LD::H + l) * 64);
        if constexpr (!DX) return;
        const PlaneView<C, BIG> px(yin, plane, z, xcell + (long long)(el >> 3) * nx);
        dst += NF * LD::H * 64;
#pragma unroll
        for (int r = 0; r < NF * N / 8; r++) px.to_lds(8 * r, unx, dst + r * 64);
        if ((NF * N) % 8 != 0 && el < (NF * N) % 8 * 8) px.to_lds(NF * N / 8 * 8, unx, dst + NF * N / 8 * 64);
    };
    // trace modes of the edge cells and of the tile's own low-edge cells, then the fluxes of the 20
    // low-edge faces and their moments, relative to the mean flux of the tile's cell; em: the means of the
    // edge cell that this lane took (those past the high edges are asked for by the lanes next to them)
    constexpr int EYH = CTX, EXH = (SPLIT ? 0 : 2 * CTX) + CTY;  // first lane of the y, x high-edge cells
    auto edges = [&](int z, auto dx_c, auto dy_c, C em[NF]) __attribute__((always_inline)) {
        constexpr bool DX = decltype(dx_c)::value, DY = decltype(dy_c)::value;
        constexpr int FC0 = DX ? 0 : CTY, NFC = (DX ? CTY : 0) + (DY ? CTX : 0);  // first and number of low-edge faces
        constexpr int LX = DY ? 2 * CTX : 0;                                     // first lane of the x edges' cells
        const int ol = opaque(lane), cx = ol & (CTX - 1), cy = ol / CTX;
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the edge cells have landed
        lds_order();
        // lanes 0..31 take the y edges' cells, 32..39 the x edges' (the others read along and drop them);
        // a mode is read as seen from the face, with degrees (r, p, q)
        const bool ay = DY && (!DX || ol < LX);
        constexpr int WD = sizeof(C) / 4 * 64;  // words of a load
        const int *const raw = reinterpret_cast<const int *>(lds + LD::RAW);
        C ew[NF][N];
        if (ay) {
#pragma unroll
            for (int i = 0; i < NF; i++)
#pragma unroll
                for (int l = 0; l < N; l++) {
                    const int ly = face_mode<K, 1>(T.u[l], T.v[l], T.w[l]);
                    ew[i][l] = from_lds(raw + ol + (i * LD::H + ly % LD::H) * WD + (ly >= LD::H ? 32 : 0), C());
                }
        } else {
#pragma unroll
            for (int i = 0; i < NF; i++)
#pragma unroll
                for (int l = 0; l < N; l++) {
                    const int val = i * N + l;
                    ew[i][l] = from_lds(raw + (ol & 7) + (NF * LD::H + val / 8) * WD + val % 8 * 8, C());
                }
        }
#pragma unroll
        for (int i = 0; i < NF; i++) em[i] = ew[i][0];
        lds_order();
        C *const lmean = le + 2 * NV * EF;
        if (ol < LX + (DX ? 2 * CTY : 0)) {
            const bool hi = ay ? ol >= CTX : ol >= LX + CTY;
            const int j = ay ? cx : ol & (CTY - 1);
            const C sg = hi ? C(-1) : C(1);
            const int stride = hi ? CX_PLANE : EF;
            const int d0 = opaque(hi ? (ay ? SL_YHI : SL_XHI) + j : LD::X + (ay ? CTY : 0) + j);
            C c1[n];
#pragma unroll
            for (int r = 0; r <= K; r++) c1[r] = (r & 1) ? sg * (C)L::E[r] : (C)L::E[r];
#pragma unroll
            for (int i = 0; i < NF; i++) {
                const int f = i == 1 ? (ay ? 2 : 1) : i == 2 ? (ay ? 1 : 2) : i;
                C *dst = lds + d0 + f * NT * stride;
                if (!hi) lmean[f * EF + (ay ? CTY : 0) + j] = em[i];
#pragma unroll
                for (int p = 0; p <= K; p++)
#pragma unroll
                    for (int q = 0; q <= K - p; q++) {
                        const bool dev = p + q == 0;
                        C s = dev ? c1[1] * ew[i][mode_of<K>(1, 0, 0)] : ew[i][mode_of<K>(0, p, q)];
#pragma unroll
                        for (int r = dev ? 2 : 1; r <= K - p - q; r++) s = fma_(c1[r], ew[i][mode_of<K>(r, p, q)], s);
                        dst[t2<K>(p, q) * stride] = s;
                    }
            }
        }
        {
            C t[NF][NT];
            if constexpr (DX) trace(I0{}, MINUS{}, t);
            if (DX && cx == 0) put_modes(le + opaque(NV * EF + cy), EF, t);
            if constexpr (DY) trace(I1{}, MINUS{}, t);
            if (DY && cy == 0) put_modes(le + opaque(NV * EF + CTY + cx), EF, t);
#pragma unroll
            for (int f = 0; f < NF; f++) {
                if (DX && cx == 0) lmean[(NF + f) * EF + cy] = w[face_field<0>(f)][0];
                if (DY && cy == 0) lmean[(NF + f) * EF + CTY + cx] = w[face_field<1>(f)][0];
            }
            C q[NF], F0[NF];
            means(q);
            if constexpr (DX) mean_flux(I0{}, q, F0);
#pragma unroll
            for (int f = 0; f < NF; f++)
                if (DX && cx == 0) lmean[(2 * NF + f) * EF + cy] = F0[f];
            if constexpr (DY) mean_flux(I1{}, q, F0);
#pragma unroll
            for (int f = 0; f < NF; f++)
                if (DY && cy == 0) lmean[(2 * NF + f) * EF + CTY + cx] = F0[f];
        }
        lds_order();
#pragma unroll 1
        for (int e = opaque(FC0 * P + lane); e < (FC0 + NFC) * P; e += 64) {
            const int fc = e / P, pt = e - fc * P, b = pt / n, c = pt - b * n;
            C pb[n], pc[n], qL[NF], qR[NF], F[NF];
            pb[0] = pc[0] = C(1);
#pragma unroll
            for (int p = 1; p <= K; p++) {
                pb[p] = leg_at<K, C>(p, b);
                pc[p] = leg_at<K, C>(p, c);
            }
#pragma unroll
            for (int f = 0; f < NF; f++) {
                C o[n];
                row_of(le + f * NT * EF + fc, EF, pb, o);
                qL[f] = point_of(o, pc, lmean[f * EF + fc]);
                row_of(le + (NV + f * NT) * EF + fc, EF, pb, o);
                qR[f] = point_of(o, pc, lmean[(NF + f) * EF + fc]);
            }
            solve(qL, qR, F);
#pragma unroll
            for (int f = 0; f < NF; f++) lx[flux_slot(f * EF * P + e)] = F[f] - lmean[(2 * NF + f) * EF + fc];
        }
        lds_order();
#pragma unroll 1
        for (int e = opaque(lane); e < NFC * NF; e += 64) {  // (face, field)
            const int f = e / NFC, fc = FC0 + e - f * NFC;
            C m[NT];
#pragma unroll
            for (int t = 0; t < NT; t++) m[t] = C(0);
#pragma unroll
            for (int b = 0; b < n; b++) {
                C pb[n], s[n];
#pragma unroll
                for (int p = 0; p <= K; p++) {
                    pb[p] = (C)L::P[p][b];
                    s[p] = C(0);
                }
#pragma unroll
                for (int c = 0; c < n; c++) {
                    const C d = lx[flux_slot((f * EF + fc) * P + b * n + c)];
#pragma unroll
                    for (int q = 0; q <= K; q++)
                        if (L::P[q][c] != 0.0) s[q] = fma_((C)(L::W[c] * L::P[q][c]), d, s[q]);
                }
                add_row(m, s, (C)L::W[b], pb);
            }
            C *dst = lx + f * NT * CX_PLANE + (fc < CTY ? SL_XLO + fc : SL_YLO + fc - CTY);
#pragma unroll
            for (int t = 0; t < NT; t++) dst[t * CX_PLANE] = m[t];
        }
        lds_order();
    };
    // the +x or +y face of every lane; both of its cells take the moments
    auto side = [&](auto ax_c, const C em[NF]) __attribute__((always_inline)) {
        constexpr int AX = decltype(ax_c)::value;
        const int ol = opaque(lane), sx = ol & (CTX - 1), sy = ol / CTX;
        // slots of the cell above, of this one, and of the moments from below
        const int up = AX == 0 ? (sx == CTX - 1 ? SL_XHI + sy : ol + 1) : (sy == CTY - 1 ? SL_YHI + sx : ol + CTX);
        const int down = AX == 0 ? (sx == 0 ? SL_XLO + sy : ol - 1) : (sy == 0 ? SL_YLO + sx : ol - CTX);
        const bool last = AX == 0 ? sx == CTX - 1 : sy == CTY - 1, first = AX == 0 ? sx == 0 : sy == 0;
        constexpr int STEP = AX == 0 ? 1 : CTX;
        C F0[NF], lm[NF], rm[NF], m[NF][NT];
        {
            C t[NF][NT];
            trace(ax_c, MINUS{}, t);
            put_modes(lx + ol, CX_PLANE, t);
            trace(ax_c, PLUS{}, t);
            put_modes(le + opaque(lane), 64, t);
        }
        lds_order();
        means(lm);
#pragma unroll
        for (int i = 0; i < NF; i++) {
            const C in = lane_value(lm[i], ol + STEP), out = lane_value(em[i], AX == 0 ? EXH + sy : EYH + sx);
            rm[i] = last ? out : in;
        }
        mean_flux(ax_c, lm, F0);
        face(ax_c, le + ol, lm, lx + up, std::integral_constant<int, CX_PLANE>{}, rm, F0, m);
        lift(ax_c, PLUS{}, m);
        lds_order();
        put_modes(lx + ol, CX_PLANE, m);
        lds_order();
        const C *src = lx + down;
#pragma unroll
        for (int f = 0; f < NF; f++)
#pragma unroll
            for (int j = 0; j < NT; j++) m[f][j] = src[(f * NT + j) * CX_PLANE];
        // from the mean flux of the cell below to this one's (the low-edge faces' moments have it already);
        // the difference is small where the flux is not, so it is taken before the moment is touched
#pragma unroll
        for (int f = 0; f < NF; f++) {
            const C d = lane_value(F0[f], ol - STEP) - F0[f];
            m[f][0] += first ? C(0) : d;
        }
        lift(ax_c, MINUS{}, m);
        pin(R);
        lds_order();
    };
    // volume integral and driving source of the Gauss planes A0 <= qa < A1 along x
    auto volume = [&](int z, auto a0_c, auto a1_c) {
        constexpr int A0 = decltype(a0_c)::value, A1 = decltype(a1_c)::value;
        constexpr int STASHED = SPLIT ? 0 : LD::STASHED;
        C mu[9][NL];  // moments of the fluxes xx xy xz yy yz zz of the momentum, x y z of the energy
#pragma unroll
        for (int j = 0; j < 9; j++)
#pragma unroll
            for (int l = 0; l < NL; l++) mu[j][l] = C(0);
        C q0[NF], fb[9];
        means(q0);
        fluxes(q0, fb);
        // driving acceleration at the points of a column, requested two columns ahead; the cache holds a
        // tile's 64 values of a point together, so a read is two whole cache lines
        C ac[3][3][n];
        auto accel = [&](int col, C o[3][n]) {
            constexpr int AR = 3 * n * n * n;
            const PlaneView<C, BIG> av(a.acache, AR * 64, (long long)z * ntx * nty + by * ntx + bx, lane);
            const int qa = col / n, qb = col % n;
#pragma unroll
            for (int c = 0; c < 3; c++)
#pragma unroll
                for (int qc = 0; qc < n; qc++) o[c][qc] = av.get(c * n * n * n + (qc * n + qb) * n + qa, 64);
        };
        if constexpr (FORCE) {
            accel(A0 * n, ac[(A0 * n) % 3]);
            accel(A0 * n + 1, ac[(A0 * n + 1) % 3]);
        }
        if constexpr (STASHED > 0) {
            lds_order();
            C *const wp = lds + opaque(lane);
#pragma unroll
            for (int i = 0; i < NF; i++)
#pragma unroll
                for (int l = 1; l < N; l++) wp[(i * (N - 1) + l - 1) * 64] = w[i][l];
            lds_order();
        }
        const C *const ws = lds + opaque(lane);  // the weights' copies
#pragma unroll
        for (int qa = A0; qa < A1; qa++) {
            C Mx[NF][NT];
#pragma unroll
            for (int i = 0; i < NF; i++)
#pragma unroll
                for (int v = 0; v <= K; v++)
#pragma unroll
                    for (int ww = 0; ww <= K - v; ww++) {
                        auto wt = [&](int l) { return STASHED && l ? ws[(i * (N - 1) + l - 1) * 64] : w[i][l]; };
                        C s = v + ww == 0 ? C(0) : wt(mode_of<K>(0, v, ww));
#pragma unroll
                        for (int u = 1; u <= K - v - ww; u++)
                            if (L::P[u][qa] != 0.0) s = fma_((C)L::P[u][qa], wt(mode_of<K>(u, v, ww)), s);
                        Mx[i][t2<K>(v, ww)] = s;
                    }
#pragma unroll
            for (int qb = 0; qb < n; qb++) {
                C Z[NF][n], mq[9][K], sq[4][n];
                const int col = qa * n + qb;
                if constexpr (FORCE)
                    if (col + 2 < A1 * n) accel(col + 2, ac[(col + 2) % 3]);
#pragma unroll
                for (int i = 0; i < NF; i++)
#pragma unroll
                    for (int ww = 0; ww <= K; ww++) {
                        C s = Mx[i][t2<K>(0, ww)];
#pragma unroll
                        for (int v = 1; v <= K - ww; v++)
                            if (L::P[v][qb] != 0.0) s = fma_((C)L::P[v][qb], Mx[i][t2<K>(v, ww)], s);
                        Z[i][ww] = s;
                    }
#pragma unroll
                for (int j = 0; j < 9; j++)
#pragma unroll
                    for (int m = 0; m < K; m++) mq[j][m] = C(0);
#pragma unroll
                for (int j = 0; j < 4; j++)
#pragma unroll
                    for (int m = 0; m < n; m++) sq[j][m] = C(0);
#pragma unroll
                for (int qc = 0; qc < n; qc++) {
                    C q[NF];
#pragma unroll
                    for (int i = 0; i < NF; i++) {
                        C s = Z[i][0];
#pragma unroll
                        for (int ww = K; ww >= 1; ww--)
                            if (L::P[ww][qc] != 0.0) s = fma_((C)L::P[ww][qc], Z[i][ww], s);
                        q[i] = s + w[i][0];  // the mean last, as on the faces
                    }
                    C f[9];
                    fluxes(q, f);
#pragma unroll
                    for (int j = 0; j < 9; j++) {
                        const C d = f[j] - fb[j];
#pragma unroll
                        for (int m = 0; m < K; m++)
                            if (L::P[m][qc] != 0.0) mq[j][m] = fma_((C)(L::W[qc] * L::P[m][qc]), d, mq[j][m]);
                    }
                    if constexpr (FORCE) {
                        C sv[4];
#pragma unroll
                        for (int c = 0; c < 3; c++) sv[c] = q[0] * ac[col % 3][c][qc];
                        sv[3] = q[1] * ac[col % 3][0][qc] + q[2] * ac[col % 3][1][qc] +
                                q[3] * ac[col % 3][2][qc];
#pragma unroll
                        for (int j = 0; j < 4; j++)
#pragma unroll
                            for (int m = 0; m < n; m++)
                                if (L::P[m][qc] != 0.0) sq[j][m] = fma_((C)(L::W[qc] * L::P[m][qc]), sv[j], sq[j][m]);
                    }
                }
                // this (x, y) column into the moments of degree <= k - 1; the source into R
#pragma unroll
                for (int l = 0; l < NL; l++) {
                    const C cf = (C)(L::W[qa] * L::W[qb] * L::P[T.u[l]][qa] * L::P[T.v[l]][qb]);
#pragma unroll
                    for (int j = 0; j < 9; j++)
                        if (L::P[T.u[l]][qa] * L::P[T.v[l]][qb] != 0.0) mu[j][l] = fma_(cf, mq[j][T.w[l]], mu[j][l]);
                }
                if constexpr (FORCE) {
#pragma unroll
                    for (int l = 0; l < N; l++) {
                        const C cf = (C)(-L::W[qa] * L::W[qb] * L::P[T.u[l]][qa] * L::P[T.v[l]][qb]);
#pragma unroll
                        for (int j = 0; j < 4; j++)
                            if (L::P[T.u[l]][qa] * L::P[T.v[l]][qb] != 0.0)
                                R[1 + j][l] = fma_(cf, sq[j][T.w[l]], R[1 + j][l]);
                    }
                    pin(R);
                }
                pin(mu);
            }
        }
        if constexpr (STASHED > 0) {
            lds_order();
#pragma unroll
            for (int i = 0; i < NF; i++)
#pragma unroll
                for (int l = 1; l < N; l++) w[i][l] = ws[(i * (N - 1) + l - 1) * 64];
        }
        // R_l -= 2/h_a sum over l' of d(l, l') mu_l', l' = l with a lower degree of the other parity along
        // axis a: d = sqrt((2u+1)(2u'+1)); the mass flux's moments are the momentum's modes (mode 0 is the
        // subtracted mean flux)
        constexpr int TENS[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
#pragma unroll
        for (int l = 1; l < N; l++)
#pragma unroll
            for (int ax = 0; ax < 3; ax++) {
                const int deg = ax == 0 ? T.u[l] : ax == 1 ? T.v[l] : T.w[l];
#pragma unroll
                for (int e = deg - 1; e >= 0; e -= 2) {
                    const int lp = ax == 0 ? mode_of<K>(e, T.v[l], T.w[l])
                                           : ax == 1 ? mode_of<K>(T.u[l], e, T.w[l]) : mode_of<K>(T.u[l], T.v[l], e);
                    const C d = (C)(-2.0 * L::E[deg] * L::E[e]) * ih[ax];
                    if (A0 == 0 && lp > 0) R[0][l] = fma_(d, w[1 + ax][lp], R[0][l]);
#pragma unroll
                    for (int i = 0; i < 3; i++) R[1 + i][l] = fma_(d, mu[TENS[i][ax]][lp], R[1 + i][l]);
                    R[4][l] = fma_(d, mu[6 + ax][lp], R[4][l]);
                }
            }
    };

    // the +z face of the plane in w, whose mean flux is F0: flux moments mz relative to F0; the next
    // plane's cells are left in w
    auto zface = [&](int z, C F0[NF]) __attribute__((always_inline)) {
        C lm[NF], rm[NF];
        means(lm);
        mean_flux(I2{}, lm, F0);
        {
            C t[NF][NT];
            trace(I2{}, PLUS{}, t);
            put_modes(lds + LD::S + opaque(lane), 64, t);
            load_cells(z + 1);
            trace(I2{}, MINUS{}, t);
            put_modes(lx + opaque(lane), 64, t);
        }
        lds_order();
        means(rm);
        face(I2{}, lds + LD::S + opaque(lane), lm, lx + opaque(lane), std::integral_constant<int, 64>{}, rm, F0, mz);
        lds_order();
    };

    // the closure's correction, the stage update and the store of the plane in R
    auto finish = [&](int z) {
        const PlaneView<C, BIG> po(a.out, plane, z, cell);
        if (K == 1 && a.corr) {  // learned closure: dy/dt = -R + c
            const PlaneView<C, BIG> pc(a.corr, plane, z, cell);
#pragma unroll
            for (int i = 0; i < NF; i++)
#pragma unroll
                for (int l = 0; l < N; l++)
                    R[i][l] -= pc.get(i * N + l, unx) - (l == 0 ? (C)a.cmean[i] : C(0));
        }
        // out = a y0 + b (yin - dt R); the stage input is read again (through the caches) rather than held
        // across the faces
        auto combine = [&](auto with0) {
            const C bb = uniform((C)a.b), aa = uniform((C)a.a);
            const PlaneView<C, BIG> p1(yin, plane, z, cell), p0(a.y0, plane, z, cell);
            C v[NF][N], v0[NF][N];
#pragma unroll
            for (int i = 0; i < NF; i++)
#pragma unroll
                for (int l = 0; l < N; l++) {
                    if (with0) v0[i][l] = p0.get(i * N + l, unx);
                    v[i][l] = p1.get(i * N + l, unx);
                }
#pragma unroll
            for (int i = 0; i < NF; i++)
#pragma unroll
                for (int l = 0; l < N; l++) {
                    R[i][l] = bb * (v[i][l] - dt * R[i][l]);
                    if (with0) R[i][l] = aa * v0[i][l] + R[i][l];
                }
        };
        if (a.mode != 0) {
            if (a.a != 0.0)
                combine(std::true_type{});
            else
                combine(std::false_type{});
        }
        if (keep) {
#pragma unroll
            for (int i = 0; i < NF; i++)
#pragma unroll
                for (int l = 0; l < N; l++) po.put(i * N + l, unx, R[i][l]);
        }
        // the next step's CFL rate from the means just stored (the same cells, values and arithmetic as
        // the reduction that the launch would otherwise be followed by)
        if constexpr (SPLIT) {
            if (a.next_rate) {
                const double r = wave_max(keep ? cfl_rate((double)R[0][0], (double)R[1][0], (double)R[2][0], (double)R[3][0],
                                                          (double)R[4][0], a.gamma, a.ih[0], a.ih[1], a.ih[2])
                                               : 0.0);
                if (lane == 0) rate_max(a.next_rate, r);
            }
        }
    };

    C F0[NF];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < NF; i++)
#pragma unroll
            for (int l = 0; l < N; l++) R[i][l] = C(0);
    };
    // the flux moments of the face below, relative to F0, onto this cell's mean flux
    auto rebase = [&]() {
        C q[NF], F[NF];
        means(q);
        mean_flux(I2{}, q, F);
#pragma unroll
        for (int f = 0; f < NF; f++) mz[f][0] += F0[f] - F[f];
    };
    C em[NF];
    if constexpr (SPLIT) {
        using SP = CellSplit<K, C>;
        if (wave < 2) {
            if (wave == 0)
                request_edges(z0, YES{}, NO{});
            else
                request_edges(z0, NO{}, YES{});
            load_cells(z0);
            clear();
            if (wave == 0) {
                edges(z0, YES{}, NO{}, em);
                side(I0{}, em);
            } else {
                edges(z0, NO{}, YES{}, em);
                side(I1{}, em);
            }
        } else if (wave == 2) {
            load_cells(z0 - 1);
            zface(z0 - 1, F0);
            rebase();
            clear();
            lift(I2{}, MINUS{}, mz);
            pin(R);
            zface(z0, F0);
            lift(I2{}, PLUS{}, mz);
        } else {
            load_cells(z0);
            clear();
            if constexpr (SP::NVOL == 1)
                volume(z0, I0{}, std::integral_constant<int, n>{});
            else if (wave == SP::VOL)
                volume(z0, I0{}, I1{});
            else if (wave == SP::VOL + 1)
                volume(z0, I1{}, I2{});
            else
                volume(z0, I2{}, std::integral_constant<int, 3>{});
        }
        if (wave != SP::VOL) {  // shares of R, in the waves' own regions
            lds_order();
            C *p = lds + opaque(lane);
#pragma unroll
            for (int i = 0; i < NF; i++)
#pragma unroll
                for (int l = 0; l < N; l++) p[(i * N + l) * 64] = R[i][l];
        }
        __syncthreads();
        if (wave != SP::VOL) return;
#pragma unroll 1
        for (int v = 0; v < SP::WAVES; v++) {
            if (v == SP::VOL) continue;
            const C *p = lds0 + SP::base(v) + opaque(lane);
#pragma unroll
            for (int i = 0; i < NF; i++)
#pragma unroll
                for (int l = 0; l < N; l++) R[i][l] += p[(i * N + l) * 64];
        }
        finish(z0);
    } else {
        load_cells(z0 - 1);
        zface(z0 - 1, F0);
#pragma unroll 1
        for (int z = z0; z < z1; z++) {
            rebase();
            clear();
            lift(I2{}, MINUS{}, mz);
            pin(R);
            request_edges(z, YES{}, YES{});
            volume(z, I0{}, std::integral_constant<int, n>{});
            pin(R);
            edges(z, YES{}, YES{}, em);
            side(I0{}, em);
            side(I1{}, em);
            zface(z, F0);
            lift(I2{}, PLUS{}, mz);
            finish(z);
        }
    }
}

template <int K, class C, bool FORCE, int RS, bool BIG>
__global__ __launch_bounds__(64 * CELL_WAVES)
    __attribute__((amdgpu_waves_per_eu(cell_waves<K, C>(), cell_waves<K, C>()))) void cell_stage_kernel(StageArgs a) {
    cell_stage<K, C, FORCE, RS, BIG, false>(a);
}

template <int K, class C>
constexpr int split_simd_waves() { return (CellSplit<K, C>::WAVES + 3) / 4; }
template <int K, class C, bool FORCE, int RS>
__global__ __launch_bounds__((64 * CellSplit<K, C>::WAVES))
    __attribute__((amdgpu_waves_per_eu(split_simd_waves<K, C>()))) void cell_split_kernel(StageArgs a) {
    cell_stage<K, C, FORCE, RS, false, true>(a);
}

template <int K, class C>
constexpr int cell_lds(int waves) { return waves * CellLds<K>::ELEMS * (int)sizeof(C); }
template <int K, class C>
constexpr int split_lds() { return CellSplit<K, C>::ELEMS * (int)sizeof(C); }

template <int K, class C, bool FORCE, int RS>
static hipError_t launch_cell_t(const StageArgs &a, hipStream_t s) {
    const long long plane = (long long)sizeof(C) * NF * Dims<K>::N * a.nx * a.ny;
    const bool big = plane >= (1LL << 31);
    if (a.wgw == 0) {  // one tile and plane per workgroup, split by task (small meshes, so never big planes)
        if (big) return hipErrorInvalidValue;
        hipLaunchKernelGGL((cell_split_kernel<K, C, FORCE, RS>), dim3((unsigned)a.nitems),
                           dim3(64 * CellSplit<K, C>::WAVES), (split_lds<K, C>()), s, a);
        return hipGetLastError();
    }
    const dim3 grid((unsigned)((a.nitems + a.wgw - 1) / a.wgw)), block(64 * a.wgw);
    if (big)
        hipLaunchKernelGGL((cell_stage_kernel<K, C, FORCE, RS, true>), grid, block, (cell_lds<K, C>(a.wgw)), s, a);
    else
        hipLaunchKernelGGL((cell_stage_kernel<K, C, FORCE, RS, false>), grid, block, (cell_lds<K, C>(a.wgw)), s, a);
    return hipGetLastError();
}

template <int K, class C>
static hipError_t launch_cell_kc(const StageArgs &a, hipStream_t s) {
    if (a.riemann) return a.forcing ? launch_cell_t<K, C, true, 1>(a, s) : launch_cell_t<K, C, false, 1>(a, s);
    return a.forcing ? launch_cell_t<K, C, true, 0>(a, s) : launch_cell_t<K, C, false, 0>(a, s);
}

hipError_t launch_stage_cell(int k, int prec, const StageArgs &a, hipStream_t s) {
    const bool f64 = prec == DG_FP64;
    if (k == 1) return f64 ? launch_cell_kc<1, double>(a, s) : launch_cell_kc<1, float>(a, s);
    if (k == 2) return f64 ? launch_cell_kc<2, double>(a, s) : launch_cell_kc<2, float>(a, s);
    return hipErrorInvalidValue;
}

template <int K, class C, bool FORCE, int RS>
static hipError_t cell_attr_t() {
    const int lds = cell_lds<K, C>(CELL_WAVES);
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&cell_stage_kernel<K, C, FORCE, RS, false>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(&cell_stage_kernel<K, C, FORCE, RS, true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e == hipSuccess)
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(&cell_split_kernel<K, C, FORCE, RS>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, split_lds<K, C>());
    return e;
}
template <int K, class C>
static hipError_t cell_setup_t(int *per_cu) {
    hipError_t e = cell_attr_t<K, C, false, 0>();
    if (e == hipSuccess) e = cell_attr_t<K, C, true, 0>();
    if (e == hipSuccess) e = cell_attr_t<K, C, false, 1>();
    if (e == hipSuccess) e = cell_attr_t<K, C, true, 1>();
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, cell_stage_kernel<K, C, true, 0, false>,
                                                         64 * CELL_WAVES, (size_t)cell_lds<K, C>(CELL_WAVES));
    return e;
}
// allows the kernels their LDS; per_cu: workgroups a compute unit holds
hipError_t stage_cell_setup(int k, int prec, int *per_cu) {
    const bool f64 = prec == DG_FP64;
    if (k == 1) return f64 ? cell_setup_t<1, double>(per_cu) : cell_setup_t<1, float>(per_cu);
    if (k == 2) return f64 ? cell_setup_t<2, double>(per_cu) : cell_setup_t<2, float>(per_cu);
    return hipErrorInvalidValue;
}

}  // namespace dgmi
