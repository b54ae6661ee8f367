// Turbulence diagnostics of arXiv 1602.09079 on the GPU: sub-cell sampling of the
// DG polynomials (Sec. 4: slices and PDFs use 4^3 points per cell), the shell
// power spectrum of the velocity (Sec. 3.3), the log-density PDF (Sec. 4.4) and
// the rms Mach number (Sec. 4.1).
#include <hip/hip_runtime.h>

#include <cmath>

#include "dg_internal.h"

namespace dgmi {

constexpr int SAMPLE_THREADS = 256;

long long sample_blocks(long long nc) { return (nc + SAMPLE_THREADS - 1) / SAMPLE_THREADS; }

__device__ inline float log10_d(float x) { return log10f(x); }
__device__ inline double log10_d(double x) { return log10(x); }

// S values of a velocity grid's row; pair: S is even and every row starts on a boundary of two elements,
// so they go out two at a time
template <int S, class C>
__device__ inline void store_row(C *o, const C v[S], int pair) {
    typedef C c2 __attribute__((ext_vector_type(2)));
    if (S % 2 == 0 && pair) {
#pragma unroll
        for (int a = 0; a < S; a += 2) *reinterpret_cast<c2 *>(o + a) = c2{v[a], v[a + 1]};
    } else {
#pragma unroll
        for (int a = 0; a < S; a++) o[a] = v[a];
    }
}

// One thread per cell (x consecutive over the lanes).  The cell is split into S equal parts per
// axis; per z slice of the S^3 part centres the five fields are evaluated by sum factorisation
// over the 1D Legendre factors at the centres (z, then y, then x).  Grid point (X, Y, Z) =
// (S ix + a, S iy + b, S iz + c).
// WHAT: SAMPLE_FIELDS, SAMPLE_VELOCITY (component A.what - 1; reads only its momentum and the density)
// or SAMPLE_STATS.
enum { SAMPLE_FIELDS, SAMPLE_VELOCITY, SAMPLE_STATS };
// Waves per SIMD.  The five fields in FP64 write rows of 24 and 32 bytes a lane, and more waves at it only
// spread the writes: 64^3 at S = 4, k = 2 180 us with the three waves that fit, 147 with one (4.6 TB/s of
// output), k = 3 209 and 182; k = 1 151 with eight, 135 with two.
template <int K, int S, class C, int WHAT>
constexpr int sample_waves() { return sizeof(C) == 8 && S >= 3 && WHAT == SAMPLE_FIELDS ? (K >= 2 ? 1 : 2) : 8; }
template <int K, int S, class C, int WHAT>
__global__ __launch_bounds__(SAMPLE_THREADS)
    __attribute__((amdgpu_waves_per_eu(1, sample_waves<K, S, C, WHAT>()))) void sample_kernel(SampleArgs A, Leg1D L) {
    constexpr int N = (K + 1) * (K + 2) * (K + 3) / 6;
    constexpr bool stats = WHAT == SAMPLE_STATS;
    __shared__ double red[stats ? SAMPLE_THREADS : 1];
    __shared__ unsigned int hist[stats ? DIAG_MAX_BINS + 2 : 1];
    if (stats && A.nbins > 0) {
        for (int j = threadIdx.x; j < A.nbins + 2; j += blockDim.x) hist[j] = 0u;
        __syncthreads();
    }
    C P[K + 1][S];
#pragma unroll
    for (int u = 0; u <= K; u++)
#pragma unroll
        for (int a = 0; a < S; a++) P[u][a] = (C)L.p[u][a];
    const long long cell = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    double msum = 0.0;
    if (cell < A.nc) {
        const C *y = static_cast<const C *>(A.y);
        const long long r = cell / A.nx;
        const int ix = (int)(cell - r * A.nx);
        const int iy = (int)(r % A.ny);
        const int iz = (int)(r / A.ny);
        const long long base = r * (long long)NF * N * A.nx + ix;
        constexpr int NW = WHAT == SAMPLE_VELOCITY ? 2 : NF;  // fields read: density and one momentum, or all
        C wt[NW][N];
#pragma unroll
        for (int i = 0; i < NW; i++) {
            const int fi = WHAT == SAMPLE_VELOCITY && i == 1 ? A.what : i;
#pragma unroll
            for (int l = 0; l < N; l++) wt[i][l] = y[base + (long long)(fi * N + l) * A.nx];
        }
        const C g = (C)A.gamma;
        // the statistics in FP64 from k = 3 on one slice at a time: unrolled, their code does not stay in the
        // instruction cache (rms Mach number at S = 4: 64^3 k = 3 151 -> 103 us, 48^3 k = 4 195 -> 139)
#pragma unroll (stats && K >= 3 && sizeof(C) == 8 ? 1 : S)
        for (int c = 0; c < S; c++) {
            auto eval = [&](int i, C q[S][S]) {
                C t1[K + 1][K + 1];
#pragma unroll
                for (int u = 0; u <= K; u++)
#pragma unroll
                    for (int v = 0; u + v <= K; v++) {
                        C t = 0;
#pragma unroll
                        for (int w = 0; u + v + w <= K; w++) t += wt[i][mode_of<K>(u, v, w)] * (C)L.p[w][c];
                        t1[u][v] = t;
                    }
                C t2[K + 1][S];
#pragma unroll
                for (int u = 0; u <= K; u++)
#pragma unroll
                    for (int b = 0; b < S; b++) {
                        C t = 0;
#pragma unroll
                        for (int v = 0; u + v <= K; v++) t += t1[u][v] * P[v][b];
                        t2[u][b] = t;
                    }
#pragma unroll
                for (int b = 0; b < S; b++)
#pragma unroll
                    for (int a = 0; a < S; a++) {
                        C t = 0;
#pragma unroll
                        for (int u = 0; u <= K; u++) t += t2[u][b] * P[u][a];
                        q[b][a] = t;
                    }
            };
            const long long Z = (long long)iz * S + c;
            if constexpr (WHAT == SAMPLE_FIELDS) {
                C *o = static_cast<C *>(A.out);
#pragma unroll
                for (int i = 0; i < NF; i++) {
                    C q[S][S];
                    eval(i, q);
#pragma unroll
                    for (int b = 0; b < S; b++) {
                        C *row = o + i * A.pf + Z * A.py + (long long)(iy * S + b) * A.px + (long long)ix * S;
#pragma unroll
                        for (int a = 0; a < S; a++) row[a] = q[b][a];
                    }
                }
            } else if constexpr (WHAT == SAMPLE_VELOCITY) {
                C *o = static_cast<C *>(A.out);
                C rho[S][S], m[S][S];
                eval(0, rho);
                eval(1, m);
#pragma unroll
                for (int b = 0; b < S; b++) {
#pragma unroll
                    for (int a = 0; a < S; a++) m[b][a] = m[b][a] / rho[b][a];
                    store_row<S>(o + Z * A.py + (long long)(iy * S + b) * A.px + (long long)ix * S, m[b], A.pair);
                }
            } else {
                C rho[S][S], m2[S][S], e[S][S], qm[S][S];
                eval(0, rho);
                eval(4, e);
#pragma unroll
                for (int i = 1; i < 4; i++) {
                    eval(i, qm);
#pragma unroll
                    for (int b = 0; b < S; b++)
#pragma unroll
                        for (int a = 0; a < S; a++) m2[b][a] = (i == 1 ? C(0) : m2[b][a]) + qm[b][a] * qm[b][a];
                }
#pragma unroll
                for (int b = 0; b < S; b++)
#pragma unroll
                    for (int a = 0; a < S; a++) {
                        const C rh = rho[b][a];
                        if (A.mach_partials) {
                            // |v|^2 / c^2 = |m|^2 / (gamma rho p), p = (gamma-1)(E - |m|^2/(2 rho))
                            const C p = (g - C(1)) * (e[b][a] - C(0.5) * m2[b][a] / rh);
                            msum += (double)(m2[b][a] / (g * rh * p));
                        }
                        if (A.nbins > 0) {
                            int bin;
                            if (!(rh > C(0)) || !(rh < __builtin_huge_valf())) {
                                bin = 0;
                            } else {
                                const double x = (double)log10_d(rh);
                                if (x < A.lo) bin = 0;
                                else if (x >= A.hi) bin = A.nbins + 1;
                                else {
                                    int bb = (int)floor((x - A.lo) / (A.hi - A.lo) * A.nbins);
                                    bin = 1 + (bb < A.nbins - 1 ? bb : A.nbins - 1);
                                }
                            }
                            atomicAdd(&hist[bin], 1u);
                        }
                    }
            }
        }
    }
    if constexpr (stats) {
        if (A.mach_partials) {
            red[threadIdx.x] = msum;
            __syncthreads();
            for (int h = SAMPLE_THREADS / 2; h > 0; h >>= 1) {
                if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
                __syncthreads();
            }
            if (threadIdx.x == 0) A.mach_partials[blockIdx.x] = red[0];
        }
        if (A.nbins > 0) {
            __syncthreads();
            for (int j = threadIdx.x; j < A.nbins + 2; j += blockDim.x)
                if (hist[j]) atomicAdd(&A.counts[j], (unsigned long long)hist[j]);
        }
    }
}

template <int K, int S>
static hipError_t launch_sample_ks(int prec, SampleArgs a, const Leg1D &L, hipStream_t s) {
    const long long nb = sample_blocks(a.nc);
    const size_t two = prec == DG_FP64 ? 16 : 8;
    a.pair = a.px % 2 == 0 && a.py % 2 == 0 && reinterpret_cast<uintptr_t>(a.out) % two == 0;
    const bool f64 = prec == DG_FP64;
    const dim3 grid(nb), block(SAMPLE_THREADS);
    if (a.what == 0) {
        if (f64) hipLaunchKernelGGL((sample_kernel<K, S, double, SAMPLE_FIELDS>), grid, block, 0, s, a, L);
        else hipLaunchKernelGGL((sample_kernel<K, S, float, SAMPLE_FIELDS>), grid, block, 0, s, a, L);
    } else if (a.what <= 3) {
        if (f64) hipLaunchKernelGGL((sample_kernel<K, S, double, SAMPLE_VELOCITY>), grid, block, 0, s, a, L);
        else hipLaunchKernelGGL((sample_kernel<K, S, float, SAMPLE_VELOCITY>), grid, block, 0, s, a, L);
    } else {
        if (f64) hipLaunchKernelGGL((sample_kernel<K, S, double, SAMPLE_STATS>), grid, block, 0, s, a, L);
        else hipLaunchKernelGGL((sample_kernel<K, S, float, SAMPLE_STATS>), grid, block, 0, s, a, L);
    }
    return hipGetLastError();
}

template <int K>
static hipError_t launch_sample_k(int S, int prec, const SampleArgs &a, const Leg1D &L, hipStream_t s) {
    switch (S) {
        case 1: return launch_sample_ks<K, 1>(prec, a, L, s);
        case 2: return launch_sample_ks<K, 2>(prec, a, L, s);
        case 3: return launch_sample_ks<K, 3>(prec, a, L, s);
        case 4: return launch_sample_ks<K, 4>(prec, a, L, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_sample(int k, int S, int prec, const SampleArgs &a, const Leg1D &L, hipStream_t s) {
    switch (k) {
        case 0: return launch_sample_k<0>(S, prec, a, L, s);
        case 1: return launch_sample_k<1>(S, prec, a, L, s);
        case 2: return launch_sample_k<2>(S, prec, a, L, s);
        case 3: return launch_sample_k<3>(S, prec, a, L, s);
        case 4: return launch_sample_k<4>(S, prec, a, L, s);
        default: return hipErrorInvalidValue;
    }
}

// Shell power of an R2C spectrum [M][M][Mh], Mh = M/2 + 1 (interleaved complex).  Element
// (kz, ky, kx) has wave vector (kx, ky or ky - M, kz or kz - M); it stands for itself and, for
// 0 < kx < M/2 (or kx > 0 when M is odd), for its conjugate at -n as well (weight 2).  The shell
// is the integer nearest to |n|, found in integer arithmetic: s = r + [|n|^2 > r (r + 1)],
// r = floor(sqrt(|n|^2)); |n|^2 < 2^31 for every M whose grid a device can hold.
__device__ inline int shell_of(int n2) {
    int r = (int)__builtin_amdgcn_sqrtf((float)n2);
    if (r * r > n2) r--;
    if ((r + 1) * (r + 1) <= n2) r++;
    return r + (n2 > r * (r + 1) ? 1 : 0);
}

// the lane `d` below (d = 1, 2, 4, 8, inside its row of 16), or the last lane of the row / half below
template <int CTRL, int ROWS>
__device__ inline double dpp_from(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, ROWS, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// One pass over the spectrum.  Workgroups of one wave: wave w takes a contiguous range of the rows
// (kz, ky), 64 consecutive kx at a time, and keeps a bin per shell in LDS.  Along a row the shell does
// not decrease, so the 64 elements fall into runs of one shell: a segmented scan over the lanes (six
// DPP steps; a lane adds the lane d below it only inside its run) leaves each run's sum in its last
// lane, which alone adds it to the bin.  The order of every sum is fixed by M, so the spectrum is
// bitwise reproducible and a shell's value does not depend on nbins.  The waves' bins go to
// part[w][shell] (`first`: written, else added to) and shells_sum_kernel adds them up.
//
// What bounds it: the scan's vector instructions, about 100 per 64 elements, beside one read of the
// spectrum (67 MB for 256^3 FP32).  A workgroup per shell that searched the rows for its kx intervals
// took 846 us there, most of it in the searches and in the few workgroups with the largest shells; this
// takes 48 (74 without the early request of the next 64 elements and with 2048 waves instead of 4096).
template <class C>
__global__ __launch_bounds__(64) void shells_kernel(const C *__restrict__ spec, int M, int nb, int first,
                                                    double *__restrict__ part) {
    extern __shared__ double bins[];
    typedef C c2 __attribute__((ext_vector_type(2)));
    const int lane = threadIdx.x, Mh = M / 2 + 1;
    const long long rows = (long long)M * M, per = (rows + gridDim.x - 1) / gridDim.x;
    const long long r0 = blockIdx.x * per, r1 = r0 + per < rows ? r0 + per : rows;
    for (int j = lane; j < nb; j += 64) bins[j] = 0.0;
    const int row16 = lane & ~15;
    for (long long r = r0; r < r1; r++) {
        int kz = (int)(r / M), ky = (int)(r - (long long)kz * M);
        if (ky > M / 2) ky -= M;
        if (kz > M / 2) kz -= M;
        const int c = ky * ky + kz * kz;
        if (shell_of(c) >= nb) continue;  // no element of this row is wanted: the shell grows with kx
        const c2 *row = reinterpret_cast<const c2 *>(spec) + r * Mh;
        c2 nxt = row[lane < Mh ? lane : 0];  // the next 64 elements are requested before these are summed
        for (int x0 = 0; x0 < Mh; x0 += 64) {
            const int kx = x0 + lane;
            const c2 v = nxt;
            nxt = row[kx + 64 < Mh ? kx + 64 : 0];
            const int s = kx < Mh ? shell_of(kx * kx + c) : nb;
            // the first lane has the smallest shell: the rest of this row is not wanted
            if (__builtin_amdgcn_readfirstlane(s) >= nb) break;
            double p = 0.0;
            if (s < nb) {
                const double re = (double)v[0], im = (double)v[1];
                const bool self_conj = kx == 0 || (M % 2 == 0 && kx == M / 2);
                p = (re * re + im * im) * (self_conj ? 1.0 : 2.0);
            }
            const int below = __builtin_amdgcn_update_dpp(-1, s, 0x138, 0xf, 0xf, false);  // the lane below's shell
            const unsigned long long heads = __ballot(lane == 0 || below != s);
            // first lane of this lane's run
            const int start = 63 - __builtin_clzll(heads & (~0ull >> (63 - lane)));
            double q;
            q = dpp_from<0x111, 0xf>(p);
            if (lane - 1 >= start && lane - 1 >= row16) p += q;
            q = dpp_from<0x112, 0xf>(p);
            if (lane - 2 >= start && lane - 2 >= row16) p += q;
            q = dpp_from<0x114, 0xf>(p);
            if (lane - 4 >= start && lane - 4 >= row16) p += q;
            q = dpp_from<0x118, 0xf>(p);
            if (lane - 8 >= start && lane - 8 >= row16) p += q;
            q = dpp_from<0x142, 0xa>(p);  // lane 15 to row 1, lane 47 to row 3
            if ((lane & 16) && start < row16) p += q;
            q = dpp_from<0x143, 0xc>(p);  // lane 31 to rows 2 and 3
            if (lane >= 32 && start < 32) p += q;
            const bool last = lane == 63 || ((heads >> ((lane + 1) & 63)) & 1ull);
            if (last && s < nb) bins[s] += p;
        }
    }
    for (int j = lane; j < nb; j += 64) {
        double *o = part + (long long)blockIdx.x * nb + j;
        *o = first ? bins[j] : *o + bins[j];
    }
}

// bins[s] = scale * (the waves' sums of shell s, in a fixed order); shells past the last one are zero
__global__ __launch_bounds__(1024) void shells_sum_kernel(const double *__restrict__ part, int waves, int nb, int nbins,
                                                         double scale, double *__restrict__ bins) {
    __shared__ double red[64][16];
    const int j = blockIdx.x * 16 + (threadIdx.x & 15), g = threadIdx.x >> 4;
    double sum = 0.0;
    if (j < nb)
#pragma unroll 8
        for (int w = g; w < waves; w += 64) sum += part[(long long)w * nb + j];
    red[g][threadIdx.x & 15] = sum;
    __syncthreads();
    if (g == 0 && j < nbins) {
        double t = 0.0;
        for (int i = 0; i < 64; i++) t += red[i][threadIdx.x];
        bins[j] = t * scale;
    }
}

// shells an M^3 grid has
static int shell_count(int M) {
    const double h = M / 2;
    return (int)floor(sqrt(3.0 * h * h) + 0.5) + 1;
}
int shells_waves(int M) {
    const long long w = SHELL_PARTS / shell_count(M), rows = (long long)M * M;
    return (int)(w < 4096 ? (w < rows ? w : rows) : (4096 < rows ? 4096 : rows));
}

hipError_t launch_shells(int prec, const void *spec, int M, int nbins, int first, double *part, hipStream_t s) {
    const int ns = shell_count(M), nb = nbins < ns ? nbins : ns, nw = shells_waves(M);
    const size_t lds = (size_t)nb * sizeof(double);
    if (prec == DG_FP64)
        hipLaunchKernelGGL(shells_kernel<double>, dim3(nw), dim3(64), lds, s, (const double *)spec, M, nb, first, part);
    else
        hipLaunchKernelGGL(shells_kernel<float>, dim3(nw), dim3(64), lds, s, (const float *)spec, M, nb, first, part);
    return hipGetLastError();
}

hipError_t launch_shells_sum(const double *part, int M, int nbins, double scale, double *bins, hipStream_t s) {
    const int ns = shell_count(M), nb = nbins < ns ? nbins : ns;
    hipLaunchKernelGGL(shells_sum_kernel, dim3((nbins + 15) / 16), dim3(1024), 0, s, part, shells_waves(M), nb, nbins,
                       scale, bins);
    return hipGetLastError();
}

__global__ void fill_zero_kernel(unsigned long long *p, long long n) {
    for (long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (long long)gridDim.x * blockDim.x)
        p[j] = 0ull;
}

hipError_t launch_fill_zero(unsigned long long *p, long long n, hipStream_t s) {
    long long nb = (n + 255) / 256;
    if (nb > 1024) nb = 1024;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(fill_zero_kernel, dim3(nb), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

}  // namespace dgmi
