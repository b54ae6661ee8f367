// Training kernels of the closure's tanh network for shapes whose activations fit in LDS (a 16-sample
// tile of every layer; 140-128-128-20 takes 37 KB): two launches per loss gradient and one that sums
// the shares, instead of thirteen.  All products on the FP32 matrix cores (16x16x4, exact products).
//
// What bounds them: latency.  A 4096-sample gradient at 140-128-128-20 is 0.8 GFLOP, 5 us at the FP32
// matrix rate.  One product per launch left a weight gradient - 152 result tiles, contraction over the
// whole batch - to 152 waves of 1024 dependent steps each (93 us a product, eight of them), and one
// workgroup to the loss (87 us).  Measured for one iteration with Adam: 863 -> 42 us (24 for the tiles,
// 13.5 for the weight gradients, 6.5 for the shares under the profiler).
//
// Contraction order.  A lane feeds four consecutive K steps from one 16-byte read: in step j lane group
// g takes index 16 s + 4 g + j, in both operands.

#include "dg_internal.h"

namespace dgmi {

typedef float f4c __attribute__((ext_vector_type(4)));

namespace {

__device__ inline f4c mfma4(float a, float b, f4c c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

constexpr int MT = 16;            // samples per workgroup of the activation kernel
constexpr int M_THREADS = 512;    // 8 waves, one 16-feature tile each in turn
constexpr int M_WAVES = M_THREADS / 64;

__host__ __device__ inline int pad16(int n) { return (n + 15) & ~15; }
// LDS row of one sample's layer of n features: whole K groups, and an offset that spreads the samples
// over the banks
__host__ __device__ inline int lds_ld(int n) { return pad16(n) + 4; }
__host__ __device__ inline int mlp_lds_floats(const MlpArgs &a) {
    return MT * (lds_ld(a.nin) + lds_ld(a.h1) + 2 * lds_ld(a.h2) + lds_ld(a.no));
}

// acc += W[row][k] X[col][k] over k < K; V: 16-byte reads.  Rows past the last one repeat row 0 and are
// dropped by the caller.  No load of a whole step is conditional, so the loads of several are in flight
// together.  The last step of a K that is no multiple of 16 is requested first; past the row's end it
// takes zeros, not weights that would meet zeros in LDS (one of them may be infinite).
template <bool V>
__device__ inline f4c rows_product(const float *W, int ldw, int row, int rows, int K, const float *xs, int ldx) {
    const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    const float *w = W + (size_t)(row < rows ? row : 0) * ldw + 4 * g;
    const float *x = xs + col * ldx + 4 * g;
    const int whole = K & ~15, rest = K - whole - 4 * g;  // rest: this lane's weights in the last step
    f4c acc = f4c{0, 0, 0, 0}, tail = acc;
    if (whole < K) {
        if (V) {
            if (rest > 0) tail = *reinterpret_cast<const f4c *>(w + whole);  // K is a multiple of 4 here
        } else {
#pragma unroll
            for (int j = 0; j < 4; j++)
                if (j < rest) tail[j] = w[whole + j];
        }
    }
#pragma unroll 8
    for (int s = 0; s < whole; s += 16) {
        f4c av;
        if (V) {
            av = *reinterpret_cast<const f4c *>(w + s);
        } else {
#pragma unroll
            for (int j = 0; j < 4; j++) av[j] = w[s + j];
        }
        const f4c bv = *reinterpret_cast<const f4c *>(x + s);
#pragma unroll
        for (int j = 0; j < 4; j++) acc = mfma4(av[j], bv[j], acc);
    }
    if (whole < K) {
        const f4c bv = *reinterpret_cast<const f4c *>(x + whole);
#pragma unroll
        for (int j = 0; j < 4; j++) acc = mfma4(tail[j], bv[j], acc);
    }
    return acc;
}

// entries m .. m + 3 of a vector of n (past its end: the last one)
__device__ inline f4c bias4(const float *b, int m, int n) {
    f4c v;
#pragma unroll
    for (int r = 0; r < 4; r++) v[r] = b[m + r < n ? m + r : n - 1];
    return v;
}

// acc += W[m][row] D[col][m] over m < K: the transposed weights (the last step as above)
__device__ inline f4c cols_product(const float *W, int ldw, int row, int rows, int K, const float *ds, int ldd) {
    const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    const float *w = W + (row < rows ? row : 0) + (size_t)(4 * g) * ldw;
    const float *d = ds + col * ldd + 4 * g;
    const int whole = K & ~15, rest = K - whole - 4 * g;
    f4c acc = f4c{0, 0, 0, 0}, tail = acc;
    if (whole < K) {
#pragma unroll
        for (int j = 0; j < 4; j++)
            if (j < rest) tail[j] = w[(size_t)(whole + j) * ldw];
    }
#pragma unroll 8
    for (int s = 0; s < whole; s += 16) {
        f4c av;
#pragma unroll
        for (int j = 0; j < 4; j++) av[j] = w[(size_t)(s + j) * ldw];
        const f4c bv = *reinterpret_cast<const f4c *>(d + s);
#pragma unroll
        for (int j = 0; j < 4; j++) acc = mfma4(av[j], bv[j], acc);
    }
    if (whole < K) {
        const f4c bv = *reinterpret_cast<const f4c *>(d + whole);
#pragma unroll
        for (int j = 0; j < 4; j++) acc = mfma4(tail[j], bv[j], acc);
    }
    return acc;
}

}  // namespace

// Activations and back-propagated signals of 16 samples: gather (and input noise), three layers forward,
// the squared error, two layers back, everything in LDS; what the weight gradients contract over goes
// to memory feature-major, [feature][bp], samples past the batch as zeros.  GRAD false: y only.
template <bool GRAD, bool V>
__global__ __launch_bounds__(M_THREADS) void mlp_tile_kernel(MlpArgs a) {
    extern __shared__ __attribute__((aligned(16))) float sm[];
    const int l0 = lds_ld(a.nin), l1 = lds_ld(a.h1), l2 = lds_ld(a.h2), lo = lds_ld(a.no);
    float *xs = sm, *h1s = xs + MT * l0, *h2s = h1s + MT * l1, *d2s = h2s + MT * l2, *dys = d2s + MT * l2;
    __shared__ double red[M_WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 15, g = lane >> 4;
    const int s0 = blockIdx.x * MT, smp = s0 + col;
    const bool live = smp < a.batch;
    const float *W1 = a.params, *b1 = W1 + (size_t)a.h1 * a.nin, *W2 = b1 + a.h1, *b2 = W2 + (size_t)a.h2 * a.h1;
    const float *W3 = b2 + a.h2, *b3 = W3 + (size_t)a.no * a.h2;
    const long long myrow = live ? (a.rows ? a.rows[smp] : smp) : 0;
    // wave w gathers samples w and w + 8, lanes along the features
#pragma unroll
    for (int s = wave; s < MT; s += M_WAVES) {
        const bool in = s0 + s < a.batch;
        const float *src = a.x + (in ? (a.rows ? a.rows[s0 + s] : s0 + s) : 0) * (long long)a.nin;
#pragma unroll 4
        for (int k = lane; k < l0; k += 64) {
            float v = src[k < a.nin ? k : 0];
            if (a.noise != 0.0f)
                v += a.noise * normal_draw(a.seed, (unsigned long long)((long long)k * a.batch + s0 + s));
            xs[s * l0 + k] = in && k < a.nin ? v : 0.0f;
        }
    }
    __syncthreads();
    // tile t of a layer's result: rows 16 t + 4 g + r of sample col
    for (int t = wave; t < pad16(a.h1) / 16; t += M_WAVES) {
        const f4c bias = bias4(b1, 16 * t + 4 * g, a.h1);
        f4c c = rows_product<V>(W1, a.nin, 16 * t + col, a.h1, a.nin, xs, l0);
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int m = 16 * t + 4 * g + r;
            c[r] = m < a.h1 ? tanhf(c[r] + bias[r]) : 0.0f;
            if (GRAD && m < a.h1) a.H1[(size_t)m * a.bp + smp] = live ? c[r] : 0.0f;
        }
        *reinterpret_cast<f4c *>(h1s + col * l1 + 16 * t + 4 * g) = c;
    }
    if (GRAD)
        for (int e = threadIdx.x; e < MT * a.nin; e += M_THREADS)
            a.X[(size_t)(e >> 4) * a.bp + s0 + (e & 15)] = xs[(e & 15) * l0 + (e >> 4)];
    __syncthreads();
    for (int t = wave; t < pad16(a.h2) / 16; t += M_WAVES) {
        const f4c bias = bias4(b2, 16 * t + 4 * g, a.h2);
        f4c c = rows_product<V>(W2, a.h1, 16 * t + col, a.h2, a.h1, h1s, l1);
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int m = 16 * t + 4 * g + r;
            c[r] = m < a.h2 ? tanhf(c[r] + bias[r]) : 0.0f;
            if (GRAD && m < a.h2) a.H2[(size_t)m * a.bp + smp] = live ? c[r] : 0.0f;
        }
        *reinterpret_cast<f4c *>(h2s + col * l2 + 16 * t + 4 * g) = c;
    }
    __syncthreads();
    double sq = 0.0;
    for (int t = wave; t < pad16(a.no) / 16; t += M_WAVES) {
        const f4c bias = bias4(b3, 16 * t + 4 * g, a.no);
        const f4c want = GRAD ? bias4(a.target + myrow * a.no, 16 * t + 4 * g, a.no) : bias;
        f4c c = rows_product<V>(W3, a.h2, 16 * t + col, a.no, a.h2, h2s, l2);
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int m = 16 * t + 4 * g + r;
            const float v = c[r] + bias[r];
            if (!GRAD) {
                if (m < a.no && live) a.y[(size_t)smp * a.no + m] = v;
                continue;
            }
            float d = 0.0f;
            if (m < a.no && live) {
                const float e = v - want[r];
                sq += (double)e * (double)e;
                d = a.dscale * e;
            }
            if (m < a.no) a.dY[(size_t)m * a.bp + smp] = d;
            c[r] = d;
        }
        if (GRAD) *reinterpret_cast<f4c *>(dys + col * lo + 16 * t + 4 * g) = c;
    }
    if (!GRAD) return;
    // this workgroup's sum of squares, in a fixed order
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) sq += __shfl_xor(sq, o, 64);
    if (lane == 0) red[wave] = sq;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = red[0];
        for (int w = 1; w < M_WAVES; w++) s += red[w];
        a.lpart[blockIdx.x] = s;
    }
    for (int t = wave; t < pad16(a.h2) / 16; t += M_WAVES) {
        f4c c = cols_product(W3, a.h2, 16 * t + col, a.h2, a.no, dys, lo);
        const f4c h = *reinterpret_cast<const f4c *>(h2s + col * l2 + 16 * t + 4 * g);
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int m = 16 * t + 4 * g + r;
            c[r] = live && m < a.h2 ? c[r] * (1.0f - h[r] * h[r]) : 0.0f;
            if (m < a.h2) a.D2[(size_t)m * a.bp + smp] = c[r];
        }
        *reinterpret_cast<f4c *>(d2s + col * l2 + 16 * t + 4 * g) = c;
    }
    __syncthreads();
    for (int t = wave; t < pad16(a.h1) / 16; t += M_WAVES) {
        f4c c = cols_product(W2, a.h1, 16 * t + col, a.h1, a.h2, d2s, l2);
        const f4c h = *reinterpret_cast<const f4c *>(h1s + col * l1 + 16 * t + 4 * g);
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int m = 16 * t + 4 * g + r;
            if (m < a.h1) a.D1[(size_t)m * a.bp + smp] = live ? c[r] * (1.0f - h[r] * h[r]) : 0.0f;
        }
    }
}

// Weight gradients D A^T of the three layers, and bias gradients (row sums of D, in FP64): a wave takes
// 16 rows by 64 columns of one of them over one of `nsplit` ranges of the batch; the shares go to
// part[split][param] and bpart[split][bias row].
constexpr int W_COLS = 4;  // 16-column tiles per wave: the rows of D it reads are used four times

__global__ __launch_bounds__(256) void mlp_wgrad_kernel(MlpArgs a) {
    const int lane = threadIdx.x & 63, col = lane & 15, g = lane >> 4;
    const int n1 = pad16(a.h1) / 16 * ((a.nin + 63) / 64), n2 = pad16(a.h2) / 16 * ((a.h1 + 63) / 64);
    const int n3 = pad16(a.no) / 16 * ((a.h2 + 63) / 64);
    int task = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int split = task / (n1 + n2 + n3);
    if (split >= a.nsplit) return;
    task -= split * (n1 + n2 + n3);
    const float *D, *A;
    int M, N;
    size_t off;  // first weight of the layer among the parameters
    int brow;    // first bias row of the layer in bpart
    const size_t o2 = (size_t)a.h1 * a.nin + a.h1, o4 = o2 + (size_t)a.h2 * a.h1 + a.h2;
    if (task < n1) {
        D = a.D1; A = a.X; M = a.h1; N = a.nin; off = 0; brow = 0;
    } else if (task < n1 + n2) {
        task -= n1;
        D = a.D2; A = a.H1; M = a.h2; N = a.h1; off = o2; brow = a.h1;
    } else {
        task -= n1 + n2;
        D = a.dY; A = a.H2; M = a.no; N = a.h2; off = o4; brow = a.h1 + a.h2;
    }
    const int nc = (N + 63) / 64, tm = task / nc, tn = task - tm * nc;
    const int row = 16 * tm + col;
    const float *d = D + (size_t)(row < M ? row : M - 1) * a.bp + 4 * g;
    const float *b[W_COLS];
#pragma unroll
    for (int c = 0; c < W_COLS; c++) {
        const int k = 64 * tn + 16 * c + col;
        b[c] = A + (size_t)(k < N ? k : N - 1) * a.bp + 4 * g;
    }
    const int lo = split * a.schunk, hi = lo + a.schunk < a.bp ? lo + a.schunk : a.bp;
    f4c acc[W_COLS];
#pragma unroll
    for (int c = 0; c < W_COLS; c++) acc[c] = f4c{0, 0, 0, 0};
    double bs = 0.0;
#pragma unroll 4
    for (int s = lo; s < hi; s += 16) {
        const f4c dv = *reinterpret_cast<const f4c *>(d + s);
        f4c bv[W_COLS];
#pragma unroll
        for (int c = 0; c < W_COLS; c++) bv[c] = *reinterpret_cast<const f4c *>(b[c] + s);
        if (tn == 0) bs += ((double)dv[0] + (double)dv[1]) + ((double)dv[2] + (double)dv[3]);
#pragma unroll
        for (int j = 0; j < 4; j++)
#pragma unroll
            for (int c = 0; c < W_COLS; c++) acc[c] = mfma4(dv[j], bv[c][j], acc[c]);
    }
    float *p = a.part + (size_t)split * a.nparams + off;
#pragma unroll
    for (int c = 0; c < W_COLS; c++) {
        const int k = 64 * tn + 16 * c + col;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int m = 16 * tm + 4 * g + r;
            if (m < M && k < N) p[(size_t)m * N + k] = acc[c][r];
        }
    }
    if (tn == 0) {
        bs += __shfl_xor(bs, 16, 64);
        bs += __shfl_xor(bs, 32, 64);
        if (g == 0 && row < M) a.bpart[(size_t)split * (a.h1 + a.h2 + a.no) + brow + row] = bs;
    }
}

// grad = the shares in split order (FP64 sums); the loss from the tiles' sums by the last workgroup
__global__ __launch_bounds__(256) void mlp_reduce_kernel(MlpArgs a) {
    if (blockIdx.x == gridDim.x - 1) {
        if (!a.loss) return;
        __shared__ double red[256];
        double s = 0.0;
        const int nt = (a.batch + MT - 1) / MT;
        for (int j = threadIdx.x; j < nt; j += 256) s += a.lpart[j];
        red[threadIdx.x] = s;
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
            __syncthreads();
        }
        if (threadIdx.x == 0) *a.loss = red[0] / ((double)a.batch * a.no);
        return;
    }
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= a.nparams) return;
    const long long o1 = (long long)a.h1 * a.nin, o2 = o1 + a.h1, o3 = o2 + (long long)a.h2 * a.h1, o4 = o3 + a.h2,
                    o5 = o4 + (long long)a.no * a.h2;
    const int nb = a.h1 + a.h2 + a.no;
    const int brow = i >= o5 ? (int)(i - o5) + a.h1 + a.h2 : i >= o3 && i < o4 ? (int)(i - o3) + a.h1
                     : i >= o1 && i < o2 ? (int)(i - o1) : -1;
    double s = 0.0;
    for (int sp = 0; sp < a.nsplit; sp++)
        s += brow >= 0 ? a.bpart[(size_t)sp * nb + brow] : (double)a.part[(size_t)sp * a.nparams + i];
    a.grad[i] = (float)s;
}

bool mlp_fused_fits(const int32_t sh[4]) {
    MlpArgs a{};
    a.nin = sh[0];
    a.h1 = sh[1];
    a.h2 = sh[2];
    a.no = sh[3];
    return mlp_lds_floats(a) * (int)sizeof(float) <= 64 * 1024 - 256;
}

// Ranges of the batch that the weight gradients are split into: 256 samples each, 32 at most.  A range
// shorter than that leaves a wave fewer products than its first loads cost; a longer one leaves compute
// units idle (4096 samples: 16 ranges x 44 waves of 140-128-128-20).
static int mlp_splits(int bp) {
    const int s = (bp + 255) / 256;
    return s < 32 ? s : 32;
}

size_t mlp_fused_bytes(const int32_t sh[4], int batch) {
    const size_t bp = pad16(batch), np = dg_mlp_nparams(sh);
    const size_t f = bp * ((size_t)sh[0] + 2 * (size_t)sh[1] + 2 * (size_t)sh[2] + sh[3]) + mlp_splits((int)bp) * ((np + 3) & ~(size_t)3);
    const size_t d = mlp_splits((int)bp) * ((size_t)sh[1] + sh[2] + sh[3]) + bp / MT;
    return f * sizeof(float) + d * sizeof(double) + 64;
}

void mlp_fused_carve(MlpArgs &a, void *work) {
    a.bp = pad16(a.batch);
    a.nsplit = mlp_splits(a.bp);
    a.schunk = ((a.bp / 16 + a.nsplit - 1) / a.nsplit) * 16;
    char *w = reinterpret_cast<char *>((reinterpret_cast<uintptr_t>(work) + 15) & ~(uintptr_t)15);
    double *d = reinterpret_cast<double *>(w);
    a.bpart = d;
    d += (size_t)a.nsplit * (a.h1 + a.h2 + a.no);
    a.lpart = d;
    d += a.bp / MT;
    float *f = reinterpret_cast<float *>((reinterpret_cast<uintptr_t>(d) + 15) & ~(uintptr_t)15);
    a.X = f; f += (size_t)a.nin * a.bp;
    a.H1 = f; f += (size_t)a.h1 * a.bp;
    a.D1 = f; f += (size_t)a.h1 * a.bp;
    a.H2 = f; f += (size_t)a.h2 * a.bp;
    a.D2 = f; f += (size_t)a.h2 * a.bp;
    a.dY = f; f += (size_t)a.no * a.bp;
    a.part = f;
}

hipError_t launch_mlp_fused(const MlpArgs &a, bool grad, hipStream_t s) {
    const int nt = (a.batch + MT - 1) / MT, lds = mlp_lds_floats(a) * (int)sizeof(float);
    // 16-byte reads of the weights' rows: every row and matrix on a 16-byte boundary
    const bool v = (reinterpret_cast<uintptr_t>(a.params) & 15) == 0 && a.nin % 4 == 0 && a.h1 % 4 == 0 && a.h2 % 4 == 0;
    if (!grad) {
        if (v) hipLaunchKernelGGL((mlp_tile_kernel<false, true>), dim3(nt), dim3(M_THREADS), lds, s, a);
        else hipLaunchKernelGGL((mlp_tile_kernel<false, false>), dim3(nt), dim3(M_THREADS), lds, s, a);
        return hipGetLastError();
    }
    if (v) hipLaunchKernelGGL((mlp_tile_kernel<true, true>), dim3(nt), dim3(M_THREADS), lds, s, a);
    else hipLaunchKernelGGL((mlp_tile_kernel<true, false>), dim3(nt), dim3(M_THREADS), lds, s, a);
    const int tasks = pad16(a.h1) / 16 * ((a.nin + 63) / 64) + pad16(a.h2) / 16 * ((a.h1 + 63) / 64) +
                      pad16(a.no) / 16 * ((a.h2 + 63) / 64);
    hipLaunchKernelGGL(mlp_wgrad_kernel, dim3((tasks * a.nsplit + 3) / 4), dim3(256), 0, s, a);
    hipLaunchKernelGGL(mlp_reduce_kernel, dim3((unsigned)((a.nparams + 255) / 256 + 1)), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace dgmi
