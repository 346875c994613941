// Learned warm start: a node-wise MLP that predicts the (preconditioned)
// optimal dual of every node from the initial state, the disturbance path
// and the stage, trained on the GPU by the kernels below.  The paper
// warm-starts its solvers from a few iterations of an accelerated gradient
// method (Sec. III-F); the MLP takes that slot, and the solver's own
// residual decides whether its prediction or the cold start is used.
//
// Features of node i (stage t_i) of an instance with initial state x0:
//   [ x0, c_i / c_scale, (mean of c over the path root->i) / c_scale,
//     one-hot(t_i) ]                       (3 nx + N + 1 values; c_0 = 0)
// Network: din -> dh -> dh -> dout (= nx + nu), ReLU, FP32 weights and
// FP32 accumulation.  Parameters are one flat array
//   [W1 (din x dh), b1, W2 (dh x dh), b2, W3 (dh x dout), b3], row-major.
// Outputs map to the node's dual rows (leaves use the first nx; the root's
// state rows are zero because they carry infinite bounds).
#include <cmath>

#include "internal.h"

namespace stotree {

namespace {

typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int kKt = 16;      // reduction rows staged in LDS at a time
constexpr int kGB = 256;     // threads per GEMM block: four wavefronts
constexpr int kLossThreads = 1024;   // threads per block of the loss passes

// C[m][n] = sum_k opA(m,k) opB(k,n) over k in [k0, k1), with
// opA(m,k) = TA ? A[k*lda+m] : A[m*lda+k], opB(k,n) = TB ? B[n*ldb+k] : B[k*ldb+n],
// on the FP32 matrix cores (v_mfma_f32_32x32x2f32: FP32 products, FP32 sums).
// Epilogue: + bias[n]; ReLU; or multiplication by the gate (G[m][n] > 0).
// With kslice > 0, blockIdx.z selects a slice of kslice rows of the reduction
// (partial sums for the weight gradients, C advances by z*M*ldc) and csum, if
// given, receives the slice's column sums of B (the bias gradients).
//
// Mapping: a block of BM x BN outputs, WR x WC wavefronts, each (BM/WR) x
// (BN/WC) of them in 32 x 32 accumulators; the operands go through LDS in rows
// of the reduction (an odd stride, so neither the transposing stores nor the
// reads conflict) with the next rows' loads in flight during the products.
// Bounds: the forward products move 40-65 MB of activations each at a
// 65,536-row minibatch of the 128-unit network and run 11-14 us of matrix
// work; the vector-unit tiles that stood here ran at 11 TFLOP/s (forward 42 us
// a layer, weight gradients 98 us).
// Operands (lane l): A[l%32][l/32], B[l/32][l%32], D[8(e/4) + 4(l/32) + e%4][l%32], e < 16.
template <bool TA, bool TB, int BM, int BN, int WR, int WC>
__global__ void __launch_bounds__(kGB) gemm_kernel(int M, int N, int K, const float *__restrict__ A, int lda,
                                                 const float *__restrict__ B, int ldb, float *__restrict__ C,
                                                 int ldc, const float *__restrict__ bias, int relu,
                                                 const float *__restrict__ gate, int ldg, int kslice,
                                                 float *__restrict__ csum)
{
    static_assert(WR * WC * 64 == kGB, "four wavefronts");
    constexpr int TM = BM / WR / 32, TN = BN / WC / 32;
    constexpr int LA = BM * kKt / kGB, LB = BN * kKt / kGB;     // staged entries per thread
    __shared__ float As[kKt][BM + 1];
    __shared__ float Bs[kKt][BN + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
    const int wm = wave / WC * (BM / WR), wn = wave % WC * (BN / WC);
    int kbeg = 0, kend = K;
    if (kslice > 0) {
        kbeg = blockIdx.z * kslice;
        kend = min(K, kbeg + kslice);
        C += (long long)blockIdx.z * M * ldc;
    }
    // entry e of a tile: consecutive threads on consecutive addresses; entries
    // past the matrix read a valid one and become zero on their way to LDS, so
    // no load sits under a branch
    float ra[LA], rb[LB];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int q = 0; q < LA; ++q) {
            const int e = tid + kGB * q, kk = TA ? e / BM : e % kKt, mm = TA ? e % BM : e / kKt;
            const int m = min(m0 + mm, M - 1), k = min(k0 + kk, kend - 1);
            ra[q] = TA ? A[(long long)k * lda + m] : A[(long long)m * lda + k];
        }
#pragma unroll
        for (int q = 0; q < LB; ++q) {
            const int e = tid + kGB * q, kk = TB ? e % kKt : e / BN, nn = TB ? e / kKt : e % BN;
            const int n = min(n0 + nn, N - 1), k = min(k0 + kk, kend - 1);
            rb[q] = TB ? B[(long long)n * ldb + k] : B[(long long)k * ldb + n];
        }
    };
    v16f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    const bool sums = csum && blockIdx.y == 0 && tid < BN;
    float bsum = 0.0f;
    fetch(kbeg);
    for (int k0 = kbeg; k0 < kend; k0 += kKt) {
#pragma unroll
        for (int q = 0; q < LA; ++q) {
            const int e = tid + kGB * q, kk = TA ? e / BM : e % kKt, mm = TA ? e % BM : e / kKt;
            As[kk][mm] = m0 + mm < M && k0 + kk < kend ? ra[q] : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < LB; ++q) {
            const int e = tid + kGB * q, kk = TB ? e % kKt : e / BN, nn = TB ? e / kKt : e % BN;
            Bs[kk][nn] = n0 + nn < N && k0 + kk < kend ? rb[q] : 0.0f;
        }
        __syncthreads();
        if (k0 + kKt < kend) fetch(k0 + kKt);
#pragma unroll
        for (int kk = 0; kk < kKt; kk += 2) {
            const int k = kk + lane / 32, c = lane & 31;
            float a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) a[i] = As[k][wm + 32 * i + c];
#pragma unroll
            for (int j = 0; j < TN; ++j) b[j] = Bs[k][wn + 32 * j + c];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        if (sums)
#pragma unroll
            for (int kk = 0; kk < kKt; ++kk) bsum += Bs[kk][tid];
        __syncthreads();
    }
    if (sums && n0 + tid < N) csum[(long long)blockIdx.z * N + n0 + tid] = bsum;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int n = n0 + wn + 32 * j + (lane & 31);
        if (n >= N) continue;
        const float bn = bias ? bias[n] : 0.0f;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int m = m0 + wm + 32 * i + 8 * (e / 4) + 4 * (lane / 32) + e % 4;
                if (m >= M) continue;
                float v = acc[i][j][e];
                if (bias) v += bn;
                if (relu) v = fmaxf(v, 0.0f);
                if (gate && !(gate[(long long)m * ldg + n] > 0.0f)) v = 0.0f;
                C[(long long)m * ldc + n] = v;
            }
    }
}

// out[j] = sum_s part[s*n + j] in double, in a fixed order: 16 threads per
// output take every 16th slice, then their sums are added pairwise.  A second
// pair of arrays (the bias gradient's) rides along: outputs n .. n + n2.
// (One thread per output walked its 128 slices one load at a time: 30 us.)
__global__ void __launch_bounds__(256) sum_rows_kernel(const float *part, int S, int n, float *out,
                                                       const float *part2, int n2, float *out2)
{
    const int j = blockIdx.x * 16 + (threadIdx.x & 15), g = threadIdx.x >> 4;
    const bool second = j >= n;
    const int jj = second ? j - n : j, nn = second ? n2 : n;
    const float *p = second ? part2 : part;
    double s = 0.0;
    if (j < n + n2)
        for (int k = g; k < S; k += 16) s += p[(long long)k * nn + jj];
    __shared__ double red[16][17];
    red[g][threadIdx.x & 15] = s;
    __syncthreads();
    for (int h = 8; h > 0; h >>= 1) {
        if (g < h) red[g][threadIdx.x & 15] += red[g + h][threadIdx.x & 15];
        __syncthreads();
    }
    if (g == 0 && j < n + n2) (second ? out2 : out)[jj] = (float)red[0][threadIdx.x];
}

// Loss 1/count sum mask (Y - T)^2 and its gradient dY = 2 mask (Y - T)/count.
// Per-block partial sums of the loss and of the mask go to part[2*block].
// Device-side count of the mask: per-block sums (fixed order) into part; every
// block of the gradient pass adds them up.
__global__ void __launch_bounds__(kLossThreads) mask_count_kernel(long long n, const float *mask, double *part)
{
    __shared__ double red[kLossThreads];
    double c = 0.0;
    for (long long k = blockIdx.x * (long long)blockDim.x + threadIdx.x; k < n;
         k += (long long)gridDim.x * blockDim.x)
        c += mask[k];
    red[threadIdx.x] = c;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// Sum of part[stride*k], k < nb <= 256, by a block of at least 256 threads (fixed
// order), in every thread.
__device__ __forceinline__ double block_sum(const double *part, int nb, int stride, double *red)
{
    if (threadIdx.x < 256) red[threadIdx.x] = (int)threadIdx.x < nb ? part[stride * threadIdx.x] : 0.0;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    const double v = red[0];
    __syncthreads();
    return v;
}

// counts: per-block counts of mask_count_kernel (each block adds them up and
// takes 1 / max(1, sum)), or null (inv_count given)
__global__ void __launch_bounds__(kLossThreads) mse_grad_kernel(long long n, const float *Y, const float *T, const float *mask,
                                                       float inv_count, const double *counts, int ncounts, float *dY,
                                                       double *part)
{
    __shared__ double red[2][kLossThreads];
    double l = 0.0, c = 0.0;
    float inv = inv_count;
    if (counts) {
        const double t = block_sum(counts, ncounts, 1, red[0]);
        inv = (float)(1.0 / (t > 1.0 ? t : 1.0));
    }
    for (long long k = blockIdx.x * (long long)blockDim.x + threadIdx.x; k < n;
         k += (long long)gridDim.x * blockDim.x) {
        const float d = Y[k] - T[k];
        const float w = mask[k];
        dY[k] = 2.0f * w * d * inv;
        l += (double)w * d * d;
        c += w;
    }
    red[0][threadIdx.x] = l;
    red[1][threadIdx.x] = c;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            red[0][threadIdx.x] += red[0][threadIdx.x + s];
            red[1][threadIdx.x] += red[1][threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = red[0][0];
        part[2 * blockIdx.x + 1] = red[1][0];
    }
}

__global__ void __launch_bounds__(256) sum_pairs_kernel(const double *part, int nb, double *out)
{
    __shared__ double red[256];
    const double l = block_sum(part, nb, 2, red), c = block_sum(part + 1, nb, 2, red);
    if (threadIdx.x == 0) {
        out[0] = l;
        out[1] = c;
    }
}

// Adam (Kingma and Ba 2015) with bias correction.
__global__ void adam_kernel(long long n, float *p, const float *g, float *m, float *v, float lr, float b1, float b2,
                            float eps, float c1, float c2)
{
    for (long long k = blockIdx.x * (long long)blockDim.x + threadIdx.x; k < n;
         k += (long long)gridDim.x * blockDim.x) {
        const float gk = g[k];
        const float mk = b1 * m[k] + (1.0f - b1) * gk;
        const float vk = b2 * v[k] + (1.0f - b2) * gk * gk;
        m[k] = mk;
        v[k] = vk;
        p[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
    }
}

struct WarmArgs {
    const InstDesc *inst;
    const int *anc;
    const double *cvec, *x0;
    int din, dout;
    float c_scale;
};

// The node passes run every instance in one launch (blockIdx.y; ninst of
// them), its rows starting at its first node; per instance a launch took 3-8 us
// for 1-3 us of work.  Ix: type of an element index inside an instance, 32 bits
// where they suffice (the divisions are several times cheaper).

// One thread per (node, state entry): its x0, c and path-mean features and
// every nx-th entry of the one-hot stage.  (The walk to the root is a chain of
// dependent loads; a thread per feature put it into almost every wavefront
// for a quarter of its lanes.)
template <typename Ix>
__global__ void features_kernel(WarmArgs a, int ninst, float *X)
{
    for (int b = blockIdx.y; b < ninst; b += gridDim.y) {
        const InstDesc I = a.inst[b];
        const int *anc = a.anc + I.sc;  // node-indexed pools share the sc offset
        const double *cv = a.cvec + I.c;
        const Ix total = (Ix)I.V * I.nx;
        float *Xb = X + I.node0 * a.din;
        for (Ix e = (Ix)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (Ix)gridDim.x * blockDim.x) {
            const int i = (int)(e / I.nx), col = (int)(e - (Ix)i * I.nx);
            float *x = Xb + (long long)i * a.din;
            double s = 0.0;
            int t = 0;                   // the stage: edges on the path to the root
            for (int j = i; j > 0; j = anc[j], ++t) s += cv[(long long)j * I.nx + col];
            x[col] = (float)a.x0[I.x0 + col];
            x[I.nx + col] = (float)(cv[e] / a.c_scale);
            x[2 * I.nx + col] = t > 0 ? (float)(s / t / a.c_scale) : 0.0f;
            for (int f = col; f <= I.N; f += I.nx) x[3 * I.nx + f] = f == t ? 1.0f : 0.0f;
        }
    }
}

// Y rows (scaled by y_scale) -> dual vector (root state rows 0), and the
// inverse map dual -> target rows with a mask of the rows that exist.
template <typename Ix>
__global__ void scatter_kernel(WarmArgs a, int ninst, const float *Y, double *y, float y_scale)
{
    for (int b = blockIdx.y; b < ninst; b += gridDim.y) {
        const InstDesc I = a.inst[b];
        const Ix W = I.nx + I.nu, nl = (Ix)I.Vnl * W, m = (Ix)I.m;
        const float *Yb = Y + I.node0 * a.dout;
        for (Ix k = (Ix)blockIdx.x * blockDim.x + threadIdx.x; k < m; k += (Ix)gridDim.x * blockDim.x) {
            Ix i, col;
            if (k < nl) { i = k / W; col = k - i * W; }
            else { i = (k - nl) / I.nx; col = k - nl - i * I.nx; i += I.Vnl; }
            const double v = (i == 0 && (int)col < I.nx) ? 0.0 : (double)Yb[(long long)i * a.dout + col] * y_scale;
            y[I.y + k] = v;
        }
    }
}

template <typename Ix>
__global__ void targets_kernel(WarmArgs a, int ninst, const double *y, float *T, float *mask, float inv_scale)
{
    for (int b = blockIdx.y; b < ninst; b += gridDim.y) {
        const InstDesc I = a.inst[b];
        const Ix total = (Ix)I.V * a.dout;
        float *Tb = T + I.node0 * a.dout, *Mb = mask + I.node0 * a.dout;
        for (Ix e = (Ix)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (Ix)gridDim.x * blockDim.x) {
            const int i = (int)(e / a.dout), col = (int)(e - (Ix)i * a.dout);
            const int w = i < I.Vnl ? I.nx + I.nu : I.nx;
            float t = 0.0f, mk = 0.0f;
            if (col < w && !(i == 0 && col < I.nx)) {
                const long long o = i < I.Vnl ? (long long)i * (I.nx + I.nu) : (long long)I.Vnl * I.nu + (long long)i * I.nx;
                t = (float)(y[I.y + o + col] * inv_scale);
                mk = 1.0f;
            }
            Tb[e] = t;
            Mb[e] = mk;
        }
    }
}

template <bool TA, bool TB, int BM, int BN, int WR, int WC>
void launch_tile(int M, int N, int K, const float *A, int lda, const float *B, int ldb, float *C, int ldc,
                 const float *bias, int relu, const float *gate, int ldg, int kslice, int nslices, float *csum,
                 hipStream_t st)
{
    const dim3 grid((N + BN - 1) / BN, (M + BM - 1) / BM, nslices);
    hipLaunchKernelGGL((gemm_kernel<TA, TB, BM, BN, WR, WC>), grid, dim3(kGB), 0, st, M, N, K, A, lda, B, ldb, C,
                       ldc, bias, relu, gate, ldg, kslice, csum);
}

// Tiles of the row products (C has one row per node row): as wide as the
// columns, so that the activations are read once, and 128 rows tall for narrow
// outputs.  Wider outputs take 32 rows (64 for up to 64 columns) below 32,768 rows
// and 64 (128) from there, although 64 rows give every compute unit a block from
// 16,384 on: it takes two to hide the loads.  Network forward by 32 / by 64 rows:
// 128 units 35.5 / 38.3 us at 16,384 rows, 41.0 / 47.2 at 20,000, 46.1 / 48.3 at
// 32,767; 160 units 61.3 / 66.3 at 20,000, 85.4 / 79.1 at 32,767.
// A 65,536-row training step with the wide tile at 64 x 128: 296 us; 128 x 128
// (three wavefronts per SIMD) 325, 32 x 128 304, 64 x 64 297; 32 reduction rows
// at a time instead of 16: 328, 8: 348.
template <bool TB>
int launch_rows(int M, int N, int K, const float *A, int lda, const float *B, int ldb, float *C, int ldc,
                const float *bias, int relu, const float *gate, int ldg, hipStream_t st)
{
    const bool tall = M >= 128 * 256;
    if (N <= 32)
        launch_tile<false, TB, 128, 32, 4, 1>(M, N, K, A, lda, B, ldb, C, ldc, bias, relu, gate, ldg, 0, 1, nullptr, st);
    else if (N <= 64 && tall)
        launch_tile<false, TB, 128, 64, 2, 2>(M, N, K, A, lda, B, ldb, C, ldc, bias, relu, gate, ldg, 0, 1, nullptr, st);
    else if (N <= 64)
        launch_tile<false, TB, 64, 64, 2, 2>(M, N, K, A, lda, B, ldb, C, ldc, bias, relu, gate, ldg, 0, 1, nullptr, st);
    else if (tall)
        launch_tile<false, TB, 64, 128, 1, 4>(M, N, K, A, lda, B, ldb, C, ldc, bias, relu, gate, ldg, 0, 1, nullptr, st);
    else
        launch_tile<false, TB, 32, 128, 1, 4>(M, N, K, A, lda, B, ldb, C, ldc, bias, relu, gate, ldg, 0, 1, nullptr, st);
    STOTREE_HIP(hipGetLastError());
    return STOTREE_OK;
}

struct Layout {
    long long W1, b1, W2, b2, W3, b3, n;
};

Layout layout(int din, int dh, int dout)
{
    Layout L;
    L.W1 = 0;
    L.b1 = L.W1 + (long long)din * dh;
    L.W2 = L.b1 + dh;
    L.b2 = L.W2 + (long long)dh * dh;
    L.W3 = L.b2 + dh;
    L.b3 = L.W3 + (long long)dh * dout;
    L.n = L.b3 + dout;
    return L;
}

// rows per slice of the weight-gradient reductions: a 65,536-row minibatch
// gives 128 slices, so a 128 x 128 weight gradient runs 512 workgroups
// (4,096-row slices left most of the chip idle: 64 workgroups, 0.75 ms each)
constexpr int kSliceRows = 512;

WarmArgs warm_args(const tree_factors *f, const double *x0, float c_scale)
{
    WarmArgs a{};
    a.inst = f->d_inst;
    a.anc = f->d_anc;
    a.cvec = f->cvec;
    a.x0 = x0;
    const InstDesc &I = f->inst[0];
    a.din = 3 * I.nx + I.N + 1;
    a.dout = I.nx + I.nu;
    a.c_scale = c_scale;
    return a;
}

int uniform_instances(const tree_factors *f, const char *who)
{
    for (const InstDesc &I : f->inst)
        if (I.nx != f->inst[0].nx || I.nu != f->inst[0].nu || I.N != f->inst[0].N) {
            set_error(std::string(who) + ": every instance needs the same nx, nu and N");
            return STOTREE_ERR_ARG;
        }
    return STOTREE_OK;
}

}  // namespace

long long mlp_param_count(int din, int dh, int dout) { return layout(din, dh, dout).n; }

int mlp_forward_impl(int rows, int din, int dh, int dout, const float *P, const float *X, float *H, float *Y,
                     hipStream_t st)
{
    const Layout L = layout(din, dh, dout);
    float *H1 = H, *H2 = H + (long long)rows * dh;
    int rc;
    if ((rc = launch_rows<false>(rows, dh, din, X, din, P + L.W1, dh, H1, dh, P + L.b1, 1, nullptr, 0, st)))
        return rc;
    if ((rc = launch_rows<false>(rows, dh, dh, H1, dh, P + L.W2, dh, H2, dh, P + L.b2, 1, nullptr, 0, st)))
        return rc;
    return launch_rows<false>(rows, dout, dh, H2, dh, P + L.W3, dout, Y, dout, P + L.b3, 0, nullptr, 0, st);
}

// (rows floats of it are spare: the length is part of the interface)
long long mlp_work_len(int rows, int din, int dh, int dout)
{
    const long long slices = (rows + kSliceRows - 1) / kSliceRows;
    const long long wmax = std::max<long long>((long long)din * dh, std::max<long long>((long long)dh * dh, (long long)dh * dout));
    return 2LL * rows * dh + slices * wmax + rows + slices * std::max(dh, dout);
}

namespace {
// dst[r][:] = src[idx[r]][:] for r < rows (cols floats per row)
template <typename Ix>
__global__ void gather_rows_kernel(long long rows, int cols, const float *src, long long src_rows,
                                   const long long *idx, float *dst, int *bad)
{
    const Ix total = (Ix)(rows * cols);
    for (Ix e = (Ix)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (Ix)gridDim.x * blockDim.x) {
        const Ix r = e / (Ix)cols;
        const int c = (int)(e - r * (Ix)cols);
        const long long s = idx[r];
        if (s < 0 || s >= src_rows) {   // an index outside the source: flagged, entry left as is
            *bad = 1;
            continue;
        }
        dst[e] = src[s * cols + c];
    }
}

// Gradient of one layer: G[W] = A' D and G[b] = column sums of D over the rows,
// in slices of kSliceRows rows (partial sums in part and partb), added up in a
// fixed order.
int layer_grad(int rows, int M, int N, const float *A, const float *D, float *part, float *partb, float *GW,
               float *Gb, hipStream_t st)
{
    const int slices = (rows + kSliceRows - 1) / kSliceRows;
    launch_tile<true, false, 64, 64, 2, 2>(M, N, rows, A, M, D, N, part, N, nullptr, 0, nullptr, 0, kSliceRows, slices,
                                           partb, st);
    hipLaunchKernelGGL(sum_rows_kernel, dim3((M * N + N + 15) / 16), dim3(256), 0, st, part, slices, M * N, GW, partb,
                       N, Gb);
    STOTREE_HIP(hipGetLastError());
    return STOTREE_OK;
}
}  // namespace

int mlp_backward_impl(int rows, int din, int dh, int dout, const float *P, const float *X, const float *H,
                      const float *dY, float *G, float *work, hipStream_t st)
{
    const Layout L = layout(din, dh, dout);
    const float *H1 = H, *H2 = H + (long long)rows * dh;
    float *dH2 = work, *dH1 = work + (long long)rows * dh, *part = work + 2LL * rows * dh;
    const int slices = (rows + kSliceRows - 1) / kSliceRows;
    const long long wmax = std::max<long long>((long long)din * dh, std::max<long long>((long long)dh * dh, (long long)dh * dout));
    float *partb = part + (long long)slices * wmax;
    int rc;
    // layer 3
    if ((rc = layer_grad(rows, dh, dout, H2, dY, part, partb, G + L.W3, G + L.b3, st))) return rc;
    if ((rc = launch_rows<true>(rows, dh, dout, dY, dout, P + L.W3, dout, dH2, dh, nullptr, 0, H2, dh, st))) return rc;
    // layer 2
    if ((rc = layer_grad(rows, dh, dh, H1, dH2, part, partb, G + L.W2, G + L.b2, st))) return rc;
    if ((rc = launch_rows<true>(rows, dh, dh, dH2, dh, P + L.W2, dh, dH1, dh, nullptr, 0, H1, dh, st))) return rc;
    // layer 1
    return layer_grad(rows, din, dh, X, dH1, part, partb, G + L.W1, G + L.b1, st);
}

int mse_grad_impl(long long n, const float *Y, const float *T, const float *mask, float inv_count, float *dY,
                  double *loss2, double *part, hipStream_t st)
{
    // 170 blocks: the (loss, count) pairs fill 340 of the 512 scratch doubles;
    // with inv_count 0 the per-block counts fill the 170 after them
    const int nb = 170;
    double *counts = nullptr;
    if (inv_count == 0.0f) {
        counts = part + 2 * nb;
        hipLaunchKernelGGL(mask_count_kernel, dim3(nb), dim3(kLossThreads), 0, st, n, mask, counts);
    }
    hipLaunchKernelGGL(mse_grad_kernel, dim3(nb), dim3(kLossThreads), 0, st, n, Y, T, mask, inv_count, counts, nb, dY, part);
    hipLaunchKernelGGL(sum_pairs_kernel, dim3(1), dim3(256), 0, st, part, nb, loss2);
    STOTREE_HIP(hipGetLastError());
    return STOTREE_OK;
}

int gather_rows_impl(long long rows, int cols, const float *src, long long src_rows, const long long *idx,
                     float *dst, int *bad, hipStream_t st)
{
    const unsigned g = (unsigned)std::min<long long>(2048, (rows * cols + 255) / 256);
    if (rows * cols < 1LL << 31)
        hipLaunchKernelGGL(gather_rows_kernel<unsigned>, dim3(g), dim3(256), 0, st, rows, cols, src, src_rows, idx, dst, bad);
    else
        hipLaunchKernelGGL(gather_rows_kernel<unsigned long long>, dim3(g), dim3(256), 0, st, rows, cols, src, src_rows, idx,
                           dst, bad);
    STOTREE_HIP(hipGetLastError());
    return STOTREE_OK;
}

int adam_impl(long long n, float *p, const float *g, float *m, float *v, float lr, float b1, float b2, float eps,
              int step, hipStream_t st)
{
    const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
    hipLaunchKernelGGL(adam_kernel, dim3(512), dim3(256), 0, st, n, p, g, m, v, lr, b1, b2, eps, c1, c2);
    STOTREE_HIP(hipGetLastError());
    return STOTREE_OK;
}

namespace {
// Grid of a node pass: enough blocks of 256 for the largest instance's
// elements (at most 1024), a row of them per instance.
struct NodeGrid {
    dim3 grid;
    bool small;                      // 32-bit element indices
};
NodeGrid node_grid(const tree_factors *f, long long per_node)
{
    long long most = 1;
    for (const InstDesc &I : f->inst) most = std::max(most, (long long)I.V * per_node);
    return {dim3((unsigned)std::min<long long>(1024, (most + 255) / 256), (unsigned)std::min(f->ninst, 32768)),
            most < 1LL << 31};
}
}  // namespace

int warm_features_impl(const tree_factors *f, const double *x0, float c_scale, float *X, hipStream_t st)
{
    int rc = uniform_instances(f, "warm_features");
    if (rc) return rc;
    const WarmArgs a = warm_args(f, x0, c_scale);
    const NodeGrid g = node_grid(f, f->inst[0].nx);
    if (g.small) hipLaunchKernelGGL(features_kernel<unsigned>, g.grid, dim3(256), 0, st, a, f->ninst, X);
    else hipLaunchKernelGGL(features_kernel<unsigned long long>, g.grid, dim3(256), 0, st, a, f->ninst, X);
    STOTREE_HIP(hipGetLastError());
    return STOTREE_OK;
}

int warm_scatter_impl(const tree_factors *f, const float *Y, float y_scale, double *y, hipStream_t st)
{
    int rc = uniform_instances(f, "warm_scatter");
    if (rc) return rc;
    const WarmArgs a = warm_args(f, nullptr, 1.0f);
    const NodeGrid g = node_grid(f, a.dout);
    if (g.small) hipLaunchKernelGGL(scatter_kernel<unsigned>, g.grid, dim3(256), 0, st, a, f->ninst, Y, y, y_scale);
    else hipLaunchKernelGGL(scatter_kernel<unsigned long long>, g.grid, dim3(256), 0, st, a, f->ninst, Y, y, y_scale);
    STOTREE_HIP(hipGetLastError());
    return STOTREE_OK;
}

int warm_targets_impl(const tree_factors *f, const double *y, float y_scale, float *T, float *mask, hipStream_t st)
{
    int rc = uniform_instances(f, "warm_targets");
    if (rc) return rc;
    const WarmArgs a = warm_args(f, nullptr, 1.0f);
    const NodeGrid g = node_grid(f, a.dout);
    if (g.small) hipLaunchKernelGGL(targets_kernel<unsigned>, g.grid, dim3(256), 0, st, a, f->ninst, y, T, mask, 1.0f / y_scale);
    else hipLaunchKernelGGL(targets_kernel<unsigned long long>, g.grid, dim3(256), 0, st, a, f->ninst, y, T, mask, 1.0f / y_scale);
    STOTREE_HIP(hipGetLastError());
    return STOTREE_OK;
}

}  // namespace stotree
