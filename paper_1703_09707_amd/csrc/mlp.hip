// Learned surrogate: a three-layer network n_in -> h -> h -> n_out that
// predicts magnification histograms from lens parameters, for the
// parameter-space exploration of the Bayesian Monte Carlo analysis that
// motivates fast map generation (arXiv:1703.09707, Sec. 1).
//
// Weights are stored in BF16 (rounded from FP32 master copies that Adam
// updates); activations and accumulation are FP32.  GELU (erf form) follows
// the first two layers; the output is a softmax, trained with cross-entropy
// against shooter histograms.  Parameter layout (FP32, flat):
// W1[n_in][h], b1[h], W2[h][h], b2[h], W3[h][n_out], b3[n_out].
//
// Networks whose layers are at most kRowsMaxDim wide run in two kernels: one
// takes a few rows of the batch through every layer, the other forms all
// weight gradients (below).  For wider ones, one LDS-tiled FP32 GEMM on the
// matrix cores serves every product of the forward and backward passes; it
// computes C[M][N] = sum_k A(m, k) B(k, n)
// with A and B read directly or transposed, B in FP32 or BF16 (widened to
// FP32 exactly), and a fused epilogue.  The products are FP32 MFMAs
// (v_mfma_f32_16x16x4f32: FP32 operands and accumulation, so activations
// stay FP32).  All reductions run in a fixed order, so results are
// deterministic.
#include <cmath>
#include <limits>
#include <vector>

#include "raysh_ctx.h"

namespace {

// The wide networks' products: 32 x 32 tiles, so that a product of a few
// hundred rows still has a workgroup for every few compute units, and
// K-chunks of 64 to keep the chain of staging round trips short.
constexpr int BM = 32, BN = 32, BK = 64, kGemmThreads = 256;
constexpr int WT = BM / 32;   // 16 x 16 MFMA tiles per wave and dimension (the 4 waves take quarters)

typedef float floatx4 __attribute__((ext_vector_type(4)));

enum Epilogue {
    EPI_STORE = 0,       // C = acc
    EPI_BIAS_GELU = 1,   // Z = acc + bias (into C), H = gelu(Z) (into C2)
    EPI_GELU_GRAD = 2,   // C = acc * gelu'(aux)
    EPI_BIAS = 3         // C = acc + bias
};

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// Round to nearest, ties to even (finite inputs).
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    const uint32_t u = __float_as_uint(f);
    const uint32_t lsb = (u >> 16) & 1u;
    return (uint16_t)((u + 0x7FFFu + lsb) >> 16);
}

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }

__device__ __forceinline__ float gelu_grad(float z) {
    return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

template <bool A_T, bool B_T, bool B_BF16, int EPI>
__global__ __launch_bounds__(kGemmThreads) void gemm_kernel(const float *__restrict__ A, int lda,
                                                            const void *__restrict__ Bv, int ldb, int M,
                                                            int N, int K, float *__restrict__ C, int ldc,
                                                            const float *__restrict__ bias,
                                                            const float *__restrict__ aux,
                                                            float *__restrict__ C2) {
    __shared__ float As[BK][BM + 4];
    __shared__ float Bs[BK][BN + 4];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    const int wm = (wave / 2) * (BM / 2), wn = (wave % 2) * (BN / 2);   // the wave's quarter of the tile
    const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;

    floatx4 acc[WT][WT];
#pragma unroll
    for (int si = 0; si < WT; ++si)
#pragma unroll
        for (int sj = 0; sj < WT; ++sj) acc[si][sj] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    for (int k0 = 0; k0 < K; k0 += BK) {
        // stage A tile: BM x BK elements, 4 per thread
        for (int e = threadIdx.x; e < BM * BK; e += kGemmThreads) {
            const int mm = A_T ? e % BM : e / BK;
            const int kk = A_T ? e / BM : e % BK;
            const int m = m0 + mm, k = k0 + kk;
            float v = 0.0f;
            if (m < M && k < K) v = A_T ? A[(int64_t)k * lda + m] : A[(int64_t)m * lda + k];
            As[kk][mm] = v;
        }
        // stage B tile: BK x BN elements
        for (int e = threadIdx.x; e < BK * BN; e += kGemmThreads) {
            const int kk = B_T ? e % BK : e / BN;
            const int nn = B_T ? e / BK : e % BN;
            const int k = k0 + kk, n = n0 + nn;
            float v = 0.0f;
            if (k < K && n < N) {
                const int64_t o = B_T ? (int64_t)n * ldb + k : (int64_t)k * ldb + n;
                v = B_BF16 ? bf16_to_f32(((const uint16_t *)Bv)[o]) : ((const float *)Bv)[o];
            }
            Bs[kk][nn] = v;
        }
        __syncthreads();
        // each wave: a 32 x 32 quarter of the tile as 2 x 2 MFMA tiles of
        // 16 x 16, four steps of k = 4 per staged chunk.  Operands of
        // v_mfma_f32_16x16x4f32: lane l gives A(row l % 16, k l / 16) and
        // B(k l / 16, column l % 16).
#pragma unroll
        for (int kq = 0; kq < BK; kq += 4) {
            const int kk = kq + lane / 16;
            float a[WT], b[WT];
#pragma unroll
            for (int si = 0; si < WT; ++si) a[si] = As[kk][wm + si * 16 + lane % 16];
#pragma unroll
            for (int sj = 0; sj < WT; ++sj) b[sj] = Bs[kk][wn + sj * 16 + lane % 16];
#pragma unroll
            for (int si = 0; si < WT; ++si)
#pragma unroll
                for (int sj = 0; sj < WT; ++sj)
                    acc[si][sj] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[si], b[sj], acc[si][sj], 0, 0, 0);
        }
        __syncthreads();
    }
    // lane l holds rows 4 (l / 16) + r, column l % 16 of each 16 x 16 tile
#pragma unroll
    for (int si = 0; si < WT; ++si)
#pragma unroll
        for (int sj = 0; sj < WT; ++sj)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm + si * 16 + 4 * (lane / 16) + r;
                const int n = n0 + wn + sj * 16 + lane % 16;
                if (m >= M || n >= N) continue;
                const int64_t o = (int64_t)m * ldc + n;
                float v = acc[si][sj][r];
                if (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU) v += bias[n];
                if (EPI == EPI_GELU_GRAD) v *= gelu_grad(aux[o]);
                C[o] = v;
                if (EPI == EPI_BIAS_GELU) C2[o] = gelu(v);
            }
}

template <bool A_T, bool B_T, bool B_BF16, int EPI>
void gemm(hipStream_t s, const float *A, int lda, const void *B, int ldb, int M, int N, int K, float *C,
          int ldc, const float *bias = nullptr, const float *aux = nullptr, float *C2 = nullptr) {
    dim3 grid((N + BN - 1) / BN, (M + BM - 1) / BM);
    hipLaunchKernelGGL((gemm_kernel<A_T, B_T, B_BF16, EPI>), grid, dim3(kGemmThreads), 0, s, A, lda, B, ldb,
                       M, N, K, C, ldc, bias, aux, C2);
}

// Softmax over each row of Z (one wave per row), the row's cross-entropy
// against T, and dZ = (P - T) / B.
__global__ __launch_bounds__(64) void softmax_xent_kernel(const float *__restrict__ Z,
                                                          const float *__restrict__ T, int B, int N,
                                                          float *__restrict__ P, float *__restrict__ dZ,
                                                          float *__restrict__ row_loss) {
    const int b = blockIdx.x;
    const float *z = Z + (int64_t)b * N;
    float mx = -INFINITY;
    for (int j = threadIdx.x; j < N; j += 64) mx = fmaxf(mx, z[j]);
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    float se = 0.0f;
    for (int j = threadIdx.x; j < N; j += 64) se += expf(z[j] - mx);
    for (int off = 32; off > 0; off >>= 1) se += __shfl_xor(se, off, 64);
    const float lse = logf(se);
    float l = 0.0f;
    for (int j = threadIdx.x; j < N; j += 64) {
        const float logp = z[j] - mx - lse;
        const float p = expf(logp);
        if (P) P[(int64_t)b * N + j] = p;
        if (T) {
            const float t = T[(int64_t)b * N + j];
            l -= t * logp;
            if (dZ) dZ[(int64_t)b * N + j] = (p - t) / (float)B;
        }
    }
    for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
    if (row_loss && threadIdx.x == 0) row_loss[b] = l;
}

// out[n] = sum_b X[b][n] in a fixed order: a workgroup takes kSumCols
// columns; thread (column c, group r) sums rows r, r + kSumGroups, ... in
// order, and the groups' partial sums are then added in order of r.
constexpr int kSumCols = 16, kSumGroups = 16;

__global__ __launch_bounds__(kSumCols * kSumGroups) void column_sum_kernel(const float *__restrict__ X, int B,
                                                                           int N, float *__restrict__ out) {
    __shared__ float part[kSumGroups][kSumCols + 1];
    const int c = threadIdx.x % kSumCols, r = threadIdx.x / kSumCols;
    const int n = blockIdx.x * kSumCols + c;
    float s = 0.0f;
    if (n < N)
        for (int b = r; b < B; b += kSumGroups) s += X[(int64_t)b * N + n];
    part[r][c] = s;
    __syncthreads();
    if (r == 0 && n < N) {
        float t = 0.0f;
        for (int g = 0; g < kSumGroups; ++g) t += part[g][c];
        out[n] = t;
    }
}

// Mean of row losses (one workgroup, fixed order).
__global__ void mean_loss_kernel(const float *__restrict__ row_loss, int B, float *__restrict__ loss) {
    __shared__ float part[256];
    float s = 0.0f;
    for (int b = threadIdx.x; b < B; b += 256) s += row_loss[b];
    part[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.0f;
        for (int i = 0; i < 256; ++i) t += part[i];
        *loss = t / (float)B;
    }
}

// Adam on FP32 masters; the BF16 copies of the weight entries are refreshed.
// at_a and at_b give each parameter's place in the two BF16 layouts (-1:
// none; at_b may be NULL).
__global__ void adam_kernel(float *__restrict__ master, uint16_t *__restrict__ w16, const int32_t *__restrict__ at_a,
                            uint16_t *__restrict__ w16b, const int32_t *__restrict__ at_b,
                            const float *__restrict__ g, float *__restrict__ m, float *__restrict__ v,
                            int64_t n, float lr, float b1, float b2, float eps, float bc1, float bc2) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float p = master[i] - lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
    master[i] = p;
    const int32_t a = at_a[i], b = at_b ? at_b[i] : -1;
    if (a >= 0) w16[a] = f32_to_bf16(p);
    if (b >= 0) w16b[b] = f32_to_bf16(p);
}

__global__ void to_bf16_kernel(const float *__restrict__ master, uint16_t *__restrict__ w16,
                               const int32_t *__restrict__ at_a, uint16_t *__restrict__ w16b,
                               const int32_t *__restrict__ at_b, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t a = at_a[i], b = at_b ? at_b[i] : -1;
    if (a >= 0) w16[a] = f32_to_bf16(master[i]);
    if (b >= 0) w16b[b] = f32_to_bf16(master[i]);
}

// ---- The whole network for a few rows in one workgroup.
//
// Rows of a batch are independent through every layer, forward and back, so
// one workgroup takes 4 RG rows through all of them with the activations in
// LDS: one launch where the layer-by-layer path takes four (forward) or six.
// At the sizes the network is used at, a product's time is its chain of
// dependent loads and the launch around it, not the matrix cores' rate.
//
// The products stay FP32 x BF16 with FP32 sums, on the BF16 matrix cores: an
// FP32 activation is split without remainder into three BF16 pieces (24 bits
// of significand in three times 8), whose products with a BF16 weight are
// exact in FP32.  v_mfma_f32_16x16x32_bf16 takes 16 rows: 4 rows of the batch
// in 4 slots each, the three pieces and a zero, so that 4 rows fill it; its
// result holds the pieces' sums in one lane's registers, and adding them
// gives the product.  Four rows a workgroup put 64 workgroups on a batch of
// 256, where 16 rows would leave 240 of 256 compute units idle.  The weights
// are read as they lie, 8 steps of k a lane in one 16-byte load
// ([k / 8][column][8]), each load a product or more ahead of its use: the
// stream of weights through the compute unit's vector cache (64 bytes a
// cycle, 160 KB forward) and the launch's own latencies bound the kernel.
// 4-256-256-64, per call: forward at batch 256 42.9 -> 8.9 us, at 4096 59 ->
// 12.5; gradient and Adam step at batch 256 152 -> 23.6 us, at 4096 1197 -> 67.
// The error against 64-bit arithmetic fell from 9e-7 to 3e-7 (forward) and
// from 3e-7 to 1.3e-7 (gradient): fewer roundings, in shorter chains.
// 16 waves are 5 % faster at batch 256 and 40 % slower at 4096 (one workgroup
// a compute unit).
constexpr int kRowWaves = 8, kRowThreads = 64 * kRowWaves;
constexpr int kRowAhead = 8;       // blocks of 32 steps whose weights are in flight
constexpr int kRowsMaxDim = 512;   // largest layer: 8 rows' activations and slopes take 96 KB of LDS
constexpr int kRowsFill = 512;     // workgroups above which a workgroup takes more rows

__host__ __device__ constexpr int pad_to(int n, int m) { return (n + m - 1) / m * m; }

// Place of weight (k, n) in the layout of a product with K steps and N columns.
inline int64_t row_layout_at(int k, int n, int N) { return ((int64_t)(k / 8) * pad_to(N, 16) + n) * 8 + k % 8; }
inline int64_t row_layout_size(int K, int N) { return (int64_t)pad_to(K, 32) * pad_to(N, 16); }

// The products in the order the kernel takes them: W1, W2, W3 and, in
// training, W3 and W2 transposed.
struct RowNet {
    int n_in, h, n_out;
    const uint16_t *W[5];
    int K[5], N[5];
    const float *b1, *b2, *b3;
    float *H[2];                    // [batch][h]: activations (training)
    float *dZ[3];                   // [batch][h], [batch][h], [batch][n_out] (training)
    float *row_loss;                // [batch] (training)
};

// A barrier for data in LDS only: loads from global memory stay in flight
// (the plain one waits for them, and with them for the next product's
// weights).
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Activations in LDS: [k / 8][RG][4 rows x 4 slots][8] BF16.
template <int RG>
__device__ __forceinline__ int act_at(int k, int g, int row) {
    return (((k / 8) * RG + g) * 16 + 4 * row) * 8 + k % 8;
}

// a split into three BF16 pieces with a = hi + mid + lo exactly, by
// truncation (each takes the next 8 bits); infinities and NaN stay in hi.
template <int RG>
__device__ __forceinline__ void act_store(uint16_t *act, int k, int g, int row, float a) {
    const uint32_t hi = __float_as_uint(a) & 0xFFFF0000u;
    const bool finite = (hi & 0x7F800000u) != 0x7F800000u;
    const float r1 = finite ? a - __uint_as_float(hi) : 0.0f;
    const uint32_t mid = __float_as_uint(r1) & 0xFFFF0000u;
    const float r2 = r1 - __uint_as_float(mid);
    uint16_t *d = act + act_at<RG>(k, g, row);
    d[0] = a != a ? 0x7FC0 : (uint16_t)(hi >> 16);
    d[8] = (uint16_t)(mid >> 16);
    d[16] = (uint16_t)(__float_as_uint(r2) >> 16);
}

// The weights a wave takes next: blocks of 32 steps of one tile of 16
// columns, n of them (past the last one the loads repeat it).
struct RowCursor {
    const uint4 *p;
    int n, stride;
};

__device__ __forceinline__ RowCursor row_cursor(const uint16_t *W, int K, int N, int tile, int kb) {
    const int lane = threadIdx.x % 64, Np = pad_to(N, 16);
    const int t = tile * 16 < Np ? tile : 0;   // a wave without a tile loads the first one, unused
    return RowCursor{(const uint4 *)W + (lane / 16 + 4 * kb) * Np + t * 16 + lane % 16, pad_to(K, 32) / 32 - kb,
                     4 * Np};
}

__device__ __forceinline__ uint4 row_load(const RowCursor &c, int u) { return c.p[(u < c.n ? u : c.n - 1) * c.stride]; }

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// One product for 4 RG rows: every tile of 16 columns of the wave's share
// (tile = wave, wave + kRowWaves, ...) summed over k and handed to
// done(g, n, z): lane l has column 16 tile + l % 16 of row l / 16 of group g.
// w holds the first kRowAhead blocks of the wave's first tile; a slot is
// loaded again as soon as it has been used, at the end of the share with the
// next product's first blocks (Wn, Kn, Nn).  The loads are outside every
// branch, so that they land in their registers without copies, which would
// wait for them.
template <int RG, class Done>
__device__ __forceinline__ void row_product(const uint16_t *act, const uint16_t *W, int K, int N,
                                            uint4 (&w)[kRowAhead], const uint16_t *Wn, int Kn, int Nn, Done done) {
    const int lane = threadIdx.x % 64, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int blocks = pad_to(K, 32) / 32, tiles = pad_to(N, 16) / 16;
    const uint16_t *row = act + ((lane / 16) * RG * 16 + lane % 16) * 8;   // the lane's operand at k = 0
    int tile = wave;
    do {
        const bool mine = tile < tiles;   // uniform; a wave without a tile only loads what comes next
        floatx4 acc[RG];
#pragma unroll
        for (int g = 0; g < RG; ++g) acc[g] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        int kb = 0;
        do {
            RowCursor from;
            if (mine && kb + kRowAhead < blocks) from = row_cursor(W, K, N, tile, kb + kRowAhead);
            else if (tile + kRowWaves < tiles) from = row_cursor(W, K, N, tile + kRowWaves, 0);
            else from = row_cursor(Wn, Kn, Nn, wave, 0);
#pragma unroll
            for (int u = 0; u < kRowAhead; ++u) {
                if (mine && kb + u < blocks) {
                    const bf16x8 b = __builtin_bit_cast(bf16x8, w[u]);
#pragma unroll
                    for (int g = 0; g < RG; ++g) {
                        const bf16x8 a = *(const bf16x8 *)(row + ((kb + u) * 4 * RG + g) * 16 * 8);
                        acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[g], 0, 0, 0);
                    }
                }
                w[u] = row_load(from, u);
            }
            kb += kRowAhead;
        } while (mine && kb < blocks);
        if (mine) {
#pragma unroll
            for (int g = 0; g < RG; ++g) done(g, 16 * tile + lane % 16, (acc[g][2] + acc[g][1]) + acc[g][0]);
        }
        tile += kRowWaves;
    } while (tile < tiles);
}

// Softmax of each row's logits (one wave a row, z is [4 RG][no]) into P; with
// TRAIN the cross-entropy against T, and dZ3 to act and dZ.
template <int RG, bool TRAIN>
__device__ __forceinline__ void row_softmax(const float *z_rows, int no, uint16_t *act, int row0, int B,
                                            const float *__restrict__ T, float *__restrict__ P,
                                            float *__restrict__ dZ, float *__restrict__ row_loss) {
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    for (int row = wave; row < 4 * RG; row += kRowWaves) {
        const int b = row0 + row;
        const float *z = z_rows + row * no;
        float mx = -INFINITY;
        for (int j = lane; j < no; j += 64) mx = fmaxf(mx, z[j]);
        for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
        float se = 0.0f;
        for (int j = lane; j < no; j += 64) se += expf(z[j] - mx);
        for (int off = 32; off > 0; off >>= 1) se += __shfl_xor(se, off, 64);
        const float lse = logf(se);
        float l = 0.0f;
        for (int j = lane; j < (TRAIN ? pad_to(no, 32) : no); j += 64) {   // act is zero up to the next product's K
            float d = 0.0f;
            if (j < no && b < B) {
                const float logp = z[j] - mx - lse;
                const float p = expf(logp);
                if (!TRAIN) {
                    P[(int64_t)b * no + j] = p;
                } else {
                    const float t = T[(int64_t)b * no + j];
                    l -= t * logp;
                    d = (p - t) / (float)B;
                    dZ[(int64_t)b * no + j] = d;
                }
            }
            if (TRAIN) act_store<RG>(act, j, row / 4, row % 4, d);
        }
        if (TRAIN) {
            for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
            if (lane == 0 && b < B) row_loss[b] = l;
        }
    }
}

// Forward pass of rows [4 RG block, ...) to softmax outputs P; with TRAIN the
// cross-entropy against T, and back to dZ3, dZ2 and dZ1 (the weight
// gradients' operands).  dim: the widest layer padded to 32.
template <int RG, bool TRAIN>
__global__ __launch_bounds__(kRowThreads) void mlp_rows_kernel(RowNet net, const float *__restrict__ x,
                                                               const float *__restrict__ T, int B, int dim,
                                                               float *__restrict__ P) {
    extern __shared__ __align__(16) uint16_t lds[];
    const int h = net.h, no = net.n_out, act_words = dim * RG * 16;
    // two sets of activations: a product reads one and its epilogue writes the
    // other (offsets into lds, not pointers: a chosen pointer would be a flat
    // one, whose loads wait for every load in flight)
    float *logits = (float *)(lds + 2 * act_words);      // [4 RG][no]
    float *bias = logits + 4 * RG * no;                  // b1, b2, b3
    float *slope = bias + 2 * h + no;                    // [2][4 RG][h]: GELU' (training)
    const int row0 = blockIdx.x * (4 * RG);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    uint4 w[kRowAhead];
    {
        const RowCursor c = row_cursor(net.W[0], net.K[0], net.N[0], wave, 0);
#pragma unroll
        for (int u = 0; u < kRowAhead; ++u) w[u] = row_load(c, u);
    }
    // the zero slots, and k past a layer's width: zero once.  What is written
    // there later (the input's columns beyond a narrower hidden layer) meets
    // the zeros that pad the weights' steps
    for (int e = threadIdx.x; e < 2 * act_words / 8; e += kRowThreads) ((uint4 *)lds)[e] = uint4{0, 0, 0, 0};
    for (int e = threadIdx.x; e < 2 * h + no; e += kRowThreads)
        bias[e] = e < h ? net.b1[e] : e < 2 * h ? net.b2[e - h] : net.b3[e - 2 * h];
    lds_barrier();
    for (int e = threadIdx.x; e < 4 * RG * net.n_in; e += kRowThreads) {
        const int row = e / net.n_in, k = e - row * net.n_in;
        if (row0 + row < B) act_store<RG>(lds, k, row / 4, row % 4, x[(int64_t)row0 * net.n_in + e]);
    }
    lds_barrier();
    const int lane_row = (threadIdx.x % 64) / 16;
    constexpr int kProducts = TRAIN ? 5 : 3;
#pragma unroll 1
    for (int l = 0; l < kProducts; ++l) {
        const int next = l + 1 < kProducts ? l + 1 : l;
        const int from = (l % 2) * act_words, to = ((l + 1) % 2) * act_words;
        row_product<RG>(lds + from, net.W[l], net.K[l], net.N[l], w, net.W[next], net.K[next], net.N[next],
                        [&](int g, int n, float z) {
                            const int row = 4 * g + lane_row, b = row0 + row;
                            if (l == 2) {
                                if (n < no) logits[row * no + n] = z + bias[2 * h + n];
                                return;
                            }
                            if (n >= h) return;
                            float a;
                            if (l < 2) {   // hidden layer: the activation, and its slope for the way back
                                z += bias[l * h + n];
                                a = gelu(z);
                                if (TRAIN) {
                                    slope[(l * 4 * RG + row) * h + n] = gelu_grad(z);
                                    if (b < B) net.H[l][(int64_t)b * h + n] = a;
                                }
                            } else {       // passed back: l = 3: dZ2, l = 4: dZ1
                                a = b < B ? z * slope[((4 - l) * 4 * RG + row) * h + n] : 0.0f;
                                if (b < B) net.dZ[4 - l][(int64_t)b * h + n] = a;
                            }
                            if (l < 4) act_store<RG>(lds + to, n, g, lane_row, a);
                        });
        lds_barrier();
        if (l == 2) {
            row_softmax<RG, TRAIN>(logits, no, lds + to, row0, B, T, P, net.dZ[2], net.row_loss);
            if (TRAIN) lds_barrier();
        }
    }
}

// Every weight and bias gradient, and the mean loss, in one launch.  A
// workgroup takes a 16 x 16 tile of one layer's gradient
// dW[m][n] = sum_b A[b][m] dZ[b][n] (336 workgroups for the 4-256-256-64
// network); its four waves share the batch in steps of 4 rows, so that a
// wave's chain is batch / 16 products, and their sums are added in order; the
// tiles of the first rows also add up their columns of dZ for the bias.  The
// last workgroup takes the mean loss.  Both operands are FP32, so these
// products stay on the FP32 MFMA.  Outputs go to the network's gradient and,
// if asked for, to the caller's copy.  4.5 us at batch 256, where three GEMMs,
// three column sums, the mean and a copy took 11-14, 3-6, 4 and 3 us each.
struct GradLayer {
    const float *A, *dZ;
    int M, N;
    int64_t w, b;   // offsets of the weight and bias gradients
    int tiles_n, first;
};

constexpr int kGradAhead = 8;   // steps whose loads are in flight

__global__ __launch_bounds__(256) void mlp_grad_kernel(GradLayer l1, GradLayer l2, GradLayer l3, int n_tiles, int B,
                                                       float *__restrict__ grad, float *__restrict__ out,
                                                       const float *__restrict__ row_loss,
                                                       float *__restrict__ loss) {
    __shared__ float part[4][16][17];
    __shared__ float col[4][64];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    if ((int)blockIdx.x == n_tiles) {   // the mean loss
        float *p = &part[0][0][0];
        float s = 0.0f;
        for (int b = threadIdx.x; b < B; b += 256) s += row_loss[b];
        p[threadIdx.x] = s;
        __syncthreads();
        if (threadIdx.x < 64) {
            float t = p[threadIdx.x] + p[threadIdx.x + 64] + p[threadIdx.x + 128] + p[threadIdx.x + 192];
            for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
            if (threadIdx.x == 0) *loss = t / (float)B;
        }
        return;
    }
    const GradLayer &L = (int)blockIdx.x >= l3.first ? l3 : (int)blockIdx.x >= l2.first ? l2 : l1;
    const int tile = blockIdx.x - L.first;
    const int m0 = (tile / L.tiles_n) * 16, n0 = (tile % L.tiles_n) * 16;
    // operands of v_mfma_f32_16x16x4f32: lane l gives A(row l % 16, k l / 16) and B(k l / 16, column l % 16)
    const int m = m0 + lane % 16, n = n0 + lane % 16, k = lane / 16;
    const bool in_m = m < L.M, in_n = n < L.N;
    const float *A = L.A + (in_m ? m : 0), *D = L.dZ + (in_n ? n : 0);
    floatx4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    float csum = 0.0f;
    const int steps = (B + 3) / 4;
    for (int s0 = wave; s0 < steps; s0 += 4 * kGradAhead) {
        float a[kGradAhead], d[kGradAhead];
#pragma unroll
        for (int u = 0; u < kGradAhead; ++u) {
            const int b = 4 * (s0 + 4 * u) + k;
            const bool in = b < B;
            const int64_t bb = in ? b : 0;
            const float av = A[bb * L.M], dv = D[bb * L.N];
            a[u] = in && in_m ? av : 0.0f;
            d[u] = in && in_n ? dv : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < kGradAhead; ++u) {
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u], d[u], acc, 0, 0, 0);
            csum += d[u];
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) part[wave][4 * k + r][lane % 16] = acc[r];
    col[wave][lane] = csum;
    __syncthreads();
    const int tm = threadIdx.x / 16, tn = threadIdx.x % 16;
    if (n0 + tn >= L.N) return;
    if (m0 + tm < L.M) {
        const float v = ((part[0][tm][tn] + part[1][tm][tn]) + part[2][tm][tn]) + part[3][tm][tn];
        const int64_t o = L.w + (int64_t)(m0 + tm) * L.N + n0 + tn;
        grad[o] = v;
        if (out) out[o] = v;
    }
    if (m0 == 0 && tm == 0) {
        float v = 0.0f;
        for (int w = 0; w < 4; ++w)
            for (int q = 0; q < 4; ++q) v += col[w][16 * q + tn];
        grad[L.b + n0 + tn] = v;
        if (out) out[L.b + n0 + tn] = v;
    }
}

}  // namespace

struct raysh_mlp {
    int device = 0;
    hipStream_t stream = nullptr;
    int n_in = 0, h = 0, n_out = 0, max_batch = 0;
    int64_t n_params = 0;
    int64_t off[6] = {};        // offsets of W1, b1, W2, b2, W3, b3 in the flat parameters
    int64_t woff[3] = {};       // offsets of W1, W2, W3 in w16
    int64_t roff[3] = {};       // offsets of W2, W3 in w16b (index 1 and 2)
    int64_t step = 0;
    float *master = nullptr, *grad = nullptr, *m = nullptr, *v = nullptr;
    bool by_rows = false;       // every layer within kRowsMaxDim: mlp_rows_kernel and mlp_grad_kernel
    // BF16 weights: by_rows, w16 in the row kernels' forward layout and w16b (W2, W3) in the transposed one;
    // otherwise w16 in the parameters' order and w16b unused.  at_a, at_b: flat parameter -> place in each, or -1.
    uint16_t *w16 = nullptr, *w16b = nullptr;
    int32_t *at_a = nullptr, *at_b = nullptr;
    float *Z1 = nullptr, *H1 = nullptr, *Z2 = nullptr, *H2 = nullptr, *Z3 = nullptr, *P = nullptr;
    float *dZ3 = nullptr, *dZ2 = nullptr, *dZ1 = nullptr, *row_loss = nullptr;
    bool has_grad = false;
    std::vector<void *> allocs;
};

namespace {

int mlp_alloc(raysh_mlp *p, void **ptr, size_t bytes) {
    hipError_t e = hipMalloc(ptr, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return set_error(RAYSH_ENOMEM, "raysh_mlp: device allocation of %zu bytes failed", bytes);
    }
    p->allocs.push_back(*ptr);
    return RAYSH_OK;
}

void mlp_release(raysh_mlp *p) {
    for (void *a : p->allocs) (void)hipFree(a);
    p->allocs.clear();
}

int check_batch(const raysh_mlp *p, int32_t batch) {
    if (batch < 1 || batch > p->max_batch)
        return set_error(RAYSH_EINVAL, "batch %d outside [1, %d]", batch, p->max_batch);
    return RAYSH_OK;
}

// Whether two of a call's buffers share memory.
bool overlap(const void *a, size_t a_bytes, const void *b, size_t b_bytes) {
    const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
    return a && b && x < y + b_bytes && y < x + a_bytes;
}

RowNet row_net(const raysh_mlp *p) {
    RowNet n{};
    n.n_in = p->n_in;
    n.h = p->h;
    n.n_out = p->n_out;
    for (int l = 0; l < 3; ++l) {
        n.W[l] = p->w16 + p->woff[l];
        n.K[l] = l == 0 ? p->n_in : p->h;
        n.N[l] = l == 2 ? p->n_out : p->h;
    }
    n.W[3] = p->w16b + p->roff[2];
    n.K[3] = p->n_out;
    n.N[3] = p->h;
    n.W[4] = p->w16b + p->roff[1];
    n.K[4] = n.N[4] = p->h;
    n.b1 = p->master + p->off[1];
    n.b2 = p->master + p->off[3];
    n.b3 = p->master + p->off[5];
    n.H[0] = p->H1;
    n.H[1] = p->H2;
    n.dZ[0] = p->dZ1;
    n.dZ[1] = p->dZ2;
    n.dZ[2] = p->dZ3;
    n.row_loss = p->row_loss;
    return n;
}

template <int RG, bool TRAIN>
void launch_rows(const raysh_mlp *p, const float *x, const float *target, int B, float *probs) {
    const int widest = p->n_in > p->h ? (p->n_in > p->n_out ? p->n_in : p->n_out) : (p->h > p->n_out ? p->h : p->n_out);
    const int dim = pad_to(widest, 32);
    // two sets of activations, the logits, the biases and, in training, two layers' slopes
    const size_t lds = 2 * sizeof(uint16_t) * dim * RG * 16 +
                       sizeof(float) * (4 * RG * p->n_out + 2 * p->h + p->n_out + (TRAIN ? 2 * 4 * RG * p->h : 0));
    hipLaunchKernelGGL((mlp_rows_kernel<RG, TRAIN>), dim3((B + 4 * RG - 1) / (4 * RG)), dim3(kRowThreads), lds,
                       p->stream, row_net(p), x, target, B, dim, probs);
}

// 4 rows a workgroup until there are two workgroups per compute unit, then 8:
// every workgroup reads all weights, so more rows share them once the device
// is full anyway.
template <bool TRAIN>
void forward_rows(const raysh_mlp *p, const float *x, const float *target, int B, float *probs) {
    if (B <= 4 * kRowsFill) launch_rows<1, TRAIN>(p, x, target, B, probs);
    else launch_rows<2, TRAIN>(p, x, target, B, probs);
}

// Forward pass into the context's activation buffers.
void forward(raysh_mlp *p, const float *x, int B) {
    hipStream_t s = p->stream;
    const float *b1 = p->master + p->off[1], *b2 = p->master + p->off[3], *b3 = p->master + p->off[5];
    gemm<false, false, true, EPI_BIAS_GELU>(s, x, p->n_in, p->w16 + p->woff[0], p->h, B, p->h, p->n_in, p->Z1,
                                            p->h, b1, nullptr, p->H1);
    gemm<false, false, true, EPI_BIAS_GELU>(s, p->H1, p->h, p->w16 + p->woff[1], p->h, B, p->h, p->h, p->Z2,
                                            p->h, b2, nullptr, p->H2);
    gemm<false, false, true, EPI_BIAS>(s, p->H2, p->h, p->w16 + p->woff[2], p->n_out, B, p->n_out, p->h,
                                       p->Z3, p->n_out, b3);
}

}  // namespace

extern "C" {

int raysh_mlp_create(raysh_mlp **out, int device, void *hip_stream, int32_t n_in, int32_t n_hidden,
                     int32_t n_out, int32_t max_batch, const float *params) {
    if (!out) return set_error(RAYSH_EINVAL, "out is NULL");
    if (n_in < 1 || n_hidden < 1 || n_out < 1 || max_batch < 1)
        return set_error(RAYSH_EINVAL, "layer sizes and max_batch must be >= 1");
    if (n_in > 4096 || n_hidden > 4096 || n_out > 4096 || max_batch > (1 << 20))
        return set_error(RAYSH_EINVAL, "layer sizes above 4096 or max_batch above 2^20");
    if (!params) return set_error(RAYSH_EINVAL, "params is NULL");
    const int64_t h = n_hidden;
    const int64_t sizes[6] = {(int64_t)n_in * h, h, h * h, h, h * n_out, n_out};
    int64_t total = 0;
    for (int64_t sz : sizes) total += sz;
    for (int64_t i = 0; i < total; ++i)
        if (!std::isfinite(params[i])) return set_error(RAYSH_EINVAL, "parameter %lld is not finite", (long long)i);
    if (device < 0) return set_error(RAYSH_EINVAL, "device < 0");
    DeviceGuard g(device);
    if (!g.ok) return set_error(RAYSH_EDEVICE, "hipSetDevice(%d) failed", device);

    raysh_mlp *p = new raysh_mlp();
    p->device = device;
    p->stream = (hipStream_t)hip_stream;
    p->n_in = n_in;
    p->h = n_hidden;
    p->n_out = n_out;
    p->max_batch = max_batch;
    p->n_params = total;
    int64_t o = 0;
    for (int i = 0; i < 6; ++i) {
        p->off[i] = o;
        o += sizes[i];
    }
    p->by_rows = n_in <= kRowsMaxDim && n_hidden <= kRowsMaxDim && n_out <= kRowsMaxDim;
    const int K[3] = {n_in, n_hidden, n_hidden}, N[3] = {n_hidden, n_hidden, n_out};
    int64_t na = 0, nb = 0;   // entries of w16 and w16b
    for (int l = 0; l < 3; ++l) {
        p->woff[l] = na;
        na += p->by_rows ? row_layout_size(K[l], N[l]) : (int64_t)K[l] * N[l];
        p->roff[l] = nb;
        if (p->by_rows && l > 0) nb += row_layout_size(N[l], K[l]);
    }
    std::vector<int32_t> at_a(total, -1), at_b(total, -1);
    for (int l = 0; l < 3; ++l)
        for (int k = 0; k < K[l]; ++k)
            for (int n = 0; n < N[l]; ++n) {
                const int64_t i = (int64_t)k * N[l] + n;
                at_a[p->off[2 * l] + i] =
                    (int32_t)(p->woff[l] + (p->by_rows ? row_layout_at(k, n, N[l]) : i));
                if (p->by_rows && l > 0)   // transposed: step n, column k
                    at_b[p->off[2 * l] + i] = (int32_t)(p->roff[l] + row_layout_at(n, k, K[l]));
            }

    const int64_t Bh = (int64_t)max_batch * h, Bo = (int64_t)max_batch * n_out;
    int r = RAYSH_OK;
    void *tmp = nullptr;
#define ALLOC(field, type, count)                                            \
    if (r == RAYSH_OK) {                                                     \
        r = mlp_alloc(p, &tmp, (size_t)(count) * sizeof(type));              \
        p->field = (type *)tmp;                                              \
    }
    ALLOC(master, float, total)
    ALLOC(grad, float, total)
    ALLOC(m, float, total)
    ALLOC(v, float, total)
    ALLOC(w16, uint16_t, na)
    ALLOC(at_a, int32_t, total)
    if (p->by_rows) {
        ALLOC(w16b, uint16_t, nb)
        ALLOC(at_b, int32_t, total)
    }
    ALLOC(H1, float, Bh)
    ALLOC(H2, float, Bh)
    if (!p->by_rows) {
        ALLOC(Z1, float, Bh)
        ALLOC(Z2, float, Bh)
        ALLOC(Z3, float, Bo)
        ALLOC(P, float, Bo)
    }
    ALLOC(dZ3, float, Bo)
    ALLOC(dZ2, float, Bh)
    ALLOC(dZ1, float, Bh)
    ALLOC(row_loss, float, max_batch)
#undef ALLOC
    hipError_t e = hipSuccess;
    if (r == RAYSH_OK) {
        e = hipMemcpy(p->master, params, total * sizeof(float), hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(p->at_a, at_a.data(), total * sizeof(int32_t), hipMemcpyHostToDevice);
        if (e == hipSuccess && p->by_rows) {
            // the layouts' padding stays zero: only real entries are ever written
            e = hipMemcpy(p->at_b, at_b.data(), total * sizeof(int32_t), hipMemcpyHostToDevice);
            if (e == hipSuccess) e = hipMemset(p->w16, 0, na * sizeof(uint16_t));
            if (e == hipSuccess) e = hipMemset(p->w16b, 0, nb * sizeof(uint16_t));
        }
        if (e == hipSuccess) e = hipMemset(p->m, 0, total * sizeof(float));
        if (e == hipSuccess) e = hipMemset(p->v, 0, total * sizeof(float));
        if (e == hipSuccess) {
            hipLaunchKernelGGL(to_bf16_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, p->stream,
                               p->master, p->w16, p->at_a, p->w16b, p->at_b, total);
            e = hipGetLastError();
        }
        if (e == hipSuccess) e = hipStreamSynchronize(p->stream);
        if (e != hipSuccess) r = hip_error(e, "raysh_mlp_create");
    }
    if (r != RAYSH_OK) {
        mlp_release(p);
        delete p;
        return r;
    }
    *out = p;
    return set_ok();
}

int64_t raysh_mlp_n_params(const raysh_mlp *p) { return p ? p->n_params : 0; }

int raysh_mlp_get_params(const raysh_mlp *p, float *params) {
    if (!p || !params) return set_error(RAYSH_EINVAL, "NULL argument");
    DeviceGuard g(p->device);
    hipError_t e = hipMemcpyAsync(params, p->master, p->n_params * sizeof(float), hipMemcpyDeviceToHost, p->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(p->stream);
    if (e != hipSuccess) return hip_error(e, "raysh_mlp_get_params");
    return set_ok();
}

int raysh_mlp_forward(raysh_mlp *p, const float *x, int32_t batch, float *probs) {
    if (!p) return set_error(RAYSH_EINVAL, "mlp is NULL");
    if (int r = check_batch(p, batch)) return r;
    if (!x || !probs) return set_error(RAYSH_EINVAL, "NULL buffer");
    DeviceGuard g(p->device);
    if (!g.ok) return set_error(RAYSH_EDEVICE, "hipSetDevice(%d) failed", p->device);
    if (int r = validate_device_ptr(x, (size_t)batch * p->n_in * 4, p->device, "x")) return r;
    if (int r = validate_device_ptr(probs, (size_t)batch * p->n_out * 4, p->device, "probs")) return r;
    if (p->by_rows) {
        // a workgroup writes its rows' outputs while others still read x
        const size_t out_bytes = (size_t)batch * p->n_out * 4;
        const bool aside = overlap(x, (size_t)batch * p->n_in * 4, probs, out_bytes);
        forward_rows<false>(p, x, nullptr, batch, aside ? p->dZ3 : probs);
        if (aside) {
            const hipError_t e = hipMemcpyAsync(probs, p->dZ3, out_bytes, hipMemcpyDeviceToDevice, p->stream);
            if (e != hipSuccess) return hip_error(e, "raysh_mlp_forward");
        }
    } else {
        forward(p, x, batch);
        hipLaunchKernelGGL(softmax_xent_kernel, dim3(batch), dim3(64), 0, p->stream, p->Z3, nullptr, batch, p->n_out,
                           probs, nullptr, nullptr);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "raysh_mlp_forward");
    return set_ok();
}

int raysh_mlp_gradient(raysh_mlp *p, const float *x, const float *target, int32_t batch, float *grads,
                       float *loss) {
    if (!p) return set_error(RAYSH_EINVAL, "mlp is NULL");
    if (int r = check_batch(p, batch)) return r;
    if (!x || !target) return set_error(RAYSH_EINVAL, "NULL buffer");
    DeviceGuard g(p->device);
    if (!g.ok) return set_error(RAYSH_EDEVICE, "hipSetDevice(%d) failed", p->device);
    if (int r = validate_device_ptr(x, (size_t)batch * p->n_in * 4, p->device, "x")) return r;
    if (int r = validate_device_ptr(target, (size_t)batch * p->n_out * 4, p->device, "target")) return r;
    if (grads)
        if (int r = validate_device_ptr(grads, (size_t)p->n_params * 4, p->device, "grads")) return r;
    if (loss)
        if (int r = validate_device_ptr(loss, 4, p->device, "loss")) return r;
    hipStream_t s = p->stream;
    const int B = batch, h = p->h, ni = p->n_in, no = p->n_out;
    float *G = p->grad;
    if (p->by_rows) {
        forward_rows<true>(p, x, target, B, nullptr);
        GradLayer l[3] = {{x, p->dZ1, ni, h, p->off[0], p->off[1], 0, 0},
                          {p->H1, p->dZ2, h, h, p->off[2], p->off[3], 0, 0},
                          {p->H2, p->dZ3, h, no, p->off[4], p->off[5], 0, 0}};
        int tiles = 0;
        for (GradLayer &g : l) {
            g.tiles_n = (g.N + 15) / 16;
            g.first = tiles;
            tiles += ((g.M + 15) / 16) * g.tiles_n;
        }
        // workgroups write grads and the loss while others still read x: in buffers that
        // share memory the loss comes after the gradient, and the caller's copy last
        const size_t x_bytes = (size_t)B * ni * 4, g_bytes = (size_t)p->n_params * 4;
        const bool in_turn =
            overlap(x, x_bytes, grads, g_bytes) || overlap(x, x_bytes, loss, 4) || overlap(grads, g_bytes, loss, 4);
        const auto launch = [&](int blocks, int n_tiles, float *copy, float *mean) {
            hipLaunchKernelGGL(mlp_grad_kernel, dim3(blocks), dim3(256), 0, s, l[0], l[1], l[2], n_tiles, B, G, copy,
                               p->row_loss, mean);
        };
        hipError_t e = hipSuccess;
        if (!in_turn) {
            launch(tiles + (loss ? 1 : 0), tiles, grads, loss);
        } else {
            launch(tiles, tiles, nullptr, nullptr);
            if (loss) launch(1, 0, nullptr, loss);   // the workgroup past the last tile takes the loss
            if (grads) e = hipMemcpyAsync(grads, G, g_bytes, hipMemcpyDeviceToDevice, s);
        }
        if (e == hipSuccess) e = hipGetLastError();
        if (e != hipSuccess) return hip_error(e, "raysh_mlp_gradient");
        p->has_grad = true;
        return set_ok();
    }
    forward(p, x, B);
    hipLaunchKernelGGL(softmax_xent_kernel, dim3(B), dim3(64), 0, s, p->Z3, target, B, no, p->P, p->dZ3,
                       p->row_loss);
    // layer 3
    gemm<true, false, false, EPI_STORE>(s, p->H2, h, p->dZ3, no, h, no, B, G + p->off[4], no);
    hipLaunchKernelGGL(column_sum_kernel, dim3((no + kSumCols - 1) / kSumCols), dim3(kSumCols * kSumGroups), 0,
                       s, p->dZ3, B, no, G + p->off[5]);
    gemm<false, true, true, EPI_GELU_GRAD>(s, p->dZ3, no, p->w16 + p->woff[2], no, B, h, no, p->dZ2, h, nullptr,
                                           p->Z2);
    // layer 2
    gemm<true, false, false, EPI_STORE>(s, p->H1, h, p->dZ2, h, h, h, B, G + p->off[2], h);
    hipLaunchKernelGGL(column_sum_kernel, dim3((h + kSumCols - 1) / kSumCols), dim3(kSumCols * kSumGroups), 0,
                       s, p->dZ2, B, h, G + p->off[3]);
    gemm<false, true, true, EPI_GELU_GRAD>(s, p->dZ2, h, p->w16 + p->woff[1], h, B, h, h, p->dZ1, h, nullptr,
                                           p->Z1);
    // layer 1
    gemm<true, false, false, EPI_STORE>(s, x, ni, p->dZ1, h, ni, h, B, G + p->off[0], h);
    hipLaunchKernelGGL(column_sum_kernel, dim3((h + kSumCols - 1) / kSumCols), dim3(kSumCols * kSumGroups), 0,
                       s, p->dZ1, B, h, G + p->off[1]);
    if (loss) hipLaunchKernelGGL(mean_loss_kernel, dim3(1), dim3(256), 0, s, p->row_loss, B, loss);
    if (grads) {
        hipError_t e = hipMemcpyAsync(grads, G, p->n_params * sizeof(float), hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return hip_error(e, "raysh_mlp_gradient");
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "raysh_mlp_gradient");
    p->has_grad = true;
    return set_ok();
}

int raysh_mlp_adam_step(raysh_mlp *p, float lr, float beta1, float beta2, float eps) {
    if (!p) return set_error(RAYSH_EINVAL, "mlp is NULL");
    if (!p->has_grad) return set_error(RAYSH_EINVAL, "no gradient computed yet");
    if (!(std::isfinite(lr) && lr > 0) || !(beta1 >= 0 && beta1 < 1) || !(beta2 >= 0 && beta2 < 1) ||
        !(std::isfinite(eps) && eps >= 0))
        return set_error(RAYSH_EINVAL, "Adam hyper-parameters out of range");
    DeviceGuard g(p->device);
    if (!g.ok) return set_error(RAYSH_EDEVICE, "hipSetDevice(%d) failed", p->device);
    p->step += 1;
    const float bc1 = (float)(1.0 - std::pow((double)beta1, (double)p->step));
    const float bc2 = (float)(1.0 - std::pow((double)beta2, (double)p->step));
    hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((p->n_params + 255) / 256)), dim3(256), 0, p->stream,
                       p->master, p->w16, p->at_a, p->w16b, p->at_b, p->grad, p->m, p->v, p->n_params, lr, beta1, beta2,
                       eps, bc1, bc2);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "raysh_mlp_adam_step");
    return set_ok();
}

int raysh_mlp_train_step(raysh_mlp *p, const float *x, const float *target, int32_t batch, float lr,
                         float beta1, float beta2, float eps, float *loss) {
    if (int r = raysh_mlp_gradient(p, x, target, batch, nullptr, loss)) return r;
    return raysh_mlp_adam_step(p, lr, beta1, beta2, eps);
}

int raysh_mlp_sync(raysh_mlp *p) {
    if (!p) return set_error(RAYSH_EINVAL, "mlp is NULL");
    DeviceGuard g(p->device);
    hipError_t e = hipStreamSynchronize(p->stream);
    if (e != hipSuccess) return hip_error(e, "raysh_mlp_sync");
    return set_ok();
}

int raysh_mlp_free(raysh_mlp *p) {
    if (!p) return set_ok();
    {
        DeviceGuard g(p->device);
        (void)hipStreamSynchronize(p->stream);
        mlp_release(p);
    }
    delete p;
    return set_ok();
}

}  // extern "C"
