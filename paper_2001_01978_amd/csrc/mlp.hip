// Warm-start network and start-vector expansion.
//
// The network maps an instance (pair energies, couplings) to one logit l_i
// per orbit; sigmoid(l_i) is trained against the half occupation <N_i>/2 of
// the exact ground state.  Reading sigmoid(l) as the BCS occupation v^2 gives
// the pair amplitude v/u = exp(l/2), and projecting that product state onto n
// pairs gives the start vector psi_k ~ prod_{i occupied in k} exp(l_i/2).
//
// Dense layers run on the matrix cores: operands are rounded from FP32 to
// BF16 as they are read, products accumulate in FP32
// (gfx950's v_mfma_f32_16x16x32_bf16: 32 products per output per
// instruction), and bias, GELU, the loss and GELU's derivative are fused into the store.
#include <cmath>

#include "pd_internal.h"

namespace pd {
namespace mlp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short shortx8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ short to_bf16(float f) {
    // round to nearest even on the upper 16 bits (inputs are finite)
    unsigned u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (short)(u >> 16);
}

__device__ __forceinline__ float gelu_tanh(float x) {
    const float c = 0.7978845608028654f;  // sqrt(2/pi)
    return 0.5f * x * (1.0f + tanhf(c * (x + 0.044715f * x * x * x)));
}

__device__ __forceinline__ float gelu_tanh_grad(float x) {
    const float c = 0.7978845608028654f;
    const float t = tanhf(c * (x + 0.044715f * x * x * x));
    return 0.5f * (1.0f + t) + 0.5f * x * (1.0f - t * t) * c * (1.0f + 3.0f * 0.044715f * x * x);
}

constexpr int kK = 32;            // k per MFMA (16x16x32)

// Eight consecutive k of one row of an operand (zero past its ends): P(row, k)
// at P[row * ld + k], or at P[k * ld + row] when trans.
__device__ __forceinline__ void load8(const float *__restrict__ P, int ld, bool trans, int row, int rows, int k, int K,
                                      float (&v)[8]) {
    if (row >= rows || k >= K) {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = 0.f;
    } else if (k + 8 <= K) {
        const float *q = trans ? P + (int64_t)k * ld + row : P + (int64_t)row * ld + k;
        const int64_t step = trans ? ld : 1;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = q[i * step];
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            v[i] = k + i < K ? (trans ? P[(int64_t)(k + i) * ld + row] : P[(int64_t)row * ld + k + i]) : 0.f;
    }
}

__device__ __forceinline__ bf16x8 pack8(const float (&v)[8]) {
    shortx8 r;
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = to_bf16(v[i]);
    return __builtin_bit_cast(bf16x8, r);
}

// Stores a 16 x 16 tile at (m0, n0): lane holds C[4 (lane / 16) + v][lane % 16].
// Returns the lane's part of the sum of squares (Loss).
__device__ __forceinline__ float store_tile(const MlpGemm &G, floatx4 acc, int m0, int n0, int lane) {
    float loss = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int gm = m0 + (lane >> 4) * 4 + v, gn = n0 + (lane & 15);
        if (gm < G.M && gn < G.N) {
            const int64_t at = (int64_t)gm * G.ldc + gn;
            float z = acc[v];
            if (G.bias) z += G.bias[gn];
            if (G.mode == kMlpTimesGeluGrad) z *= gelu_tanh_grad(G.aux[at]);
            G.C[at] = z;
            if (G.mode == kMlpGelu) G.out2[at] = gelu_tanh(z);
            if (G.mode == kMlpLoss) {
                // loss = mean (sigmoid(l) - t)^2; out2 = d loss / d l
                const float sg = 1.0f / (1.0f + expf(-z));
                const float d = sg - G.aux[at];
                loss += d * d;
                G.out2[at] = 2.0f * d * sg * (1.0f - sg) / G.count;
            }
        }
    }
    return loss;
}

// One or two products C = op(A) op(B) (MlpGemm) in a launch.  The layers are
// small (256 x 256 x 324), so what counts is how many waves share the work
// and how long each one's chain is: a wave per 16 x 16 tile gives 256 waves
// where tiles of 64 gave 16 workgroups, and it reads its operands straight into
// the matrix instruction's layout (lane l holds row l % 16 at k = 8 (l / 16) ..
// 8 (l / 16) + 7), kDepth steps of k ahead.  The sums run over k in the same order
// for either tile size.  Loss gradients of 256 rows through 324 x 256 x 256 x 24:
// 254 us with 16 launches (64 x 64 tiles, a kernel each for the column sums,
// GELU's derivative and the loss), 39 us with these 6; a launch takes 5-10 us,
// mostly its latency.
constexpr int kDepth = 4;
__device__ __forceinline__ void gemm_tile16(const MlpGemm &G, int tile) {
    const int lane = threadIdx.x, r = lane & 15, kq = (lane >> 4) * 8;
    const int ntn = (G.N + 15) / 16;
    const int m0 = tile / ntn * 16, n0 = tile % ntn * 16;
    floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
    float colsum = 0.f;
    float a[2][kDepth][8], b[2][kDepth][8];
    auto load = [&](int k0, int buf) {
#pragma unroll
        for (int d = 0; d < kDepth; ++d) {
            load8(G.A, G.lda, G.ta, m0 + r, G.M, k0 + d * kK + kq, G.K, a[buf][d]);
            load8(G.B, G.ldb, !G.tb, n0 + r, G.N, k0 + d * kK + kq, G.K, b[buf][d]);
        }
    };
    load(0, 0);
    for (int k0 = 0; k0 < G.K; k0 += 2 * kDepth * kK) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int kh = k0 + half * kDepth * kK;
            if (kh >= G.K) break;
            if (kh + kDepth * kK < G.K) load(kh + kDepth * kK, half ^ 1);
#pragma unroll
            for (int d = 0; d < kDepth; ++d) {
                if (kh + d * kK >= G.K) break;
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pack8(a[half][d]), pack8(b[half][d]), acc, 0, 0, 0);
#pragma unroll
                for (int e = 0; e < 8; ++e) colsum += b[half][d][e];
            }
        }
    }
    if (G.colsum && m0 == 0) {
        float c = colsum;
        c += __shfl_xor(c, 16, 64);
        c += __shfl_xor(c, 32, 64);
        if (lane < 16 && n0 + lane < G.N) G.colsum[n0 + lane] = c;
    }
    float loss = store_tile(G, acc, m0, n0, lane);
    if (G.mode == kMlpLoss) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) loss += __shfl_xor(loss, o, 64);
        if (lane == 0) G.partial[tile] = loss;
    }
}

// Large layers: a 64 x 64 tile per workgroup of four waves (2 x 2 tiles of the
// matrix instruction each), which reads an operand element a quarter as often.
// Both operands are staged k-contiguous, each thread converting 8 consecutive k
// of one row into one 16-byte LDS write; the next step's elements are asked for
// before this step is multiplied.
constexpr int kTile = 64;
constexpr int kRow = kK + 8;      // LDS row of a staged tile: 32 BF16 + 16 bytes of padding
__device__ __forceinline__ void gemm_tile64(const MlpGemm &G, int tile) {
    __shared__ __align__(16) short As[kTile][kRow], Bs[kTile][kRow];
    __shared__ float lsum[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ntn = (G.N + kTile - 1) / kTile;
    const int m0 = tile / ntn * kTile, n0 = tile % ntn * kTile;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32;
    const int srow = tid >> 2, sk = (tid & 3) * 8;     // this thread's staging row and k offset
    floatx4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    float a[8], b[8], colsum = 0.f;
    load8(G.A, G.lda, G.ta, m0 + srow, G.M, sk, G.K, a);
    load8(G.B, G.ldb, !G.tb, n0 + srow, G.N, sk, G.K, b);
    for (int k0 = 0; k0 < G.K; k0 += kK) {
        *reinterpret_cast<bf16x8 *>(&As[srow][sk]) = pack8(a);
        *reinterpret_cast<bf16x8 *>(&Bs[srow][sk]) = pack8(b);
#pragma unroll
        for (int e = 0; e < 8; ++e) colsum += b[e];
        __syncthreads();
        if (k0 + kK < G.K) {
            load8(G.A, G.lda, G.ta, m0 + srow, G.M, k0 + kK + sk, G.K, a);
            load8(G.B, G.ldb, !G.tb, n0 + srow, G.N, k0 + kK + sk, G.K, b);
        }
        const int r = lane & 15, kq = (lane >> 4) * 8;
        bf16x8 av[2], bv[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            av[i] = *reinterpret_cast<const bf16x8 *>(&As[wm + i * 16 + r][kq]);
            bv[i] = *reinterpret_cast<const bf16x8 *>(&Bs[wn + i * 16 + r][kq]);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[i], bv[j], acc[i][j], 0, 0, 0);
        __syncthreads();
    }
    if (G.colsum && m0 == 0) {
        colsum += __shfl_xor(colsum, 1, 64);
        colsum += __shfl_xor(colsum, 2, 64);
        if ((tid & 3) == 0 && n0 + srow < G.N) G.colsum[n0 + srow] = colsum;
    }
    float loss = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) loss += store_tile(G, acc[i][j], m0 + wm + i * 16, n0 + wn + j * 16, lane);
    if (G.mode == kMlpLoss) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) loss += __shfl_xor(loss, o, 64);
        if (lane == 0) lsum[wave] = loss;
        __syncthreads();
        if (tid == 0) G.partial[tile] = (lsum[0] + lsum[1]) + (lsum[2] + lsum[3]);
    }
}

template <int SIZE>
__global__ __launch_bounds__(SIZE * 4) void gemm_kernel(MlpGemmSet S) {
    const int t0 = S.tiles[0], t1 = S.tiles[1];
    const int b = blockIdx.x;
    if (b < t0 + t1) {
        const MlpGemm &G = S.g[b < t0 ? 0 : 1];
        if constexpr (SIZE == 16)
            gemm_tile16(G, b < t0 ? b : b - t0);
        else
            gemm_tile64(G, b < t0 ? b : b - t0);
    } else if (threadIdx.x < 64) {
        // the loss: its partial sums in a fixed order
        float s = 0.f;
        for (int i = threadIdx.x; i < S.npartial; i += 64) s += S.partial[i];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if (threadIdx.x == 0) *S.loss = s * S.scale;
    }
}

// Adam (Kingma & Ba 2015) with bias correction.
__global__ void adam_kernel(int count, float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                            float *__restrict__ v, float lr, float b1, float b2, float eps, float c1, float c2) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float mi = b1 * m[i] + (1.f - b1) * gi;
        const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
        m[i] = mi;
        v[i] = vi;
        p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    }
}

// psi_k = exp(0.5 * (sum_{i occupied in k} l_i - lmax)); lmax = sum of the n largest l.
__global__ void warm_expand_kernel(int omega, int n, int64_t dim, const float *__restrict__ logits, double lmax,
                                   double *__restrict__ psi) {
    __shared__ double l[64];
    if ((int)threadIdx.x < omega) l[threadIdx.x] = (double)logits[threadIdx.x];
    __syncthreads();
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < dim; k += (int64_t)gridDim.x * blockDim.x) {
        uint64_t r = (uint64_t)k;
        int m = n;
        double s = 0.0;
        for (int p = omega - 1; p >= 0; --p) {
            uint64_t c = g_binom.v[p][m];
            if (m > 0 && c <= r) {
                r -= c;
                --m;
                s += l[p];
            }
        }
        psi[k] = exp(0.5 * (s - lmax));
    }
}

}  // namespace mlp

// Tiles of 16 up to the count at which tiles of 64 fill half the CUs.  Forward
// passes, tiles of 16 against 64: 512 rows through 256 x 256 28 against 63 us, 1024
// through 512 x 512 65 against 84, 4096 through 256 x 256 77 against 60, 2048 through
// 1024 x 1024 317 against 162.
constexpr int64_t kSmallTiles = 2048;
int mlp_tiles(int M, int N, int size) { return ((M + size - 1) / size) * ((N + size - 1) / size); }

hipError_t launch_mlp_gemms(MlpGemmSet S, hipStream_t s) {
    int64_t small = 0;
    for (int i = 0; i < 2; ++i)
        if (S.g[i].M > 0) small += (int64_t)((S.g[i].M + 15) / 16) * ((S.g[i].N + 15) / 16);
    const int size = small <= kSmallTiles ? 16 : 64;
    int blocks = 0;
    for (int i = 0; i < 2; ++i) {
        S.tiles[i] = S.g[i].M > 0 ? mlp_tiles(S.g[i].M, S.g[i].N, size) : 0;
        blocks += S.tiles[i];
    }
    if (S.loss) ++blocks;
    if (size == 16)
        hipLaunchKernelGGL((mlp::gemm_kernel<16>), dim3(blocks), dim3(64), 0, s, S);
    else
        hipLaunchKernelGGL((mlp::gemm_kernel<64>), dim3(blocks), dim3(256), 0, s, S);
    return hipGetLastError();
}

// Tiles (and partial sums of the loss) of the product that takes the loss.
int mlp_loss_tiles(int M, int N) {
    return mlp_tiles(M, N, (int64_t)((M + 15) / 16) * ((N + 15) / 16) <= kSmallTiles ? 16 : 64);
}

hipError_t launch_adam(int count, float *p, const float *g, float *m, float *v, float lr, float b1, float b2,
                       float eps, int step, hipStream_t s) {
    const float c1 = 1.0f - std::pow(b1, (float)step), c2 = 1.0f - std::pow(b2, (float)step);
    hipLaunchKernelGGL(mlp::adam_kernel, dim3((count + 255) / 256 < 1024 ? (count + 255) / 256 : 1024), dim3(256), 0,
                       s, count, p, g, m, v, lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_warm_expand(int omega, int n, int64_t dim, const float *logits, double lmax, double *psi,
                              hipStream_t s) {
    int64_t g = (dim + 255) / 256;
    if (g > 4096) g = 4096;
    if (g < 1) g = 1;
    hipLaunchKernelGGL(mlp::warm_expand_kernel, dim3((unsigned)g), dim3(256), 0, s, omega, n, dim, logits, lmax, psi);
    return hipGetLastError();
}

}  // namespace pd
