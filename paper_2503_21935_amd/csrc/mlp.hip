// mlp.hip -- surrogate network kernels: BF16 matrix-core GEMMs with FP32
// accumulation and fused epilogues, loss, reductions, Adam; the C ABI of
// include/mlp.h.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/mlp.h"
#include "me_internal.h"

typedef __bf16 bf16;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

#define MLP_KPAD 32  // first-layer inputs padded to one MFMA K step
#define MLP_DW_SPLITS 16  // batch splits of the weight-gradient GEMMs
#ifndef MLPF_TILE_ROWS
#define MLPF_TILE_ROWS 128  // rows per block of the fused inference kernel (64: 5 % slower)
#endif

// ---------------------------------------------------------------------------
// GEMM: C[m][n] = sum_k A(m, k) B(k, n), A(m, k) = A[m * a_sm + k * a_sk],
// B(k, n) = B[k * b_sk + n * b_sn], BF16 operands, FP32 accumulation on
// v_mfma_f32_16x16x32_bf16.  A 256-thread block computes a 64 x 64 tile, each
// wave 32 x 32 (2 x 2 MFMA tiles).  Fragment layouts (16x16x32): lane l holds
// A[l%16][8(l/16) .. +7], B[8(l/16) .. +7][l%16] and D[4(l/16) + v][l%16].
// Requirements: K % 32 == 0; rows/columns beyond M/N are computed on clamped
// operands and not stored.
// ---------------------------------------------------------------------------
enum { EPI_FWD_TRAIN = 0, EPI_FWD_INFER = 1, EPI_BWD_DH = 2, EPI_DW = 3 };

struct epi_args {
    const float* bias;  // FWD: [N]
    float* z;           // FWD_TRAIN: pre-activations [M][N]
    bf16* h;            // FWD: activations [M][ldh]
    int ldh;
    const float* zprev; // BWD_DH: pre-activations of the previous layer [M][N]
    bf16* dz;           // BWD_DH: output gradient w.r.t. those pre-activations [M][N]
    float* g;           // DW: gradient [M][N] row-major with leading dimension ldg
    int ldg;
    int64_t zstride;    // DW with split K: elements between the partial slabs of blockIdx.z
    int ncols_store;    // DW: columns actually stored (n_in for the first layer)
};

// Logistic function with the hardware reciprocal (v_rcp_f32, about 1 ulp):
// a correctly rounded division costs ten instructions per activation, and the
// value is rounded to BF16 (8 bits) or enters an FP32 gradient next.
__device__ __forceinline__ float sigmoidf_(float z) { return __builtin_amdgcn_rcpf(1.f + __expf(-z)); }

template <bool AK1, bool BK1>
__device__ __forceinline__ void load_frags(const bf16* __restrict__ A, int64_t a_sm, int64_t a_sk,
                                           const bf16* __restrict__ B, int64_t b_sk, int64_t b_sn, int row0,
                                           int col0, int k0, int M, int N, int lane, bf16x8 (&a)[2],
                                           bf16x8 (&b)[2]) {
    const int kk = k0 + 8 * (lane >> 4);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        int r = row0 + 16 * i + (lane & 15);
        r = r < M ? r : M - 1;
        const bf16* p = A + (int64_t)r * a_sm + (int64_t)kk * a_sk;
        if constexpr (AK1) {
            a[i] = *reinterpret_cast<const bf16x8*>(p);
        } else {
#pragma unroll
            for (int v = 0; v < 8; ++v) a[i][v] = p[(int64_t)v * a_sk];
        }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        int c = col0 + 16 * j + (lane & 15);
        c = c < N ? c : N - 1;
        const bf16* p = B + (int64_t)kk * b_sk + (int64_t)c * b_sn;
        if constexpr (BK1) {
            b[j] = *reinterpret_cast<const bf16x8*>(p);
        } else {
#pragma unroll
            for (int v = 0; v < 8; ++v) b[j][v] = p[(int64_t)v * b_sk];
        }
    }
}

// Split K: block z of gridDim.z handles k in [z kspan, (z + 1) kspan) (kspan a
// multiple of 32); only the DW epilogue supports it (one partial slab per z).
template <int EPI, bool AK1, bool BK1>
__global__ __launch_bounds__(256) void k_gemm(int M, int N, int K, int kspan, const bf16* __restrict__ A,
                                              int64_t a_sm, int64_t a_sk, const bf16* __restrict__ B,
                                              int64_t b_sk, int64_t b_sn, epi_args e) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row0 = blockIdx.y * 64 + (wave >> 1) * 32;
    const int col0 = blockIdx.x * 64 + (wave & 1) * 32;
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int kb = blockIdx.z * kspan, ke = min(K, kb + kspan);
    for (int k0 = kb; k0 < ke; k0 += 32) {
        bf16x8 a[2], b[2];
        load_frags<AK1, BK1>(A, a_sm, a_sk, B, b_sk, b_sn, row0, col0, k0, M, N, lane, a, b);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int c = col0 + 16 * j + (lane & 15);
            if (c >= N) continue;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = row0 + 16 * i + 4 * (lane >> 4) + v;
                if (r >= M) continue;
                const float x = acc[i][j][v];
                if constexpr (EPI == EPI_FWD_TRAIN || EPI == EPI_FWD_INFER) {
                    const float z = x + e.bias[c];
                    if constexpr (EPI == EPI_FWD_TRAIN) e.z[(int64_t)r * N + c] = z;
                    e.h[(int64_t)r * e.ldh + c] = (bf16)(z * sigmoidf_(z));
                } else if constexpr (EPI == EPI_BWD_DH) {
                    const float z = e.zprev[(int64_t)r * N + c];
                    const float s = sigmoidf_(z);
                    e.dz[(int64_t)r * N + c] = (bf16)(x * s * (1.f + z * (1.f - s)));
                } else {
                    if (c < e.ncols_store) e.g[(int64_t)blockIdx.z * e.zstride + (int64_t)r * e.ldg + c] = x;
                }
            }
        }
}

// ---------------------------------------------------------------------------
// Fused inference for width 256: a block of 256 threads (4 waves) carries a
// tile of 128 rows through every layer with the activations in LDS, so the
// only HBM traffic is the input, the output and (from L2) the weights.  Per
// layer, wave w computes output columns 64w..64w+63 for all 128 rows (4 x 8
// MFMA tiles of 16 x 16, K steps of 32); after a barrier the bias + SiLU
// epilogue writes the BF16 activations over the layer's input.  Numerics as
// in the layered path: BF16 inputs, weights and activations, FP32
// accumulation, FP32 bias, activation and output layer.
// The weights are the first operand of the products, the rows the second, so
// a lane ends up with four consecutive columns of one row and stores them with
// one instruction; the weights come in fragment order (1 KB per load
// instruction) and one K step ahead of their use.  Two blocks per CU, so
// that one's epilogue (activation functions) runs beside the other's products.
// The input is a row of features or, with MOM, an event's momenta, whose
// features (those of k_features) are then formed on the way into LDS.
// 2^20 rows take 0.52 ms (0.75 with the rows first and row-major weights), 0.83 PFLOP/s.
// Bound by issue: the matrix cores are busy 38 % of the cycles and the vector
// unit another 60 %, two thirds of that exp and rcp; the two hardly overlap
// (wave priorities, a phase offset between the blocks, four smaller blocks per CU
// and loads pinned one step ahead all measured the same or slower).
// ---------------------------------------------------------------------------
#define MLPF_W 256
#define MLPF_PITCH (MLPF_W + 8)  // bf16 per LDS row: rows 528 B apart, no bank conflicts
#define MLPF_MAXDEPTH 8

struct mlpf_args {
    const bf16* w[MLPF_MAXDEPTH];   // hidden layers, [256][K] (K = 32 for the first, padded)
    bool frag;                      // in fragment order (else row-major)
    const float* b[MLPF_MAXDEPTH];  // their biases [256]
    const float* wout;              // output weights [256]
    const float* bout;              // output bias [1]
};

// 1 / sqrt(shat) of an event from its incoming momenta.
__device__ __forceinline__ double inv_sqrt_shat(const double* __restrict__ p) {
    const double E = p[0] + p[4], px = p[1] + p[5], py = p[2] + p[6], pz = p[3] + p[7];
    return 1.0 / sqrt(E * E - px * px - py * py - pz * pz);
}

// ROWS rows per 256-thread block (a multiple of 16 dividing 256).
template <int ROWS, bool MOM>
__global__ __launch_bounds__(256, 8192 / (ROWS * 32)) void k_mlp_infer(const float* __restrict__ x,
                                                                        const double* __restrict__ mom, int64_t n,
                                                                        int n_in, int depth, mlpf_args a,
                                                                        float* __restrict__ y) {
    constexpr int RT = ROWS / 16;      // 16-row MFMA tiles
    constexpr int TPR = 256 / ROWS;    // threads per row in the output layer
    __shared__ __attribute__((aligned(16))) bf16 H[ROWS * MLPF_PITCH];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t row0 = (int64_t)blockIdx.x * ROWS;
    // the whole tile's loads in flight at once (clamped, then masked)
    constexpr int PER = ROWS * MLP_KPAD / 256;  // elements per thread: column k of every 8th row
    const int k = threadIdx.x % MLP_KPAD, r0 = threadIdx.x / MLP_KPAD;
    const auto at = [&](int j) {
        const int64_t gr = row0 + r0 + (256 / MLP_KPAD) * j;
        return (gr < n ? gr : n - 1) * n_in + (k < n_in ? k : 0);
    };
    const auto put = [&](int j, float v) {
        const int r = r0 + (256 / MLP_KPAD) * j;
        H[r * MLPF_PITCH + k] = (bf16)((row0 + r < n && k < n_in) ? v : 0.f);
    };
    if constexpr (MOM) {
        __shared__ double inv[ROWS];
        double v[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) v[j] = mom[at(j)];
        if (threadIdx.x < ROWS) {
            const int64_t gr = row0 + threadIdx.x;
            inv[threadIdx.x] = inv_sqrt_shat(mom + (gr < n ? gr : n - 1) * n_in);
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            float f = (float)(v[j] * inv[r0 + (256 / MLP_KPAD) * j]);
            asm volatile("" : "+v"(f));  // rounded to FP32 first, as k_features stores it: not folded into one conversion
            put(j, f);
        }
    } else {
        float v[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) v[j] = x[at(j)];
#pragma unroll
        for (int j = 0; j < PER; ++j) put(j, v[j]);
    }
    __syncthreads();
    const int li = lane & 15, lg = lane >> 4;
    auto layer = [&](auto KS, int l) __attribute__((always_inline)) {
        constexpr int ks = KS;  // K steps
        f32x4 acc[4][RT];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) acc[t][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
        constexpr int wt = ks * 512;          // from tile to tile
        const int wk = a.frag ? 512 : 32;     // from K step to K step
        const bf16* W = a.w[l] + 4 * wave * wt + (a.frag ? 8 * lane : li * (32 * ks) + 8 * lg);
        bf16x8 w[2][4];
#pragma unroll
        for (int t = 0; t < 4; ++t) w[0][t] = *reinterpret_cast<const bf16x8*>(W + t * wt);
#pragma unroll
        for (int k = 0; k < ks; ++k) {
            if (k + 1 < ks) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    w[(k + 1) & 1][t] = *reinterpret_cast<const bf16x8*>(W + t * wt + (k + 1) * wk);
            }
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const bf16x8 h = *reinterpret_cast<const bf16x8*>(H + (16 * rt + li) * MLPF_PITCH + 32 * k + 8 * lg);
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    acc[t][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[k & 1][t], h, acc[t][rt], 0, 0, 0);
            }
        }
        __syncthreads();  // every wave has read the layer's input
        // acc[t][rt][v]: column 64 wave + 16 t + 4 lg + v of row 16 rt + li
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int c = 64 * wave + 16 * t + 4 * lg;
            const f32x4 bc = *reinterpret_cast<const f32x4u*>(a.b[l] + c);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                bf16x4 h;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float z = acc[t][rt][v] + bc[v];
                    h[v] = (bf16)(z * sigmoidf_(z));
                }
                *reinterpret_cast<bf16x4*>(H + (16 * rt + li) * MLPF_PITCH + c) = h;
            }
        }
        __syncthreads();
    };
    layer(std::integral_constant<int, 1>{}, 0);
    for (int l = 1; l < depth; ++l) layer(std::integral_constant<int, MLPF_W / 32>{}, l);
    // output layer: y = sum_k h[k] w[k] + b; TPR adjacent threads per row, each
    // over MLPF_W / TPR columns in 16-byte reads, then a butterfly
    {
        const int r = threadIdx.x / TPR, part = threadIdx.x % TPR;
        constexpr int CW = MLPF_W / TPR;
        const bf16x8* hr = reinterpret_cast<const bf16x8*>(H + r * MLPF_PITCH + part * CW);
        const float* wo = a.wout + part * CW;
        float s = 0.f;
#pragma unroll 4
        for (int k8 = 0; k8 < CW / 8; ++k8) {
            const bf16x8 v = hr[k8];
#pragma unroll
            for (int q = 0; q < 8; ++q) s = fmaf((float)v[q], wo[8 * k8 + q], s);
        }
#pragma unroll
        for (int o = 1; o < TPR; o <<= 1) s += __shfl_xor(s, o);
        const int64_t gr = row0 + r;
        if (part == 0 && gr < n) y[gr] = s + a.bout[0];
    }
}

// ---------------------------------------------------------------------------
// Element-wise and reduction kernels
// ---------------------------------------------------------------------------

// X[j][k] = bf16(x[src(j)][k]) for k < n_in, zero for n_in <= k < 32.
__global__ void k_prep_input(const float* __restrict__ x, const int32_t* __restrict__ idx, int64_t n, int n_in,
                             bf16* __restrict__ X) {
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    const int64_t src = idx ? idx[j] : j;
    for (int k = 0; k < MLP_KPAD; ++k) X[j * MLP_KPAD + k] = (bf16)(k < n_in ? x[src * n_in + k] : 0.f);
}

// y[m] = sum_k H[m][k] w[k] + b (FP32 accumulation)
__global__ void k_last_fwd(const bf16* __restrict__ H, int64_t M, int width, const float* __restrict__ w,
                           const float* __restrict__ b, float* __restrict__ y) {
    const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= M) return;
    const bf16x8* h = reinterpret_cast<const bf16x8*>(H + m * width);
    float s = 0.f;
    for (int k8 = 0; k8 < width / 8; ++k8) {
        const bf16x8 v = h[k8];
#pragma unroll
        for (int q = 0; q < 8; ++q) s = fmaf((float)v[q], w[8 * k8 + q], s);
    }
    y[m] = s + b[0];
}

// dy[m] = 2 (y[m] - t[src(m)]) / M; per-block partial sums of the squared residual.
__global__ void k_loss(const float* __restrict__ y, const float* __restrict__ t, const int32_t* __restrict__ idx,
                       int64_t M, float* __restrict__ dy, float* __restrict__ partial) {
    __shared__ float red[256];
    const int64_t m = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    float r2 = 0.f;
    if (m < M) {
        const float r = y[m] - t[idx ? idx[m] : m];
        dy[m] = 2.f * r / (float)M;
        r2 = r * r;
    }
    red[threadIdx.x] = r2;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

__global__ void k_loss_final(const float* __restrict__ partial, int nblocks, int64_t M, float* __restrict__ loss) {
    __shared__ float red[256];
    float s = 0.f;
    for (int i = threadIdx.x; i < nblocks; i += 256) s += partial[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = red[0] / (float)M;
}

// dZ[m][n] = bf16(dy[m] w[n] silu'(Z[m][n]))
__global__ void k_last_bwd(const float* __restrict__ dy, const float* __restrict__ w, const float* __restrict__ Z,
                           int64_t M, int width, bf16* __restrict__ dZ) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= M * width) return;
    const int64_t m = i / width;
    const int n = (int)(i % width);
    const float z = Z[i];
    const float s = sigmoidf_(z);
    dZ[i] = (bf16)(dy[m] * w[n] * s * (1.f + z * (1.f - s)));
}

// part[z][n] = sum over rows m of chunk z of coef(m) A[m][n] (coef = dy[m] or 1);
// block (x, z) covers 64 columns of row chunk z; k_sum_splits adds the chunks.
template <typename TA>
__global__ void k_colsum_part(const TA* __restrict__ A, const float* __restrict__ coef, int64_t M, int N,
                              int64_t rows, float* __restrict__ part) {
    __shared__ float red[4][64];
    const int c = blockIdx.x * 64 + (threadIdx.x & 63);
    const int rg = threadIdx.x >> 6;
    const int64_t m0 = (int64_t)blockIdx.y * rows, m1 = (m0 + rows < M) ? m0 + rows : M;
    float s = 0.f;
    if (c < N)
        for (int64_t m = m0 + rg; m < m1; m += 4) s = fmaf(coef ? coef[m] : 1.f, (float)A[m * N + c], s);
    red[rg][threadIdx.x & 63] = s;
    __syncthreads();
    if (rg == 0 && c < N)
        part[(int64_t)blockIdx.y * N + c] =
            red[0][threadIdx.x] + red[1][threadIdx.x] + red[2][threadIdx.x] + red[3][threadIdx.x];
}

// out[0] = sum_m dy[m]
__global__ void k_sum(const float* __restrict__ v, int64_t M, float* __restrict__ out) {
    __shared__ float red[256];
    float s = 0.f;
    for (int64_t m = threadIdx.x; m < M; m += 256) s += v[m];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = red[0];
}

struct layer_map {
    int64_t w_off[16], b_off[16];
    int fan_in[16];
};

// Adam with bias correction on the flat FP32 parameters, then the BF16 copies
// of the weight matrices (first layer padded to 32 inputs).
// Offset of element (n, k) of a [rows][K] matrix (rows a multiple of 16, K of
// 32) stored in fragment order: for each 16-row tile and 32-column step the
// 64 lanes' 16-byte B fragments of v_mfma_f32_16x16x32_bf16 (lane n % 16 +
// 16 ((k % 32) / 8) holds columns 8 ((k % 32) / 8) .. + 7 of row n) lie
// contiguously, so one load instruction reads 1 KB in lane order.
__device__ __forceinline__ int64_t frag_off(int n, int k, int K) {
    return ((int64_t)((n >> 4) * (K >> 5) + (k >> 5)) * 64 + (n & 15) + 16 * ((k & 31) >> 3)) * 8 + (k & 7);
}

__global__ void k_adam(float* __restrict__ theta, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, int64_t np, float lr, float c1, float c2, layer_map L,
                       int depth, int width, bf16* const* __restrict__ wbf, bf16* const* __restrict__ wbft,
                       bf16* const* __restrict__ wfr, bf16* const* __restrict__ wtfr) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= np) return;
    const float gi = g[i];
    const float mi = 0.9f * m[i] + 0.1f * gi;
    const float vi = 0.999f * v[i] + 0.001f * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float th = theta[i] - lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
    theta[i] = th;
    for (int l = 0; l < depth; ++l) {
        const int64_t o = L.w_off[l];
        const int fi = L.fan_in[l];
        if (i >= o && i < o + (int64_t)width * fi) {
            const int64_t r = (i - o) / fi, k = (i - o) % fi;
            const int ld = (l == 0) ? MLP_KPAD : fi;
            wbf[l][r * ld + k] = (bf16)th;
            if (l > 0) wbft[l][k * width + r] = (bf16)th;
            if (wfr) {
                wfr[l][frag_off((int)r, (int)k, ld)] = (bf16)th;
                if (l > 0) wtfr[l][frag_off((int)k, (int)r, width)] = (bf16)th;
            }
        }
    }
}

// Fragment-order copies (see frag_off) of W_l (pads k >= fan_in zero) or, with
// trans, of W_l^T, from the master parameters.
__global__ void k_to_bf16_frag(const float* __restrict__ theta, int64_t o, int rows, int fi, int ld, int trans,
                               bf16* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)rows * ld) return;
    if (!trans) {
        const int r = (int)(i / ld), k = (int)(i % ld);
        out[frag_off(r, k, ld)] = (bf16)(k < fi ? theta[o + (int64_t)r * fi + k] : 0.f);
    } else {
        const int k = (int)(i / rows), r = (int)(i % rows);  // row k of W^T, [fi][rows]
        out[frag_off(k, r, rows)] = (bf16)theta[o + (int64_t)r * fi + k];
    }
}

// BF16 copies from the master parameters (after set_params / init)
__global__ void k_to_bf16(const float* __restrict__ theta, int64_t o, int rows, int fi, int ld, bf16* __restrict__ w) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)rows * ld) return;
    const int64_t r = i / ld, k = i % ld;
    w[i] = (bf16)(k < fi ? theta[o + r * fi + k] : 0.f);
}

// transposed BF16 copy wt[k][r] = theta[o + r fi + k] of a hidden weight matrix
__global__ void k_to_bf16_t(const float* __restrict__ theta, int64_t o, int rows, int fi, bf16* __restrict__ wt) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)rows * fi) return;
    const int64_t k = i / rows, r = i % rows;
    wt[i] = (bf16)theta[o + r * fi + k];
}

// ---------------------------------------------------------------------------
// Fused training step for width 256 (one cooperative launch; one grid-wide
// barrier inside a step, one between steps).  The batch's rows are
// independent through the whole forward and backward chain, so phase 1 gives
// each block tiles of FT_R rows and carries them through every layer forward
// (activations, and the derivatives of the activation functions, in LDS), the output layer and loss, and
// every layer backward down to the first pre-activation gradient, reading the
// BF16 weights (and their transposes) in MFMA fragment order from L2, each
// layer's fragments loaded during the previous layer's epilogue.  Each tile's
// activations (but the last layer's) and gradients also go to global memory transposed
// ([feature][batch], fragment order, from the registers that hold them; the input from
// LDS), and its share of the output layer's gradient to a per-tile partial.  The
// only cross-row work is
// the weight and bias gradients, sums over the batch: after the barrier,
// phase 2 computes them as GEMMs dW_l = dZ_l^T H_{l-1} on 32 x 32 tiles, one
// per block, each wave over a quarter of the batch; the quarters are added in
// LDS in a fixed order (the result does not depend on the grid) and the block
// applies Adam to the tile's FP32 masters and refreshes their BF16 copies, so
// every parameter is updated by the block that formed its gradient; where no
// block has two tiles the masters and moments stay in its LDS from step to
// step.  Rounding points are those of the layered path.
// A step of 4096 rows at depth 4 takes 41 us (68 before): 20 in phase 1, of which
// 1 us per product is one CU's share of the weights through its L1 and 5 the
// first reads after the barrier, which come from memory; 11 in phase 2 (half a
// megabyte of operands per block); the rest the two barriers with their cache
// write-back and invalidation.  What the 27 us were, by stamps of single blocks, which
// run beside each other, so that the parts add up to more: the loss added in one
// chain of dependent loads by a block with an item of its own (20), 256 LDS reads for 16
// partial losses (2), operands left dirty for the barrier to write back (3),
// moments read and written in every step (2), registers spilled to memory
// that each barrier's invalidation makes cold, and loads under conditions that
// make the counted waits wait for everything (6 together).
// ---------------------------------------------------------------------------
#define FT_R 16        // rows per phase-1 tile
#define FT_S 4         // batch quarters of the weight-gradient sums, one per wave
#define FT_MAXDEPTH 4  // the derivatives of every layer's activations stay in LDS

struct ft_args {
    const float* x;           // [*][n_in]
    const float* t;           // targets
    const int32_t* idx;       // batch rows (nullptr: the first M)
    int64_t M;                // batch size (multiple of FT_S * 32)
    int n_in, depth;
    bf16* wfr[FT_MAXDEPTH];   // W_l [256][ld] in fragment order (ld 32 for the first layer)
    bf16* wtfr[FT_MAXDEPTH];  // W_l^T [fan_in][256] in fragment order (layers >= 1)
    bf16* wbf[FT_MAXDEPTH];   // row-major BF16 copies (other kernels), written by the launch's last step
    bf16* wbft[FT_MAXDEPTH];
    float* theta;             // FP32 masters (flat layout)
    float *m, *v;             // Adam moments
    float* grad_out;          // gradient only (no update) when non-null
    layer_map L;
    int64_t wout_off, bout_off, np;
    bf16* XT;                 // [32][M], fragment order with K = M
    bf16* HT[FT_MAXDEPTH];    // [256][M], the same
    bf16* DZT[FT_MAXDEPTH];   // [256][M], the same
    float* opart;             // [257][M / FT_R]: output-layer gradient per tile (weights, then bias)
    float* lossp;             // [gridDim.x]
    unsigned* bar;            // grid barrier state (zeroed once at allocation)
    float* loss;              // [nsteps] or nullptr
    float lr, c1, c2;         // one step (lrs == nullptr): its rate and bias corrections
    const float* lrs;         // [nsteps] rates of the steps, or nullptr
    int64_t step0;            // Adam steps taken before this launch
    int nsteps;               // steps in this launch, batch st on rows idx[st M ..] (or st M ..)
};

// B fragments of rows 64 wave + 16 t + 0..15 of the [256][K] matrix Wm kept in
// fragment order (K / 32 MFMA k-steps).
template <int K>
__device__ __forceinline__ void ft_load_w(const bf16* __restrict__ Wm, int wave, int lane, bf16x8 (&b)[8][4]) {
    unsigned off = 16u * (unsigned)lane;
    asm volatile("" : "+v"(off));  // scalar base plus this: no vector addresses to keep (and spill) across the steps
    const char* base = reinterpret_cast<const char*>(Wm) + (int64_t)wave * (4 * (K / 32) * 1024);
#pragma unroll
    for (int ks = 0; ks < K / 32; ++ks)
#pragma unroll
        for (int t = 0; t < 4; ++t)
            b[ks][t] = *reinterpret_cast<const bf16x8*>(base + (t * (K / 32) + ks) * 1024 + off);
}

// acc[t] = (16-row LDS tile A, pitch MLPF_PITCH) x (the loaded rows)^T.
template <int K>
__device__ __forceinline__ void ft_mma(const bf16* A, const bf16x8 (&b)[8][4], int li, int lg, f32x4 acc[4]) {
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < K / 32; ++ks) {
        const bf16x8 av = *reinterpret_cast<const bf16x8*>(A + li * MLPF_PITCH + 32 * ks + 8 * lg);
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, b[ks][t], acc[t], 0, 0, 0);
    }
}

// The weights of product k of a tile's chain after the first layer (k = 1 ..
// 2 (D - 1)): W_k forward for k < D, then W_l^T backward for l = D - 1 .. 1.
template <int D, int K>
__device__ __forceinline__ void ft_load_chain(const ft_args& a, int wave, int lane, bf16x8 (&b)[8][4]) {
    if constexpr (K >= 1 && K <= D - 1) ft_load_w<MLPF_W>(a.wfr[K], wave, lane, b);
    else if constexpr (K >= D && K <= 2 * (D - 1)) ft_load_w<MLPF_W>(a.wtfr[2 * D - 1 - K], wave, lane, b);
}

// Grid-wide barrier of a cooperative launch (every block resident).  Each
// thread waits for its own memory operations, then one thread per block
// publishes the block's writes (agent-scope release: the L2 write-back),
// arrives on bar[0] and waits for the generation in bar[32] to move; the last
// block to arrive resets the count and moves the generation.  One release
// and one acquire per block, where a fence in every wave would write the L2
// back once per wave.  The other waves do `meanwhile` during the wait.
template <class F>
__device__ __forceinline__ void ft_grid_sync(unsigned* bar, F&& meanwhile) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        const unsigned g = __hip_atomic_load(&bar[32], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned prev = __hip_atomic_fetch_add(&bar[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (prev == gridDim.x - 1) {
            __hip_atomic_store(&bar[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&bar[32], g + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            while (__hip_atomic_load(&bar[32], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == g)
                __builtin_amdgcn_s_sleep(1);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    } else if (threadIdx.x >= 64) {
        meanwhile();
    }
    __syncthreads();
}

// Four batch rows of a feature, batch tile m0, to the [feature][batch] array dst in
// fragment order with K = M.  Written through to memory as it is produced (three
// layers' activations and four layers' gradients, 14.7 MB per step at depth 4 and 4096
// rows): left dirty in the L2, it is written back at the grid barrier, where every
// block waits for it.
// Feature 16 f + li (f the same in the whole wave), rows 4 lg .. 4 lg + 3.
__device__ __forceinline__ void ft_store4(bf16x4 h, int f, int li, int lg, bf16* dst, int64_t M, int64_t m0) {
    const int b = (int)(m0 & 31) + 4 * lg;
    bf16* at = dst + ((int64_t)f * (M >> 5) + (m0 >> 5)) * 512 + (128 * (b >> 3) + li * 8 + (b & 7));
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(at), __builtin_bit_cast(unsigned long long, h),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Column c of the 16-row LDS tile S (batch rows m0 .. m0 + 15) to the
// [feature][batch] array dst in fragment order with K = M (two 16-byte stores).
__device__ __forceinline__ void ft_store_t(const bf16* S, int c, bf16* dst, int64_t M, int64_t m0) {
    bf16x8 v0, v1;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        v0[r] = S[r * MLPF_PITCH + c];
        v1[r] = S[(8 + r) * MLPF_PITCH + c];
    }
    const int64_t base = ((int64_t)(c >> 4) * (M >> 5) + (m0 >> 5)) * 512 + (c & 15) * 8;
    const int q = (int)(m0 & 31) >> 3;  // 0 or 2
    *reinterpret_cast<bf16x8*>(dst + base + 128 * q) = v0;
    *reinterpret_cast<bf16x8*>(dst + base + 128 * (q + 1)) = v1;
}

// Adam on a parameter (FP32 master, moments) with gradient g.
__device__ __forceinline__ void ft_adam(float g, float& m, float& v, float& th, float lr, float c1, float c2) {
    m = fmaf(0.1f, g, 0.9f * m);  // explicit: which product is fused must not depend on the surroundings
    v = fmaf(0.001f * g, g, 0.999f * v);
    th = th - lr * (m / c1) / (sqrtf(v / c2) + 1e-8f);
}

// The update of a parameter without BF16 copies (biases, output layer), or
// its gradient only.
__device__ __forceinline__ void ft_update(const ft_args& a, int64_t i, float g, float lr, float c1, float c2) {
    if (a.grad_out) {
        a.grad_out[i] = g;
        return;
    }
    float m = a.m[i], v = a.v[i], th = a.theta[i];
    ft_adam(g, m, v, th, lr, c1, c2);
    a.m[i] = m;
    a.v[i] = v;
    a.theta[i] = th;
}

// f(0) .. f(N - 1) with constant arguments
template <int N, int K = 0, class F>
__device__ __forceinline__ void ft_each(F&& f) {
    if constexpr (K < N) {
        f(std::integral_constant<int, K>{});
        ft_each<N, K + 1>(f);
    }
}

// Sum of src[0 .. n): thread q of eight adjacent ones adds q, q + 8, ..., 32 loads
// in flight, and the eight are combined by shuffles.
__device__ __forceinline__ float ft_sum8(const float* __restrict__ src, int n, int q) {
    float g = 0.f;
    for (int i = q; i < n; i += 256) {
        float v[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) v[u] = src[i + 8 * u < n ? i + 8 * u : i];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 32; ++u) g = i + 8 * u < n ? g + v[u] : g;
    }
    g += __shfl_xor(g, 1);
    g += __shfl_xor(g, 2);
    return g + __shfl_xor(g, 4);
}

// The 16 input rows (padded to MLP_KPAD features) and targets of the tile at
// batch row m0 of step st into LDS, by N threads u = 0 .. N - 1.
template <int N>
__device__ __forceinline__ void ft_rows(const ft_args& a, int st, int64_t m0, int u, bf16* Hs, float* tgs) {
    constexpr int E = FT_R * MLP_KPAD, Q = (E + N - 1) / N;
    const int32_t* idx = a.idx ? a.idx + (int64_t)st * a.M : nullptr;
    const float* x = a.idx ? a.x : a.x + (int64_t)st * a.M * a.n_in;
    const float* tg = a.idx ? a.t : a.t + (int64_t)st * a.M;
    int64_t src[Q];
    float xv[Q], tv[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int e = u + N * q, r = (e < E ? e : u) / MLP_KPAD;
        src[q] = idx ? idx[m0 + r] : m0 + r;
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int k = (u + N * q) % MLP_KPAD;
        xv[q] = x[src[q] * a.n_in + (k < a.n_in ? k : 0)];
        tv[q] = tg[src[q]];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int e = u + N * q, r = e / MLP_KPAD, k = e % MLP_KPAD;
        if (e < E) {
            Hs[r * MLPF_PITCH + k] = (bf16)(k < a.n_in ? xv[q] : 0.f);
            if (k == 0) tgs[r] = tv[q];
        }
    }
}

template <int D>
__global__ __launch_bounds__(256, 1) void k_mlp_train_fused(ft_args a) {
    constexpr int W = MLPF_W, P = MLPF_PITCH;
    static_assert(FT_R == 16 && W == 256, "one 16-row MFMA tile per phase-1 step, one thread per feature");
    // layer input and output, pre-activation gradients: two each, so that a layer
    // needs one barrier (the first Hs is the tile's input)
    __shared__ __attribute__((aligned(16))) bf16 Hs[2][FT_R * P], Gs[2][FT_R * P];
    __shared__ float part[4096 + 128];                          // phase 2: [wave][32][32] partial tiles, [wave][32] of the biases
    __shared__ float dact[D][FT_R][W + 4];                      // derivatives of the activations (each lane's own)
    __shared__ float bs[D][W];                                  // hidden biases of this step
    __shared__ float wos[W + 1];                                // output weights and bias
    __shared__ float dys[FT_R], tgs[FT_R], sq[FT_R], corr[3];
    __shared__ __attribute__((aligned(16))) float red[256];
    __shared__ __attribute__((aligned(16))) bf16 wq[32 * 40];   // phase 2: the item's new weights, rows 80 bytes apart
    // Moments and masters of the block's phase-2 item (four weights per thread; its
    // biases).  Where no block has two items they stay here from the first step
    // of the launch to the last.
    __shared__ float held[12][256], heldb[3][32];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t M = a.M;
    const int nrt = (int)(M / FT_R);
    // B fragments: bw0 the first layer's (one k-step); the products after it
    // alternate between bwa (odd) and bwb (even), and the weights of product
    // k + 2 are loaded into a buffer as soon as product k has used it, so
    // every load has a whole layer's work to arrive.  The depth is a constant:
    // loads under a condition cannot be counted, and the first layer's
    // would be waited for with all that were issued after them.
    bf16x8 bw0[8][4], bwa[8][4], bwb[8][4];
    for (int st = 0; st < a.nsteps; ++st) {
        // Offsets are formed in each step and phase: kept from step to step they
        // spill, and after a grid barrier a spilled value comes from memory.
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        int lane = tid & 63, li = lane & 15, lg = lane >> 4;
        float loss_acc = 0.f;
        float bv[D], wv = a.theta[a.wout_off + tid], wb = a.theta[a.bout_off];
#pragma unroll
        for (int l = 0; l < D; ++l) bv[l] = a.theta[a.L.b_off[l] + tid];

        // ---------------- phase 1: rows through forward and backward ----------------
        if (st == 0 && (int)blockIdx.x < nrt) ft_rows<256>(a, st, (int64_t)blockIdx.x * FT_R, tid, Hs[0], tgs);
        for (int rt = blockIdx.x; rt < nrt; rt += gridDim.x) {
            const int64_t m0 = (int64_t)rt * FT_R;
            ft_load_w<MLP_KPAD>(a.wfr[0], wave, lane, bw0);
            ft_load_chain<D, 1>(a, wave, lane, bwa);
            ft_load_chain<D, 2>(a, wave, lane, bwb);
            // (for every tile: under a condition, all the loads above would be waited for)
#pragma unroll
            for (int l = 0; l < D; ++l) bs[l][tid] = bv[l];
            wos[tid] = wv;
            wos[W] = wb;
            __syncthreads();
            if (tid < MLP_KPAD) ft_store_t(Hs[0], tid, a.XT, M, m0);
            // A lane's elements of a layer: columns 64 wave + 16 t + li of rows 4 lg + v,
            // the same in every layer and in both directions.
            ft_each<D>([&](auto LL) __attribute__((always_inline)) {
                constexpr int l = LL;
                f32x4 acc[4];
                if constexpr (l == 0) {
                    ft_mma<MLP_KPAD>(Hs[0], bw0, li, lg, acc);
                } else if constexpr (l & 1) {  // product l
                    ft_mma<W>(Hs[1], bwa, li, lg, acc);
                    ft_load_chain<D, l + 2>(a, wave, lane, bwa);
                } else {
                    ft_mma<W>(Hs[0], bwb, li, lg, acc);
                    ft_load_chain<D, l + 2>(a, wave, lane, bwb);
                }
                bf16* out = Hs[(l + 1) & 1];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int c = 64 * wave + 16 * t + li;
                    const float bc = bs[l][c];
                    bf16x4 h;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float z = acc[t][v] + bc;
                        const float s = sigmoidf_(z);
                        h[v] = (bf16)(z * s);
                        dact[l][4 * lg + v][c] = s * (1.f + z * (1.f - s));
                        out[(4 * lg + v) * P + c] = h[v];
                    }
                    if constexpr (l + 1 < D) ft_store4(h, 4 * wave + t, li, lg, a.HT[l], M, m0);
                }
                __syncthreads();
            });
            const bf16* hl = Hs[D & 1];
            // output layer, residual, loss (16 threads per row)
            {
                const int r = tid >> 4, q16 = tid & 15;
                const bf16x8* hr = reinterpret_cast<const bf16x8*>(hl + r * P + q16 * 16);
                float s = 0.f;
#pragma unroll
                for (int k8 = 0; k8 < 2; ++k8) {
                    const bf16x8 hv = hr[k8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) s = fmaf((float)hv[q], wos[q16 * 16 + 8 * k8 + q], s);
                }
#pragma unroll
                for (int o = 1; o < 16; o <<= 1) s += __shfl_xor(s, o);
                if (q16 == 0) {
                    const float res = s + wos[W] - tgs[r];
                    dys[r] = 2.f * res / (float)M;
                    loss_acc += res * res;
                }
            }
            __syncthreads();
            // this tile's share of the output layer's gradient
            {
                const int c = tid;
                float gw = 0.f, gb = 0.f;
#pragma unroll
                for (int r = 0; r < FT_R; ++r) {
                    gw = fmaf(dys[r], (float)hl[r * P + c], gw);
                    gb += dys[r];
                }
                a.opart[(int64_t)c * nrt + rt] = gw;
                if (c == 0) a.opart[(int64_t)W * nrt + rt] = gb;
            }
            // dZ of the last hidden layer
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int c = 64 * wave + 16 * t + li;
                const float woc = wos[c];
                bf16x4 g;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    g[v] = (bf16)(dys[4 * lg + v] * woc * dact[D - 1][4 * lg + v][c]);
                    Gs[0][(4 * lg + v) * P + c] = g[v];
                }
                ft_store4(g, 4 * wave + t, li, lg, a.DZT[D - 1], M, m0);
            }
            __syncthreads();
            // backward through the hidden layers: dZ_{l-1} = (dZ_l W_l) silu'(Z_{l-1})
            // (product 2 D - 1 - l: bwa when l is even)
            ft_each<D - 1>([&](auto II) __attribute__((always_inline)) {
                constexpr int l = D - 1 - II, k = 2 * D - 1 - l, in = II & 1;
                f32x4 acc[4];
                if constexpr ((l & 1) == 0) {
                    ft_mma<W>(Gs[in], bwa, li, lg, acc);
                    ft_load_chain<D, k + 2>(a, wave, lane, bwa);
                } else {
                    ft_mma<W>(Gs[in], bwb, li, lg, acc);
                    ft_load_chain<D, k + 2>(a, wave, lane, bwb);
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int c = 64 * wave + 16 * t + li;
                    bf16x4 g;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        g[v] = (bf16)(acc[t][v] * dact[l - 1][4 * lg + v][c]);
                        Gs[1 - in][(4 * lg + v) * P + c] = g[v];
                    }
                    ft_store4(g, 4 * wave + t, li, lg, a.DZT[l - 1], M, m0);
                }
                __syncthreads();
            });
            const int next = rt + (int)gridDim.x;
            if (next < nrt) ft_rows<256>(a, st, (int64_t)next * FT_R, tid, Hs[0], tgs);
        }
        if ((tid & 15) == 0) sq[tid >> 4] = loss_acc;  // the threads that hold any
        __syncthreads();
        if (tid == 0) {
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < FT_R; ++i) s += sq[i];
            a.lossp[blockIdx.x] = s;
        }
        // during the wait: the update's constants, and the next step's first tile
        const bool pre = st + 1 < a.nsteps && (int)blockIdx.x < nrt;
        ft_grid_sync(a.bar, [&]() __attribute__((always_inline)) {
            if (wave == 1) {
                const float k = (float)(a.step0 + st + 1);
                const float c1 = a.lrs ? 1.f - powf(0.9f, k) : a.c1, c2 = a.lrs ? 1.f - powf(0.999f, k) : a.c2;
                const float lr = a.lrs ? a.lrs[st] : a.lr;
                if (lane == 0) corr[0] = c1, corr[1] = c2, corr[2] = lr;
            }
            if (pre) ft_rows<192>(a, st + 1, (int64_t)blockIdx.x * FT_R, tid - 64, Hs[0], tgs);
        });

        // ---------------- phase 2: weight gradients and the update ----------------
        const float c1 = corr[0], c2 = corr[1], lr = corr[2];
        tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        lane = tid & 63, li = lane & 15, lg = lane >> 4;
        // the loss, by the last block (which seldom has an item), added in block order
        if (blockIdx.x == gridDim.x - 1 && a.loss) {
            float s = 0.f;
            for (int o = 0; o < (int)gridDim.x; o += 256) {
                __syncthreads();
                red[tid] = o + tid < (int)gridDim.x ? a.lossp[o + tid] : 0.f;
                __syncthreads();
                if (tid == 0) {
#pragma unroll 16
                    for (int i = 0; i < 64; ++i) {
                        const f32x4 v = reinterpret_cast<const f32x4*>(red)[i];
                        s = (((s + v[0]) + v[1]) + v[2]) + v[3];
                    }
                }
            }
            if (tid == 0) a.loss[st] = s / (float)M;
        }
        // items: per layer l, 8 x (padded fan-in / 32) tiles of 32 x 32 of dW_l
        // (n-tile major), then eight output-layer items
        constexpr int nw = 8 + 64 * (D - 1), nitems = nw + 8;
        // Items that share operand rows are neighbours in this order; blocks go
        // round-robin over the 8 XCDs, so slot v of XCD x takes item x q + v:
        // each XCD's L2 then fetches about an eighth of the operands instead
        // of nearly all of them.
        constexpr int q8 = (nitems + 7) / 8;
        const bool hold = 8 * q8 <= (int)gridDim.x, last = st + 1 == a.nsteps, fresh = !hold || st == 0;
        for (int vb = blockIdx.x; vb < 8 * q8; vb += gridDim.x) {
            const int it = (vb % 8) * q8 + vb / 8;
            if (it >= nitems) continue;
            if (it >= nw) {
                // output layer, columns 32 oq .. 32 oq + 31 (the last item also takes
                // the bias, in wave 0's first lanes' second sum): eight threads per
                // column add the per-tile partials in a fixed interleave, combine them
                // by shuffles and update
                const int oq = it - nw;
                const int c = 32 * oq + (tid >> 3), q = tid & 7;
                const float g = ft_sum8(a.opart + (int64_t)c * nrt, nrt, q);
                if (q == 0) ft_update(a, a.wout_off + c, g, lr, c1, c2);
                if (oq == 7 && wave == 0) {
                    const float d = ft_sum8(a.opart + (int64_t)W * nrt, nrt, q);
                    if (lane == 0) ft_update(a, a.bout_off, d, lr, c1, c2);
                }
                continue;
            }
            const int l = it < 8 ? 0 : 1 + (it - 8) / 64, j = it < 8 ? it : (it - 8) % 64;
            const int kt = l == 0 ? 1 : 8;
            const int nb = j / kt, kb = j % kt;
            const int fi = l == 0 ? a.n_in : W, ld = l == 0 ? MLP_KPAD : W;
            // operands in fragment order: the fragment of 16-row tile f at batch
            // step m / 32 starts at (f (M / 32) + m / 32) 512
            const bf16* A = a.DZT[l];                       // dZ_l^T [n][m]
            const bf16* B = (l == 0) ? a.XT : a.HT[l - 1];  // H_{l-1}^T [k][m]
            const bf16* Ar[2];
            const bf16* Br[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                Ar[i] = A + (int64_t)(2 * nb + i) * (M >> 5) * 512;
                Br[i] = B + (int64_t)(2 * kb + i) * (M >> 5) * 512;
            }
            const int lane8 = lane * 8;
            f32x4 acc[2][2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int k = 0; k < 2; ++k) acc[i][k] = f32x4{0.f, 0.f, 0.f, 0.f};
            float bsum[2] = {0.f, 0.f};
            auto mstep = [&](const bf16x8 (&av)[2], const bf16x8 (&bv)[2]) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
#pragma unroll
                    for (int q = 0; q < 8; ++q) bsum[i] += (float)av[i][q];
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        acc[i][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[i], bv[k], acc[i][k], 0, 0, 0);
                }
            };
            // this wave's quarter of the batch
            const int64_t mq = M / FT_S, mb = (int64_t)wave * mq;
            constexpr int U = 8;  // batch steps whose loads are all in flight together
            int64_t m = mb;
            for (; m + 32 * U <= mb + mq; m += 32 * U) {
                bf16x8 av[U][2], bv[U][2];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        av[u][i] = *reinterpret_cast<const bf16x8*>(Ar[i] + 16 * (m + 32 * u) + lane8);
                        bv[u][i] = *reinterpret_cast<const bf16x8*>(Br[i] + 16 * (m + 32 * u) + lane8);
                    }
#pragma unroll
                for (int u = 0; u < U; ++u) mstep(av[u], bv[u]);
            }
            for (; m < mb + mq; m += 32) {
                bf16x8 av[2], bv[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    av[i] = *reinterpret_cast<const bf16x8*>(Ar[i] + 16 * m + lane8);
                    bv[i] = *reinterpret_cast<const bf16x8*>(Br[i] + 16 * m + lane8);
                }
                mstep(av, bv);
            }
            // the wave's partial tile: element (n, k) = acc[i][k'][v], n = 16 i + 4 lg + v, k = 16 k' + li
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int k = 0; k < 2; ++k)
#pragma unroll
                    for (int v = 0; v < 4; ++v) part[(wave * 32 + 16 * i + 4 * lg + v) * 32 + 16 * k + li] = acc[i][k][v];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                bsum[i] += __shfl_xor(bsum[i], 16);
                bsum[i] += __shfl_xor(bsum[i], 32);
                if (lg == 0) part[4096 + wave * 32 + 16 * i + li] = bsum[i];
            }
            // four of the tile's 1024 weights per thread, 8 rows apart: element tid + 256 r
            const int n0 = tid >> 5, kk = 32 * kb + (tid & 31);
            const int64_t i0 = a.L.w_off[l] + (int64_t)(32 * nb + n0) * fi + kk, ib = a.L.b_off[l] + 32 * nb + tid;
            const bool mine = kk < fi, bias = kb == 0 && tid < 32;
            if (fresh && !a.grad_out) {
                float x[12];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int64_t i = mine ? i0 + (int64_t)(8 * r) * fi : a.L.w_off[l];
                    x[r] = a.m[i], x[4 + r] = a.v[i], x[8 + r] = a.theta[i];
                }
#pragma unroll
                for (int r = 0; r < 12; ++r) held[r][tid] = x[r];
                if (bias) heldb[0][tid] = a.m[ib], heldb[1][tid] = a.v[ib], heldb[2][tid] = a.theta[ib];
            }
            __syncthreads();
            // the four quarters added in wave order
            float g[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int e = tid + 256 * r;
                g[r] = ((part[e] + part[1024 + e]) + part[2048 + e]) + part[3072 + e];
            }
            if (a.grad_out) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (mine) a.grad_out[i0 + (int64_t)(8 * r) * fi] = g[r];
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float mo = held[r][tid], vo = held[4 + r][tid], th = held[8 + r][tid];
                    ft_adam(g[r], mo, vo, th, lr, c1, c2);
                    held[r][tid] = mo, held[4 + r][tid] = vo, held[8 + r][tid] = th;
                    wq[(n0 + 8 * r) * 40 + (tid & 31)] = mine ? (bf16)th : (bf16)0.f;
                }
            }
            if (bias) {
                const float gb = ((part[4096 + tid] + part[4096 + 32 + tid]) + part[4096 + 64 + tid]) + part[4096 + 96 + tid];
                if (a.grad_out) {
                    a.grad_out[ib] = gb;
                } else {
                    float mo = heldb[0][tid], vo = heldb[1][tid], th = heldb[2][tid];
                    ft_adam(gb, mo, vo, th, lr, c1, c2);
                    heldb[0][tid] = mo, heldb[1][tid] = vo, heldb[2][tid] = th;
                    a.theta[ib] = th;
                    if (!hold || last) a.m[ib] = mo, a.v[ib] = vo;
                }
            }
            __syncthreads();  // wq is complete; part is rewritten by the next item
            if (!a.grad_out) {
                // The fragment-order copies feed the next step: lane f of fragment (n, k)
                // holds columns 8 (f / 16) .. + 7 of row f % 16, one 16-byte store per
                // thread, the first half of the block W, the second W^T.
                const int half = tid >> 7, t16 = (tid >> 6) & 1;
                if (half == 0) {
                    const bf16x8 v = *reinterpret_cast<const bf16x8*>(wq + (16 * t16 + li) * 40 + 8 * lg);
                    *reinterpret_cast<bf16x8*>(a.wfr[l] + ((int64_t)((2 * nb + t16) * (ld >> 5) + kb) * 64 + lane) * 8) = v;
                } else if (l > 0) {
                    bf16x8 v;
#pragma unroll
                    for (int q = 0; q < 8; ++q) v[q] = wq[(8 * lg + q) * 40 + 16 * t16 + li];
                    *reinterpret_cast<bf16x8*>(a.wtfr[l] + ((int64_t)((2 * kb + t16) * (W >> 5) + nb) * 64 + lane) * 8) = v;
                }
                if (!hold || last) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int64_t i = i0 + (int64_t)(8 * r) * fi;
                        if (mine) a.m[i] = held[r][tid], a.v[i] = held[4 + r][tid], a.theta[i] = held[8 + r][tid];
                    }
                }
                // the row-major copies feed only other kernels
                if (last) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int rr = 32 * nb + n0 + 8 * r;
                        const bf16 v = wq[(n0 + 8 * r) * 40 + (tid & 31)];
                        if (mine) a.wbf[l][rr * ld + kk] = v;
                        if (mine && l > 0) a.wbft[l][kk * W + rr] = v;
                    }
                }
            }
        }
        if (st + 1 < a.nsteps) ft_grid_sync(a.bar, []() {});  // the next step reads the updated weights
    }
}

// Blocks of 256 threads, FEAT_EV events each: the events' 1 / sqrt(shat) once, then
// momenta and features in address order (one event per thread, 192 bytes apart,
// took 0.65 ms for 2^20 events of six particles; now 0.07 ms).
#define FEAT_EV 128
__global__ void k_features(const double* __restrict__ mom, int64_t n, int npart, float* __restrict__ x) {
    __shared__ double inv[FEAT_EV];
    const int64_t first = (int64_t)blockIdx.x * FEAT_EV;
    const int nc = 4 * npart, ne = (int)(n - first < FEAT_EV ? n - first : FEAT_EV);
    if ((int)threadIdx.x < ne) inv[threadIdx.x] = inv_sqrt_shat(mom + (first + threadIdx.x) * nc);
    __syncthreads();
    for (int e = threadIdx.x; e < ne * nc; e += 256) x[first * nc + e] = (float)(mom[first * nc + e] * inv[e / nc]);
}

// Rows of bf16(features), zero-padded to 32, from momenta: what k_features and
// k_prep_input make in two passes.
__global__ void k_prep_momenta(const double* __restrict__ mom, int64_t n, int n_in, bf16* __restrict__ X) {
    __shared__ double inv[FEAT_EV];
    const int64_t first = (int64_t)blockIdx.x * FEAT_EV;
    const int ne = (int)(n - first < FEAT_EV ? n - first : FEAT_EV);
    if ((int)threadIdx.x < ne) inv[threadIdx.x] = inv_sqrt_shat(mom + (first + threadIdx.x) * n_in);
    __syncthreads();
    for (int e = threadIdx.x; e < ne * MLP_KPAD; e += 256) {
        const int r = e / MLP_KPAD, k = e % MLP_KPAD;
        float f = k < n_in ? (float)(mom[(first + r) * n_in + k] * inv[r]) : 0.f;
        asm volatile("" : "+v"(f));  // rounded to FP32 first, as k_features stores it
        X[(first + r) * MLP_KPAD + k] = (bf16)f;
    }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

static void (*ft_kernel(int depth))(ft_args) {
    static_assert(FT_MAXDEPTH == 4, "one kernel per depth");
    return depth == 1 ? k_mlp_train_fused<1> : depth == 2 ? k_mlp_train_fused<2>
         : depth == 3 ? k_mlp_train_fused<3> : k_mlp_train_fused<4>;
}

struct me_mlp {
    int n_in, width, depth;
    int64_t np;
    layer_map L;
    int64_t wout_off, bout_off;
    float *theta, *grad, *m, *v;
    float* dwpart;           // split-K partial slabs of one weight gradient [MLP_DW_SPLITS][width][fan_in]
    std::vector<bf16*> wbf;  // per hidden layer, [width][ld]
    bf16** d_wbf;            // device array of those pointers
    std::vector<bf16*> wbft; // transposed copies [fan_in][width] (layers >= 1; the backward pass)
    bf16** d_wbft;
    std::vector<bf16*> wfr;  // fragment-order copies of W_l and W_l^T for the one-kernel step
    std::vector<bf16*> wtfr; // (width 256 only; empty otherwise)
    bf16 **d_wfr, **d_wtfr;
    bool fused;              // training step as one cooperative kernel where it applies
    int fgrid;               // its grid: co-resident blocks
    int64_t fcap;            // batch capacity of its buffers
    bf16 *XT, *HTb, *DZTb;   // transposed input, activations and gradients [feature][batch]
    float *flossp, *fopart;
    unsigned* fbar;          // grid barrier state of the fused kernel
    int64_t cap;             // activation capacity (rows)
    bf16* X;
    std::vector<bf16*> H;
    std::vector<float*> Z;
    bf16 *dZa, *dZb;
    float *y, *dy, *partial, *loss_tmp;
    int64_t step;
};

#define HCHK(expr)                                                                                   \
    do {                                                                                             \
        hipError_t _e = (expr);                                                                      \
        if (_e != hipSuccess) return me_fail(ME_EDEVICE, std::string(#expr ": ") + hipGetErrorString(_e)); \
    } while (0)

static uint64_t splitmix(uint64_t& s) {
    s += 0x9E3779B97F4A7C15ull;
    uint64_t z = s;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

static void free_acts(me_mlp* p) {
    auto f = [](void* q) {
        if (q) (void)hipFree(q);
    };
    f(p->X);
    for (auto q : p->H) f(q);
    for (auto q : p->Z) f(q);
    f(p->dZa);
    f(p->dZb);
    f(p->y);
    f(p->dy);
    f(p->partial);
    p->X = nullptr;
    p->H.assign(p->depth, nullptr);
    p->Z.assign(p->depth, nullptr);
    p->dZa = p->dZb = nullptr;
    p->y = p->dy = p->partial = nullptr;
    p->cap = 0;
}

static int ensure_acts(me_mlp* p, int64_t rows) {
    if (rows <= p->cap) return ME_OK;
    HCHK(hipDeviceSynchronize());
    free_acts(p);
    const int64_t W = p->width;
    HCHK(hipMalloc(&p->X, rows * MLP_KPAD * sizeof(bf16)));
    for (int l = 0; l < p->depth; ++l) {
        HCHK(hipMalloc(&p->H[l], rows * W * sizeof(bf16)));
        HCHK(hipMalloc(&p->Z[l], rows * W * sizeof(float)));
    }
    HCHK(hipMalloc(&p->dZa, rows * W * sizeof(bf16)));
    HCHK(hipMalloc(&p->dZb, rows * W * sizeof(bf16)));
    HCHK(hipMalloc(&p->y, rows * sizeof(float)));
    HCHK(hipMalloc(&p->dy, rows * sizeof(float)));
    HCHK(hipMalloc(&p->partial, ((rows + 255) / 256 + 1) * sizeof(float)));
    p->cap = rows;
    return ME_OK;
}

static hipError_t refresh_bf16(me_mlp* p, hipStream_t s) {
    for (int l = 0; l < p->depth; ++l) {
        const int fi = p->L.fan_in[l], ld = (l == 0) ? MLP_KPAD : fi;
        const int64_t tot = (int64_t)p->width * ld;
        hipLaunchKernelGGL(k_to_bf16, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, p->theta, p->L.w_off[l],
                           p->width, fi, ld, p->wbf[l]);
        if (l > 0) {
            const int64_t nt = (int64_t)p->width * fi;
            hipLaunchKernelGGL(k_to_bf16_t, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, s, p->theta,
                               p->L.w_off[l], p->width, fi, p->wbft[l]);
        }
        if (p->d_wfr) {
            hipLaunchKernelGGL(k_to_bf16_frag, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, p->theta,
                               p->L.w_off[l], p->width, fi, ld, 0, p->wfr[l]);
            if (l > 0)
                hipLaunchKernelGGL(k_to_bf16_frag, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, p->theta,
                                   p->L.w_off[l], p->width, fi, ld, 1, p->wtfr[l]);
        }
    }
    return hipGetLastError();
}

template <int EPI, bool AK1, bool BK1>
// Returns the number of K splits launched (partial slabs for EPI_DW).
static int gemm(hipStream_t s, int M, int N, int K, const bf16* A, int64_t a_sm, int64_t a_sk, const bf16* B,
                int64_t b_sk, int64_t b_sn, const epi_args& e, int splits = 1) {
    const int kspan = ((K + splits - 1) / splits + 31) / 32 * 32;
    splits = (K + kspan - 1) / kspan;
    dim3 grid((unsigned)((N + 63) / 64), (unsigned)((M + 63) / 64), (unsigned)splits);
    hipLaunchKernelGGL((k_gemm<EPI, AK1, BK1>), grid, dim3(256), 0, s, M, N, K, kspan, A, a_sm, a_sk, B, b_sk, b_sn,
                       e);
    return splits;
}

// out[i] = sum over z < splits of part[z n + i] (fixed order: deterministic)
__global__ void k_sum_splits(const float* __restrict__ part, int splits, int64_t n, float* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float acc = 0.f;
    for (int z = 0; z < splits; ++z) acc += part[(int64_t)z * n + i];
    out[i] = acc;
}

// out[n] = sum_m coef(m) A[m][n] over all M rows, in row chunks (partials in
// p->dwpart, summed in a fixed order).
static void colsum(hipStream_t s, const bf16* A, const float* coef, int64_t M, int N, float* scratch, float* out) {
    const int64_t chunks = std::min<int64_t>(64, (M + 63) / 64);
    const int64_t rows = (M + chunks - 1) / chunks;
    hipLaunchKernelGGL((k_colsum_part<bf16>), dim3((unsigned)((N + 63) / 64), (unsigned)chunks), dim3(256), 0, s, A,
                       coef, M, N, rows, scratch);
    hipLaunchKernelGGL(k_sum_splits, dim3((unsigned)((N + 255) / 256)), dim3(256), 0, s, scratch, (int)chunks,
                       (int64_t)N, out);
}

// Forward over rows [0, M) of p->X; training keeps Z and every H.
static void forward(me_mlp* p, int64_t M, bool train, hipStream_t s) {
    const int W = p->width;
    const bf16* in = p->X;
    int ld_in = MLP_KPAD, K = MLP_KPAD;
    for (int l = 0; l < p->depth; ++l) {
        epi_args e{};
        e.bias = p->theta + p->L.b_off[l];
        e.z = train ? p->Z[l] : nullptr;
        bf16* out = train ? p->H[l] : ((l & 1) ? p->dZb : p->dZa);  // inference ping-pongs
        e.h = out;
        e.ldh = W;
        // Z = in . W_l^T: A = in [M][K] (k contiguous), B(k, n) = W_l[n][k] (k contiguous)
        if (train)
            gemm<EPI_FWD_TRAIN, true, true>(s, (int)M, W, K, in, ld_in, 1, p->wbf[l], 1, K, e);
        else
            gemm<EPI_FWD_INFER, true, true>(s, (int)M, W, K, in, ld_in, 1, p->wbf[l], 1, K, e);
        in = out;
        ld_in = W;
        K = W;
    }
    hipLaunchKernelGGL(k_last_fwd, dim3((unsigned)((M + 255) / 256)), dim3(256), 0, s, in, M, W,
                       p->theta + p->wout_off, p->theta + p->bout_off, p->y);
}

// Loss and gradients (into p->grad) for rows [0, M) with targets t[idx].
static void backward(me_mlp* p, const float* t, const int32_t* idx, int64_t M, float* loss, hipStream_t s) {
    const int W = p->width;
    const unsigned nb = (unsigned)((M + 255) / 256);
    hipLaunchKernelGGL(k_loss, dim3(nb), dim3(256), 0, s, p->y, t, idx, M, p->dy, p->partial);
    if (loss) hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(256), 0, s, p->partial, (int)nb, M, loss);
    bf16* Hl = p->H[p->depth - 1];
    // output layer: dw_out = sum_m dy[m] H[m][:], db_out = sum dy
    colsum(s, Hl, p->dy, M, W, p->dwpart, p->grad + p->wout_off);
    hipLaunchKernelGGL(k_sum, dim3(1), dim3(256), 0, s, p->dy, M, p->grad + p->bout_off);
    hipLaunchKernelGGL(k_last_bwd, dim3((unsigned)((M * W + 255) / 256)), dim3(256), 0, s, p->dy,
                       p->theta + p->wout_off, p->Z[p->depth - 1], M, W, p->dZa);
    bf16* dz = p->dZa;
    bf16* dz_next = p->dZb;
    for (int l = p->depth - 1; l >= 0; --l) {
        const bf16* hin = (l == 0) ? p->X : p->H[l - 1];
        const int fi = p->L.fan_in[l], ldin = (l == 0) ? MLP_KPAD : W;
        // dW_l[n][k] = sum_m dZ[m][n] hin[m][k]: A(n, m) = dZ[m][n], B(m, k) = hin[m][k]
        // split over the batch (K): 16 x 16 blocks instead of 16, partial slabs summed after
        const int splits = (int)std::min<int64_t>(MLP_DW_SPLITS, std::max<int64_t>(1, M / 256));
        epi_args e{};
        e.g = splits > 1 ? p->dwpart : p->grad + p->L.w_off[l];
        e.ldg = fi;
        e.ncols_store = fi;
        e.zstride = (int64_t)W * fi;
        const int used = gemm<EPI_DW, false, false>(s, W, ldin, (int)M, dz, 1, W, hin, ldin, 1, e, splits);
        if (splits > 1) {
            const int64_t nw = (int64_t)W * fi;
            hipLaunchKernelGGL(k_sum_splits, dim3((unsigned)((nw + 255) / 256)), dim3(256), 0, s, p->dwpart, used, nw,
                               p->grad + p->L.w_off[l]);
        }
        colsum(s, dz, nullptr, M, W, p->dwpart, p->grad + p->L.b_off[l]);
        if (l > 0) {
            // dH_{l-1}[m][k] = sum_n dZ[m][n] W_l[n][k]; fused silu'(Z_{l-1})
            epi_args e2{};
            e2.zprev = p->Z[l - 1];
            e2.dz = dz_next;
            gemm<EPI_BWD_DH, true, false>(s, (int)M, W, W, dz, W, 1, p->wbf[l], W, 1, e2);
            bf16* tmp = dz;
            dz = dz_next;
            dz_next = tmp;
        }
    }
}

extern "C" {

int mlp_create(int n_in, int width, int depth, uint64_t seed, me_mlp** out) {
    if (!out || n_in < 1 || n_in > MLP_KPAD || width < 64 || width % 64 || width > 1024 || depth < 1 || depth > 16)
        return me_fail(ME_EINVAL, "mlp_create: need 1 <= n_in <= 32, width a multiple of 64 up to 1024, depth 1..16");
    me_mlp* p = new (std::nothrow) me_mlp();
    if (!p) return me_fail(ME_ENOMEM, "host allocation");
    p->n_in = n_in;
    p->width = width;
    p->depth = depth;
    int64_t o = 0;
    int fi = n_in;
    for (int l = 0; l < depth; ++l) {
        p->L.w_off[l] = o;
        p->L.fan_in[l] = fi;
        o += (int64_t)width * fi;
        p->L.b_off[l] = o;
        o += width;
        fi = width;
    }
    p->wout_off = o;
    o += width;
    p->bout_off = o;
    o += 1;
    p->np = o;
    p->H.assign(depth, nullptr);
    p->Z.assign(depth, nullptr);
    p->wbf.assign(depth, nullptr);
    p->wbft.assign(depth, nullptr);
    p->wfr.assign(depth, nullptr);
    p->wtfr.assign(depth, nullptr);
    std::vector<float> h(o, 0.f);
    uint64_t st = seed;
    for (int l = 0; l < depth; ++l) {
        const double a = std::sqrt(6.0 / p->L.fan_in[l]);
        for (int64_t i = 0; i < (int64_t)width * p->L.fan_in[l]; ++i)
            h[p->L.w_off[l] + i] = (float)(a * (2.0 * ((splitmix(st) >> 11) * (1.0 / 9007199254740992.0)) - 1.0));
    }
    {
        const double a = std::sqrt(6.0 / width);
        for (int64_t i = 0; i < width; ++i)
            h[p->wout_off + i] = (float)(a * (2.0 * ((splitmix(st) >> 11) * (1.0 / 9007199254740992.0)) - 1.0));
    }
    auto bad = [&](hipError_t e) {
        if (e != hipSuccess) {
            mlp_free(p);
            return true;
        }
        return false;
    };
    if (bad(hipMalloc(&p->theta, o * sizeof(float))) || bad(hipMalloc(&p->grad, o * sizeof(float))) ||
        bad(hipMalloc(&p->m, o * sizeof(float))) || bad(hipMalloc(&p->v, o * sizeof(float))) ||
        bad(hipMalloc(&p->dwpart, (size_t)MLP_DW_SPLITS * width * width * sizeof(float))))
        return me_fail(ME_ENOMEM, "mlp_create: device allocation");
    for (int l = 0; l < depth; ++l) {
        const int ld = (l == 0) ? MLP_KPAD : p->L.fan_in[l];
        if (bad(hipMalloc(&p->wbf[l], (size_t)width * ld * sizeof(bf16))))
            return me_fail(ME_ENOMEM, "mlp_create: device allocation");
        if (l > 0 && bad(hipMalloc(&p->wbft[l], (size_t)width * p->L.fan_in[l] * sizeof(bf16))))
            return me_fail(ME_ENOMEM, "mlp_create: device allocation");
    }
    p->fused = (width == MLPF_W && depth <= FT_MAXDEPTH && n_in <= MLP_KPAD);
    p->fgrid = 0;
    if (p->fused) {
        for (int l = 0; l < depth; ++l) {
            const int ld = (l == 0) ? MLP_KPAD : p->L.fan_in[l];
            if (bad(hipMalloc(&p->wfr[l], (size_t)width * ld * sizeof(bf16))) ||
                (l > 0 && bad(hipMalloc(&p->wtfr[l], (size_t)width * ld * sizeof(bf16)))))
                return me_fail(ME_ENOMEM, "mlp_create: device allocation");
        }
        if (bad(hipMalloc(&p->d_wfr, depth * sizeof(bf16*))) ||
            bad(hipMemcpy(p->d_wfr, p->wfr.data(), depth * sizeof(bf16*), hipMemcpyHostToDevice)) ||
            bad(hipMalloc(&p->d_wtfr, depth * sizeof(bf16*))) ||
            bad(hipMemcpy(p->d_wtfr, p->wtfr.data(), depth * sizeof(bf16*), hipMemcpyHostToDevice)))
            return me_fail(ME_EDEVICE, "mlp_create: device allocation");
        int dev = 0, cus = 0, per = 0;
        if (bad(hipGetDevice(&dev)) || bad(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) ||
            bad(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, ft_kernel(depth), 256, 0)))
            return me_fail(ME_EDEVICE, "mlp_create: occupancy query");
        p->fgrid = cus * per;
        if (p->fgrid < 1) p->fused = false;
    }
    if (bad(hipMalloc(&p->d_wbf, depth * sizeof(bf16*))) ||
        bad(hipMemcpy(p->d_wbf, p->wbf.data(), depth * sizeof(bf16*), hipMemcpyHostToDevice)) ||
        bad(hipMalloc(&p->d_wbft, depth * sizeof(bf16*))) ||
        bad(hipMemcpy(p->d_wbft, p->wbft.data(), depth * sizeof(bf16*), hipMemcpyHostToDevice)) ||
        bad(hipMemcpy(p->theta, h.data(), o * sizeof(float), hipMemcpyHostToDevice)) ||
        bad(hipMemset(p->m, 0, o * sizeof(float))) || bad(hipMemset(p->v, 0, o * sizeof(float))) ||
        bad(hipMemset(p->grad, 0, o * sizeof(float))) || bad(refresh_bf16(p, nullptr)) ||
        bad(hipDeviceSynchronize()))
        return me_fail(ME_EDEVICE, "mlp_create: initialisation");
    p->step = 0;
    *out = p;
    return ME_OK;
}

int mlp_n_params(const me_mlp* p, int64_t* n) {
    if (!p || !n) return me_fail(ME_EINVAL, "null argument");
    *n = p->np;
    return ME_OK;
}

int mlp_dims(const me_mlp* p, int* n_in, int* width, int* depth) {
    if (!p) return me_fail(ME_EINVAL, "null network");
    if (n_in) *n_in = p->n_in;
    if (width) *width = p->width;
    if (depth) *depth = p->depth;
    return ME_OK;
}

int mlp_get_params(me_mlp* p, float* host, int64_t n) {
    if (!p || !host || n != p->np) return me_fail(ME_EINVAL, "mlp_get_params: null or wrong size");
    HCHK(hipDeviceSynchronize());
    HCHK(hipMemcpy(host, p->theta, n * sizeof(float), hipMemcpyDeviceToHost));
    return ME_OK;
}

int mlp_set_params(me_mlp* p, const float* host, int64_t n) {
    if (!p || !host || n != p->np) return me_fail(ME_EINVAL, "mlp_set_params: null or wrong size");
    HCHK(hipDeviceSynchronize());
    HCHK(hipMemcpy(p->theta, host, n * sizeof(float), hipMemcpyHostToDevice));
    HCHK(refresh_bf16(p, nullptr));
    HCHK(hipDeviceSynchronize());
    return ME_OK;
}

// The one-kernel inference, from features or from momenta; false: not this network's form.
static bool infer_fused(const me_mlp* p, const float* x, const double* mom, int64_t n, float* y, hipStream_t s) {
    if (p->width != MLPF_W || p->n_in > MLP_KPAD || p->depth > MLPF_MAXDEPTH) return false;
    mlpf_args a{};
    a.frag = p->d_wfr != nullptr;  // networks of the one-kernel step keep such copies
    for (int l = 0; l < p->depth; ++l) {
        a.w[l] = a.frag ? p->wfr[l] : p->wbf[l];
        a.b[l] = p->theta + p->L.b_off[l];
    }
    a.wout = p->theta + p->wout_off;
    a.bout = p->theta + p->bout_off;
    constexpr int rows = MLPF_TILE_ROWS;
    const dim3 grid((unsigned)((n + rows - 1) / rows));
    if (mom)
        hipLaunchKernelGGL((k_mlp_infer<rows, true>), grid, dim3(256), 0, s, nullptr, mom, n, p->n_in, p->depth, a, y);
    else
        hipLaunchKernelGGL((k_mlp_infer<rows, false>), grid, dim3(256), 0, s, x, nullptr, n, p->n_in, p->depth, a, y);
    return true;
}

// The layered inference in chunks; prep(o, m) fills the input rows of samples o .. o + m - 1.
extern "C++" template <class Prep>
static int forward_layers(me_mlp* p, int64_t n, float* y, hipStream_t s, Prep&& prep) {
    const int64_t chunk = 1 << 16;
    int rc = ensure_acts(p, std::min<int64_t>(n, chunk));
    if (rc != ME_OK) return rc;
    for (int64_t o = 0; o < n; o += chunk) {
        const int64_t m = std::min<int64_t>(chunk, n - o);
        prep(o, m);
        forward(p, m, false, s);
        HCHK(hipMemcpyAsync(y + o, p->y, m * sizeof(float), hipMemcpyDeviceToDevice, s));
    }
    HCHK(hipGetLastError());
    return ME_OK;
}

int mlp_forward(me_mlp* p, const float* x, int64_t n, float* y, void* stream) {
    if (!p || n < 0) return me_fail(ME_EINVAL, "mlp_forward: null or negative n");
    if (n == 0) return ME_OK;
    if (!x || !y) return me_fail(ME_EINVAL, "mlp_forward: null buffer");
    hipStream_t s = (hipStream_t)stream;
    if (infer_fused(p, x, nullptr, n, y, s)) {
        HCHK(hipGetLastError());
        return ME_OK;
    }
    return forward_layers(p, n, y, s, [&](int64_t o, int64_t m) {
        hipLaunchKernelGGL(k_prep_input, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, s, x + o * p->n_in, nullptr, m,
                           p->n_in, p->X);
    });
}

// Batch buffers of the fused step (grow on the first call with a larger batch;
// that call synchronises the device).
static int ensure_fused(me_mlp* p, int64_t M) {
    if (M <= p->fcap) return ME_OK;
    HCHK(hipDeviceSynchronize());
    auto f = [](void* q) {
        if (q) (void)hipFree(q);
    };
    f(p->XT);
    f(p->HTb);
    f(p->DZTb);
    f(p->flossp);
    f(p->fopart);
    f(p->fbar);
    p->fbar = nullptr;
    p->XT = p->HTb = p->DZTb = nullptr;
    p->flossp = p->fopart = nullptr;
    p->fcap = 0;
    const int64_t W = p->width;
    HCHK(hipMalloc(&p->XT, MLP_KPAD * M * sizeof(bf16)));
    HCHK(hipMalloc(&p->HTb, p->depth * W * M * sizeof(bf16)));
    HCHK(hipMalloc(&p->DZTb, p->depth * W * M * sizeof(bf16)));
    HCHK(hipMalloc(&p->flossp, p->fgrid * sizeof(float)));
    HCHK(hipMalloc(&p->fopart, (W + 1) * (M / FT_R) * sizeof(float)));
    HCHK(hipMalloc(&p->fbar, 64 * sizeof(unsigned)));
    HCHK(hipMemset(p->fbar, 0, 64 * sizeof(unsigned)));
    p->fcap = M;
    return ME_OK;
}

static bool fused_applies(const me_mlp* p, int64_t n) {
    return p->fused && n >= FT_S * 32 && n % (FT_S * 32) == 0 && n <= (int64_t)1 << 24;
}

// nsteps training steps (grad_out == nullptr; rates lr_dev[nsteps] on the
// device, or lr for a single step) or the gradient only, as one launch of the
// fused cooperative kernel.
static int fused_step(me_mlp* p, const float* x, const float* t, const int32_t* idx, int64_t n, int64_t nsteps,
                      float lr, const float* lr_dev, float* loss, float* grad_out, hipStream_t s) {
    int rc = ensure_fused(p, n);
    if (rc != ME_OK) return rc;
    ft_args a{};
    a.x = x;
    a.t = t;
    a.idx = idx;
    a.M = n;
    a.n_in = p->n_in;
    a.depth = p->depth;
    for (int l = 0; l < p->depth; ++l) {
        a.wfr[l] = p->wfr[l];
        a.wtfr[l] = p->wtfr[l];
        a.wbf[l] = p->wbf[l];
        a.wbft[l] = p->wbft[l];
        a.HT[l] = p->HTb + (int64_t)l * p->width * n;
        a.DZT[l] = p->DZTb + (int64_t)l * p->width * n;
    }
    a.theta = p->theta;
    a.m = p->m;
    a.v = p->v;
    a.grad_out = grad_out;
    a.L = p->L;
    a.wout_off = p->wout_off;
    a.bout_off = p->bout_off;
    a.np = p->np;
    a.XT = p->XT;
    a.opart = p->fopart;
    a.lossp = p->flossp;
    a.bar = p->fbar;
    a.loss = loss;
    a.nsteps = (int)nsteps;
    a.step0 = p->step;
    a.lrs = lr_dev;
    a.lr = lr;
    if (!grad_out) {
        a.c1 = 1.f - std::pow(0.9f, (float)(p->step + 1));
        a.c2 = 1.f - std::pow(0.999f, (float)(p->step + 1));
        p->step += nsteps;
    } else {
        a.c1 = a.c2 = 1.f;
    }
    void* args[] = {&a};
    HCHK(hipLaunchCooperativeKernel((const void*)ft_kernel(p->depth), dim3((unsigned)p->fgrid), dim3(256), args, 0, s));
    return ME_OK;
}

static int grad_common(me_mlp* p, const float* x, const float* t, const int32_t* idx, int64_t n, float* loss,
                       hipStream_t s) {
    if (!p || !x || !t || n <= 0 || n % 64) return me_fail(ME_EINVAL, "batch must be a positive multiple of 64");
    int rc = ensure_acts(p, n);
    if (rc != ME_OK) return rc;
    hipLaunchKernelGGL(k_prep_input, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, x, idx, n, p->n_in, p->X);
    forward(p, n, true, s);
    backward(p, t, idx, n, loss, s);
    HCHK(hipGetLastError());
    return ME_OK;
}

int mlp_set_fused_step(me_mlp* p, int on) {
    if (!p) return me_fail(ME_EINVAL, "null network");
    if (on && !(p->width == MLPF_W && p->depth <= FT_MAXDEPTH && p->n_in <= MLP_KPAD && p->fgrid > 0))
        return me_fail(ME_ESTATE, "the fused step needs width 256, depth <= 4 and n_in <= 32");
    p->fused = on != 0;
    return ME_OK;
}

int mlp_backward(me_mlp* p, const float* x, const float* t, const int32_t* idx, int64_t n, float* grad_dev,
                 float* loss_dev, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    if (p && x && t && grad_dev && fused_applies(p, n))
        return fused_step(p, x, t, idx, n, 1, 0.f, nullptr, loss_dev, grad_dev, s);
    int rc = grad_common(p, x, t, idx, n, loss_dev, s);
    if (rc != ME_OK) return rc;
    if (grad_dev) HCHK(hipMemcpyAsync(grad_dev, p->grad, p->np * sizeof(float), hipMemcpyDeviceToDevice, s));
    return ME_OK;
}

int mlp_train_step(me_mlp* p, const float* x, const float* t, const int32_t* idx, int64_t n, float lr,
                   float* loss_dev, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    if (p && x && t && fused_applies(p, n)) return fused_step(p, x, t, idx, n, 1, lr, nullptr, loss_dev, nullptr, s);
    int rc = grad_common(p, x, t, idx, n, loss_dev, s);
    if (rc != ME_OK) return rc;
    p->step += 1;
    const float c1 = 1.f - std::pow(0.9f, (float)p->step), c2 = 1.f - std::pow(0.999f, (float)p->step);
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((p->np + 255) / 256)), dim3(256), 0, s, p->theta, p->m, p->v, p->grad,
                       p->np, lr, c1, c2, p->L, p->depth, p->width, p->d_wbf, p->d_wbft, p->d_wfr, p->d_wtfr);
    HCHK(hipGetLastError());
    return ME_OK;
}

int mlp_train_steps(me_mlp* p, const float* x, const float* t, const int32_t* idx, int64_t n, int64_t nsteps,
                    const float* lr_dev, float* loss_dev, void* stream) {
    if (!p || !x || !t || !lr_dev || nsteps < 0 || nsteps > INT32_MAX)
        return me_fail(ME_EINVAL, "mlp_train_steps: null argument or bad step count");
    if (nsteps == 0) return ME_OK;
    hipStream_t s = (hipStream_t)stream;
    if (fused_applies(p, n)) return fused_step(p, x, t, idx, n, nsteps, 0.f, lr_dev, loss_dev, nullptr, s);
    // layered path: one step at a time, rates read back first
    std::vector<float> lr((size_t)nsteps);
    HCHK(hipStreamSynchronize(s));
    HCHK(hipMemcpy(lr.data(), lr_dev, nsteps * sizeof(float), hipMemcpyDeviceToHost));
    for (int64_t st = 0; st < nsteps; ++st) {
        const int32_t* ix = idx ? idx + st * n : nullptr;
        const float* xs = idx ? x : x + st * n * p->n_in;
        const float* ts = idx ? t : t + st * n;
        const int rc = mlp_train_step(p, xs, ts, ix, n, lr[st], loss_dev ? loss_dev + st : nullptr, stream);
        if (rc != ME_OK) return rc;
    }
    return ME_OK;
}

int mlp_free(me_mlp* p) {
    if (!p) return ME_OK;
    (void)hipDeviceSynchronize();
    free_acts(p);
    auto f = [](void* q) {
        if (q) (void)hipFree(q);
    };
    f(p->theta);
    f(p->grad);
    f(p->dwpart);
    f(p->m);
    f(p->v);
    for (auto q : p->wbf) f(q);
    for (auto q : p->wbft) f(q);
    f(p->d_wbf);
    f(p->d_wbft);
    for (auto q : p->wfr) f(q);
    for (auto q : p->wtfr) f(q);
    f(p->d_wfr);
    f(p->d_wtfr);
    f(p->XT);
    f(p->HTb);
    f(p->DZTb);
    f(p->flossp);
    f(p->fopart);
    f(p->fbar);
    delete p;
    return ME_OK;
}

int me_features(const double* momenta, int64_t n, int npart, float* x, void* stream) {
    if (n < 0 || npart < 2 || npart > 8) return me_fail(ME_EINVAL, "me_features: bad size");
    if (n == 0) return ME_OK;
    if (!momenta || !x) return me_fail(ME_EINVAL, "me_features: null buffer");
    me_each_launch(n, FEAT_EV, 256, [&](int64_t first, unsigned blocks) {
        hipLaunchKernelGGL(k_features, dim3(blocks), dim3(256), 0, (hipStream_t)stream, momenta + first * 4 * npart,
                           n - first, npart, x + first * 4 * npart);
    });
    HCHK(hipGetLastError());
    return ME_OK;
}

}  // extern "C"

// helpers for the unweighting driver in me_unweight.hip
int mlp_forward_momenta(me_mlp* p, const double* momenta, int64_t n, float* y, hipStream_t s) {
    if (infer_fused(p, nullptr, momenta, n, y, s)) {
        HCHK(hipGetLastError());
        return ME_OK;
    }
    return forward_layers(p, n, y, s, [&](int64_t o, int64_t m) {
        hipLaunchKernelGGL(k_prep_momenta, dim3((unsigned)((m + FEAT_EV - 1) / FEAT_EV)), dim3(256), 0, s,
                           momenta + o * p->n_in, m, p->n_in, p->X);
    });
}
int mlp_n_in(const me_mlp* p) { return p->n_in; }
