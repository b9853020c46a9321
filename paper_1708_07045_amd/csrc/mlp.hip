// Learned importance-sampling proposal over ligand configurations: a 3-layer
// SiLU network on gfx950 with BF16 MFMA products and FP32 accumulation,
// trained by its own forward/backward kernels and Adam, plus the defensive
// mixture proposal and its inverse-CDF sampler.
//
// The BF16 network runs in three kernels: k_net takes a tile of rows through
// the whole forward pass (and, in training, back through the data gradients)
// with its activations in LDS and registers, k_wgrad forms the weight
// gradients, k_update makes the Adam step and the BF16 working copies of the
// weights.  MFMA 16 x 16 x 16 (v_mfma_f32_16x16x16_bf16), per 64-lane
// wavefront:
//   A[i][k]: lane = i + 16*(k/4), element k%4      (row i, 4 consecutive k)
//   B[k][j]: lane = j + 16*(k/4), element k%4      (column j, 4 consecutive k)
//   D[i][j]: lane = j + 16*(i/4), element i%4
// A second implementation, one kernel per step of the textbook pass, keeps
// operands and activations in FP32 (GEMMs on v_mfma_f32_16x16x4_f32, A[i][k] at
// lane i + 16 k and B[k][j] at lane j + 16 k of each 16 x 16 x 4 step, D as
// above): the same network in FP32 throughout, for checking gradients against
// an FP64 reference to FP32 rounding.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/fftdg.h"

namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int KP = 64;  // padded input width of the first layer

__device__ __forceinline__ uint16_t f2bf(float f) {  // round to nearest even
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)(u >> 16);  // inf / nan
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ float silu(float z) { return z / (1.0f + expf(-z)); }
__device__ __forceinline__ float dsilu(float z) {
    const float s = 1.0f / (1.0f + expf(-z));
    return s * (1.0f + z * (1.0f - s));
}

// ------------------------------------------------- BF16 network
// Working copy of a weight matrix as B operand [N][K], K a multiple of 32, in
// the order the wavefronts read it: per 16 columns and 32 k one block of 512
// elements, lane (n % 16) + 16 ((k % 16) / 4) holding 8 of them (two MFMA
// steps), so a fragment is one 16-byte load a lane and 1 KB contiguous.
__host__ __device__ __forceinline__ int64_t frag_index(int n, int k, int K) {
    return ((int64_t)(n >> 4) * (K >> 5) + (k >> 5)) * 512 + ((n & 15) + 16 * ((k & 15) >> 2)) * 8 + ((k >> 4) & 1) * 4 +
           (k & 3);
}

struct NetArgs {
    const float *X;            // rows [.][n_in]
    const int32_t *idx;        // rows of X taken (nullptr: the first ones)
    int n_in, H, B;            // inputs, width, rows
    const uint16_t *W1, *W2, *W3, *W2t, *W3t, *W4;  // working copies (frag_index; W4 plain)
    const float *b1, *b2, *b3, *b4;
    int skip_col;
    float skip_scale;
    float *y;                  // forward: output per row
    // training
    const float *t, *w;        // target and loss weight per row of X
    const float *wsum;         // sum of the batch's weights (nullptr: each block forms it)
    int ld;                    // row stride of the transposed arrays (padded rows)
    uint16_t *A0t, *H1t, *H2t, *dZ1t, *dZ2t, *dZ3t;  // [features][ld], rows in batch_pos order
    uint16_t *H3t;             // [H][ld]
    float *dZf;                // FP32 dZ of layers 1, 2, 3, [3][H][ld]
    float *dy, *lrow;          // dL/dy and weighted squared error per row [ld]
};

// Place of batch row b in a transposed operand of the weight gradients:
// within 32 rows, rows 4 q .. and 16 + 4 q .. together, so that lane group q
// loads its rows of two MFMA steps as 16 bytes.
__host__ __device__ __forceinline__ int batch_pos(int b) {
    return (b & ~31) + 8 * ((b & 15) >> 2) + 4 * ((b >> 4) & 1) + (b & 3);
}

// Sum of the batch's loss weights: 256 strided sums, added pairwise (128
// apart, 64 apart, then within the first wavefront).  weight_terms forms the
// strided sums; weight_sum, after a barrier, gives the total to thread 0.
__device__ __forceinline__ void weight_terms(const float *__restrict__ w, const int32_t *__restrict__ idx, int B,
                                             float *sh) {
    if (threadIdx.x < 256) {
        float a = 0.f;
        for (int b = threadIdx.x; b < B; b += 256) a += w[idx ? idx[b] : b];
        sh[threadIdx.x] = a;
    }
}
__device__ __forceinline__ float weight_sum(const float *sh) {  // by the first wavefront
    const int t = threadIdx.x;
    float v = (sh[t] + sh[t + 128]) + (sh[t + 64] + sh[t + 192]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
    return v;
}
__global__ __launch_bounds__(256) void k_wsum(const float *__restrict__ w, const int32_t *__restrict__ idx, int B,
                                              float *__restrict__ out) {
    __shared__ float sh[256];
    weight_terms(w, idx, B, sh);
    __syncthreads();
    if (threadIdx.x < 64) {
        const float W = weight_sum(sh);
        if (threadIdx.x == 0) out[0] = W;
    }
}

// 16 MT rows through the network, 8 wavefronts.  Wavefront w has the columns
// of the 16-wide tiles w, w + 8, ... (NTW of them); the activations of a layer
// are the LDS tile `act`, replaced once every wavefront is done with it.
// TRAIN (MT = 1): keeps the pre-activations in registers, goes back through
// the data gradients, and leaves activations and gradients transposed (a
// lane's four rows are contiguous there) for k_wgrad.  Bound: latency of three (five) dependent
// layers, each a wavefront's weights (16 KB of 1 KB loads at width 256) from
// L2; one kernel a batch instead of a launch and a round trip through
// memory per step: 20000 rows forward (width 256) 2.9 ms in blocks of 512 ->
// 25 us; a training step of 512 rows 600 us in 31 launches -> 37 us in 3.
template <int NTW, int MT, bool TRAIN, bool FULL>
__global__ __launch_bounds__(512) void k_net(NetArgs a) {
    constexpr int HM = 128 * NTW, LDA = HM + 8;  // rows 16 bytes apart modulo the banks
    static_assert(!TRAIN || MT == 1, "training tiles are 16 rows");
    __shared__ __align__(16) uint16_t act[16 * MT][LDA];
    __shared__ __align__(16) float s_dy[16], s_w[TRAIN ? 256 : 1], s_w4[TRAIN ? HM : 1];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, c16 = lane & 15, q = lane >> 4;
    const int H = a.H, NT = H >> 4, b0 = (int)blockIdx.x * 16 * MT;
    for (int e = threadIdx.x; e < 16 * MT * KP; e += 512) {
        const int k = e / (16 * MT), r = e - k * (16 * MT), b = b0 + r;
        float v = 0.f;
        if (b < a.B && k < a.n_in) v = a.X[(size_t)(a.idx ? a.idx[b] : b) * a.n_in + k];
        const uint16_t h = f2bf(v);
        act[r][k] = h;
        if (TRAIN) a.A0t[(size_t)k * a.ld + batch_pos(b)] = h;
    }
    if constexpr (TRAIN) {
        if (!a.wsum) weight_terms(a.w, a.idx, a.B, s_w);
        for (int k = threadIdx.x; k < H; k += 512) s_w4[k] = bf2f(a.W4[k]);
    }
    __syncthreads();
    f32x4 acc[MT][NTW];
    struct alignas(16) Frag {
        bf16x4 lo, hi;
    };
    // one slice of 32 k: the lane's fragments of the wavefront's tiles, and
    // their two MFMA steps (k ascending)
    auto load = [&](Frag *f, const uint16_t *__restrict__ W, int kp, int KB) {
#pragma unroll
        for (int t = 0; t < NTW; ++t) {
            const int nt = FULL ? wave + 8 * t : min(wave + 8 * t, NT - 1);  // a tile past the last: computed, not kept
            __builtin_memcpy(&f[t], W + ((size_t)nt * KB + kp) * 512 + lane * 8, 16);
        }
    };
    auto step = [&](const Frag *f, int kp) {
        bf16x4 x0[MT], x1[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            x0[m] = *reinterpret_cast<const bf16x4 *>(&act[16 * m + c16][32 * kp + 4 * q]);
            x1[m] = *reinterpret_cast<const bf16x4 *>(&act[16 * m + c16][32 * kp + 16 + 4 * q]);
        }
#pragma unroll
        for (int t = 0; t < NTW; ++t)
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x0[m], f[t].lo, acc[m][t], 0, 0, 0);
                acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x1[m], f[t].hi, acc[m][t], 0, 0, 0);
            }
    };
    // acc = act W^T over KB slices of 32 k (KB even).  Every load of UN
    // slices is issued before the first is used.
    auto product = [&](auto kbc, const uint16_t *__restrict__ W, int KBr) {
        constexpr int KBC = decltype(kbc)::value;  // 0: KBr slices
        constexpr int UN = KBC == 0 ? 2 : (KBC * NTW <= 16 ? KBC : (NTW < 8 ? 4 : (TRAIN ? 1 : 2)));
        const int KB = KBC ? KBC : KBr;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int t = 0; t < NTW; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        Frag f[UN][NTW];
#pragma unroll
        for (int u = 0; u < UN; ++u) load(f[u], W, u, KB);
#pragma unroll 1
        for (int k0 = 0; k0 < KB; k0 += UN) {
            Frag g[UN][NTW];
            if (UN != KBC) {
#pragma unroll
                for (int u = 0; u < UN; ++u) load(g[u], W, min(k0 + UN, KB - UN) + u, KB);
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) step(f[u], k0 + u);
            if (UN != KBC) {
#pragma unroll
                for (int u = 0; u < UN; ++u)
#pragma unroll
                    for (int t = 0; t < NTW; ++t) f[u][t] = g[u][t];
            }
        }
    };
    constexpr int KH = FULL ? HM / 32 : 0;  // slices of a hidden layer, where known
    const std::integral_constant<int, KH> hid{};
    const std::integral_constant<int, KP / 32> inp{};
    // the lane's values of a tile column (rows 4 q .. 4 q + 3) into the act
    // tile, and transposed to device memory
    auto put = [&](int m, int n, const float *v, uint16_t *__restrict__ tr, bool perm) {
        struct alignas(8) {
            uint16_t h[4];
        } o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o.h[e] = f2bf(v[e]);
            act[16 * m + 4 * q + e][n] = o.h[e];
        }
        if (TRAIN) __builtin_memcpy(tr + (size_t)n * a.ld + (perm ? batch_pos(b0 + 4 * q) : b0 + 4 * q), &o, 8);
    };
    float Z[TRAIN ? 3 : 1][NTW][4];
    auto layer = [&](auto lc, auto kbc, const uint16_t *__restrict__ W, const float *__restrict__ bias,
                     uint16_t *__restrict__ tr) {
        constexpr int l = decltype(lc)::value;
        product(kbc, W, H >> 5);
        __syncthreads();  // every wavefront has read the old activations
#pragma unroll
        for (int t = 0; t < NTW; ++t) {
            const int n = 16 * (wave + 8 * t) + c16;
            if (!FULL && n >= H) continue;
            const float bn = bias[n];
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                float h[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float z = acc[m][t][e] + bn;
                    if (TRAIN) Z[l][t][e] = z;
                    h[e] = silu(z);
                }
                put(m, n, h, tr, l < 2);
            }
        }
        __syncthreads();
    };
    layer(std::integral_constant<int, 0>{}, inp, a.W1, a.b1, TRAIN ? a.H1t : nullptr);
    layer(std::integral_constant<int, TRAIN ? 1 : 0>{}, hid, a.W2, a.b2, TRAIN ? a.H2t : nullptr);
    layer(std::integral_constant<int, TRAIN ? 2 : 0>{}, hid, a.W3, a.b3, TRAIN ? a.H3t : nullptr);
    auto output = [&](int r, float s, float W) {  // row r of the block, s = H3 . W4; W: the batch's weights
        const int b = b0 + r;
        float dy = 0.f, ls = 0.f;
        if (b < a.B) {
            const size_t i = a.idx ? a.idx[b] : b;
            const float sk = a.skip_col >= 0 ? a.skip_scale * a.X[i * a.n_in + a.skip_col] : 0.f;
            const float y = s + a.b4[0] + sk;
            if (!TRAIN) a.y[b] = y;
            if (TRAIN) {
                const float d = y - a.t[i];
                dy = 2.f * a.w[i] * d / W;
                ls = a.w[i] * d * d;
            }
        }
        if (TRAIN) {
            s_dy[r] = dy;
            a.dy[b] = dy;
            a.lrow[b] = ls;
            if (b == 0) a.lrow[a.ld] = W;
        }
    };
    if constexpr (!TRAIN) {  // 32 lanes a row
        for (int r0 = 0; r0 < 16 * MT; r0 += 16) {
            const int r = r0 + ((int)threadIdx.x >> 5), l = threadIdx.x & 31;
            float s = 0.f;
            for (int k = l; k < H; k += 32) s += bf2f(act[r][k]) * bf2f(a.W4[k]);
#pragma unroll
            for (int off = 16; off > 0; off >>= 1) s += __shfl_xor(s, off);
            if (l == 0) output(r, s, 1.f);
        }
    } else {
        // one lane a row, in order of k: Adam divides a gradient by its own
        // size, so training keeps every sum in one fixed order
        if (threadIdx.x < 64) {
            float W = a.wsum ? a.wsum[0] : weight_sum(s_w);
            W = __shfl(W, 0);
            if (threadIdx.x < 16) {
                float s = 0.f;
                for (int k = 0; k < H; k += 8) {
                    const uint4 h = *reinterpret_cast<const uint4 *>(&act[threadIdx.x][k]);
                    const float4 u = *reinterpret_cast<const float4 *>(&s_w4[k]),
                                 v = *reinterpret_cast<const float4 *>(&s_w4[k + 4]);
                    auto two = [&](uint32_t x, float p, float q2) {
                        s += bf2f((uint16_t)(x & 0xffffu)) * p;
                        s += bf2f((uint16_t)(x >> 16)) * q2;
                    };
                    two(h.x, u.x, u.y), two(h.y, u.z, u.w), two(h.z, v.x, v.y), two(h.w, v.z, v.w);
                }
                output(threadIdx.x, s, W);
            }
        }
        __syncthreads();
        auto back = [&](auto lc, uint16_t *__restrict__ tr) {
            constexpr int l = decltype(lc)::value;
            // acc: dH of layer l (l < 2); the output's share for l = 2
            float *__restrict__ zf = a.dZf + (size_t)l * H * a.ld;
#pragma unroll
            for (int t = 0; t < NTW; ++t) {
                const int n = 16 * (wave + 8 * t) + c16;
                if (!FULL && n >= H) continue;
                struct alignas(16) {
                    float v[4];
                } o;
                const float w4 = l == 2 ? s_w4[n] : 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float g = l == 2 ? s_dy[4 * q + e] * w4 : acc[0][t][e];
                    o.v[e] = b0 + 4 * q + e < a.B ? g * dsilu(Z[l][t][e]) : 0.f;
                }
                __builtin_memcpy(zf + (size_t)n * a.ld + b0 + 4 * q, &o, 16);
                put(0, n, o.v, tr, true);
            }
            if (l > 0) __syncthreads();
        };
        back(std::integral_constant<int, 2>{}, a.dZ3t);
        product(hid, a.W3t, H >> 5);
        __syncthreads();
        back(std::integral_constant<int, TRAIN ? 1 : 0>{}, a.dZ2t);
        product(hid, a.W2t, H >> 5);
        __syncthreads();
        back(std::integral_constant<int, 0>{}, a.dZ1t);
    }
}

struct GradArgs {
    int H, n_in, ld, B;
    const uint16_t *A0t, *H1t, *H2t, *dZ1t, *dZ2t, *dZ3t, *H3t;
    const float *dZf, *dy, *lrow;
    float *gW1, *gb1, *gW2, *gb2, *gW3, *gb3, *gW4, *gb4, *loss;
};
// Weight gradients dZ^T H over the batch, a 16 x 32 tile a wavefront, and the
// sums over the batch of the biases, the output layer and the loss, 16
// columns a block: the columns are staged through LDS by the whole block and
// added up by one lane each.  Every sum runs over the batch in one order, row
// by row (slice by slice of 16 in the products): what limits the kernel is
// that chain, 32 MFMA or 512 additions for a batch of 512 (8 us; one lane a
// column straight from memory took 110).
__global__ __launch_bounds__(256) void k_wgrad(GradArgs a) {
    constexpr int RB = 512;  // rows staged at once
    __shared__ __align__(16) float col[16][RB + 4];
    __shared__ __align__(16) float sdy[RB];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, r16 = lane & 15, q = lane >> 4;
    const int H = a.H, nm = H / 16, n1 = nm * (KP / 32), n2 = nm * (H / 32), tb = (n1 + 2 * n2 + 3) / 4;
    if ((int)blockIdx.x >= tb) {
        const int id = (int)blockIdx.x - tb;  // columns 16 id ..: db1, db2, db3, dW4; then db4 and the loss
        if (16 * id >= 4 * H) {
            const bool ls = id > H / 4;
            const float *src = ls ? a.lrow : a.dy;
            if (ls) {
                float l = 0.f;
                for (int b = threadIdx.x; b < a.B; b += 256) l += src[b];
                sdy[threadIdx.x] = l;
                __syncthreads();
                for (int s = 128; s > 0; s >>= 1) {
                    if ((int)threadIdx.x < s) sdy[threadIdx.x] += sdy[threadIdx.x + s];
                    __syncthreads();
                }
                if (threadIdx.x == 0) a.loss[0] = sdy[0] / a.lrow[a.ld];
                return;
            }
            float s = 0.f;
            for (int b0 = 0; b0 < a.B; b0 += RB) {
                __syncthreads();
                for (int r = threadIdx.x; r < RB; r += 256) sdy[r] = b0 + r < a.B ? src[b0 + r] : 0.f;
                __syncthreads();
                if (threadIdx.x == 0)
                    for (int r = 0; r < min(RB, a.B - b0); ++r) s += sdy[r];
            }
            if (threadIdx.x == 0) a.gb4[0] = s;
            return;
        }
        const int layer = 16 * id / H, n0 = 16 * id - layer * H;  // 16 divides H
        float s = 0.f;
        for (int b0 = 0; b0 < a.B; b0 += RB) {
            const int nb = min(RB, a.ld - b0);  // staged rows, a multiple of 64
            __syncthreads();
            for (int e = threadIdx.x; e < 16 * (nb / 4); e += 256) {
                const int c = e / (nb / 4), r = 4 * (e - c * (nb / 4));
                float4 v;
                if (layer < 3) {
                    v = *reinterpret_cast<const float4 *>(a.dZf + ((size_t)layer * H + n0 + c) * a.ld + b0 + r);
                } else {
                    uint16_t h[4];
                    __builtin_memcpy(h, a.H3t + (size_t)(n0 + c) * a.ld + b0 + r, 8);
                    v = float4{bf2f(h[0]), bf2f(h[1]), bf2f(h[2]), bf2f(h[3])};
                }
                *reinterpret_cast<float4 *>(&col[c][r]) = v;
            }
            if (layer == 3)
                for (int r = threadIdx.x; r < nb; r += 256) sdy[r] = a.dy[b0 + r];
            __syncthreads();
            if (threadIdx.x < 16) {
                const int rows = min(nb, a.B - b0);
                int r = 0;
                if (layer < 3) {
                    for (; r + 16 <= rows; r += 16) {
                        float4 v[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const float4 *>(&col[threadIdx.x][r + 4 * u]);
#pragma unroll
                        for (int u = 0; u < 4; ++u) s += v[u].x, s += v[u].y, s += v[u].z, s += v[u].w;
                    }
                    for (; r < rows; ++r) s += col[threadIdx.x][r];
                } else {
                    for (; r + 16 <= rows; r += 16) {
                        float4 v[4], d[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            v[u] = *reinterpret_cast<const float4 *>(&col[threadIdx.x][r + 4 * u]);
                            d[u] = *reinterpret_cast<const float4 *>(&sdy[r + 4 * u]);
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            s += d[u].x * v[u].x;
                            s += d[u].y * v[u].y;
                            s += d[u].z * v[u].z;
                            s += d[u].w * v[u].w;
                        }
                    }
                    for (; r < rows; ++r) s += sdy[r] * col[threadIdx.x][r];
                }
            }
        }
        if (threadIdx.x < 16) {
            float *o = layer == 0 ? a.gb1 : layer == 1 ? a.gb2 : layer == 2 ? a.gb3 : a.gW4;
            o[n0 + threadIdx.x] = s;
        }
        return;
    }
    int id = 4 * (int)blockIdx.x + wave;
    if (id >= n1 + 2 * n2) return;
    const uint16_t *A, *B;
    float *C;
    int ldc, bw;  // columns of C, tiles across
    if (id < n1) A = a.dZ1t, B = a.A0t, C = a.gW1, ldc = a.n_in, bw = KP / 32;
    else if (id < n1 + n2) id -= n1, A = a.dZ2t, B = a.H1t, C = a.gW2, ldc = H, bw = H / 32;
    else id -= n1 + n2, A = a.dZ3t, B = a.H2t, C = a.gW3, ldc = H, bw = H / 32;
    const int m0 = 16 * (id / bw), n0 = 32 * (id % bw);
    if (n0 >= ldc) return;  // padded inputs only
    struct alignas(16) Frag {
        bf16x4 lo, hi;
    };
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    const int nkb = a.ld / 32;  // slices of 32 rows, an even number
    const uint16_t *pa = A + (size_t)(m0 + r16) * a.ld + 8 * q, *pb = B + (size_t)(n0 + r16) * a.ld + 8 * q;
    auto slices = [&](auto uc, int kb) {
        constexpr int U = decltype(uc)::value;  // loads of U slices in flight
        Frag fa[U], fb[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            __builtin_memcpy(&fa[u], pa + 32 * (kb + u), 16);
#pragma unroll
            for (int j = 0; j < 2; ++j) __builtin_memcpy(&fb[u][j], pb + (size_t)16 * j * a.ld + 32 * (kb + u), 16);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fa[u].lo, fb[u][j].lo, acc[j], 0, 0, 0);
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fa[u].hi, fb[u][j].hi, acc[j], 0, 0, 0);
            }
    };
    int kb = 0;
    for (; kb + 8 <= nkb; kb += 8) slices(std::integral_constant<int, 8>{}, kb);
    for (; kb < nkb; kb += 2) slices(std::integral_constant<int, 2>{}, kb);
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int c = n0 + 16 * j + r16;
            if (c < ldc) C[(size_t)(m0 + 4 * q + e) * ldc + c] = acc[j][e];
        }
}

struct UpdateArgs {
    float *p;
    const float *g;
    float *m, *v;
    int n, n_in, H;
    float lr, b1, b2, eps, c1, c2;
    uint16_t *W1, *W2, *W3, *W2t, *W3t, *W4;
};
// Adam on the flat FP32 master parameters (ADAM), and the BF16 working copies.
template <bool ADAM>
__global__ __launch_bounds__(256) void k_update(UpdateArgs a) {
    int i = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (i >= a.n) return;
    float p = a.p[i];
    if (ADAM) {
        const float gi = a.g[i];
        const float mi = a.b1 * a.m[i] + (1.f - a.b1) * gi;
        const float vi = a.b2 * a.v[i] + (1.f - a.b2) * gi * gi;
        a.m[i] = mi;
        a.v[i] = vi;
        p -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
        a.p[i] = p;
    }
    // flat layout W1, b1, W2, b2, W3, b3, W4, b4
    const uint16_t h = f2bf(p);
    const int H = a.H, F = a.n_in;
    if (i < H * F) {
        a.W1[frag_index(i / F, i % F, KP)] = h;
        return;
    }
    i -= H * F + H;
    if (i < 0) return;
    if (i < H * H) {
        a.W2[frag_index(i / H, i % H, H)] = h;
        a.W2t[frag_index(i % H, i / H, H)] = h;
        return;
    }
    i -= H * H + H;
    if (i < 0) return;
    if (i < H * H) {
        a.W3[frag_index(i / H, i % H, H)] = h;
        a.W3t[frag_index(i % H, i / H, H)] = h;
        return;
    }
    i -= H * H + H;
    if (i >= 0 && i < H) a.W4[i] = h;
}

// ------------------------------------------------- FP32 network, step by step
// C[M][N] = A[M][K] * B[N][K]^T, FP32 operands and accumulation.
// M, N multiples of 64; K multiple of 16; lda, ldb multiples of 4.
// mode 0: C (+ bias[n] if bias) -> Cout (fp32, ldc)
// mode 1: Z = C + bias[n] -> Cout; H = silu(Z) -> Hout (ldh)
__global__ __launch_bounds__(256) void k_gemm(const float *__restrict__ A, int lda, const float *__restrict__ B, int ldb,
                                              int K, const float *__restrict__ bias, int mode,
                                              float *__restrict__ Cout, int ldc, float *__restrict__ Hout, int ldh) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int m0 = blockIdx.y * 64 + (wave >> 1) * 32, n0 = blockIdx.x * 64 + (wave & 1) * 32;
    const int r = lane & 15;
    f32x4 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < K; k += 16) {
        // four 16 x 16 x 4 steps; lane (r, q = lane / 16) supplies k + 4 s + q
        const int q = lane >> 4;
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
            float fa[2], fb[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                fa[t] = A[(size_t)(m0 + t * 16 + r) * lda + k + 4 * s4 + q];
                fb[t] = B[(size_t)(n0 + t * 16 + r) * ldb + k + 4 * s4 + q];
            }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[a], fb[b], acc[a][b], 0, 0, 0);
        }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = m0 + a * 16 + (lane >> 4) * 4 + e;
                const int j = n0 + b * 16 + (lane & 15);
                float v = acc[a][b][e];
                if (bias) v += bias[j];
                Cout[(size_t)i * ldc + j] = v;
                if (mode == 1) Hout[(size_t)i * ldh + j] = silu(v);
            }
}

// rows idx[b] of X [N][n_in] (fp32) -> A0 [Bp][KP] zero padded
__global__ void k_gather(const float *__restrict__ X, int n_in, const int32_t *__restrict__ idx, int B, int Bp,
                         float *__restrict__ A0) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= Bp * KP) return;
    const int b = e / KP, k = e - b * KP;
    float v = 0.f;
    if (b < B && k < n_in) v = X[(size_t)(idx ? idx[b] : b) * n_in + k];
    A0[e] = v;
}

// y[b] = H3[b] . W4 + b4 (FP32), plus skip_scale times input column skip_col of the row (FP32)
// when skip_col >= 0
__global__ void k_out(const float *__restrict__ H3, int W, const float *__restrict__ W4, const float *b4,
                      int B, const float *__restrict__ X, int n_in, const int32_t *__restrict__ idx, int skip_col,
                      float skip_scale, float *__restrict__ y) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    float s = 0.f;
    for (int k = 0; k < W; ++k) s += H3[(size_t)b * W + k] * W4[k];
    const float sk = skip_col >= 0 ? skip_scale * X[(size_t)(idx ? idx[b] : b) * n_in + skip_col] : 0.f;
    y[b] = s + b4[0] + sk;
}

// dy = 2 w (y - t) / sum(w) and the loss; one workgroup, fixed reduction tree
__global__ __launch_bounds__(256) void k_loss(const float *__restrict__ y, const float *__restrict__ t_all,
                                              const float *__restrict__ w_all, const int32_t *__restrict__ idx, int B,
                                              float *__restrict__ dy, float *__restrict__ loss_out) {
    __shared__ float sw[256], sl[256];
    float a = 0.f, l = 0.f;
    for (int b = threadIdx.x; b < B; b += 256) {
        const int i = idx ? idx[b] : b;
        const float d = y[b] - t_all[i];
        a += w_all[i];
        l += w_all[i] * d * d;
    }
    sw[threadIdx.x] = a;
    sl[threadIdx.x] = l;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            sw[threadIdx.x] += sw[threadIdx.x + s];
            sl[threadIdx.x] += sl[threadIdx.x + s];
        }
        __syncthreads();
    }
    const float W = sw[0];
    for (int b = threadIdx.x; b < B; b += 256) {
        const int i = idx ? idx[b] : b;
        dy[b] = 2.f * w_all[i] * (y[b] - t_all[i]) / W;
    }
    if (threadIdx.x == 0) loss_out[0] = sl[0] / W;
}

// output layer gradients: dW4[k] = sum_b dy_b H3[b][k], db4 = sum_b dy_b
__global__ void k_out_grad(const float *__restrict__ dy, const float *__restrict__ H3, int W, int B,
                           float *__restrict__ gW4, float *__restrict__ gb4) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k > W) return;
    float s = 0.f;
    if (k < W)
        for (int b = 0; b < B; ++b) s += dy[b] * H3[(size_t)b * W + k];
    else
        for (int b = 0; b < B; ++b) s += dy[b];
    if (k < W) gW4[k] = s; else gb4[0] = s;
}

// dZ[b][n] = dH[b][n] * silu'(Z[b][n]) with dH = dy_b W4[n] (from_out) or the
// given fp32 dH; writes dZ [Bp][N] and its transpose [N][Bp] (rows
// b >= B are zero) and keeps fp32 dZ for the bias gradient.
__global__ void k_dz(const float *__restrict__ dH, const float *__restrict__ dy, const float *__restrict__ W4,
                     const float *__restrict__ Z, int N, int B, int Bp, float *__restrict__ dZf, float *__restrict__ dZ,
                     float *__restrict__ dZt) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= Bp * N) return;
    const int b = e / N, n = e - b * N;
    float v = 0.f;
    if (b < B) {
        const float g = dH ? dH[e] : dy[b] * W4[n];
        v = g * dsilu(Z[e]);
    }
    dZf[e] = v;
    const float h = v;
    dZ[e] = h;
    dZt[(size_t)n * Bp + b] = h;
}

// column sums: out[n] = sum_b M[b][n], b < B
__global__ void k_colsum(const float *__restrict__ M, int N, int B, float *__restrict__ out) {
    const int n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= N) return;
    float s = 0.f;
    for (int b = 0; b < B; ++b) s += M[(size_t)b * N + n];
    out[n] = s;
}

// transpose: out[c][r] = in[r][c], in [R][C]
__global__ void k_transpose(const float *__restrict__ in, int R, int C, float *__restrict__ out) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= R * C) return;
    const int r = e / C, c = e - r * C;
    out[(size_t)c * R + r] = in[e];
}

// copy a [rows][cols_src] fp32 block into [rows][cols_dst] (first cols_src columns)
__global__ void k_copy_cols(const float *__restrict__ src, int rows, int cs, int cd, float *__restrict__ dst) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= rows * cd) return;
    const int r = e / cd, c = e - r * cd;
    dst[e] = src[(size_t)r * cs + c];
}

// Adam on the flat FP32 master parameters
__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int n, float lr, float b1, float b2, float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

// working copy of a weight matrix [R][C] in [R][ldd] (zero padded)
__global__ void k_w_copy(const float *__restrict__ W, int R, int C, int ldd, float *__restrict__ out) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= R * ldd) return;
    const int r = e / ldd, c = e - r * ldd;
    out[e] = c < C ? W[(size_t)r * C + c] : 0.f;
}

// Defensive mixture proposal over P configurations and inverse-CDF draws:
//   q_c = (1 - alpha) softmax(yhat / tau)_c + alpha / P       (FP64)
//   idx_k = smallest c with u_k * cdf[P-1] < cdf[c]
// One workgroup; the CDF is a fixed-order block scan.
__global__ __launch_bounds__(256) void k_proposal(const float *__restrict__ yhat, int P, double alpha, double tau,
                                                  int K, const double *__restrict__ u, int32_t *__restrict__ idx,
                                                  double *__restrict__ q, double *__restrict__ cdf) {
    __shared__ double sh[256];
    double mx = -INFINITY;
    for (int c = threadIdx.x; c < P; c += 256) mx = fmax(mx, (double)yhat[c] / tau);
    sh[threadIdx.x] = mx;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] = fmax(sh[threadIdx.x], sh[threadIdx.x + s]);
        __syncthreads();
    }
    const double M = sh[0];
    __syncthreads();
    double sum = 0.0;
    for (int c = threadIdx.x; c < P; c += 256) sum += exp((double)yhat[c] / tau - M);
    sh[threadIdx.x] = sum;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    const double S = sh[0];
    __syncthreads();
    for (int c = threadIdx.x; c < P; c += 256) q[c] = (1.0 - alpha) * exp((double)yhat[c] / tau - M) / S + alpha / P;
    __syncthreads();
    // CDF: contiguous slices per thread, then a scan of the slice totals
    const int per = (P + 255) / 256;
    const int c0 = threadIdx.x * per, c1 = min(P, c0 + per);
    double run = 0.0;
    for (int c = c0; c < c1; ++c) run += q[c];
    sh[threadIdx.x] = run;
    __syncthreads();
    if (threadIdx.x == 0)
        for (int t = 1; t < 256; ++t) sh[t] += sh[t - 1];
    __syncthreads();
    double base = threadIdx.x > 0 ? sh[threadIdx.x - 1] : 0.0;
    for (int c = c0; c < c1; ++c) {
        base += q[c];
        cdf[c] = base;
    }
    __syncthreads();
    const double tot = cdf[P - 1];
    for (int k = threadIdx.x; k < K; k += 256) {
        const double x = u[k] * tot;
        int lo = 0, hi = P - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (x < cdf[mid]) hi = mid; else lo = mid + 1;
        }
        idx[k] = lo;
    }
}

struct Buf {
    void *p = nullptr;
    size_t n = 0;
};

}  // namespace

struct fftdg_mlp {
    int device = 0;
    hipStream_t stream = nullptr;
    std::string err;
    int n_in = 0, width = 0, max_batch = 0, Bmax = 0;
    int64_t np = 0;
    bool fp32 = false;             // operands and activations FP32 (else BF16)
    Buf P, G, Mm, Vv;              // fp32 master params, grads, Adam moments
    Buf W1, W2, W3, W4, W2t, W3t;  // working copies in the operand type (BF16: frag_index order)
    // BF16: transposed activations and gradients of a batch (dZf, dy also FP32)
    Buf A0t, H1t, H2t, H3t, dZ1t, dZ2t, dZ3t, dZf, dy, lrow, wsum, loss;
    // FP32: activations and gradients of a batch, step by step
    Buf A0, H1, H2, H3, Z1, Z2, Z3, y, dZ, dZt, dH, gtmp;
    Buf pcdf;
    int64_t step = 0;
    int skip_col = -1;  // output adds skip_scale * x[skip_col] (none if < 0)
    float skip_scale = 0.f;
};

namespace {

int merr(fftdg_mlp *m, int code, const std::string &s) {
    if (m) m->err = s;
    return code;
}
#define MCHK(m, expr)                                                                                   \
    do {                                                                                                \
        hipError_t e_ = (expr);                                                                         \
        if (e_ != hipSuccess) return merr(m, FFTDG_E_DEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

int balloc(fftdg_mlp *m, Buf &b, size_t bytes) {
    if (bytes <= b.n) return FFTDG_OK;
    if (b.p) (void)hipFree(b.p);
    b.p = nullptr;
    b.n = 0;
    if (hipMalloc(&b.p, bytes) != hipSuccess) {
        (void)hipGetLastError();
        b.p = nullptr;
        return merr(m, FFTDG_E_NOMEM, "device allocation failed");
    }
    b.n = bytes;
    return FFTDG_OK;
}

inline unsigned nb(size_t n, int t = 256) { return (unsigned)((n + t - 1) / t); }

// offsets of the flat parameter layout
struct Lay {
    int64_t W1, b1, W2, b2, W3, b3, W4, b4, n;
    Lay(int F, int H) {
        W1 = 0;
        b1 = W1 + (int64_t)H * F;
        W2 = b1 + H;
        b2 = W2 + (int64_t)H * H;
        W3 = b2 + H;
        b3 = W3 + (int64_t)H * H;
        W4 = b3 + H;
        b4 = W4 + H;
        n = b4 + 1;
    }
};

int refresh_f32(fftdg_mlp *m) {
    const int F = m->n_in, H = m->width;
    const Lay L(F, H);
    const float *p = (const float *)m->P.p;
    hipStream_t st = m->stream;
    hipLaunchKernelGGL(k_w_copy, dim3(nb((size_t)H * KP)), dim3(256), 0, st, p + L.W1, H, F, KP, (float *)m->W1.p);
    hipLaunchKernelGGL(k_w_copy, dim3(nb((size_t)H * H)), dim3(256), 0, st, p + L.W2, H, H, H, (float *)m->W2.p);
    hipLaunchKernelGGL(k_w_copy, dim3(nb((size_t)H * H)), dim3(256), 0, st, p + L.W3, H, H, H, (float *)m->W3.p);
    hipLaunchKernelGGL(k_w_copy, dim3(nb((size_t)H)), dim3(256), 0, st, p + L.W4, 1, H, H, (float *)m->W4.p);
    hipLaunchKernelGGL(k_transpose, dim3(nb((size_t)H * H)), dim3(256), 0, st, (const float *)m->W2.p, H, H,
                       (float *)m->W2t.p);
    hipLaunchKernelGGL(k_transpose, dim3(nb((size_t)H * H)), dim3(256), 0, st, (const float *)m->W3.p, H, H,
                       (float *)m->W3t.p);
    MCHK(m, hipGetLastError());
    return FFTDG_OK;
}

UpdateArgs update_args(fftdg_mlp *m, const float *g, float lr, float c1, float c2) {
    return UpdateArgs{(float *)m->P.p, g, (float *)m->Mm.p, (float *)m->Vv.p, (int)m->np, m->n_in, m->width, lr, 0.9f,
                      0.999f, 1e-8f, c1, c2, (uint16_t *)m->W1.p, (uint16_t *)m->W2.p, (uint16_t *)m->W3.p,
                      (uint16_t *)m->W2t.p, (uint16_t *)m->W3t.p, (uint16_t *)m->W4.p};
}

// the working copies of the weights from the FP32 master parameters
int refresh_w(fftdg_mlp *m) {
    if (m->fp32) return refresh_f32(m);
    hipLaunchKernelGGL(k_update<false>, dim3(nb((size_t)m->np)), dim3(256), 0, m->stream,
                       update_args(m, nullptr, 0.f, 1.f, 1.f));
    MCHK(m, hipGetLastError());
    return FFTDG_OK;
}

int gemm_f32(fftdg_mlp *m, const float *A, int lda, const float *B, int ldb, int M, int N, int K, const float *bias, int mode,
         float *C, int ldc, float *Hh, int ldh) {
    hipLaunchKernelGGL(k_gemm, dim3(N / 64, M / 64), dim3(256), 0, m->stream, A, lda, B, ldb, K, bias, mode, C,
                       ldc, Hh, ldh);
    MCHK(m, hipGetLastError());
    return FFTDG_OK;
}

// forward pass over B rows (rows of X selected by idx, or the first B rows)
int forward_f32(fftdg_mlp *m, const float *X, const int32_t *idx, int B, int Bp) {
    const int H = m->width;
    const Lay L(m->n_in, H);
    const float *p = (const float *)m->P.p;
    hipLaunchKernelGGL(k_gather, dim3(nb((size_t)Bp * KP)), dim3(256), 0, m->stream, X, m->n_in, idx, B, Bp,
                       (float *)m->A0.p);
    int rc;
    if ((rc = gemm_f32(m, (float *)m->A0.p, KP, (float *)m->W1.p, KP, Bp, H, KP, p + L.b1, 1, (float *)m->Z1.p, H,
                      (float *)m->H1.p, H)))
        return rc;
    if ((rc = gemm_f32(m, (float *)m->H1.p, H, (float *)m->W2.p, H, Bp, H, H, p + L.b2, 1, (float *)m->Z2.p, H, (float *)m->H2.p,
                      H)))
        return rc;
    if ((rc = gemm_f32(m, (float *)m->H2.p, H, (float *)m->W3.p, H, Bp, H, H, p + L.b3, 1, (float *)m->Z3.p, H, (float *)m->H3.p,
                      H)))
        return rc;
    hipLaunchKernelGGL(k_out, dim3(nb((size_t)B)), dim3(256), 0, m->stream, (const float *)m->H3.p, H,
                       (const float *)m->W4.p, p + L.b4, B, X, m->n_in, idx, m->skip_col, m->skip_scale,
                       (float *)m->y.p);
    MCHK(m, hipGetLastError());
    return FFTDG_OK;
}

NetArgs net_args(fftdg_mlp *m, const float *X, const int32_t *idx, int B) {
    const Lay L(m->n_in, m->width);
    const float *p = (const float *)m->P.p;
    NetArgs a{};
    a.X = X, a.idx = idx, a.n_in = m->n_in, a.H = m->width, a.B = B;
    a.W1 = (const uint16_t *)m->W1.p, a.W2 = (const uint16_t *)m->W2.p, a.W3 = (const uint16_t *)m->W3.p;
    a.W2t = (const uint16_t *)m->W2t.p, a.W3t = (const uint16_t *)m->W3t.p, a.W4 = (const uint16_t *)m->W4.p;
    a.b1 = p + L.b1, a.b2 = p + L.b2, a.b3 = p + L.b3, a.b4 = p + L.b4;
    a.skip_col = m->skip_col, a.skip_scale = m->skip_scale;
    return a;
}
template <int NTW, int MT, bool TRAIN>
void launch_net_w(fftdg_mlp *m, const NetArgs &a, int rows) {
    const dim3 g((unsigned)((rows + 16 * MT - 1) / (16 * MT))), t(512);
    if (m->width == 128 * NTW) hipLaunchKernelGGL((k_net<NTW, MT, TRAIN, true>), g, t, 0, m->stream, a);
    else hipLaunchKernelGGL((k_net<NTW, MT, TRAIN, false>), g, t, 0, m->stream, a);
}
template <int MT, bool TRAIN>
void launch_net(fftdg_mlp *m, const NetArgs &a, int rows) {
    if (m->width <= 128) launch_net_w<1, MT, TRAIN>(m, a, rows);
    else if (m->width <= 256) launch_net_w<2, MT, TRAIN>(m, a, rows);
    else if (m->width <= 512) launch_net_w<4, MT, TRAIN>(m, a, rows);
    else launch_net_w<8, MT, TRAIN>(m, a, rows);
}
// all n rows in one launch; two 16-row tiles a block share its weight loads
// once that still gives every compute unit a block
int forward_bf16(fftdg_mlp *m, const float *X, int n, float *y) {
    NetArgs a = net_args(m, X, nullptr, n);
    a.y = y;
    if (n >= 32 * 256) launch_net<2, false>(m, a, n);
    else launch_net<1, false>(m, a, n);
    MCHK(m, hipGetLastError());
    return FFTDG_OK;
}
// gradient of a batch of B rows (padded to 64) into g, loss in m->loss
int backward_bf16(fftdg_mlp *m, const float *X, const float *t, const float *w, const int32_t *idx, int B, float *g) {
    const Lay L(m->n_in, m->width);
    const int ld = (B + 63) / 64 * 64, H = m->width;
    NetArgs a = net_args(m, X, idx, B);
    a.t = t, a.w = w, a.ld = ld;
    a.A0t = (uint16_t *)m->A0t.p, a.H1t = (uint16_t *)m->H1t.p, a.H2t = (uint16_t *)m->H2t.p;
    a.dZ1t = (uint16_t *)m->dZ1t.p, a.dZ2t = (uint16_t *)m->dZ2t.p, a.dZ3t = (uint16_t *)m->dZ3t.p;
    a.H3t = (uint16_t *)m->H3t.p, a.dZf = (float *)m->dZf.p, a.dy = (float *)m->dy.p, a.lrow = (float *)m->lrow.p;
    if (B > 4096) {  // past that a launch costs less than every block adding up the weights
        hipLaunchKernelGGL(k_wsum, dim3(1), dim3(256), 0, m->stream, w, idx, B, (float *)m->wsum.p);
        a.wsum = (const float *)m->wsum.p;
    }
    launch_net<1, true>(m, a, ld);
    const GradArgs ga{H, m->n_in, ld, B, a.A0t, a.H1t, a.H2t, a.dZ1t, a.dZ2t, a.dZ3t, a.H3t, a.dZf, a.dy, a.lrow,
                      g + L.W1, g + L.b1, g + L.W2, g + L.b2, g + L.W3, g + L.b3, g + L.W4, g + L.b4,
                      (float *)m->loss.p};
    const int tiles = (H / 16) * (KP / 32) + 2 * (H / 16) * (H / 32);
    hipLaunchKernelGGL(k_wgrad, dim3((tiles + 3) / 4 + H / 4 + 2), dim3(256), 0, m->stream, ga);
    MCHK(m, hipGetLastError());
    return FFTDG_OK;
}

int backward_f32(fftdg_mlp *m, const float *X, const float *t, const float *w, const int32_t *idx, int B, float *g) {
    const int H = m->width, F = m->n_in;
    const int Bp = (B + 63) / 64 * 64;
    const Lay L(F, H);
    hipStream_t st = m->stream;
    int rc;
    if ((rc = forward_f32(m, X, idx, B, Bp))) return rc;
    hipLaunchKernelGGL(k_loss, dim3(1), dim3(256), 0, st, (const float *)m->y.p, t, w, idx, B, (float *)m->dy.p,
                       (float *)m->loss.p);
    hipLaunchKernelGGL(k_out_grad, dim3(nb((size_t)H + 1)), dim3(256), 0, st, (const float *)m->dy.p,
                       (const float *)m->H3.p, H, B, g + L.W4, g + L.b4);
    // layer 3
    hipLaunchKernelGGL(k_dz, dim3(nb((size_t)Bp * H)), dim3(256), 0, st, (const float *)nullptr,
                       (const float *)m->dy.p, (const float *)m->W4.p, (const float *)m->Z3.p, H, B, Bp,
                       (float *)m->dZf.p, (float *)m->dZ.p, (float *)m->dZt.p);
    hipLaunchKernelGGL(k_colsum, dim3(nb((size_t)H)), dim3(256), 0, st, (const float *)m->dZf.p, H, B, g + L.b3);
    hipLaunchKernelGGL(k_transpose, dim3(nb((size_t)Bp * H)), dim3(256), 0, st, (const float *)m->H2.p, Bp, H,
                       (float *)m->H2t.p);
    if ((rc = gemm_f32(m, (float *)m->dZt.p, Bp, (float *)m->H2t.p, Bp, H, H, Bp, nullptr, 0, g + L.W3, H,
                   nullptr, 0)))
        return rc;
    if ((rc = gemm_f32(m, (float *)m->dZ.p, H, (float *)m->W3t.p, H, Bp, H, H, nullptr, 0, (float *)m->dH.p, H,
                   nullptr, 0)))
        return rc;
    // layer 2
    hipLaunchKernelGGL(k_dz, dim3(nb((size_t)Bp * H)), dim3(256), 0, st, (const float *)m->dH.p,
                       (const float *)nullptr, (const float *)nullptr, (const float *)m->Z2.p, H, B, Bp,
                       (float *)m->dZf.p, (float *)m->dZ.p, (float *)m->dZt.p);
    hipLaunchKernelGGL(k_colsum, dim3(nb((size_t)H)), dim3(256), 0, st, (const float *)m->dZf.p, H, B, g + L.b2);
    hipLaunchKernelGGL(k_transpose, dim3(nb((size_t)Bp * H)), dim3(256), 0, st, (const float *)m->H1.p, Bp, H,
                       (float *)m->H1t.p);
    if ((rc = gemm_f32(m, (float *)m->dZt.p, Bp, (float *)m->H1t.p, Bp, H, H, Bp, nullptr, 0, g + L.W2, H,
                   nullptr, 0)))
        return rc;
    if ((rc = gemm_f32(m, (float *)m->dZ.p, H, (float *)m->W2t.p, H, Bp, H, H, nullptr, 0, (float *)m->dH.p, H,
                   nullptr, 0)))
        return rc;
    // layer 1 (no input gradient)
    hipLaunchKernelGGL(k_dz, dim3(nb((size_t)Bp * H)), dim3(256), 0, st, (const float *)m->dH.p,
                       (const float *)nullptr, (const float *)nullptr, (const float *)m->Z1.p, H, B, Bp,
                       (float *)m->dZf.p, (float *)m->dZ.p, (float *)m->dZt.p);
    hipLaunchKernelGGL(k_colsum, dim3(nb((size_t)H)), dim3(256), 0, st, (const float *)m->dZf.p, H, B, g + L.b1);
    hipLaunchKernelGGL(k_transpose, dim3(nb((size_t)Bp * KP)), dim3(256), 0, st, (const float *)m->A0.p, Bp, KP,
                       (float *)m->A0t.p);
    if ((rc = gemm_f32(m, (float *)m->dZt.p, Bp, (float *)m->A0t.p, Bp, H, KP, Bp, nullptr, 0,
                   (float *)m->gtmp.p, KP, nullptr, 0)))
        return rc;
    hipLaunchKernelGGL(k_copy_cols, dim3(nb((size_t)H * F)), dim3(256), 0, st, (const float *)m->gtmp.p, H, KP, F,
                       g + L.W1);
    MCHK(m, hipGetLastError());
    return FFTDG_OK;
}
int backward(fftdg_mlp *m, const float *X, const float *t, const float *w, const int32_t *idx, int B, float *g) {
    return m->fp32 ? backward_f32(m, X, t, w, idx, B, g) : backward_bf16(m, X, t, w, idx, B, g);
}

}  // namespace

extern "C" {

int fftdg_mlp_create(fftdg_mlp **out, int device, void *stream, int32_t n_in, int32_t width, int32_t max_batch) {
    return fftdg_mlp_create_ex(out, device, stream, n_in, width, max_batch, 0);
}

int fftdg_mlp_create_ex(fftdg_mlp **out, int device, void *stream, int32_t n_in, int32_t width, int32_t max_batch,
                        int32_t fp32_operands) {
    if (!out) return FFTDG_E_INVALID;
    *out = nullptr;
    if (n_in < 1 || n_in > KP || width < 64 || width % 64 || width > 1024 || max_batch < 1 || max_batch > (1 << 22) ||
        (fp32_operands != 0 && fp32_operands != 1))
        return FFTDG_E_INVALID;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) {
        (void)hipGetLastError();
        return FFTDG_E_DEVICE;
    }
    if (device < 0 || device >= ndev) return FFTDG_E_INVALID;
    if (hipSetDevice(device) != hipSuccess) {
        (void)hipGetLastError();
        return FFTDG_E_DEVICE;
    }
    fftdg_mlp *m = new (std::nothrow) fftdg_mlp();
    if (!m) return FFTDG_E_NOMEM;
    m->device = device;
    m->stream = (hipStream_t)stream;
    m->n_in = n_in;
    m->width = width;
    m->max_batch = max_batch;
    m->fp32 = fp32_operands != 0;
    m->Bmax = (max_batch + 63) / 64 * 64;
    const Lay L(n_in, width);
    m->np = L.n;
    const size_t H = width, Bm = m->Bmax;
    int rc = 0;
    Buf *f32n[] = {&m->P, &m->G, &m->Mm, &m->Vv};
    for (Buf *b : f32n)
        if (!rc) rc = balloc(m, *b, sizeof(float) * L.n);
    const size_t bf = m->fp32 ? sizeof(float) : sizeof(uint16_t);  // operand element
    auto make = [&](std::initializer_list<Buf *> bufs, size_t bytes) {
        for (Buf *b : bufs)
            if (!rc) rc = balloc(m, *b, bytes);
    };
    make({&m->W1}, bf * H * KP);
    make({&m->W2, &m->W3, &m->W2t, &m->W3t}, bf * H * H);
    make({&m->W4}, bf * H);
    make({&m->A0t}, bf * Bm * KP);
    make({&m->loss}, sizeof(float) * 4);
    if (m->fp32) {
        make({&m->A0}, bf * Bm * KP);
        make({&m->H1, &m->H2, &m->H3, &m->H1t, &m->H2t, &m->dZ, &m->dZt, &m->Z1, &m->Z2, &m->Z3, &m->dZf, &m->dH},
             sizeof(float) * Bm * H);
        make({&m->y, &m->dy}, sizeof(float) * Bm);
        make({&m->gtmp}, sizeof(float) * H * KP);
    } else {
        make({&m->H1t, &m->H2t, &m->H3t, &m->dZ1t, &m->dZ2t, &m->dZ3t}, bf * Bm * H);
        make({&m->dZf}, sizeof(float) * 3 * Bm * H);
        make({&m->dy}, sizeof(float) * Bm);
        make({&m->lrow}, sizeof(float) * (Bm + 64));
        make({&m->wsum}, sizeof(float));
        if (!rc && hipMemset(m->W1.p, 0, bf * H * KP) != hipSuccess) {  // padded inputs weigh nothing
            (void)hipGetLastError();
            rc = FFTDG_E_DEVICE;
        }
    }
    if (rc) {
        fftdg_mlp_destroy(m);
        return rc;
    }
    std::vector<float> zero(L.n, 0.f);
    if (hipMemcpy(m->P.p, zero.data(), sizeof(float) * L.n, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(m->Mm.p, zero.data(), sizeof(float) * L.n, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(m->Vv.p, zero.data(), sizeof(float) * L.n, hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipGetLastError();
        fftdg_mlp_destroy(m);
        return FFTDG_E_DEVICE;
    }
    if ((rc = refresh_w(m)) || hipStreamSynchronize(m->stream) != hipSuccess) {
        fftdg_mlp_destroy(m);
        return rc ? rc : FFTDG_E_DEVICE;
    }
    *out = m;
    return FFTDG_OK;
}

void fftdg_mlp_destroy(fftdg_mlp *m) {
    if (!m) return;
    (void)hipSetDevice(m->device);
    (void)hipStreamSynchronize(m->stream);
    Buf *all[] = {&m->P,   &m->G,   &m->Mm,   &m->Vv,   &m->W1,   &m->W2,   &m->W3,   &m->W4, &m->W2t, &m->W3t,
                  &m->A0t, &m->H1t, &m->H2t,  &m->dZ1t, &m->dZ2t, &m->dZ3t, &m->H3t, &m->lrow, &m->wsum, &m->loss,
                  &m->A0,  &m->H1,  &m->H2,   &m->H3,   &m->Z1,   &m->Z2,   &m->Z3,   &m->y,  &m->dy,  &m->dZf,
                  &m->dZ,  &m->dZt, &m->dH,   &m->gtmp, &m->pcdf};
    for (Buf *b : all)
        if (b->p) (void)hipFree(b->p);
    delete m;
}

const char *fftdg_mlp_last_error(const fftdg_mlp *m) { return m ? m->err.c_str() : "network is NULL"; }

int64_t fftdg_mlp_num_params(const fftdg_mlp *m) { return m ? m->np : -1; }

int fftdg_mlp_set_params(fftdg_mlp *m, const float *p_host, int64_t n) {
    if (!m) return FFTDG_E_INVALID;
    if (!p_host || n != m->np) return merr(m, FFTDG_E_INVALID, "set_params: wrong size or NULL");
    MCHK(m, hipSetDevice(m->device));
    MCHK(m, hipMemcpyAsync(m->P.p, p_host, sizeof(float) * n, hipMemcpyHostToDevice, m->stream));
    std::vector<float> zero(n, 0.f);
    MCHK(m, hipMemcpyAsync(m->Mm.p, zero.data(), sizeof(float) * n, hipMemcpyHostToDevice, m->stream));
    MCHK(m, hipMemcpyAsync(m->Vv.p, zero.data(), sizeof(float) * n, hipMemcpyHostToDevice, m->stream));
    m->step = 0;
    int rc = refresh_w(m);
    if (rc) return rc;
    MCHK(m, hipStreamSynchronize(m->stream));
    return FFTDG_OK;
}

int fftdg_mlp_get_params(fftdg_mlp *m, float *p_host, int64_t n) {
    if (!m) return FFTDG_E_INVALID;
    if (!p_host || n != m->np) return merr(m, FFTDG_E_INVALID, "get_params: wrong size or NULL");
    MCHK(m, hipSetDevice(m->device));
    MCHK(m, hipMemcpyAsync(p_host, m->P.p, sizeof(float) * n, hipMemcpyDeviceToHost, m->stream));
    MCHK(m, hipStreamSynchronize(m->stream));
    return FFTDG_OK;
}

int fftdg_mlp_set_skip(fftdg_mlp *m, int32_t col, float scale) {
    if (!m) return FFTDG_E_INVALID;
    if (col < -1 || col >= m->n_in || !std::isfinite(scale))
        return merr(m, FFTDG_E_INVALID, "set_skip: column out of range or non-finite scale");
    m->skip_col = col;
    m->skip_scale = col >= 0 ? scale : 0.f;
    return FFTDG_OK;
}

int fftdg_mlp_forward(fftdg_mlp *m, const float *x, int32_t n, float *y) {
    if (!m) return FFTDG_E_INVALID;
    if (!x || !y || n < 0) return merr(m, FFTDG_E_INVALID, "forward: NULL pointer or negative size");
    MCHK(m, hipSetDevice(m->device));
    if (!m->fp32) return n > 0 ? forward_bf16(m, x, n, y) : FFTDG_OK;
    for (int32_t b0 = 0; b0 < n; b0 += m->max_batch) {
        const int B = std::min(m->max_batch, n - b0), Bp = (B + 63) / 64 * 64;
        int rc = forward_f32(m, x + (size_t)b0 * m->n_in, nullptr, B, Bp);
        if (rc) return rc;
        MCHK(m, hipMemcpyAsync(y + b0, m->y.p, sizeof(float) * B, hipMemcpyDeviceToDevice, m->stream));
    }
    return FFTDG_OK;
}

int fftdg_mlp_grad(fftdg_mlp *m, const float *x_all, const float *t_all, const float *w_all, const int32_t *idx,
                   int32_t B, float *grad, float *loss_host) {
    if (!m) return FFTDG_E_INVALID;
    if (!x_all || !t_all || !w_all || !grad || B < 1 || B > m->max_batch)
        return merr(m, FFTDG_E_INVALID, "grad: NULL pointer or batch size outside 1..max_batch");
    MCHK(m, hipSetDevice(m->device));
    int rc = backward(m, x_all, t_all, w_all, idx, B, grad);
    if (rc) return rc;
    if (loss_host) {
        MCHK(m, hipMemcpyAsync(loss_host, m->loss.p, sizeof(float), hipMemcpyDeviceToHost, m->stream));
        MCHK(m, hipStreamSynchronize(m->stream));
    }
    return FFTDG_OK;
}

int fftdg_mlp_train_step(fftdg_mlp *m, const float *x_all, const float *t_all, const float *w_all,
                         const int32_t *idx, int32_t B, float lr, float *loss_host) {
    if (!m) return FFTDG_E_INVALID;
    if (!(lr > 0.f) || !std::isfinite(lr)) return merr(m, FFTDG_E_INVALID, "train_step: learning rate must be > 0");
    int rc = fftdg_mlp_grad(m, x_all, t_all, w_all, idx, B, (float *)m->G.p, nullptr);
    if (rc) return rc;
    ++m->step;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - powf(b1, (float)m->step), c2 = 1.f - powf(b2, (float)m->step);
    if (m->fp32) {
        hipLaunchKernelGGL(k_adam, dim3(nb((size_t)m->np)), dim3(256), 0, m->stream, (float *)m->P.p,
                           (const float *)m->G.p, (float *)m->Mm.p, (float *)m->Vv.p, (int)m->np, lr, b1, b2, 1e-8f,
                           c1, c2);
        MCHK(m, hipGetLastError());
        if ((rc = refresh_w(m))) return rc;
    } else {
        hipLaunchKernelGGL(k_update<true>, dim3(nb((size_t)m->np)), dim3(256), 0, m->stream,
                           update_args(m, (const float *)m->G.p, lr, c1, c2));
        MCHK(m, hipGetLastError());
    }
    if (loss_host) {
        MCHK(m, hipMemcpyAsync(loss_host, m->loss.p, sizeof(float), hipMemcpyDeviceToHost, m->stream));
        MCHK(m, hipStreamSynchronize(m->stream));
    }
    return FFTDG_OK;
}

int fftdg_proposal_sample(fftdg_mlp *m, const float *yhat, int32_t P, double alpha, double tau, int32_t K,
                          const double *u, int32_t *idx, double *q) {
    if (!m) return FFTDG_E_INVALID;
    if (!yhat || !u || !idx || !q || P < 1 || K < 0)
        return merr(m, FFTDG_E_INVALID, "proposal_sample: NULL pointer or bad size");
    if (!(alpha >= 0.0 && alpha <= 1.0) || !(tau > 0.0) || !std::isfinite(tau))
        return merr(m, FFTDG_E_INVALID, "proposal_sample: need 0 <= alpha <= 1 and tau > 0");
    MCHK(m, hipSetDevice(m->device));
    if (m->pcdf.n < sizeof(double) * (size_t)P) {
        if (m->pcdf.p) (void)hipFree(m->pcdf.p);
        m->pcdf.p = nullptr;
        m->pcdf.n = 0;
        if (hipMalloc(&m->pcdf.p, sizeof(double) * (size_t)P) != hipSuccess) {
            (void)hipGetLastError();
            return merr(m, FFTDG_E_NOMEM, "proposal_sample: allocation failed");
        }
        m->pcdf.n = sizeof(double) * (size_t)P;
    }
    hipLaunchKernelGGL(k_proposal, dim3(1), dim3(256), 0, m->stream, yhat, P, alpha, tau, K, u, idx, q,
                       (double *)m->pcdf.p);
    MCHK(m, hipGetLastError());
    return FFTDG_OK;
}

}  // extern "C"
