// Learned pairwise bridge-force surrogate: an MLP whose forward and backward matrix products run
// as hand-written BF16 MFMA kernels (v_mfma_f32_16x16x32_bf16, FP32 accumulation) on gfx950.
// See include/pf_mlp.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/pf_mlp.h"

namespace pfm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// n / d for d >= 1, from n / 4 and d / 4: the reciprocal's quotient with one correction by its exact
// remainder, then the special cases (d infinite, n infinite or NaN).  It is the IEEE division without the
// scaling for small d and without the second correction, half its instructions.  The factor 1/4 changes no
// bit of the result and keeps the reciprocal of the largest finite d normal, as the hardware flushes
// subnormal ones to zero (without it SiLU is 0 below z = -87.3, where it is about -1e-36; 65536 rows of
// 4 -> 128 x 4 -> 1 take 31.7 us with it and 31.6 without).  With the remainder exact the result differs from
// the correctly rounded quotient in about one of 10^7 cases, by one unit in the last place.
__device__ __forceinline__ float quotient(float n4, float d4) {
    const float r = __builtin_amdgcn_rcpf(d4), q = n4 * r;
    return __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-d4, q, n4), r, q), d4, n4);
}
// a constant in a scalar register (as a literal it would lengthen each instruction that takes it)
__device__ __forceinline__ float scalar(float k) {
    asm("" : "+s"(k));
    return k;
}
// z / (1 + exp(-z)) from z4 = z / 4, with quarter = 1/4 and c = -4 log2(e)
__device__ __forceinline__ float silu4(float z4, float quarter, float c) {
    return quotient(z4, __builtin_fmaf(__builtin_amdgcn_exp2f(z4 * c), quarter, quarter));
}
constexpr float SILU_C = -4.0f * 0x1.715476p+0f;
__device__ __forceinline__ float silu(float z) {
    const float quarter = scalar(0.25f);
    return quotient(quarter * z, __builtin_fmaf(__expf(-z), quarter, quarter));
}
__device__ __forceinline__ float silu_grad(float z) {
    const float quarter = scalar(0.25f), s = quotient(0.25f, __builtin_fmaf(__expf(-z), quarter, quarter));
    return s * (1.0f + z * (1.0f - s));
}

// C[M][N] = A[M][K] B[K][N] (+ bias[n]), BF16 operands contiguous along K, FP32 accumulation, N a
// multiple of 16.  K advances 32 at a time through one MFMA.  Operand layout of
// v_mfma_f32_16x16x32_bf16: lane l holds A[l % 16][8 (l / 16) + j] and B[8 (l / 16) + j][l % 16],
// j = 0..7; the result D[4 (l / 16) + r][l % 16], r = 0..3.  Epilogue: Cf (FP32, may be NULL) receives
// the sum z; Cb (BF16, may be NULL) receives z, or silu(z) when act != 0.  Elements outside
// [M) x [N) x [K) read as zero and are not written.
struct Gemm {
    const __bf16 *A;
    long long sam;
    const __bf16 *B;
    long long sbn;
    float *Cf;
    __bf16 *Cb;
    long long scm;
    const float *bias;
    int M, N, K, act;
    int vec;  // k_gemm_bf16_rows: 16-byte operand loads (K, row strides multiples of 8, aligned bases)
};

// A block of 4 waves computes 64 rows across up to
// 16 NT columns (blockIdx.y picks the column chunk): the B columns are staged in LDS, 128 K values
// at a time (rows padded by 16 bytes so that the 16 lanes reading one K chunk of 16 columns hit
// distinct banks), and each wave takes a 16-row strip, loading its A fragment (one 16-byte load
// per lane when g.vec, else element by element) and reusing it for the NT products of the strip.
// The BF16 strip is written through LDS as 16-byte row segments.  Every wave takes part in the
// staging, also one past the last row.
template <int NT>
__global__ __launch_bounds__(256) void k_gemm_bf16_rows(Gemm g) {
    constexpr int KC = 128, LD = KC + 8;
    __shared__ __attribute__((aligned(16))) __bf16 wl[16 * NT][LD];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int tm = blockIdx.x * 4 + wave;
    const int n0 = blockIdx.y * 16 * NT;
    const int row = tm * 16 + (lane & 15), kq = 8 * (lane >> 4);
    const bool active = tm * 16 < g.M;
    f32x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16x8 zero = {};
    for (int kc = 0; kc < g.K; kc += KC) {
        for (int e = tid * 8; e < 16 * NT * KC; e += 256 * 8) {
            const int r = e / KC, c = e - r * KC;
            bf16x8 v = zero;
            if (n0 + r < g.N) {
                const __bf16 *src = g.B + (long long)(n0 + r) * g.sbn + kc + c;
                if (g.vec) {
                    if (kc + c < g.K) v = *(const bf16x8 *)src;
                } else {
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (kc + c + j < g.K) v[j] = src[j];
                }
            }
            *(bf16x8 *)&wl[r][c] = v;
        }
        __syncthreads();
        if (active) {
            for (int k0 = 0; k0 < KC && kc + k0 < g.K; k0 += 32) {
                const int k = kc + k0 + kq;
                bf16x8 a = zero;
                if (row < g.M) {
                    const __bf16 *src = g.A + row * g.sam + k;
                    if (g.vec) {
                        if (k < g.K) a = *(const bf16x8 *)src;
                    } else {
#pragma unroll
                        for (int j = 0; j < 8; ++j)
                            if (k + j < g.K) a[j] = src[j];
                    }
                }
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    if (n0 + 16 * t >= g.N) break;  // uniform
                    const bf16x8 b = *(const bf16x8 *)&wl[16 * t + (lane & 15)][k0 + kq];
                    acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[t], 0, 0, 0);
                }
            }
        }
        __syncthreads();
    }
    // epilogue: z = acc + bias; FP32 z element by element; the BF16 strip (16 x 16 NT) goes to
    // this wave's part of the (now free) staging area, then out as 16-byte row segments
    __bf16 *strip = &wl[0][0] + wave * (16 * 16 * NT);
    const int ncols = min(16 * NT, g.N - n0);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        if (16 * t >= ncols) break;
        const int nl = 16 * t + (lane & 15), n = n0 + nl;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int ml = 4 * (lane >> 4) + r, m = tm * 16 + ml;
            const float z = acc[t][r] + (g.bias && n < g.N ? g.bias[n] : 0.0f);
            if (active && g.Cf && m < g.M && n < g.N) g.Cf[m * g.scm + n] = z;
            strip[ml * (16 * NT) + nl] = (__bf16)(g.act ? silu(z) : z);
        }
    }
    __syncthreads();
    if (!active || !g.Cb) return;
    // 16 rows x ncols columns, ncols a multiple of 16: 8-element segments
    const int segs = ncols / 8;
    for (int q = lane; q < 16 * segs; q += 64) {
        const int ml = q / segs, c = (q - ml * segs) * 8, m = tm * 16 + ml;
        if (m >= g.M) continue;
        __bf16 *dst = g.Cb + m * g.scm + n0 + c;
        const bf16x8 v = *(const bf16x8 *)&strip[ml * (16 * NT) + c];
        if (g.vec)
            *(bf16x8 *)dst = v;
        else
            for (int j = 0; j < 8; ++j) dst[j] = v[j];
    }
}

// Output layer with one output: y = A w + b over K (a multiple of 8) BF16 inputs, 16 lanes per
// row (each takes 8 consecutive inputs per 128), summed across the 16 lanes in a fixed order.
__global__ __launch_bounds__(256) void k_last_layer(const __bf16 *__restrict__ A, int M, int K,
                                                    const __bf16 *__restrict__ w, const float *__restrict__ bias,
                                                    float *__restrict__ y) {
    const long long t = (long long)blockIdx.x * 256 + threadIdx.x;
    const int row = (int)(t >> 4), sub = (int)(t & 15);
    float acc = 0.0f;
    if (row < M) {
        for (int k = 8 * sub; k < K; k += 128) {
            const bf16x8 a = *(const bf16x8 *)(A + (long long)row * K + k);
            const bf16x8 b = *(const bf16x8 *)(w + k);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc = fmaf((float)a[j], (float)b[j], acc);
        }
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 16);
    if (row < M && sub == 0) y[row] = acc + bias[0];
}

// BF16 copy of an FP32 array
__global__ void k_to_bf16(const float *__restrict__ x, __bf16 *__restrict__ y, int n) {
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) y[i] = (__bf16)x[i];
}

// BF16 copies of the weights of every layer, row-major [out][in] and transposed [in][out]
struct LayerMap {
    int n;                       // layers incl. the output layer
    int in[10], out[10];
    long long w[10], b[10];      // offsets in the parameter vector
    long long wb[10];            // offsets in the BF16 weight copies
};
__global__ void k_refresh_weights(LayerMap lm, const float *__restrict__ p, __bf16 *__restrict__ wb,
                                  __bf16 *__restrict__ wt) {
    for (int l = 0; l < lm.n; ++l) {
        const int I = lm.in[l], O = lm.out[l];
        for (int i = blockIdx.x * 256 + threadIdx.x; i < I * O; i += gridDim.x * 256) {
            const int o = i / I, k = i - o * I;
            const __bf16 v = (__bf16)p[lm.w[l] + i];
            wb[lm.wb[l] + i] = v;
            wt[lm.wb[l] + (long long)k * O + o] = v;
        }
    }
}

// What the training form of the fused kernel leaves behind: per hidden layer the FP32 pre-activations
// Z, the BF16 activations A and error terms dZ ([row][H]), the BF16 output gradient dY, and per block
// the FP64 loss sum, the FP32 sum of dY and the FP32 column sums of every dZ.
struct TrainBuf {
    const float *t;
    float *Z[8];
    __bf16 *A[8], *dZ[8], *dY;
    double *loss;
    float *dysum, *dzsum;  // [block], [block][layer][H]
};

// Forward pass (inference), or forward and backward pass (TRAIN), of a network of hidden width H in
// one launch.  A block of four waves carries 16 RS rows through every layer; a wave computes H / 4
// output columns of all of them, so each wave holds only its own slice of a layer's weights, in
// registers (loaded one layer ahead), and the weights need neither LDS nor a barrier.  The rows'
// activations (BF16) pass from layer to layer through LDS, two buffers, one barrier a layer.  The
// products run transposed, D = W act^T, so that a lane holds four consecutive columns of one row and
// stores them as 8 bytes; each product's K order is that of the layer-by-layer path.  RS = 1 where
// the batch would otherwise leave CUs idle, 4 on large batches (each weight fragment then serves
// four products).  The first layer takes the FP32 inputs rounded to BF16 (K padded with zeros to 32);
// the output layer is a dot product of each row with the output weights in a fixed order.
//
// Inference can take its row count from the device (n_dev, at most M); blocks past it return.
//
// What bounds it: the SiLU of every hidden unit on large batches (the exponential and the division
// take more issue slots than the matrix instructions), the layers' latencies on small ones.
// 4 -> 128 x 4 -> 1: gradients of 8192 rows 8997 -> 130 us a call and a training step of 205 rows
// 377 -> 50 us, this kernel 28.6 and 19.0 us of them, against the layer-by-layer path of 29 launches with
// serial column sums (1553 us each at 8192 rows) and strided single-tile weight gradients (193 us each).
struct NoTrain {};  // inference: 200 bytes of kernel arguments fewer
template <int H, int RS, bool TRAIN>
__global__ __launch_bounds__(256) void k_mlp_fused(const float *__restrict__ x, int M, int nin, LayerMap lm,
                                                   const __bf16 *__restrict__ Wb, const __bf16 *__restrict__ Wt,
                                                   const float *__restrict__ P, float *__restrict__ y,
                                                   std::conditional_t<TRAIN, TrainBuf, NoTrain> tb,
                                                   const int *__restrict__ n_dev) {
    typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
    constexpr int NT = H / 64, KS = H / 32, LD = H + 8, ROWS = 16 * RS;
    __shared__ __attribute__((aligned(16))) __bf16 act[2][ROWS][LD];
    __shared__ float dyl[ROWS], dyf[ROWS];
    __shared__ double el[ROWS];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int rl = lane & 15, kq = 8 * (lane >> 4), fq = 4 * (lane >> 4);
    const int r0 = blockIdx.x * ROWS;
    if constexpr (!TRAIN) {
        if (n_dev) M = min(M, *n_dev);
        if (r0 >= M) return;  // whole block
    }
    const int L = lm.n - 1;
    const float quarter = scalar(0.25f), silu_c = scalar(SILU_C);
    auto feat = [&](int t) { return 16 * (wave * NT + t); };  // first column of this wave's tile t
    // this wave's slice of a square layer's weights, row-major [H][H]
    auto load_w = [&](const __bf16 *W, bf16x8 (&w)[NT][KS]) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int k = 0; k < KS; ++k) w[t][k] = *(const bf16x8 *)(W + (feat(t) + rl) * H + 32 * k + kq);
    };
    // biases, inference a quarter of them
    auto load_b = [&](int l, f32x4 (&bias)[NT]) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) bias[t][r] = (TRAIN ? 1.0f : quarter) * P[lm.b[l] + feat(t) + fq + r];
    };
    // pre-activations -> BF16 activations in LDS buffer c (and, training, Z and A)
    auto activate = [&](int l, int c, int s, const f32x4 (&acc)[NT], const f32x4 (&bias)[NT]) {
        const int row = r0 + 16 * s + rl;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            bf16x4 v;
            f32x4 z;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if constexpr (TRAIN) {
                    z[r] = acc[t][r] + bias[t][r];
                    v[r] = (__bf16)silu(z[r]);
                } else {  // z / 4 in the one rounding of the sum
                    v[r] = (__bf16)silu4(__builtin_fmaf(acc[t][r], quarter, bias[t][r]), quarter, silu_c);
                }
            }
            *(bf16x4 *)&act[c][16 * s + rl][feat(t) + fq] = v;
            if constexpr (TRAIN)
                if (row < M) {
                    const long long o = (long long)row * H + feat(t) + fq;
                    *(f32x4 *)(tb.Z[l] + o) = z;
                    *(bf16x4 *)(tb.A[l] + o) = v;
                }
        }
    };
    // products of this wave's columns with 16 rows of LDS buffer c
    auto product = [&](int c, int s, const bf16x8 (&w)[NT][KS], f32x4 (&acc)[NT]) {
        bf16x8 b[KS];
#pragma unroll
        for (int k = 0; k < KS; ++k) b[k] = *(const bf16x8 *)&act[c][16 * s + rl][32 * k + kq];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < KS; ++k) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[t][k], b[k], acc[t], 0, 0, 0);
        }
    };
    bf16x8 w[NT][KS];
    // ---- layer 0 (K = nin <= 16, one product step)
    {
        bf16x8 w0[NT];
        f32x4 bias[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int j = 0; j < 8; ++j)
                w0[t][j] = kq + j < nin ? Wb[lm.wb[0] + (feat(t) + rl) * nin + kq + j] : (__bf16)0.0f;
        load_b(0, bias);
        if (L > 1) load_w(Wb + lm.wb[1], w);
#pragma unroll
        for (int s = 0; s < RS; ++s) {
            const int row = r0 + 16 * s + rl;
            bf16x8 b;
#pragma unroll
            for (int j = 0; j < 8; ++j)
                b[j] = row < M && kq + j < nin ? (__bf16)x[(long long)row * nin + kq + j] : (__bf16)0.0f;
            f32x4 acc[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0[t], b, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            activate(0, 0, s, acc, bias);
        }
        __syncthreads();
    }
    // ---- hidden layers
    int cur = 0;
    for (int l = 1; l < L; ++l) {
        f32x4 bias[NT];
        load_b(l, bias);
        bf16x8 wn[NT][KS];
        constexpr bool AHEAD = NT * KS <= 8;  // two layers' slices fit the registers
        if (AHEAD && l + 1 < L) load_w(Wb + lm.wb[l + 1], wn);
#pragma unroll
        for (int s = 0; s < RS; ++s) {
            f32x4 acc[NT];
            product(cur, s, w, acc);
            activate(l, cur ^ 1, s, acc, bias);
        }
        if (AHEAD) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int k = 0; k < KS; ++k) w[t][k] = wn[t][k];
        } else if (l + 1 < L) {
            load_w(Wb + lm.wb[l + 1], w);
        }
        cur ^= 1;
        __syncthreads();
    }
    const __bf16 *wo = Wb + lm.wb[L];
    if constexpr (!TRAIN) {
        // ---- output layer: four lanes per row, H / 4 inputs each
        const int rr = tid >> 2, part = tid & 3;
        if (rr < ROWS) {
            float s = 0.0f;
#pragma unroll
            for (int q = 0; q < H / 32; ++q) {
                const int k = (H / 4) * part + 8 * q;
                const bf16x8 a = *(const bf16x8 *)&act[cur][rr][k];
                const bf16x8 b = *(const bf16x8 *)(wo + k);
#pragma unroll
                for (int j = 0; j < 8; ++j) s = fmaf((float)a[j], (float)b[j], s);
            }
            s += __shfl_xor(s, 1, 4);
            s += __shfl_xor(s, 2, 4);
            if (part == 0 && r0 + rr < M) y[r0 + rr] = s + P[lm.b[L]];
        }
    } else {
        // ---- output layer as the layer-by-layer path sums it (sixteen lanes per row, eight inputs per
        // 128 each), loss and its gradient 2 (y - t) / M
        if (L > 1) load_w(Wt + lm.wb[L - 1], w);
#pragma unroll
        for (int s = 0; s < RS; ++s) {
            const int rr = 16 * s + (tid >> 4), sub = tid & 15, row = r0 + rr;
            float o = 0.0f;
            for (int k = 8 * sub; k < H; k += 128) {
                const bf16x8 a = *(const bf16x8 *)&act[cur][rr][k];
                const bf16x8 b = *(const bf16x8 *)(wo + k);
#pragma unroll
                for (int j = 0; j < 8; ++j) o = fmaf((float)a[j], (float)b[j], o);
            }
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) o += __shfl_xor(o, off, 16);
            if (sub == 0) {
                const float e = row < M ? o + P[lm.b[L]] - tb.t[row] : 0.0f;
                const float g = 2.0f * e / (float)M;
                const __bf16 gb = (__bf16)g;
                el[rr] = (double)e * e;
                dyf[rr] = g;
                dyl[rr] = (float)gb;
                if (row < M) tb.dY[row] = gb;
            }
        }
        __syncthreads();
        if (tid == 0) {
            double le = 0.0;
            float ds = 0.0f;
            for (int r = 0; r < ROWS; ++r) {
                le += el[r];
                ds += dyf[r];
            }
            tb.loss[blockIdx.x] = le;
            tb.dysum[blockIdx.x] = ds;
        }
        // ---- backward: dA of the top hidden layer is the outer product of dY and the output weights
        for (int l = L - 1; l >= 0; --l) {
            f32x4 sum[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) sum[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < RS; ++s) {
                const int row = r0 + 16 * s + rl;
                f32x4 z[NT], acc[NT];
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    z[t] = *(const f32x4 *)(tb.Z[l] + (long long)min(row, M - 1) * H + feat(t) + fq);
                if (l == L - 1) {
#pragma unroll
                    for (int t = 0; t < NT; ++t)
#pragma unroll
                        for (int r = 0; r < 4; ++r) acc[t][r] = dyl[16 * s + rl] * (float)wo[feat(t) + fq + r];
                } else {
                    product(cur, s, w, acc);
                }
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    bf16x4 v;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const float d = row < M ? acc[t][r] * silu_grad(z[t][r]) : 0.0f;
                        sum[t][r] += d;
                        v[r] = (__bf16)d;
                    }
                    *(bf16x4 *)&act[cur ^ 1][16 * s + rl][feat(t) + fq] = v;
                    if (row < M) *(bf16x4 *)(tb.dZ[l] + (long long)row * H + feat(t) + fq) = v;
                }
            }
            // the transposed weights of the next product (it takes dZ_l through layer l's weights)
            if (l < L - 1 && l > 0) load_w(Wt + lm.wb[l], w);
            // column sums of dZ over the block's rows (16 lanes share a column quad)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int off = 1; off < 16; off <<= 1) sum[t][r] += __shfl_xor(sum[t][r], off, 16);
            if (rl == 0)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    *(f32x4 *)(tb.dzsum + ((long long)blockIdx.x * L + l) * H + feat(t) + fq) = sum[t];
            cur ^= 1;
            __syncthreads();
        }
    }
}

// Weight gradients dW_l[o][i] = sum_b dZ_l[b][o] A_{l-1}[b][i] of the layers l0, l0 + 1, .. (blockIdx.z):
// a block forms one 128 x 128 tile (blockIdx.x) over one chunk of rows (blockIdx.y) and writes it to
// its own FP32 partials, which k_grads sums in order, so the batch is split over the card without
// atomics.  The sum runs over rows, the strided direction of both operands: 32 rows at a time are
// staged in LDS transposed (two rows packed per dword), from where the fragments are 16-byte reads.
struct DwArgs {
    const __bf16 *dZ[9], *A[9];  // [row][O], [row][I] of each layer
    int n, chunk;                // rows, rows per chunk (a multiple of 32)
    float *part;                 // [chunk][np]
    long long np;
};

__global__ __launch_bounds__(256) void k_dw(DwArgs g, LayerMap lm, int l0) {
    constexpr int LD = 40;  // 32 rows and 16 bytes of padding
    __shared__ __attribute__((aligned(16))) __bf16 zt[128][LD], at[128][LD];
    const int l = l0 + blockIdx.z, O = lm.out[l], I = lm.in[l];
    const int tiles_i = (I + 127) / 128, tiles = ((O + 127) / 128) * tiles_i;
    if ((int)blockIdx.x >= tiles) return;  // whole block
    const int o0 = (blockIdx.x / tiles_i) * 128, i0 = (blockIdx.x % tiles_i) * 128;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, rl = lane & 15, kq = 8 * (lane >> 4);
    const int b0 = blockIdx.y * g.chunk, b1 = min(b0 + g.chunk, g.n);
    // wave (wo, wi) takes the 64 x 64 quarter; tiles past the matrix are skipped
    const int wo = 64 * (wave >> 1), wi = 64 * (wave & 1);
    const int no = max(0, min(4, (O - o0 - wo + 15) / 16)), ni = max(0, min(4, (I - i0 - wi + 15) / 16));
    f32x4 acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[a][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    // staging: thread = (row pair, group of eight columns)
    const int pr = tid & 15, gc = 8 * (tid >> 4);
    auto fetch = [&](const __bf16 *X, int ld, int c0, int row) {
        bf16x8 v = {};
        if (row < b1) {
            const __bf16 *src = X + (long long)row * ld + c0 + gc;
            if (ld % 8 == 0) {
                if (c0 + gc < ld) v = *(const bf16x8 *)src;
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (c0 + gc + j < ld) v[j] = src[j];
            }
        }
        return v;
    };
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x8 z0 = fetch(g.dZ[l], O, o0, b0 + 2 * pr), z1 = fetch(g.dZ[l], O, o0, b0 + 2 * pr + 1);
    bf16x8 x0 = fetch(g.A[l], I, i0, b0 + 2 * pr), x1 = fetch(g.A[l], I, i0, b0 + 2 * pr + 1);
    for (int b = b0; b < b1; b += 32) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            *(bf16x2 *)&zt[gc + j][2 * pr] = bf16x2{z0[j], z1[j]};
            *(bf16x2 *)&at[gc + j][2 * pr] = bf16x2{x0[j], x1[j]};
        }
        __syncthreads();
        if (b + 32 < b1) {  // the next rows are in flight during the products
            z0 = fetch(g.dZ[l], O, o0, b + 32 + 2 * pr);
            z1 = fetch(g.dZ[l], O, o0, b + 33 + 2 * pr);
            x0 = fetch(g.A[l], I, i0, b + 32 + 2 * pr);
            x1 = fetch(g.A[l], I, i0, b + 33 + 2 * pr);
        }
        bf16x8 fz[4], fx[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            fz[a] = *(const bf16x8 *)&zt[wo + 16 * a + rl][kq];
            fx[a] = *(const bf16x8 *)&at[wi + 16 * a + rl][kq];
        }
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (a < no && c < ni) acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fz[a], fx[c], acc[a][c], 0, 0, 0);
        __syncthreads();
    }
    float *out = g.part + (long long)blockIdx.y * g.np + lm.w[l];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int o = o0 + wo + 16 * a + 4 * (lane >> 4) + r, i = i0 + wi + 16 * c + rl;
                if (o < O && i < I) out[(long long)o * I + i] = acc[a][c][r];
            }
}

// Gradients from their partials, in a fixed order: weights (one thread each, over the row chunks),
// biases (64 threads each, over the blocks of the column sums), the loss; with adam != 0 the Adam step
// on them and the BF16 copies of the new weights.
struct GradArgs {
    const float *part;                   // [chunk][np]
    const float *dzsum, *dysum;          // [block][layer][hidden], [block]
    const double *lossp;                 // [block]
    int chunks, blocks, n, hidden;
    long long np;
    float *G, *P, *Mo, *Vo;
    __bf16 *Wb, *Wt;
    double *loss;
    int adam;
    float lr, c1, c2;
};

__global__ __launch_bounds__(256) void k_grads(GradArgs g, LayerMap lm) {
    const int tid = threadIdx.x;
    auto update = [&](long long i, float gi) -> float {
        g.G[i] = gi;
        if (!g.adam) return 0.0f;
        const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
        const float mi = b1 * g.Mo[i] + (1.0f - b1) * gi;
        const float vi = b2 * g.Vo[i] + (1.0f - b2) * gi * gi;
        g.Mo[i] = mi;
        g.Vo[i] = vi;
        const float pn = g.P[i] - g.lr * (mi / g.c1) / (sqrtf(vi / g.c2) + eps);
        g.P[i] = pn;
        return pn;
    };
    if (blockIdx.y < (unsigned)lm.n) {  // the weights of layer blockIdx.y
        const int l = blockIdx.y, I = lm.in[l], O = lm.out[l];
        for (int k = blockIdx.x * 256 + tid; k < I * O; k += gridDim.x * 256) {
            const float *src = g.part + lm.w[l] + k;
            float s = 0.0f;
            int c = 0;
            for (; c + 8 <= g.chunks; c += 8) {
                float v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = src[(long long)(c + j) * g.np];
#pragma unroll
                for (int j = 0; j < 8; ++j) s += v[j];
            }
            for (; c < g.chunks; ++c) s += src[(long long)c * g.np];
            const float pn = update(lm.w[l] + k, s);
            if (g.adam) {
                const __bf16 v = (__bf16)pn;
                g.Wb[lm.wb[l] + k] = v;
                g.Wt[lm.wb[l] + (long long)(k % I) * O + k / I] = v;
            }
        }
        return;
    }
    // biases: a block takes 16 columns of one hidden layer (or the output bias), 16 threads a column
    __shared__ float ps[16][17];
    __shared__ double pl[256];
    const int per = g.hidden / 16, L = lm.n - 1;
    const int col = tid & 15, grp = tid >> 4;
    for (int job = blockIdx.x; job <= L * per; job += gridDim.x) {
        const bool last = job == L * per;
        const int l = last ? L : job / per, c = last ? 0 : 16 * (job % per) + col;
        const float *src = last ? g.dysum : g.dzsum + (long long)l * g.hidden + c;
        const long long st = last ? 1 : (long long)L * g.hidden;
        float s = 0.0f;
        int b = grp;
        for (; b + 112 < g.blocks; b += 128) {
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = src[(b + 16 * j) * st];
#pragma unroll
            for (int j = 0; j < 8; ++j) s += v[j];
        }
        for (; b < g.blocks; b += 16) s += src[b * st];
        ps[grp][col] = s;
        if (last) {
            double e = 0.0;
            for (int k = tid; k < g.blocks; k += 256) e += g.lossp[k];
            pl[tid] = e;
        }
        __syncthreads();
        if (grp == 0 && (!last || col == 0)) {
            float tot = 0.0f;
#pragma unroll
            for (int k = 0; k < 16; ++k) tot += ps[k][col];
            update(lm.b[l] + c, tot);
        }
        if (last) {
            for (int wd = 128; wd > 0; wd >>= 1) {
                if (tid < wd) pl[tid] += pl[tid + wd];
                __syncthreads();
            }
            if (tid == 0) *g.loss = pl[0] / g.n;
        }
        __syncthreads();
    }
}

// dZ = dA * silu'(Z) (FP32 and BF16)
__global__ void k_silu_back(const float *__restrict__ dA, const float *__restrict__ Z, float *__restrict__ dZ,
                            __bf16 *__restrict__ dZb, int n) {
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        const float v = dA[i] * silu_grad(Z[i]);
        dZ[i] = v;
        dZb[i] = (__bf16)v;
    }
}

// Column sums of dZ [n][O] over the rows of one block (64 rows), one thread per column
__global__ __launch_bounds__(256) void k_colsum(const float *__restrict__ dZ, int n, int O, float *__restrict__ out,
                                                long long stride) {
    const int j = blockIdx.y * 256 + threadIdx.x, r0 = blockIdx.x * 64, r1 = min(r0 + 64, n);
    if (j >= O) return;
    float s = 0.f;
#pragma unroll 8
    for (int r = r0; r < r1; ++r) s += dZ[(long long)r * O + j];
    out[blockIdx.x * stride + j] = s;
}

// Mean-squared-error terms of the layer-by-layer path, 64 rows a block (one wave): dY = 2 (y - t) / n,
// the FP64 sum of (y - t)^2 and the FP32 sum of dY
__global__ __launch_bounds__(64) void k_loss(const float *__restrict__ y, const float *__restrict__ t, int n,
                                             __bf16 *__restrict__ dyb, double *__restrict__ loss,
                                             float *__restrict__ dysum) {
    const int i = blockIdx.x * 64 + threadIdx.x;
    const float e = i < n ? y[i] - t[i] : 0.0f, g = 2.0f * e / (float)n;
    if (i < n) dyb[i] = (__bf16)g;
    double s = (double)e * e;
    float d = g;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        s += __shfl_xor(s, off, 64);
        d += __shfl_xor(d, off, 64);
    }
    if (threadIdx.x == 0) {
        loss[blockIdx.x] = s;
        dysum[blockIdx.x] = d;
    }
}

}  // namespace pfm

using namespace pfm;

struct pf_mlp {
    pf_mlp_config cfg;
    hipStream_t stream = nullptr;
    char *ws = nullptr;
    LayerMap lm{};
    long long np = 0, nwb = 0;
    // workspace offsets
    size_t P, G, Mo, Vo, Wb, Wt, Xb, Y, dYb, loss, dA, dZ, dZb, Z[10], A[10];
    size_t dzl, part, dzsum, dysum, lossp;
    int max_chunks = 1;
    int adam_t = 0;
    std::string err;
};

namespace {

thread_local std::string g_mlp_init_error;

int mfail(pf_mlp *h, int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (h)
        h->err = buf;
    else
        g_mlp_init_error = buf;
    return code;
}

#define MCHK(h, call)                                                                              \
    do {                                                                                           \
        hipError_t e_ = (call);                                                                    \
        if (e_ != hipSuccess) return mfail((h), PF_LBM_EDEVICE, "%s: %s", #call, hipGetErrorString(e_)); \
    } while (0)

template <typename X>
X *at(pf_mlp *h, size_t off) {
    return (X *)(h->ws + off);
}

void gemm(pf_mlp *h, const __bf16 *A, long long sam, const __bf16 *B, long long sbn, float *Cf, __bf16 *Cb,
          long long scm, const float *bias, int M, int N, int K, int act) {
    Gemm g{A, sam, B, sbn, Cf, Cb, scm, bias, M, N, K, act, 0};
    g.vec = K % 8 == 0 && sam % 8 == 0 && sbn % 8 == 0 && scm % 8 == 0 && ((uintptr_t)A % 16) == 0 &&
            ((uintptr_t)B % 16) == 0 && ((uintptr_t)Cb % 16) == 0;
    constexpr int NT = 8;
    const dim3 grid((unsigned)(((M + 15) / 16 + 3) / 4), (unsigned)((N + 16 * NT - 1) / (16 * NT)));
    k_gemm_bf16_rows<NT><<<grid, 256, 0, h->stream>>>(g);
}

int grid_for(long long n) { return (int)std::max(1LL, std::min(4096LL, (n + 255) / 256)); }

// forward pass of n samples; leaves A_l (and with keep_z the FP32 pre-activations Z_l, which only
// the backward pass needs) and the output in the workspace
int run_forward(pf_mlp *h, const float *x, int n, bool keep_z, float *y_out = nullptr) {
    const LayerMap &lm = h->lm;
    const int nin = h->cfg.n_in;
    k_to_bf16<<<grid_for((long long)n * nin), 256, 0, h->stream>>>(x, at<__bf16>(h, h->Xb), n * nin);
    for (int l = 0; l < lm.n; ++l) {
        const int I = lm.in[l], O = lm.out[l];
        const __bf16 *Ain = l == 0 ? at<__bf16>(h, h->Xb) : at<__bf16>(h, h->A[l - 1]);
        const bool last = l == lm.n - 1;
        const __bf16 *Wl = at<__bf16>(h, h->Wb) + lm.wb[l];
        const float *bl = at<float>(h, h->P) + lm.b[l];
        float *Zl = last ? (y_out ? y_out : at<float>(h, h->Y)) : (keep_z ? at<float>(h, h->Z[l]) : nullptr);
        if (last) {
            const long long th = (long long)n * 16;
            k_last_layer<<<(unsigned)((th + 255) / 256), 256, 0, h->stream>>>(Ain, n, I, Wl, bl, Zl);
        } else {
            // Z = A_in W^T + b: B[k][n] = W[n][k]
            gemm(h, Ain, I, Wl, I, Zl, at<__bf16>(h, h->A[l]), O, bl, n, O, I, 1);
        }
    }
    MCHK(h, hipGetLastError());
    return PF_LBM_OK;
}

// row chunks of the weight gradients: about 96 blocks a layer where the rows and the partials'
// space allow, whole 32-row steps
int dw_chunks(const pf_mlp *h, int n, int &chunk) {
    const int tiles = ((h->cfg.hidden + 127) / 128) * ((h->cfg.hidden + 127) / 128);
    int c = std::max(1, std::min(std::min(h->max_chunks, 96 / tiles), (n + 63) / 64));
    chunk = ((n + c - 1) / c + 31) / 32 * 32;
    return (n + chunk - 1) / chunk;
}

// the sums over the partials, and with lr > 0 the Adam step
void finish_grads(pf_mlp *h, int n, int chunks, int blocks, float lr) {
    GradArgs g{};
    g.part = at<float>(h, h->part);
    g.dzsum = at<float>(h, h->dzsum);
    g.dysum = at<float>(h, h->dysum);
    g.lossp = at<double>(h, h->lossp);
    g.chunks = chunks;
    g.blocks = blocks;
    g.n = n;
    g.hidden = h->cfg.hidden;
    g.np = h->np;
    g.G = at<float>(h, h->G);
    g.P = at<float>(h, h->P);
    g.Mo = at<float>(h, h->Mo);
    g.Vo = at<float>(h, h->Vo);
    g.Wb = at<__bf16>(h, h->Wb);
    g.Wt = at<__bf16>(h, h->Wt);
    g.loss = at<double>(h, h->loss);
    g.adam = lr > 0.0f;
    if (g.adam) {
        ++h->adam_t;
        g.lr = lr;
        g.c1 = 1.0f - std::pow(0.9f, (float)h->adam_t);
        g.c2 = 1.0f - std::pow(0.999f, (float)h->adam_t);
    }
    const int H = h->cfg.hidden, gx = std::max((H * H + 255) / 256, (h->lm.n - 1) * (H / 16) + 1);
    k_grads<<<dim3((unsigned)std::min(gx, 1024), (unsigned)h->lm.n + 1), 256, 0, h->stream>>>(g, h->lm);
}

// layer-by-layer backward pass after run_forward: error terms, partial weight gradients and sums
void run_backward(pf_mlp *h, const float *t, int n, int chunks, int chunk) {
    const LayerMap &lm = h->lm;
    const int H = h->cfg.hidden, L = lm.n - 1, nb = (n + 63) / 64;
    k_loss<<<nb, 64, 0, h->stream>>>(at<float>(h, h->Y), t, n, at<__bf16>(h, h->dYb), at<double>(h, h->lossp),
                                     at<float>(h, h->dysum));
    const __bf16 *dZb = at<__bf16>(h, h->dYb);
    const int tiles = ((H + 127) / 128) * ((H + 127) / 128);
    for (int l = L; l >= 0; --l) {
        const int I = lm.in[l], O = lm.out[l];
        DwArgs d{};
        d.dZ[l] = dZb;
        d.A[l] = l == 0 ? at<__bf16>(h, h->Xb) : at<__bf16>(h, h->A[l - 1]);
        d.n = n;
        d.chunk = chunk;
        d.part = at<float>(h, h->part);
        d.np = h->np;
        k_dw<<<dim3((unsigned)tiles, (unsigned)chunks, 1), 256, 0, h->stream>>>(d, lm, l);
        if (l == 0) break;
        // dA_in[b][i] = sum_o dZ[b][o] W[o][i]: B-operand (k = o, n = i) from the transposed copy
        gemm(h, dZb, O, at<__bf16>(h, h->Wt) + lm.wb[l], O, at<float>(h, h->dA), nullptr, I, nullptr, n, I, O, 0);
        // dZ of the layer below and its column sums
        float *dZn = at<float>(h, h->dZ) + (size_t)(l & 1) * h->cfg.max_batch * H;
        __bf16 *dZbn = at<__bf16>(h, h->dZb) + (size_t)(l & 1) * h->cfg.max_batch * H;
        k_silu_back<<<grid_for((long long)n * I), 256, 0, h->stream>>>(at<float>(h, h->dA), at<float>(h, h->Z[l - 1]), dZn,
                                                                        dZbn, n * I);
        k_colsum<<<dim3((unsigned)nb, (unsigned)((H + 255) / 256)), 256, 0, h->stream>>>(
            dZn, n, H, at<float>(h, h->dzsum) + (size_t)(l - 1) * H, (long long)L * H);
        dZb = dZbn;
    }
}

// rows a fused block carries: 16, and 64 where 16-row blocks would exceed two per CU
int fused_rows(int n) { return n > 16 * 512 ? 64 : 16; }

template <int H, bool TRAIN, class B>
void launch_fused(pf_mlp *h, const float *x, int n, float *y, const B &tb, const int *n_dev) {
    const int rows = fused_rows(n);
    const unsigned g = (unsigned)((n + rows - 1) / rows);
    if (rows == 64)
        k_mlp_fused<H, 4, TRAIN><<<g, 256, 0, h->stream>>>(x, n, h->cfg.n_in, h->lm, at<__bf16>(h, h->Wb),
                                                           at<__bf16>(h, h->Wt), at<float>(h, h->P), y, tb, n_dev);
    else
        k_mlp_fused<H, 1, TRAIN><<<g, 256, 0, h->stream>>>(x, n, h->cfg.n_in, h->lm, at<__bf16>(h, h->Wb),
                                                           at<__bf16>(h, h->Wt), at<float>(h, h->P), y, tb, n_dev);
}

// the one-launch network passes exist for these widths; others run layer by layer
bool fused_width(int H) { return H == 64 || H == 128 || H == 256; }

template <bool TRAIN, class B>
void launch_fused_any(pf_mlp *h, const float *x, int n, float *y, const B &tb, const int *n_dev = nullptr) {
    if (h->cfg.hidden == 64)
        launch_fused<64, TRAIN>(h, x, n, y, tb, n_dev);
    else if (h->cfg.hidden == 128)
        launch_fused<128, TRAIN>(h, x, n, y, tb, n_dev);
    else
        launch_fused<256, TRAIN>(h, x, n, y, tb, n_dev);
}

// loss, parameter gradients into G and with lr > 0 the Adam step
int loss_and_grad(pf_mlp *h, const float *x, const float *t, int n, float lr) {
    const LayerMap &lm = h->lm;
    const int H = h->cfg.hidden, L = lm.n - 1;
    int chunk = 0;
    const int chunks = dw_chunks(h, n, chunk);
    if (fused_width(H)) {
        TrainBuf tb{};
        tb.t = t;
        DwArgs d{};
        for (int l = 0; l < L; ++l) {
            tb.Z[l] = at<float>(h, h->Z[l]);
            tb.A[l] = at<__bf16>(h, h->A[l]);
            tb.dZ[l] = at<__bf16>(h, h->dzl) + (size_t)l * h->cfg.max_batch * H;
            d.dZ[l] = tb.dZ[l];
            d.A[l + 1] = tb.A[l];
        }
        tb.dY = at<__bf16>(h, h->dYb);
        tb.loss = at<double>(h, h->lossp);
        tb.dysum = at<float>(h, h->dysum);
        tb.dzsum = at<float>(h, h->dzsum);
        k_to_bf16<<<grid_for((long long)n * h->cfg.n_in), 256, 0, h->stream>>>(x, at<__bf16>(h, h->Xb), n * h->cfg.n_in);
        launch_fused_any<true>(h, x, n, nullptr, tb);
        d.dZ[L] = tb.dY;
        d.A[0] = at<__bf16>(h, h->Xb);
        d.n = n;
        d.chunk = chunk;
        d.part = at<float>(h, h->part);
        d.np = h->np;
        const int tiles = ((H + 127) / 128) * ((H + 127) / 128);
        k_dw<<<dim3((unsigned)tiles, (unsigned)chunks, (unsigned)lm.n), 256, 0, h->stream>>>(d, lm, 0);
        finish_grads(h, n, chunks, (n + fused_rows(n) - 1) / fused_rows(n), lr);
    } else {
        const int rc = run_forward(h, x, n, true);
        if (rc != PF_LBM_OK) return rc;
        run_backward(h, t, n, chunks, chunk);
        finish_grads(h, n, chunks, (n + 63) / 64, lr);
    }
    MCHK(h, hipGetLastError());
    return PF_LBM_OK;
}

uint64_t splitmix64(uint64_t &s) {
    uint64_t z = (s += 0x9E3779B97F4A7C15ull);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

int upload_params(pf_mlp *h, const float *params) {
    MCHK(h, hipMemcpyAsync(h->ws + h->P, params, sizeof(float) * h->np, hipMemcpyHostToDevice, h->stream));
    MCHK(h, hipMemsetAsync(h->ws + h->Mo, 0, sizeof(float) * h->np, h->stream));
    MCHK(h, hipMemsetAsync(h->ws + h->Vo, 0, sizeof(float) * h->np, h->stream));
    k_refresh_weights<<<grid_for(h->nwb), 256, 0, h->stream>>>(h->lm, at<float>(h, h->P), at<__bf16>(h, h->Wb),
                                                                 at<__bf16>(h, h->Wt));
    MCHK(h, hipGetLastError());
    MCHK(h, hipStreamSynchronize(h->stream));
    h->adam_t = 0;
    return PF_LBM_OK;
}

}  // namespace

__attribute__((visibility("hidden"))) void pfm_internal_info(const pf_mlp *h, int *n_in, int *max_batch,
                                                             void **stream) {
    *n_in = h ? h->cfg.n_in : 0;
    *max_batch = h ? h->cfg.max_batch : 0;
    *stream = h ? (void *)h->stream : nullptr;
}

__attribute__((visibility("hidden"))) bool pfm_internal_forward_counted(pf_mlp *h, const float *x, int max_rows,
                                                                        const int *n_dev, float *y) {
    if (!fused_width(h->cfg.hidden)) return false;
    launch_fused_any<false>(h, x, max_rows, y, NoTrain{}, n_dev);
    return true;
}

extern "C" {

int pf_mlp_init(const pf_mlp_config *cfg, uint64_t seed, void *workspace, size_t ws_bytes, void *hip_stream,
                pf_mlp **out, size_t *ws_bytes_needed) {
    g_mlp_init_error.clear();
    if (!cfg) return mfail(nullptr, PF_LBM_EINVAL, "cfg is NULL");
    if (cfg->struct_size < sizeof(pf_mlp_config)) return mfail(nullptr, PF_LBM_EINVAL, "bad struct_size");
    if (cfg->n_in < 1 || cfg->n_in > 16) return mfail(nullptr, PF_LBM_EINVAL, "n_in must be in [1, 16]");
    if (cfg->hidden < 16 || cfg->hidden > 512 || cfg->hidden % 16)
        return mfail(nullptr, PF_LBM_EINVAL, "hidden must be a multiple of 16 in [16, 512]");
    if (cfg->layers < 1 || cfg->layers > 8) return mfail(nullptr, PF_LBM_EINVAL, "layers must be in [1, 8]");
    if (cfg->max_batch < 1 || cfg->max_batch > 65536) return mfail(nullptr, PF_LBM_EINVAL, "max_batch in [1, 65536]");
    pf_mlp tmp;
    tmp.cfg = *cfg;
    LayerMap &lm = tmp.lm;
    lm.n = cfg->layers + 1;
    long long np = 0, nwb = 0;
    for (int l = 0; l < lm.n; ++l) {
        lm.in[l] = l == 0 ? cfg->n_in : cfg->hidden;
        lm.out[l] = l == lm.n - 1 ? 1 : cfg->hidden;
        lm.w[l] = np;
        np += (long long)lm.in[l] * lm.out[l];
        lm.b[l] = np;
        np += lm.out[l];
        lm.wb[l] = nwb;
        nwb += (long long)lm.in[l] * lm.out[l];
    }
    tmp.np = np;
    tmp.nwb = nwb;
    const long long B = cfg->max_batch, H = cfg->hidden;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = (off + bytes + 255) / 256 * 256;
        return o;
    };
    tmp.P = take(4 * np);
    tmp.G = take(4 * np);
    tmp.Mo = take(4 * np);
    tmp.Vo = take(4 * np);
    tmp.Wb = take(2 * nwb);
    tmp.Wt = take(2 * nwb);
    tmp.Xb = take(2 * B * cfg->n_in);
    tmp.Y = take(4 * B);
    tmp.dYb = take(2 * B);
    tmp.loss = take(8);
    // error terms: layer by layer FP32 dA, two FP32 and two BF16 dZ; fused, one BF16 dZ a layer (at
    // most 8), in the same space
    tmp.dzl = tmp.dA = take(4 * B * H);
    tmp.dZ = take(4 * 2 * B * H);
    tmp.dZb = take(2 * 2 * B * H);
    // partial gradients: up to 96 row chunks within 32 MB (at least one), sums per 16 rows (fused, up
    // to 8192 rows) or 64 rows
    tmp.max_chunks = (int)std::max(1LL, std::min(96LL, (32LL << 20) / (4 * np)));
    tmp.part = take((size_t)4 * np * tmp.max_chunks);
    const long long sb = std::max(std::min((B + 15) / 16, 512LL), (B + 63) / 64);
    tmp.dzsum = take((size_t)4 * sb * cfg->layers * H);
    tmp.dysum = take((size_t)4 * sb);
    tmp.lossp = take((size_t)8 * sb);
    for (int l = 0; l < lm.n - 1; ++l) {
        tmp.Z[l] = take(4 * B * H);
        tmp.A[l] = take(2 * B * H);
    }
    if (ws_bytes_needed) *ws_bytes_needed = off;
    if (!workspace) return PF_LBM_OK;
    if (!out) return mfail(nullptr, PF_LBM_EINVAL, "out is NULL");
    if (ws_bytes < off) return mfail(nullptr, PF_LBM_ENOMEM, "workspace of %zu bytes, %zu needed", ws_bytes, off);
    if ((uintptr_t)workspace % 256) return mfail(nullptr, PF_LBM_EINVAL, "workspace must be 256-byte aligned");
    pf_mlp *h = new (std::nothrow) pf_mlp(tmp);
    if (!h) return mfail(nullptr, PF_LBM_ENOMEM, "host allocation failed");
    h->ws = (char *)workspace;
    h->stream = (hipStream_t)hip_stream;
    // seeded initialisation: W ~ U(-sqrt(6 / in), sqrt(6 / in)), b = 0
    std::vector<float> p((size_t)np, 0.0f);
    uint64_t s = seed;
    for (int l = 0; l < lm.n; ++l) {
        const double a = std::sqrt(6.0 / lm.in[l]);
        for (long long i = 0; i < (long long)lm.in[l] * lm.out[l]; ++i) {
            const double u = (double)(splitmix64(s) >> 11) * (1.0 / 9007199254740992.0);
            p[lm.w[l] + i] = (float)((2.0 * u - 1.0) * a);
        }
    }
    const int rc = upload_params(h, p.data());
    if (rc != PF_LBM_OK) {
        g_mlp_init_error = h->err;
        delete h;
        return rc;
    }
    *out = h;
    return PF_LBM_OK;
}

int32_t pf_mlp_num_params(const pf_mlp *h) { return h ? (int32_t)h->np : 0; }

int pf_mlp_set_params(pf_mlp *h, const float *params) {
    if (!h || !params) return mfail(h, PF_LBM_EINVAL, "handle or params is NULL");
    return upload_params(h, params);
}

int pf_mlp_get_params(pf_mlp *h, float *params) {
    if (!h || !params) return mfail(h, PF_LBM_EINVAL, "handle or params is NULL");
    MCHK(h, hipMemcpyAsync(params, h->ws + h->P, sizeof(float) * h->np, hipMemcpyDeviceToHost, h->stream));
    MCHK(h, hipStreamSynchronize(h->stream));
    return PF_LBM_OK;
}

int pf_mlp_forward(pf_mlp *h, const float *x, int32_t n, float *y) {
    if (!h || !x || !y) return mfail(h, PF_LBM_EINVAL, "NULL argument");
    if (n < 1 || n > h->cfg.max_batch) return mfail(h, PF_LBM_EINVAL, "n must be in [1, max_batch]");
    // the one-launch pass reads inputs while other blocks write outputs; the layer-by-layer path copies the
    // inputs first, so outputs may lie over them
    const uintptr_t x0 = (uintptr_t)x, y0 = (uintptr_t)y;
    const bool apart = y0 + sizeof(float) * (size_t)n <= x0 || x0 + sizeof(float) * (size_t)n * h->cfg.n_in <= y0;
    if (fused_width(h->cfg.hidden) && apart) {
        launch_fused_any<false>(h, x, n, y, NoTrain{});
        MCHK(h, hipGetLastError());
        return PF_LBM_OK;
    }
    return run_forward(h, x, n, false, y);
}

int pf_mlp_gradients(pf_mlp *h, const float *x, const float *t, int32_t n, float *grad, double *loss) {
    if (!h || !x || !t || !grad) return mfail(h, PF_LBM_EINVAL, "NULL argument");
    if (n < 1 || n > h->cfg.max_batch) return mfail(h, PF_LBM_EINVAL, "n must be in [1, max_batch]");
    const int rc = loss_and_grad(h, x, t, n, 0.0f);
    if (rc != PF_LBM_OK) return rc;
    MCHK(h, hipMemcpyAsync(grad, h->ws + h->G, sizeof(float) * h->np, hipMemcpyDeviceToHost, h->stream));
    if (loss) MCHK(h, hipMemcpyAsync(loss, h->ws + h->loss, sizeof(double), hipMemcpyDeviceToHost, h->stream));
    MCHK(h, hipStreamSynchronize(h->stream));
    return PF_LBM_OK;
}

int pf_mlp_train_step(pf_mlp *h, const float *x, const float *t, int32_t n, float lr, double *loss) {
    if (!h || !x || !t) return mfail(h, PF_LBM_EINVAL, "NULL argument");
    if (n < 1 || n > h->cfg.max_batch) return mfail(h, PF_LBM_EINVAL, "n must be in [1, max_batch]");
    if (!(lr > 0.0f)) return mfail(h, PF_LBM_EINVAL, "lr must be positive");
    const int rc = loss_and_grad(h, x, t, n, lr);
    if (rc != PF_LBM_OK) return rc;
    if (loss) {
        MCHK(h, hipMemcpyAsync(loss, h->ws + h->loss, sizeof(double), hipMemcpyDeviceToHost, h->stream));
        MCHK(h, hipStreamSynchronize(h->stream));
    }
    return PF_LBM_OK;
}

void pf_mlp_destroy(pf_mlp *h) { delete h; }

const char *pf_mlp_last_error(const pf_mlp *h) { return h ? h->err.c_str() : g_mlp_init_error.c_str(); }

}  // extern "C"
