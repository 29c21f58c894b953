// mlp.hip -- training and inference kernels of the learned Newton initial
// guess (the grte_mlp_* calls of include/grte.h).
//
// Training data are rows of six binary32 values, (f_0..f_4, log(T^{n+1}/T^n)),
// written by grte_log_pairs from converged steps of the solver itself.  One
// training step on a minibatch of B rows is two kernels:
//   mlp_grad_kernel  forward and backward pass of 16 rows at a time, the three
//                    64 x 64 products on the binary32 matrix instructions ->
//                    per-block partial gradient (deterministic, no atomics);
//   mlp_adam_kernel  sums the partials in a fixed order, applies Adam with bias
//                    correction to the binary32 master parameters and writes
//                    their bfloat16 copy (round to nearest even).
// The loss is the mean squared error of the standardised target.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <mutex>
#include <new>
#include <vector>

#include "../../include/grte.h"
#include "mlp_common.hpp"

namespace {
constexpr int GROWS = 16;              // rows of one pass of a gradient block
constexpr int GRAD_BLOCKS = 256;       // most gradient blocks of one minibatch (each takes rows until none is left)
}

// Workspace of grte_mlp_train_noalloc: per-block partial gradients, partial
// losses and the loss history, in one file-scope device array that each device
// holds until the process ends.  In host code the array's name only stands
// for it: its address on a device comes from hipGetSymbolAddress, taken once
// per device with that device current, and kept.
constexpr int NOALLOC_MAX_BATCH = 16384;                      // rows per minibatch
constexpr int NOALLOC_MAX_BLOCKS = GRAD_BLOCKS;
constexpr int NOALLOC_MAX_STEPS = 65536;                      // loss-history entries
constexpr size_t NOALLOC_FLOATS =
    (size_t)NOALLOC_MAX_BLOCKS * MLP_NPARAM + NOALLOC_MAX_BLOCKS + NOALLOC_MAX_STEPS;   // 4.98 MB

static __device__ __align__(256) float scratch[NOALLOC_FLOATS];

namespace {

using f32x4 = __attribute__((ext_vector_type(4))) float;
using f32x16 = __attribute__((ext_vector_type(16))) float;
using bf16x8 = __attribute__((ext_vector_type(8))) __bf16;

int grad_blocks(int B) { return std::min((B + GROWS - 1) / GROWS, GRAD_BLOCKS); }

// One gradient block: four wavefronts, GROWS rows at a time.  Lane l = 16 q + u of
// wavefront w holds hidden unit 16 w + u of the rows 4 q .. 4 q + 3, in both layers and
// both passes -- the result layout of the 16 x 16 x 4 matrix instruction, so activations,
// their derivatives and the sums over rows stay in registers and only h1 and dL/dz2
// pass through LDS, as operands.  The weights of the products are read once per block.
//   z2 = h1 W2^T, dL/dh1 = dL/dz2 W2     (16 x 64 per wavefront's 16 columns)
//   dL/dW2 = dL/dz2^T h1                 (16 rows of W2 per wavefront, sums kept over all rows)
// Bound: the chain of one pass (weights and rows from memory, 32 dependent matrix
// instructions, four barriers), hence the least rows per block that the instruction
// takes and as many blocks as compute units.  4096 rows on an MI355X: 9.3 us; one
// wavefront per 64 rows with each row's 64-unit vectors in one lane took 138 us.
constexpr int GS = MLP_H + 4;          // LDS row stride

__global__ void __launch_bounds__(256) mlp_grad_kernel(const float *theta, const float *norm, const float *data,
                                                       long long n, long long start, int B, float *gpart,
                                                       float *lpart)
{
    __shared__ __align__(16) float sH[GROWS * GS], sD[GROWS * GS], sY[4][GROWS], sX[GROWS][8];
    const int t = threadIdx.x, w = t >> 6, u = t & 15, q = (t & 63) >> 4, unit = 16 * w + u;
    // W2 as operands, k-slot (g, q, e) = input 16 g + 4 q + e
    float wf[16], wb[16], w1[MLP_IN];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            wf[4 * g + e] = theta[MLP_OW2 + MLP_H * unit + 16 * g + 4 * q + e];
            wb[4 * g + e] = theta[MLP_OW2 + MLP_H * (16 * g + 4 * q + e) + unit];
        }
#pragma unroll
    for (int c = 0; c < MLP_IN; ++c) w1[c] = theta[MLP_OW1 + MLP_IN * unit + c];
    const float b1 = theta[MLP_OB1 + unit], b2 = theta[MLP_OB2 + unit], w3 = theta[MLP_OW3 + unit], b3 = theta[MLP_OB3];
    f32x4 gW2[4] = {};
    float gW1[MLP_IN] = {}, gb1 = 0.0f, gb2 = 0.0f, gW3 = 0.0f, gb3 = 0.0f, loss = 0.0f;
    for (int r0 = blockIdx.x * GROWS; r0 < B; r0 += gridDim.x * GROWS) {
        if (t < GROWS * 6) {                           // standardised inputs and target
            const int r = t / 6, c = t - 6 * r, k = c < MLP_IN ? c : 2 * MLP_IN;
            float v = 0.0f;
            if (r0 + r < B) v = (data[(start + r0 + r) % n * 6 + c] - norm[k]) / norm[c < MLP_IN ? k + MLP_IN : k + 1];
            sX[r][c] = v;
        }
        __syncthreads();
        float x[4][MLP_IN], d1[4], d2[4], h2[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float z = b1;
#pragma unroll
            for (int c = 0; c < MLP_IN; ++c) {
                x[r][c] = sX[4 * q + r][c];
                z = fmaf(w1[c], x[r][c], z);
            }
            sH[(4 * q + r) * GS + unit] = gelu_both(z, d1[r]);
        }
        __syncthreads();
        f32x4 z2 = {b2, b2, b2, b2};
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 h = *reinterpret_cast<const float4 *>(&sH[u * GS + 16 * g + 4 * q]);
            z2 = __builtin_amdgcn_mfma_f32_16x16x4f32(h.x, wf[4 * g], z2, 0, 0, 0);
            z2 = __builtin_amdgcn_mfma_f32_16x16x4f32(h.y, wf[4 * g + 1], z2, 0, 0, 0);
            z2 = __builtin_amdgcn_mfma_f32_16x16x4f32(h.z, wf[4 * g + 2], z2, 0, 0, 0);
            z2 = __builtin_amdgcn_mfma_f32_16x16x4f32(h.w, wf[4 * g + 3], z2, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            h2[r] = gelu_both(z2[r], d2[r]);
            float y = w3 * h2[r];                      // over the wavefront's 16 units
            y += __shfl_xor(y, 1);
            y += __shfl_xor(y, 2);
            y += __shfl_xor(y, 4);
            y += __shfl_xor(y, 8);
            if (u == 0) sY[w][4 * q + r] = y;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 4 * q + r;
            const float e = b3 + ((sY[0][row] + sY[1][row]) + (sY[2][row] + sY[3][row])) - sX[row][MLP_IN];
            const bool in = r0 + row < B;
            const float dy = in ? 2.0f * e / (float)B : 0.0f;
            loss += in ? e * e : 0.0f;
            gb3 += dy;
            gW3 = fmaf(dy, h2[r], gW3);
            d2[r] *= dy * w3;
            gb2 += d2[r];
            sD[row * GS + unit] = d2[r];
        }
        __syncthreads();
        f32x4 dh = {};
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 d = *reinterpret_cast<const float4 *>(&sD[u * GS + 16 * g + 4 * q]);
            dh = __builtin_amdgcn_mfma_f32_16x16x4f32(d.x, wb[4 * g], dh, 0, 0, 0);
            dh = __builtin_amdgcn_mfma_f32_16x16x4f32(d.y, wb[4 * g + 1], dh, 0, 0, 0);
            dh = __builtin_amdgcn_mfma_f32_16x16x4f32(d.z, wb[4 * g + 2], dh, 0, 0, 0);
            dh = __builtin_amdgcn_mfma_f32_16x16x4f32(d.w, wb[4 * g + 3], dh, 0, 0, 0);
        }
#pragma unroll
        for (int c = 0; c < GROWS / 4; ++c) {
            const float d = sD[(4 * c + q) * GS + unit];
#pragma unroll
            for (int g = 0; g < 4; ++g)
                gW2[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(d, sH[(4 * c + q) * GS + 16 * g + u], gW2[g], 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float d = dh[r] * d1[r];
            gb1 += d;
#pragma unroll
            for (int c = 0; c < MLP_IN; ++c) gW1[c] = fmaf(d, x[r][c], gW1[c]);
        }
        // (no barrier here: each array is written again only behind one that follows its last reads)
    }
    // the sums over the four lanes of a unit, then this block's gradient
    auto rows = [](float v) {
        v += __shfl_xor(v, 16);
        return v + __shfl_xor(v, 32);
    };
    float *g = gpart + (size_t)blockIdx.x * MLP_NPARAM;
#pragma unroll
    for (int c = 0; c < MLP_IN; ++c) gW1[c] = rows(gW1[c]);
    gb1 = rows(gb1);
    gb2 = rows(gb2);
    gW3 = rows(gW3);
    gb3 = rows(gb3);
    loss = rows(loss);
    if (q == 0) {
#pragma unroll
        for (int c = 0; c < MLP_IN; ++c) g[MLP_OW1 + MLP_IN * unit + c] = gW1[c];
        g[MLP_OB1 + unit] = gb1;
        g[MLP_OB2 + unit] = gb2;
        g[MLP_OW3 + unit] = gW3;
    }
    if (t == 0) {
        g[MLP_OB3] = gb3;
        lpart[blockIdx.x] = loss;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) g[MLP_OW2 + MLP_H * (16 * w + 4 * q + r) + 16 * k + u] = gW2[k][r];
}

// Adam on AE parameters per block: thread (a, s) sums the partials s, s + AS, .. of
// parameter a, then the AS sums are joined in order.  Bound by the latency of the
// partials' loads: 16 per thread in flight, 128 bytes of a partial per block.  256
// partials: 5.3 us (64 bytes 6.4; 64 partials by one thread per parameter 20).
constexpr int AE = 32, AS = 16;

__global__ void __launch_bounds__(AE *AS) mlp_adam_kernel(float *theta, float *am, float *av, uint16_t *wbf,
                                                          const float *gpart, int nblk, const float *lpart, int B,
                                                          float *lhist, int hidx, float lr, float c1, float c2)
{
    __shared__ float part[AS][AE + 1];
    const int a = threadIdx.x % AE, s = threadIdx.x / AE, e = blockIdx.x * AE + a;
    float g = 0.0f;
    if (e < MLP_NPARAM) {
#pragma unroll 16
        for (int b = s; b < nblk; b += AS) g += gpart[(size_t)b * MLP_NPARAM + e];
    } else if (lhist && e == MLP_NPARAM) {             // the spare column of the last block: the loss
        for (int b = s; b < nblk; b += AS) g += lpart[b];
    }
    part[s][a] = g;
    __syncthreads();
    if (s > 0) return;
#pragma unroll
    for (int k = 1; k < AS; ++k) g += part[k][a];
    if (lhist && e == MLP_NPARAM) lhist[hidx] = g / (float)B;
    if (e >= MLP_NPARAM) return;
    const float beta1 = 0.9f, beta2 = 0.999f;
    const float m = beta1 * am[e] + (1.0f - beta1) * g;
    const float v = beta2 * av[e] + (1.0f - beta2) * g * g;
    am[e] = m;
    av[e] = v;
    // c1 = 1 - beta1^k, c2 = 1 - beta2^k (bias correction, computed on the host in binary64)
    const float th = theta[e] - lr * (m / c1) / (sqrtf(v / c2) + 1e-8f);
    theta[e] = th;
    wbf[e] = f_to_bf16(th);
}
constexpr int ADAM_GRID = (MLP_NPARAM + AE) / AE;      // covers MLP_NPARAM + 1 columns

__global__ void mlp_round_kernel(const float *theta, uint16_t *wbf)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < MLP_NPARAM) wbf[e] = f_to_bf16(theta[e]);
}

// mean and standard deviation of the six columns (binary64 sums in row order)
__global__ void __launch_bounds__(256) mlp_norm_kernel(const float *data, long long n, float *norm)
{
    __shared__ double s1[256][6], s2[256][6];
    const int t = threadIdx.x;
    double a[6] = {0, 0, 0, 0, 0, 0}, b[6] = {0, 0, 0, 0, 0, 0};
    for (long long r = t; r < n; r += 256)
        for (int q = 0; q < 6; ++q) {
            const double v = data[r * 6 + q];
            a[q] += v;
            b[q] += v * v;
        }
    for (int q = 0; q < 6; ++q) {
        s1[t][q] = a[q];
        s2[t][q] = b[q];
    }
    __syncthreads();
    if (t < 6) {
        double sa = 0.0, sb = 0.0;
        for (int k = 0; k < 256; ++k) {
            sa += s1[k][t];
            sb += s2[k][t];
        }
        const double mean = sa / (double)n;
        const double var = fmax(sb / (double)n - mean * mean, 0.0);
        const double sd = var > 0.0 ? sqrt(var) : 1.0;
        if (t < 5) {
            norm[t] = (float)mean;
            norm[5 + t] = (float)sd;
        } else {
            norm[10] = (float)mean;
            norm[11] = (float)sd;
        }
    }
}

// Inference: a wavefront takes 32 rows at a time through both layers on the 32 x 32 x 16
// bfloat16 matrix instruction, units by rows, binary32 sums.  The weights are bfloat16;
// each binary32 input is split into three bfloat16 terms whose sum it is (8 + 8 + 8 of
// its 24 bits), so every product is exact and the sums are those of binary32 arithmetic.
// Layer 1 is one instruction per 32 units: 15 slots of the 16 hold the terms of the five
// inputs, the last the bias.  Lane 32 h + c gets the units 8 (r / 4) + 4 h + r % 4 of row
// c, which are the operand of layer 2 as they stand (W2's columns in the same order), so
// nothing passes through LDS but b2 and W3.
// Bound: the gelu evaluations (128 per row, 14 vector instructions each, one of them a
// quarter-rate exp2); 2^20 rows on an MI355X: 85 us per call (213 us with one row per lane
// and vector products); two or three wavefronts per SIMD make no difference.
struct Split {
    unsigned hi, mid, lo;              // bfloat16 terms in the upper halves
};
__device__ __forceinline__ Split split3(float v)
{
    Split s;
    s.hi = __float_as_uint(v);
    const float r = v - __uint_as_float(s.hi & 0xffff0000u);
    s.mid = __float_as_uint(r);
    s.lo = __float_as_uint(r - __uint_as_float(s.mid & 0xffff0000u));
    return s;
}
// the upper halves of a and b as two bfloat16 values, a first
__device__ __forceinline__ unsigned pack_hi(unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// One row by the whole wavefront, lane l unit l of both layers, in plain binary32 sums: what
// the rows need whose values are not finite on the way.  The split turns an infinity into
// NaN (inf - inf), and so does an infinite weight with a zero term.  Behind the main loop, not in
// it, where its registers cost 3 us of 85.
__device__ __forceinline__ float eval_row(const uint16_t *wbf, const float *norm, const float *f, int l)
{
    float z = bf16_to_f(wbf[MLP_OB1 + l]);
#pragma unroll
    for (int k = 0; k < MLP_IN; ++k) z += bf16_to_f(wbf[MLP_OW1 + MLP_IN * l + k]) * ((f[k] - norm[k]) / norm[MLP_IN + k]);
    const float h = gelu_f(z);
    z = bf16_to_f(wbf[MLP_OB2 + l]);
    for (int j = 0; j < MLP_H; ++j) z += bf16_to_f(wbf[MLP_OW2 + MLP_H * l + j]) * __shfl(h, j);
    const float t = bf16_to_f(wbf[MLP_OW3 + l]) * gelu_f(z);
    float y = bf16_to_f(wbf[MLP_OB3]);
    for (int j = 0; j < MLP_H; ++j) y += __shfl(t, j);
    return y;
}

__global__ void __launch_bounds__(256) mlp_predict_kernel(const uint16_t *wbf, const float *norm, const float *data,
                                                          long long n, float *y)
{
    __shared__ __align__(16) float sB2[MLP_H], sW3[MLP_H];
    const int t = threadIdx.x, l = t & 63, c = l & 31, h = l >> 5;
    if (t < MLP_H) {
        sB2[t] = bf16_to_f(wbf[MLP_OB2 + t]);
        sW3[t] = bf16_to_f(wbf[MLP_OW3 + t]);
    }
    float mean[MLP_IN], sd[MLP_IN];
#pragma unroll
    for (int k = 0; k < MLP_IN; ++k) {
        mean[k] = norm[k];
        sd[k] = norm[MLP_IN + k];
    }
    const float b3 = bf16_to_f(wbf[MLP_OB3]);
    // layer 1, slots of the lower lanes: hi 0..4, mid 0..2; of the upper: mid 3, 4, lo 0..4, bias
    uint4 w1[2], w2[2][4];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const uint16_t *r = wbf + MLP_OW1 + MLP_IN * (32 * m + c);
        const unsigned bias = wbf[MLP_OB1 + 32 * m + c];
        const unsigned a0 = r[0], a1 = r[1], a2 = r[2], a3 = r[3], a4 = r[4];
        w1[m] = h == 0 ? make_uint4(a0 | a1 << 16, a2 | a3 << 16, a4 | a0 << 16, a1 | a2 << 16)
                       : make_uint4(a3 | a4 << 16, a0 | a1 << 16, a2 | a3 << 16, a4 | bias << 16);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint2 *q = reinterpret_cast<const uint2 *>(wbf + MLP_OW2 + MLP_H * (32 * m + c) + 16 * k + 4 * h);
            const uint2 lo = q[0], hi = q[2];
            w2[m][k] = make_uint4(lo.x, lo.y, hi.x, hi.y);
        }
    }
    __syncthreads();
    auto mma = [](const uint4 &a, const uint4 &b, const f32x16 &acc) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc,
                                                       0, 0, 0);
    };
    const long long tiles = (n + 31) / 32, stride = (long long)gridDim.x * 4;
    bool bad = false;
    for (long long tile = (long long)blockIdx.x * 4 + (t >> 6); tile < tiles; tile += stride) {
        const long long row = tile * 32 + c;
        const float *f = data + (row < n ? row : n - 1) * 6;
        Split x[MLP_IN];
#pragma unroll
        for (int k = 0; k < MLP_IN; ++k) x[k] = split3((f[k] - mean[k]) / sd[k]);
        const uint4 xb = h == 0 ? make_uint4(pack_hi(x[0].hi, x[1].hi), pack_hi(x[2].hi, x[3].hi),
                                             pack_hi(x[4].hi, x[0].mid), pack_hi(x[1].mid, x[2].mid))
                                : make_uint4(pack_hi(x[3].mid, x[4].mid), pack_hi(x[0].lo, x[1].lo),
                                             pack_hi(x[2].lo, x[3].lo), pack_hi(x[4].lo, 0x3f800000u));
        f32x16 z2[2];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 b = *reinterpret_cast<const float4 *>(&sB2[32 * m + 8 * g + 4 * h]);
                z2[m][4 * g] = b.x;
                z2[m][4 * g + 1] = b.y;
                z2[m][4 * g + 2] = b.z;
                z2[m][4 * g + 3] = b.w;
            }
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const f32x16 zero = {};
            const f32x16 z1 = mma(w1[m], xb, zero);
#pragma unroll
            for (int k = 0; k < 2; ++k) {              // eight of the lane's units: one slot group of layer 2
                unsigned hi[4], mid[4], lo[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const Split a = split3(gelu_finite(z1[8 * k + 2 * j])), b = split3(gelu_finite(z1[8 * k + 2 * j + 1]));
                    hi[j] = pack_hi(a.hi, b.hi);
                    mid[j] = pack_hi(a.mid, b.mid);
                    lo[j] = pack_hi(a.lo, b.lo);
                }
                const uint4 vl = make_uint4(lo[0], lo[1], lo[2], lo[3]), vm = make_uint4(mid[0], mid[1], mid[2], mid[3]),
                            vh = make_uint4(hi[0], hi[1], hi[2], hi[3]);
#pragma unroll
                for (int o = 0; o < 2; ++o) {
                    z2[o] = mma(w2[o][2 * m + k], vl, z2[o]);
                    z2[o] = mma(w2[o][2 * m + k], vm, z2[o]);
                    z2[o] = mma(w2[o][2 * m + k], vh, z2[o]);
                }
            }
        }
        float s = 0.0f;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 w = *reinterpret_cast<const float4 *>(&sW3[32 * m + 8 * g + 4 * h]);
                s = fmaf(w.x, gelu_finite(z2[m][4 * g]), s);
                s = fmaf(w.y, gelu_finite(z2[m][4 * g + 1]), s);
                s = fmaf(w.z, gelu_finite(z2[m][4 * g + 2]), s);
                s = fmaf(w.w, gelu_finite(z2[m][4 * g + 3]), s);
            }
        s += __shfl_xor(s, 32);
        s += b3;
        if (h == 0 && row < n) y[row] = s;
        bad |= !isfinite(s);
    }
    if (!__any(bad)) return;
    for (long long tile = (long long)blockIdx.x * 4 + (t >> 6); tile < tiles; tile += stride) {
        const long long row = tile * 32 + c;
        unsigned long long again = __ballot(h == 0 && row < n && !isfinite(y[row]));
        while (again) {
            const int k = __builtin_ctzll(again);
            again &= again - 1;
            const float v = eval_row(wbf, norm, data + (tile * 32 + k) * 6, l);
            if (l == k) y[row] = v;
        }
    }
}
constexpr int PREDICT_BLOCKS = 1024;   // four per compute unit, each wavefront's weights loaded once

grte_status mhip(hipError_t e, const char *what)
{
    if (e == hipSuccess) return GRTE_OK;
    fprintf(stderr, "grte_mlp: %s failed: %s\n", what, hipGetErrorString(e));
    return GRTE_E_HIP;
}

#define MCHK(x)                                                 \
    do {                                                        \
        grte_status _s = mhip((x), #x);                         \
        if (_s != GRTE_OK) return _s;                           \
    } while (0)

grte_status ensure_gpart(grte_mlp *m, int nblk)
{
    if (nblk <= m->gcap) return GRTE_OK;
    if (m->gpart) (void)hipFree(m->gpart);
    if (m->lpart) (void)hipFree(m->lpart);
    m->gpart = nullptr;
    m->lpart = nullptr;
    m->gcap = 0;
    if (hipMalloc((void **)&m->gpart, (size_t)nblk * MLP_NPARAM * sizeof(float)) != hipSuccess ||
        hipMalloc((void **)&m->lpart, (size_t)nblk * sizeof(float)) != hipSuccess)
        return GRTE_E_NOMEM;
    m->gcap = nblk;
    return GRTE_OK;
}

// per-block partial gradients and losses into gpart/lpart (grad_blocks(B) blocks)
grte_status launch_grad_into(grte_mlp *m, const float *data, long long n, long long start, int B, float *gpart,
                             float *lpart)
{
    hipLaunchKernelGGL(mlp_grad_kernel, dim3(grad_blocks(B)), dim3(256), 0, m->stream, m->theta, m->norm, data, n,
                       start, B, gpart, lpart);
    MCHK(hipGetLastError());
    return GRTE_OK;
}

grte_status launch_grad(grte_mlp *m, const float *data, long long n, long long start, int B)
{
    const int nblk = grad_blocks(B);
    grte_status st = ensure_gpart(m, nblk);
    if (st != GRTE_OK) return st;
    return launch_grad_into(m, data, n, start, B, m->gpart, m->lpart);
}

// `steps` Adam steps on minibatches of B rows, taken cyclically from the n
// rows; the per-block partials go to gpart/lpart, the loss of step k to
// lhist[k] (device, null: not recorded).  Allocates nothing.
grte_status train_steps(grte_mlp *m, const float *data, long long n, int steps, int B, float lr, float *gpart,
                        float *lpart, float *lhist)
{
    const int nblk = grad_blocks(B);
    long long start = 0;
    for (int k = 0; k < steps; ++k) {
        grte_status st = launch_grad_into(m, data, n, start, B, gpart, lpart);
        if (st != GRTE_OK) return st;
        start = (start + B) % n;
        const int kk = ++m->adam_k;
        const float c1 = (float)(1.0 - std::pow(0.9, kk)), c2 = (float)(1.0 - std::pow(0.999, kk));
        hipLaunchKernelGGL(mlp_adam_kernel, dim3(ADAM_GRID), dim3(AE * AS), 0, m->stream, m->theta,
                           m->am, m->av, m->wbf, gpart, nblk, lpart, B, lhist, k, lr, c1, c2);
        MCHK(hipGetLastError());
    }
    return GRTE_OK;
}

// ---- the training entry point that allocates nothing (grte_mlp_train_noalloc):
// the device address of the file-scope workspace, per device
constexpr int NOALLOC_MAX_DEVICES = 64;
std::mutex scratch_mutex;
float *scratch_ptr[NOALLOC_MAX_DEVICES] = {};

grte_status scratch_on_device(float **out)
{
    int dev = -1;
    MCHK(hipGetDevice(&dev));
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return GRTE_E_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_ptr[dev]) {
        void *p = nullptr;
        MCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return GRTE_E_HIP;
        scratch_ptr[dev] = (float *)p;
    }
    *out = scratch_ptr[dev];
    return GRTE_OK;
}

}  // namespace

extern "C" {

grte_status grte_mlp_destroy(grte_mlp *m)
{
    if (!m) return GRTE_OK;
    void *ps[] = {m->theta, m->wbf, m->am, m->av, m->norm, m->gpart, m->lpart, m->lhist};
    for (void *p : ps)
        if (p) (void)hipFree(p);
    delete m;
    return GRTE_OK;
}

grte_status grte_mlp_create(grte_mlp **out)
{
    if (!out) return GRTE_E_INVAL;
    *out = nullptr;
    grte_mlp *m = new (std::nothrow) grte_mlp();
    if (!m) return GRTE_E_NOMEM;
    if (hipMalloc((void **)&m->theta, MLP_NPARAM * sizeof(float)) != hipSuccess ||
        hipMalloc((void **)&m->wbf, (MLP_NPARAM + 3) * sizeof(uint16_t)) != hipSuccess ||
        hipMalloc((void **)&m->am, MLP_NPARAM * sizeof(float)) != hipSuccess ||
        hipMalloc((void **)&m->av, MLP_NPARAM * sizeof(float)) != hipSuccess ||
        hipMalloc((void **)&m->norm, MLP_NNORM * sizeof(float)) != hipSuccess) {
        grte_mlp_destroy(m);
        return GRTE_E_NOMEM;
    }
    const float unit[MLP_NNORM] = {0, 0, 0, 0, 0, 1, 1, 1, 1, 1, 0, 1};
    std::vector<float> z(MLP_NPARAM, 0.0f);
    if (hipMemcpy(m->theta, z.data(), MLP_NPARAM * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(m->am, z.data(), MLP_NPARAM * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(m->av, z.data(), MLP_NPARAM * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(m->norm, unit, sizeof(unit), hipMemcpyHostToDevice) != hipSuccess) {
        grte_mlp_destroy(m);
        return GRTE_E_HIP;
    }
    hipLaunchKernelGGL(mlp_round_kernel, dim3((MLP_NPARAM + 255) / 256), dim3(256), 0, nullptr, m->theta, m->wbf);
    if (hipDeviceSynchronize() != hipSuccess) {
        grte_mlp_destroy(m);
        return GRTE_E_HIP;
    }
    *out = m;
    return GRTE_OK;
}

grte_status grte_mlp_set_stream(grte_mlp *m, void *hip_stream)
{
    if (!m) return GRTE_E_INVAL;
    m->stream = (hipStream_t)hip_stream;
    return GRTE_OK;
}

grte_status grte_mlp_set_params(grte_mlp *m, const float *theta)
{
    if (!m || !theta) return GRTE_E_INVAL;
    for (int e = 0; e < MLP_NPARAM; ++e)
        if (!std::isfinite(theta[e])) return GRTE_E_INVAL;
    MCHK(hipMemcpyAsync(m->theta, theta, MLP_NPARAM * sizeof(float), hipMemcpyHostToDevice, m->stream));
    MCHK(hipMemsetAsync(m->am, 0, MLP_NPARAM * sizeof(float), m->stream));
    MCHK(hipMemsetAsync(m->av, 0, MLP_NPARAM * sizeof(float), m->stream));
    hipLaunchKernelGGL(mlp_round_kernel, dim3((MLP_NPARAM + 255) / 256), dim3(256), 0, m->stream, m->theta, m->wbf);
    MCHK(hipGetLastError());
    MCHK(hipStreamSynchronize(m->stream));
    m->adam_k = 0;
    return GRTE_OK;
}

grte_status grte_mlp_get_params(grte_mlp *m, float *theta, unsigned short *theta_bf16)
{
    if (!m) return GRTE_E_INVAL;
    if (theta) MCHK(hipMemcpyAsync(theta, m->theta, MLP_NPARAM * sizeof(float), hipMemcpyDeviceToHost, m->stream));
    if (theta_bf16)
        MCHK(hipMemcpyAsync(theta_bf16, m->wbf, MLP_NPARAM * sizeof(uint16_t), hipMemcpyDeviceToHost, m->stream));
    MCHK(hipStreamSynchronize(m->stream));
    return GRTE_OK;
}

grte_status grte_mlp_set_norm(grte_mlp *m, const float *norm)
{
    if (!m || !norm) return GRTE_E_INVAL;
    for (int q = 0; q < MLP_NNORM; ++q)
        if (!std::isfinite(norm[q])) return GRTE_E_INVAL;
    for (int q = 0; q < MLP_IN; ++q)
        if (!(norm[MLP_IN + q] > 0)) return GRTE_E_INVAL;
    if (!(norm[11] > 0)) return GRTE_E_INVAL;
    MCHK(hipMemcpyAsync(m->norm, norm, MLP_NNORM * sizeof(float), hipMemcpyHostToDevice, m->stream));
    MCHK(hipStreamSynchronize(m->stream));
    return GRTE_OK;
}

grte_status grte_mlp_get_norm(grte_mlp *m, float *norm)
{
    if (!m || !norm) return GRTE_E_INVAL;
    MCHK(hipMemcpyAsync(norm, m->norm, MLP_NNORM * sizeof(float), hipMemcpyDeviceToHost, m->stream));
    MCHK(hipStreamSynchronize(m->stream));
    return GRTE_OK;
}

grte_status grte_mlp_fit_norm(grte_mlp *m, const float *data, long long n)
{
    if (!m || !data || n < 2) return GRTE_E_INVAL;
    hipLaunchKernelGGL(mlp_norm_kernel, dim3(1), dim3(256), 0, m->stream, data, n, m->norm);
    MCHK(hipGetLastError());
    MCHK(hipStreamSynchronize(m->stream));
    return GRTE_OK;
}

grte_status grte_mlp_grad(grte_mlp *m, const float *data, long long n, float *grad, float *loss)
{
    if (!m || !data || !grad || n < 1 || n > (1 << 24)) return GRTE_E_INVAL;
    const int B = (int)n;
    grte_status st = launch_grad(m, data, n, 0, B);
    if (st != GRTE_OK) return st;
    const int nblk = grad_blocks(B);
    std::vector<float> gp((size_t)nblk * MLP_NPARAM), lp(nblk);
    MCHK(hipMemcpyAsync(gp.data(), m->gpart, gp.size() * sizeof(float), hipMemcpyDeviceToHost, m->stream));
    MCHK(hipMemcpyAsync(lp.data(), m->lpart, lp.size() * sizeof(float), hipMemcpyDeviceToHost, m->stream));
    MCHK(hipStreamSynchronize(m->stream));
    for (int e = 0; e < MLP_NPARAM; ++e) {
        float g = 0.0f;
        for (int b = 0; b < nblk; ++b) g += gp[(size_t)b * MLP_NPARAM + e];
        grad[e] = g;
    }
    if (loss) {
        float l = 0.0f;
        for (int b = 0; b < nblk; ++b) l += lp[b];
        *loss = l / (float)B;
    }
    return GRTE_OK;
}

grte_status grte_mlp_train(grte_mlp *m, const float *data, long long n, int steps, int batch, float lr,
                           float *loss_hist)
{
    if (!m || !data || n < 1 || steps < 1 || batch < 1 || batch > (1 << 20) || !(lr > 0)) return GRTE_E_INVAL;
    const int B = (int)std::min<long long>(batch, n);
    const int nblk = grad_blocks(B);
    if (loss_hist && steps > m->hcap) {
        if (m->lhist) (void)hipFree(m->lhist);
        m->lhist = nullptr;
        m->hcap = 0;
        if (hipMalloc((void **)&m->lhist, (size_t)steps * sizeof(float)) != hipSuccess) return GRTE_E_NOMEM;
        m->hcap = steps;
    }
    grte_status st = ensure_gpart(m, nblk);
    if (st != GRTE_OK) return st;
    st = train_steps(m, data, n, steps, B, lr, m->gpart, m->lpart, loss_hist ? m->lhist : nullptr);
    if (st != GRTE_OK) return st;
    if (loss_hist)
        MCHK(hipMemcpyAsync(loss_hist, m->lhist, (size_t)steps * sizeof(float), hipMemcpyDeviceToHost, m->stream));
    MCHK(hipStreamSynchronize(m->stream));
    return GRTE_OK;
}

grte_status grte_mlp_train_noalloc(grte_mlp *m, const float *data, long long n, int steps, int batch, float lr,
                                   float *loss_hist)
{
    if (!m || !data || n < 1 || steps < 1 || batch < 1 || !(lr > 0)) return GRTE_E_INVAL;
    const int B = (int)std::min<long long>(batch, n);
    if (B > NOALLOC_MAX_BATCH || (loss_hist && steps > NOALLOC_MAX_STEPS)) {
        fprintf(stderr, "grte_mlp_train_noalloc: minibatch %d rows (at most %d) or %d loss-history steps "
                        "(at most %d) beyond the fixed workspace\n", B, NOALLOC_MAX_BATCH, steps, NOALLOC_MAX_STEPS);
        return GRTE_E_UNSUPPORTED;
    }
    float *ws = nullptr;
    grte_status st = scratch_on_device(&ws);
    if (st != GRTE_OK) return st;
    float *gpart = ws;                                              // NOALLOC_MAX_BLOCKS x MLP_NPARAM
    float *lpart = gpart + (size_t)NOALLOC_MAX_BLOCKS * MLP_NPARAM;  // NOALLOC_MAX_BLOCKS
    float *lhist = lpart + NOALLOC_MAX_BLOCKS;                      // NOALLOC_MAX_STEPS
    st = train_steps(m, data, n, steps, B, lr, gpart, lpart, loss_hist ? lhist : nullptr);
    if (st != GRTE_OK) return st;
    if (loss_hist)
        MCHK(hipMemcpyAsync(loss_hist, lhist, (size_t)steps * sizeof(float), hipMemcpyDeviceToHost, m->stream));
    MCHK(hipStreamSynchronize(m->stream));
    return GRTE_OK;
}

grte_status grte_mlp_predict(grte_mlp *m, const float *data, long long n, float *y)
{
    if (!m || !data || !y || n < 1) return GRTE_E_INVAL;
    const unsigned blocks = (unsigned)std::min<long long>((n + 127) / 128, PREDICT_BLOCKS);
    hipLaunchKernelGGL(mlp_predict_kernel, dim3(blocks), dim3(256), 0, m->stream, m->wbf, m->norm, data, n, y);
    MCHK(hipGetLastError());
    MCHK(hipStreamSynchronize(m->stream));
    return GRTE_OK;
}

}  // extern "C"
