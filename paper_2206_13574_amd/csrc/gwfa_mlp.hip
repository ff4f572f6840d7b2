// gwfa_mlp.hip -- training and batch inference of the diagonal keep/drop
// network used by the learned pruning mode (8 -> 64 ReLU -> 64 ReLU -> 1).
//
// The forward pass is the inference arithmetic of gwfa_mlp_dev.h: inputs
// x = bf16(feature * scale), bfloat16 weights, activations rounded to
// bfloat16 after each ReLU, float32 sums in the same order, so a trained
// network scores a diagonal in training exactly as the alignment kernel does.
// Loss: binary cross-entropy on the logit, positives weighted by pos_weight,
// averaged over the samples of the call.  The backward pass treats the
// bfloat16 roundings as the identity.  Adam keeps float32 master weights and
// moments and writes the bfloat16 copy the kernels read.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "gwfa_internal.h"
#include "gwfa_mlp_dev.h"

namespace gwfa_train {

using namespace gwfa_nn;

// One workgroup's partial sums: the gradient, then the loss, padded.
constexpr int PART = 4864;
constexpr int GRAD_WAVES = 4;       // waves of a gradient workgroup
constexpr int GRAD_BLOCKS = 256;    // at most: one per compute unit

// LDS written by some lanes of a wave is read by others: its DS operations run
// in order, only the compiler has to keep them so.
__device__ __forceinline__ void wave_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

__device__ __forceinline__ float softplus(float z) { return fmaxf(z, 0.0f) + log1pf(expf(-fabsf(z))); }
__device__ __forceinline__ float sigmoid(float z) {
    const float e = expf(-fabsf(z));
    return z >= 0.0f ? 1.0f / (1.0f + e) : e / (1.0f + e);
}

// Forward and backward of 16 samples per wave and step, all products on the
// matrix cores: the forward pass in bfloat16 (the values are bfloat16), the
// backward pass and the weight gradients in float32 (v_mfma_f32_16x16x4_f32),
// so nothing is rounded that a float32 sum would not round.  Lane (g = l/16,
// m = l%16) holds:
//   h1   unit 16c + 4g + i of sample m          (layer 1, transposed)
//   a2   unit 16c + m of sample 4g + i          (layer 2, and g2 = dL/da2)
// Products over samples take sample 4g + q in step q, so g2 and g1 are operands
// as they lie; h1 and g2 are turned once each through LDS.  Every wave keeps
// its whole gradient in registers over its samples; the waves of a workgroup
// are added in LDS and the workgroups by k_grad_sum, without atomics and in
// a fixed order.
// 32,768 samples: about 27 us, bound by the waves' chain of steps (two per wave,
// then the sum in LDS), the matrix work being 4 us; one thread per sample and
// per parameter took 300 us.
__global__ __launch_bounds__(64 * GRAD_WAVES, 1) void k_grad(const float* __restrict__ feat, int64_t stride,
                                                             Scale8 scale, const uint8_t* __restrict__ label, int64_t n,
                                                             float pos_weight, float inv_n,
                                                             const uint16_t* __restrict__ w, float* __restrict__ part) {
    constexpr int LD = 68;                       // row of a turned tile
    struct Tile { float h[16 * LD], g[16 * LD], x[16 * 17]; };
    __shared__ float w2f[64 * 65];               // W2 as float
    __shared__ union { Tile tile[GRAD_WAVES]; float sum[PART]; } L;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int col = lane & 15, grp = lane >> 4;
    Tile& T = L.tile[wv];
    for (int p = threadIdx.x; p < 4096; p += 64 * GRAD_WAVES) w2f[(p >> 6) * 65 + (p & 63)] = bf2f(w[MW_W2 + p]);
    // weights as operands, kept over the samples
    const __bf16 zero = bf_bits(0);
    bf16x8 w1a[4], w2b[2][4];
    float b1[16], b2[4], w3[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
        for (int i = 0; i < 8; ++i) w1a[c][i] = grp == 0 ? bf_bits(w[(16 * c + col) * 8 + i]) : zero;
#pragma unroll
        for (int i = 0; i < 4; ++i) b1[4 * c + i] = bf2f(w[MW_B1 + 16 * c + 4 * grp + i]);
        b2[c] = bf2f(w[MW_B2 + 16 * c + col]);
        w3[c] = bf2f(w[MW_W3 + 16 * c + col]);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const uint16_t* row = w + MW_W2 + (16 * c + col) * 64 + 32 * ks + 4 * grp;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                w2b[ks][c][i] = bf_bits(row[i]);
                w2b[ks][c][4 + i] = bf_bits(row[16 + i]);
            }
        }
    }
    const float b3 = bf2f(w[MW_B3]);
    f32x4 d2[4][4], d1[4];                       // dW2 by unit pair; dW1 with db1 as column 8
    float db2[4], dw3[4], db3 = 0.0f, loss = 0.0f;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        db2[c] = 0.0f; dw3[c] = 0.0f;
        d1[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 4; ++k) d2[c][k] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __syncthreads();
    const int64_t tiles = (n + 15) / 16;
    for (int64_t t = (int64_t)blockIdx.x * GRAD_WAVES + wv; t < tiles; t += (int64_t)gridDim.x * GRAD_WAVES) {
        // the rows that fill up the last tile: every activation and gradient 0, so
        // that no weight, infinite ones among them, is multiplied into the sums
        const bool row = 16 * t + col < n;
        // inputs: two features per lane, column 8 is 1 (the bias)
        {
            const int64_t b = 16 * t + col;
            const bool ok = b < n;
            const float* f = feat + (ok ? b : 0) * stride + 2 * grp;
            const float s0 = scale.s[2 * grp], s1 = scale.s[2 * grp + 1];
            T.x[col * 17 + 2 * grp] = ok ? round_bf16(f[0] * s0) : 0.0f;
            T.x[col * 17 + 2 * grp + 1] = ok ? round_bf16(f[1] * s1) : 0.0f;
            T.x[col * 17 + 8 + 2 * grp] = ok && grp == 0 ? 1.0f : 0.0f;
            T.x[col * 17 + 9 + 2 * grp] = 0.0f;
        }
        bool pos[4], ok[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t b = 16 * t + 4 * grp + i;
            ok[i] = b < n;
            pos[i] = ok[i] && label[ok[i] ? b : 0] != 0;
        }
        wave_order();
        bf16x8 xb;
#pragma unroll
        for (int i = 0; i < 8; ++i) xb[i] = grp == 0 ? bf_of(T.x[col * 17 + i]) : zero;
        float h[16];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            f32x4 d;
#pragma unroll
            for (int i = 0; i < 4; ++i) d[i] = b1[4 * c + i];
            d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1a[c], xb, d, 0, 0, 0);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                h[4 * c + i] = row ? round_bf16(fmaxf(d[i], 0.0f)) : 0.0f;
                T.h[col * LD + 16 * c + 4 * grp + i] = h[4 * c + i];
            }
        }
        f32x4 a2[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) a2[c] = f32x4{b2[c], b2[c], b2[c], b2[c]};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8 a;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                a[i] = bf_of(h[8 * ks + i]);
                a[4 + i] = bf_of(h[8 * ks + 4 + i]);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) a2[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w2b[ks][c], a2[c], 0, 0, 0);
        }
        // logits of samples 4g + i, loss and dL/dz; g2 = dL/da2
        float g2[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float h2[4], z = 0.0f;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                h2[c] = round_bf16(fmaxf(a2[c][i], 0.0f));
                z = fmaf(w3[c], h2[c], z);
            }
#pragma unroll
            for (int o = 8; o >= 1; o >>= 1) z += __shfl_xor(z, o, 64);
            z += b3;
            const float sz = sigmoid(z);
            const float dz = ok[i] ? (pos[i] ? pos_weight * (sz - 1.0f) : sz) * inv_n : 0.0f;
            if (col == 0 && ok[i]) {
                loss += pos[i] ? pos_weight * softplus(-z) : softplus(z);
                db3 += dz;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                dw3[c] = fmaf(dz, h2[c], dw3[c]);
                g2[c][i] = ok[i] && a2[c][i] > 0.0f ? dz * w3[c] : 0.0f;
                db2[c] += g2[c][i];
                T.g[(4 * grp + i) * LD + 16 * c + col] = g2[c][i];
            }
        }
        wave_order();
        float hb[4][4];                          // h1 of unit 16k + m, sample 4g + q
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q) hb[k][q] = T.h[(4 * grp + q) * LD + 16 * k + col];
        f32x4 a1[4];                             // dL/dh1 of unit 16k + m, sample 4g + i
#pragma unroll
        for (int k = 0; k < 4; ++k) a1[k] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 16; ++q) {           // unit 16g + q of layer 2
            const float ga = T.g[col * LD + 16 * grp + q];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                a1[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(ga, w2f[(16 * grp + q) * 65 + 16 * k + col], a1[k], 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float xv = T.x[(4 * grp + q) * 17 + col];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    d2[c][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(g2[c][q], hb[k][q], d2[c][k], 0, 0, 0);
                d1[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(hb[c][q] > 0.0f ? a1[c][q] : 0.0f, xv, d1[c], 0, 0, 0);
            }
        }
        wave_order();                            // the tile's rows are read before they are written again
    }
    // the biases' and w3's lanes: sum over the four groups
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        db2[c] += __shfl_xor(db2[c], 16, 64); db2[c] += __shfl_xor(db2[c], 32, 64);
        dw3[c] += __shfl_xor(dw3[c], 16, 64); dw3[c] += __shfl_xor(dw3[c], 32, 64);
    }
    db3 += __shfl_xor(db3, 16, 64); db3 += __shfl_xor(db3, 32, 64);
    loss += __shfl_xor(loss, 16, 64); loss += __shfl_xor(loss, 32, 64);
    for (int v = 0; v < GRAD_WAVES; ++v) {
        __syncthreads();
        if (wv == v) {
            auto add = [&](int p, float x) { L.sum[p] = v == 0 ? x : L.sum[p] + x; };
#pragma unroll
            for (int c = 0; c < 4; ++c) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int j = 16 * c + 4 * grp + i;
                    if (col < 8) add(j * 8 + col, d1[c][i]);
                    if (col == 8) add(MW_B1 + j, d1[c][i]);
#pragma unroll
                    for (int k = 0; k < 4; ++k) add(MW_W2 + j * 64 + 16 * k + col, d2[c][k][i]);
                }
                if (grp == 0) {
                    add(MW_B2 + 16 * c + col, db2[c]);
                    add(MW_W3 + 16 * c + col, dw3[c]);
                }
            }
            if (lane == 0) { add(MW_B3, db3); add(MLP_N, loss * inv_n); }
        }
    }
    __syncthreads();
    for (int p = threadIdx.x; p <= MLP_N; p += 64 * GRAD_WAVES) part[(int64_t)blockIdx.x * PART + p] = L.sum[p];
}

// Sums the workgroups' parts: 32 values per workgroup, eight lanes a value.
__global__ __launch_bounds__(256) void k_grad_sum(const float* __restrict__ part, int blocks, float* __restrict__ grad,
                                                  float* __restrict__ loss) {
    __shared__ float s[8][32];
    const int p = blockIdx.x * 32 + (threadIdx.x & 31), q = threadIdx.x >> 5;
    float a = 0.0f;
    if (p <= MLP_N)
#pragma unroll 8
        for (int b = q; b < blocks; b += 8) a += part[(int64_t)b * PART + p];
    s[q][threadIdx.x & 31] = a;
    __syncthreads();
    if (q == 0 && p <= MLP_N) {
#pragma unroll
        for (int k = 1; k < 8; ++k) a += s[k][threadIdx.x];
        if (p < MLP_N) grad[p] = a; else *loss = a;
    }
}

__global__ void k_adam(float* __restrict__ master, float* __restrict__ m1, float* __restrict__ m2,
                       const float* __restrict__ grad, uint16_t* __restrict__ wb, float lr, float beta1, float beta2,
                       float eps, float bc1, float bc2) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= MLP_N) return;
    const float g = grad[p];
    const float a = beta1 * m1[p] + (1.0f - beta1) * g;
    const float b = beta2 * m2[p] + (1.0f - beta2) * g * g;
    m1[p] = a;
    m2[p] = b;
    const float upd = (a / bc1) / (sqrtf(b / bc2) + eps);
    const float w = master[p] - lr * upd;
    master[p] = w;
    wb[p] = f2bf(w);
}

__global__ void k_cast(const float* __restrict__ src, uint16_t* __restrict__ dst, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = f2bf(src[i]);
}

// Lanes 0..31: a of lanes l and l+32 added; lanes 32..63: b of them.
__device__ __forceinline__ float sum_rows32(float a, float b) {
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(x[0]) + __uint_as_float(x[1]);
}
// Rows of 16 lanes: a of rows 0 and 1 added, b of rows 0 and 1, a of rows 2
// and 3, b of rows 2 and 3.
__device__ __forceinline__ float sum_rows16(float a, float b) {
    const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(x[0]) + __uint_as_float(x[1]);
}

// Logits of n samples, bit for bit those of the alignment kernel's inference
// routine (same products, roundings and order of the sums), persistent waves
// with the weights in registers.  A wave takes 64 samples, one per lane,
// and scores them 16 at a time.  The weights of layer 1 stand in all four
// quarters of the product's 32 positions and the samples of tile t in quarter
// t, so each lane's inputs are its operand as they lie; layer 2 is taken
// transposed (units by samples), so its inputs are layer 1's outputs and the
// last sum is 16 products in a lane and five exchanges of rows (no LDS).
// 1,000,003 samples: 29 us (36 MB: 1.2 TB/s); with the weights gathered from
// LDS for every tile and 20 exchanges 81 us.  Bound by the roundings and
// packing between the layers (about 120 vector instructions per 16 samples).
__global__ __launch_bounds__(256, 3) void k_logits(const float* __restrict__ feat, int64_t stride, Scale8 scale,
                                                int64_t n, const uint16_t* __restrict__ w, float* __restrict__ out) {
    const int lane = threadIdx.x & 63, col = lane & 15, grp = lane >> 4;
    bf16x8 w1a[4], w2a[2][4];
    f32x4 b1[4], b2[4], w3[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
        for (int i = 0; i < 8; ++i) w1a[c][i] = bf_bits(w[(16 * c + col) * 8 + i]);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int j = 16 * c + 4 * grp + i;
            b1[c][i] = bf2f(w[MW_B1 + j]);
            b2[c][i] = bf2f(w[MW_B2 + j]);
            w3[c][i] = bf2f(w[MW_W3 + j]);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const uint16_t* row = w + MW_W2 + (16 * c + col) * 64 + 32 * ks + 4 * grp;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                w2a[ks][c][i] = bf_bits(row[i]);
                w2a[ks][c][4 + i] = bf_bits(row[16 + i]);
            }
        }
    }
    const float b3 = bf2f(w[MW_B3]);
    // Weights that are not finite must not meet the zeros that stand for the other
    // quarters' samples (0 times infinity is not a number): then only the first
    // quarter holds weights, and every tile's samples are brought there.
    uint32_t top = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < 8; ++i) top = max(top, (uint32_t)(w[(16 * c + col) * 8 + i] & 0x7f80u));
    const bool first_only = __ballot(top == 0x7f80u) != 0;
    if (first_only && grp != 0) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int i = 0; i < 8; ++i) w1a[c][i] = bf_bits(0);
    }
    const bool wide = (stride & 3) == 0 && (reinterpret_cast<uintptr_t>(feat) & 15) == 0;   // rows of 16-byte words
    const int64_t waves = (int64_t)gridDim.x * 4;
    for (int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); g * 64 < n; g += waves) {
        const int64_t b = g * 64 + lane;
        const bool ok = b < n;
        const float* f = feat + (ok ? b : 0) * stride;
        float x[8];
        if (wide) {
            const float4 lo = *reinterpret_cast<const float4*>(f), hi = *reinterpret_cast<const float4*>(f + 4);
            x[0] = lo.x; x[1] = lo.y; x[2] = lo.z; x[3] = lo.w;
            x[4] = hi.x; x[5] = hi.y; x[6] = hi.z; x[7] = hi.w;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = f[i];
        }
        bf16x8 xp;
#pragma unroll
        for (int i = 0; i < 8; ++i) xp[i] = bf_of(round_bf16(x[i] * scale.s[i]));
        float z_out = 0.0f;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            bf16x8 xb;
#pragma unroll
            for (int i = 0; i < 8; ++i) xb[i] = grp == t ? xp[i] : bf_bits(0);
            if (first_only) {
                const int4 p = __builtin_bit_cast(int4, xp);
                const int4 q = make_int4(__shfl(p.x, 16 * t + col, 64), __shfl(p.y, 16 * t + col, 64),
                                         __shfl(p.z, 16 * t + col, 64), __shfl(p.w, 16 * t + col, 64));
                xb = __builtin_bit_cast(bf16x8, grp == 0 ? q : make_int4(0, 0, 0, 0));
            }
            bf16x8 h[2];   // units 32ks + 4g + i and 32ks + 16 + 4g + i of sample 16t + m
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const f32x4 d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1a[c], xb, b1[c], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < 4; ++i) h[c >> 1][4 * (c & 1) + i] = (__bf16)fmaxf(d[i], 0.0f);
            }
            // the last layer in the order of the alignment kernel's routine: over
            // units 16c + u, then pairs of u that differ in bit 3 (group g xor 2), bit
            // 2 (group g xor 1), bit 1 and bit 0 (i)
            float q[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                f32x4 a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2a[0][c], h[0], b2[c], 0, 0, 0);
                a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2a[1][c], h[1], a, 0, 0, 0);
#pragma unroll
                for (int i = 0; i < 4; ++i) q[i] = fmaf(w3[c][i], round_bf16(fmaxf(a[i], 0.0f)), q[i]);
            }
            // rows 0, 1: q0, rows 2, 3: q1 (q2, q3); then rows q0, q2, q1, q3
            const float z = sum_rows16(sum_rows32(q[0], q[1]), sum_rows32(q[2], q[3]));
            const float y = sum_rows16(z, z);                     // rows 0, 1: q0 + q2; rows 2, 3: q1 + q3
            const float logit = b3 + sum_rows32(y, y);            // (by every lane, not under a branch of some)
            z_out = grp == t ? logit : z_out;
        }
        if (ok) out[b] = z_out;
    }
}

}  // namespace gwfa_train

// ---------------------------------------------------------------------------
// launch helpers
// ---------------------------------------------------------------------------
int64_t gwfa_mlp_scratch_floats() { return (int64_t)gwfa_train::GRAD_BLOCKS * gwfa_train::PART; }

hipError_t gwfa_launch_mlp_grad(const float* feat, int64_t stride, const Scale8& scale, const uint8_t* label,
                                int64_t n, float pos_weight, const uint16_t* w, float* scr, float* grad, float* loss,
                                hipStream_t st) {
    using namespace gwfa_train;
    (void)hipGetLastError();   // report only this call's launch status
    // workgroups enough for one 16-sample step per wave, at most one per
    // compute unit (each ends by writing 19 KB of sums)
    const int blocks = (int)std::min<int64_t>(GRAD_BLOCKS, (n + 16 * GRAD_WAVES - 1) / (16 * GRAD_WAVES));
    if (n > 0)
        hipLaunchKernelGGL(k_grad, dim3(blocks), dim3(64 * GRAD_WAVES), 0, st, feat, stride, scale, label, n, pos_weight,
                           1.0f / (float)n, w, scr);
    hipLaunchKernelGGL(k_grad_sum, dim3((MLP_N + 1 + 31) / 32), dim3(256), 0, st, scr, n > 0 ? blocks : 0, grad, loss);
    return hipGetLastError();
}

hipError_t gwfa_launch_mlp_adam(float* master, float* m1, float* m2, const float* grad, uint16_t* wb, float lr,
                                float beta1, float beta2, float eps, float bc1, float bc2, hipStream_t st) {
    using namespace gwfa_train;
    (void)hipGetLastError();
    hipLaunchKernelGGL(k_adam, dim3((MLP_N + 255) / 256), dim3(256), 0, st, master, m1, m2, grad, wb, lr, beta1,
                       beta2, eps, bc1, bc2);
    return hipGetLastError();
}

hipError_t gwfa_launch_mlp_cast(const float* src, uint16_t* dst, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    (void)hipGetLastError();
    hipLaunchKernelGGL(gwfa_train::k_cast, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src, dst, n);
    return hipGetLastError();
}

hipError_t gwfa_launch_mlp_logits(const float* feat, int64_t stride, const Scale8& scale, int64_t n,
                                  const uint16_t* w, float* out, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    (void)hipGetLastError();
    // workgroups that fit the chip at once (three a compute unit), fewer for few samples
    const unsigned blocks = (unsigned)std::min<int64_t>(768, (n + 255) / 256);
    hipLaunchKernelGGL(gwfa_train::k_logits, dim3(blocks), dim3(256), 0, st, feat, stride, scale, n, w, out);
    return hipGetLastError();
}
