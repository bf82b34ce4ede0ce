// Wave-level inference of the 2 -> 64 -> 64 -> 3 equation-of-state surrogate.
//
// The hidden layer is computed transposed, Z2^T = W2 H1^T, with
// v_mfma_f32_32x32x16_bf16: A = W2 (rows: output neurons, loaded as 8
// contiguous BF16 per lane), B = H1^T (rows: input neurons, columns: samples).
// For the B operand lane l holds input neurons 16 ks + 8 (l / 32) + j of
// samples 32 nt + l % 32, so each lane evaluates its own first-layer
// activations; no transpose through memory is needed.  The accumulator gives
// lane l the output neurons 32 mt + 8 (v / 4) + 4 (l / 32) + v % 4 of the same
// samples; the output layer is a per-lane partial dot product completed with
// the partner lane l ^ 32.
#pragma once

#include <type_traits>

#include "lbm_device.hpp"

namespace lbm {
namespace mlp {

constexpr int H = 64;
constexpr int OFF_W1 = 0, OFF_B1 = 128, OFF_W2 = 192, OFF_B2 = 4288, OFF_W3 = 4352, OFF_B3 = 4544;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// hidden activation: ReLU, max(z, 0), taken on the bit pattern: a set sign bit reads as a negative
// integer and gives +0, a positive value passes unchanged.  One integer max
// per value; the float max would first quiet its input (a second
// instruction per value on matrix-core results).  Differs from fmaxf only
// for a NaN input, which the residual check sends to the fallback anyway.
__device__ __forceinline__ float relu(float z) { return __int_as_float(max(__float_as_int(z), 0)); }

// ReLU of two BF16 values packed in a word, as a 16-bit integer max with 0
// on each half.  Rounding to BF16 is monotone and keeps the sign, so this
// equals rounding relu(a), relu(b): bit for bit, also for -0 and NaN.
typedef short s16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t relu_bf16x2(uint32_t p) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, p), (s16x2){0, 0}));
}

__device__ __forceinline__ __bf16 to_bf16(float v) { return __builtin_bit_cast(__bf16, bf16_hw(v)); }

__device__ __forceinline__ void normalise(const float *norm, float rho, float e, float &x0, float &x1) {
    x0 = 2.0f * (rho - norm[0]) / (norm[1] - norm[0]) - 1.0f;
    x1 = 2.0f * (e - norm[2]) / (norm[3] - norm[2]) - 1.0f;
}

// Parameter pointers of one forward pass with both hidden layers on MFMA
struct Net {
    const uint16_t *w2b;        // [64][w2_ld] BF16, row-major [out][in]
    const float *b2, *w3, *b3;  // [64], [NOUT][64], [NOUT]
    int w2_ld;
};

// ---------------------------------------------------------------------------
// Stand-alone form: first layer on the vector ALU in FP32, hidden layer on
// BF16 MFMA or (F32) on the FP32 matrix instruction.  The small layers and the
// hidden weights sit in LDS, written once per workgroup, and one read of a
// weight serves NT tiles of 32 samples: what bounds it is the vector ALU (per
// tile 112 instructions in the first layer, 32 (1 + NOUT) in the last), not the
// parameter reads that a pass of one tile spends its time on (1,000,003 samples,
// three outputs: 113 us with one wavefront per workgroup converting W2 for
// itself, 25 us so).
template <int NOUT, bool F32> struct NetLds {
    static constexpr int W2LD = F32 ? 68 : 72;  // padded rows: conflict-free 16-byte reads
    // first layer by input position: BF16 position k is neuron k; F32 position
    // 32 h + s is neuron 2 s + h (the matrix instruction's k index of step s in
    // lane half h), and W2's columns follow the same order
    float w1x[H], w1y[H], b1[H], b2[H], w3[NOUT][H], b3[4];
    typename std::conditional<F32, float, uint16_t>::type w2[H * W2LD];
};
// w2b: the hidden weights in BF16 where a copy of them is kept (16-byte aligned), else null
template <int NOUT, bool F32>
__device__ __forceinline__ void net_to_lds(NetLds<NOUT, F32> &n, const float *__restrict__ P,
                                           const uint16_t *__restrict__ w2b, int tid, int nt) {
    for (int k = tid; k < H; k += nt) {
        const int q = F32 ? 2 * (k & 31) + (k >> 5) : k;
        n.w1x[k] = P[OFF_W1 + 2 * q];
        n.w1y[k] = P[OFF_W1 + 2 * q + 1];
        n.b1[k] = P[OFF_B1 + q];
        n.b2[k] = P[OFF_B2 + k];
        for (int o = 0; o < NOUT; o++) n.w3[o][k] = P[OFF_W3 + o * H + k];
    }
    if (tid < NOUT) n.b3[tid] = P[OFF_B3 + tid];
    if constexpr (!F32) {
        if (w2b) {
            for (int r = tid; r < H * H / 8; r += nt)
                *(uint4 *)&n.w2[r / (H / 8) * n.W2LD + 8 * (r % (H / 8))] = ((const uint4 *)w2b)[r];
            return;
        }
    }
    for (int r = tid; r < H * H; r += nt) {
        const int m = r / H, q = r % H;
        const float v = P[OFF_W2 + r];
        if constexpr (F32) n.w2[m * n.W2LD + 32 * (q & 1) + (q >> 1)] = v;
        else n.w2[m * n.W2LD + q] = bf16_hw(v);
    }
}
// Normalised outputs of 32 NT samples: lane l holds samples 64 p + l, p < NT / 2.
// Uniform control flow over the wavefront.
template <int NOUT, bool F32, int NT>
__device__ __forceinline__ void forward_tiles(const float (&x0)[NT / 2], const float (&x1)[NT / 2],
                                              const NetLds<NOUT, F32> &n, float (&y)[NT / 2][NOUT]) {
    const int lane = threadIdx.x & 63, hh = lane >> 5, c = lane & 31;
    float xs0[NT], xs1[NT];
#pragma unroll
    for (int t = 0; t < NT; t++) {
        xs0[t] = __shfl(x0[t / 2], 32 * (t & 1) + c, 64);
        xs1[t] = __shfl(x1[t / 2], 32 * (t & 1) + c, 64);
    }
    // accumulators seeded with b2 of their neurons 32 mt + 8 (v / 4) + 4 hh + v % 4
    f32x16 acc[NT][2], seed[2];
#pragma unroll
    for (int mt = 0; mt < 2; mt++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const float4 b = *(const float4 *)&n.b2[32 * mt + 8 * q + 4 * hh];
            seed[mt][4 * q] = b.x;
            seed[mt][4 * q + 1] = b.y;
            seed[mt][4 * q + 2] = b.z;
            seed[mt][4 * q + 3] = b.w;
        }
#pragma unroll
    for (int ks = 0; ks < (F32 ? 8 : 4); ks++) {
        // input positions of this lane half in this group: 8 of a BF16 k-step,
        // or those of four FP32 k-steps
        constexpr int G = F32 ? 4 : 8;
        const int k0 = F32 ? 32 * hh + 4 * ks : 16 * ks + 8 * hh;
        float wx[G], wy[G], b[G];
#pragma unroll
        for (int j = 0; j < G; j += 4) {
            *(float4 *)&wx[j] = *(const float4 *)&n.w1x[k0 + j];
            *(float4 *)&wy[j] = *(const float4 *)&n.w1y[k0 + j];
            *(float4 *)&b[j] = *(const float4 *)&n.b1[k0 + j];
        }
        const uint4 a0 = *(const uint4 *)&n.w2[c * n.W2LD + k0], a1 = *(const uint4 *)&n.w2[(32 + c) * n.W2LD + k0];
#pragma unroll
        for (int t = 0; t < NT; t++) {
            float hv[G];
#pragma unroll
            for (int j = 0; j < G; j++) hv[j] = relu(fmaf(wx[j], xs0[t], fmaf(wy[j], xs1[t], b[j])));
            if constexpr (F32) {
                const float *w0 = (const float *)&a0, *w1 = (const float *)&a1;
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const bool first = ks == 0 && j == 0;
                    acc[t][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(w0[j], hv[j], first ? seed[0] : acc[t][0], 0, 0, 0);
                    acc[t][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(w1[j], hv[j], first ? seed[1] : acc[t][1], 0, 0, 0);
                }
            } else {
                const uint4 bp = {bf16x2_hw(hv[0], hv[1]), bf16x2_hw(hv[2], hv[3]), bf16x2_hw(hv[4], hv[5]),
                                  bf16x2_hw(hv[6], hv[7])};
                const bf16x8 bv = __builtin_bit_cast(bf16x8, bp);
                acc[t][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a0), bv,
                                                                   ks == 0 ? seed[0] : acc[t][0], 0, 0, 0);
                acc[t][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a1), bv,
                                                                   ks == 0 ? seed[1] : acc[t][1], 0, 0, 0);
            }
        }
        // bounds the live registers to one group's parameters
        __builtin_amdgcn_sched_barrier(0);
    }
    float ys[NT][NOUT];
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
        for (int k = 0; k < NOUT; k++) ys[t][k] = 0.0f;
#pragma unroll
    for (int mt = 0; mt < 2; mt++)
#pragma unroll
        for (int q = 0; q < 4; q++) {
            float w[NOUT][4];
#pragma unroll
            for (int k = 0; k < NOUT; k++) *(float4 *)w[k] = *(const float4 *)&n.w3[k][32 * mt + 8 * q + 4 * hh];
#pragma unroll
            for (int t = 0; t < NT; t++)
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const float h2 = relu(acc[t][mt][4 * q + r]);
#pragma unroll
                    for (int k = 0; k < NOUT; k++) ys[t][k] = fmaf(w[k][r], h2, ys[t][k]);
                }
        }
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
        for (int k = 0; k < NOUT; k++) {
            ys[t][k] += __shfl_xor(ys[t][k], 32, 64);
            // lane l's sample of pair p sits in tile 2 p + l / 32
            if (hh == (t & 1)) y[t / 2][k] = ys[t][k] + n.b3[k];
        }
}

// ---------------------------------------------------------------------------
// Both hidden layers on MFMA (the surrogate pass's form).  Layer 1 is the
// contraction of [w1_0, w1_1, b1] with [x0, x1, 1] padded to K = 16: one
// v_mfma_f32_32x32x16_bf16 per 32 neurons and 32 samples, its operands
// rounded to BF16.  Its accumulator gives lane l (h = l / 32) neurons
// 32 mt + 8 q + 4 h + r (q, r < 4) of its sample; the layer-2 B operand of
// k-step ks wants 8 consecutive k-indices 16 ks + 8 h + j.  Numbering the
// layer-2 inputs by
//   sigma(16 ks + 8 h + j) = 32 (ks / 2) + 8 (2 (ks % 2) + j / 4) + 4 h + j % 4
// makes that operand the accumulator entries 8 (ks % 2) + j of tile ks / 2,
// so no value crosses lanes; the A operand reads W2 with its columns in the
// same order (w2_perm_col).  Layer 2 starts its accumulators at b2.
__host__ __device__ constexpr int w2_perm_col(int k) {
    return 32 * ((k >> 4) >> 1) + 8 * (2 * ((k >> 4) & 1) + ((k & 7) >> 2)) + 4 * ((k >> 3) & 1) + (k & 3);
}
// per-lane layer-1 A operands (neurons 32 mt + l % 32 in lanes 0..31: their
// w1 row and bias; zero in lanes 32..63)
struct L1Ops {
    bf16x8 a[2];
};
__device__ __forceinline__ L1Ops l1_operands(const float *w1, const float *b1) {
    const int lane = threadIdx.x & 63, c = lane & 31;
    L1Ops o;
#pragma unroll
    for (int mt = 0; mt < 2; mt++) {
        uint4 u = {0u, 0u, 0u, 0u};
        if (lane < 32) {
            const int m = 32 * mt + c;
            u.x = bf16x2_hw(w1[2 * m], w1[2 * m + 1]);
            u.y = bf16x2_hw(b1[m], 0.0f);
        }
        o.a[mt] = __builtin_bit_cast(bf16x8, u);
    }
    return o;
}
// normalised outputs 0..NOUT-1 of this lane's sample; uniform control flow.
// p.w2b: BF16 W2 with permuted columns (row stride p.w2_ld elements).
template <int NOUT>
__device__ __forceinline__ void forward_wave_l1mfma(float x0, float x1, const Net &p, const L1Ops &l1, float y[NOUT]) {
    const int lane = threadIdx.x & 63;
    const int hh = lane >> 5, c = lane & 31;
    const unsigned a_off = (unsigned)(c * p.w2_ld + 8 * hh) * 2u;
#pragma unroll
    for (int nt = 0; nt < 2; nt++) {
        const float xs0 = __shfl(x0, 32 * nt + c, 64), xs1 = __shfl(x1, 32 * nt + c, 64);
        uint4 bu = {0u, 0u, 0u, 0u};
        if (hh == 0) {
            bu.x = bf16x2_hw(xs0, xs1);
            bu.y = bf16x2_hw(1.0f, 0.0f);
        }
        const bf16x8 b1 = __builtin_bit_cast(bf16x8, bu);
        f32x16 z1[2];
#pragma unroll
        for (int mt = 0; mt < 2; mt++) {
#pragma unroll
            for (int v = 0; v < 16; v++) z1[mt][v] = 0.0f;
            z1[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(l1.a[mt], b1, z1[mt], 0, 0, 0);
        }
        // layer 2, accumulators seeded with b2 of the output neurons
        f32x16 acc[2];
#pragma unroll
        for (int mt = 0; mt < 2; mt++)
#pragma unroll
            for (int v = 0; v < 16; v++) acc[mt][v] = p.b2[32 * mt + 8 * (v >> 2) + 4 * hh + (v & 3)];
#pragma unroll
        for (int ks = 0; ks < 4; ks++) {
            const int t = ks >> 1, o = 8 * (ks & 1);
            uint4 bp;
            bp.x = relu_bf16x2(bf16x2_hw(z1[t][o + 0], z1[t][o + 1]));
            bp.y = relu_bf16x2(bf16x2_hw(z1[t][o + 2], z1[t][o + 3]));
            bp.z = relu_bf16x2(bf16x2_hw(z1[t][o + 4], z1[t][o + 5]));
            bp.w = relu_bf16x2(bf16x2_hw(z1[t][o + 6], z1[t][o + 7]));
            const bf16x8 b = __builtin_bit_cast(bf16x8, bp);
#pragma unroll
            for (int mt = 0; mt < 2; mt++) {
                const uint4 raw =
                    *(const uint4 *)((const char *)p.w2b + a_off + (unsigned)((32 * mt * p.w2_ld + 16 * ks) * 2));
                acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, raw), b, acc[mt], 0, 0, 0);
            }
        }
        float ys[NOUT];
#pragma unroll
        for (int k = 0; k < NOUT; k++) ys[k] = 0.0f;
#pragma unroll
        for (int mt = 0; mt < 2; mt++)
#pragma unroll
            for (int v = 0; v < 16; v++) {
                const int o = 32 * mt + 8 * (v >> 2) + 4 * hh + (v & 3);
                const float h2 = relu(acc[mt][v]);
#pragma unroll
                for (int k = 0; k < NOUT; k++) ys[k] = fmaf(p.w3[k * H + o], h2, ys[k]);
            }
#pragma unroll
        for (int k = 0; k < NOUT; k++) {
            ys[k] += __shfl_xor(ys[k], 32, 64);
            if (hh == nt) y[k] = ys[k] + p.b3[k];
        }
    }
}

}  // namespace mlp
}  // namespace lbm
