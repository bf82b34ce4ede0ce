// Learned equation-of-state surrogate (rho, e) -> (T, P, c_s^2): a
// 2 -> 64 -> 64 -> 3 ReLU network standing in for the caloric inversion of
// Section 3.2 (explicit for van der Waals, eq. lbm_temp; iterative for a
// general equation of state).  Inference runs inside the per-cell passes
// with a residual check and an exact FP64 Newton fallback; training uses the
// library's own forward, backward and Adam kernels.
//
// In training a workgroup of four wavefronts handles 64 samples.  The 64x64
// hidden layer and the two 64x64x64 products of the backward pass run through
// wave_tile64, a 32x32 tile per wavefront: BF16 MFMA (v_mfma_f32_32x32x16_bf16,
// FP32 accumulate) or FP32 MFMA (v_mfma_f32_32x32x2_f32), both returning the
// result in the accumulator layout:
//   tile (mt, nt) in {0,1}^2, accumulator v in 0..15, lane l holds
//   row 32 mt + 8 (v / 4) + 4 (l / 32) + v % 4, column 32 nt + l % 32.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include <cmath>
#include <cstring>
#include <type_traits>

#include "lbm_internal.hpp"
#include "lbm_mlp_device.hpp"

using namespace lbm;

namespace lbm {
namespace mlp {

constexpr int NP = LBM_MLP_NPARAMS;
constexpr int LD = 65;  // padded LDS row stride (floats) of a 64x64 activation tile

__device__ __forceinline__ int acc_row(int mt, int v, int lane) { return 32 * mt + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3); }
__device__ __forceinline__ int acc_col(int nt, int lane) { return 32 * nt + (lane & 31); }

// Tile (mt, nt) of C(i, j) = sum_k A(i, k) B(k, j), i, j, k in [0, 64), by one
// wavefront; A and B are strided FP32 views: A(i, k) = A[i * ai + k * ak],
// B(k, j) = B[k * bk + j * bj].  Entry v of the result is the one at (acc_row,
// acc_col).  BF16: operands rounded to BF16; else the FP32 matrix instruction.
template <bool BF16>
__device__ __forceinline__ f32x16 wave_tile64(const float *A, int ai, int ak, const float *B, int bk, int bj, int mt,
                                              int nt) {
    const int lane = threadIdx.x & 63, i = 32 * mt + (lane & 31), j = 32 * nt + (lane & 31);
    f32x16 c;
    for (int v = 0; v < 16; v++) c[v] = 0.0f;
    if constexpr (BF16) {
#pragma unroll
        for (int ks = 0; ks < 4; ks++) {
            bf16x8 a, b;
            const int k0 = 16 * ks + 8 * (lane >> 5);
#pragma unroll
            for (int q = 0; q < 8; q++) {
                a[q] = to_bf16(A[i * ai + (k0 + q) * ak]);
                b[q] = to_bf16(B[(k0 + q) * bk + j * bj]);
            }
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
        }
    } else {
#pragma unroll 8
        for (int s = 0; s < 32; s++) {
            const int k = 2 * s + (lane >> 5);
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(A[i * ai + k * ak], B[k * bk + j * bj], c, 0, 0, 0);
        }
    }
    return c;
}

// ---------------------------------------------------------------------------
// Stand-alone forward.  A workgroup of four wavefronts puts the network into
// LDS and takes blocks of 4 x 32 NT samples in turn; NT = 4 once each of 256
// compute units has a workgroup with it, else 2 (more wavefronts, less work each).
constexpr int FWD_BLOCKS = 1024;  // four workgroups for each of 256 compute units
template <bool F32, int NT>
__global__ void __launch_bounds__(256, 2) k_forward(const float *__restrict__ P, const float *__restrict__ norm,
                                                 const float *__restrict__ x, float *__restrict__ y, int B) {
    __shared__ __attribute__((aligned(16))) NetLds<3, F32> net;
    net_to_lds(net, P, (const uint16_t *)nullptr, threadIdx.x, 256);
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (long long b0 = (blockIdx.x * 4ll + w) * (32 * NT); b0 < B; b0 += gridDim.x * 4ll * (32 * NT)) {
        float x0[NT / 2], x1[NT / 2], o[NT / 2][3];
#pragma unroll
        for (int p = 0; p < NT / 2; p++) {
            const long long b = min(b0 + 64 * p + lane, (long long)B - 1);
            normalise(norm, x[2 * b], x[2 * b + 1], x0[p], x1[p]);
        }
        forward_tiles<3, F32, NT>(x0, x1, net, o);
#pragma unroll
        for (int p = 0; p < NT / 2; p++) {
            const long long b = b0 + 64 * p + lane;
            if (b < B)
                for (int k = 0; k < 3; k++) y[3 * b + k] = o[p][k] * norm[5 + 2 * k] + norm[4 + 2 * k];
        }
    }
}

// the surrogate pass's form (both hidden layers on BF16 MFMA, W2 columns
// permuted), four wavefronts per workgroup, 64 samples each in turn
__global__ void __launch_bounds__(256, 2) k_forward_l1mfma(const float *__restrict__ P, const float *__restrict__ norm,
                                                        const float *__restrict__ x, float *__restrict__ y, int B) {
    __shared__ __attribute__((aligned(16))) uint16_t sW2[H * 72];
    __shared__ float sOut[4 * H + 4];  // b2, w3, b3
    for (int r = threadIdx.x; r < H * H; r += 256)
        sW2[(r / H) * 72 + r % H] = bf16_hw(P[OFF_W2 + (r / H) * H + w2_perm_col(r % H)]);
    for (int r = threadIdx.x; r < 4 * H + 3; r += 256) sOut[r] = P[OFF_B2 + r];
    __syncthreads();
    const Net net{sW2, sOut, sOut + H, sOut + 4 * H, 72};
    const L1Ops l1 = l1_operands(P + OFF_W1, P + OFF_B1);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (long long b0 = (blockIdx.x * 4ll + w) * 64; b0 < B; b0 += gridDim.x * 256ll) {
        const long long b = b0 + lane, bc = b < B ? b : B - 1;
        float x0, x1, o[3];
        normalise(norm, x[2 * bc], x[2 * bc + 1], x0, x1);
        forward_wave_l1mfma<3>(x0, x1, net, l1, o);
        if (b < B)
            for (int k = 0; k < 3; k++) y[3 * b + k] = o[k] * norm[5 + 2 * k] + norm[4 + 2 * k];
    }
}

// ---------------------------------------------------------------------------
// Per-cell passes with the surrogate.  T comes from the network; a cell whose
// caloric residual |e(rho, T_hat) - e| / (c_v T_hat) exceeds tol (or is not
// finite) takes one FP64 Newton step on e(rho, T) = e from T_hat -- exact for
// van der Waals, whose e is linear in T; with the Peng-Robinson equation of
// state the residual is taken with e(rho, T_hat) and c_v(rho, T_hat) in FP64,
// and a failing cell runs Newton's method from T_hat to convergence.  The
// residual check validates the temperature only, so P and c_s^2 come from the
// equation of state at the accepted T (explicit once T is known); the network's
// P and c_s^2 outputs are trained and reported but not used here.
//   MLP_STEP    the fields of the multi-kernel step, counters kept
//   MLP_EXPORT  rho, u, T, P to the caller's arrays
//   MLP_SUMS    the conservation partials
// A workgroup keeps the network in LDS and takes runs of 256-cell units as the
// explicit read-back does (512^3 cells: 3.4 ms; with the parameters read from
// global memory by every wavefront 9.4 ms for the fields, and 1.6 ms more to
// export them).  Bound by the vector ALU; on small lattices by the latency of
// putting the network into LDS, so the hidden weights come from their BF16 copy,
// two 16-byte reads a lane, and blocks without cells end at once (Peng-Robinson
// step of 129 x 30 cells: 25.8 us with the parameters read from global memory,
// 29.5 with all of them converted by every block, so 18.9).
enum { MLP_STEP, MLP_EXPORT, MLP_SUMS };
template <int D, int MODE>
__global__ void __launch_bounds__(BX, 2) k_cells_mlp(Grid g, Phys<float> ph, MomSrc<float> m, Fields<float> fl,
                                                  const float *__restrict__ Pn,
                                                  const uint16_t *__restrict__ W2b, const float *__restrict__ norm,
                                                  float tol, unsigned long long *counters, ReadOut o) {
    __shared__ __attribute__((aligned(16))) NetLds<1, false> net;
    double acc[RED_VALS] = {0, 0, 0, 0, 0, 0, 0};
    unsigned n_fb = 0, n_cell = 0, n_it = 0;
    long long u0, u1;
    unsigned per_plane;
    read_units(g, u0, u1, per_plane);
    if (MODE != MLP_SUMS && u0 == u1) return;  // a small lattice leaves most blocks without work
    if (u0 < u1) net_to_lds(net, Pn, W2b, threadIdx.x, BX);
    __syncthreads();
    for (long long un = u0; un < u1; un++) {
        const int z = (int)((unsigned long long)un / per_plane);
        const unsigned p = (unsigned)(un - (long long)z * per_plane) * BX + threadIdx.x;
        int y = (int)(p / (unsigned)g.nx), x = (int)(p - (unsigned)y * (unsigned)g.nx);
        const bool active = y < g.ny;  // other lanes evaluate the plane's last cell and write nothing
        if (!active) {
            x = g.nx - 1;
            y = g.ny - 1;
        }
        const long long c = cell_index<D>(g, x, y, z);
        const CellKin<float> k = cell_kin<D>(g, ph, m, fl.lap, x, y, z);
        const float rho = k.rho, e = k.e;
        float x0[1], x1[1], yh[1][1];
        normalise(norm, rho, e, x0[0], x1[0]);
        forward_tiles<1, false, 2>(x0, x1, net, yh);
        float T = yh[0][0] * norm[5] + norm[4];
        float Pr, c2, ec = 0.0f;
        bool fb;
        if (ph.pr) {
            const double rd = (double)rho, ed = (double)e;
            const double L = pr_log(ph, rd);
            EosPoint q = pr_eos(ph, rd, (double)T, L);
            fb = !(fabs(q.e - ed) <= (double)tol * q.cv * fabs((double)T));
            if (fb) {
                int it = 0;
                const double Td = pr_temperature(ph, rd, ed, (double)T, L, it);
                q = pr_eos(ph, rd, Td, L);
                T = (float)Td;
                n_it += active ? (unsigned)it : 0u;
            }
            if (MODE == MLP_STEP) ec = (float)pr_eos(ph, rd, (double)T, L).e;
            Pr = (float)q.P;
            c2 = (float)q.cs2;
        } else {
            float r = fabsf(ph.cv * T - ph.a * rho - e) / (ph.cv * fabsf(T));
            fb = !(r <= tol);
            if (fb) {
                double Td = (double)T, rd = (double)rho, cv = (double)ph.cv, a = (double)ph.a;
                Td = Td - (cv * Td - a * rd - (double)e) / cv;  // Newton on e(rho, T) - e = 0
                double omb = 1.0 - (double)ph.b * rd;
                T = (float)Td;
                Pr = (float)(rd * (double)ph.R * Td / omb - a * rd * rd);
                c2 = (float)((double)ph.R * Td * (1.0 + (double)ph.R / cv) / (omb * omb) - 2.0 * a * rd);
            } else {
                Pr = vdw_pressure(ph, rho, T);
                c2 = vdw_cs2(ph, rho, T);
            }
        }
        n_fb += fb && active ? 1u : 0u;
        n_cell += active ? 1u : 0u;
        if (!active) continue;
        if constexpr (MODE == MLP_STEP) {
            float theta = Pr * k.inv_rho;
            for (int a = 0; a < D; a++) {
                fl.u[a * g.N + c] = k.u[a];
                fl.F[a * g.N + c] = k.F[a];
                fl.Lam[a * g.N + c] = rho * k.u[a] * (k.u[a] * k.u[a] + 3.0f * (theta - 1.0f / 3.0f));
            }
            fl.T[c] = T;
            fl.P[c] = Pr;
            fl.h[c] = e + theta;
            fl.cs2[c] = c2;
            if (ph.pr) fl.e[c] = ec;
        } else {
            read_cell<D, float, MODE == MLP_SUMS>(g, k, T, Pr, c, (double)ph.b, o, acc);
        }
    }
    if constexpr (MODE == MLP_STEP) {
        unsigned long long *slot = counter_slot(counters);
        wave_count(&slot[0], n_fb);
        wave_count(&slot[1], n_cell);
        if (ph.pr) {
            wave_count(&slot[2], n_it);
            wave_count(&slot[3], n_cell);
        }
    }
    if constexpr (MODE == MLP_SUMS) block_partials(acc, o.partials);
}

// ---------------------------------------------------------------------------
// Training.  A workgroup processes 64 samples of the batch and writes its
// partial gradient (NP values) and partial squared error; a second kernel sums
// the partials in a fixed order.  Loss L = 1/(3B) sum (yhat - that)^2.
//
// Bound by latency: a chain of LDS passes with a barrier between them, each sum
// over samples or neurons in sequence by one lane.  The four wavefronts share
// every pass -- a tile of each product, a quarter of the rows, or one of the
// independent sums each (8192 samples, BF16: 17.6 us with one wavefront doing
// all of them, now 9.6, of which the loads and the launch are about half).
template <bool BF16>
__global__ void __launch_bounds__(256) k_train_partial(const float *__restrict__ P, const float *__restrict__ xn,
                                                       const float *__restrict__ tn, int B, float *__restrict__ gpart,
                                                       float *__restrict__ lpart) {
    __shared__ float H1[64 * LD], H2[64 * LD], DZ[64 * LD], W2[64 * LD], X[64 * 2], DY[64 * 3];
    __shared__ float Pr[3 * 64];  // residuals
    __shared__ float sB2[H], sW3[3 * H + 3];  // b2; w3, b3
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int mt = w >> 1, nt = w & 1;  // this wavefront's tile of each product
    const int b = blockIdx.x * 64 + lane;
    float *G = gpart + (long long)blockIdx.x * NP;
    // every load of the kernel first: behind a barrier each would cost its
    // latency again (the parameters are the last update's, fresh from memory)
    const float x0 = xn[2 * b], x1 = xn[2 * b + 1], target = w < 3 ? tn[3 * b + w] : 0.0f;
    if (threadIdx.x < H) sB2[threadIdx.x] = P[OFF_B2 + threadIdx.x];
    if (threadIdx.x < 3 * H + 3) sW3[threadIdx.x] = P[OFF_W3 + threadIdx.x];
    if (w == 0) {
        X[2 * lane] = x0;
        X[2 * lane + 1] = x1;
    }
#pragma unroll
    for (int r = 0; r < 16; r++) {
        const int q = threadIdx.x + 256 * r;
        W2[(q / H) * LD + q % H] = P[OFF_W2 + q];
    }
#pragma unroll
    for (int r = 0; r < 16; r++) {
        const int j = 16 * w + r;
        H1[lane * LD + j] = relu(fmaf(P[OFF_W1 + 2 * j], x0, fmaf(P[OFF_W1 + 2 * j + 1], x1, P[OFF_B1 + j])));
    }
    __syncthreads();
    {
        const f32x16 acc = wave_tile64<BF16>(H1, LD, 1, W2, 1, LD, mt, nt);  // Z2 = H1 W2^T
        const int cc = acc_col(nt, lane);
        const float b2 = sB2[cc];
#pragma unroll
        for (int v = 0; v < 16; v++) H2[acc_row(mt, v, lane) * LD + cc] = relu(acc[v] + b2);
    }
    __syncthreads();
    // output k = w of the lane's sample, and its residual
    const float scale = 2.0f / (3.0f * (float)B);
    if (w < 3) {
        float s = sW3[3 * H + w];
#pragma unroll 16
        for (int n = 0; n < H; n++) s = fmaf(sW3[w * H + n], H2[lane * LD + n], s);
        const float r = s - target;
        Pr[64 * w + lane] = r;
        DY[3 * lane + w] = scale * r;  // dL / dyhat
    }
    __syncthreads();
    // dZ2[b][n] = (sum_k DY[b][k] W3[k][n]) ReLU'(z2), lane n, a quarter of the
    // samples (the unit is active where its output H2 is positive)
    {
        const float w0 = sW3[lane], w1 = sW3[H + lane], w2 = sW3[2 * H + lane];
#pragma unroll
        for (int r = 0; r < 16; r++) {
            const int bb = 16 * w + r;
            float h2 = H2[bb * LD + lane];
            float d = DY[3 * bb] * w0 + DY[3 * bb + 1] * w1 + DY[3 * bb + 2] * w2;
            DZ[bb * LD + lane] = h2 > 0.0f ? d : 0.0f;  // ReLU'
        }
    }
    // output layer: dW3[k][n] = sum_b DY[b][k] H2[b][n], k = w; db3[k] = sum_b
    // DY[b][k] and the loss by the fourth wavefront
    if (w < 3) {
        float s = 0.0f;
#pragma unroll 16
        for (int bb = 0; bb < 64; bb++) s = fmaf(DY[3 * bb + w], H2[bb * LD + lane], s);
        G[OFF_W3 + w * H + lane] = s;
    } else {
        if (lane < 3) {
            float s = 0.0f;
#pragma unroll 16
            for (int bb = 0; bb < 64; bb++) s += DY[3 * bb + lane];
            G[OFF_B3 + lane] = s;
        }
        const float r0 = Pr[lane], r1 = Pr[64 + lane], r2 = Pr[128 + lane];
        float sq = fmaf(r2, r2, fmaf(r1, r1, r0 * r0));
        for (int o = 32; o > 0; o >>= 1) sq += __shfl_xor(sq, o, 64);
        if (lane == 0) lpart[blockIdx.x] = sq;
    }
    __syncthreads();
    // dW2[n][k] = sum_b dZ2[b][n] H1[b][k]
    {
        const f32x16 acc = wave_tile64<BF16>(DZ, 1, LD, H1, LD, 1, mt, nt);
#pragma unroll
        for (int v = 0; v < 16; v++) G[OFF_W2 + acc_row(mt, v, lane) * H + acc_col(nt, lane)] = acc[v];
    }
    // dH1[b][k] = sum_n dZ2[b][n] W2[n][k], then dZ1 in the place of H2
    {
        const f32x16 acc = wave_tile64<BF16>(DZ, LD, 1, W2, LD, 1, mt, nt);
        const int cc = acc_col(nt, lane);
#pragma unroll
        for (int v = 0; v < 16; v++) {
            const int r = acc_row(mt, v, lane);
            H2[r * LD + cc] = H1[r * LD + cc] > 0.0f ? acc[v] : 0.0f;
        }
    }
    __syncthreads();
    // lane n, j: db2[n] = sum_b dZ2[b][n]; dW1[j][i] = sum_b dZ1[b][j] X[b][i];
    // db1[j] = sum_b dZ1[b][j]; one of the four sums per wavefront
    {
        const float *D = w == 3 ? DZ : H2;
        float s = 0.0f;
        if (w < 2) {
#pragma unroll 16
            for (int bb = 0; bb < 64; bb++) s = fmaf(D[bb * LD + lane], X[2 * bb + w], s);
            G[OFF_W1 + 2 * lane + w] = s;
        } else {
#pragma unroll 16
            for (int bb = 0; bb < 64; bb++) s += D[bb * LD + lane];
            G[(w == 2 ? OFF_B1 : OFF_B2) + lane] = s;
        }
    }
}

// Sum of the per-block partial gradients, in a fixed order: a workgroup takes
// 64 parameters; its 16 wavefronts each sum a contiguous sixteenth of the blocks
// for those parameters (a lane per parameter, loads coalesced across the lanes
// and eight in flight), and lane p of the first wavefront adds the sums in pairs.
// The last workgroup sums the block losses in FP64.  Bound by the latency of the
// partials, which other XCDs have written (128 blocks: 17.6 us with four
// wavefronts and one lane adding up the losses, now 2.8).
constexpr int SUM_WAVES = 16;
__global__ void __launch_bounds__(64 * SUM_WAVES) k_sum_partials(const float *__restrict__ gpart,
                                                                 const float *__restrict__ lpart, int nblk, int B,
                                                                 float *__restrict__ grad, float *__restrict__ loss) {
    __shared__ float part[SUM_WAVES][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (blockIdx.x == gridDim.x - 1) {
        if (w || !loss) return;
        double t = 0.0;
        for (int k = lane; k < nblk; k += 64) t += (double)lpart[k];
        t = wave_sum(t);
        if (lane == 0) loss[0] = (float)(t / (3.0 * (double)B));
        return;
    }
    const int p = blockIdx.x * 64 + lane;
    const int k0 = (int)(((long long)w * nblk) / SUM_WAVES), k1 = (int)(((long long)(w + 1) * nblk) / SUM_WAVES);
    float s = 0.0f;
    if (p < NP) {
#pragma unroll 8
        for (int k = k0; k < k1; k++) s += gpart[(long long)k * NP + p];
    }
    part[w][lane] = s;
    __syncthreads();
    if (w == 0 && p < NP) {
        // in pairs: four roundings after those of a wavefront's run, where one
        // after the other would be 15
        float t[SUM_WAVES];
#pragma unroll
        for (int q = 0; q < SUM_WAVES; q++) t[q] = part[q][lane];
#pragma unroll
        for (int n = SUM_WAVES / 2; n > 0; n /= 2)
#pragma unroll
            for (int q = 0; q < n; q++) t[q] += t[q + n];
        grad[p] = t[0];
    }
}

__global__ void k_adam(float *P, const float *grad, float *m, float *v, float lr, float bc1, float bc2) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= NP) return;
    const float gp = grad[p];
    float mm = 0.9f * m[p] + 0.1f * gp;
    float vv = 0.999f * v[p] + 0.001f * gp * gp;
    m[p] = mm;
    v[p] = vv;
    P[p] -= lr * (mm / bc1) / (sqrtf(vv / bc2) + 1e-8f);
}

__global__ void k_accumulate_loss(const float *loss, double *acc) {
    if (threadIdx.x == 0 && blockIdx.x == 0) acc[0] += (double)loss[0];
}

// counter-based uniform doubles: splitmix64 of (seed, stream, index)
__device__ __forceinline__ double uniform01(unsigned long long seed, unsigned long long k) {
    unsigned long long z = seed + 0x9E3779B97F4A7C15ull * (k + 1);
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return (double)(z >> 11) * (1.0 / 9007199254740992.0);
}

// samples (rho, T) uniform in the box; x = (rho, e), t = (T, P, c_s^2)
__global__ void k_make_samples(int n, unsigned long long seed, Phys<double> ph, double r0, double r1, double T0,
                               double T1, float *x, double *t) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double rho = r0 + (r1 - r0) * uniform01(seed, 2ull * i);
    double T = T0 + (T1 - T0) * uniform01(seed, 2ull * i + 1);
    if (ph.pr) {  // Peng-Robinson targets
        const EosPoint q = pr_eos(ph, rho, T);
        x[2 * i] = (float)rho;
        x[2 * i + 1] = (float)q.e;
        t[3 * i] = T;
        t[3 * i + 1] = q.P;
        t[3 * i + 2] = q.cs2;
        return;
    }
    double e = ph.cv * T - ph.a * rho;
    double omb = 1.0 - ph.b * rho;
    x[2 * i] = (float)rho;
    x[2 * i + 1] = (float)e;
    t[3 * i] = T;
    t[3 * i + 1] = rho * ph.R * T / omb - ph.a * rho * rho;
    t[3 * i + 2] = ph.R * T * (1.0 + ph.R / ph.cv) / (omb * omb) - 2.0 * ph.a * rho;
}

// per-output mean and standard deviation, FP64, deterministic (one block)
__global__ void __launch_bounds__(256) k_target_stats(int n, const double *t, double *stats) {
    __shared__ double sh[256];
    for (int k = 0; k < 3; k++) {
        double s = 0.0;
        for (int i = threadIdx.x; i < n; i += 256) s += t[3 * i + k];
        sh[threadIdx.x] = s;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
            __syncthreads();
        }
        double mean = sh[0] / n;
        __syncthreads();
        double q = 0.0;
        for (int i = threadIdx.x; i < n; i += 256) {
            double d = t[3 * i + k] - mean;
            q += d * d;
        }
        sh[threadIdx.x] = q;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            stats[2 * k] = mean;
            stats[2 * k + 1] = sqrt(sh[0] / n);
        }
        __syncthreads();
    }
}

__global__ void k_normalise_samples(int n, const float *x, const double *t, const float *norm, float *xn, float *tn) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float a, b;
    normalise(norm, x[2 * i], x[2 * i + 1], a, b);
    xn[2 * i] = a;
    xn[2 * i + 1] = b;
    for (int k = 0; k < 3; k++) tn[3 * i + k] = (float)((t[3 * i + k] - (double)norm[4 + 2 * k]) / (double)norm[5 + 2 * k]);
}

}  // namespace mlp
}  // namespace lbm

// ---------------------------------------------------------------------------
static Phys<float> make_phys_f32(const lbm_params &p) {
    Phys<float> ph;
    ph.a = (float)p.a; ph.b = (float)p.b; ph.R = (float)p.R; ph.cv = (float)p.cv;
    ph.mu = (float)p.mu; ph.eta = (float)p.eta; ph.k = (float)p.k; ph.kappa = (float)p.kappa;
    ph.inv_cv = (float)(1.0 / p.cv); ph.k_over_mu = (float)(p.k / p.mu); ph.eta_over_mu = (float)(p.eta / p.mu);
    ph.sgn_eps = (float)p.upwind_eps;
    ph.sc_cmu = (float)p.sc_cmu; ph.sc_ceta = (float)p.sc_ceta; ph.sc_ck = (float)p.sc_ck;
    ph.pr = lbm_eos_is_pr(p.eos) ? 1 : 0;
    ph.pr_m = p.pr_m; ph.pr_Tc = p.pr_Tc; ph.pr_c0 = p.pr_c0; ph.pr_c1 = p.pr_c1;
    return ph;
}
template <int D, int MODE>
static int launch_cells_mlp(lbm_ctx *c, const MomSrc<float> &m, const Fields<float> &fl, const ReadOut &o) {
    hipLaunchKernelGGL((mlp::k_cells_mlp<D, MODE>), dim3(READ_BLOCKS), dim3(BX), 0, c->stream, c->grid,
                       make_phys_f32(c->p), m, fl, c->mlp_params, c->mlp_w2b, c->mlp_norm, (float)c->p.mlp_tol, c->mlp_counters, o);
    return lbm_note(hipGetLastError());
}
template <int D, class C> int launch_fields_mlp(lbm_ctx *c, Fields<C> fl) {
    if constexpr (!std::is_same<C, float>::value) {
        (void)c;
        (void)fl;
        return LBM_EINVAL;
    } else {
        const MomSrc<C> m{fl.rho, (long long)c->p.nx * c->p.ny, (long long)c->grid.N, D + 1};
        return launch_cells_mlp<D, mlp::MLP_STEP>(c, m, fl, ReadOut{});
    }
}
template <int D, class C>
int launch_readback_mlp(lbm_ctx *c, const MomSrc<C> &m, Fields<C> fl, const ReadOut &o) {
    if constexpr (!std::is_same<C, float>::value) {
        (void)c;
        (void)m;
        (void)fl;
        (void)o;
        return LBM_EINVAL;
    } else {
        return o.partials ? launch_cells_mlp<D, mlp::MLP_SUMS>(c, m, fl, o)
                          : launch_cells_mlp<D, mlp::MLP_EXPORT>(c, m, fl, o);
    }
}
#define INSTANTIATE(D, C)                                     \
    template int launch_fields_mlp<D, C>(lbm_ctx *, Fields<C>); \
    template int launch_readback_mlp<D, C>(lbm_ctx *, const MomSrc<C> &, Fields<C>, const ReadOut &);
INSTANTIATE(2, float)
INSTANTIATE(3, float)
INSTANTIATE(2, double)
INSTANTIATE(3, double)
#undef INSTANTIATE

// ---------------------------------------------------------------------------
// Scratch of lbm_mlp_loss_grad_noalloc: the per-block gradient partials (NP
// values per 64 samples) and squared-error partials of a batch of at most
// LBM_MLP_NOALLOC_MAX_BATCH samples, 2.3 MB on every GPU the library runs on,
// held until the process ends.  Host code never passes `scratch` itself to a
// kernel (in host code the name is a stand-in, not a device address): it
// takes the address of each device's copy with hipGetSymbolAddress, once per
// device, and passes that.
namespace {
constexpr int NOALLOC_BLOCKS = LBM_MLP_NOALLOC_MAX_BATCH / 64;
constexpr int NOALLOC_FLOATS = NOALLOC_BLOCKS * mlp::NP + NOALLOC_BLOCKS;
constexpr int NOALLOC_MAX_DEVICES = 64;
__device__ __align__(256) float scratch[NOALLOC_FLOATS];

std::mutex g_scratch_mutex;
float *g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};

// device address of the current device's scratch array (looked up on the
// first call on that device)
int scratch_address(float **out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return lbm_note(hipGetLastError());
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return LBM_EDEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) return lbm_note(e != hipSuccess ? e : hipErrorInvalidSymbol);
        g_scratch_ptr[dev] = (float *)p;
    }
    *out = g_scratch_ptr[dev];
    return LBM_OK;
}
}  // namespace

namespace {
struct DevBuf {
    void *p = nullptr;
    ~DevBuf() {
        if (p) (void)hipFree(p);
    }
    bool alloc(size_t n) { return lbm_note(hipMalloc(&p, n)) == LBM_OK; }
    template <class T> T *as() { return (T *)p; }
};
}  // namespace

extern "C" {

int lbm_mlp_forward(const float *params, const float *norm, const float *x, float *y, int B, int precision,
                    void *stream) {
    if (B < 0 || (precision != LBM_MLP_BF16 && precision != LBM_MLP_F32 && precision != LBM_MLP_BF16_L1))
        return LBM_EINVAL;
    if (B == 0) return LBM_OK;
    if (!params || !norm || !x || !y) return LBM_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    // workgroups of 4 x 32 NT samples
    auto grid = [&](int nt) {
        const long long n = ((long long)B + 128 * nt - 1) / (128 * nt);
        return dim3((unsigned)std::min<long long>(n, mlp::FWD_BLOCKS));
    };
    const bool wide = B >= 256 * 512;
    if (precision == LBM_MLP_BF16_L1)
        hipLaunchKernelGGL(mlp::k_forward_l1mfma, grid(2), dim3(256), 0, s, params, norm, x, y, B);
    else if (precision == LBM_MLP_BF16 && wide)
        hipLaunchKernelGGL((mlp::k_forward<false, 4>), grid(4), dim3(256), 0, s, params, norm, x, y, B);
    else if (precision == LBM_MLP_BF16)
        hipLaunchKernelGGL((mlp::k_forward<false, 2>), grid(2), dim3(256), 0, s, params, norm, x, y, B);
    else if (wide)
        hipLaunchKernelGGL((mlp::k_forward<true, 4>), grid(4), dim3(256), 0, s, params, norm, x, y, B);
    else
        hipLaunchKernelGGL((mlp::k_forward<true, 2>), grid(2), dim3(256), 0, s, params, norm, x, y, B);
    return lbm_note(hipGetLastError());
}

int lbm_mlp_adam(float *params, const float *grad, float *m, float *v, int t, float lr, void *stream) {
    if (!params || !grad || !m || !v || t < 1 || !(lr > 0)) return LBM_EINVAL;
    hipLaunchKernelGGL(mlp::k_adam, dim3((mlp::NP + 255) / 256), dim3(256), 0, (hipStream_t)stream, params, grad, m,
                       v, lr, (float)(1.0 - pow(0.9, (double)t)), (float)(1.0 - pow(0.999, (double)t)));
    return lbm_note(hipGetLastError());
}

static int loss_grad_impl(const float *params, const float *xn, const float *tn, int B, float *grad, float *loss,
                          int precision, hipStream_t s, float *gpart, float *lpart) {
    const int nblk = B / 64;
    if (precision == LBM_MLP_BF16)
        hipLaunchKernelGGL(mlp::k_train_partial<true>, dim3(nblk), dim3(256), 0, s, params, xn, tn, B, gpart, lpart);
    else
        hipLaunchKernelGGL(mlp::k_train_partial<false>, dim3(nblk), dim3(256), 0, s, params, xn, tn, B, gpart, lpart);
    hipLaunchKernelGGL(mlp::k_sum_partials, dim3((mlp::NP + 63) / 64 + 1), dim3(64 * mlp::SUM_WAVES), 0, s, gpart,
                       lpart, nblk, B, grad, loss);
    return lbm_note(hipGetLastError());
}

int lbm_mlp_loss_grad(const float *params, const float *xn, const float *tn, int B, float *grad, float *loss,
                      int precision, void *stream) {
    if (B <= 0 || B % 64 || (precision != LBM_MLP_BF16 && precision != LBM_MLP_F32)) return LBM_EINVAL;
    if (!params || !xn || !tn || !grad || !loss) return LBM_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    DevBuf gp, lp;
    if (!gp.alloc(sizeof(float) * (size_t)(B / 64) * mlp::NP) || !lp.alloc(sizeof(float) * (size_t)(B / 64)))
        return LBM_ENOMEM;
    int rc = loss_grad_impl(params, xn, tn, B, grad, loss, precision, s, gp.as<float>(), lp.as<float>());
    // the scratch buffers are released when this call returns
    if (hipStreamSynchronize(s) != hipSuccess) return LBM_EDEVICE;
    return rc;
}

int lbm_mlp_loss_grad_noalloc(const float *params, const float *xn, const float *tn, int B, float *grad,
                              float *loss, int precision, void *stream) {
    if (B <= 0 || B % 64 || B > LBM_MLP_NOALLOC_MAX_BATCH || (precision != LBM_MLP_BF16 && precision != LBM_MLP_F32))
        return LBM_EINVAL;
    if (!params || !xn || !tn || !grad || !loss) return LBM_EINVAL;
    float *sp = nullptr;
    const int rc = scratch_address(&sp);
    if (rc) return rc;
    // every partial of the B / 64 blocks is written before it is summed, so
    // nothing of a previous call's contents is read
    return loss_grad_impl(params, xn, tn, B, grad, loss, precision, (hipStream_t)stream, sp,
                          sp + (size_t)NOALLOC_BLOCKS * mlp::NP);
}

// Peng-Robinson specific energy e(rho, T) on the host (the same relation the
// kernels evaluate), for the input range of the training box
static double host_pr_energy(const lbm_params &p, double rho, double T) {
    const double r2 = std::sqrt(2.0);
    const double L = std::log((1.0 + (1.0 + r2) * p.b * rho) / (1.0 + (1.0 - r2) * p.b * rho)) / (2.0 * r2 * p.b);
    return p.pr_c0 * T + 0.5 * p.pr_c1 * T * T - p.a * (1.0 + p.pr_m) * (1.0 + p.pr_m * (1.0 - std::sqrt(T / p.pr_Tc))) * L;
}

int lbm_mlp_train(const lbm_params *prm, const double *box, int n, uint64_t seed, int epochs, int batch, float lr,
                  int precision, float *host_params, float *host_norm, double *host_loss) {
    if (!prm || !box || !host_params || !host_norm) return LBM_EINVAL;
    if (batch <= 0 || batch % 64 || n < batch || epochs < 1 || !(lr > 0)) return LBM_EINVAL;
    if (precision != LBM_MLP_BF16 && precision != LBM_MLP_F32) return LBM_EINVAL;
    if (!(box[1] > box[0] && box[3] > box[2] && box[0] > 0 && box[2] > 0)) return LBM_EINVAL;
    if (!(prm->cv > 0) || !(prm->b * box[1] < 1.0)) return LBM_EINVAL;
    if (lbm_eos_is_pr(prm->eos) && !(prm->pr_Tc > 0 && prm->pr_c0 > 0 && prm->b > 0)) return LBM_EINVAL;
    hipStream_t s = nullptr;
    const int nbat = n / batch;
    DevBuf x, t, xn, tn, P, m, v, grad, loss, gpart, lpart, stats, norm, lacc;
    bool ok = x.alloc(sizeof(float) * 2 * (size_t)n) && t.alloc(sizeof(double) * 3 * (size_t)n) &&
              xn.alloc(sizeof(float) * 2 * (size_t)n) && tn.alloc(sizeof(float) * 3 * (size_t)n) &&
              P.alloc(sizeof(float) * mlp::NP) && m.alloc(sizeof(float) * mlp::NP) &&
              v.alloc(sizeof(float) * mlp::NP) && grad.alloc(sizeof(float) * mlp::NP) && loss.alloc(sizeof(float)) &&
              gpart.alloc(sizeof(float) * (size_t)(batch / 64) * mlp::NP) &&
              lpart.alloc(sizeof(float) * (size_t)(batch / 64)) && stats.alloc(sizeof(double) * 6) &&
              norm.alloc(sizeof(float) * 16) && lacc.alloc(sizeof(double));
    if (!ok) return LBM_ENOMEM;
    Phys<double> ph;
    ph.a = prm->a; ph.b = prm->b; ph.R = prm->R; ph.cv = prm->cv;
    ph.mu = ph.eta = ph.k = ph.kappa = 0; ph.inv_cv = 1.0 / prm->cv; ph.k_over_mu = ph.eta_over_mu = 0; ph.sgn_eps = 0;
    ph.sc_cmu = ph.sc_ceta = ph.sc_ck = 0;
    ph.pr = lbm_eos_is_pr(prm->eos) ? 1 : 0;
    ph.pr_m = prm->pr_m; ph.pr_Tc = prm->pr_Tc; ph.pr_c0 = prm->pr_c0; ph.pr_c1 = prm->pr_c1;
    hipLaunchKernelGGL(mlp::k_make_samples, dim3((n + 255) / 256), dim3(256), 0, s, n, (unsigned long long)seed, ph,
                       box[0], box[1], box[2], box[3], x.as<float>(), t.as<double>());
    hipLaunchKernelGGL(mlp::k_target_stats, dim3(1), dim3(256), 0, s, n, t.as<double>(), stats.as<double>());
    double st[6];
    if (hipMemcpy(st, stats.p, sizeof(st), hipMemcpyDeviceToHost) != hipSuccess) return LBM_EDEVICE;
    // input ranges of the box: rho in [r0, r1]; e rises with T and falls
    // with rho (van der Waals e = c_v T - a rho: [c_v T0 - a r1, c_v T1 - a r0];
    // Peng-Robinson likewise, its departure term being negative and growing
    // with density)
    float nh[16] = {0};
    nh[0] = (float)box[0];
    nh[1] = (float)box[1];
    if (ph.pr) {
        nh[2] = (float)host_pr_energy(*prm, box[1], box[2]);
        nh[3] = (float)host_pr_energy(*prm, box[0], box[3]);
    } else {
        nh[2] = (float)(prm->cv * box[2] - prm->a * box[1]);
        nh[3] = (float)(prm->cv * box[3] - prm->a * box[0]);
    }
    for (int k = 0; k < 3; k++) {
        nh[4 + 2 * k] = (float)st[2 * k];
        nh[5 + 2 * k] = (float)(st[2 * k + 1] > 0 ? st[2 * k + 1] : 1.0);
    }
    if (hipMemcpy(norm.p, nh, sizeof(float) * 16, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(P.p, host_params, sizeof(float) * mlp::NP, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemset(m.p, 0, sizeof(float) * mlp::NP) != hipSuccess ||
        hipMemset(v.p, 0, sizeof(float) * mlp::NP) != hipSuccess)
        return LBM_EDEVICE;
    hipLaunchKernelGGL(mlp::k_normalise_samples, dim3((n + 255) / 256), dim3(256), 0, s, n, x.as<float>(),
                       t.as<double>(), norm.as<float>(), xn.as<float>(), tn.as<float>());
    long long it = 0;
    const long long total = (long long)epochs * nbat;
    for (int ep = 0; ep < epochs; ep++) {
        if (ep == epochs - 1 && hipMemset(lacc.p, 0, sizeof(double)) != hipSuccess) return LBM_EDEVICE;
        for (int bi = 0; bi < nbat; bi++, it++) {
            const float *xb = xn.as<float>() + 2LL * bi * batch;
            const float *tb = tn.as<float>() + 3LL * bi * batch;
            int rc = loss_grad_impl(P.as<float>(), xb, tb, batch, grad.as<float>(), loss.as<float>(), precision, s,
                                    gpart.as<float>(), lpart.as<float>());
            if (rc) return rc;
            if (ep == epochs - 1)
                hipLaunchKernelGGL(mlp::k_accumulate_loss, dim3(1), dim3(64), 0, s, loss.as<float>(), lacc.as<double>());
            const double lr_t = 0.5 * lr * (1.0 + cos(M_PI * (double)it / (double)total));  // cosine decay
            const double t1 = (double)(it + 1);
            hipLaunchKernelGGL(mlp::k_adam, dim3((mlp::NP + 255) / 256), dim3(256), 0, s, P.as<float>(),
                               grad.as<float>(), m.as<float>(), v.as<float>(), (float)lr_t,
                               (float)(1.0 - pow(0.9, t1)), (float)(1.0 - pow(0.999, t1)));
        }
    }
    if (lbm_note(hipGetLastError())) return LBM_EDEVICE;
    double la = 0;
    if (hipMemcpy(host_params, P.p, sizeof(float) * mlp::NP, hipMemcpyDeviceToHost) != hipSuccess ||
        hipMemcpy(&la, lacc.p, sizeof(double), hipMemcpyDeviceToHost) != hipSuccess)
        return LBM_EDEVICE;
    std::memcpy(host_norm, nh, sizeof(float) * LBM_MLP_NNORM);
    if (host_loss) *host_loss = la / nbat;
    return LBM_OK;
}

static uint16_t host_bf16(float v) {
    uint32_t u;
    std::memcpy(&u, &v, 4);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;
    return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

int lbm_mlp_set(lbm_ctx *c, const float *host_params, const float *host_norm) {
    if (!c || !host_params || !host_norm) return LBM_EINVAL;
    if (!lbm_eos_uses_mlp(c->p.eos)) return LBM_EINVAL;
    for (int i = 0; i < mlp::H * mlp::H; i++) c->mlp_w2b_host[i] = host_bf16(host_params[mlp::OFF_W2 + i]);
    if (hipMemcpyAsync(c->mlp_params, host_params, sizeof(float) * LBM_MLP_NPARAMS, hipMemcpyHostToDevice,
                       c->stream) != hipSuccess ||
        hipMemcpyAsync(c->mlp_w2b, c->mlp_w2b_host, sizeof(uint16_t) * mlp::H * mlp::H, hipMemcpyHostToDevice,
                       c->stream) != hipSuccess ||
        hipMemcpyAsync(c->mlp_norm, host_norm, sizeof(float) * LBM_MLP_NNORM, hipMemcpyHostToDevice, c->stream) !=
            hipSuccess ||
        hipStreamSynchronize(c->stream) != hipSuccess)
        return LBM_EDEVICE;
    c->mlp_ready = true;
    return LBM_OK;
}

int lbm_eos_stats(lbm_ctx *c, double *frac, double *iters) {
    if (!c) return LBM_EINVAL;
    unsigned long long all[COUNTER_SLOTS * COUNTER_STRIDE], h[4] = {0, 0, 0, 0};
    if (hipMemcpyAsync(all, c->mlp_counters, sizeof(all), hipMemcpyDeviceToHost, c->stream) != hipSuccess ||
        hipStreamSynchronize(c->stream) != hipSuccess)
        return LBM_EDEVICE;
    for (int s = 0; s < COUNTER_SLOTS; s++)
        for (int k = 0; k < 4; k++) h[k] += all[s * COUNTER_STRIDE + k];
    if (frac) *frac = h[1] ? (double)h[0] / (double)h[1] : 0.0;
    if (iters) *iters = h[3] ? (double)h[2] / (double)h[3] : 0.0;
    if (hipMemsetAsync(c->mlp_counters, 0, sizeof(all), c->stream) != hipSuccess) return LBM_EDEVICE;
    return LBM_OK;
}

int lbm_mlp_stats(lbm_ctx *c, double *frac) {
    if (!c || !frac) return LBM_EINVAL;
    return lbm_eos_stats(c, frac, nullptr);
}

}  // extern "C"
