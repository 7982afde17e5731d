// Learned low-fidelity level: a permutation-invariant set network
//   phi(x) = ReLU(W2 ReLU(W1 x + b1) + b2)     per bubble, 4 -> 128 -> 128
//   s      = pool_scale * sum_bubbles phi(x)
//   y      = W4 ReLU(W3 s + b3) + b4            128 -> 128 -> 5
// trained on the solver's QoIs and used as an extra control variate of the
// OF-MLMC estimator (its coefficient from eq. (alpha-matvec) absorbs its
// error).
//
// The 128-wide contractions (and their backward products) run on the matrix
// cores with bf16 operands (round to nearest even from float) and float
// accumulation (v_mfma_f32_32x32x16_bf16), the 4-wide input layer on them in
// float (v_mfma_f32_32x32x2_f32: each product and sum rounded as the chain of
// FMAs b + x0 w0 + x1 w1 + x2 w2 + x3 w3).  The 5-wide output layer, pooling,
// loss and Adam are vector code in float.  Every reduction has a fixed order,
// so results do not depend on scheduling.
//
// A training step is four launches: the pool (phi_pool_kernel), the head with
// its backward part (head_kernel<true>), the backward part of phi
// (phi_back_kernel, which recomputes the activations: storing and re-reading
// them took 30 times the bytes) and the sum of the workgroups' partial
// gradients (grad_sum_kernel).
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <type_traits>

#include "nn_kernels.h"

namespace ofm {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(2 * sizeof(float)))) float floatx2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
struct alignas(16) u16x8 { uint16_t v[8]; };
struct alignas(16) u32x4 { uint32_t v[4]; };
struct alignas(8) u32x2 { uint32_t v[2]; };

__device__ __forceinline__ uint16_t to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);   // round to nearest, ties to even
    return (uint16_t)(u >> 16);
}

// Two floats as packed bf16 (round to nearest even).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    const floatx2 f = { lo, hi };
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}

// In one operation: with a visible infinity the compiler makes it a maximum
// behind a canonicalisation, two.  A NaN gives 0, as fmaxf(v, 0) does.
__device__ __forceinline__ float relu(float v) {
    float inf = __builtin_inff();
    asm("" : "+s"(inf));
    return __builtin_amdgcn_fmed3f(v, 0.f, inf);
}

__device__ __forceinline__ bf16x8 frag(const uint16_t* p)
{
    u16x8 t = *reinterpret_cast<const u16x8*>(p);
    return __builtin_bit_cast(bf16x8, t);
}

// Output element e (0..15) of a 32x32 MFMA block held by `lane`: column
// lane % 32, row (e / 4) * 8 + (lane / 32) * 4 + e % 4.
__device__ __forceinline__ int mfma_row(int e, int lane) { return (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3); }

__device__ __forceinline__ floatx16 splat16(float v)
{
    floatx16 r;
#pragma unroll
    for (int e = 0; e < 16; ++e) r[e] = v;
    return r;
}

// Hidden unit that row m of an input-layer block stands for when the block is
// computed with units as rows (below): lane / 32 = h then holds, in elements
// 8 t .. 8 t + 7, the units 16 t + 8 h .. 16 t + 8 h + 7 of its bubble, which
// is the left operand of the next layer's MFMA as it stands.
__device__ __forceinline__ int unit_of_row(int m)
{
    return 16 * (m >> 4) + 8 * ((m >> 2) & 1) + 4 * ((m >> 3) & 1) + (m & 3);
}

constexpr int HP = 128 + 8;   // LDS pitch of 128 bf16: 16-byte fragments stay aligned
constexpr int RP = 64 + 8;    // the same for 64

// A 128 x 128 weight matrix into LDS [n][k], pitch HP (256 threads), and eight
// of its rows at one column as a fragment.
__device__ __forceinline__ void stage_weights(const uint16_t* __restrict__ W, uint16_t* sW, int tid)
{
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int e = (q * 256 + tid) * 8;
        *reinterpret_cast<u16x8*>(&sW[(e >> 7) * HP + (e & 127)]) = *reinterpret_cast<const u16x8*>(&W[e]);
    }
}
__device__ __forceinline__ bf16x8 column_frag(const uint16_t* sW, int n0, int k)
{
    u16x8 v;
#pragma unroll
    for (int i = 0; i < 8; ++i) v.v[i] = sW[(n0 + i) * HP + k];
    return __builtin_bit_cast(bf16x8, v);
}

// ---------------------------------------------------------------------------
// phi and the sum pool.  A wavefront takes 64 bubbles of one set at a time:
// the input layer as W1 X^T (two blocks of 32 bubbles), whose result, after
// ReLU and rounding, is already the left operand of the 128 x 128 layer
// (unit_of_row), so that activations never pass through LDS; W2 is read from
// LDS as the right operand, each fragment used for both blocks.  Layer 2 goes
// by blocks of 32 columns: bias, ReLU and column sums of one block are vector
// work that the matrix products of the next hide.  A set's sum adds its
// groups of 64 in order, two at a time, whichever wavefront computed them, so
// that its result does not depend on the launch.
//
// Per 64 bubbles: 64 bf16 and 16 float MFMAs (1.32 us of a SIMD's matrix core
// at the rates measured for them alone) and 640 vector operations (1.47 us),
// which overlap in part: 2.3 us.  16384 sets of 500: 1117 us before (input
// layer on the vector units, activations through LDS, 128 rows a workgroup),
// 305 now (365 before the activations took one operation each and the next
// inputs were loaded ahead).
//
// PER_WAVE: a set per wavefront (the next group's inputs loaded ahead);
// otherwise a set per workgroup, its groups dealt to the four wavefronts.
// ---------------------------------------------------------------------------
template <bool PER_WAVE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(PER_WAVE ? 2 : 3)))
phi_pool_kernel(const float* __restrict__ x, const int32_t* __restrict__ offsets, int n_sets,
                const float* __restrict__ P, const uint16_t* __restrict__ W2bf, float pool_scale,
                uint16_t* __restrict__ s_bf)
{
    __shared__ __align__(16) uint16_t sW[128 * HP];             // W2 [n][k]
    __shared__ __align__(16) float sb1[128];
    __shared__ float colsum[PER_WAVE ? 1 : 4][128];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, half = lane >> 5;
    stage_weights(W2bf, sW, tid);
    if (tid < 128) sb1[tid] = P[NN_B1 + tid];
    float a1[4][2], b2[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
#pragma unroll
        for (int k = 0; k < 2; ++k) a1[u][k] = P[NN_W1 + (u * 32 + unit_of_row(col)) * 4 + 2 * k + half];
        b2[u] = P[NN_B2 + u * 32 + col];
    }
    __syncthreads();

    // this lane's inputs of the bubbles c .. min(c + 64, r1) - 1
    auto load = [&](int c, int r1, float (&xb)[2][2]) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int r = c + i * 32 + col;
#pragma unroll
            for (int k = 0; k < 2; ++k) xb[i][k] = r < r1 ? x[(int64_t)r * 4 + 2 * k + half] : 0.f;
        }
    };

    // their column sums (every lane gets those of its four columns)
    auto group_of = [&](auto full_c, int c, int r1, const float (&xb)[2][2], float (&cs)[4]) {
        constexpr bool FULL = decltype(full_c)::value;    // 64 bubbles: no row check
        bf16x8 h[2][8];                           // ReLU(z1), the left operands of layer 2
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            floatx16 d[2];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 b = *reinterpret_cast<const float4*>(&sb1[u * 32 + 16 * (g >> 1) + 8 * half + 4 * (g & 1)]);
                d[0][4 * g] = b.x; d[0][4 * g + 1] = b.y; d[0][4 * g + 2] = b.z; d[0][4 * g + 3] = b.w;
            }
            d[1] = d[0];
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int i = 0; i < 2; ++i) d[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[u][k], xb[i][k], d[i], 0, 0, 0);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    u32x4 p;
#pragma unroll
                    for (int q = 0; q < 4; ++q) p.v[q] = pack_bf16(relu(d[i][8 * t + 2 * q]), relu(d[i][8 * t + 2 * q + 1]));
                    h[i][2 * u + t] = __builtin_bit_cast(bf16x8, p);
                }
        }
        auto product = [&](int j, floatx16 (&acc)[2]) {
            acc[0] = acc[1] = splat16(0.f);
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const bf16x8 b = frag(&sW[(j * 32 + col) * HP + t * 16 + half * 8]);
#pragma unroll
                for (int i = 0; i < 2; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(h[i][t], b, acc[i], 0, 0, 0);
            }
        };
        auto column = [&](int j, const floatx16 (&acc)[2]) {
            float v = 0.f;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float r = fmaxf(acc[i][e] + b2[j], 0.f);
                    v += FULL || c + i * 32 + mfma_row(e, lane) < r1 ? r : 0.f;
                }
            cs[j] = v + __shfl_xor(v, 32, 64);
        };
        floatx16 acc[2][2];
        product(0, acc[0]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j + 1 < 4) product(j + 1, acc[(j + 1) & 1]);
            column(j, acc[j & 1]);
        }
    };
    auto group = [&](int c, int r1, const float (&xb)[2][2], float (&cs)[4]) {
        if (c + 64 <= r1)
            group_of(std::true_type{}, c, r1, xb, cs);
        else
            group_of(std::false_type{}, c, r1, xb, cs);
    };

    if constexpr (PER_WAVE) {
        // one group of 64 an iteration (at least one a set); the next one's
        // inputs, also those of the next set, are loaded ahead
        const int step = gridDim.x * 4;
        int set = blockIdx.x * 4 + wave;
        if (set >= n_sets) return;
        int c = offsets[set], r1 = offsets[set + 1];
        float xb[2][2], sum[4] = { 0.f, 0.f, 0.f, 0.f }, first[4] = { 0.f, 0.f, 0.f, 0.f };
        bool odd = false;
        load(c, r1, xb);
#pragma clang loop unroll(disable)
        while (set < n_sets) {
            const bool last = c + 64 >= r1;
            const int nset = last ? set + step : set;
            int nc = c + 64, nr1 = r1;
            if (last && nset < n_sets) { nc = offsets[nset]; nr1 = offsets[nset + 1]; }
            float xn[2][2], cs[4];
            load(nc, nset < n_sets ? nr1 : nc, xn);
            group(c, r1, xb, cs);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (odd) sum[j] += first[j] + cs[j];
                first[j] = cs[j];
            }
            odd = !odd;
            if (last) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (odd) sum[j] += first[j];
                    if (half == 0) s_bf[(int64_t)set * 128 + j * 32 + col] = to_bf16(pool_scale * sum[j]);
                    sum[j] = 0.f;
                }
                odd = false;
            }
            set = nset;
            c = nc;
            r1 = nr1;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int k = 0; k < 2; ++k) xb[i][k] = xn[i][k];
        }
    } else {
        for (int set = blockIdx.x; set < n_sets; set += gridDim.x) {
            const int r0 = offsets[set], r1 = offsets[set + 1];
            float sum = 0.f;                      // of column tid (tid < 128)
            for (int c0 = r0; c0 < r1; c0 += 256) {
                const int c = c0 + wave * 64;
                float cs[4] = { 0.f, 0.f, 0.f, 0.f };
                if (c < r1) {
                    float xb[2][2];
                    load(c, r1, xb);
                    group(c, r1, xb, cs);
                }
                if (half == 0)
#pragma unroll
                    for (int j = 0; j < 4; ++j) colsum[wave][j * 32 + col] = cs[j];
                __syncthreads();
                if (tid < 128) {
                    sum += colsum[0][tid] + colsum[1][tid];
                    sum += colsum[2][tid] + colsum[3][tid];
                }
                __syncthreads();
            }
            if (tid < 128) s_bf[(int64_t)set * 128 + tid] = to_bf16(pool_scale * sum);
        }
    }
}

// ---------------------------------------------------------------------------
// Head: z3 = W3 s + b3, y = W4 ReLU(z3) + b4, 32 sets a workgroup and pass.
// Wavefront w computes columns 32 w .. 32 w + 31 of z3 (operands straight
// from memory in fragment order); the output layer is one thread per (set,
// output), a chain of 128 FMAs over LDS.
//
// TRAIN: also the loss, dz3 = (dy W4) [z3 > 0], ds = dz3 W3 (bf16 operands)
// and this workgroup's part of the gradients of W3, b3, W4, b4.  An element
// of dz3 as computed (sets in registers, columns over lanes) is the left
// operand of dW3 = dz3^T s as it stands, with the sets taken in the order the
// registers hold them; ds needs it with columns in registers: through LDS.
// ---------------------------------------------------------------------------
template <bool TRAIN>
__global__ void __launch_bounds__(256) head_kernel(const uint16_t* __restrict__ s_bf, const uint16_t* __restrict__ W3bf,
                                                   const float* __restrict__ P, int n_sets,
                                                   const float* __restrict__ mean, const float* __restrict__ stdv,
                                                   float* __restrict__ y_phys, const float* __restrict__ y_true,
                                                   float* __restrict__ ds, float* __restrict__ part)
{
    constexpr int AP = 129;
    __shared__ __align__(16) uint16_t smem[TRAIN ? 128 * HP : 64 * AP];   // TRAIN: first W3
    float* sA = reinterpret_cast<float*>(smem);         // ReLU(z3) [set][k]
    uint16_t* sZ = smem + 64 * HP;                      // TRAIN: dz3 as bf16 [set][n]
    __shared__ float sW4[NN_DOUT * 128];
    __shared__ float sY[TRAIN ? 32 * NN_DOUT : 1];      // dy
    __shared__ float sQ[TRAIN ? 256 : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lc = lane & 31, half = lane >> 5, n = wave * 32 + lc;
    const float b3 = P[NN_B3 + n];
    for (int e = tid; e < NN_DOUT * 128; e += 256) sW4[e] = P[NN_W4 + e];
    float w4[NN_DOUT];
    bf16x8 wt[TRAIN ? 8 : 1];                           // W3 with column n over K (ds)
    floatx16 dW3[TRAIN ? 4 : 1];
    float db3 = 0.f, dw4[3] = { 0.f, 0.f, 0.f }, db4 = 0.f, loss = 0.f;
    if constexpr (TRAIN) {
#pragma unroll
        for (int o = 0; o < NN_DOUT; ++o) w4[o] = P[NN_W4 + o * 128 + n];
        stage_weights(W3bf, smem, tid);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 8; ++t) wt[t] = column_frag(smem, t * 16 + half * 8, n);
#pragma unroll
        for (int q = 0; q < 4; ++q) dW3[q] = splat16(0.f);
    }
    for (int s0 = blockIdx.x * 32; s0 < n_sets; s0 += gridDim.x * 32) {
        const int sr = min(s0 + lc, n_sets - 1);
        floatx16 acc = splat16(0.f);
#pragma unroll
        for (int t = 0; t < 8; ++t)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(&s_bf[(int64_t)sr * 128 + t * 16 + half * 8]),
                                                          frag(&W3bf[n * 128 + t * 16 + half * 8]), acc, 0, 0, 0);
        __syncthreads();                                // the pass before has read sA, sY and sZ
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            acc[e] += b3;
            sA[mfma_row(e, lane) * AP + n] = fmaxf(acc[e], 0.f);
        }
        __syncthreads();
        if (tid < 32 * NN_DOUT) {
            const int s = tid & 31, o = tid >> 5, set = s0 + s;
            float y = P[NN_B4 + o];
            #pragma unroll 16
            for (int k = 0; k < 128; ++k) y += sA[s * AP + k] * sW4[o * 128 + k];
            float dy = 0.f;
            if (set < n_sets) {
                if (y_phys) y_phys[(int64_t)set * NN_DOUT + o] = y * stdv[o] + mean[o];
                if constexpr (TRAIN) {
                    const float d = y - (y_true[(int64_t)set * NN_DOUT + o] - mean[o]) / stdv[o];
                    dy = 2.f * d / (float)(n_sets * NN_DOUT);
                    loss += d * d;
                }
            }
            if constexpr (TRAIN) sY[s * NN_DOUT + o] = dy;
        }
        if constexpr (TRAIN) {
            __syncthreads();
            u32x4 af[2];
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float d[2];
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        const int e = 8 * t + 2 * q + b, s = mfma_row(e, lane);
                        float v = 0.f;
#pragma unroll
                        for (int o = 0; o < NN_DOUT; ++o) v += sY[s * NN_DOUT + o] * w4[o];
                        d[b] = acc[e] > 0.f ? v : 0.f;
                        db3 += d[b];
                        sZ[s * HP + n] = to_bf16(d[b]);
                    }
                    af[t].v[q] = pack_bf16(d[0], d[1]);
                }
            // dW3[n][k] over this pass's sets, in the registers' order
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) {
                    u16x8 b;
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        b.v[i] = s_bf[(int64_t)min(s0 + mfma_row(8 * t + i, lane), n_sets - 1) * 128 + kb * 32 + lc];
                    dW3[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[t]),
                                                                     __builtin_bit_cast(bf16x8, b), dW3[kb], 0, 0, 0);
                }
            // dW4: this thread's column, outputs tid / 128, + 2, + 4
            for (int s = 0; s < 32; ++s) {
                const float a = sA[s * AP + (tid & 127)];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const int o = (tid >> 7) + 2 * q;
                    if (o < NN_DOUT) dw4[q] += sY[s * NN_DOUT + o] * a;
                }
                if (tid < NN_DOUT) db4 += sY[s * NN_DOUT + tid];
            }
            __syncthreads();
            floatx16 dsa = splat16(0.f);
#pragma unroll
            for (int t = 0; t < 8; ++t)
                dsa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(&sZ[lc * HP + t * 16 + half * 8]), wt[t], dsa, 0, 0, 0);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int set = s0 + mfma_row(e, lane);
                if (set < n_sets) ds[(int64_t)set * 128 + n] = dsa[e];
            }
        }
    }
    if constexpr (TRAIN) {
        float* g = part + (int64_t)blockIdx.x * NN_PART_HEAD;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
            for (int e = 0; e < 16; ++e) g[(wave * 32 + mfma_row(e, lane)) * 128 + kb * 32 + lc] = dW3[kb][e];
        db3 += __shfl_xor(db3, 32, 64);
        if (half == 0) g[NN_B3 - NN_W3 + n] = db3;
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int o = (tid >> 7) + 2 * q;
            if (o < NN_DOUT) g[NN_W4 - NN_W3 + o * 128 + (tid & 127)] = dw4[q];
        }
        if (tid < NN_DOUT) g[NN_B4 - NN_W3 + tid] = db4;
        sQ[tid] = loss;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if (tid < w) sQ[tid] += sQ[tid + w];
            __syncthreads();
        }
        if (tid == 0) g[NN_PART_HEAD - 1] = sQ[0];
    }
}

// ---------------------------------------------------------------------------
// Backward part of phi over the bubbles of the workgroup's sets, 64 at a time:
//   dz2 = pool_scale ds[set] [z2 > 0],  dW2 = dz2^T h1,  db2 = sum dz2,
//   dz1 = (dz2 W2) [z1 > 0],            dW1 = dz1^T x,   db1 = sum dz1,
// with h1 and z2 computed again from x.  Wavefront w owns 32 hidden units of
// the input layer and 32 of the second: it computes its units of h1 in both
// orders (for the left operand of z2 and the right one of dW2), its columns
// of z2, its rows of dW2 (64 accumulators a lane, kept over all bubbles) and
// its columns of dh1.  dz2 as computed (bubbles in registers, units over
// lanes) is the left operand of dW2; dh1 needs it with units in registers:
// through LDS, like h1.
// One workgroup a CU (a set each, at most 256) in lockstep over three barriers:
// bound by each group's chain of 56 MFMAs, 700 vector and 120 LDS operations a
// wavefront.  256 sets of 500 took 2.2 ms in 12 launches over 500 MB of stored
// activations, gradients and GEMM splits before, 40 us now.  (Half sets to 512
// workgroups: 47 us, and twice the parts to sum.)  A set stays with its
// workgroup, so that few or very uneven sets leave CUs idle: a gradient call
// over one set of 500, 73 us; of 10^5, 6.4 ms; of 10^6, 64 ms (282 us, 9.8 and
// 91 ms with the stored activations spread over rows).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
phi_back_kernel(const float* __restrict__ x, const int32_t* __restrict__ offsets, int n_sets,
                const float* __restrict__ P, const uint16_t* __restrict__ W2bf, const float* __restrict__ ds,
                float pool_scale, float* __restrict__ part)
{
    __shared__ __align__(16) uint16_t smem[128 * HP + 128 * RP];
    uint16_t* sH = smem;                                // h1 [bubble][unit]
    uint16_t* sD = smem + 64 * HP;                      // dz2 [bubble][unit]
    uint16_t* sT = smem + 128 * HP;                     // h1 [unit][bubble, in the registers' order]
    __shared__ float4 sX[64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lc = lane & 31, half = lane >> 5, n = wave * 32 + lc;
    // groups of this workgroup's sets, up to 65 (the other loads hide these)
    int total = 0;
    for (int set = blockIdx.x + lane * gridDim.x; set < n_sets; set += 64 * gridDim.x)
        total += min((offsets[set + 1] - offsets[set] + 63) >> 6, 65);
    bf16x8 w2[8], w2t[8];                               // W2 row n; W2 column n
    stage_weights(W2bf, smem, tid);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        w2[t] = frag(&smem[n * HP + t * 16 + half * 8]);
        w2t[t] = column_frag(smem, t * 16 + half * 8, n);
    }
    float a1[2], b1[2], bias1[16];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        a1[k] = P[NN_W1 + (wave * 32 + unit_of_row(lc)) * 4 + 2 * k + half];
        b1[k] = P[NN_W1 + n * 4 + 2 * k + half];
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) bias1[e] = P[NN_B1 + wave * 32 + unit_of_row(mfma_row(e, lane))];
    const float bn1 = P[NN_B1 + n], bn2 = P[NN_B2 + n];
    floatx16 dW2[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) dW2[q] = splat16(0.f);
    float db2 = 0.f, db1 = 0.f, dw1[4] = { 0.f, 0.f, 0.f, 0.f };
    // The sums so far, added to this workgroup's part: at the end, and after
    // each 64 groups before it (a float sum over all bubbles of a large set, one
    // after another, loses digits: 1e-3 of W1's gradient at 3 x 10^5 like ones,
    // 1e-5 in blocks of 4096).
    int groups = 0;
    bool begun = false;
    auto add = [&](float* p, float v) { *p = begun ? *p + v : v; };
    auto store = [&]() {
        // (the empty statement: addresses not worked out ahead of the groups and
        // held over them)
        float* g = part + (int64_t)blockIdx.x * NN_PART_PHI;
        uint32_t at = NN_W2 + (wave * 32 + 4 * half) * 128 + lc;
        asm volatile("" : "+s"(g), "+v"(at));
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
#pragma unroll
            for (int e = 0; e < 16; ++e) add(&g[at + mfma_row(e, 0) * 128 + kb * 32], dW2[kb][e]);
            dW2[kb] = splat16(0.f);
        }
        db2 += __shfl_xor(db2, 32, 64);
        db1 += __shfl_xor(db1, 32, 64);
#pragma unroll
        for (int k = 0; k < 4; ++k) dw1[k] += __shfl_xor(dw1[k], 32, 64);
        if (half == 0) {
            add(&g[NN_B2 + n], db2);
            add(&g[NN_B1 + n], db1);
#pragma unroll
            for (int k = 0; k < 4; ++k) add(&g[NN_W1 + n * 4 + k], dw1[k]);
        }
        db2 = db1 = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) dw1[k] = 0.f;
        begun = true;
        groups = 0;
    };
    auto all_sets = [&](auto many_c) {
        for (int set = blockIdx.x; set < n_sets; set += gridDim.x) {
            const int r0 = offsets[set], r1 = offsets[set + 1];
            const float dsc = pool_scale * ds[(int64_t)set * 128 + n];
            const uint32_t dlo = to_bf16(dsc), dhi = dlo << 16;
            float xn[2][2];                                 // inputs of the next 64 bubbles
            auto load = [&](int c) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int r = c + i * 32 + lc;
#pragma unroll
                    for (int k = 0; k < 2; ++k) xn[i][k] = r < r1 ? x[(int64_t)r * 4 + 2 * k + half] : 0.f;
                }
            };
            load(r0);
            for (int c = r0; c < r1; c += 64) {
                float xb[2][2];
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int k = 0; k < 2; ++k) xb[i][k] = xn[i][k];
                load(c + 64);
                __syncthreads();                            // the pass before has read sX, sH, sT and sD
                if (wave == 0)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int k = 0; k < 2; ++k) reinterpret_cast<float*>(&sX[i * 32 + lc])[2 * k + half] = xb[i][k];
                uint32_t on1 = 0;                           // bit 16 i + e: z1 > 0
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    floatx16 d, dt = splat16(bn1);
#pragma unroll
                    for (int e = 0; e < 16; ++e) d[e] = bias1[e];
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        d = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[k], xb[i][k], d, 0, 0, 0);      // [unit][bubble]
                        dt = __builtin_amdgcn_mfma_f32_32x32x2f32(xb[i][k], b1[k], dt, 0, 0, 0);    // [bubble][unit]
                    }
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        u32x4 p;
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            p.v[q] = pack_bf16(relu(d[8 * t + 2 * q]), relu(d[8 * t + 2 * q + 1]));
                        *reinterpret_cast<u32x4*>(&sH[(i * 32 + lc) * HP + wave * 32 + t * 16 + half * 8]) = p;
                    }
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        u32x2 p;
#pragma unroll
                        for (int q = 0; q < 2; ++q)
                            p.v[q] = pack_bf16(relu(dt[4 * g + 2 * q]), relu(dt[4 * g + 2 * q + 1]));
                        *reinterpret_cast<u32x2*>(&sT[n * RP + i * 32 + 16 * (g >> 1) + 8 * half + 4 * (g & 1)]) = p;
                    }
#pragma unroll
                    for (int e = 0; e < 16; ++e) on1 |= dt[e] > 0.f ? 1u << (16 * i + e) : 0u;
                }
                __syncthreads();
                floatx16 z[2] = { splat16(0.f), splat16(0.f) };
#pragma unroll
                for (int t = 0; t < 8; ++t)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        z[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(&sH[(i * 32 + lc) * HP + t * 16 + half * 8]), w2[t],
                                                                      z[i], 0, 0, 0);
                int count = 0;
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        u32x4 af;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int e = 8 * t + 2 * q, row = i * 32 + mfma_row(e, lane);
                            const bool p0 = z[i][e] + bn2 > 0.f && c + row < r1;
                            const bool p1 = z[i][e + 1] + bn2 > 0.f && c + row + 1 < r1;
                            count += (p0 ? 1 : 0) + (p1 ? 1 : 0);
                            sD[row * HP + n] = (uint16_t)(p0 ? dlo : 0u);
                            sD[(row + 1) * HP + n] = (uint16_t)(p1 ? dlo : 0u);
                            af.v[q] = (p0 ? dlo : 0u) | (p1 ? dhi : 0u);
                        }
#pragma unroll
                        for (int kb = 0; kb < 4; ++kb)
                            dW2[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                __builtin_bit_cast(bf16x8, af), frag(&sT[(kb * 32 + lc) * RP + i * 32 + t * 16 + half * 8]),
                                dW2[kb], 0, 0, 0);
                    }
                db2 += count ? dsc * (float)count : 0.f;    // dsc may be infinite or NaN (a label that is)
                __syncthreads();
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    floatx16 dh = splat16(0.f);
#pragma unroll
                    for (int t = 0; t < 8; ++t)
                        dh = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(&sD[(i * 32 + lc) * HP + t * 16 + half * 8]), w2t[t],
                                                                    dh, 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const float d = (on1 >> (16 * i + e)) & 1u ? dh[e] : 0.f;
                        const float4 xv = sX[i * 32 + mfma_row(e, lane)];
                        dw1[0] += d * xv.x;
                        dw1[1] += d * xv.y;
                        dw1[2] += d * xv.z;
                        dw1[3] += d * xv.w;
                        db1 += d;
                    }
                }
                if constexpr (decltype(many_c)::value)
                    if (++groups == 64) store();
            }
        }
    };
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) total = min(total + __shfl_xor(total, off, 64), 65);
    // a loop of its own where they are few: the stores in it cost a call over
    // 256 sets of 500 4 %
    if (total > 64) {
        all_sets(std::true_type{});
        store();
    } else {
        all_sets(std::false_type{});
        store();
    }
}

// Gradients and loss from the workgroups' parts: 64 parameters a workgroup,
// each wavefront a quarter of the parts, in a fixed order.
__global__ void __launch_bounds__(256) grad_sum_kernel(const float* __restrict__ part_phi, int n_phi,
                                                       const float* __restrict__ part_head, int n_head, int n_err,
                                                       float* __restrict__ G, float* __restrict__ loss)
{
    __shared__ float sh[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lane;               // NN_NPARAM: the loss
    const bool phi = i < NN_W3;
    const float* p = phi ? part_phi + i : part_head + (i - NN_W3);
    const int np = i > NN_NPARAM ? 0 : phi ? n_phi : n_head, stride = phi ? NN_PART_PHI : NN_PART_HEAD;
    const int per = (np + 3) / 4, b0 = wave * per, b1 = min(np, b0 + per);
    float s = 0.f;
#pragma unroll 8
    for (int b = b0; b < b1; ++b) s += p[(int64_t)b * stride];
    sh[wave][lane] = s;
    __syncthreads();
    if (wave == 0) {
        const float t = (sh[0][lane] + sh[1][lane]) + (sh[2][lane] + sh[3][lane]);
        if (i < NN_NPARAM) G[i] = t;
        if (i == NN_NPARAM) *loss = t / (float)n_err;
    }
}

// Adam (bias-corrected), float masters; refreshes the bf16 shadows.
__global__ void __launch_bounds__(256) adam_kernel(float* __restrict__ P, const float* __restrict__ G,
                                                   float* __restrict__ m, float* __restrict__ v, int n, float lr,
                                                   float b1, float b2, float eps, float c1, float c2,
                                                   uint16_t* __restrict__ W2bf, uint16_t* __restrict__ W3bf)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const float g = G[i];
    const float mi = b1 * m[i] + (1.f - b1) * g;
    const float vi = b2 * v[i] + (1.f - b2) * g * g;
    m[i] = mi;
    v[i] = vi;
    const float p = P[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    P[i] = p;
    if (i >= NN_W2 && i < NN_W2 + 128 * 128) W2bf[i - NN_W2] = to_bf16(p);
    if (i >= NN_W3 && i < NN_W3 + 128 * 128) W3bf[i - NN_W3] = to_bf16(p);
}

__global__ void __launch_bounds__(256) shadow_kernel(const float* __restrict__ P, uint16_t* __restrict__ W2bf,
                                                     uint16_t* __restrict__ W3bf)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= 128 * 128) return;
    W2bf[i] = to_bf16(P[NN_W2 + i]);
    W3bf[i] = to_bf16(P[NN_W3 + i]);
}

// He-uniform initialisation from a counter-based generator (SplitMix64 of
// seed ^ index); biases zero.
__device__ __forceinline__ uint64_t sm64(uint64_t z)
{
    z += 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__global__ void __launch_bounds__(256) init_params_kernel(float* __restrict__ P, uint64_t seed)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= NN_NPARAM) return;
    int fan_in = 0;
    if (i < NN_B1) fan_in = 4;
    else if (i >= NN_W2 && i < NN_B2) fan_in = 128;
    else if (i >= NN_W3 && i < NN_B3) fan_in = 128;
    else if (i >= NN_W4 && i < NN_B4) fan_in = 128;
    if (fan_in == 0) { P[i] = 0.f; return; }
    const double u = (double)(sm64(seed ^ (uint64_t)i) >> 11) * (1.0 / 9007199254740992.0);
    const double lim = sqrt(6.0 / fan_in);
    P[i] = (float)((2.0 * u - 1.0) * lim);
}

// Per-bubble inputs ((c - centre)/R, ln(r/r_median)/sigma).
__global__ void __launch_bounds__(256) features_kernel(const double* __restrict__ bub, int64_t rows, int ndim,
                                                       double cx, double cy, double cz, double R, double rmed,
                                                       double sigma, float* __restrict__ x)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= rows) return;
    const double* b = bub + 4 * i;
    x[4 * i + 0] = (float)((b[0] - cx) / R);
    x[4 * i + 1] = (float)(ndim > 1 ? (b[1] - cy) / R : 0.0);
    x[4 * i + 2] = (float)(ndim > 2 ? (b[2] - cz) / R : 0.0);
    x[4 * i + 3] = (float)(log(b[3] / rmed) / sigma);
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static int cdiv64(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

hipError_t nn_phi_pool(const float* x, const int32_t* offsets, int n_sets, int64_t rows, const float* P,
                       const uint16_t* W2bf, float pool_scale, uint16_t* s_bf, hipStream_t st)
{
    // A set per wavefront wastes nothing inside a set: taken where the sets give
    // each SIMD a wavefront, or have one group of 64 each on average, so that
    // three wavefronts of a workgroup would idle.  Fewer, larger sets finish
    // earlier dealt to four wavefronts.  A forward call by wavefronts against
    // by workgroups: 256 sets of 500, 47 us against 35; 1000 of 500, 50 against
    // 49; 1000 of 100, 34 against 38; 2000 of 500, 63 against 65; 4096 of 100,
    // 48 against 61; 1000 of 60, 32 against 37.  Measured with sets of like
    // size: the rule does not see a large set among many small ones, whose
    // groups one wavefront then takes in turn (1000 sets of 1 and one of 60000,
    // 2.1 ms; one set of 10^5 alone, dealt to four, 1.2).
    if (n_sets >= 1024 || rows <= 64 * (int64_t)n_sets)
        hipLaunchKernelGGL((phi_pool_kernel<true>), dim3(n_sets < 4096 ? (n_sets + 3) / 4 : 1024), dim3(256), 0, st, x, offsets,
                           n_sets, P, W2bf, pool_scale, s_bf);
    else
        hipLaunchKernelGGL((phi_pool_kernel<false>), dim3(n_sets), dim3(256), 0, st, x, offsets, n_sets, P, W2bf, pool_scale,
                           s_bf);
    return hipGetLastError();
}

hipError_t nn_head(const uint16_t* s_bf, const uint16_t* W3bf, const float* P, int n_sets, const float* mean,
                   const float* stdv, float* y_phys, hipStream_t s)
{
    hipLaunchKernelGGL((head_kernel<false>), dim3(cdiv64(n_sets, 32)), dim3(256), 0, s, s_bf, W3bf, P, n_sets, mean, stdv,
                       y_phys, nullptr, nullptr, nullptr);
    return hipGetLastError();
}

// workgroups (and parts of the gradient) of the training kernels
int nn_parts_head(int n_sets) { return cdiv64(n_sets, 32) < 64 ? cdiv64(n_sets, 32) : 64; }
int nn_parts_phi(int n_sets) { return n_sets < 256 ? n_sets : 256; }

hipError_t nn_head_train(const uint16_t* s_bf, const uint16_t* W3bf, const float* P, int n_sets, const float* mean,
                         const float* stdv, const float* y_true, float* ds, float* part, hipStream_t s)
{
    hipLaunchKernelGGL((head_kernel<true>), dim3(nn_parts_head(n_sets)), dim3(256), 0, s, s_bf, W3bf, P, n_sets, mean, stdv,
                       nullptr, y_true, ds, part);
    return hipGetLastError();
}

hipError_t nn_phi_back(const float* x, const int32_t* offsets, int n_sets, const float* P, const uint16_t* W2bf,
                       const float* ds, float pool_scale, float* part, hipStream_t s)
{
    hipLaunchKernelGGL(phi_back_kernel, dim3(nn_parts_phi(n_sets)), dim3(256), 0, s, x, offsets, n_sets, P, W2bf, ds,
                       pool_scale, part);
    return hipGetLastError();
}

hipError_t nn_grad_sum(const float* part_phi, const float* part_head, int n_sets, float* G, float* loss, hipStream_t s)
{
    hipLaunchKernelGGL(grad_sum_kernel, dim3(NN_NPARAM / 64 + 1), dim3(256), 0, s, part_phi, nn_parts_phi(n_sets), part_head,
                       nn_parts_head(n_sets), n_sets * NN_DOUT, G, loss);
    return hipGetLastError();
}

hipError_t nn_adam(float* P, const float* G, float* m, float* v, float lr, float b1, float b2, float eps, int t,
                   uint16_t* W2bf, uint16_t* W3bf, hipStream_t s)
{
    const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
    hipLaunchKernelGGL(adam_kernel, dim3(cdiv64(NN_NPARAM, 256)), dim3(256), 0, s, P, G, m, v, NN_NPARAM, lr, b1, b2,
                       eps, c1, c2, W2bf, W3bf);
    return hipGetLastError();
}

hipError_t nn_shadow(const float* P, uint16_t* W2bf, uint16_t* W3bf, hipStream_t s)
{
    hipLaunchKernelGGL(shadow_kernel, dim3(64), dim3(256), 0, s, P, W2bf, W3bf);
    return hipGetLastError();
}

hipError_t nn_init_params(float* P, uint64_t seed, hipStream_t s)
{
    hipLaunchKernelGGL(init_params_kernel, dim3(cdiv64(NN_NPARAM, 256)), dim3(256), 0, s, P, seed);
    return hipGetLastError();
}

hipError_t nn_features(const double* bub, int64_t rows, int ndim, const double* center, double R, double rmed,
                       double sigma, float* x, hipStream_t s)
{
    hipLaunchKernelGGL(features_kernel, dim3(cdiv64(rows, 256)), dim3(256), 0, s, bub, rows, ndim, center[0], center[1],
                       center[2], R, rmed, sigma, x);
    return hipGetLastError();
}

}  // namespace ofm
