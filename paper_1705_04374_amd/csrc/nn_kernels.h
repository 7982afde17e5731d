// Launchers of the set-network kernels (nn_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

namespace ofm {

// flat parameter layout (float): W1[128][4] b1[128] W2[128][128] b2[128]
// W3[128][128] b3[128] W4[5][128] b4[5]; W[out][in]
constexpr int NN_DIN = 4, NN_WIDTH = 128, NN_DOUT = 5;
constexpr int NN_W1 = 0;
constexpr int NN_B1 = NN_W1 + 128 * 4;
constexpr int NN_W2 = NN_B1 + 128;
constexpr int NN_B2 = NN_W2 + 128 * 128;
constexpr int NN_W3 = NN_B2 + 128;
constexpr int NN_B3 = NN_W3 + 128 * 128;
constexpr int NN_W4 = NN_B3 + 128;
constexpr int NN_B4 = NN_W4 + NN_DOUT * 128;
constexpr int NN_NPARAM = NN_B4 + NN_DOUT;

// A workgroup's part of the gradients: those of phi (W1, b1, W2, b2), and
// those of the head (W3, b3, W4, b4) and the squared errors' sum.
constexpr int NN_PART_PHI = NN_W3;
constexpr int NN_PART_HEAD = NN_NPARAM - NN_W3 + 1;

// s_bf: the pooled activations as bf16, [n_sets][128]
hipError_t nn_phi_pool(const float* x, const int32_t* offsets, int n_sets, int64_t rows, const float* P,
                       const uint16_t* W2bf, float pool_scale, uint16_t* s_bf, hipStream_t st);
hipError_t nn_head(const uint16_t* s_bf, const uint16_t* W3bf, const float* P, int n_sets, const float* mean,
                   const float* stdv, float* y_phys, hipStream_t s);
int nn_parts_head(int n_sets);
int nn_parts_phi(int n_sets);
// ds: d loss / d pooled activations [n_sets][128]; part [nn_parts_head][NN_PART_HEAD]
hipError_t nn_head_train(const uint16_t* s_bf, const uint16_t* W3bf, const float* P, int n_sets, const float* mean,
                         const float* stdv, const float* y_true, float* ds, float* part, hipStream_t s);
// part [nn_parts_phi][NN_PART_PHI]
hipError_t nn_phi_back(const float* x, const int32_t* offsets, int n_sets, const float* P, const uint16_t* W2bf,
                       const float* ds, float pool_scale, float* part, hipStream_t s);
hipError_t nn_grad_sum(const float* part_phi, const float* part_head, int n_sets, float* G, float* loss, hipStream_t s);
hipError_t nn_adam(float* P, const float* G, float* m, float* v, float lr, float b1, float b2, float eps, int t,
                   uint16_t* W2bf, uint16_t* W3bf, hipStream_t s);
hipError_t nn_shadow(const float* P, uint16_t* W2bf, uint16_t* W3bf, hipStream_t s);
hipError_t nn_init_params(float* P, uint64_t seed, hipStream_t s);
hipError_t nn_features(const double* bub, int64_t rows, int ndim, const double* center, double R, double rmed,
                       double sigma, float* x, hipStream_t s);

}  // namespace ofm
