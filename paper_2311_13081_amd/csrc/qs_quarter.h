// Quarter-lane layout of the bf16 actor's kernel: lane L = j + 16 k holds
// quarter k of env j; register c of quarter k holds observation feature
// q_phi(c, k).
#pragma once
#include "qs_device.h"

namespace qs {

typedef float f4q __attribute__((ext_vector_type(4)));

constexpr int Q_C = 37;          // K-chunks of layer 1

// Observation feature of chunk c, quarter k (or -1 for padding).
__host__ __device__ constexpr int q_phi(int c, int k) {
  return c < 5 ? (4 * c + k < 18 ? 4 * c + k : -1) : 18 + 4 * (c - 5) + k;
}

// The 18 observed state features of the lane's env (p, R row-major, v, w),
// with the actor's observation noise when enabled, in the quarter layout:
// F[c] = feature 4c + k (0 past the end).
template <bool EXTRAS>
__device__ inline void quarter_state_features(const DevCfg& c, uint32_t e, uint32_t ep, int t_ep,
                                              int k, const float x[NS], float F[5],
                                              const SetPoint& sp) {
  float Rm[9];
  rotmat(x + 3, Rm);
  float sf[20] = {x[0], x[1], x[2], Rm[0], Rm[1], Rm[2], Rm[3], Rm[4], Rm[5], Rm[6],
                  Rm[7], Rm[8], x[7], x[8], x[9], x[10], x[11], x[12], 0.0f, 0.0f};
  if (EXTRAS) {
    sp.apply(c, sf);
    add_obs_noise<1>(c, e, ep, t_ep, sf);
  }
#pragma unroll
  for (int cc = 0; cc < 5; ++cc)
    F[cc] = k == 0 ? sf[4 * cc] : k == 1 ? sf[4 * cc + 1] : k == 2 ? sf[4 * cc + 2]
                                                                    : sf[4 * cc + 3];
}

// ReLU mask word of a quarter-lane record (row REC_M + k of the lane's env,
// k its quarter): bit 8 n + r is set when layer-1 neuron 16 n + 4 k + r of
// the env has a positive pre-activation, bit 8 n + 4 + r the same for layer
// 2.  z1, z2: the lane's result tiles, before or after the ReLU (z > 0 and
// relu(z) > 0 agree, NaN included).
__device__ inline uint32_t quarter_mask(const f4q z1[4], const f4q z2[4]) {
  uint32_t m = 0u;
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      m |= (z1[n][r] > 0.0f ? 1u : 0u) << (8 * n + r);
      m |= (z2[n][r] > 0.0f ? 1u : 0u) << (8 * n + 4 + r);
    }
  return m;
}

}  // namespace qs
