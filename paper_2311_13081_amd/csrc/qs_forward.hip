// Forward kernels of the batched quadrotor step: initialisation and reset,
// snapshots, and the plain five-kernel step (the fused kernels live in
// qs_tile.hip, qs_split.hip and qs_fused.hip, dynamics-only rollouts in qs_dynamics.hip).
//
// Layout: one env per lane, struct-of-arrays in HBM ([K][N]) so every global
// access of a wave is a contiguous 256-byte segment.
// Fused multiply-adds only where one expression of the source holds the
// product and the sum: the kernels that promise equal results then round the
// shared arithmetic the same way (left to the optimiser, fusing depends on what
// surrounds the inlined code).
#pragma clang fp contract(on)
#include "qs_forward.h"
#include "qs_tile.h"

namespace qs {

// ---------------------------------------------------------------------------
// Init / reset / snapshots
// ---------------------------------------------------------------------------

// Draws per-env parameters (when params != 0) and episode-0 start states.
__global__ void k_init(DevCfg c, SimBufs b, int params) {
  const int N = c.n_envs;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N) return;
  float th[NP];
  if (params) {
    env_params(c, (uint32_t)e, th);
#pragma unroll
    for (int i = 0; i < NP; ++i) b.theta[i * N + e] = th[i];
  } else {
#pragma unroll
    for (int i = 0; i < NP; ++i) th[i] = b.theta[i * N + e];
  }
  float s[NS];
  const float ah = reset_state(c, (uint32_t)e, 0u, th[0], th[4], th[5], th[6], s);
#pragma unroll
  for (int i = 0; i < NS; ++i) b.state[i * N + e] = s[i];
  for (int i = 0; i < NH * NA; ++i) b.ring[i * N + e] = ah;
  b.head[e] = 0;
  b.t_ep[e] = 0;
  b.ep[e] = 0;
  b.ret[e] = 0.0f;
  b.ret[(size_t)N + e] = 0.0f;
  b.last_len[e] = 0;
}

// Snapshot copies.  Each thread loads a batch of rows before storing any of
// them: the source and destination may not be assumed disjoint, so a
// load-store-load sequence would wait out one memory round trip per row.
__global__ void k_get_state(SimBufs b, int N, float* state, float* hist, int32_t* t_ep,
                            int32_t* ep, float* ret, int32_t* last_len) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N) return;
  if (state) {
    float v[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) v[i] = b.state[i * N + e];
#pragma unroll
    for (int i = 0; i < NS; ++i) state[i * N + e] = v[i];
  }
  if (hist) {
    const int h = b.head[e];
#pragma unroll
    for (int s0 = 0; s0 < NH; s0 += 8) {
      float v[8 * NA];
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const int slot = (h + s0 + s) & (NH - 1);
#pragma unroll
        for (int a = 0; a < NA; ++a) v[s * NA + a] = b.ring[(slot * NA + a) * N + e];
      }
#pragma unroll
      for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int a = 0; a < NA; ++a) hist[((s0 + s) * NA + a) * N + e] = v[s * NA + a];
    }
  }
  if (t_ep) t_ep[e] = b.t_ep[e];
  if (ep) ep[e] = b.ep[e];
  if (ret) {
    const float r0 = b.ret[e], r1 = b.ret[(size_t)N + e];
    ret[e] = r0;
    ret[(size_t)N + e] = r1;
  }
  if (last_len) last_len[e] = b.last_len[e];
}

__global__ void k_set_state(SimBufs b, int N, const float* state, const float* hist,
                            const int32_t* t_ep, const int32_t* ep, const float* ret,
                            const int32_t* last_len) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N) return;
  if (state) {
    float v[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) v[i] = state[i * N + e];
#pragma unroll
    for (int i = 0; i < NS; ++i) b.state[i * N + e] = v[i];
  }
  if (hist) {
#pragma unroll
    for (int i0 = 0; i0 < NH * NA; i0 += 32) {
      float v[32];
#pragma unroll
      for (int i = 0; i < 32; ++i) v[i] = hist[(i0 + i) * N + e];
#pragma unroll
      for (int i = 0; i < 32; ++i) b.ring[(i0 + i) * N + e] = v[i];
    }
    b.head[e] = 0;
  }
  if (t_ep) b.t_ep[e] = t_ep[e];
  if (ep) b.ep[e] = ep[e];
  if (ret) {
    const float r0 = ret[e], r1 = ret[(size_t)N + e];
    b.ret[e] = r0;
    b.ret[(size_t)N + e] = r1;
  }
  if (last_len) b.last_len[e] = last_len[e];
}

// ---------------------------------------------------------------------------
// Plain path: five kernels per step, every intermediate through HBM.
// ---------------------------------------------------------------------------

// obs[146][N] = {p, R(q), v, w, H oldest..newest}
__global__ void __launch_bounds__(256) k_plain_obs(DevCfg c, SimBufs b, float* __restrict__ obs) {
  const int N = c.n_envs;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N) return;
  float q[4], f[18];
#pragma unroll
  for (int i = 0; i < 4; ++i) q[i] = b.state[(3 + i) * N + e];
  rotmat(q, f + 3);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    f[i] = b.state[i * N + e];
    f[12 + i] = b.state[(7 + i) * N + e];
    f[15 + i] = b.state[(10 + i) * N + e];
  }
  SetPoint sp;
  sp.load(c, N, e);
  sp.apply(c, f);
  add_obs_noise<0>(c, (uint32_t)e, (uint32_t)b.ep[e], b.t_ep[e], f);
#pragma unroll
  for (int i = 0; i < 18; ++i) obs[i * N + e] = f[i];
  const int h = b.head[e];
  for (int s = 0; s < NH; ++s) {
    const int slot = (h + s) & (NH - 1);
#pragma unroll
    for (int a = 0; a < NA; ++a)
      obs[(size_t)(18 + s * NA + a) * N + e] = b.ring[(slot * NA + a) * N + e];
  }
}

// The three actor layers of the plain path: the tile kernel's products in its
// order and operand layout (qs_tile.h), two 16-env tiles per wave, so the
// actions equal the fused kernels' bit for bit; only the layer outputs go
// through HBM ([64][N], [64][N], [4][N]).  Lanes of envs past the batch load
// the last env and store nothing.
constexpr int P_ENVS = 128;  // envs of a workgroup (4 waves of 2 tiles)

// h1[64][N] = ReLU(W1 obs + b1).
__global__ void __launch_bounds__(256) k_plain_l1(int N, const float* __restrict__ W,
                                                  const float* __restrict__ in,
                                                  float* __restrict__ out) {
  __shared__ u4t sW[T_G2 * T_P * 64];
  __shared__ uint32_t flags[4];
  const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int first = blockIdx.x * P_ENVS + 32 * (threadIdx.x >> 6);
  // every input load in flight before the weights are staged
  float v[2][4][8], F[2][5];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int e = min(first + 16 * b + li, N - 1);
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int i = 0; i < 8; ++i) v[b][c][i] = in[(size_t)(18 + NA * (8 * c + i) + lg) * N + e];
#pragma unroll
    for (int i = 0; i < 5; ++i) F[b][i] = in[(size_t)min(4 * i + lg, 17) * N + e];
    if (lg >= 2) F[b][4] = 0.0f;  // features 18, 19: padding
  }
  __builtin_amdgcn_sched_barrier(0);
  set_flag(!stage_fragments<4>(W, sW, T_G2, tile_src), flags);
  __syncthreads();
  if (first >= N) return;
  u4t x[4][2][T_P], xs[1][2][T_P];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint32_t p[T_P];
        split_pair(v[b][c][2 * q], v[b][c][2 * q + 1], p);
#pragma unroll
        for (int s = 0; s < T_P; ++s) x[c][b][s][q] = p[s];
      }
    state_operand(F[b], xs[0][b]);
  }
  f4t a1[4][2];
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    f4t h[1][2], as[1][2];
    Frags<1> f;
    split_sum<4, 1, 2>([&](int c) { f.load(sW, 4 * n + c, 0, lane); return f; }, x, h);
    split_sum<1, 1, 2>([&](int) { f.load(sW, T_GS + n, 0, lane); return f; }, xs, as);
#pragma unroll
    for (int b = 0; b < 2; ++b) a1[n][b] = h[0][b] + as[0][b];
  }
  const bool bad_actor = any_flag(flags);
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int oe = first + 16 * b + li;
    const uint64_t nan = nan_slots(a1[0][b], [&](int s) {
      return in[(size_t)(18 + NA * s + lg) * N + min(oe, N - 1)];
    });
#pragma unroll
    for (int r = 0; r < 4; ++r) a1[0][b][r] = relu_bits(a1[0][b][r]);
    carry_nan(a1[0][b], (bad_actor ? ~0ull : nan) | nan_lanes(F[b]));
    if (oe < N)
#pragma unroll
      for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          out[(size_t)(16 * n + 4 * lg + r) * N + oe] = relu_bits(a1[n][b][r]);
  }
}

// h2[64][N] = ReLU(W2 h1 + b2).
__global__ void __launch_bounds__(256) k_plain_l2(int N, const float* __restrict__ W,
                                                  const float* __restrict__ in,
                                                  float* __restrict__ out) {
  __shared__ u4t sW[(T_G - T_G2) * T_P * 64];
  __shared__ uint32_t flags[4];
  const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int first = blockIdx.x * P_ENVS + 32 * (threadIdx.x >> 6);
  f4t h1[4][2];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int e = min(first + 16 * b + li, N - 1);
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) h1[n][b][r] = in[(size_t)(16 * n + 4 * lg + r) * N + e];
  }
  __builtin_amdgcn_sched_barrier(0);
  set_flag(!stage_fragments<4>(W, sW, T_G - T_G2,
                               [](int g, int l, int e) { return tile_src(T_G2 + g, l, e); }),
           flags);
  __syncthreads();
  if (first >= N) return;
  u4t x[2][2][T_P];
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int b = 0; b < 2; ++b) hidden_operand(h1[2 * m][b], h1[2 * m + 1][b], x[m][b]);
  f4t a2[4][2];
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    f4t acc[1][2], b2;
    Frags<1> f;
    split_sum<2, 1, 2>([&](int m) { f.load(sW, 2 * n + m, 0, lane); return f; }, x, acc);
#pragma unroll
    for (int r = 0; r < 4; ++r) b2[r] = W[OFF_B2 + 16 * n + 4 * lg + r];
#pragma unroll
    for (int b = 0; b < 2; ++b) a2[n][b] = acc[0][b] + b2;
  }
  const bool bad_actor = any_flag(flags);
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int oe = first + 16 * b + li;
#pragma unroll
    for (int r = 0; r < 4; ++r) a2[0][b][r] = relu_bits(a2[0][b][r]);
    carry_nan(a2[0][b], (bad_actor ? ~0ull : 0ull) | __ballot(h1[0][b][0] != h1[0][b][0]));
    if (oe < N)
#pragma unroll
      for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          out[(size_t)(16 * n + 4 * lg + r) * N + oe] = relu_bits(a2[n][b][r]);
  }
}

// act[4][N] = tanh(W3 h2 + b3).
__global__ void __launch_bounds__(256) k_plain_l3(int N, const float* __restrict__ W,
                                                  const float* __restrict__ in,
                                                  float* __restrict__ out) {
  __shared__ __attribute__((aligned(16))) float sW[NA * T_W3_LD + NA];  // W3 rows, then b3
  const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int first = blockIdx.x * P_ENVS + 32 * (threadIdx.x >> 6);
  f4t h2[4][2];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int e = min(first + 16 * b + li, N - 1);
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) h2[n][b][r] = in[(size_t)(16 * n + 4 * lg + r) * N + e];
  }
  stage_lds(sW, NA * T_W3_LD, W, [](int i) {
    const int r = i / T_W3_LD, k = i % T_W3_LD;
    return k < NHID ? OFF_W3 + r * NHID + k : -1;
  });
  stage_lds(sW + NA * T_W3_LD, NA, W, [](int i) { return OFF_B3 + i; });
  __syncthreads();
  if (first >= N) return;
  float z3[NA];
  Layer3 l3;
  l3.load(sW, sW + NA * T_W3_LD);
  tile_layer3<2>(l3.w, l3.b, h2, z3);
  const int oe = first + 16 * (lg & 1) + li;
  if (oe < N)
#pragma unroll
    for (int o = 0; o < NA; ++o)
      if ((o & 1) == (lg >> 1)) out[(size_t)o * N + oe] = tanh_act(z3[o]);
}

// Dynamics, reward, history push, episode bookkeeping and reset.  DIST: the
// dynamics carry the episode disturbance terms (instantiated as the fused
// kernel instantiates its dynamics: with the training extras or a set point).
template <bool DIST>
__global__ void __launch_bounds__(256) k_plain_dyn(DevCfg c, SimBufs b,
                                                   const float* __restrict__ act,
                                                   float* __restrict__ reward_out,
                                                   uint8_t* __restrict__ done_out,
                                                   float* __restrict__ state_out) {
  const int N = c.n_envs;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N) return;
  float th[NP], x[NS], a[NA], u[NA];
#pragma unroll
  for (int i = 0; i < NP; ++i) th[i] = b.theta[i * N + e];
#pragma unroll
  for (int i = 0; i < NS; ++i) x[i] = b.state[i * N + e];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    a[i] = act[i * N + e];
    u[i] = action_to_rpm(c, a[i]);
  }
  Body<float> B = make_body<float>(th);
  if (DIST) {
    float dist[6];
    disturbance(c, (uint32_t)e, (uint32_t)b.ep[e], dist);
    set_disturbance(B, dist);
  }
  rk4_step<float, DIST>(B, c.arm, c.km, c.g, c.dt, (c.flags & F_RENORM_Q) != 0, x, u);
  const float r = reward(c, x, a);
  int h = b.head[e];
#pragma unroll
  for (int i = 0; i < NA; ++i) b.ring[(h * NA + i) * N + e] = a[i];
  h = (h + 1) & (NH - 1);
  int t_ep = b.t_ep[e] + 1;
  const uint32_t d = episode_end(c, x, t_ep);
  EpAcc acc;
  acc.load(b, N, e);
  acc.add(r, d && (c.flags & F_AUTORESET), t_ep);
  acc.store(b, N, (uint32_t)e);
  if (d && (c.flags & F_AUTORESET)) {
    const int ep = b.ep[e] + 1;
    b.ep[e] = ep;
    t_ep = 0;
    const float ah = reset_state(c, (uint32_t)e, (uint32_t)ep, th[0], th[4], th[5], th[6], x);
    for (int i = 0; i < NH * NA; ++i) b.ring[i * N + e] = ah;
    h = 0;
  }
  b.head[e] = h;
  b.t_ep[e] = t_ep;
#pragma unroll
  for (int i = 0; i < NS; ++i) b.state[i * N + e] = x[i];
  if (reward_out) reward_out[e] = r;
  if (done_out) done_out[e] = (uint8_t)d;
  if (state_out)
#pragma unroll
    for (int i = 0; i < NS; ++i) state_out[i * N + e] = x[i];
}

// Observations of the current state (for a caller that runs its own policy
// or critic): the actor observation with the noise of the coming step, and
// the critic's privileged observation {p, R, v, w, w_m, f_r, tau_r} (Sec. IV).
__global__ void __launch_bounds__(256) k_observe(DevCfg c, SimBufs b, float* __restrict__ aobs,
                                                 float* __restrict__ cobs) {
  const int N = c.n_envs;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N) return;
  float x[NS], f[18];
#pragma unroll
  for (int i = 0; i < NS; ++i) x[i] = b.state[i * N + e];
  rotmat(x + 3, f + 3);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    f[i] = x[i];
    f[12 + i] = x[7 + i];
    f[15 + i] = x[10 + i];
  }
  const uint32_t ep = (uint32_t)b.ep[e];
  if (cobs) {
    float d[6];
    disturbance(c, (uint32_t)e, ep, d);
#pragma unroll
    for (int i = 0; i < 18; ++i) cobs[i * N + e] = f[i];
#pragma unroll
    for (int i = 0; i < 4; ++i) cobs[(18 + i) * N + e] = x[13 + i];
#pragma unroll
    for (int i = 0; i < 6; ++i) cobs[(22 + i) * N + e] = d[i];
  }
  if (aobs) {
    SetPoint sp;
    sp.load(c, N, e);
    sp.apply(c, f);
    add_obs_noise(c, (uint32_t)e, ep, b.t_ep[e], f);
#pragma unroll
    for (int i = 0; i < 18; ++i) aobs[i * N + e] = f[i];
    const int h = b.head[e];
    for (int s = 0; s < NH; ++s) {
      const int slot = (h + s) & (NH - 1);
#pragma unroll
      for (int a = 0; a < NA; ++a)
        aobs[(size_t)(18 + s * NA + a) * N + e] = b.ring[(slot * NA + a) * N + e];
    }
  }
}

// Ends the episodes of the envs with mask[e] != 0 and starts their next ones,
// as an in-step reset does: episode + 1, step 0, the start state of (env,
// episode + 1), the history filled with the env's hover action, and the
// episode accumulators closed (the running return and the step count become
// the last finished episode's).
__global__ void k_reset_envs(DevCfg c, SimBufs b, const uint8_t* __restrict__ mask) {
  const int N = c.n_envs;
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N || !mask[e]) return;
  float th[NP], s[NS];
#pragma unroll
  for (int i = 0; i < NP; ++i) th[i] = b.theta[(size_t)i * N + e];
  const int ep = b.ep[e] + 1;
  const float ah = reset_state(c, (uint32_t)e, (uint32_t)ep, th[0], th[4], th[5], th[6], s);
#pragma unroll
  for (int i = 0; i < NS; ++i) b.state[(size_t)i * N + e] = s[i];
  for (int i = 0; i < NH * NA; ++i) b.ring[(size_t)i * N + e] = ah;
  b.ret[(size_t)N + e] = b.ret[e];
  b.ret[e] = 0.0f;
  b.last_len[e] = b.t_ep[e];
  b.head[e] = 0;
  b.t_ep[e] = 0;
  b.ep[e] = ep;
}

// Rewards of given transitions under the configured reward constants: r(s',
// a) of the reward equation (Sec. IV) for M post-step states s [17][M] and
// actions a [4][M] (e.g. a replay buffer re-scored after the constants
// changed).
__global__ void __launch_bounds__(256) k_reward_batch(DevCfg c, const float* __restrict__ s,
                                                      const float* __restrict__ a, int M,
                                                      float* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= M) return;
  float x[NS], u[NA];
#pragma unroll
  for (int k = 0; k < NS; ++k) x[k] = s[(size_t)k * M + i];
#pragma unroll
  for (int k = 0; k < NA; ++k) u[k] = a[(size_t)k * M + i];
  out[i] = reward(c, x, u);
}

// Copies the state to a [17][N] slice (start state of a recorded rollout).
__global__ void k_copy_state(SimBufs b, int N, float* __restrict__ out) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N) return;
#pragma unroll
  for (int i = 0; i < NS; ++i) out[i * N + e] = b.state[i * N + e];
}


// ---------------------------------------------------------------------------
// Host-side launchers
// ---------------------------------------------------------------------------

static inline unsigned nblk(int n, int bs) { return (unsigned)((n + bs - 1) / bs); }

hipError_t launch_init(const DevCfg& c, const SimBufs& b, int params, hipStream_t st) {
  hipLaunchKernelGGL(k_init, dim3(nblk(c.n_envs, 256)), dim3(256), 0, st, c, b, params);
  return hipGetLastError();
}

hipError_t launch_get_state(const SimBufs& b, int N, float* state, float* hist, int32_t* t_ep,
                            int32_t* ep, float* ret, int32_t* last_len, hipStream_t st) {
  hipLaunchKernelGGL(k_get_state, dim3(nblk(N, 256)), dim3(256), 0, st, b, N, state, hist, t_ep,
                     ep, ret, last_len);
  return hipGetLastError();
}

hipError_t launch_set_state(const SimBufs& b, int N, const float* state, const float* hist,
                            const int32_t* t_ep, const int32_t* ep, const float* ret,
                            const int32_t* last_len, hipStream_t st) {
  hipLaunchKernelGGL(k_set_state, dim3(nblk(N, 256)), dim3(256), 0, st, b, N, state, hist, t_ep,
                     ep, ret, last_len);
  return hipGetLastError();
}

hipError_t launch_plain_step(const DevCfg& c, const SimBufs& b, const PlainBufs& p,
                             const float* W, const float* ext_act, float* reward, uint8_t* done,
                             float* state_out, hipStream_t st) {
  const int N = c.n_envs;
  const dim3 g(nblk(N, 256)), blk(256);
  const float* act = ext_act;
  if (!ext_act) {
    hipLaunchKernelGGL(k_plain_obs, g, blk, 0, st, c, b, p.obs);
    const dim3 g2(nblk(N, P_ENVS));
    hipLaunchKernelGGL(k_plain_l1, g2, blk, 0, st, N, W, p.obs, p.h1);
    hipLaunchKernelGGL(k_plain_l2, g2, blk, 0, st, N, W, p.h1, p.h2);
    hipLaunchKernelGGL(k_plain_l3, g2, blk, 0, st, N, W, p.h2, p.act);
    act = p.act;
  }
  const bool ex = (c.flags & (F_DISTURB | F_OBS_NOISE)) != 0 || c.target != nullptr;
  hipLaunchKernelGGL(ex ? k_plain_dyn<true> : k_plain_dyn<false>, g, blk, 0, st, c, b, act,
                     reward, done, state_out);
  return hipGetLastError();
}


hipError_t launch_observe(const DevCfg& c, const SimBufs& b, float* actor_obs, float* critic_obs,
                          hipStream_t st) {
  hipLaunchKernelGGL(k_observe, dim3(nblk(c.n_envs, 256)), dim3(256), 0, st, c, b, actor_obs,
                     critic_obs);
  return hipGetLastError();
}

hipError_t launch_reset_envs(const DevCfg& c, const SimBufs& b, const uint8_t* mask,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_reset_envs, dim3(nblk(c.n_envs, 256)), dim3(256), 0, st, c, b, mask);
  return hipGetLastError();
}

hipError_t launch_reward_batch(const DevCfg& c, const float* s, const float* a, int M, float* out,
                               hipStream_t st) {
  hipLaunchKernelGGL(k_reward_batch, dim3(nblk(M, 256)), dim3(256), 0, st, c, s, a, M, out);
  return hipGetLastError();
}

hipError_t launch_copy_state(const SimBufs& b, int N, float* out, hipStream_t st) {
  hipLaunchKernelGGL(k_copy_state, dim3(nblk(N, 256)), dim3(256), 0, st, b, N, out);
  return hipGetLastError();
}


hipError_t launch_recompute(const DevCfg& c, const SimBufs& b, const float* W, int T, int K,
                            const float* ck_in, float* rec, hipStream_t st) {
  // the kernel of taped rollouts, in record mode: one segment of T steps
  const RecSpan one{{rec}, 0, K, T};
  const TapedKernel tk = taped_kernel(c);
  if (tk == TAPED_SPLIT)
    return launch_split(c, b, W, T, 0, nullptr, nullptr, nullptr, nullptr, 1, ck_in, one, st);
  if (tk == TAPED_BF16)
    return launch_bf16_quarter(c, b, W, T, 0, nullptr, nullptr, nullptr, nullptr, 1, ck_in, one,
                               st);
  return launch_tile(tk == TAPED_TILE2 ? 2 : 1, c, b, W, T, 0, nullptr, nullptr, nullptr, nullptr,
                     1, ck_in, one, st);
}

}  // namespace qs
