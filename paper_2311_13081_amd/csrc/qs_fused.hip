// Fused multi-step kernel of the batched quadrotor step with one env per
// lane: observation, actor (vector ALUs; the bf16 option on bf16 matrix
// cores), action map, RK4, reward, history push, termination and reset for T
// steps in one launch.
//
// Layout: struct-of-arrays in HBM ([K][N]) so every global access of a wave is
// a contiguous 256-byte segment; actor weights are staged in LDS once per
// workgroup.
#include "qs_actor.h"
#include "qs_forward.h"

namespace qs {
// ---------------------------------------------------------------------------
// Fused multi-step kernel
// ---------------------------------------------------------------------------

// T steps of the whole step (observation, actor, action map, RK4, reward,
// history push, termination, truncation, reset, episode accumulators) with
// state and history kept in registers.  Outputs indexed by t_base + t.
// Inactive lanes of the last wave shadow the wave's first env (read only) so
// every MFMA operand is finite.  EXTRAS (the training extras or a set point are
// on): the episode disturbance enters the dynamics and the actor sees its
// observation with noise and the set-point shift; without them the kernel
// carries none of that code.  The loop issues no vector-memory load: loads and
// stores share one completion counter, so a wait for a load issued in the loop
// would also wait for every output store issued before it.
enum FusedActor { ACT_VALU, ACT_BF16 };

template <bool EXTRAS, FusedActor ACT>
__global__ void __launch_bounds__(256)
k_fused(DevCfg c, SimBufs b, const float* __restrict__ W, int T, int t_base,
        float* __restrict__ rewards, uint8_t* __restrict__ dones, float* __restrict__ states) {
  __shared__ __attribute__((aligned(16))) float lds[ACT == ACT_VALU ? V_TOTAL : MB_TOTAL];
  const int N = c.n_envs;
  constexpr int DRAW = ACT == ACT_BF16 ? 1 : 0;
  if constexpr (ACT == ACT_VALU) stage_actor(W, lds);
  if constexpr (ACT == ACT_BF16) stage_actor_bf16(W, lds);
  __syncthreads();
  const int env = blockIdx.x * blockDim.x + threadIdx.x;
  const int first = env - (threadIdx.x & 63);
  if (first >= N) return;  // whole wave past the end
  const bool active = env < N;
  const int e = active ? env : first;

  float th[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) th[i] = b.theta[i * N + e];
  Body<float> B = make_body<float>(th);
  const bool renorm = (c.flags & F_RENORM_Q) != 0;

  float x[NS];
  float H[NH * NA];
  EpAcc acc;
#pragma unroll
  for (int i = 0; i < NS; ++i) x[i] = b.state[i * N + e];
  const int head0 = b.head[e];
#pragma unroll
  for (int sl = 0; sl < NH; ++sl) {
    const int slot = (head0 + sl) & (NH - 1);
#pragma unroll
    for (int a = 0; a < NA; ++a) H[sl * NA + a] = b.ring[(slot * NA + a) * N + e];
  }
  int t_ep = b.t_ep[e], ep = b.ep[e];
  acc.load(b, N, e);
  SetPoint sp;
  if (EXTRAS) sp.load(c, N, e);
  if (EXTRAS) {
    float d[6];
    disturbance(c, (uint32_t)e, (uint32_t)ep, d);
    set_disturbance(B, d);
  }
  bool was_reset = false;
  const float wh = hover_rpm(c, th[0], th[4], th[5], th[6]);
  const float ah = rpm_to_action(c, wh);
  // next episode's start state drawn ahead (long launches only)
  const bool ahead = T >= 2 * RESERVE_PERIOD;
  float nx[NRES];
  bool have = ahead;
  if (ahead) draw_ahead<DRAW>(c, (uint32_t)e, (uint32_t)(ep + 1), wh, nx);

  if (states && t_base == 0 && active)
#pragma unroll
    for (int i = 0; i < NS; ++i) states[i * N + e] = x[i];

  for (int t = 0; t < T; ++t) {
    // Keeps the weight reads inside the step: hoisting them out of the time
    // loop would pin thousands of loop-invariant values in registers.
    __asm__ volatile("" ::: "memory");
    const uint32_t eo = opaque((uint32_t)e);
    const int gt = t_base + t;
    float a[NA];
    {
      float Rm[9];
      rotmat(x + 3, Rm);
      float z3[NA];
      // the observed state features (the set-point shift and the noise
      // under EXTRAS)
      float so[NS];
#pragma unroll
      for (int i = 0; i < NS; ++i) so[i] = x[i];
      if constexpr (EXTRAS) {
        if ((c.flags & F_OBS_NOISE) || c.target) {
          float f[18] = {x[0],  x[1],  x[2],  Rm[0], Rm[1], Rm[2], Rm[3], Rm[4],  Rm[5],
                         Rm[6], Rm[7], Rm[8], x[7],  x[8],  x[9],  x[10], x[11], x[12]};
          sp.apply(c, f);
          add_obs_noise<DRAW>(c, (uint32_t)e, (uint32_t)ep, t_ep, f);
#pragma unroll
          for (int i = 0; i < 3; ++i) {
            so[i] = f[i];
            so[7 + i] = f[12 + i];
            so[10 + i] = f[15 + i];
          }
#pragma unroll
          for (int i = 0; i < 9; ++i) Rm[i] = f[3 + i];
        }
      }
      if constexpr (ACT == ACT_BF16)
        actor_mfma_bf16(lds, so, Rm, H, z3);
      else
        actor_valu(lds, so, Rm, H, z3);
#pragma unroll
      for (int i = 0; i < NA; ++i) a[i] = tanh_act(z3[i]);
    }
    float u[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) u[i] = action_to_rpm(c, a[i]);
    rk4_step<float, EXTRAS>(B, c.arm, c.km, c.g, c.dt, renorm, x, u);
    const float r = reward(c, x, a);
    ++t_ep;
    const uint32_t d = episode_end(c, x, t_ep);
    const bool rst = d && (c.flags & F_AUTORESET);
    acc.add(r, rst, t_ep);
    // history push and the reset fill in one pass: one select per slot
#pragma unroll
    for (int i = 0; i < (NH - 1) * NA; ++i) H[i] = rst ? ah : H[i + NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) H[(NH - 1) * NA + i] = rst ? ah : a[i];
    if (rst) {
      ++ep;
      t_ep = 0;
      was_reset = true;
      reset_from_reserve<DRAW>(c, (uint32_t)e, (uint32_t)ep, wh, nx, have, x);
      if (EXTRAS) {
        float dd[6];
        disturbance(c, (uint32_t)e, (uint32_t)ep, dd);
        set_disturbance(B, dd);
      }
    }
    if (ahead && (t & (RESERVE_PERIOD - 1)) == RESERVE_PERIOD - 1 && !have) {
      draw_ahead<DRAW>(c, (uint32_t)e, (uint32_t)(ep + 1), wh, nx);
      have = true;
    }
    if (active) {
      if (rewards) rewards[(size_t)gt * N + eo] = r;
      if (dones) dones[(size_t)gt * N + eo] = (uint8_t)d;
      if (states)
#pragma unroll
        for (int i = 0; i < NS; ++i) states[((size_t)(gt + 1) * NS + i) * N + eo] = x[i];
    }
  }
  if (!active) return;
  const uint32_t ef = opaque((uint32_t)e);
#pragma unroll
  for (int i = 0; i < NS; ++i) b.state[(size_t)i * N + ef] = x[i];
  // The ring keeps slots older than this launch in place; only the T newest
  // logical slots (all 32 after a reset) are written.
  const int head1 = (head0 + T) & (NH - 1);
#pragma unroll
  for (int sl = 0; sl < NH; ++sl) {
    if (was_reset || sl >= NH - T) {
      const int slot = (head1 + sl) & (NH - 1);
#pragma unroll
      for (int a = 0; a < NA; ++a) b.ring[(size_t)(slot * NA + a) * N + ef] = H[sl * NA + a];
    }
  }
  b.head[ef] = head1;
  b.t_ep[ef] = t_ep;
  b.ep[ef] = ep;
  acc.store(b, N, ef);
}

static inline unsigned nblk(int n, int bs) { return (unsigned)((n + bs - 1) / bs); }

hipError_t launch_fused(const DevCfg& c, const SimBufs& b, const float* W, int T, int t_base,
                        float* rewards, uint8_t* dones, float* states, hipStream_t st) {
  const dim3 g(nblk(c.n_envs, 256)), blk(256);
  const bool ex = (c.flags & (F_DISTURB | F_OBS_NOISE)) != 0 || c.target != nullptr;
  const bool bf = (c.flags & F_ACTOR_BF16) != 0;
  auto k = bf ? (ex ? k_fused<true, ACT_BF16> : k_fused<false, ACT_BF16>)
              : (ex ? k_fused<true, ACT_VALU> : k_fused<false, ACT_VALU>);
  hipLaunchKernelGGL(k, g, blk, 0, st, c, b, W, T, t_base, rewards, dones, states);
  return hipGetLastError();
}

}  // namespace qs
