// Fused multi-step kernel with the actor split over the four waves of a
// workgroup, for batches too small to give every SIMD a wave of the tile
// kernel (4096 envs make 256 one-tile waves for 1024 SIMDs).
//
// A workgroup advances one 16-env tile.  Each of its 4 waves holds it in the
// tile layout (qs_tile.h), so every env sits on 16 lanes.  Wave w evaluates
// unit tile w (16 units) of layers 1 and 2, a quarter of the matrix work; the
// layer-1 results are split into their bf16 parts by the wave that owns them
// and exchanged through LDS as layer-2 operands, the layer-2 results as fp32
// tiles, with one barrier per layer.  Every wave then evaluates layer 3 and
// the dynamics of the 16 envs: the same arithmetic on identical inputs, so
// the copies agree bit for bit, and the products are the tile kernel's in its
// order, so its results are the same too.  Wave 0 writes the outputs.
// Fused multiply-adds only where one expression of the source holds the
// product and the sum: the kernels that promise equal results then round the
// shared arithmetic the same way (left to the optimiser, fusing depends on what
// surrounds the inlined code).
#pragma clang fp contract(on)
#include "qs_forward.h"
#include "qs_tile.h"

namespace qs {

// Exchange buffers: layer-2 operands [part][chunk][lane] (a tile fills half of
// each lane's 16 bytes), layer-2 result tiles [tile][lane].
struct SplitXch {
  u4t x1[3][2][64];
  f4t x2[4][64];
};

// Layers 1 to 3 of the workgroup's 16 envs: z3 of the lane's env in every lane
// of every wave.  When rec != NULL (the step's record), writes this wave's
// tile of the layer pre-activations (rows 16 w + 4 lg + r; zoff addresses row
// 4 lg of this lane's env) and its byte of the ReLU mask word (tile_mask; moff
// addresses the word), for lanes with on set.
__device__ inline void actor_split(const float* lds, SplitXch& xc, const TileHist<1>& H,
                                   const float F[5], float z3[NA], float* __restrict__ rec,
                                   bool on, uint32_t zoff, uint32_t moff) {
  const int lane = threadIdx.x & 63, lg = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const u4t* frag = reinterpret_cast<const u4t*>(lds);
  f4t a1[1][1], a2[1][1];
  a1[0][0] = *reinterpret_cast<const f4t*>(&lds[T_B1 + 16 * w + 4 * lg]);
  a2[0][0] = *reinterpret_cast<const f4t*>(&lds[T_B2 + 16 * w + 4 * lg]);
#pragma unroll
  for (int c = 0; c < 5; ++c) {
    u4t x[1][3];
    if (c < 4) {
#pragma unroll
      for (int s = 0; s < 3; ++s) x[0][s] = H.h[0][s][c];
    } else {
      state_operand(F, x[0]);
    }
    Frags<1> f;
    f.load(frag, 4 * c + w, lane);
    tile_products<1, 1>(f, x, a1);
  }
  uint32_t mask = 0u;
  if (rec) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (on) rec[(size_t)(REC_Z1 + 16 * w + r) * RB + zoff] = a1[0][0][r];
      mask |= (a1[0][0][r] > 0.0f ? 1u : 0u) << r;
    }
  }
  relu_tiles(a1);
  {
    uint32_t p[3], q[3];
    split_pair(a1[0][0][0], a1[0][0][1], p);
    split_pair(a1[0][0][2], a1[0][0][3], q);
#pragma unroll
    for (int s = 0; s < 3; ++s)
      *(reinterpret_cast<uint2*>(&xc.x1[s][w >> 1][lane]) + (w & 1)) = uint2{p[s], q[s]};
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    u4t x[1][3];
#pragma unroll
    for (int s = 0; s < 3; ++s) x[0][s] = xc.x1[s][m][lane];
    Frags<1> f;
    f.load(frag, T_G1 + 4 * m + w, lane);
    tile_products<1, 1>(f, x, a2);
  }
  if (rec) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (on) rec[(size_t)(REC_Z2 + 16 * w + r) * RB + zoff] = a2[0][0][r];
      mask |= (a2[0][0][r] > 0.0f ? 1u : 0u) << (4 + r);
    }
    if (on) reinterpret_cast<uint8_t*>(rec + (size_t)REC_M * RB + moff)[w] = (uint8_t)mask;
  }
  relu_tiles(a2);
  xc.x2[w][lane] = a2[0][0];
  __syncthreads();
  f4t h2[4][1];
#pragma unroll
  for (int n = 0; n < 4; ++n) h2[n][0] = xc.x2[n][lane];
  tile_layer3<1>(lds + T_W3, lds + T_B3, h2, z3);
}

// T steps of the whole env step for 16 envs per workgroup (blockDim 256).
// A barrier separates each layer's writes of the exchange buffers from the
// reads, and the next step's writes of a buffer come after the barrier that
// follows every wave's reads of it, so two barriers per step suffice.
// As the tile kernel: with tape != NULL, checkpoints every ckpt_every steps;
// with ck_in != NULL the launch starts from that checkpoint (no write-back of
// the env state); with rs.buf[0] != NULL the record of the span rs.  Wave 0
// writes everything except the layer pre-activations and the mask bytes,
// which each wave writes for its own tile.
template <bool EXTRAS>
__global__ void __launch_bounds__(256)
k_split(DevCfg c, SimBufs b, const float* __restrict__ W, int T, int t_base,
        float* __restrict__ rewards, uint8_t* __restrict__ dones, float* __restrict__ states,
        float* __restrict__ tape, int ckpt_every, const float* __restrict__ ck_in,
        RecSpan rs) {
  __shared__ __attribute__((aligned(16))) float lds[T_TOTAL];
  __shared__ SplitXch xc;
  const int N = c.n_envs;
  const int env0 = blockIdx.x * 16;
  if (env0 >= N) return;  // the whole workgroup (no barrier is reached)
  stage_tile(W, lds);
  __syncthreads();
  const int lane = threadIdx.x & 63, j = lane & 15, k = lane >> 4;
  const bool writer = threadIdx.x < 64;  // wave 0
  const int env = env0 + j;
  const bool active = env < N;
  const int e = active ? env : env0;
  // from a checkpoint (the backward's recompute): no write-back of the env
  // state; the steps of the span rs are recorded (rec_at)
  const bool REC = ck_in != nullptr;

  float th[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) th[i] = b.theta[(size_t)i * N + e];
  Body<float> B = make_body<float>(th);
  const bool renorm = (c.flags & F_RENORM_Q) != 0;

  float x[NS];
  TileHist<1> H;
  int head0 = 0, t_ep = 0, ep = 0;
  if (REC) {
#pragma unroll
    for (int i = 0; i < NS; ++i) x[i] = ck_in[(size_t)i * N + e];
#pragma unroll
    for (int q = 0; q < 16; ++q)
      H.set_pair(0, q, ck_in[(size_t)(NS + 2 * q * NA + k) * N + e],
                 ck_in[(size_t)(NS + (2 * q + 1) * NA + k) * N + e]);
    t_ep = __float_as_int(ck_in[(size_t)CK_TEP * N + e]);
    ep = __float_as_int(ck_in[(size_t)CK_EP * N + e]);
  } else {
#pragma unroll
    for (int i = 0; i < NS; ++i) x[i] = b.state[(size_t)i * N + e];
    head0 = b.head[e];
    float v[NH];
#pragma unroll
    for (int s = 0; s < NH; ++s)
      v[s] = b.ring[(size_t)(((head0 + s) & (NH - 1)) * NA + k) * N + e];
#pragma unroll
    for (int q = 0; q < 16; ++q) H.set_pair(0, q, v[2 * q], v[2 * q + 1]);
    t_ep = b.t_ep[e];
    ep = b.ep[e];
  }
  // episode accumulators: the recompute from a checkpoint leaves them alone
  EpAcc acc;
  if (REC)
    acc.cur = acc.last = 0.0f, acc.len = 0;
  else
    acc.load(b, N, e);
  SetPoint sp;
  if (EXTRAS) sp.load(c, N, e);
  bool was_reset = false;
  const float wh = hover_rpm(c, th[0], th[4], th[5], th[6]);
  const float ah = rpm_to_action(c, wh);
  if (EXTRAS) {
    float d[6];
    disturbance(c, (uint32_t)e, (uint32_t)ep, d);
    set_disturbance(B, d);
  }
  // next episode's start state drawn ahead (long launches only)
  const bool ahead = T >= 2 * RESERVE_PERIOD && (c.flags & F_AUTORESET) != 0;
  float nx[NRES];
  bool have = ahead;
  if (ahead) draw_ahead<0>(c, (uint32_t)e, (uint32_t)(ep + 1), wh, nx);

  if (states && t_base == 0 && active && writer)
#pragma unroll
    for (int i = 0; i < NS; ++i)
      if ((i & 3) == k) states[(size_t)i * N + e] = x[i];

  for (int t = 0; t < T; ++t) {
    __asm__ volatile("" ::: "memory");
    const uint32_t eo = opaque((uint32_t)e);
    const int gt = t_base + t;
    RecAt ra;
    const bool rec_on = rec_at(rs, gt, ra);  // wave uniform
    const int rt_step = ra.step;
    if (tape && (gt % ckpt_every) == 0 && active && writer) {
      float* ck = tape + (size_t)(gt / ckpt_every) * CK_F * N;
#pragma unroll
      for (int i = 0; i < NS; ++i)
        if ((i & 3) == k) ck[(size_t)i * N + eo] = x[i];
      const uint32_t kc = opaque((uint32_t)(k * N + e));
#pragma unroll
      for (int s = 0; s < NH; ++s) ck[(size_t)(NS + s * NA) * N + kc] = H.get(0, s);
      if (k == 0) {
        ck[(size_t)CK_TEP * N + eo] = __int_as_float(t_ep);
        ck[(size_t)CK_EP * N + eo] = __int_as_float(ep);
      }
    }
    float F[1][5];
    tile_features<1, EXTRAS>(c, sp, (uint32_t)e, (uint32_t)ep, t_ep, x, k, F);
    float* rt = rec_on ? ra.base + rec_step(rt_step, N) : nullptr;
    const uint32_t zoff = opaque((uint32_t)(rb_at(env0 + j, REC_F) + 4 * k * RB));
    const uint32_t moff = opaque((uint32_t)(rb_at(env0 + j, REC_F) + k * RB));
    float z3[NA];
    actor_split(lds, xc, H, F[0], z3, rt, active, zoff, moff);
    float a[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) a[i] = tanh_act(z3[i]);
    float ak[1];
    to_tiles<1>(a, k, ak);
    if (rec_on && active && writer) {
      const uint32_t koff = opaque((uint32_t)(rb_at(e, REC_F) + k * RB));
      const uint32_t roff = opaque((uint32_t)rb_at(e, REC_F));
#pragma unroll
      for (int cc = 0; cc < 5; ++cc)
        if (4 * cc + k < 18) rt[(size_t)(REC_O + 4 * cc) * RB + koff] = F[0][cc];
      float* act = ra.base + rec_act(ra.n, N);
      const uint32_t aoff = opaque((uint32_t)(rb_at(e, (NH + ra.n) * NA) + k * RB));
      if (rt_step == 0) {
#pragma unroll
        for (int s = 0; s < NH; ++s) act[(size_t)(s * NA) * RB + aoff] = H.get(0, s);
      }
      act[(size_t)((NH + rt_step) * NA) * RB + aoff] = ak[0];
#pragma unroll
      for (int i = 0; i < NS; ++i)
        if ((i & 3) == k) rt[(size_t)(REC_X + i) * RB + roff] = x[i];
      rt[(size_t)REC_A * RB + koff] = ak[0];
    }
    // the action goes to the history ring in memory as it is applied (the
    // last 32 of a launch; the older ones would be overwritten)
    if (!REC && t >= T - NH && active && writer)
      b.ring[(size_t)(((head0 + t) & (NH - 1)) * NA + k) * N + eo] = ak[0];
    uint32_t ap[1][T_P];
    split_pair(ak[0], 0.0f, ap[0]);
#pragma unroll
    for (int c4 = 0; c4 < 4; ++c4) H.push_chunk(c4, ap);
    float u[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) u[i] = action_to_rpm(c, a[i]);
    rk4_step<float, EXTRAS>(B, c.arm, c.km, c.g, c.dt, renorm, x, u);
    const float r = reward(c, x, a);
    ++t_ep;
    const uint32_t d = episode_end(c, x, t_ep);
    const bool rst = d && (c.flags & F_AUTORESET);
    acc.add(r, rst, t_ep);
    if (__ballot(rst)) {  // wave uniform
      const float ahk[1] = {ah};
      H.fill(&rst, ahk);
      if (rst) {
        ++ep;
        t_ep = 0;
        was_reset = true;
        reset_from_reserve<0>(c, (uint32_t)e, (uint32_t)ep, wh, nx, have, x);
        if (EXTRAS) {
          float dd[6];
          disturbance(c, (uint32_t)e, (uint32_t)ep, dd);
          set_disturbance(B, dd);
        }
      }
    }
    if (ahead && (t & (RESERVE_PERIOD - 1)) == RESERVE_PERIOD - 1 && !have) {
      draw_ahead<0>(c, (uint32_t)e, (uint32_t)(ep + 1), wh, nx);
      have = true;
    }
    if (active && writer) {
      if (k == 0 && rewards) rewards[(size_t)gt * N + eo] = r;
      if (k == 1 && dones) dones[(size_t)gt * N + eo] = (uint8_t)d;
      if (states)
#pragma unroll
        for (int i = 0; i < NS; ++i)
          if ((i & 3) == k) states[((size_t)(gt + 1) * NS + i) * N + eo] = x[i];
    }
  }
  if (!active || !writer || REC) return;
  const uint32_t ef = opaque((uint32_t)e);
#pragma unroll
  for (int i = 0; i < NS; ++i)
    if ((i & 3) == k) b.state[(size_t)i * N + ef] = x[i];
  const int head1 = (head0 + T) & (NH - 1);
  // after a reset in this launch the slots older than the episode's t_ep
  // actions hold the hover action
  if (was_reset)
#pragma unroll 1
    for (int s = 0; s < NH - t_ep; ++s)
      b.ring[(size_t)(((head1 + s) & (NH - 1)) * NA + k) * N + ef] = ah;
  if (k == 0) {
    b.head[ef] = head1;
    b.t_ep[ef] = t_ep;
    b.ep[ef] = ep;
    acc.store(b, N, ef);
  }
}

hipError_t launch_split(const DevCfg& c, const SimBufs& b, const float* W, int T, int t_base,
                        float* rewards, uint8_t* dones, float* states, float* tape,
                        int ckpt_every, const float* ck_in, const RecSpan& rs, hipStream_t st) {
  if (!rec_span_ok(rs)) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)((c.n_envs + 15) / 16);
  const bool ex = (c.flags & (F_DISTURB | F_OBS_NOISE)) != 0 || c.target != nullptr;
  auto k = ex ? k_split<true> : k_split<false>;
  hipLaunchKernelGGL(k, dim3(grid), dim3(256), 0, st, c, b, W, T, t_base, rewards, dones, states,
                     tape, ckpt_every, ck_in, rs);
  return hipGetLastError();
}

}  // namespace qs
