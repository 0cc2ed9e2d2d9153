// Fused multi-step kernel with the actor split over the four waves of a
// workgroup, for batches too small to give every SIMD a wave of the tile
// kernel (4096 envs make 256 one-tile waves for 1024 SIMDs).
//
// A workgroup advances one 16-env tile.  Each of its 4 waves holds it in the
// tile layout (qs_tile.h), so every env sits on 16 lanes.  Wave w evaluates
// unit tile w (16 units) of layers 1 and 2, a quarter of the matrix work, from
// weight fragments that it keeps in registers (84 of them: no staging of
// the actor in LDS and no weight reads in the loop); the layer-1 results are
// split into their bf16 parts by the wave that owns them and exchanged through LDS
// as layer-2 operands, the layer-2 results
// as fp32 tiles, with one barrier per layer (and one for the noise).  Every wave then evaluates layer
// 3 and the dynamics of the 16 envs: the same arithmetic on identical inputs,
// so the copies agree bit for bit, and the products are the tile kernel's in
// its order, so its results are the same too.  Wave 0 writes the outputs.
//
// What bounds it is the serial chain of a step: features, 6 dependent matrix
// products, exchange, 12 products, exchange, layer 3, tanh, four right-hand
// sides.  The history products of layer 1 (24 of its 30) are off the chain:
// they run beside the right-hand sides of the step before.  4096 envs: 2.25 us
// per step (3.15 us with fp32 products, the actor in LDS and every product on
// the chain; with noise 3.0).  One wave per SIMD with up to 512 registers; two waves of 256
// spill and take 2.67 us there, 3.96 us at 8192 envs against 3.38 us for the
// tile kernel.
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

// A wave's share of the actor: the fragments of unit tile w, its biases, and
// layer 3.
struct SplitActor {
  Frags<1> hist[4], state, l2[2];
  f4t b2, b3, w3[4];

  // false where a weight of the lane's share has no split
  __device__ inline bool load(const float* __restrict__ W, int w, int lane) {
    const int lg = lane >> 4;
    uint32_t third = 0;
    const auto get = [&](int g, u4t (&a)[T_P]) {
      load_fragment(W, g, lane, a);
      third |= (a[2][0] | a[2][1]) | (a[2][2] | a[2][3]);
    };
#pragma unroll
    for (int c = 0; c < 4; ++c) get(4 * w + c, hist[c].a[0]);
    get(T_GS + w, state.a[0]);
#pragma unroll
    for (int m = 0; m < 2; ++m) get(T_G2 + 2 * w + m, l2[m].a[0]);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      b2[r] = W[OFF_B2 + 16 * w + 4 * lg + r];
      b3[r] = lg == 0 ? W[OFF_B3 + r] : 0.0f;
#pragma unroll
      for (int n = 0; n < 4; ++n) w3[n][r] = W[OFF_W3 + (lane & 3) * NHID + 16 * n + 4 * lg + r];
    }
    bool ok = true;
    if (__builtin_expect(__ballot(maybe_unsplit(third)) != 0, 0)) {
      const u4t t[7] = {hist[0].a[0][2], hist[1].a[0][2], hist[2].a[0][2], hist[3].a[0][2],
                        state.a[0][2],   l2[0].a[0][2],   l2[1].a[0][2]};
#pragma unroll
      for (int i = 0; i < 7; ++i)
        ok = ok && !(unsplit(t[i][0]) || unsplit(t[i][1]) || unsplit(t[i][2]) || unsplit(t[i][3]));
    }
    return ok;
  }
  // layer 1's history sums of the wave's unit tile
  __device__ inline void history(const TileHist<1>& H, f4t (&a1)[1][1]) const {
    u4t x[4][1][T_P];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int s = 0; s < T_P; ++s) x[c][0][s] = H.h[0][s][c];
    split_sum<4, 1, 1>([&](int c) { return hist[c]; }, x, a1);
  }
};

// The rest of layer 1 (the state features and the bias; a1 holds the history
// sums), layers 2 and 3 of the workgroup's 16 envs: z3 of the lane's env
// in every lane of every wave.  When rec != NULL (the step's record), writes
// this wave's tile of the layer pre-activations (rows 16 w + 4 lg + r; zoff
// addresses row 4 lg of this lane's env) and its byte of the ReLU mask word
// (tile_mask; moff addresses the word), for lanes with on set.  lost: lanes that
// carry_nan whatever their features are, in the wave's tile.
__device__ inline void actor_split(const SplitActor& A, SplitXch& xc, f4t (&a1)[1][1],
                                   const float (&F)[5], uint64_t lost, float z3[NA],
                                   float* __restrict__ rec, bool on, uint32_t zoff, uint32_t moff,
                                   int w) {
  const int lane = threadIdx.x & 63;
  {
    u4t x[1][1][T_P];
    state_operand(F, x[0][0]);
    f4t as[1][1];
    split_sum<1, 1, 1>([&](int) { return A.state; }, x, as);
    a1[0][0] += as[0][0];
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
  uint64_t nan;
  f4t a2[1][1];
  {
    u4t x[2][1][T_P];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int s = 0; s < T_P; ++s) x[m][0][s] = xc.x1[s][m][lane];
    // (while the reads are on their way)
    __builtin_amdgcn_sched_barrier(0);
    nan = lost | nan_lanes(F);
    __builtin_amdgcn_sched_barrier(0);
    split_sum<2, 1, 1>([&](int m) { return A.l2[m]; }, x, a2);
    a2[0][0] += A.b2;
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
  carry_nan(a2[0][0], nan);
  xc.x2[w][lane] = a2[0][0];
  __syncthreads();
  f4t h2[4][1];
#pragma unroll
  for (int n = 0; n < 4; ++n) h2[n][0] = xc.x2[n][lane];
  tile_layer3<1>(A.w3, A.b3, h2, z3);
}

// T steps of the whole env step for 16 envs per workgroup (blockDim 256).
// A barrier separates each layer's writes of the exchange buffers from the
// reads, and the next step's writes of a buffer come after the barrier that
// follows every wave's reads of it, so two barriers per step suffice; with
// observation noise a third stands between its draws and their use.
// TAPE: as the tile kernel: with tape != NULL, checkpoints every ckpt_every
// steps; with ck_in != NULL the launch starts from that checkpoint (no
// write-back of the env state); with rs.buf[0] != NULL the record of the span
// rs.  Wave 0 writes everything except the layer pre-activations and the mask
// bytes, which each wave writes for its own tile.
template <bool EXTRAS, bool TAPE>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
k_split(DevCfg c, SimBufs b, const float* __restrict__ W, int T, int t_base,
        float* __restrict__ rewards, uint8_t* __restrict__ dones, float* __restrict__ states,
        float* __restrict__ tape, int ckpt_every, const float* __restrict__ ck_in,
        RecSpan rs) {
  __shared__ SplitXch xc;
  __shared__ float next_start[NRES * 256];
  __shared__ float2 normals[EXTRAS ? 5 : 1][64];
  const int N = c.n_envs;
  const int env0 = blockIdx.x * 16;
  const int lane = threadIdx.x & 63, j = lane & 15, k = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  SplitActor A;
  // (of the wave's share; its layer-2 tile tells the other waves)
  const bool bad_actor = __ballot(!A.load(W, w, lane)) != 0;
  const bool writer = w == 0;
  const int env = env0 + j;
  const bool active = env < N;
  const int e = active ? env : env0;
  // from a checkpoint (the backward's recompute): no write-back of the env
  // state; the steps of the span rs are recorded (rec_at)
  const bool REC = TAPE && ck_in != nullptr;

  float th[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) th[i] = b.theta[(size_t)i * N + e];
  Body<float> B = make_body<float>(th);
  const bool renorm = (c.flags & F_RENORM_Q) != 0;

  float x[NS];
  TileHist<1> H;
  int head0 = 0, t_ep = 0, ep = 0;
  EpAcc acc;
  if (REC) {
#pragma unroll
    for (int i = 0; i < NS; ++i) x[i] = ck_in[(size_t)i * N + e];
#pragma unroll
    for (int q = 0; q < 16; ++q)
      H.set_pair(0, q, ck_in[(size_t)(NS + 2 * q * NA + k) * N + e],
                 ck_in[(size_t)(NS + (2 * q + 1) * NA + k) * N + e]);
    t_ep = __float_as_int(ck_in[(size_t)CK_TEP * N + e]);
    ep = __float_as_int(ck_in[(size_t)CK_EP * N + e]);
    acc.cur = acc.last = 0.0f, acc.len = 0;
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
    acc.load(b, N, e);
  }
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
  // next episode's start state drawn ahead (long launches only), kept in LDS
  const bool ahead = T >= 2 * RESERVE_PERIOD && (c.flags & F_AUTORESET) != 0;
  float* nxp = next_start + threadIdx.x;
  const auto draw_next = [&]() {
    float nx[NRES];
    draw_ahead<0>(c, (uint32_t)e, (uint32_t)(ep + 1), wh, nx);
#pragma unroll
    for (int i = 0; i < NRES; ++i) nxp[i * 256] = nx[i];
  };
  bool have = ahead;
  if (ahead) draw_next();

  const uint32_t ok = 4u * (uint32_t)(k * N + e);  // byte offset of row k of the env
  if (states && t_base == 0 && active && writer) store_rows<4, NS>(states, N, ok, k, x);

  // The observation noise of a step is drawn by the four waves together at the end
  // of the step before (wave w pair w of every lane, the last wave pair 4 too) and
  // read after a barrier: drawn whole by every wave it took a quarter of a step (4096
  // envs with noise 3.53 us a step, now 3.21; without 2.40).
  const bool noisy = EXTRAS && (c.flags & F_OBS_NOISE) != 0;
  const auto draw_noise = [&]() {
    normals[EXTRAS ? w : 0][lane] = draw_normal_pair(c, (uint32_t)e, (uint32_t)ep, t_ep, k, w);
    if (w == 3)
      normals[EXTRAS ? 4 : 0][lane] = draw_normal_pair(c, (uint32_t)e, (uint32_t)ep, t_ep, k, 4);
  };
  if (noisy) draw_noise();

  f4t a1[1][1];  // layer 1's history sums of the coming step
  A.history(H, a1);
  // lanes that carry_nan in the first step
  uint64_t lost = nan_slots(a1[0][0], [&](int s) {
    if (REC) return ck_in[(size_t)(NS + s * NA + k) * N + e];
    return b.ring[(size_t)(((head0 + s) & (NH - 1)) * NA + k) * N + e];
  });
  if (bad_actor) lost = ~0ull;
  drain_loads();
  for (int t = 0; t < T; ++t) {
    const uint32_t so = opaque(ok);
    const int gt = t_base + t;
    RecAt ra;
    const bool rec_on = TAPE && rec_at(rs, gt, ra);  // wave uniform
    if (TAPE && tape && (gt % ckpt_every) == 0 && active && writer) {
      float* ck = tape + (size_t)(gt / ckpt_every) * CK_F * N;
      store_rows<4, NS>(ck, N, so, k, x);
#pragma unroll
      for (int s = 0; s < NH; ++s) at_byte(ck + (size_t)(NS + s * NA) * N, so) = H.get(0, s);
      if (k == 0) {
        at_byte(ck + (size_t)CK_TEP * N, so) = __int_as_float(t_ep);
        at_byte(ck + (size_t)CK_EP * N, so) = __int_as_float(ep);
      }
    }
    float F[1][5];
    if (noisy) __syncthreads();
    tile_features<1, EXTRAS>(c, sp, x, k, F, [&](float* zc, float* zs) {
#pragma unroll
      for (int q = 0; q < 5; ++q) {
        const float2 z = normals[EXTRAS ? q : 0][lane];
        zc[q] = z.x;
        zs[q] = z.y;
      }
    });
    float* rt = rec_on ? ra.base + rec_step(ra.step, N) : nullptr;
    const uint32_t zoff = TAPE ? opaque((uint32_t)(rb_at(env0 + j, REC_F) + 4 * k * RB)) : 0u;
    const uint32_t moff = TAPE ? opaque((uint32_t)(rb_at(env0 + j, REC_F) + k * RB)) : 0u;
    float z3[NA];
    actor_split(A, xc, a1, F[0], lost, z3, TAPE ? rt : nullptr, active, zoff, moff, w);
    lost = bad_actor ? ~0ull : 0ull;
    float a[NA], ak[1];
#pragma unroll
    for (int i = 0; i < NA; ++i) a[i] = tanh_act(z3[i]);
    to_tiles<1>(a, k, ak);
    if (TAPE && rec_on && active && writer) {
#pragma unroll
      for (int q = 0; q < 5; ++q)
        if (4 * q + k < 18) rt[(size_t)(REC_O + 4 * q) * RB + moff] = F[0][q];
      const int cap = opaque_uniform(rs.len);  // (not formed ahead of the loop)
      float* act = ra.base + rec_act(cap, N);
      const uint32_t aoff = opaque((uint32_t)(rb_at(e, (NH + cap) * NA) + k * RB));
      if (ra.step == 0) {
#pragma unroll
        for (int s = 0; s < NH; ++s) act[(size_t)(s * NA) * RB + aoff] = H.get(0, s);
      }
      act[(size_t)((NH + ra.step) * NA) * RB + aoff] = ak[0];
      rt[(size_t)REC_A * RB + moff] = ak[0];
      store_rows<4, NS>(rt + REC_X * RB, RB, 4u * moff, k, x);
    }
    // the action goes to the history ring in memory as it is applied (the
    // last 32 of a launch; the older ones would be overwritten)
    if (!REC && t >= T - NH && active && writer)
      b.ring[(size_t)(((head0 + t) & (NH - 1)) * NA) * N + (so >> 2)] = ak[0];
    uint32_t ap[1][T_P];
    split_pair(ak[0], 0.0f, ap[0]);
    H.push(ap);
    // beside the right-hand sides (no dependence between the two)
    A.history(H, a1);
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
      A.history(H, a1);
      if (rst) {
        ++ep;
        t_ep = 0;
        was_reset = true;
        if (have) {
#pragma unroll
          for (int i = 0; i < NRES; ++i) x[i] = nxp[i * 256];
#pragma unroll
          for (int i = NRES; i < NS; ++i) x[i] = wh;
          have = false;
        } else {
          reset_draw<0>(c, (uint32_t)e, (uint32_t)ep, wh, x);
        }
        if (EXTRAS) {
          float dd[6];
          disturbance(c, (uint32_t)e, (uint32_t)ep, dd);
          set_disturbance(B, dd);
        }
      }
    }
    if (ahead && (t & (RESERVE_PERIOD - 1)) == RESERVE_PERIOD - 1 && !have) {
      draw_next();
      have = true;
    }
    // (every wave has read this step's normals: two barriers ago)
    if (noisy && t + 1 < T) draw_noise();
    if (active && writer) {
      if (k == 0) {
        if (rewards) at_byte(rewards + (size_t)gt * N, so) = r;
        if (dones) at_byte(dones + (size_t)gt * N, so >> 2) = (uint8_t)d;
      }
      if (states) store_rows<4, NS>(states + (size_t)(gt + 1) * NS * N, N, so, k, x);
    }
  }
  if (!active || !writer || REC) return;
  store_rows<4, NS>(b.state, N, ok, k, x);
  const int head1 = (head0 + T) & (NH - 1);
  // after a reset in this launch the slots older than the episode's t_ep
  // actions hold the hover action
  if (was_reset)
#pragma unroll 1
    for (int s = 0; s < NH - t_ep; ++s)
      b.ring[(size_t)(((head1 + s) & (NH - 1)) * NA) * N + (ok >> 2)] = ah;
  if (k == 0) {
    b.head[e] = head1;
    b.t_ep[e] = t_ep;
    b.ep[e] = ep;
    acc.store(b, N, e);
  }
}

hipError_t launch_split(const DevCfg& c, const SimBufs& b, const float* W, int T, int t_base,
                        float* rewards, uint8_t* dones, float* states, float* tape,
                        int ckpt_every, const float* ck_in, const RecSpan& rs, hipStream_t st) {
  if (!rec_span_ok(rs)) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)((c.n_envs + 15) / 16);
  const bool ex = (c.flags & (F_DISTURB | F_OBS_NOISE)) != 0 || c.target != nullptr;
  const bool tp = tape || ck_in || rs.buf[0];
  auto k = ex ? (tp ? k_split<true, true> : k_split<true, false>)
              : (tp ? k_split<false, true> : k_split<false, false>);
  hipLaunchKernelGGL(k, dim3(grid), dim3(256), 0, st, c, b, W, T, t_base, rewards, dones, states,
                     tape, ckpt_every, ck_in, rs);
  return hipGetLastError();
}

}  // namespace qs
