// Fused multi-step kernel with the actor on bf16 matrix cores (fp32 products
// by splitting, qs_tile.h): each wave advances 16 or 32 envs (one or two
// 16-env tiles) for T steps of observation, actor, action map, RK4, reward,
// history push, termination and reset in one launch, state and history in
// registers.
//
// The dynamics of an env run replicated on its 4 / TILES lanes (identical
// inputs and arithmetic, identical results); memory writes are split among
// them.
// Fused multiply-adds only where one expression of the source holds the
// product and the sum: the kernels that promise equal results then round the
// shared arithmetic the same way (left to the optimiser, fusing depends on what
// surrounds the inlined code).
#pragma clang fp contract(on)
#include "qs_forward.h"
#include "qs_tile.h"

namespace qs {

// The record of a step (the backward's): rows through a buffer view of the
// segment's record, s[b] the byte offset of tile b's envs in the step and z the
// lane's of row 4 lg of its env there, so that an address costs no vector
// instruction.  Envs past the batch record their shadow into the padding of the
// last block.
template <int TILES>
struct StepRec {
  static constexpr bool KEEPS_FEATURES = true;
  __amdgpu_buffer_rsrc_t buf;
  bool on;  // wave uniform
  uint32_t s[TILES], z, mask[TILES];
  template <int ROW, int SHIFT>
  __device__ inline void rows(const f4t (&v)[4][TILES]) {
    if (!on) return;
#pragma unroll
    for (int b = 0; b < TILES; ++b) {
#pragma unroll
      for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          bst1(v[n][b][r], buf, z, s[b] + 4u * (ROW + 16 * n + r) * RB);
      mask[b] = opaque(mask[b] | tile_mask<TILES>(v, b) << SHIFT);
    }
  }
  __device__ inline void layer1(const f4t (&v)[4][TILES]) { rows<REC_Z1, 0>(v); }
  __device__ inline void layer2(const f4t (&v)[4][TILES]) { rows<REC_Z2, 4>(v); }
};

constexpr int T_MAX_THREADS = 512;

// Values of a lane that a step needs once, in columns of LDS (one per lane)
// instead of the registers of the actor: the body, the episode accumulators, the
// hover speed and each tile's hover action, and the next start state.  Left to
// the compiler they are spilled to memory, and reading a spill back waits for
// every store issued before it: recorded steps of 65536 envs took 19.1 us with 85
// spills (and 1.1 GB written for 0.64 GB of record per 16 steps), now 12.  Spills
// that are left, by the compiler's count: 9 (two tiles), 20 (with the record), 32 and
// 48 (one, two tiles with the extras), 30 and 59 (with both); without the extras
// those in the loop lie around draws and resets, with them a step stores 16 to 27
// and reads as many back around the noise.
enum { PK_NEXT = 0, PK_ACC = NRES, PK_HOVER = PK_ACC + 3, PK_AH = PK_HOVER + 1, PK_BODY = PK_AH + 2 };
constexpr int PK_F = PK_BODY + sizeof(Body<float>) / 4;
struct Park {
  float* p;
  __device__ inline float& operator[](int i) const { return p[i * T_MAX_THREADS]; }
  // the members a body has without (11) or with the episode disturbance
  template <bool DIST>
  __device__ inline Body<float> body() const {
    struct { float v[PK_F - PK_BODY]; } f = {};
#pragma unroll
    for (int i = 0; i < (DIST ? PK_F - PK_BODY : 11); ++i) f.v[i] = (*this)[PK_BODY + i];
    return __builtin_bit_cast(Body<float>, f);
  }
  __device__ inline void put(const Body<float>& b) const {
    struct F { float v[PK_F - PK_BODY]; };
    const F f = __builtin_bit_cast(F, b);
#pragma unroll
    for (int i = 0; i < PK_F - PK_BODY; ++i) (*this)[PK_BODY + i] = f.v[i];
  }
  __device__ inline EpAcc acc() const {
    return {(*this)[PK_ACC], (*this)[PK_ACC + 1], __float_as_int((*this)[PK_ACC + 2])};
  }
  __device__ inline void put(const EpAcc& a) const {
    (*this)[PK_ACC] = a.cur;
    (*this)[PK_ACC + 1] = a.last;
    (*this)[PK_ACC + 2] = __int_as_float(a.len);
  }
};

// T steps; outputs indexed by t_base + t.  Lanes of envs past the batch
// shadow the wave's first env (loads only) so every operand is finite.
// EXTRAS: the training extras or a set point are on.  TAPE: the modes of
// differentiable rollouts: with tape != NULL a CK_F-row checkpoint every
// ckpt_every steps; with ck_in != NULL the launch starts from that checkpoint
// and leaves the env state alone (the backward's recompute); with rs.buf[0] !=
// NULL it writes the backward's record of the span rs.
//
// Two waves per SIMD (256 registers each): the matrix products of one wave
// overlap the vector instructions of the other.
template <int TILES, bool EXTRAS, bool TAPE>
__global__ void __launch_bounds__(T_MAX_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_tile(DevCfg c, SimBufs b, const float* __restrict__ W, int T, int t_base,
       float* __restrict__ rewards, uint8_t* __restrict__ dones, float* __restrict__ states,
       float* __restrict__ tape, int ckpt_every, const float* __restrict__ ck_in, RecSpan rs) {
  constexpr int SUB = 4 / TILES;  // lanes per env
  __shared__ __attribute__((aligned(16))) float lds[T_TOTAL + PK_F * T_MAX_THREADS];
  static_assert((T_TOTAL + PK_F * T_MAX_THREADS + T_MAX_THREADS / 64) * 4 <= 160 * 1024,
                "weights and columns fit in LDS");
  __shared__ uint32_t flags[T_MAX_THREADS / 64];
  const int N = c.n_envs;
  const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  set_flag(!stage_tile(W, lds), flags);
  __syncthreads();
  const int wave = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  const int env0 = __builtin_amdgcn_readfirstlane(wave * 16 * TILES);
  if (env0 >= N) return;
  // own env (dynamics): tile lg % TILES, this lane the sub-th of its SUB
  const int sub = lg / TILES;
  const int env = env0 + 16 * (lg % TILES) + li;
  const bool active = env < N;
  const int e = active ? env : env0;
  int et[TILES];  // the lane's env in each tile
#pragma unroll
  for (int t = 0; t < TILES; ++t) et[t] = env0 + 16 * t + li < N ? env0 + 16 * t + li : env0;
  const bool REC = TAPE && ck_in != nullptr;

  float th[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) th[i] = b.theta[(size_t)i * N + e];
  const Park park{lds + T_TOTAL + threadIdx.x};
  const bool renorm = (c.flags & F_RENORM_Q) != 0;

  float x[NS];
  TileHist<TILES> H;
  int head0 = 0, t_ep = 0, ep = 0;
  if (REC) {
#pragma unroll
    for (int i = 0; i < NS; ++i) x[i] = ck_in[(size_t)i * N + e];
#pragma unroll
    for (int t = 0; t < TILES; ++t)
#pragma unroll
      for (int q = 0; q < 16; ++q)
        H.set_pair(t, q, ck_in[(size_t)(NS + 2 * q * NA + lg) * N + et[t]],
                   ck_in[(size_t)(NS + (2 * q + 1) * NA + lg) * N + et[t]]);
    t_ep = __float_as_int(ck_in[(size_t)CK_TEP * N + e]);
    ep = __float_as_int(ck_in[(size_t)CK_EP * N + e]);
    park.put(EpAcc{0.0f, 0.0f, 0});
  } else {
#pragma unroll
    for (int i = 0; i < NS; ++i) x[i] = b.state[(size_t)i * N + e];
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
      const int hd = b.head[et[t]];
      float v[NH];
#pragma unroll
      for (int s = 0; s < NH; ++s)
        v[s] = b.ring[(size_t)(((hd + s) & (NH - 1)) * NA + lg) * N + et[t]];
#pragma unroll
      for (int q = 0; q < 16; ++q) H.set_pair(t, q, v[2 * q], v[2 * q + 1]);
    }
    head0 = b.head[e];
    t_ep = b.t_ep[e];
    ep = b.ep[e];
    EpAcc acc;
    acc.load(b, N, e);
    park.put(acc);
  }
  SetPoint sp;
  if (EXTRAS) sp.load(c, N, e);
  bool was_reset = false;
  {
    const float wh = hover_rpm(c, th[0], th[4], th[5], th[6]), ah = rpm_to_action(c, wh);
    const float v[4] = {ah, ah, ah, ah};
    float aht[TILES];
    to_tiles<TILES>(v, lg, aht);
    park[PK_HOVER] = wh;
#pragma unroll
    for (int t = 0; t < TILES; ++t) park[PK_AH + t] = aht[t];
    Body<float> B = make_body<float>(th);
    if (EXTRAS) {
      float d[6];
      disturbance(c, (uint32_t)e, (uint32_t)ep, d);
      set_disturbance(B, d);
    }
    park.put(B);
  }
  // next episode's start state drawn ahead (long launches only)
  const bool ahead = T >= 2 * RESERVE_PERIOD && (c.flags & F_AUTORESET) != 0;
  const auto draw_next = [&]() {
    float nx[NRES];
    draw_ahead<0>(c, (uint32_t)e, (uint32_t)(ep + 1), park[PK_HOVER], nx);
#pragma unroll
    for (int i = 0; i < NRES; ++i) park[PK_NEXT + i] = nx[i];
  };
  bool have = ahead;
  if (ahead) draw_next();

  const uint32_t osub = 4u * (uint32_t)(sub * N + e);  // row sub of the env
  if (states && t_base == 0 && active) store_rows<SUB, NS>(states, N, osub, sub, x);

  f4t a1[4][TILES];  // layer 1's history sums of the coming step
  FragPipe<TILES> fp;
  const auto history = [&]() {
    fp.start(lds);
#pragma unroll
    for (int n = 0; n < 4; n += T_NN<TILES>) tile_history<TILES>(fp, H, n, a1);
  };
  history();
  const bool bad_actor = any_flag(flags);
  uint64_t lost[TILES];  // lanes that carry_nan in the first step
#pragma unroll
  for (int t = 0; t < TILES; ++t) {
    const uint64_t m = nan_slots(a1[0][t], [&](int s) {
      if (REC) return ck_in[(size_t)(NS + s * NA + lg) * N + et[t]];
      return b.ring[(size_t)(((b.head[et[t]] + s) & (NH - 1)) * NA + lg) * N + et[t]];
    });
    lost[t] = bad_actor ? ~0ull : m;
  }
  drain_loads();
  for (int t = 0; t < T; ++t) {
    // keeps the weight reads inside the step (hoisted out of the time loop
    // they would pin the registers)
    __asm__ volatile("" ::: "memory");
    const uint32_t so = opaque(osub);
    const int gt = t_base + t;
    RecAt ra;
    const bool rec_on = TAPE && rec_at(rs, gt, ra);  // wave uniform
    if (TAPE && tape && (gt % ckpt_every) == 0) {
      float* ck = tape + (size_t)(gt / ckpt_every) * CK_F * N;
      if (active) {
        store_rows<SUB, NS>(ck, N, so, sub, x);
        if (sub == 0) {
          at_byte(ck + (size_t)CK_TEP * N, so) = __int_as_float(t_ep);
          at_byte(ck + (size_t)CK_EP * N, so) = __int_as_float(ep);
        }
      }
#pragma unroll
      for (int tl = 0; tl < TILES; ++tl) {
        const uint32_t kc = opaque(4u * (uint32_t)(lg * N + et[tl]));
        if (env0 + 16 * tl + li < N)
#pragma unroll
          for (int s = 0; s < NH; ++s) at_byte(ck + (size_t)(NS + s * NA) * N, kc) = H.get(tl, s);
      }
    }
    float F[TILES][5];
    tile_features<TILES, EXTRAS>(c, sp, x, lg, F, [&](float* zc, float* zs) {
      draw_normals<TILES>(c, (uint32_t)e, (uint32_t)ep, t_ep, lg, zc, zs);
    });
    // the wave in its actor goes first: its products are the serial part, the
    // other wave's vector instructions fill in
    __builtin_amdgcn_s_setprio(1);
    float z3[NA];
    StepRec<TILES> sr;
    if constexpr (TAPE) {
      sr.on = rec_on;
      sr.buf = span_rsrc(ra.base, rec_on ? 4u * (uint32_t)rec_floats(opaque_uniform(rs.len), N) : 0u);
      const uint32_t l = opaque((uint32_t)lane);  // (not formed ahead of the loop)
      sr.z = 4u * (4 * (l >> 4) * RB + (l & 15));
#pragma unroll
      for (int tl = 0; tl < TILES; ++tl) {
        sr.mask[tl] = 0u;
        sr.s[tl] = 4u * (uint32_t)(rec_step(ra.step, N) + rb_at(env0 + 16 * tl, REC_F));
      }
      tile_actor<TILES>(lds, fp, a1, F, lost, z3, sr);
    } else {
      tile_actor<TILES>(lds, fp, a1, F, lost, z3, NoRec{});
    }
#pragma unroll
    for (int tl = 0; tl < TILES; ++tl) lost[tl] = bad_actor ? ~0ull : 0ull;
    __builtin_amdgcn_s_setprio(0);
    float a[NA], at[TILES];
#pragma unroll
    for (int i = 0; i < NA; ++i) a[i] = tanh_act(z3[i]);
    to_tiles<TILES>(a, lg, at);
    if (TAPE && rec_on) {
      const uint32_t l = opaque((uint32_t)lane), ko = 4u * ((l >> 4) * RB + (l & 15));  // row lg
      const int cap = opaque_uniform(rs.len);  // (not formed ahead of the loop)
#pragma unroll
      for (int tl = 0; tl < TILES; ++tl) {
        // the state features, masks and actions; the history features are
        // earlier actions, kept on the segment's action tape (the
        // checkpoint's history first, then a_t)
        const uint32_t act =
            4u * (uint32_t)(rec_act(cap, N) + rb_at(env0 + 16 * tl, (NH + cap) * NA));
#pragma unroll
        for (int q = 0; q < 5; ++q)
          if (q < 4 || lg < 2) bst1(F[tl][q], sr.buf, ko, sr.s[tl] + 4u * (REC_O + 4 * q) * RB);
        bst1(at[tl], sr.buf, ko, sr.s[tl] + 4u * REC_A * RB);
        bst1(__uint_as_float(sr.mask[tl]), sr.buf, ko, sr.s[tl] + 4u * REC_M * RB);
        if (ra.step == 0) {
#pragma unroll
          for (int s = 0; s < NH; ++s) bst1(H.get(tl, s), sr.buf, ko, act + 4u * (s * NA) * RB);
        }
        bst1(at[tl], sr.buf, ko, act + 4u * (uint32_t)((NH + ra.step) * NA) * RB);
      }
      // row sub of the own env, from the wave's first
      const uint32_t xo = 4u * ((l >> 4) / TILES * RB + 16 * ((l >> 4) % TILES) + (l & 15));
      store_rows<SUB, NS>(ra.base + rec_step(ra.step, N) + rb_at(env0, REC_F) + REC_X * RB, RB,
                          xo, sub, x);
    }
    // the action goes to the history ring in memory as it is applied (the
    // last 32 of a launch; the older ones would be overwritten)
    if (!REC && t >= T - NH && active)
      store_ring<SUB>(b.ring, N, (head0 + t) & (NH - 1), so, sub, a);
    uint32_t ap[TILES][T_P];
#pragma unroll
    for (int tl = 0; tl < TILES; ++tl) split_pair(at[tl], 0.0f, ap[tl]);
    H.push(ap);
    float u[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) u[i] = action_to_rpm(c, a[i]);
    // ahead of each (two tiles) or every other (one tile) right-hand side the
    // history sums of one or two unit tiles for the next step
    __asm__ volatile("" ::: "memory");  // the body is read here, not ahead of the actor
    const Body<float> B = park.body<EXTRAS>();
    rk4_step<float, EXTRAS>(B, c.arm, c.km, c.g, c.dt, renorm, x, u, [&](int k) {
      __builtin_amdgcn_sched_barrier(0);
      if (k % T_NN<TILES> == 0) tile_history<TILES>(fp, H, k, a1);
    });
    __builtin_amdgcn_sched_barrier(0);
    const float r = reward(c, x, a);
    ++t_ep;
    const uint32_t d = episode_end(c, x, t_ep);
    const bool rst = d && (c.flags & F_AUTORESET);
    EpAcc acc = park.acc();
    acc.add(r, rst, t_ep);
    park.put(acc);
    const uint64_t any = __ballot(rst);
    if (any) {  // wave uniform
      bool on[TILES];
#pragma unroll
      for (int tl = 0; tl < TILES; ++tl) on[tl] = (any >> (16 * tl + li)) & 1u;
      float aht[TILES];
#pragma unroll
      for (int tl = 0; tl < TILES; ++tl) aht[tl] = park[PK_AH + tl];
      H.fill(on, aht);
      reset_history<TILES>(lds, on, aht, a1);
      if (rst) {
        ++ep;
        t_ep = 0;
        was_reset = true;
        const float wh = park[PK_HOVER];
        if (have) {
#pragma unroll
          for (int i = 0; i < NRES; ++i) x[i] = park[PK_NEXT + i];
#pragma unroll
          for (int i = NRES; i < NS; ++i) x[i] = wh;
          have = false;
        } else {
          reset_draw<0>(c, (uint32_t)e, (uint32_t)ep, wh, x);
        }
        if (EXTRAS) {
          float dd[6];
          disturbance(c, (uint32_t)e, (uint32_t)ep, dd);
          Body<float> Bn = B;
          set_disturbance(Bn, dd);
          park.put(Bn);
        }
      }
    }
    if (ahead && (t & (RESERVE_PERIOD - 1)) == RESERVE_PERIOD - 1 && !have) {
      draw_next();
      have = true;
    }
    if (active) {
      if (sub == 0) {
        if (rewards) at_byte(rewards + (size_t)gt * N, so) = r;
        if (dones) at_byte(dones + (size_t)gt * N, so >> 2) = (uint8_t)d;
      }
      if (states) store_rows<SUB, NS>(states + (size_t)(gt + 1) * NS * N, N, so, sub, x);
    }
  }
  if (!active || REC) return;
  const uint32_t ef = opaque((uint32_t)e);
  store_rows<SUB, NS>(b.state, N, osub, sub, x);
  const int head1 = (head0 + T) & (NH - 1);
  // after a reset in this launch the slots older than the episode's t_ep
  // actions hold the hover action
  if (was_reset)
#pragma unroll 1
    for (int s = 0; s < NH - t_ep; ++s) {
      const float ah = rpm_to_action(c, park[PK_HOVER]);
      const float v[NA] = {ah, ah, ah, ah};
      store_ring<SUB>(b.ring, N, (head1 + s) & (NH - 1), osub, sub, v);
    }
  if (sub == 0) {
    b.head[ef] = head1;
    b.t_ep[ef] = t_ep;
    b.ep[ef] = ep;
    park.acc().store(b, N, ef);
  }
}

template <int TILES, bool EXTRAS>
static hipError_t launch(const DevCfg& c, const SimBufs& b, const float* W, int T, int t_base,
                         float* rewards, uint8_t* dones, float* states, float* tape,
                         int ckpt_every, const float* ck_in, const RecSpan& rs, hipStream_t st) {
  // A CU holds one workgroup (the staged weights take more than half of its
  // LDS).  The batch is spread over the 256 CUs with 4 to 8 waves each: fewer
  // than 4 would leave SIMDs idle, more than 8 do not fit.
  const int waves = (c.n_envs + 16 * TILES - 1) / (16 * TILES);
  int per = (waves + 255) / 256;
  per = per < 4 ? 4 : per > 8 ? 8 : per;
  const dim3 g((unsigned)((waves + per - 1) / per)), blk((unsigned)per * 64);
  auto k = tape || ck_in || rs.buf[0] ? k_tile<TILES, EXTRAS, true>
                                      : k_tile<TILES, EXTRAS, false>;
  hipLaunchKernelGGL(k, g, blk, 0, st, c, b, W, T, t_base, rewards, dones, states, tape,
                     ckpt_every, ck_in, rs);
  return hipGetLastError();
}

hipError_t launch_tile(int tiles, const DevCfg& c, const SimBufs& b, const float* W, int T,
                       int t_base, float* rewards, uint8_t* dones, float* states, float* tape,
                       int ckpt_every, const float* ck_in, const RecSpan& rs, hipStream_t st) {
  if (!rec_span_ok(rs)) return hipErrorInvalidValue;
  const bool ex = (c.flags & (F_DISTURB | F_OBS_NOISE)) != 0 || c.target != nullptr;
  auto f = tiles == 2 ? (ex ? launch<2, true> : launch<2, false>)
                      : (ex ? launch<1, true> : launch<1, false>);
  return f(c, b, W, T, t_base, rewards, dones, states, tape, ckpt_every, ck_in, rs, st);
}

}  // namespace qs
