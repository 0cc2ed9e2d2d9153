// Discrete adjoint of a taped rollout.
//
// The taped forward stored checkpoints (state, history) every K steps.  The
// backward walks the segments last to first; per segment:
//   1. recompute: the taped forward's kernel restarts from the checkpoint and
//      records x_t, a_t, the layer pre-activations z1, z2 and the state
//      features of o_t per step (the history features are earlier actions);
//   2. reverse sweep (k_bwd_reverse): four lanes per env, the adjoints of
//      the state and of the action history in registers, stepping back
//      through reward, quaternion renormalisation, the four RK4 stages, the
//      action map, the actor (on MFMA) and the history shift; per-env
//      parameter gradients accumulate in registers; the layer cotangents
//      dz1 and dz3 of every (step, env) go to scratch;
//   3. weight gradients (k_bwd_dw): sum over (step, env) rows of dz (x) input
//      on bf16 MFMA with split operands, one workgroup per (64-env chunk, step group)
//      accumulating into its own partial; biases come from a constant-one
//      input column.
// Finally k_bwd_reduce adds the workgroup partials in a fixed order, so the
// result does not depend on scheduling.
//
// Fused multiply-adds only where one expression of the source holds the product
// and the sum, so kernels that promise equal results round alike.
#pragma clang fp contract(on)
#include <type_traits>

#include "qs_actor.h"
#include "qs_backward.h"
#include "qs_forward.h"
#include "qs_reverse.h"

namespace qs {

static inline unsigned nb(int n, int bs) { return (unsigned)((n + bs - 1) / bs); }

__global__ void k_fill(float* __restrict__ p, size_t n, float v) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// lam = (dS_T, 0), gth = 0.
__global__ void k_bwd_init(int N, const float* __restrict__ dS_T, float* __restrict__ lam,
                           float* __restrict__ gth) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N) return;
  for (int i = 0; i < NS; ++i) lam[(size_t)i * N + e] = dS_T ? dS_T[(size_t)i * N + e] : 0.0f;
  for (int i = NS; i < LAM_F; ++i) lam[(size_t)i * N + e] = 0.0f;
  for (int i = 0; i < NP; ++i) gth[(size_t)i * N + e] = 0.0f;
}

// Reverse sweep in the quarter-lane layout (16 envs per wave, lane L = j +
// 16 k: env j, quarter k), the adjoint of the forward step.  Per lane:
// the state adjoint (17) and the dynamics VJP, replicated over the 4 quarters
// of an env; the history adjoint of action component k (32 slots).  The actor
// VJP runs on matrix cores:
//   dz2 = W3^T dz3: one K=4 fp32 product per 16-neuron tile (quarter k supplies
//         dz3[k]);
//   dz1 = W2^T dz2, do = W1^T dz1: bf16 products of split operands (qs_tile.h),
//         each layer's result registers split into the next one's operands.
// The rows of W1^T are taken in the forward's observation order, so tile p
// of do leaves in quarter k exactly the features PHI(4p + r, k): history
// slot 4p + r - 5, component k (the lane's own history adjoint) or, for
// chunks 0..4, state features 4c + k, gathered across quarters with 20
// lane shuffles.  One wave per SIMD, bound by the serial chain of a step (the
// stages of the dynamics, then the layers): 16 steps of 16384 envs took 164 us
// with fp32 products and a branch around each load and store, now 107 (the
// split form at 1024 envs 100 and 83).
//
// LDS (floats): R_W3 [4][64] = W3; R_FRAG the transposed layers' fragments
// (stage_transposed).
constexpr int R_W3 = 0, R_FRAG = R_W3 + NA * NHID, R_TOTAL = R_FRAG + 4 * RT_FRAGS;

__host__ __device__ constexpr int r_phi(int c, int k) {
  return c < 5 ? (4 * c + k < 18 ? 4 * c + k : -1) : c < 37 ? 18 + 4 * (c - 5) + k : -1;
}

__device__ inline void stage_reverse(const float* __restrict__ W, float* lds, bool bf16) {
  stage_lds(lds + R_W3, NA * NHID, W, [](int i) { return OFF_W3 + i; }, bf16);
  stage_transposed(W, reinterpret_cast<u4t*>(lds + R_FRAG),
                   [](int p, int i) { return r_phi(4 * p + (i & 3), i >> 2); }, bf16);
}

// Inputs of one reverse step: the recorded state and action, this lane's
// ReLU mask word (tile_mask: the signs of its 16 layer-1 and 16 layer-2
// pre-activations, neurons 16 q + 4 k + r), the reward and state cotangents.
struct StepIn {
  float x[NS], a[NA], dS[NS], dR;
  uint32_t zm;
};

// vx, vk: the lane's byte offsets of its env's column and of row k of it in a
// step's record, sr the step's; ve = 4 e.
__device__ __forceinline__ void load_step(StepIn& in, __amdgpu_buffer_rsrc_t rrec, uint32_t sr,
                                          uint32_t vx, uint32_t vk, uint32_t ve,
                                          const float* __restrict__ d_rewards,
                                          const float* __restrict__ d_states, int t, int N) {
#pragma unroll
  for (int i = 0; i < NS; ++i) in.x[i] = bld1(rrec, vx, sr + 4u * (REC_X + i) * RB);
#pragma unroll
  for (int i = 0; i < NA; ++i) in.a[i] = bld1(rrec, vx, sr + 4u * (REC_A + i) * RB);
  in.zm = __float_as_uint(bld1(rrec, vk, sr + 4u * REC_M * RB));
  load_cotangents(in.dS, in.dR, d_rewards, d_states, t, N, ve);
}

// The observation's share of the adjoints, from do (dob: tile p, register r
// of quarter k = the cotangent of feature PHI(4p + r, k)): shifts the
// history adjoint (H_t[s] feeds H_{t+1}[s-1]), gathers the 18 state features
// from the quarters, adds them (through R(q)) to gx and forms the state
// adjoint before the step, ls = gx + dS.  sgn: do's sign (dz_sign).
__device__ __forceinline__ void reverse_observation(const float dob[40], const float x[NS],
                                                    const float dS[NS], float sgn, int j,
                                                    float gx[NS], float lH[NH], float ls[NS]) {
  // descending s reads the older adjoint before it is overwritten
#pragma unroll
  for (int s = NH - 1; s >= 0; --s) lH[s] = fmaf(sgn, dob[5 + s], s >= 1 ? lH[s - 1] : 0.0f);
  // state features 4cc + q live in quarter q: gather them into every lane
  float gf[20];
#pragma unroll
  for (int cc = 0; cc < 5; ++cc)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      gf[4 * cc + q] = __int_as_float(
          __builtin_amdgcn_ds_bpermute((j + 16 * q) << 2, __float_as_int(dob[cc])));
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    gx[i] = fmaf(sgn, gf[i], gx[i]);
    gx[7 + i] = fmaf(sgn, gf[12 + i], gx[7 + i]);
    gx[10 + i] = fmaf(sgn, gf[15 + i], gx[10 + i]);
  }
  {
    float gq[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    const float q[4] = {x[3], x[4], x[5], x[6]};
    rotmat_vjp(q, gf + 3, gq);
#pragma unroll
    for (int i = 0; i < 4; ++i) gx[3 + i] = fmaf(sgn, gq[i], gx[3 + i]);
  }
#pragma unroll
  for (int i = 0; i < NS; ++i) ls[i] = gx[i] + dS[i];
}

// Exchange space of the split sweep, after the staged weights: dz2 and dz1 as
// operands [part][chunk][64] (16 bytes, a tile filling half of each) and do tiles
// [10][64] (f4).
constexpr int R_XCH = (2 * T_P + 2 * T_P + 10) * 64 * 4;
// Batches up to this size run the split sweep (four times the waves; the
// quarter-lane sweep leaves most SIMDs idle there; a workgroup of either takes a CU,
// so beyond 4096 envs the split one needs a second round: forward and backward of
// 4097 envs x 64 steps 790 us on the quarter-lane sweep, 1065 on the split one).
constexpr int REVERSE_SPLIT_MAX_ENVS = 4096;
// From this size (fp32 actor) the one-env-per-lane sweep (qs_reverse1.hip): one
// round of 64-env waves, one per SIMD, up to 65536 envs, and no repeated dynamics
// adjoint; the quarter-lane sweep takes a round per 16384 envs.  Forward and backward
// of 64 steps, quarter-lane against one-lane: 32768 envs 1825 and 1957 us, 32769
// 2490 and 2306, 49152 2660 and 2455, 65535 3550 and 3080.  The present kernels
// cross at 32769 envs; the line is still where their fp32-product forms did.
constexpr int REVERSE_LANE_MIN_ENVS = 65536;

// Reverse sweep of one segment.  SPLIT = false: 16 envs per wave in the
// quarter-lane layout.  SPLIT = true: 16 envs per workgroup of 4 waves, each
// in that layout; wave w evaluates neuron tile w of dz2 and dz1 and the do
// tiles w, w + 4, w + 8 on MFMA, the tiles go through LDS (three barriers a
// step, each exchange buffer rewritten only after the barrier that follows
// every wave's reads of it), and every wave runs the dynamics and the
// observation adjoints.  The MFMA chains of each tile are the same in both,
// so they agree bit for bit.
template <bool SPLIT>
__global__ void __launch_bounds__(256)
k_bwd_reverse(DevCfg c, const float* __restrict__ theta, const float* __restrict__ W,
              const float* __restrict__ ck, const float* __restrict__ rec, int n, int t0,
              const float* __restrict__ d_rewards,
              const float* __restrict__ d_states, float* __restrict__ lam,
              float* __restrict__ gth_io, float* __restrict__ dz) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  stage_reverse(W, lds, (c.flags & F_ACTOR_BF16) != 0);
  __syncthreads();
  const int N = c.n_envs;
  const int lane = threadIdx.x & 63, j = lane & 15, k = lane >> 4;
  const int w = SPLIT ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
  const int env0 = SPLIT ? blockIdx.x * 16 : (blockIdx.x * blockDim.x + threadIdx.x - lane) / 4;
  if (env0 >= N) return;  // SPLIT: the whole workgroup
  const int env = env0 + j;
  const bool active = env < N;
  const int e = active ? env : env0;
  const u4t* frag = reinterpret_cast<const u4t*>(lds + R_FRAG);
  u4t(*xd2)[2][64] = reinterpret_cast<u4t(*)[2][64]>(lds + R_TOTAL);
  u4t(*xd1)[2][64] = xd2 + T_P;
  f4t* xdo = reinterpret_cast<f4t*>(xd1 + T_P);
  // this wave's tile of a layer as half of the next layer's operands, and the
  // whole operands after the barrier
  const auto put = [&](u4t(*xc)[2][64], const f4t& d) {
    uint32_t p[T_P], q[T_P];
    split_pair(d[0], d[1], p);
    split_pair(d[2], d[3], q);
#pragma unroll
    for (int s = 0; s < T_P; ++s)
      *(reinterpret_cast<uint2*>(&xc[s][w >> 1][lane]) + (w & 1)) = uint2{p[s], q[s]};
  };
  const auto get = [&](u4t(*xc)[2][64], u4t(&x)[2][1][T_P]) {
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int s = 0; s < T_P; ++s) x[m][0][s] = xc[s][m][lane];
  };

  float th[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) th[i] = theta[(size_t)i * N + e];
  // the episode disturbance of the segment (no resets in a taped rollout)
  float dist[6];
  disturbance(c, (uint32_t)e, (uint32_t)__float_as_int(ck[(size_t)CK_EP * N + e]), dist);
  const Quad B = make_rev_quad(c, th, dist);
  const RevStep rs = make_rev_step(c);
  const bool renorm = (c.flags & F_RENORM_Q) != 0;
  const float sgn = wave_const(dz_sign(env0));  // of all 16 envs

  float ls[NS], lH[NH], gth[NP];
#pragma unroll
  for (int i = 0; i < NS; ++i) ls[i] = lam[(size_t)i * N + e];
#pragma unroll
  for (int s = 0; s < NH; ++s) lH[s] = lam[(size_t)(NS + s * NA + k) * N + e];
#pragma unroll
  for (int i = 0; i < NP; ++i) gth[i] = gth_io[(size_t)i * N + e];

  // The per-step inputs (record rows and cotangents) of step tl - 1 are
  // loaded while step tl is processed, so their latency hides behind it.
  // Byte offsets.  Lanes of envs >= N store zeros into their slots of the padded
  // block, so no store is under a branch.
  const uint32_t rbp = (uint32_t)rb_pad(N);
  const __amdgpu_buffer_rsrc_t rrec = span_rsrc(rec, 4u * (uint32_t)rec_floats(n, N));
  const __amdgpu_buffer_rsrc_t rdz = span_rsrc(dz, 4u * (uint32_t)n * DZ_F * rbp);
  const uint32_t vx = 4u * (uint32_t)rb_at(e, REC_F), vk = vx + 4u * (uint32_t)(k * RB);
  const uint32_t ve = 4u * (uint32_t)e, vz = 4u * (uint32_t)rb_at(env, DZ_F);
  const uint32_t vz1 = vz + 4u * (uint32_t)(k * RB), vz4 = vz + 4u * (uint32_t)(4 * k * RB);
  StepIn cur, nxt;
  load_step(cur, rrec, 4u * (uint32_t)(n - 1) * (REC_F * rbp), vx, vk, ve, d_rewards, d_states,
            t0 + n - 1, N);
  drain_loads();
  for (int tl = n - 1; tl >= 0; --tl) {
    __asm__ volatile("" ::: "memory");
    const int tp = tl > 0 ? tl - 1 : 0;
    load_step(nxt, rrec, 4u * (uint32_t)tp * (REC_F * rbp), vx, vk, ve, d_rewards, d_states,
              t0 + tp, N);
    const uint32_t sz = 4u * (uint32_t)tl * (DZ_F * rbp);  // the step's cotangents
    const uint32_t zm = active ? cur.zm : 0u;

    float gx[NS], ga[NA];
    // newest history slot: component i lives in quarter i of the same env
    float hn[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i)
      hn[i] = __int_as_float(
          __builtin_amdgcn_ds_bpermute((j + 16 * i) << 2, __float_as_int(lH[NH - 1])));
    reverse_dynamics(c, rs, B, renorm, cur.x, cur.a, d_rewards ? cur.dR : 1.0f, ls, hn, gx, ga, gth);

    // --- actor VJP on matrix cores --------------------------------------------
    float d3[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) d3[i] = ga[i] * (1.0f - cur.a[i] * cur.a[i]);
    const float d3e = k == 0 ? d3[0] : k == 1 ? d3[1] : k == 2 ? d3[2] : d3[3];
    const float d3k = active ? sgn * d3e : 0.0f;
    if (!SPLIT || w == 0) bst1(d3k, rdz, vz1, sz + 4u * DZ_3 * RB);
    // do = W1^T dz1 in observation order: tile p, register r of quarter k is
    // the cotangent of feature PHI(4p + r, k)
    float dob[40];
    if (!SPLIT) {
      // dz2 = (W3^T dz3) * [z2 > 0]: tile q rows 16q + 4k + r, env j
      f4 dz2[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        dz2[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(lds[R_W3 + k * NHID + 16 * q + j], d3k,
                                                      f4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          dz2[q][r] = (zm >> (8 * q + 4 + r)) & 1u ? dz2[q][r] : 0.0f;
        }
      }
      // dz1 = (W2^T dz2) * [z1 > 0]
      u4t xo[2][1][T_P];
#pragma unroll
      for (int m = 0; m < 2; ++m) hidden_operand(dz2[2 * m], dz2[2 * m + 1], xo[m][0]);
      f4t dz1[4][1];
#pragma unroll
      for (int mt = 0; mt < 4; mt += 2)
        transposed_sum<2, 1>(frag, 2 * mt, lane, xo, reinterpret_cast<f4t(&)[2][1]>(dz1[mt]));
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          dz1[mt][0][r] = (zm >> (8 * mt + r)) & 1u ? dz1[mt][0][r] : 0.0f;
          bst1(dz1[mt][0][r], rdz, vz4, sz + 4u * (16 * mt + r) * RB);
        }
#pragma unroll
      for (int m = 0; m < 2; ++m) hidden_operand(dz1[2 * m][0], dz1[2 * m + 1][0], xo[m][0]);
#pragma unroll
      for (int p = 0; p < 10; p += 2) {
        f4t o[2][1];
        transposed_sum<2, 1>(frag, RT_G1 + 2 * p, lane, xo, o);
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int r = 0; r < 4; ++r) dob[4 * (p + q) + r] = o[q][0][r];
      }
    } else {
      // dz2 tile w
      f4 d2 = __builtin_amdgcn_mfma_f32_16x16x4f32(lds[R_W3 + k * NHID + 16 * w + j], d3k,
                                                   f4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        d2[r] = (zm >> (8 * w + 4 + r)) & 1u ? d2[r] : 0.0f;
      }
      put(xd2, d2);
      __syncthreads();
      u4t xo[2][1][T_P];
      get(xd2, xo);
      // dz1 tile w
      f4t d1[1][1];
      transposed_sum<1, 1>(frag, 2 * w, lane, xo, d1);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        d1[0][0][r] = (zm >> (8 * w + r)) & 1u ? d1[0][0][r] : 0.0f;
        bst1(d1[0][0][r], rdz, vz4, sz + 4u * (16 * w + r) * RB);
      }
      put(xd1, d1[0][0]);
      __syncthreads();
      get(xd1, xo);
      // do tiles w, w + 4, w + 8
#pragma unroll
      for (int pi = 0; pi < 3; ++pi) {
        const int p = w + 4 * pi;
        if (p < 10) {
          f4t o[1][1];
          transposed_sum<1, 1>(frag, RT_G1 + 2 * p, lane, xo, o);
          xdo[p * 64 + lane] = o[0][0];
        }
      }
      __syncthreads();
#pragma unroll
      for (int p = 0; p < 10; ++p) {
        const f4t v = xdo[p * 64 + lane];
#pragma unroll
        for (int r = 0; r < 4; ++r) dob[4 * p + r] = v[r];
      }
    }
    reverse_observation(dob, cur.x, cur.dS, sgn, j, gx, lH, ls);
    cur = nxt;
  }
  if (!active || w != 0) return;
  const uint32_t ef = opaque((uint32_t)e);
  const uint32_t kf = opaque((uint32_t)(k * N + e));
#pragma unroll
  for (int i = 0; i < NS; ++i)
    if ((i & 3) == k) lam[(size_t)i * N + ef] = ls[i];
#pragma unroll
  for (int s = 0; s < NH; ++s) lam[(size_t)(NS + s * NA) * N + kf] = lH[s];
  if (k == 0)
#pragma unroll
    for (int i = 0; i < NP; ++i) gth_io[(size_t)i * N + ef] = gth[i];
}

// Weight gradients of one segment: for every (step, env) row,
//   dW1 += dz1 o^T, dW2 += dz2 relu(z1)^T, dW3 += dz3 relu(z2)^T, db += dz,
// the rows being the contraction dimension.  The products run on bf16 matrix
// cores with both operands split (qs_tile.h), 32 envs a product: A[i][k] (lane
// i + 16 lg, 8 elements) = dz of neuron 16 n + i, B[k][j] = input column 16 t + j,
// element e of both at env 32 s + 16 (e / 4) + 4 lg + e % 4 of slab pair s; result
// register r of a tile holds neuron 16 n + 4 lg + r, column 16 t + li.
//
// One workgroup of 8 waves per (64-env block, step group).  The input
// columns fall in column tiles of 16: layer 1's 146 columns and its constant one
// (the bias) make the tiles 0..9, layer 2's 64 columns the tiles 10..13, layer
// 3's the tiles 14..17.  Waves g and g + 4 run column group g on the two slab
// pairs of each step (two waves per SIMD, so one's loads and splitting overlap
// the other's matrix work); at the end the second's sums, of the opposite sign
// (dz_sign), are taken from the first's through LDS.  A group owns three tiles with their 4 neuron tiles -- {g, g + 4} of
// layer 1 and 10 + g of layer 2 --, neuron tile g of the shared tiles 8 and 9, tile
// 14 + g of layer 3 (A's rows are the 4 outputs, repeated) and layer 2's bias of
// its neuron tile (a product with ones; group 2 layer 3's too), so the groups
// issue the same products.  The dz rows (A operands, the same for the four groups)
// are loaded once per step by the eight waves together, whole 256-byte rows
// per lane group, split once and staged in LDS; each wave loads its own input
// columns (B operands) from the record or the LDS copy of the action tape and
// splits them.  The history features of o_t are the actions of the 32
// previous steps, read from the segment's action tape (one contiguous span
// per 64-env block).
//
// A step of 65536 envs reads 58 MB (11 us at a copy's rate) and takes 6 us of
// products and 8 us of vector instructions per SIMD, mostly splitting: 17 us, as
// the two waves of a SIMD meet at a barrier every step.  It took 21 us with fp32
// products (13 us of them) and dz2 read from memory (16384 envs: 5.6, now 4.7).
constexpr int DW_GL = 3;  // B operands a group may read from the record: i of dw_tile
// accumulators (f4) of a wave: tile i < 3, neuron tile n at 4 i + n, the shared
// tiles 8 and 9, layer 3's tile, and the biases (layer 2's in columns 0..7,
// layer 3's in columns 8..15 of group 2)
constexpr int DW_A_T8 = 12, DW_A_T9 = 13, DW_A_L3 = 14, DW_A_BIAS = 15, DW_NACC = 16;
constexpr int DW_T9 = 16 * 9;  // first column of tile 9: two columns, then the constant one

// column tile of operand i < 3 of group G
__host__ __device__ constexpr int dw_tile(int G, int i) { return i < 2 ? G + 4 * i : 10 + G; }
static_assert(dw_tile(3, 1) == 7 && dw_tile(0, 2) == 10 && dw_tile(3, 2) == 13 && DW_T9 + 2 == NO,
              "column groups");

// LDS staging of one step's dz rows for a half: [part][row][64 envs] in bf16, a
// row's eight 16-byte granules (4 s + lg: the operand of slab pair s, lane group
// lg) permuted by its index, so that the 16 rows a read touches lie on distinct
// banks.
constexpr int DW_ROWS = 2 * NHID + NA;  // dz1, dz2, dz3
constexpr int DW_PART = DW_ROWS * 128, DW_ABUF = T_P * DW_PART / 4;  // bytes; floats per half
__device__ inline int dw_granule(int row, int gr) { return row * 128 + 16 * (gr ^ ((row >> 1) & 7)); }
constexpr int DW_AP = RB + 4;  // pitch of the tape window: rows on distinct banks

__device__ inline f4 const4(float v) { return f4{v, v, v, v}; }

// Raw buffer view of a device array (bounds-checked by the hardware against
// `bytes`: out-of-range loads read zero).  Loads take a 32-bit per-lane byte
// offset, a uniform byte offset and a constant, so the per-tile and per-step
// parts of an address stay scalar.
__device__ inline __amdgpu_buffer_rsrc_t buf_rsrc(const float* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, (int)bytes, 0x00020000);
}
__device__ inline f4 bld4(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

// Tiles 1..9 hold history columns: tile 1 mixes the last two state features
// with history and is read from the record with a per-lane offset (the
// source step depends on the column); tiles 2..9 hold action-tape values
// only and read an LDS copy of the block's tape window: the DW_CH steps [w0,
// w0 + DW_CH) observe slots w0 .. w0 + DW_CH + NH - 2, which the workgroup
// copies in (rows (slot - w0) * NA + a, pitch DW_AP) and refills every
// DW_CH steps, so each tape value is read from memory once per window
// instead of once for each of the 32 steps that observe it.
constexpr int DW_CH = 16, DW_TW = (DW_CH + NH) * NA, DW_TBUF = DW_TW * DW_AP;

// The record's B operands of a slab pair: tiles dw_tile(G, 0), dw_tile(G, 2) and
// 14 + G, two slabs each.
struct DwOps {
  f4 v[DW_GL][2];
};
// Offsets of one step: of this step's block in the record (bytes, wave uniform),
// the lane's of tile 1 (group 1), and the step's first row of the tape window.
struct DwAddr {
  uint32_t rs, h1;
  int tape;
};

template <int G>
__device__ inline void dw_addr(DwAddr& d, int tl, int K, int chunk, int N, int lane, int w0) {
  const int li = lane & 15, lg = lane >> 4;
  const uint32_t rbp = (uint32_t)rb_pad(N), rstep = (uint32_t)REC_F * rbp;
  const uint32_t blk = (uint32_t)tl * rstep + (uint32_t)chunk * (REC_F * RB);
  d.rs = 4u * blk;
  d.tape = (tl - w0) * NA;
  d.h1 = 0;
  if (G == 1) {
    // history slot sl of step tl is tape slot tl + sl of the block
    const uint32_t tape = (uint32_t)K * rstep + (uint32_t)chunk * ((NH + K) * NA * RB);
    const int hc = li < 2 ? 0 : li - 2;
    const uint32_t o_hist = tape + (uint32_t)((tl + (hc >> 2)) * NA + (hc & 3)) * RB;
    d.h1 = 4u * (4 * lg + (li < 2 ? blk + (REC_O + 16 + li) * RB : o_hist));
  }
}

// Issues the record's B loads of slab pair s of a step; they are split when they
// are used, so the loads stay in flight during the previous pair's matrix work.
// loff: the lane's byte offset 4 (li * RB + 4 lg).
template <int G>
__device__ inline void dw_load_pair(DwOps& o, __amdgpu_buffer_rsrc_t rrec, const DwAddr& d,
                                    uint32_t loff, int s) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const uint32_t b = 128 * s + 64 * q;
    if (G == 0) o.v[0][q] = bld4(rrec, loff + b, d.rs + 4 * (REC_O * RB));
    if (G == 1) o.v[0][q] = bld4(rrec, d.h1 + b, 0);
    o.v[1][q] = bld4(rrec, loff + b, d.rs + 4 * ((REC_Z1 + 16 * G) * RB));
    o.v[2][q] = bld4(rrec, loff + b, d.rs + 4 * ((REC_Z2 + 16 * G) * RB));
  }
}

// Copies tape slots [w0, w0 + DW_CH + NH) of 64-env block `chunk` (those
// below NH + K) into the window tw, every thread of the 512 issuing its six
// 16-byte loads before its first store.
constexpr int DW_TLD = DW_TW * (RB / 4) / 512;
static_assert(DW_TW * (RB / 4) % 512 == 0, "the window splits evenly over the workgroup");
__device__ inline void dw_stage_tape(float* tw, __amdgpu_buffer_rsrc_t rrec, int chunk, int K,
                                     int N, int w0) {
  const uint32_t rbp = (uint32_t)rb_pad(N);
  // the block's tape, in bytes from the record's start
  const uint32_t base =
      4u * ((uint32_t)K * REC_F * rbp + (uint32_t)chunk * (uint32_t)((NH + K) * NA * RB));
  const int rows = min(DW_TW, (NH + K - w0) * NA);
  f4 v[DW_TLD];
#pragma unroll
  for (int j = 0; j < DW_TLD; ++j) {
    const int k = (int)threadIdx.x + 512 * j, r = k >> 4, c = 4 * (k & 15);
    const int rr = r < rows ? r : rows - 1;
    v[j] = bld4(rrec, 4u * (uint32_t)((w0 * NA + rr) * RB + c), base);
  }
#pragma unroll
  for (int j = 0; j < DW_TLD; ++j) {
    const int k = (int)threadIdx.x + 512 * j, r = k >> 4, c = 4 * (k & 15);
    if (r < rows) *reinterpret_cast<f4*>(&tw[r * DW_AP + c]) = v[j];
  }
}

// A wave's share of a step's dz rows, wave g of half h: neurons 16 g + 8 h .. + 7
// of layers 1 and 2 (lane l takes envs 4 (l & 15) .. + 3 of neuron 16 g + 8 h + 4 j
// + (l >> 4), j < 2) and, of half 0, row g of layer 3.  dz2 is formed here, (W3^T
// dz3) [z2 > 0] from dz3 and the record's mask words: it takes neither a store in
// the sweep nor a load.
struct DwRows {
  f4 d1[2], d3[4], m[2];
};
__device__ inline void dw_a_load(DwRows& r, __amdgpu_buffer_rsrc_t rdz,
                                 __amdgpu_buffer_rsrc_t rrec, int tl, int chunk, int N, int g,
                                 int h, int lane) {
  const uint32_t rbp = (uint32_t)rb_pad(N);
  const uint32_t so = 4u * ((uint32_t)tl * (DZ_F * rbp) + (uint32_t)chunk * (DZ_F * RB));
  const uint32_t ro = 4u * ((uint32_t)tl * (REC_F * rbp) + (uint32_t)chunk * (REC_F * RB));
  const uint32_t v = 16u * (uint32_t)(lane & 15), vr = v + 4u * (uint32_t)((lane >> 4) * RB);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    r.d1[j] = bld4(rdz, vr, so + 4u * (uint32_t)((16 * g + 8 * h + 4 * j) * RB));
    r.m[j] = bld4(rrec, v, ro + 4u * (uint32_t)((REC_M + 2 * h + j) * RB));
  }
#pragma unroll
  for (int i = 0; i < NA; ++i) r.d3[i] = bld4(rdz, v, so + 4u * (uint32_t)((DZ_3 + i) * RB));
}
// Where a wave's rows go: envs 4 m .. 4 m + 3 of a row lie in granule 4 (m / 8) +
// m % 4, its half (m / 4) % 2.  off: the byte offset of neuron 16 g + 8 h + (l >> 4)
// of layer 1 (four neurons further: + 512, with the permutation's bit 1 turned).
struct DwPlace {
  int off, off3;
};
__device__ inline DwPlace dw_place(int g, int h, int lane) {
  const int m = lane & 15, gr = 4 * (m >> 3) + (m & 3), half = 8 * ((m >> 2) & 1);
  return {dw_granule(16 * g + 8 * h + (lane >> 4), gr) + half, dw_granule(2 * NHID + g, gr) + half};
}
// Splits and stages piece q of the share: neurons + 4 q of layer 1 (q < 2), + 4 (q -
// 2) of layer 2 (q < 4), layer 3's row (q = 4).  w3[neuron]: layer 3's four weights
// of it.
template <int Q>
__device__ inline void dw_stage(const DwRows& r, const f4* w3, char* sA, const DwPlace& at, int g,
                                int h, int lane) {
  constexpr int J = Q & 1;
  f4 v;
  if (Q < 2) {
    v = r.d1[J];
  } else if (Q < 4) {
    const f4 w = w3[16 * g + 8 * h + 4 * J + (lane >> 4)];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      float d = w[0] * r.d3[0][m];
#pragma unroll
      for (int i = 1; i < NA; ++i) d = fmaf(w[i], r.d3[i][m], d);
      // neuron 16 g + 4 k + i: bit 8 g + 4 + i of word k
      v[m] = keep_if(d, __float_as_uint(r.m[J][m]) >> (lane >> 4), 8 * g + 4);
    }
  } else {
    v = r.d3[g];
  }
  uint32_t p[T_P], q[T_P];
  split_pair(v[0], v[1], p);
  split_pair(v[2], v[3], q);
  char* a = sA + (Q == 4 ? at.off3 : (at.off ^ (32 * J)) + 512 * J + (Q < 2 ? 0 : NHID * 128));
  if (Q < 4 || (h == 0 && lane < 16))
#pragma unroll
    for (int s = 0; s < T_P; ++s) *reinterpret_cast<uint2*>(a + s * DW_PART) = uint2{p[s], q[s]};
}

// B operand of a slab pair from its two slabs: ReLU of the pre-activation columns
// (RELU) and the forward's bf16 rounding of its inputs (BF16: one part).  Envs >=
// N of the last block need nothing: their dz slots are zero (cleared at
// allocation; the sweeps write zeros there) and their record slots are zero or
// finite copies of a batch env's values, so they add nothing.
template <bool RELU, bool BF16>
__device__ inline void dw_operand(f4 lo, f4 hi, u4t (&x)[T_P]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    if (RELU) {
      lo[m] = relu_bits(lo[m]);
      hi[m] = relu_bits(hi[m]);
    }
  }
  if (BF16) {
    x[0] = u4t{pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]), pack_bf16(hi[0], hi[1]),
               pack_bf16(hi[2], hi[3])};
  } else {
    hidden_operand(lo, hi, x);
  }
}
// The products of A operand a with M B operands: the small terms first.
template <int M, bool BF16>
__device__ inline void dw_products(f4* acc, const u4t (&a)[T_P], const u4t (*x)[T_P]) {
  constexpr int AP[6] = {2, 0, 1, 1, 0, 0}, XP[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    if (BF16 && XP[k] > 0) continue;
#pragma unroll
    for (int i = 0; i < M; ++i) acc[i] = mfma_bf(a[AP[k]], x[i][XP[k]], acc[i]);
  }
}

// Slab pair s of a step.  sA: the step's staged rows; tw: the tape window; tape:
// the step's first row in it.  stage(q), q < 5: the pieces of the next step's
// staging, placed where matrix instructions can cover them.
template <int G, bool BF16, typename Stage>
__device__ inline void dw_pair(f4* acc, const DwOps& o, const char* sA, const float* tw, int tape,
                               int s, int lane, Stage&& stage) {
  const int li = lane & 15, lg = lane >> 4;
  // the A operands of rows row0 + li, row0 a multiple of 16
  const char* la = sA + dw_granule(li, 4 * s + lg);
  const auto rows = [&](int row0, u4t (&a)[T_P]) {
#pragma unroll
    for (int p = 0; p < T_P; ++p)
      a[p] = *reinterpret_cast<const u4t*>(la + row0 * 128 + p * DW_PART);
  };
  // tile t of the tape window: history columns 16 t - 18 ..
  const auto tape_tile = [&](int t, u4t (&x)[T_P]) {
    const int c = t == 9 && li >= 2 ? 0 : li;
    const float* w = tw + (tape + 16 * t - 18 + c) * DW_AP + 32 * s + 4 * lg;
    f4 lo = *reinterpret_cast<const f4*>(w), hi = *reinterpret_cast<const f4*>(w + 16);
    if (t == 9) {
      const float one = li == 2 ? 1.0f : 0.0f;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        lo[m] = li < 2 ? lo[m] : one;
        hi[m] = li < 2 ? hi[m] : one;
      }
    }
    dw_operand<false, BF16>(lo, hi, x);
  };
  // Neuron tiles in the outer loop: two operands of 12 registers a side at a time.
  u4t a[2][T_P], x[2][T_P], y[2][T_P];
  if (G < 2)
    dw_operand<false, BF16>(o.v[0][0], o.v[0][1], x[0]);
  else
    tape_tile(G, x[0]);
  tape_tile(G + 4, x[1]);
  rows(0, a[0]);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    if (n < 3) rows(16 * (n + 1), a[(n + 1) & 1]);
    f4 c[2] = {acc[n], acc[4 + n]};
    dw_products<2, BF16>(c, a[n & 1], x);
    acc[n] = c[0];
    acc[4 + n] = c[1];
    if (n == 0) tape_tile(8, y[0]);
    if (n == 1) tape_tile(9, y[1]);
    if (n == 2) stage(std::integral_constant<int, 0>());
    if (n == 3) stage(std::integral_constant<int, 1>());
    __builtin_amdgcn_sched_barrier(0);
  }
  rows(16 * G, a[0]);
  dw_products<2, BF16>(acc + DW_A_T8, a[0], y);
  dw_operand<true, BF16>(o.v[1][0], o.v[1][1], x[0]);
  stage(std::integral_constant<int, 4>());
  rows(NHID, a[0]);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    if (n < 3) rows(NHID + 16 * (n + 1), a[(n + 1) & 1]);
    dw_products<1, BF16>(acc + 8 + n, a[n & 1], x);
    if (n == 0) stage(std::integral_constant<int, 2>());
    if (n == 1) stage(std::integral_constant<int, 3>());
    if (n == 2) dw_operand<true, BF16>(o.v[2][0], o.v[2][1], x[1]);
    __builtin_amdgcn_sched_barrier(0);
  }
  // layer 3: rows 128 + li % 4
  u4t a3[T_P], ag[T_P];
#pragma unroll
  for (int p = 0; p < T_P; ++p)
    a3[p] = *reinterpret_cast<const u4t*>(sA + dw_granule(2 * NHID + (li & 3), 4 * s + lg) +
                                          p * DW_PART);
  rows(NHID + 16 * G, ag);
  dw_products<1, BF16>(acc + DW_A_L3, a3, x + 1);
  // biases
  const uint32_t one = 0x3f803f80u, b2 = li < 8 ? one : 0u, b3 = li < 8 ? 0u : one;
#pragma unroll
  for (int p = T_P - 1; p >= 0; --p) {
    acc[DW_A_BIAS] = mfma_bf(ag[p], u4t{b2, b2, b2, b2}, acc[DW_A_BIAS]);
    if (G == 2) acc[DW_A_BIAS] = mfma_bf(a3[p], u4t{b3, b3, b3, b3}, acc[DW_A_BIAS]);
  }
}

// Steps t_lo .. t_hi - 1 of the group, half h taking slab pair h of each.  A step's
// B loads are issued one step ahead into the other of two operand buffers (a copy
// between them would wait for the loads in flight); its dz share is loaded two
// steps ahead and staged one ahead, beside the products, into the other of two
// staging buffers: one barrier a step, and no phase that only stages.
// sA: the staging buffers.
// Barrier discipline: the four column groups run separate instantiations of
// this loop, so their waves reach the workgroup barriers at different
// program locations; the hardware barrier counts arriving waves, and every
// wave executes the same sequence of barriers (one before the loop, one at the end
// of every iteration, another where the tape window is refilled; iters and the refills
// are uniform over the workgroup), so they pair up.
// A loop in the kernel body with the group switched per step would keep the
// barriers in uniform code, but it keeps every group's operand slots live
// across the switch and spills.
template <int G, bool BF16>
__device__ inline void dw_accumulate(f4* acc, const float* __restrict__ rec,
                                     const float* __restrict__ dz, int N, int chunk, int t_lo,
                                     int t_hi, int K, int half, char* sA, float* tw,
                                     const f4* w3) {
  const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int iters = t_hi - t_lo;
  if (iters <= 0) return;
  const uint32_t rbp = (uint32_t)rb_pad(N);
  const __amdgpu_buffer_rsrc_t rrec =
      buf_rsrc(rec, 4u * ((uint32_t)K * REC_F * rbp + (uint32_t)(NH + K) * NA * rbp));
  const __amdgpu_buffer_rsrc_t rdz = buf_rsrc(dz, 4u * ((uint32_t)K * DZ_F * rbp));
  const uint32_t loff = 4u * (uint32_t)(li * RB + 4 * lg);
  const DwPlace at = dw_place(G, half, lane);
  const auto step = [&](int i) { return t_lo + (i < iters ? i : iters - 1); };
  int w0 = t_lo;  // first slot of the tape window
  dw_stage_tape(tw, rrec, chunk, K, N, w0);
  DwRows an;
  dw_a_load(an, rdz, rrec, step(0), chunk, N, G, half, lane);
  const auto stage_to = [&](char* a) {
    return [&, a](auto q) { dw_stage<decltype(q)::value>(an, w3, a, at, G, half, lane); };
  };
  {
    const auto st = stage_to(sA);
    st(std::integral_constant<int, 0>());
    st(std::integral_constant<int, 1>());
    st(std::integral_constant<int, 2>());
    st(std::integral_constant<int, 3>());
    st(std::integral_constant<int, 4>());
  }
  DwOps ob0, ob1;
  DwAddr d;
  dw_addr<G>(d, step(0), K, chunk, N, lane, w0);
  dw_load_pair<G>(ob0, rrec, d, loff, half);
  dw_a_load(an, rdz, rrec, step(1), chunk, N, G, half, lane);
  __syncthreads();
  // One step: operands cur, the next step's into nxt.  Loads past the last step
  // read it again (a load under a branch would leave the waits counting it
  // conservatively).
  const auto body = [&](const DwOps& cur, DwOps& nxt, int i) {
    const int tape = d.tape;
    // the next step's window (refilled below when the next step opens one)
    const bool refill = i + 1 < iters && (i + 1) % DW_CH == 0;
    const int w0n = refill ? w0 + DW_CH : w0;
    dw_addr<G>(d, step(i + 1), K, chunk, N, lane, w0n);
    dw_load_pair<G>(nxt, rrec, d, loff, half);
    __builtin_amdgcn_sched_barrier(0);
    dw_pair<G, BF16>(acc, cur, sA + (i & 1) * (4 * DW_ABUF), tw, tape, half, lane,
                     stage_to(sA + (~i & 1) * (4 * DW_ABUF)));
    __builtin_amdgcn_sched_barrier(0);
    dw_a_load(an, rdz, rrec, step(i + 2), chunk, N, G, half, lane);
    if (refill) {
      __syncthreads();  // every wave is done with the window
      w0 = w0n;
      dw_stage_tape(tw, rrec, chunk, K, N, w0);
    }
    __syncthreads();
  };
  for (int i = 0; i < iters; i += 2) {
    body(ob0, ob1, i);
    if (i + 1 < iters) body(ob1, ob0, i + 1);
  }
}

// The workgroup's 64-env chunks x, x + gx, ... in turn.  (A chunk's last iteration
// ends with a barrier, so no wave still reads its staged step or its window when
// the next one is staged.)
template <int G, bool BF16>
__device__ inline void dw_chunks(f4* acc, const float* __restrict__ rec,
                                 const float* __restrict__ dz, int N, int t_lo, int t_hi, int K,
                                 int half, char* sA, float* tw, const f4* w3) {
  const int n_chunks = (N + RB - 1) / RB;
  for (int chunk = blockIdx.x; chunk < n_chunks; chunk += gridDim.x)
    dw_accumulate<G, BF16>(acc, rec, dz, N, chunk, t_lo, t_hi, K, half, sA, tw, w3);
}

// A partial slot holds the sums in the accumulators' own register layout:
// [group 4][accumulator DW_NACC][lane 64][register 4] floats, so a wave adds
// its sums with whole-wave vector loads and stores; dw_slot maps a flat
// gradient index to its place in a slot (k_bwd_reduce gathers with it).
constexpr int DW_SLOT = 4 * DW_NACC * 64 * 4;

__host__ __device__ constexpr int dw_pos(int g, int a, int lane, int r) {
  return ((g * DW_NACC + a) * 64 + lane) * 4 + r;
}
// a 16x16 product tile: row rr (neuron within the tile), column c
__host__ __device__ constexpr int dw_tile_pos(int g, int a, int rr, int c) {
  return dw_pos(g, a, c + 16 * (rr / 4), rr % 4);
}

// flat gradient index (torch Linear layout) -> place in a slot
__device__ inline int dw_slot(int idx) {
  if (idx < OFF_B1) {
    const int nrn = idx / NO, col = idx % NO, t = col / 16, c = col % 16;
    if (t >= 8) return dw_tile_pos(nrn / 16, t == 8 ? DW_A_T8 : DW_A_T9, nrn % 16, c);
    return dw_tile_pos(t % 4, 4 * (t / 4) + nrn / 16, nrn % 16, c);
  }
  if (idx < OFF_W2) {
    const int nrn = idx - OFF_B1;  // the constant column 146
    return dw_tile_pos(nrn / 16, DW_A_T9, nrn % 16, NO - DW_T9);
  }
  if (idx < OFF_B2) {
    const int nrn = (idx - OFF_W2) / NHID, col = (idx - OFF_W2) % NHID;
    return dw_tile_pos(col / 16, 8 + nrn / 16, nrn % 16, col % 16);
  }
  if (idx < OFF_W3) {
    const int nrn = idx - OFF_B2;
    return dw_tile_pos(nrn / 16, DW_A_BIAS, nrn % 16, 0);
  }
  if (idx < OFF_B3) {
    const int o = (idx - OFF_W3) / NHID, col = (idx - OFF_W3) % NHID;
    return dw_tile_pos(col / 16, DW_A_L3, o, col % 16);
  }
  return dw_tile_pos(2, DW_A_BIAS, idx - OFF_B3, 8);
}

// grid (gx, S step groups), 512 threads; workgroup x takes the 64-env
// chunks x, x + gx, ... in turn, step group sg the steps [sg * per, min(n,
// (sg + 1) * per)), per = ceil(n / S); it accumulates into its own partial
// slot (x * S + sg) across segments.  n: the segment's steps, K: the capacity of
// its buffers.
template <bool BF16>
__global__ void __launch_bounds__(512)
k_bwd_dw(int N, const float* __restrict__ W, const float* __restrict__ rec,
         const float* __restrict__ dz, int n, int K, int S, float* __restrict__ gpart) {
  // two staging buffers during the loop, then the exchange of sums
  __shared__ __attribute__((aligned(16))) float smem[2 * DW_ABUF + DW_TBUF + NHID * NA];
  float* tw = smem + 2 * DW_ABUF;  // the action-tape window
  f4* w3 = reinterpret_cast<f4*>(tw + DW_TBUF);  // layer 3's weights by neuron
  if (threadIdx.x < NHID * NA) {
    const float w = W[OFF_W3 + (threadIdx.x & 3) * NHID + (threadIdx.x >> 2)];
    tw[DW_TBUF + threadIdx.x] = BF16 ? (float)(__bf16)w : w;
  }
  __syncthreads();
  static_assert(2 * DW_ABUF * 4 >= 4 * DW_NACC * 64 * 16, "exchange fits the staging space");
  f4(*xacc)[DW_NACC][64] = reinterpret_cast<f4(*)[DW_NACC][64]>(smem);
  const int sg = blockIdx.y;
  // the wave index is uniform across the wave: keep it (and every offset
  // derived from it) in scalar registers
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = wv & 3, half = wv >> 2;
  const int per = (n + S - 1) / S;
  const int t_lo = sg * per, t_hi = (t_lo + per) < n ? (t_lo + per) : n;
  f4 acc[DW_NACC];
#pragma unroll
  for (int i = 0; i < DW_NACC; ++i) acc[i] = const4(0.0f);
  char* sA = reinterpret_cast<char*>(smem);
  // one loop over the workgroup's chunks inside each group's instantiation
  // (a loop around the switch would keep every group's operand slots live
  // and spill)
  switch (g) {
    case 0: dw_chunks<0, BF16>(acc, rec, dz, N, t_lo, t_hi, K, half, sA, tw, w3); break;
    case 1: dw_chunks<1, BF16>(acc, rec, dz, N, t_lo, t_hi, K, half, sA, tw, w3); break;
    case 2: dw_chunks<2, BF16>(acc, rec, dz, N, t_lo, t_hi, K, half, sA, tw, w3); break;
    default: dw_chunks<3, BF16>(acc, rec, dz, N, t_lo, t_hi, K, half, sA, tw, w3); break;
  }
  __syncthreads();  // the staging space becomes the exchange buffer
  // half 1 hands its sums, of the opposite sign, to half 0
  if (half == 1)
#pragma unroll
    for (int i = 0; i < DW_NACC; ++i) xacc[g][i][lane] = acc[i];
  __syncthreads();
  if (half == 1) return;
#pragma unroll
  for (int i = 0; i < DW_NACC; ++i) {
    const f4 o = xacc[g][i][lane];
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[i][r] -= o[r];
  }
  // add into this group's part of the slot: all loads, then all stores
  f4* gp = reinterpret_cast<f4*>(gpart + ((size_t)blockIdx.x * S + sg) * DW_SLOT) + g * DW_NACC * 64;
  f4 old[DW_NACC];
#pragma unroll
  for (int i = 0; i < DW_NACC; ++i) old[i] = gp[i * 64 + lane];
#pragma unroll
  for (int i = 0; i < DW_NACC; ++i) {
#pragma unroll
    for (int r = 0; r < 4; ++r) old[i][r] += acc[i][r];
    gp[i * 64 + lane] = old[i];
  }
}

// grad[i] = sum over the G partial slots of slot g's entry for i, in a fixed
// order:
// DR_SPLIT threads per output each add a contiguous range of slots in
// ascending order, then the range sums are added in ascending range order, in
// double (the kernel waits for memory, 11 us either way): in single precision these
// sums alone add a tenth to the error of the actor gradients (16384 envs x 32 steps
// 1.06e-7, with this 9.4e-8).
constexpr int DR_OUT = 32, DR_SPLIT = 8;
__global__ void __launch_bounds__(DR_OUT * DR_SPLIT)
k_bwd_reduce(const float* __restrict__ gpart, int G, float* __restrict__ out) {
  __shared__ double part[DR_SPLIT][DR_OUT];
  const int tx = threadIdx.x % DR_OUT, ty = threadIdx.x / DR_OUT;
  const int i = blockIdx.x * DR_OUT + tx;
  const int per = (G + DR_SPLIT - 1) / DR_SPLIT;
  const int g0 = ty * per, g1 = (g0 + per) < G ? (g0 + per) : G;
  double s = 0.0;
  if (i < NW) {
    const int pl = dw_slot(i);
#pragma unroll 8
    for (int gg = g0; gg < g1; ++gg) s += gpart[(size_t)gg * DW_SLOT + pl];
  }
  part[ty][tx] = s;
  __syncthreads();
  if (ty != 0 || i >= NW) return;
  double t = part[0][tx];
#pragma unroll
  for (int r = 1; r < DR_SPLIT; ++r) t += part[r][tx];
  out[i] = (float)t;
}

__global__ void k_copy(const float* __restrict__ src, float* __restrict__ dst, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

// ---------------------------------------------------------------------------

hipError_t bwd_alloc(BwdBufs& bw, int N, int K, int H) {
  bw.N = N;
  bw.K = K;
  bw.H = H;
  // Weight-gradient pass: one workgroup per CU (the double-buffered staging
  // takes most of the LDS), so about n_cu workgroups: up to n_cu 64-env
  // chunks, each split into step groups to fill the CUs; beyond n_cu chunks,
  // n_cu workgroups that each take every n_cu-th chunk in turn (one partial
  // slot per workgroup, whose sums stay in registers across its chunks).
  // A group takes at least two steps: its start (the tape window, a first step
  // staged beside nothing) costs more than the second step (forward and backward
  // of 1024 envs x 64 steps 612 us; with groups of one step, on twice the CUs, 640;
  // no difference at 64 and 256 envs).
  const int chunks = (int)nb(N, 64);
  int n_cu = 256;
  {
    int dev = 0;
    if (hipGetDevice(&dev) == hipSuccess)
      (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  }
  int S = n_cu / chunks;
  if (S > K / 2) S = K / 2;
  if (S < 1) S = 1;
  bw.dw_gx = chunks < n_cu ? chunks : n_cu;
  bw.dw_groups = S;
  bw.n_parts = bw.dw_gx * S;
  hipError_t e;
  // a horizon of J segments uses min(J, BWD_NBUF) of the rotating buffers, fewer
  // where they are large or where a recompute runs beside the sweep (overlap):
  // elsewhere every segment kept spares its recompute (16384 envs x 128 steps, K =
  // 16: 2350 us with four, 1982 with eight).  Forward and backward of 128 steps, K =
  // 8 (64 steps, K = 16), four buffers with the overlap against eight without: 6000
  // envs 1575 (797) against 2255 (866) us, 12288 2180 (920) against 2470 (978), 16320
  // 2695 (1033) against 2544 (1009), so the line by compute units lies within a few
  // percent of the crossing.
  const size_t seg_bytes = rec_floats(K, N) * 4, dz_bytes = (size_t)K * DZ_F * rb_pad(N) * 4;
  const int most = chunks < n_cu ? BWD_NBUF_MIN : BWD_NBUF;
  int nseg = (H + K - 1) / K < most ? (H + K - 1) / K : most;
  while (nseg > BWD_NBUF_MIN && (double)nseg * (double)(seg_bytes + dz_bytes) > BWD_MORE_BYTES)
    --nseg;
  const auto add_buffer = [&]() -> hipError_t {
    const int i = bw.nbuf;
    hipError_t e = hipMalloc(&bw.seg[i], seg_bytes);
    if (e == hipSuccess) e = hipMalloc(&bw.dz[i], dz_bytes);
    // zeroed once: whole wavefronts past the last env never write their slots
    // of the last 64-env block, which must read as finite (record) and zero
    // (cotangents) in the weight-gradient pass
    if (e == hipSuccess) e = hipMemset(bw.seg[i], 0, seg_bytes);
    if (e == hipSuccess) e = hipMemset(bw.dz[i], 0, dz_bytes);
    if (e == hipSuccess) ++bw.nbuf;
    return e;
  };
  for (int i = 0; i < BWD_NBUF; ++i) {
    if ((e = hipEventCreateWithFlags(&bw.e_rec[i], hipEventDisableTiming)) != hipSuccess) return e;
    if ((e = hipEventCreateWithFlags(&bw.e_rev[i], hipEventDisableTiming)) != hipSuccess) return e;
    if ((e = hipEventCreateWithFlags(&bw.e_dw[i], hipEventDisableTiming)) != hipSuccess) return e;
  }
  while (bw.nbuf < nseg && bw.nbuf < BWD_NBUF_MIN)
    if ((e = add_buffer()) != hipSuccess) return e;
  int dev = 0;
  if ((e = hipGetDevice(&dev)) != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&bw.n_cu, hipDeviceAttributeMultiprocessorCount, dev)) !=
      hipSuccess)
    return e;
  if ((e = hipEventCreateWithFlags(&bw.e_init, hipEventDisableTiming)) != hipSuccess) return e;
  if ((e = hipStreamCreateWithFlags(&bw.s_rec, hipStreamNonBlocking)) != hipSuccess) return e;
  if ((e = hipStreamCreateWithFlags(&bw.s_dw, hipStreamNonBlocking)) != hipSuccess) return e;
  if ((e = hipMalloc(&bw.lam, (size_t)LAM_F * N * 4)) != hipSuccess) return e;
  if ((e = hipMalloc(&bw.gth, (size_t)NP * N * 4)) != hipSuccess) return e;
  if ((e = hipMalloc(&bw.gpart, (size_t)bw.n_parts * DW_SLOT * 4)) != hipSuccess) return e;
  if ((e = hipMalloc(&bw.gsum, (size_t)NW * 4)) != hipSuccess) return e;
  if ((e = hipFuncSetAttribute((const void*)k_bwd_reverse<false>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, R_TOTAL * 4)) !=
      hipSuccess)
    return e;
  if ((e = hipFuncSetAttribute((const void*)k_bwd_reverse<true>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (R_TOTAL + R_XCH) * 4)) !=
      hipSuccess)
    return e;
  if ((e = reverse1_prepare()) != hipSuccess) return e;
  // The buffers past the fourth only save time: last, so that they take nothing the
  // handle needs, and each only where it is a small part of the free memory, most of
  // which is left to the caller.
  size_t free_bytes = 0, all_bytes = 0;
  while (bw.nbuf < nseg && hipMemGetInfo(&free_bytes, &all_bytes) == hipSuccess &&
         seg_bytes + dz_bytes <= free_bytes / BWD_MORE_SHARE) {
    if (add_buffer() == hipSuccess) continue;
    const int i = bw.nbuf;
    if (bw.seg[i]) (void)hipFree(bw.seg[i]);
    if (bw.dz[i]) (void)hipFree(bw.dz[i]);
    bw.seg[i] = bw.dz[i] = nullptr;
    break;
  }
  (void)hipGetLastError();  // of the calls for optional memory
  return hipSuccess;
}

void bwd_free(BwdBufs& bw) {
  for (int i = 0; i < BWD_NBUF; ++i) {
    if (bw.seg[i]) (void)hipFree(bw.seg[i]);
    if (bw.dz[i]) (void)hipFree(bw.dz[i]);
    if (bw.e_rec[i]) (void)hipEventDestroy(bw.e_rec[i]);
    if (bw.e_rev[i]) (void)hipEventDestroy(bw.e_rev[i]);
    if (bw.e_dw[i]) (void)hipEventDestroy(bw.e_dw[i]);
  }
  if (bw.e_init) (void)hipEventDestroy(bw.e_init);
  if (bw.s_rec) (void)hipStreamDestroy(bw.s_rec);
  if (bw.s_dw) (void)hipStreamDestroy(bw.s_dw);
  void* ptrs[] = {bw.lam, bw.gth, bw.gpart, bw.gsum};
  for (void* p : ptrs)
    if (p) (void)hipFree(p);
  bw = BwdBufs{};
}

#define BWD_TRY(x)                 \
  do {                             \
    hipError_t e_ = (x);           \
    if (e_ != hipSuccess) return e_; \
  } while (0)

// Segments run last to first.  Per segment (buffers in turn):
//   recompute stream: waits for the weight-gradient pass that last used the
//     buffer, then records the segment;
//   caller stream: waits for the record, runs the reverse sweep (the
//     segment-to-segment adjoint carry keeps these in order);
//   weight-gradient stream: waits for the sweep, reduces the segment.
// So the recompute of the next segments and the weight gradients of the
// previous ones overlap the sweep.  The caller's stream finally waits for
// the last weight-gradient pass before the fixed-order partial sum.
// Overlap only pays while the sweep leaves compute units idle (a workgroup of
// the recompute takes a whole one); for large batches the sweep (one wave per
// SIMD, most registers) fills the chip and everything stays on the caller's
// stream in order.  Both sides measured: bwd_alloc.
// serial: every kernel on st (the scratch-array variant, one buffer).
static hipError_t backward_segments(const DevCfg& c, const SimBufs& b, const BwdBufs& bw,
                                    bool serial, const float* W, const float* tape, int K, int T,
                                    const float* d_rewards, const float* d_states,
                                    float* grad_actor, float* grad_params, int* held,
                                    hipStream_t st) {
  const int N = c.n_envs;
  const size_t np = (size_t)bw.n_parts * DW_SLOT;
  hipLaunchKernelGGL(k_fill, dim3(nb((int)np, 256)), dim3(256), 0, st, bw.gpart, np, 0.0f);
  hipLaunchKernelGGL(k_bwd_init, dim3(nb(N, 256)), dim3(256), 0, st, N,
                     d_states ? d_states + (size_t)T * NS * N : nullptr, bw.lam, bw.gth);
  const int nbuf = bw.nbuf;
  const bool overlap = !serial && (int)nb(N, 64) < bw.n_cu;
  hipStream_t s_rec = overlap ? bw.s_rec : st, s_dw = overlap ? bw.s_dw : st;
  if (overlap) {
    BWD_TRY(hipEventRecord(bw.e_init, st));
    BWD_TRY(hipStreamWaitEvent(s_rec, bw.e_init, 0));
    BWD_TRY(hipStreamWaitEvent(s_dw, bw.e_init, 0));
  }
  const int J = (T + K - 1) / K;
  int last = 0;
  for (int j = J - 1, idx = 0; j >= 0; --j, ++idx) {
    const int t0 = j * K;
    const int n = (T - t0) < K ? (T - t0) : K;
    const int buf = idx % nbuf;
    // the record may be in the buffer already: written by the taped rollout
    // (on the caller's stream, ahead of this call) or by a recompute of an
    // earlier backward on the same tape
    if (held && held[buf] == j) {
      // nothing to recompute
    } else {
      if (held) held[buf] = j;
      if (overlap && idx >= nbuf) BWD_TRY(hipStreamWaitEvent(s_rec, bw.e_dw[buf], 0));
      BWD_TRY(launch_recompute(c, b, W, n, K, tape + (size_t)j * CK_F * N, bw.seg[buf], s_rec));
      if (overlap) {
        BWD_TRY(hipEventRecord(bw.e_rec[buf], s_rec));
        BWD_TRY(hipStreamWaitEvent(st, bw.e_rec[buf], 0));
      }
    }
    if (N >= REVERSE_LANE_MIN_ENVS && !(c.flags & F_ACTOR_BF16))
      BWD_TRY(launch_reverse1(c, b.theta, W, tape + (size_t)j * CK_F * N, bw.seg[buf], n, t0,
                              d_rewards, d_states, bw.lam, bw.gth, bw.dz[buf], st));
    else if (N <= REVERSE_SPLIT_MAX_ENVS)
      hipLaunchKernelGGL(k_bwd_reverse<true>, dim3(nb(N, 16)), dim3(256), (R_TOTAL + R_XCH) * 4,
                         st, c, b.theta, W, tape + (size_t)j * CK_F * N, bw.seg[buf], n, t0,
                         d_rewards, d_states, bw.lam, bw.gth, bw.dz[buf]);
    else
      hipLaunchKernelGGL(k_bwd_reverse<false>, dim3(nb(N, 64)), dim3(256), R_TOTAL * 4, st, c,
                         b.theta, W, tape + (size_t)j * CK_F * N, bw.seg[buf], n, t0, d_rewards,
                         d_states, bw.lam, bw.gth, bw.dz[buf]);
    BWD_TRY(hipGetLastError());
    if (overlap) {
      BWD_TRY(hipEventRecord(bw.e_rev[buf], st));
      BWD_TRY(hipStreamWaitEvent(s_dw, bw.e_rev[buf], 0));
    }
    hipLaunchKernelGGL((c.flags & F_ACTOR_BF16) ? k_bwd_dw<true> : k_bwd_dw<false>,
                       dim3(bw.dw_gx, bw.dw_groups), dim3(512), 0, s_dw, N, W, bw.seg[buf],
                       bw.dz[buf], n, K, bw.dw_groups, bw.gpart);
    BWD_TRY(hipGetLastError());
    if (overlap) BWD_TRY(hipEventRecord(bw.e_dw[buf], s_dw));
    last = buf;
  }
  if (overlap) BWD_TRY(hipStreamWaitEvent(st, bw.e_dw[last], 0));
  hipLaunchKernelGGL(k_bwd_reduce, dim3(nb(NW, DR_OUT)), dim3(DR_OUT * DR_SPLIT), 0, st, bw.gpart,
                     bw.n_parts,
                     grad_actor ? grad_actor : bw.gsum);
  if (grad_params)
    hipLaunchKernelGGL(k_copy, dim3(nb(NP * N, 256)), dim3(256), 0, st, bw.gth, grad_params,
                       (size_t)NP * N);
  return hipGetLastError();
}

hipError_t run_backward(const DevCfg& c, const SimBufs& b, BwdBufs& bw, const float* W,
                        const float* tape, int K, int T, const float* d_rewards,
                        const float* d_states, float* grad_actor, float* grad_params,
                        int held[BWD_NBUF], hipStream_t st) {
  return backward_segments(c, b, bw, false, W, tape, K, T, d_rewards, d_states, grad_actor,
                           grad_params, held, st);
}

// Layout of the scratch array in floats, every part starting on a 256-byte
// boundary: one segment record, its layer cotangents, the adjoint carry,
// the parameter gradients, the weight-gradient partials, the actor-gradient
// sink.
static inline size_t up64(size_t f) { return (f + 63) & ~(size_t)63; }

size_t bwd_scratch_floats(const BwdBufs& bw) {
  const int N = bw.N, K = bw.K;
  return up64(rec_floats(K, N)) + up64((size_t)K * DZ_F * rb_pad(N)) + up64((size_t)LAM_F * N) +
         up64((size_t)NP * N) + up64((size_t)bw.n_parts * DW_SLOT) + up64((size_t)NW);
}

hipError_t run_backward_in(const DevCfg& c, const SimBufs& b, const BwdBufs& bw, float* scratch,
                           const float* W, const float* tape, int K, int T,
                           const float* d_rewards, const float* d_states, float* grad_actor,
                           float* grad_params, hipStream_t st) {
  const int N = c.n_envs;
  BwdBufs sb = bw;  // shape, groups and device attributes of the handle's backward
  for (int i = 0; i < BWD_NBUF; ++i) sb.seg[i] = sb.dz[i] = nullptr;
  float* p = scratch;
  const size_t f_rec = rec_floats(K, N), f_dz = (size_t)K * DZ_F * rb_pad(N);
  sb.seg[0] = p;
  p += up64(f_rec);
  sb.dz[0] = p;
  p += up64(f_dz);
  sb.lam = p;
  p += up64((size_t)LAM_F * N);
  sb.gth = p;
  p += up64((size_t)NP * N);
  sb.gpart = p;
  p += up64((size_t)bw.n_parts * DW_SLOT);
  sb.gsum = p;
  // the array keeps whatever the last call on this device left in it; the
  // record and cotangent slots of envs >= N in the last 64-env block may go
  // unwritten here and must read as finite and zero
  // (k_fill: one float per thread; both sizes are below 2^31 by the
  // scratch bound the caller checked)
  hipLaunchKernelGGL(k_fill, dim3(nb((int)f_rec, 256)), dim3(256), 0, st, sb.seg[0], f_rec, 0.0f);
  hipLaunchKernelGGL(k_fill, dim3(nb((int)f_dz, 256)), dim3(256), 0, st, sb.dz[0], f_dz, 0.0f);
  BWD_TRY(hipGetLastError());
  sb.nbuf = 1;
  return backward_segments(c, b, sb, true, W, tape, K, T, d_rewards, d_states, grad_actor,
                           grad_params, nullptr, st);
}

}  // namespace qs
