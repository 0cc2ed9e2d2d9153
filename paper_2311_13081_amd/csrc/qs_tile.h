// Actor on bf16 matrix cores in 16-env tiles, shared by the tile kernel, the
// split-actor kernel and the plain step.
//
// Tile layout: lane L = li + 16 lg holds, for each 16-env tile b of the wave,
// lane group lg's share of env 16 b + li: action component lg of the 32
// history slots, and the state features 4 e + lg (e = 0..4).  That is the B
// operand of v_mfma_f32_16x16x32_bf16 (8 elements per lane):
//   chunk c = 0..3 of layer 1: element e is history slot 8 c + e (oldest
//       first), component lg;
//   chunk 4: element e < 5 is state feature 4 e + lg (p, R row-major, v, w; 0
//       past feature 17), element 5 the constant one of the bias (weight b1 in
//       lane group 0, 0 elsewhere), the rest 0;
//   chunk m of layer 2: element e is hidden unit 32 m + 16 (e / 4) + 4 lg + e %
//       4, the order in which the layer-1 result registers arrive (register r
//       of result tile n: unit 16 n + 4 lg + r of env 16 b + li).
//
// fp32 products by splitting.  An fp32 value from about 2^-110 up to bf16's
// largest is the sum of three bf16 values (its bf16 rounding, the rounding of what
// is left, and the rest: 24 bits in all, exact; smaller ones lose bits below
// 2^-133, and infinities, NaN and magnitudes that round past bf16's largest have no
// split: "No split" below), and a product of two such sums keeps the six terms down to
// 2^-16 of the leading one; the three left out are below 2^-25.  The six
// products run at 16 times the rate of the fp32 shapes, 2.7 times per fp32
// product, and overlap with vector instructions, which the fp32 shapes do
// not.  A sum takes the five small terms of all its inputs first and the
// leading ones last, so it is rounded at its own size only once per leading
// product, and biases are added at the end: against 64 bits that is closer than
// the fp32 chain (relative rms error at K = 160 6e-8 against 2.3e-7) and
// without the bias of a chain that rounds 30 times at full size (2.6 times the
// rms error, and a mean error of 1e-8 in the actions, which a closed loop turns
// into an offset).  The order of the terms is the same in every kernel, so they
// agree bit for bit.
#pragma once
#include <type_traits>

#include "qs_device.h"

namespace qs {

typedef float f4t __attribute__((ext_vector_type(4)));
typedef uint32_t u4t __attribute__((ext_vector_type(4)));
typedef __bf16 bf8t __attribute__((ext_vector_type(8)));
typedef __bf16 bf2t __attribute__((ext_vector_type(2)));
typedef float f2t __attribute__((ext_vector_type(2)));

constexpr int T_P = 3;  // bf16 parts of a value

// LDS: operand fragments of 64 lanes x 16 bytes ([group][part][lane], so a
// read is one conflict-free b128 per lane), then layer 2's and 3's biases and
// layer 3's weights.  Groups, in the order a step reads them: layer 1's history
// chunk c of unit tile n at 4 n + c, its state chunk at 16 + n, layer 2's chunk m
// of unit tile n at 20 + 2 n + m.
constexpr int T_GS = 16, T_G2 = 20, T_G = 28;
constexpr int T_W3_LD = 68;  // layer-3 row pitch: the 16-byte reads stay aligned
constexpr int T_B2 = T_G * T_P * 256, T_W3 = T_B2 + NHID, T_B3 = T_W3 + NA * T_W3_LD,
              T_TOTAL = T_B3 + 4;  // floats

// Source index (into the flat actor) of element e of lane l in group g, -1
// for padding.
__device__ inline int tile_src(int g, int l, int e) {
  const int li = l & 15, lg = l >> 4;
  if (g < T_GS) return OFF_W1 + (16 * (g >> 2) + li) * NO + 18 + NA * (8 * (g & 3) + e) + lg;
  if (g < T_G2) {
    const int unit = 16 * (g - T_GS) + li;
    if (e == 5 && lg == 0) return OFF_B1 + unit;
    return e < 5 && 4 * e + lg < 18 ? OFF_W1 + unit * NO + 4 * e + lg : -1;
  }
  const int n = (g - T_G2) >> 1, m = (g - T_G2) & 1;
  return OFF_W2 + (16 * n + li) * NHID + 32 * m + 16 * (e >> 2) + 4 * lg + (e & 3);
}

// Two fp32 values to packed bf16 (round to nearest even), first one low.
__device__ inline uint32_t pack_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2t{a, b}, bf2t));
}
__device__ inline float bf_lo(uint32_t p) { return __uint_as_float(p << 16); }
__device__ inline float bf_hi(uint32_t p) { return __uint_as_float(p & 0xffff0000u); }

// No split.  The second and third part of an infinity or NaN are NaN, so every sum of
// its env's column is NaN, of the sign that the ReLU (a maximum of the bit patterns)
// takes as zero; the columns of other envs are as without it.  For an infinite input
// that leaves finite actions, as mixed infinities do in an fp32 chain.  But a NaN input or
// weight has to give NaN actions: an env that has lost its state, or a policy that
// has diverged, would otherwise look sound.  So NaN is carried past the products: a
// lane that has one among its features (or its history at the start of a launch; a
// NaN action shows in the next step's state) makes one of its layer-2 units NaN
// (carry_nan), and with a weight that has no split every lane does, in every step.
// Four instructions a tile and step.
// (As masks of the wave's lanes, which take no vector register.)
__device__ __forceinline__ uint64_t nan_lanes(const float (&F)[5]) {
  return __ballot(__builtin_isunordered(F[0], F[1])) | __ballot(__builtin_isunordered(F[2], F[3])) |
         __ballot(F[4] != F[4]);
}
__device__ __forceinline__ void carry_nan(f4t& h2, uint64_t nan) {
  h2[0] = pick(__builtin_amdgcn_inverse_ballot_w64(nan), __uint_as_float(0x7fc00000u), h2[0]);
}
// Whether v holds in a thread of the workgroup: set_flag, a barrier, any_flag.  flags: a
// word per wave.
__device__ inline void set_flag(bool v, uint32_t* flags) {
  const uint64_t m = __ballot(v);
  if ((threadIdx.x & 63) == 0) flags[threadIdx.x >> 6] = m != 0;
}
__device__ inline bool any_flag(const uint32_t* flags) {
  const int last = (int)(blockDim.x >> 6) - 1;
  return __ballot(flags[min((int)(threadIdx.x & 63), last)] != 0) != 0;
}

// The parts of a pair of values, packed: p[0] + p[1] + p[2] is the value.
__device__ inline void split_pair(float a, float b, uint32_t p[T_P]) {
  p[0] = pack_bf16(a, b);
  a -= bf_lo(p[0]);
  b -= bf_hi(p[0]);
  p[1] = pack_bf16(a, b);
  p[2] = pack_bf16(a - bf_lo(p[1]), b - bf_hi(p[1]));
}

// Weights are looked at by their third parts, words w: bit 14 of a half is set where it
// is 2 or more, infinite or NaN (the weight 2^18 or more, or without a split), so the
// bits of a thread's share or-ed together (an instruction for three words: this is
// in every launch) mostly settle it.
__device__ inline bool maybe_unsplit(uint32_t bits) { return (bits & 0x40004000u) != 0; }
__device__ inline bool unsplit(uint32_t w) { return __builtin_isunordered(bf_lo(w), bf_hi(w)); }

// The fragment of group g of lane l, straight from the actor.
__device__ inline void load_fragment(const float* __restrict__ W, int g, int l, u4t (&a)[T_P]) {
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int s = tile_src(g, l, e);
    v[e] = W[s < 0 ? 0 : s];
    if (s < 0) v[e] = 0.0f;
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    uint32_t p[T_P];
    split_pair(v[2 * q], v[2 * q + 1], p);
#pragma unroll
    for (int s = 0; s < T_P; ++s) a[s][q] = p[s];
  }
}

// Stages n groups of fragments at dst, src(g, l, e) the source index of element e
// of lane l in group g (-1 for padding), every thread of the workgroup taking
// (group, lane) pairs, the loads of MAXT pairs in flight at a time.  bf16: the
// weights rounded to bf16 first.  False where a weight of the thread's share has no
// split.
template <int MAXT, typename Src>
__device__ inline bool stage_fragments(const float* __restrict__ W, u4t* dst, int groups, Src src,
                                       bool bf16 = false) {
  const int nt = blockDim.x, n = groups * 64;
  uint32_t third = 0;
  for (int base = threadIdx.x; base < n; base += MAXT * nt) {
    float v[MAXT][8];
#pragma unroll
    for (int j = 0; j < MAXT; ++j) {
      const int t = min(base + j * nt, n - 1);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int s = src(t >> 6, t & 63, e);
        v[j][e] = W[s < 0 ? 0 : s];
        if (s < 0) v[j][e] = 0.0f;
        if (bf16) v[j][e] = (float)(__bf16)v[j][e];
      }
    }
#pragma unroll
    for (int j = 0; j < MAXT; ++j) {
      const int t = base + j * nt;
      if (t >= n) break;
      u4t o[T_P];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint32_t p[T_P];
        split_pair(v[j][2 * q], v[j][2 * q + 1], p);
#pragma unroll
        for (int s = 0; s < T_P; ++s) o[s][q] = p[s];
      }
#pragma unroll
      for (int s = 0; s < T_P; ++s) dst[((t >> 6) * T_P + s) * 64 + (t & 63)] = o[s];
      third |= (o[2][0] | o[2][1]) | (o[2][2] | o[2][3]);
    }
  }
  bool ok = true;
  if (maybe_unsplit(third))
    for (int t = threadIdx.x; t < n; t += nt) {
      const u4t w = dst[((t >> 6) * T_P + 2) * 64 + (t & 63)];  // the thread's own
      ok = ok && !(unsplit(w[0]) || unsplit(w[1]) || unsplit(w[2]) || unsplit(w[3]));
    }
  return ok;
}

// The whole actor into LDS; false where a weight of the thread's share has no split.
__device__ inline bool stage_tile(const float* __restrict__ W, float* lds) {
  const bool ok = stage_fragments<4>(W, reinterpret_cast<u4t*>(lds), T_G, tile_src);
  for (int i = threadIdx.x; i < NHID + NA * T_W3_LD + NA; i += blockDim.x) {
    if (i < NHID) {
      lds[T_B2 + i] = W[OFF_B2 + i];
    } else if (i < NHID + NA * T_W3_LD) {
      const int r = (i - NHID) / T_W3_LD, k = (i - NHID) % T_W3_LD;
      lds[T_W3 + i - NHID] = k < NHID ? W[OFF_W3 + r * NHID + k] : 0.0f;
    } else {
      const int o = i - NHID - NA * T_W3_LD;
      lds[T_B3 + o] = W[OFF_B3 + o];
    }
  }
  return ok;
}

__device__ inline f4t mfma_bf(u4t a, u4t b, f4t c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8t, a),
                                                 __builtin_bit_cast(bf8t, b), c, 0, 0, 0);
}

// Fragments of NN unit tiles, group g + stride j for tile j.
template <int NN>
struct Frags {
  u4t a[NN][T_P];
  __device__ inline void load(const u4t* w, int g, int stride, int lane) {
#pragma unroll
    for (int j = 0; j < NN; ++j)
#pragma unroll
      for (int s = 0; s < T_P; ++s) a[j][s] = w[((g + stride * j) * T_P + s) * 64 + lane];
  }
};

// The five small terms of fragment j x operand x[b], from the smallest up, for NN
// unit tiles and TILES env tiles.
template <int NN, int TILES>
__device__ inline void small_terms(const Frags<NN>& f, const u4t (&x)[TILES][T_P],
                                   f4t (&acc)[NN][TILES]) {
  constexpr int WP[5] = {2, 0, 1, 1, 0}, XP[5] = {0, 2, 1, 0, 1};
#pragma unroll
  for (int k = 0; k < 5; ++k)
#pragma unroll
    for (int j = 0; j < NN; ++j)
#pragma unroll
      for (int b = 0; b < TILES; ++b) acc[j][b] = mfma_bf(f.a[j][WP[k]], x[b][XP[k]], acc[j][b]);
}

// The sum over CH chunks of fragment x operand: the small terms of every chunk,
// then the leading products.  frag(c): chunk c's fragments; x[c]: its operands.
template <int CH, int NN, int TILES, typename F>
__device__ inline void split_sum(F&& frag, const u4t (&x)[CH][TILES][T_P],
                                 f4t (&acc)[NN][TILES]) {
  u4t lead[CH][NN];
#pragma unroll
  for (int j = 0; j < NN; ++j)
#pragma unroll
    for (int b = 0; b < TILES; ++b) acc[j][b] = f4t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int c = 0; c < CH; ++c) {
    const Frags<NN> f = frag(c);
    small_terms<NN, TILES>(f, x[c], acc);
#pragma unroll
    for (int j = 0; j < NN; ++j) lead[c][j] = f.a[j][0];
  }
#pragma unroll
  for (int c = 0; c < CH; ++c)
#pragma unroll
    for (int j = 0; j < NN; ++j)
#pragma unroll
      for (int b = 0; b < TILES; ++b) acc[j][b] = mfma_bf(lead[c][j], x[c][b][0], acc[j][b]);
}

// Unit tiles taken together: enough independent sums (NN x TILES >= 2) for the
// matrix pipe.
template <int TILES>
constexpr int T_NN = TILES == 1 ? 2 : 1;

// The fragments of a step, read from LDS in its order, one read ahead: while
// the products of NN unit tiles run, the next ones' fragments (12 registers
// each) are on their way.
template <int TILES>
struct FragPipe {
  static constexpr int NN = T_NN<TILES>;
  const u4t* w;
  Frags<NN> next;
  // An LDS read reaches 64 KB past its address: the groups further out get an
  // address of their own, formed where it is used (hoisted out of the time loop
  // it would cost a register, or a spill).
  __device__ inline void load(int g, int stride) {
    constexpr int FAR = 20;  // T_P KB a group
    const int lane = threadIdx.x & 63;
    if (g + stride * (NN - 1) > FAR)
      next.load(w, g, stride, (int)opaque((uint32_t)lane));
    else
      next.load(w, g, stride, lane);
  }
  // read i of the step (28 / NN of them): NN = 1 every group in turn; NN = 2 the
  // history chunks of tiles 0, 1, of tiles 2, 3, the state chunks, layer 2
  __device__ inline void read(int i) {
    if constexpr (NN == 1) {
      load(i % T_G, 0);
    } else {
      i %= T_G / 2;
      const int g = i < 8 ? 8 * (i >> 2) + (i & 3)
                    : i < 10 ? T_GS + 2 * (i - 8)
                             : T_G2 + 4 * ((i - 10) >> 1) + ((i - 10) & 1);
      load(g, i < 8 ? 4 : i < 10 ? 1 : 2);
    }
  }
  __device__ inline void start(const float* lds) {
    w = reinterpret_cast<const u4t*>(lds);
    read(0);
  }
  // fragments of read i; the one after it is issued
  __device__ inline Frags<NN> take(int i) {
    const Frags<NN> f = next;
    read(i + 1);
    __builtin_amdgcn_sched_barrier(0);
    return f;
  }
};

// Operand of layer-2 chunk m from two layer-1 result tiles (ReLU applied).
__device__ inline void hidden_operand(const f4t& lo, const f4t& hi, u4t (&x)[T_P]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    uint32_t p[T_P];
    const float a = q < 2 ? lo[2 * q] : hi[2 * q - 4], b = q < 2 ? lo[2 * q + 1] : hi[2 * q - 3];
    split_pair(a, b, p);
#pragma unroll
    for (int s = 0; s < T_P; ++s) x[s][q] = p[s];
  }
}

// State operand (chunk 4) of one tile from its five features, with the constant
// one of the bias.
__device__ inline void state_operand(const float F[5], u4t (&x)[T_P]) {
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    uint32_t p[T_P];
    split_pair(F[2 * q], q < 2 ? F[2 * q + 1] : 1.0f, p);
#pragma unroll
    for (int s = 0; s < T_P; ++s) x[s][q] = p[s];
  }
#pragma unroll
  for (int s = 0; s < T_P; ++s) x[s][3] = 0u;
}

// Per-lane values V[k] of the lane's own env (k = lane group) to out[b] = V[lg]
// of env 16 b + li.  One tile: every lane group holds the same env, a
// select.  Two tiles: own env = tile lg & 1; rows 0 and 2 hold tile 0, rows 1
// and 3 tile 1, so lane groups 0, 1 offer V[0], V[1] and groups 2, 3 offer V[2],
// V[3], and one swap of odd with even rows sorts them by tile.
template <int TILES>
__device__ inline void to_tiles(const float V[4], int lg, float out[TILES]) {
  static_assert(TILES == 1 || TILES == 2, "tiles per wave");
  if constexpr (TILES == 1) {
    const float lo = pick(lg & 1, V[1], V[0]), hi = pick(lg & 1, V[3], V[2]);
    out[0] = pick(lg & 2, hi, lo);
  } else {
    const float X = pick(lg < 2, V[0], V[2]), Y = pick(lg < 2, V[1], V[3]);
    const auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(X), __float_as_uint(Y), false,
                                                    false);
    out[0] = __uint_as_float(q[0]);
    out[1] = __uint_as_float(q[1]);
  }
}

// The uniforms of the observation noise that a lane needs: those of half h of
// each of the step's five blocks (h = 0 feeds features 4 q, 4 q + 1, h = 1 the
// next two), h = lg / 2 for one tile and for two.  The lanes of an env draw
// different blocks (block 4 all of them) and swap: one tile, lane group q
// draws block q; two tiles, groups 0, 1 draw blocks 0 and 1, groups 2, 3 blocks
// 2 and 3 of the same env.
template <int TILES>
__device__ inline void noise_uniforms(const DevCfg& c, uint32_t e, uint32_t ep, int t_ep, int lg,
                                      float u0[5], float u1[5]) {
  const uint32_t base = (uint32_t)t_ep * 5u;
  float u[4];
  uniforms4(c.seed_lo, c.seed_hi, e, ep, base + 4u, STREAM_NOISE, u);
  u0[4] = pick(lg < 2, u[0], u[2]);
  u1[4] = pick(lg < 2, u[1], u[3]);
#pragma unroll
  for (int k = 0; k < TILES; ++k) {
    uniforms4(c.seed_lo, c.seed_hi, e, ep,
              base + (uint32_t)(TILES == 1 ? lg : 2 * (lg >> 1) + k), STREAM_NOISE, u);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      // halves 0 of rows 0, 1 | halves 1 of rows 0, 1, and the same of rows 2, 3
      const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(u[i]),
                                                      __float_as_uint(u[2 + i]), false, false);
      float* o = i ? u1 : u0;
      if constexpr (TILES == 1) {
        const auto a = __builtin_amdgcn_permlane16_swap(s[0], s[0], false, false);
        const auto b = __builtin_amdgcn_permlane16_swap(s[1], s[1], false, false);
        o[0] = __uint_as_float(a[0]);
        o[1] = __uint_as_float(a[1]);
        o[2] = __uint_as_float(b[0]);
        o[3] = __uint_as_float(b[1]);
      } else {
        o[k] = __uint_as_float(s[0]);
        o[2 + k] = __uint_as_float(s[1]);
      }
    }
  }
}

// The observed state features 4 q + lg (p, R row-major, v, w; 0 past the end)
// of each tile's env, with the set-point shift and the noise under EXTRAS.
// The noise costs more than the rest of the step's vector work, so a lane
// evaluates only the normals of the features it hands out: one of a pair for
// one tile, a pair for two.
// noise(zc, zs): the five pairs of normals of the lane's half.
template <int TILES, bool EXTRAS, typename Noise>
__device__ inline void tile_features(const DevCfg& c, const SetPoint& sp, const float x[NS], int lg,
                                     float (&F)[TILES][5], Noise&& noise) {
  float f[20];
  rotmat(x + 3, f + 3);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    f[i] = x[i];
    f[12 + i] = x[7 + i];
    f[15 + i] = x[10 + i];
  }
  f[18] = f[19] = 0.0f;
  if (EXTRAS) {
    sp.apply(c, f);
    if (c.flags & F_OBS_NOISE) {
      float zcs[5], zss[5];
      noise(zcs, zss);
#pragma unroll
      for (int q = 0; q < 5; ++q) {
        const float zc = zcs[q], zs = zss[q];
        // the pair 4 q + 2 h, 4 q + 2 h + 1 of this lane's half h
        const bool lo = lg < 2;
        f[4 * q] = fmaf(pick(lo, noise_std(c, 4 * q), 0.0f), zc, f[4 * q]);
        f[4 * q + 1] = fmaf(pick(lo, noise_std(c, 4 * q + 1), 0.0f), zs, f[4 * q + 1]);
        f[4 * q + 2] = fmaf(pick(lo, 0.0f, noise_std(c, 4 * q + 2)), zc, f[4 * q + 2]);
        f[4 * q + 3] = fmaf(pick(lo, 0.0f, noise_std(c, 4 * q + 3)), zs, f[4 * q + 3]);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    float o[TILES];
    to_tiles<TILES>(f + 4 * q, lg, o);
#pragma unroll
    for (int t = 0; t < TILES; ++t) F[t][q] = o[t];
  }
}

// The normals drawn by the lane itself.
template <int TILES>
__device__ inline void draw_normals(const DevCfg& c, uint32_t e, uint32_t ep, int t_ep, int lg,
                                    float zc[5], float zs[5]) {
  float u0[5], u1[5];
  noise_uniforms<TILES>(c, e, ep, t_ep, lg, u0, u1);
#pragma unroll
  for (int q = 0; q < 5; ++q) box_muller(u0[q], u1[q], zc[q], zs[q]);
}
// One of its pairs: block q of the step, the half of lane group lg.
__device__ inline float2 draw_normal_pair(const DevCfg& c, uint32_t e, uint32_t ep, int t_ep,
                                          int lg, int q) {
  float u[4];
  float2 z;
  uniforms4(c.seed_lo, c.seed_hi, e, ep, (uint32_t)t_ep * 5u + (uint32_t)q, STREAM_NOISE, u);
  box_muller(pick(lg < 2, u[0], u[2]), pick(lg < 2, u[1], u[3]), z.x, z.y);
  return z;
}

// Layer 3 (fp32 16-block 4x4x1, one product per layer-2 result register: block
// b takes that register's unit for its lane group and 4 envs as B, the
// unit's 4 output weights as A, row o = lane & 3) from the layer-2 results h2
// (ReLU applied): z3 of the lane's own env in every lane.  Each lane group
// ends with the partial sum over its units; swapping 32 lanes and adding,
// then 16 lanes and adding, completes them ((0 + 2) + (1 + 3)).
// w3[n]: weights of units 16 n + 4 lg .. + 3 for output lane & 3; b3: the bias in
// lane group 0, zero in the others.
template <int TILES>
__device__ inline void tile_layer3(const f4t w3[4], const f4t& b3, const f4t (&h2)[4][TILES],
                                   float z3[NA]) {
  f4t acc[TILES];
#pragma unroll
  for (int n = 0; n < 4; ++n) {
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int b = 0; b < TILES; ++b)
        acc[b] = __builtin_amdgcn_mfma_f32_4x4x1f32(w3[n][v], h2[n][b][v],
                                                    (n == 0 && v == 0) ? b3 : acc[b], 0, 0, 0);
  }
#pragma unroll
  for (int o = 0; o < NA; ++o) {
    uint32_t s[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const uint32_t v = __float_as_uint(acc[b % TILES][o]);
      const auto p = __builtin_amdgcn_permlane32_swap(v, v, false, false);
      s[b] = __float_as_uint(__uint_as_float(p[0]) + __uint_as_float(p[1]));
    }
    const auto q = __builtin_amdgcn_permlane16_swap(s[0], s[1], false, false);
    z3[o] = __uint_as_float(q[0]) + __uint_as_float(q[1]);
  }
}

// Layer 3's operands from LDS (rows of pitch T_W3_LD).
struct Layer3 {
  f4t w[4], b;
  __device__ inline void load(const float* w3, const float* b3) {
    const int lane = threadIdx.x & 63, lg = lane >> 4;
#pragma unroll
    for (int n = 0; n < 4; ++n)
      w[n] = *reinterpret_cast<const f4t*>(&w3[(lane & 3) * T_W3_LD + 16 * n + 4 * lg]);
#pragma unroll
    for (int r = 0; r < 4; ++r) b[r] = lg == 0 ? b3[r] : 0.0f;
  }
};

template <int NN, int TILES>
__device__ inline void relu_tiles(f4t (&a)[NN][TILES]) {
#pragma unroll
  for (int n = 0; n < NN; ++n)
#pragma unroll
    for (int b = 0; b < TILES; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) a[n][b][r] = relu_bits(a[n][b][r]);
}

// Action history of a wave's tiles: component lg of slots 2 q, 2 q + 1 packed in
// word q (of 16), one word array per part.
template <int TILES>
struct TileHist {
  u4t h[TILES][T_P][4];

  // slots (2 q, 2 q + 1) of tile b
  __device__ inline void set_pair(int b, int q, float s0, float s1) {
    uint32_t p[T_P];
    split_pair(s0, s1, p);
#pragma unroll
    for (int s = 0; s < T_P; ++s) h[b][s][q >> 2][q & 3] = p[s];
  }
  // One slot older: every slot moves down by one, p[b] (the parts of a value
  // in the low halves) becomes slot 31.
  __device__ inline void push(const uint32_t (&p)[TILES][T_P]) {
#pragma unroll
    for (int b = 0; b < TILES; ++b)
#pragma unroll
      for (int s = 0; s < T_P; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          u4t v = h[b][s][c];
          const uint32_t next = c < 3 ? (uint32_t)h[b][s][c < 3 ? c + 1 : 3][0] : p[b][s];
          v[0] = __builtin_amdgcn_alignbit(v[1], v[0], 16);
          v[1] = __builtin_amdgcn_alignbit(v[2], v[1], 16);
          v[2] = __builtin_amdgcn_alignbit(v[3], v[2], 16);
          v[3] = __builtin_amdgcn_alignbit(next, v[3], 16);
          h[b][s][c] = v;
        }
  }
  // where on[b]: every slot of the lane's env in tile b becomes v[b]
  __device__ inline void fill(const bool on[TILES], const float v[TILES]) {
#pragma unroll
    for (int b = 0; b < TILES; ++b) {
      uint32_t p[T_P];
      split_pair(v[b], v[b], p);
#pragma unroll
      for (int s = 0; s < T_P; ++s)
#pragma unroll
        for (int q = 0; q < 16; ++q)
          h[b][s][q >> 2][q & 3] = on[b] ? p[s] : h[b][s][q >> 2][q & 3];
    }
  }
  // the value of slot sl (the sum of its parts, exact; an infinity is its first part)
  __device__ inline float get(int b, int sl) const {
    const int q = sl >> 1;
    float p[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const uint32_t w = h[b][s][q >> 2][q & 3];
      p[s] = sl & 1 ? bf_hi(w) : bf_lo(w);
    }
    return pick(fabsf(p[0]) < __uint_as_float(0x7f800000u), p[0] + (p[1] + p[2]), p[0]);
  }
};

// The lanes with a NaN among their 32 history values slot(s) of a tile, of which a1 are
// layer 1's sums: these are NaN in every unit then, so most launches look no further.
template <typename Slot>
__device__ inline uint64_t nan_slots(const f4t& a1, Slot&& slot) {
  uint64_t m = 0;
  if (__builtin_expect(__ballot(a1[0] != a1[0]) != 0, 0)) {
#pragma unroll 1
    for (int s = 0; s < NH; ++s) {
      const float v = slot(s);
      m |= __ballot(v != v);
    }
  }
  return m;
}

// Layer 1's history sums of unit tiles n0 .. n0 + NN - 1.  They need the actions
// only, so a step's share is evaluated while the step before integrates its
// dynamics: the matrix products and the vector instructions of one wave
// overlap.
template <int TILES>
__device__ inline void tile_history(FragPipe<TILES>& fp, const TileHist<TILES>& H, int n0,
                                    f4t (&a1)[4][TILES]) {
  constexpr int NN = T_NN<TILES>;
  u4t x[4][TILES][T_P];
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int b = 0; b < TILES; ++b)
#pragma unroll
      for (int s = 0; s < T_P; ++s) x[c][b][s] = H.h[b][s][c];
  split_sum<4, NN, TILES>([&](int c) { return fp.take(4 * (n0 / NN) + c); }, x,
                          reinterpret_cast<f4t(&)[NN][TILES]>(a1[n0]));
}

// Layer 1's history sums a1 of the envs that reset (on[b]: the lane's env of tile b)
// and whose history is now the hover action aht[b] throughout.  A column of a
// product depends on its own env only, so one pass of products serves the resets of
// both tiles wherever no two share a column (else a second pass), and its sums are
// those tile_history would form.  Half the products of doing two tiles again: 1000
// steps of 65536 envs of which one in 32 resets in 40% of the wave-steps, 11.35 ->
// 10.2 ms.
template <int TILES>
__device__ inline void reset_history(const float* lds, const bool (&on)[TILES],
                                     const float (&aht)[TILES], f4t (&a1)[4][TILES]) {
  const u4t* w = reinterpret_cast<const u4t*>(lds);
  const int lane = threadIdx.x & 63;
  bool todo[TILES];
#pragma unroll
  for (int b = 0; b < TILES; ++b) todo[b] = on[b];
  bool more;
  do {
    // the first of the lane's tiles that is still to do
    bool take[TILES], left = false;
    float ah = 0.0f;
    bool used = false;
#pragma unroll
    for (int b = 0; b < TILES; ++b) {
      take[b] = todo[b] && !used;
      used = used || take[b];
      ah = pick(take[b], aht[b], ah);
      todo[b] = todo[b] && !take[b];
      left = left || todo[b];
    }
    more = __ballot(left) != 0;
    uint32_t p[T_P];
    split_pair(ah, ah, p);
    u4t x[4][1][T_P];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int s = 0; s < T_P; ++s) x[c][0][s] = u4t{p[s], p[s], p[s], p[s]};
#pragma unroll
    for (int n = 0; n < 4; n += 2) {
      f4t acc[2][1];
      split_sum<4, 2, 1>(
          [&](int c) {
            __builtin_amdgcn_sched_barrier(0);  // (registers: one chunk's reads at a time)
            Frags<2> f;
            f.load(w, 4 * n + c, 4, lane);
            return f;
          },
          x, acc);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int b = 0; b < TILES; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r) a1[n + j][b][r] = pick(take[b], acc[j][0][r], a1[n + j][b][r]);
    }
  } while (more);
}

// The rest of the actor for the wave's tiles: z3 (pre-tanh) of the lane's own
// env in every lane.  a1: layer 1's history sums (consumed); F: the state
// features 4 e + lg of each tile's env.  rec takes the layer results before the
// ReLU (the record of taped rollouts).  lost: lanes that carry_nan whatever their
// features are.
template <int TILES, typename Rec>
__device__ inline void tile_actor(const float* lds, FragPipe<TILES>& fp, f4t (&a1)[4][TILES],
                                  const float (&F)[TILES][5], const uint64_t (&lost)[TILES],
                                  float z3[NA], Rec&& rec) {
  constexpr int NN = T_NN<TILES>;
  const int lg = (int)opaque((threadIdx.x & 63) >> 4);
  // (with a record the features are kept anyway, and are looked at where the mask is
  // used)
  constexpr bool LATE = std::remove_reference_t<Rec>::KEEPS_FEATURES;
  uint64_t nan[TILES];
#pragma unroll
  for (int b = 0; b < TILES; ++b)
    if (!LATE) nan[b] = lost[b] | nan_lanes(F[b]);
  {
    u4t x[1][TILES][T_P];
#pragma unroll
    for (int b = 0; b < TILES; ++b) state_operand(F[b], x[0][b]);
#pragma unroll
    for (int n = 0; n < 4; n += NN) {
      f4t as[NN][TILES];
      split_sum<1, NN, TILES>([&](int) { return fp.take((T_GS + n) / NN); }, x, as);
#pragma unroll
      for (int j = 0; j < NN; ++j)
#pragma unroll
        for (int b = 0; b < TILES; ++b) a1[n + j][b] += as[j][b];
    }
  }
  rec.layer1(a1);
  relu_tiles(a1);
  f4t a2[4][TILES];
  {
    u4t x[2][TILES][T_P];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int b = 0; b < TILES; ++b) hidden_operand(a1[2 * m][b], a1[2 * m + 1][b], x[m][b]);
#pragma unroll
    for (int n = 0; n < 4; n += NN) {
      split_sum<2, NN, TILES>([&](int m) { return fp.take((T_G2 + 2 * n) / NN + m); }, x,
                              reinterpret_cast<f4t(&)[NN][TILES]>(a2[n]));
#pragma unroll
      for (int j = 0; j < NN; ++j) {
        const f4t b2 = *reinterpret_cast<const f4t*>(&lds[T_B2 + 16 * (n + j) + 4 * lg]);
#pragma unroll
        for (int b = 0; b < TILES; ++b) a2[n + j][b] += b2;
      }
    }
  }
  rec.layer2(a2);
  relu_tiles(a2);
#pragma unroll
  for (int b = 0; b < TILES; ++b) {
    if (LATE) nan[b] = lost[b] | nan_lanes(F[b]);
    carry_nan(a2[0][b], nan[b]);
  }
  Layer3 l3;
  l3.load(lds + T_W3, lds + T_B3);
  tile_layer3<TILES>(l3.w, l3.b, a2, z3);
}

// No record.
struct NoRec {
  static constexpr bool KEEPS_FEATURES = false;
  template <typename A>
  __device__ inline void layer1(const A&) {}
  template <typename A>
  __device__ inline void layer2(const A&) {}
};

// ReLU mask word of a record (row REC_M + lg of the env's column, lg the
// lane group): bit 8 n + r is set when layer-1 unit 16 n + 4 lg + r of the
// env has a positive pre-activation, bit 8 n + 4 + r the same for layer 2.
// z: the lane's result tiles of one layer; layer 2's bits are these << 4.
template <int TILES>
__device__ inline uint32_t tile_mask(const f4t (&z)[4][TILES], int b) {
  uint32_t m = 0u;
#pragma unroll
  for (int n = 0; n < 4; ++n)
#pragma unroll
    for (int r = 0; r < 4; ++r) m |= (z[n][b][r] > 0.0f ? 1u : 0u) << (8 * n + r);
  return m;
}

}  // namespace qs
