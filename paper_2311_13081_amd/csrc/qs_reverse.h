// Reverse of one env step's dynamics, shared by the reverse sweeps of every
// lane layout (qs_backward.hip, qs_reverse1.hip).
#pragma once
#include "qs_device.h"
#include "qs_tile.h"

namespace qs {

// Layer cotangents per (step, env): dz1, then dz3 at DZ_3.  dz2 follows from dz3,
// the masks and layer 3 (k_bwd_dw); its rows between the two stay unused, which
// keeps the size of the caller's scratch array.
constexpr int DZ_3 = 2 * NHID, DZ_F = DZ_3 + NA;

// Of half the envs (32..63 of a 64-env block, k_bwd_dw's second slab pair) the
// cotangents are those of the negated loss, from dz3 to do: dz_sign at dz3, again
// where do joins the adjoints, and k_bwd_dw takes the halves' difference.  A bf16
// matrix product drops what lies far below its largest term toward minus infinity
// (0.007 units in the last place in the mean, whatever the signs), the same way in
// every product, and a recurrence of a hundred steps keeps it: parameter gradients of
// 128 steps 5.6e-7 off in their median, now 9e-9; actor gradients, where it adds up
// over the envs, 1.14e-7 off at 16384 envs x 32 steps, now 1.06e-7.
__device__ inline float dz_sign(int env) { return (env & 32) ? -1.0f : 1.0f; }

constexpr int LAM_F = NS + NH * NA;     // state and history adjoints carried between segments

// v where bit b of the mask word m is set, +0 elsewhere (the sign-extended
// one-bit field is all ones or zero)
__device__ inline float keep_if(float v, uint32_t m, int b) {
  return __uint_as_float(__float_as_uint(v) & (uint32_t)__builtin_amdgcn_sbfe((int)m, b, 1));
}

// The actor's transposed layers as fragments of 16 outputs (qs_tile.h's operand
// layout, products and order of terms): dz1 = W2^T dz2, output tile mt, chunk m
// (units 32 m + ..) at group 2 mt + m; do = W1^T dz1, output tile p, chunk m at 8
// + 2 p + m.  feat(p, i): the observation feature of row i of tile p (-1: none).
constexpr int RT_G1 = 8, RT_G = RT_G1 + 20, RT_FRAGS = RT_G * T_P * 64;  // u4t
template <typename Feat>
__device__ inline void stage_transposed(const float* __restrict__ W, u4t* dst, Feat feat,
                                        bool bf16) {
  stage_fragments<4>(
      W, dst, RT_G,
      [feat](int g, int l, int e) {
        const int li = l & 15, unit = 32 * (g & 1) + 16 * (e >> 2) + 4 * (l >> 4) + (e & 3);
        if (g < RT_G1) return OFF_W2 + unit * NHID + 16 * (g >> 1) + li;
        const int f = feat((g - RT_G1) >> 1, li);
        return f >= 0 ? OFF_W1 + unit * NO + f : -1;
      },
      bf16);
}
// Both chunks of NN output tiles whose fragments start at group g.
template <int NN, int TILES>
__device__ inline void transposed_sum(const u4t* w, int g, int lane, const u4t (&x)[2][TILES][T_P],
                                      f4t (&acc)[NN][TILES]) {
  split_sum<2, NN, TILES>(
      [&](int m) {
        Frags<NN> f;
        f.load(w, g + m, 2, lane);
        return f;
      },
      x, acc);
}

// Cotangents of step t for env byte offset ve = 4 e; a null pointer reads as zero
// (an empty buffer), with no branch: at a join the waits count every load and
// store of either side, so a load under one would be waited for at once.  The
// reward's cotangent defaults to one, at its use.
__device__ __forceinline__ void load_cotangents(float dS[NS], float& dR,
                                                const float* __restrict__ d_rewards,
                                                const float* __restrict__ d_states, int t, int N,
                                                uint32_t ve) {
  const uint32_t row = 4u * (uint32_t)N;
  const __amdgpu_buffer_rsrc_t rr = span_rsrc(
      d_rewards ? d_rewards + (size_t)t * N : nullptr, d_rewards ? row : 0u);
  const __amdgpu_buffer_rsrc_t rs = span_rsrc(
      d_states ? d_states + (size_t)t * NS * N : nullptr, d_states ? NS * row : 0u);
  dR = bld1(rr, ve, 0);
#pragma unroll
  for (int i = 0; i < NS; ++i) dS[i] = bld1(rs, ve, (uint32_t)i * row);
}
// Step sizes of the reverse step, in scalar registers.
struct RevStep {
  float h, hh, h6, h26;  // h, h / 2, h / 6, h^2 / 6
};
__device__ inline float wave_const(float v) {
  return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v)));
}
__device__ inline RevStep make_rev_step(const DevCfg& c) {
  const float h6 = wave_const(c.dt / 6.0f);
  return {c.dt, 0.5f * c.dt, h6, c.dt * h6};
}
// A body whose members the compiler takes as given: it otherwise moves their
// divisions into the time loop.
__device__ inline Quad make_rev_quad(const DevCfg& c, const float th[NP], const float d[6]) {
  Quad q = make_quad(c, th);
  set_disturbance(q, d);
  __asm__ volatile("" : "+v"(q.inv_m), "+v"(q.inv_Tm), "+v"(q.inv_J[0]), "+v"(q.inv_J[1]), "+v"(q.inv_J[2]));
  __asm__ volatile("" : "+v"(q.kx), "+v"(q.ky), "+v"(q.kz), "+v"(q.ax), "+v"(q.ay), "+v"(q.az));
  return q;
}

// A stage of the recomputed step: attitude, body rates, rotor speeds, and of its
// right-hand side the rates' derivative, F / m and 1 / |q|^2.
struct Stage {
  float q[4], o[3], w[4];
  float dw[3], fm, rn2;
};
// Sums over the stages of a step that the parameter gradients are formed from.
struct ThetaSums {
  float m = 0.0f, U[3] = {0.0f, 0.0f, 0.0f}, A[3] = {0.0f, 0.0f, 0.0f};
  float c0 = 0.0f, c1 = 0.0f, c2 = 0.0f, Tm = 0.0f;
};

// Right-hand side at s (quad_rhs's rows), keeping what its reverse reads.
__device__ __forceinline__ void stage_rhs(const Quad& B, float g, Stage& s, float k[10]) {
  quad_rhs<true>(B, g, s.q, s.o, s.w, k, &s.fm, &s.rn2);
#pragma unroll
  for (int i = 0; i < 3; ++i) s.dw[i] = k[7 + i];
}

// Vector-Jacobian product of the right-hand side at s for the cotangents gq, gv,
// go, gw of q', v', o' and w': adds to sq, so, sw and to gu (the actions' share,
// over 1 / Tm) and the parameter sums.  (p' = v is left to the caller.)
__device__ __forceinline__ void stage_vjp(const Quad& B, const Stage& s, const float u[NA],
                                          const float gq[4], const float gv[3], const float go[3],
                                          const float gw[4], float sq[4], float so[3], float sw[4],
                                          float gu[NA], ThetaSums& t) {
  const float *q = s.q, *o = s.o, *w = s.w;
  // q' = 1/2 q (x) (0, o)
  float hg[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) hg[i] = 0.5f * gq[i];
  sq[0] = fmaf(hg[1], o[0], fmaf(hg[2], o[1], fmaf(hg[3], o[2], sq[0])));
  sq[1] = fmaf(-hg[0], o[0], fmaf(-hg[2], o[2], fmaf(hg[3], o[1], sq[1])));
  sq[2] = fmaf(-hg[0], o[1], fmaf(hg[1], o[2], fmaf(-hg[3], o[0], sq[2])));
  sq[3] = fmaf(-hg[0], o[2], fmaf(-hg[1], o[1], fmaf(hg[2], o[0], sq[3])));
  so[0] = fmaf(-hg[0], q[1], fmaf(hg[1], q[0], fmaf(hg[2], q[3], fmaf(-hg[3], q[2], so[0]))));
  so[1] = fmaf(-hg[0], q[2], fmaf(-hg[1], q[3], fmaf(hg[2], q[0], fmaf(hg[3], q[1], so[1]))));
  so[2] = fmaf(-hg[0], q[3], fmaf(hg[1], q[2], fmaf(-hg[2], q[1], fmaf(hg[3], q[0], so[2]))));
  // v' = sc P(q) - g e_z + f / m, P = (2(xz+wy), 2(yz-wx), ww+zz-xx-yy), sc = F / (m |q|^2)
  const float px = fmaf(q[1], q[3], q[0] * q[2]), py = fmaf(q[2], q[3], -(q[0] * q[1]));
  const float pz = fmaf(q[0], q[0], fmaf(q[3], q[3], fmaf(-q[1], q[1], -(q[2] * q[2]))));
  const float gsc = fmaf(gv[2], pz, 2.0f * fmaf(gv[0], px, gv[1] * py));
  const float sc = s.fm * s.rn2, s2 = sc + sc;
  const float a0 = s2 * gv[0], a1 = s2 * gv[1], a2 = s2 * gv[2];
  const float k2 = (gsc * s2) * s.rn2;  // from sc's 1 / |q|^2
  sq[0] = fmaf(a0, q[2], fmaf(-a1, q[1], fmaf(a2, q[0], fmaf(-k2, q[0], sq[0]))));
  sq[1] = fmaf(a0, q[3], fmaf(-a1, q[0], fmaf(-a2, q[1], fmaf(-k2, q[1], sq[1]))));
  sq[2] = fmaf(a0, q[0], fmaf(a1, q[3], fmaf(-a2, q[2], fmaf(-k2, q[2], sq[2]))));
  sq[3] = fmaf(a0, q[1], fmaf(a1, q[2], fmaf(a2, q[3], fmaf(-k2, q[3], sq[3]))));
  const float gF = (gsc * B.inv_m) * s.rn2;
  t.m = fmaf(gsc, sc, fmaf(gv[0], B.f[0], fmaf(gv[1], B.f[1], fmaf(gv[2], B.f[2], t.m))));
  // o' = tau / J - k o o (gyroscopic)
  const float Gx = B.kx * go[0], Gy = B.ky * go[1], Gz = B.kz * go[2];
  so[0] = fmaf(-Gy, o[2], fmaf(-Gz, o[1], so[0]));
  so[1] = fmaf(-Gx, o[2], fmaf(-Gz, o[0], so[1]));
  so[2] = fmaf(-Gx, o[1], fmaf(-Gy, o[0], so[2]));
  t.A[0] = fmaf(go[0], o[1] * o[2], t.A[0]);
  t.A[1] = fmaf(go[1], o[2] * o[0], t.A[1]);
  t.A[2] = fmaf(go[2], o[0] * o[1], t.A[2]);
#pragma unroll
  for (int i = 0; i < 3; ++i) t.U[i] = fmaf(go[i], s.dw[i], t.U[i]);
  // torques and collective thrust -> rotor thrusts (their sum is 4 gF)
  const float gA = B.ax * go[0], gB = B.ay * go[1];
  const float a = fmaf(-B.az, go[2], gF), b = fmaf(B.az, go[2], gF), p = gA + gB, m = gA - gB;
  const float gT[4] = {a - p, b - m, a + p, b + m};
  t.c0 += gF;
  // thrust curve T = c0 + c1 w + c2 w^2, motor lag w' = (u - w) / Tm
  const float d2 = B.c2 + B.c2;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float gTw = gT[i] * w[i];
    t.c1 += gTw;
    t.c2 = fmaf(gTw, w[i], t.c2);
    sw[i] = fmaf(gT[i], fmaf(d2, w[i], B.c1), fmaf(-B.inv_Tm, gw[i], sw[i]));
    gu[i] += gw[i];
    t.Tm = fmaf(gw[i], u[i] - w[i], t.Tm);
  }
}

// Reverse of one step's dynamics: recomputes the RK4 stages from the recorded
// state x and action a, then steps back through the reward, the quaternion
// renormalisation and the four stages.  In: ls (state adjoint after the
// step), hn (adjoint of the newest history slot, i.e. of a).
// Out: gx (state adjoint before the step, without the observation's share),
// ga (action adjoint, the history coupling included); gth accumulates the
// parameter gradients d/d(m, Jxx, Jyy, Jzz, c0, c1, c2, Tm).
//
// Bound by vector-ALU issue (it is most of a sweep's instructions), so the
// forward's shape is used: what enters the velocity rows reaches nothing but the
// position, whose adjoint passes all stages unchanged, so their stage cotangents
// are closed forms of h; each stage keeps five values of its right-hand side for
// its reverse; parameter gradients are scaled once a step, from sums.  About 250
// instructions a step fewer than the plain product rule over four right-hand
// sides (1390 to 1140).
__device__ __forceinline__ void reverse_dynamics(const DevCfg& c, const RevStep& rs, const Quad& B,
                                                 bool renorm, const float x[NS],
                                                 const float a[NA], float dR, const float ls[NS],
                                                 const float hn[NA], float gx[NS], float ga[NA],
                                                 float gth[NP]) {
  const float h = rs.h, hh = rs.hh, h6 = rs.h6;
  float u[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) u[i] = fmaf(a[i] + 1.0f, c.rpm_half_range, c.rpm_min);
  Stage st[4];
  float k[10], sum[10], sv[3];  // of the stages; the first three's velocity rows
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    st[0].q[i] = x[3 + i];
    st[0].w[i] = x[13 + i];
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) st[0].o[i] = x[10 + i];
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    stage_rhs(B, c.g, st[n], k);
#pragma unroll
    for (int i = 0; i < 10; ++i)
      sum[i] = n == 0 ? k[i] : n == 3 ? sum[i] + k[i] : fmaf(2.0f, k[i], sum[i]);
    if (n == 3) break;
#pragma unroll
    for (int i = 0; i < 3; ++i) sv[i] = n == 0 ? k[4 + i] : sv[i] + k[4 + i];
    const float hs = n == 2 ? h : hh;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      st[n + 1].q[i] = fmaf(hs, k[i], x[3 + i]);
      st[n + 1].w[i] = fmaf(hs * B.inv_Tm, u[i] - st[n].w[i], x[13 + i]);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) st[n + 1].o[i] = fmaf(hs, k[7 + i], x[10 + i]);
  }
  // post-step state (renormalised): position, attitude, velocity, rates
  float sp[3], sn[10];
#pragma unroll
  for (int i = 0; i < 3; ++i) sp[i] = x[i] + fmaf(rs.h26, sv[i], h * x[7 + i]);
#pragma unroll
  for (int i = 0; i < 10; ++i) sn[i] = fmaf(h6, sum[i], x[3 + i]);
  float rn = 1.0f;
  if (renorm) {
    // the forward's reciprocal square root (rk4_step)
    rn = rsqrt_r(fmaf(sn[0], sn[0], fmaf(sn[1], sn[1], fmaf(sn[2], sn[2], sn[3] * sn[3]))));
#pragma unroll
    for (int i = 0; i < 4; ++i) sn[i] *= rn;
  }

  // --- reward and history coupling -----------------------------------------
  float g[NS];
  const float r2 = -2.0f * dR, rp = c.C_rp * r2, rv = c.C_rv * r2, rw = c.C_rw * r2,
              ra = c.C_ra * r2;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    g[i] = fmaf(rp, sp[i], ls[i]);
    g[7 + i] = fmaf(rv, sn[4 + i], ls[7 + i]);
    g[10 + i] = fmaf(rw, sn[7 + i], ls[10 + i]);
  }
  g[3] = fmaf(-(c.C_rq * r2), sn[0], ls[3]);
#pragma unroll
  for (int i = 4; i < 7; ++i) g[i] = ls[i];
#pragma unroll
  for (int i = 13; i < NS; ++i) g[i] = ls[i];
  // the newest history slot's adjoint joins the action's
#pragma unroll
  for (int i = 0; i < NA; ++i) ga[i] = fmaf(ra, a[i] - c.C_rab, hn[i]);

  // --- renormalisation ------------------------------------------------------
  if (renorm) {
    const float d = fmaf(sn[0], g[3], fmaf(sn[1], g[4], fmaf(sn[2], g[5], sn[3] * g[6])));
#pragma unroll
    for (int i = 0; i < 4; ++i) g[3 + i] = fmaf(-sn[i], d, g[3 + i]) * rn;
  }

  // --- RK4 stages in reverse ----------------------------------------------
  // rows: attitude 0..3, rates 4..6, rotors 7..10
  float gk[11], gu[NA] = {0.0f, 0.0f, 0.0f, 0.0f}, gv1[3], gv2[3], gv4[3];
  ThetaSums t;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    // h as six sixths, as the forward adds them: h / 6 is rounded, and the same way
    // in every step (2.3e-8 low for h = 0.01), so with h itself here the actor
    // gradients of 48 steps at 65536 envs are off by 1.6e-7 instead of 1.3e-7
    const float p6 = h6 * g[i];
    gx[i] = g[i];
    gx[7 + i] = fmaf(6.0f, p6, g[7 + i]);
    gv4[i] = h6 * g[7 + i];
    gv1[i] = fmaf(h, p6, gv4[i]);
    gv2[i] = gv4[i] + gv1[i];  // stages 2 and 3
  }
  constexpr auto row = [](int i) { return i < 4 ? 3 + i : 6 + i; };
  // The stages' shares, h times smaller than the adjoint they go to, are summed by
  // themselves: added to it term by term, each term is rounded at the adjoint's size
  // (parameter gradients of 128 steps at 16384 envs off by 6.0e-6 instead of 3.0e-6).
  float acc[11];
#pragma unroll
  for (int i = 0; i < 11; ++i) gk[i] = h6 * g[row(i)];
#pragma unroll
  for (int n = 3; n >= 0; --n) {
    float gs[11];
#pragma unroll
    for (int i = 0; i < 11; ++i) gs[i] = n == 0 ? acc[i] : 0.0f;
    stage_vjp(B, st[n], u, gk, n == 3 ? gv4 : n == 0 ? gv1 : gv2, gk + 4, gk + 7, gs, gs + 4,
              gs + 7, gu, t);
    const float hs = n == 3 ? h : hh;  // the step to this stage's state
    const float hg = n >= 2 ? h6 + h6 : h6;
#pragma unroll
    for (int i = 0; i < 11; ++i) {
      if (n == 0) {
        gx[row(i)] = g[row(i)] + gs[i];
      } else {
        acc[i] = n == 3 ? gs[i] : acc[i] + gs[i];
        gk[i] = fmaf(hs, gs[i], hg * g[row(i)]);
      }
    }
  }
  const float gs = c.rpm_half_range * B.inv_Tm;
#pragma unroll
  for (int i = 0; i < NA; ++i) ga[i] = fmaf(gu[i], gs, ga[i]);
  const float A0 = B.inv_J[0] * t.A[0], A1 = B.inv_J[1] * t.A[1], A2 = B.inv_J[2] * t.A[2];
  gth[0] = fmaf(-B.inv_m, t.m, gth[0]);
  gth[1] += fmaf(-B.inv_J[0], t.U[0], A2 - A1);
  gth[2] += fmaf(-B.inv_J[1], t.U[1], A0 - A2);
  gth[3] += fmaf(-B.inv_J[2], t.U[2], A1 - A0);
  gth[4] = fmaf(4.0f, t.c0, gth[4]);
  gth[5] += t.c1;
  gth[6] += t.c2;
  gth[7] = fmaf(-(B.inv_Tm * B.inv_Tm), t.Tm, gth[7]);
}

}  // namespace qs
