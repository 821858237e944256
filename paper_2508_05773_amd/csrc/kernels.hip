// gfx950 kernels of one BR-MPPI control update (arXiv 2508.05773).
//
//   k_noise   : Philox4x32-10 + Box-Muller normals of every (sample, step)
//               in parallel (for the rollout variants that read them).
//   k_rollout : S rollouts of the tractor-trailer model, each step projected
//               onto the barrier-rate equalities (eq. (9)) with the
//               soft-bound closed form (eqs. (11)-(12)), contouring cost
//               (eqs. (13)-(15)) accumulated; writes the applied inputs
//               [3T][S] and the cost of every sample.  One or several lanes
//               per sample; noise drawn in the kernel or read from k_noise.
//               k_rollout_drawn: up to 8192 samples, the update's only launch;
//               k_rollout_batch: the tiles of a batch from one queue.
//   k_reduce  : weights exp(-(J - m)/lambda) (Sec. III-B) and the weighted
//               average of the applied inputs (eq. (5)) from HBM, in units of
//               32 samples and groups of 32 units merged by log-sum-exp; the
//               last block writes the new nominal sequence, the receding-
//               horizon shift and, on request, a closed-loop FP64 plant step
//               (eq. (6)).  A single-instance rollout whose tiles are whole
//               units does the same reduction itself from LDS (fused
//               epilogue): the applied inputs then never reach HBM.
//
// A sample's state, barrier rates and row terms stay in registers.  Obstacles
// (with their shape matrices) and a window of the path are staged in LDS per
// tile.  Positions are carried relative to the start position, headings to the
// quarter turn nearest the start heading and progress to the start progress, so
// that FP32 keeps sub-micrometre resolution far from the origin.
#include <math.h>

#include <type_traits>

#include "brmppi_internal.h"

namespace brm {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): 10 rounds of two 32x32->64 products,
// Weyl-sequence key schedule.
// ---------------------------------------------------------------------------
// a ^ b ^ c in one instruction (the compiler forms two)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t out[4]) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * (uint64_t)c0;
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * (uint64_t)c2;
    const uint32_t n0 = xor3((uint32_t)(p1 >> 32), c1, k0);
    const uint32_t n2 = xor3((uint32_t)(p0 >> 32), c3, k1);
    c1 = (uint32_t)p1;
    c3 = (uint32_t)p0;
    c0 = n0;
    c2 = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  out[0] = c0;
  out[1] = c1;
  out[2] = c2;
  out[3] = c3;
}

// (r >> 9 + 1/2) / 2^23, exact in FP32: r's top 23 bits as the mantissa of a
// value in [1, 2), less 1 - 2^-24.  Two instructions; a shift, a conversion and a
// multiply-add cost the batched rollout, which draws as it goes, 2 % more (64 instances
// 731 -> 717 us).
__device__ __forceinline__ float unif23(uint32_t r) {
  return __uint_as_float(__builtin_amdgcn_alignbit(0x7fu, r, 9)) - (1.0f - 0x1p-24f);
}

// Box-Muller on the pairs (u0, u1) and (u2, u3): radius sqrt(-2 ln u0),
// angle 2 pi u1.  The uniforms lie in [2^-24, 1), so the hardware log2,
// square root, sine and cosine need none of the library's range reduction or
// special cases; the hardware sine and cosine take the angle in revolutions,
// so 2 pi u1 is never rounded.  Over all 2^23 uniforms the radius is within
// 4.9e-7 and the sine and cosine within 1.3e-7 of the exact values.
constexpr float kLn2 = 0.693147182f;
__device__ __forceinline__ float bm_radius(float u) {
  return __builtin_amdgcn_sqrtf(-2.0f * kLn2 * __builtin_amdgcn_logf(u));
}
__device__ __forceinline__ void box_muller4(const uint32_t r[4], float* n) {
  const float u0 = unif23(r[0]), u1 = unif23(r[1]), u2 = unif23(r[2]), u3 = unif23(r[3]);
  const float rad0 = bm_radius(u0), rad1 = bm_radius(u2);
  n[0] = rad0 * __builtin_amdgcn_cosf(u1);
  n[1] = rad0 * __builtin_amdgcn_sinf(u1);
  n[2] = rad1 * __builtin_amdgcn_cosf(u3);
  n[3] = rad1 * __builtin_amdgcn_sinf(u3);
}

__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// Loads and stores through global-address-space pointers.  Pointers read from
// a descriptor are generic, and a generic (flat) access also counts against
// the LDS/scalar wait counter: every wait for an LDS or scalar result would
// then wait for the step-ahead HBM loads as well.
typedef float gvec4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float gld(const float* p) {
  return *(const __attribute__((address_space(1))) float*)p;
}
__device__ __forceinline__ float4 gld4(const float4* p) {
  const gvec4 v = *(const __attribute__((address_space(1))) gvec4*)p;
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void gst(float* p, float v) { *(__attribute__((address_space(1))) float*)p = v; }
// LDS reads and writes through local-address-space pointers (and gst4, a
// 16-byte global store).  The instance merge is a function of its own, not
// inlined into the kernel, where a pointer argument is generic: a generic
// access to LDS compiles to a flat access, which is slower and counts against
// both wait counters.  Every pointer passed to the LDS helpers points into LDS.
typedef __attribute__((address_space(3))) float lds_float;
typedef __attribute__((address_space(3))) double lds_double;
typedef __attribute__((address_space(3))) gvec4 lds_vec4;
__device__ __forceinline__ float lds(const float* p) { return *(const lds_float*)p; }
__device__ __forceinline__ double lds(const double* p) { return *(const lds_double*)p; }
__device__ __forceinline__ float4 lds(const float4* p) {
  const gvec4 v = *(const lds_vec4*)p;
  return make_float4(v.x, v.y, v.z, v.w);
}
// the first three floats of a 16-byte entry (one ds_read_b96: a fourth register
// would be written late, and its next use would wait for the read)
typedef float gvec3 __attribute__((ext_vector_type(3)));
struct Vec3 {
  float x, y, z;
};
__device__ __forceinline__ Vec3 lds3(const float4* p) {
  const gvec3 v = *(const __attribute__((address_space(3))) gvec3*)p;
  return Vec3{v.x, v.y, v.z};
}
__device__ __forceinline__ void lds_put(float* p, float v) { *(lds_float*)p = v; }
__device__ __forceinline__ void lds_put(double* p, double v) { *(lds_double*)p = v; }
__device__ __forceinline__ void lds_put(float4* p, float4 v) {
  gvec4 w;
  w.x = v.x;
  w.y = v.y;
  w.z = v.z;
  w.w = v.w;
  *(lds_vec4*)p = w;
}
__device__ __forceinline__ void gst4(float4* p, float4 v) {
  gvec4 w;
  w.x = v.x;
  w.y = v.y;
  w.z = v.z;
  w.w = v.w;
  *(__attribute__((address_space(1))) gvec4*)p = w;
}

// Per-lane choices inside the step are written as selects marked
// unpredictable, so that the compiler keeps them as lane selects instead of
// divergent branches (each of which costs exec-mask instructions and splits
// the step into separately scheduled regions).
__device__ __forceinline__ float sel(bool c, float a, float b) { return __builtin_unpredictable(c) ? a : b; }
// The same with the lane mask in a scalar register pair, for several selects
// under one mask: runs of v_cndmask that read vcc were measured at 16 cycles
// each as soon as four waves run on a CU, the form with another mask at 4.
__device__ __forceinline__ float sel_mask(uint64_t mask, float a, float b) {
  float r;
  asm("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(r) : "v"(b), "v"(a), "s"(mask));
  return r;
}

// Units of the rollout.  Time is counted in steps and angles in revolutions: vh = Ts
// v and ah = Ts^2 a are metres a step, the inputs act as Ts^3 j on ah and Ts omega on
// the steer angle, and the step needs no multiplication by Ts.  Revolutions are what
// the hardware sine and cosine take, and wrapping one is x - rint(x).  Progress stays
// in metres: counted in waypoints it is rounded at another place of its binade, 7 % more
// error of the costs over the long route's 100 steps.
constexpr float kTurn = 6.283185307179586f;      // radians a revolution
constexpr float kInvTurn = 0.15915494309189535f;
constexpr float kInvTurnLo = (float)(0.15915494309189535 - (double)kInvTurn);
__device__ __forceinline__ float wrap_rev(float x) { return x - rintf(x); }
// absolute error of order 1e-7 (the Box-Muller check over [0, 1) revolutions)
__device__ __forceinline__ void sincos_rev(float x, float* s, float* c) {
  *s = __builtin_amdgcn_sinf(x);
  *c = __builtin_amdgcn_cosf(x);
}

// Frame of a rollout: its origin is the start position, and its axes are turned by
// the quarter turns (c, s: the cosine and sine of `turn`, 0 and +-1) nearest the start
// heading, so that headings are small.  A quarter turn moves no bit of a coordinate;
// in revolutions an angle just past one is held to 1.9e-7 rad, where radians hold it to
// 1.2e-7, and a vehicle that parks along an axis has its heading there (costs of 3000
// samples, 40 steps, 8 vehicles in a bay, against FP64, over 16 scenes: 2.6e-7 with the
// path's axes, 2.2e-7 in radians, 1.6e-7 with these).
struct Frame {
  float ox, oy, turn, c, s;
};
__device__ __forceinline__ Frame frame_at(float px, float py, float th1) {
  Frame F;
  F.ox = px;
  F.oy = py;
  const float q = rintf(4.0f * kInvTurn * th1);
  F.turn = 0.25f * q;
  // q mod 4, in -2 .. 2 (any q that FP32 holds; a non-finite heading makes the
  // sample's cost non-finite whatever the axes are)
  const float m = fmaf(-4.0f, rintf(F.turn), q);
  F.c = m == 0.0f ? 1.0f : (fabsf(m) == 2.0f ? -1.0f : 0.0f);
  F.s = m == 1.0f ? 1.0f : (m == -1.0f ? -1.0f : 0.0f);
  return F;
}
__device__ __forceinline__ void into_frame(const Frame& F, float& x, float& y) {
  const float a = fmaf(F.s, y, F.c * x), b = fmaf(F.c, y, -(F.s * x));
  x = a;
  y = b;
}
// an angle in radians, in revolutions from the frame's axis
__device__ __forceinline__ float into_frame(const Frame& F, float th) {
  return fmaf(th, kInvTurnLo, fmaf(th, kInvTurn, -F.turn));
}
// the same less whole turns, which are found before the result is rounded
__device__ __forceinline__ float into_frame_wrapped(const Frame& F, float th) {
  const float n = rintf(fmaf(th, kInvTurn, -F.turn));
  return fmaf(th, kInvTurnLo, fmaf(th, kInvTurn, -(F.turn + n)));
}
// a waypoint (its headings only matter up to whole turns)
__device__ __forceinline__ float4 into_frame(const Frame& F, float4 w) {
  float x = w.x - F.ox, y = w.y - F.oy;
  into_frame(F, x, y);
  return make_float4(x, y, into_frame_wrapped(F, w.z), into_frame_wrapped(F, w.w));
}
// Obstacle row staged in LDS: the obstacle's centre in the rollout's frame
// at t0 and its motion in a step; for e = 2 the shape matrix Q = R'
// diag((mx+r)^-2, (my+r)^-2) R of eq. (16), with qa, qd the half sum and half
// difference of its diagonal, and Q rho for the motion rho of a step; the map
// A = diag((mx+r)^-1, (my+r)^-1) R into the obstacle's scaled frame, in which
// h = y0^e + y1^e - 1 (e4 = 1 for e = 4); the row's footprint disc (dA, dB).
// In the order that one 16-byte read brings what is used together.
struct alignas(16) ObsL {
  float cx, cy, qd, e4;
  float q11, q12, q22, qa;
  float mx, my, rx, ry;    // motion of a step, Q rho
  float rr, dA, dB, pad;   // rho' Q rho; disc centre p + dA e1 - dB f2
  float a00, a01, a10, a11;
};

struct RefPoint {
  float x, y, th1, th2;
};

// Reference zeta(psi): linear interpolation between waypoints, headings by the
// wrapped difference, clamped to the ends.  f is the fractional waypoint index
// relative to k0.  The window in LDS (in the rollout's frame) serves every lane
// unless one leaves it: then (a wave-uniform, rare case) the lanes outside read their
// points from HBM.  LDS is read through the local address space and HBM through the
// global one, each consumed on its own side of the branch: no flat access, whose wait
// would also drain the step-ahead HBM loads in flight.
__device__ __forceinline__ RefPoint reference(float f, int k0, int n_path, const float4* __restrict__ spath,
                                              int w0, int nw, const float4* __restrict__ gpath) {
  float fi = floorf(f);
  fi = fminf(fmaxf(fi, -1.0e7f), 1.0e7f);  // NaN -> -1e7 -> clamped to the start
  float t = fmaxf(f - fi, 0.0f);           // NaN -> 0
  const int graw = k0 + (int)fi;
  const int gi = min(max(graw, 0), n_path - 2);
  t = sel(graw > gi, 1.0f, t);
  t = sel(graw < 0, 0.0f, t);
  const int li = gi - w0;
  const int lc = min(max(li, 0), nw - 2);
  float4 A = lds(spath + lc), B = lds(spath + lc + 1);
  const bool outside = li != lc;
  if (__any(outside)) {
    // one point after the other, the frame in scalar registers: no more vector
    // registers here than the step has to spare
    auto uni = [](float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); };
    const float4 fr = lds(spath + kPathWin);
    const Frame F{uni(fr.x), uni(fr.y), uni(fr.z), uni(fr.w), uni(lds(&spath[kPathWin + 1].x))};
    auto from_hbm = [&](float4& W, int g) __attribute__((always_inline)) {
      const float4 w = into_frame(F, gld4(gpath + g));
      W.x = outside ? w.x : W.x;
      W.y = outside ? w.y : W.y;
      W.z = outside ? w.z : W.z;
      W.w = outside ? w.w : W.w;
      asm volatile("" : "+v"(W.x), "+v"(W.y), "+v"(W.z), "+v"(W.w)::"memory");
    };
    from_hbm(A, gi);
    from_hbm(B, gi + 1);
  }
  RefPoint r;
  r.x = fmaf(t, B.x - A.x, A.x);
  r.y = fmaf(t, B.y - A.y, A.y);
  r.th1 = fmaf(t, wrap_rev(B.z - A.z), A.z);
  r.th2 = fmaf(t, wrap_rev(B.w - A.w), A.w);
  return r;
}

// ---------------------------------------------------------------------------
// Rollout
// ---------------------------------------------------------------------------
// Launch shapes: G lanes share one sample (G = 1, 2, 4, 8).  Every lane of a group
// carries the full state; obstacle o's barrier row is computed by group lane
// o % G, and the rows' projection terms are summed over the group by DPP
// butterflies in a canonical tree of eight virtual lanes (below), so that
// every lane ends with the same sums, bit for bit, as a one-lane sample.  The normals
// are drawn in the rollout or come from the noise buffer filled by k_noise or from
// a run of steps drawn into LDS (the same Philox and Box-Muller code).  Results are
// therefore bitwise identical for every G, source of normals and block size.
//
// What bounds the step is the number of instructions, of any kind: a wave
// issues at most one every 4 cycles (transcendentals 8), and with one wave per
// SIMD (the eight-lane form at up to 8192 samples) scalar instructions, waits
// and nops cost as much as arithmetic.  Hence the units above and the row
// algebra below, whose obstacle rows are half the arithmetic of the
// gradient-by-gradient expansion of eq. (17): about 290 instructions a step in
// the eight-lane form with one row per lane, where the expansion took 430.
// Measured with it, before -> now: closed-loop update of 8192 samples, 50
// steps, 8 ellipses 63.7 -> 53.1 us (46.2 since); solve of 65536 samples, 100 steps, 32
// ellipses 1038 -> 658 us (610 since); of 5000 samples, 120 steps, 7 super-ellipses 168 ->
// 129 us (117 since).

// One row of eq. (9), divided by its guarded barrier value hh and with the
// inputs' scale factors left out: u^alpha = -(L + P U0 + Q U1) - alpha with
// L = Lf / hh, and U0 = Ts^3 j, U1 = G1 omega (G1 of the sample's step).
struct RowTerms {
  float L, P, Q;
};

// guarded barrier: copysign(max(|hhat|, h_eps), hhat) with 0 -> +h_eps (hhat is
// a sum whose zero is an exact cancellation, +0).  The NaN-propagating maximum: a
// NaN stays one, and its sample's cost is then non-finite.
__device__ __forceinline__ float barrier_rcp(float hhat, float h_eps) {
  return rcp(copysignf(__builtin_elementwise_maximum(fabsf(hhat), h_eps), hhat));
}

// Row sums of the 2x2 normal equations of the eliminated projection,
// accumulated in FP64.  With s = L + alpha + abar (abar the auxiliary input's
// own optimum) the equations are
//   diag(M_j, M_w) + Ma sum (G0 P, G1 Q)(G0 P, G1 Q)',
//   right-hand side p_u - Ma sum (G0 P, G1 Q) s,
// so the row sums need only P, Q and s.
struct Acc5 {
  double PP, PQ, QQ, Ps, Qs;
};

__device__ __forceinline__ Acc5 acc_zero() { return Acc5{0.0, 0.0, 0.0, 0.0, 0.0}; }

__device__ __forceinline__ void acc_row(Acc5& A, const RowTerms& R, float s) {
  const double p = (double)R.P, q = (double)R.Q, sd = (double)s;
  A.PP = fma(p, p, A.PP);
  A.PQ = fma(p, q, A.PQ);
  A.QQ = fma(q, q, A.QQ);
  A.Ps = fma(p, sd, A.Ps);
  A.Qs = fma(q, sd, A.Qs);
}

__device__ __forceinline__ Acc5 acc_add(const Acc5& a, const Acc5& b) {
  return Acc5{a.PP + b.PP, a.PQ + b.PQ, a.QQ + b.QQ, a.Ps + b.Ps, a.Qs + b.Qs};
}

// Barrier value, drift term and input gradient of one row: hhat, Lf = Ts
// (d hhat / dt along the drift), d hhat / d ah = g0, and g1 with
// Ts d hhat / d delta = G1 g1
struct ObsRow {
  float hhat, Lf, g0, g1;
};

// What the rear-axle rows of a sample's step share: position, e1 and vh e1
// (e2 its left normal), heading increment w = vh tan(delta)/l1 of the step, and
// the coefficients of the e = 2 rows.
struct StepGeom {
  float px, py, c1, s1, vc, vs, vh, ah, w, k2;
  float ca, b1, b2, ha, hb, hc, la, lb, lc;
  float m1, m2, tau;     // moving obstacles: coefficients, the step's index
};

template <bool MOV>
__device__ __forceinline__ StepGeom step_geom(float px, float py, float c1, float s1, float vc, float vs, float vh,
                                              float ah, float kd, float w, float tau) {
  StepGeom g;
  g.px = px; g.py = py; g.c1 = c1; g.s1 = s1; g.vc = vc; g.vs = vs; g.vh = vh; g.ah = ah; g.w = w; g.tau = tau;
  const float C2 = fmaf(-2.0f * s1, s1, 1.0f), S2 = 2.0f * s1 * c1;
  const float m = fmaf(3.0f, ah, 2.0f * vh);
  g.k2 = vh * w;
  g.ca = fmaf(2.0f, vh, ah);
  g.b1 = fmaf(-w, g.k2, g.ca + ah);
  g.b2 = kd * m;
  g.ha = vh * vh;
  g.hb = g.ha * C2;
  g.hc = g.ha * S2;
  g.la = vh * m;
  const float l3 = 3.0f * (vh * g.k2);
  g.lb = fmaf(g.la, C2, -(l3 * S2));
  g.lc = fmaf(g.la, S2, l3 * C2);
  if constexpr (MOV) {
    g.m1 = fmaf(2.0f, vh, m);              // 4 vh + 3 ah
    g.m2 = 3.0f * w;
  } else {
    g.m1 = g.m2 = 0.0f;
  }
  return g;
}

// Obstacle row, eqs. (16)-(17) with e = 2.  With d = p - p_o, q = d + vh e1,
// d_dd = ah e1 + k2 e2 (k2 = vh w) and the products y1 = d'Q e1, y2 = vh d'Q e2,
//   hhat = q'Qq - 1 + d'Q d_dd = d'Qd - 1 + (2 vh + ah) y1 + w y2 + vh^2 E11,
//   Lf   = (2 vh + 2 ah - w k2) y1 + kd m y2 + vh m E11 + 3 vh k2 E12
// with m = 2 vh + 3 ah, E11 = e1'Q e1 = qa + qd cos 2th + q12 sin 2th, E12 =
// e1'Q e2 = q12 cos 2th - qd sin 2th; the last two terms of each are three
// products with the step's coefficients.  A moving obstacle (motion rho a
// step: d_d = vh e1 - rho) adds rho'Q rho - 2 d'Q rho - 2 vh e1'Q rho to hhat
// and 2 rho'Q rho - 2 d'Q rho - (4 vh + 3 ah) e1'Q rho - 3 k2 e2'Q rho to Lf.
template <bool MOV>
__device__ __forceinline__ ObsRow obstacle_row(const ObsL& ob, const StepGeom& g) {
  float dx = g.px - ob.cx, dy = g.py - ob.cy;
  if constexpr (MOV) {
    dx = fmaf(-ob.mx, g.tau, dx);
    dy = fmaf(-ob.my, g.tau, dy);
  }
  const float Qx = fmaf(ob.q12, dy, ob.q11 * dx), Qy = fmaf(ob.q22, dy, ob.q12 * dx);
  ObsRow R;
  R.g0 = fmaf(Qy, g.s1, Qx * g.c1);
  R.g1 = fmaf(Qy, g.vc, -(Qx * g.vs));
  float h = fmaf(dy, Qy, fmaf(dx, Qx, -1.0f));
  h = fmaf(g.ca, R.g0, h);
  h = fmaf(g.w, R.g1, h);
  h = fmaf(g.ha, ob.qa, h);
  h = fmaf(g.hb, ob.qd, h);
  R.hhat = fmaf(g.hc, ob.q12, h);
  float l = g.b1 * R.g0;
  l = fmaf(g.b2, R.g1, l);
  l = fmaf(g.la, ob.qa, l);
  l = fmaf(g.lb, ob.qd, l);
  R.Lf = fmaf(g.lc, ob.q12, l);
  if constexpr (MOV) {
    const float r1 = fmaf(ob.ry, g.s1, ob.rx * g.c1);
    const float r2 = fmaf(ob.ry, g.vc, -(ob.rx * g.vs));     // vh e2'Q rho
    const float dr = fmaf(ob.ry, dy, ob.rx * dx) - ob.rr;
    // hhat: rr - 2 dR - 2 vh r1 = -2 (dr + vh r1) - rr
    R.hhat = fmaf(-2.0f, fmaf(g.vh, r1, dr), R.hhat) - ob.rr;
    R.Lf = fmaf(-2.0f, dr, fmaf(-g.m1, r1, fmaf(-g.m2, r2, R.Lf)));
  }
  return R;
}

// Super-ellipse row (e = 4), eqs. (16)-(17), in the obstacle's scaled frame:
// y = A d, h = y0^4 + y1^4 - 1.  Per axis, with E = A e1, F = A e2, the rate
// dl = vh E - A rho and the drift acceleration ep = ah E + k2 F (a step's
// units), hhat = sum y^4 + 4 y^3 (dl + ep/2) + 6 y^2 dl^2 - 1 and Lf = sum
// P dl + V ep + (3 ah w F - k2 w E) 2 y^3, P and V the partials of hhat in y
// and dl; g0 and g1 collect the partial 2 y^3 in ep along E and vh F.
__device__ __forceinline__ ObsRow obstacle_row_e4(const ObsL& ob, const StepGeom& g) {
  const float dx = fmaf(-ob.mx, g.tau, g.px - ob.cx), dy = fmaf(-ob.my, g.tau, g.py - ob.cy);
  const float a0[2] = {ob.a00, ob.a10}, a1[2] = {ob.a01, ob.a11};
  float h = -1.0f, l = 0.0f, g0 = 0.0f, g2 = 0.0f;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float y = fmaf(a1[i], dy, a0[i] * dx);
    const float E = fmaf(a1[i], g.s1, a0[i] * g.c1), F = fmaf(a1[i], g.c1, -(a0[i] * g.s1));
    const float rho = fmaf(a1[i], ob.my, a0[i] * ob.mx);
    const float dl = fmaf(g.vh, E, -rho), ep = fmaf(g.k2, F, g.ah * E);
    const float c = fmaf(0.5f, ep, dl);
    const float y2 = y * y, yc = y * c, d2 = dl * dl;
    const float A = 2.0f * y2 * y;
    h = fmaf(y2, fmaf(6.0f, d2, fmaf(4.0f, yc, y2)), h);
    const float P = 4.0f * y * fmaf(3.0f, d2, fmaf(3.0f, yc, y2));
    const float V = 4.0f * y2 * fmaf(3.0f, dl, y);
    l = fmaf(P, dl, l);
    l = fmaf(V, ep, l);
    g0 = fmaf(A, E, g0);
    g2 = fmaf(A, F, g2);
  }
  ObsRow R;
  R.hhat = h;
  R.g0 = g0;
  R.g1 = g.vh * g2;
  R.Lf = fmaf(3.0f * g.ah * g.w, g2, fmaf(-(g.k2 * g.w), g0, l));
  return R;
}

// Kinematics of a footprint disc centre c = p + A e1 - B f2 along the drift
// (inputs zero), for the rows of a footprint other than the rear axle (Sec.
// IV-C), in the units of a step: e1, e2 the tractor's heading and its left
// normal, f2, n2 the trailer's; every quantity is P0 + A PA - B PB with the
// step's parts below.
//   velocity  c'   = v e1 + A w1 e2 - B w2 n2
//   accel.    c''  = a e1 + v w1 e2 + A (w1' e2 - w1^2 e1) - B (w2' n2 - w2^2 f2)
//   jerk      c''' = -v w1^2 e1 + (2 a w1 + v w1') e2 + A (-3 w1 w1' e1 - w1^3 e2)
//                    + B (3 w2 w2' f2 + (w2^3 - w2'') n2)
// with w1 = th1', w2 = th2' of eq. (6) and their drift derivatives; and the
// partials through which the inputs act: dc'/d delta, dc''/da, dc''/d delta.
struct DiscBasis {
  float f2x, f2y;                                  // position: P0 = p, PA = e1, PB = f2
  float v0x, v0y, vAx, vAy, vBx, vBy;              // velocity
  float a0x, a0y, aAx, aAy, aBx, aBy;              // drift acceleration
  float j0x, j0y, jAx, jAy, jBx, jBy;              // drift jerk
  float gAx, gAy, gBx, gBy;                        // d velocity / d delta (P0 = 0)
  float ha0x, ha0y, haAx, haAy, haBx, haBy;        // d acceleration / d a
  float hd0x, hd0y, hdAx, hdAy, hdBx, hdBy;        // d acceleration / d delta
};

__device__ __forceinline__ DiscBasis disc_basis(float v, float a, float c1, float s1, float cp, float sp, float tn,
                                                float sec2, float inv_l1, float inv_l2, float ch) {
  DiscBasis D;
  const float e2x = -s1, e2y = c1;
  D.f2x = c1 * cp + s1 * sp;          // theta2 = theta1 - phi
  D.f2y = s1 * cp - c1 * sp;
  const float n2x = -D.f2y, n2y = D.f2x;
  const float kd = tn * inv_l1, dkd = sec2 * inv_l1;
  const float W = inv_l2 * (sp - ch * cp * tn);             // w2 = v W
  const float Wp = inv_l2 * (cp + ch * sp * tn);            // dW/dphi (d2W/dphi2 = -W)
  const float Wd = -inv_l2 * ch * cp * sec2;                // dW/d delta
  const float Wpd = inv_l2 * ch * sp * sec2;                // d2W/dphi d delta
  const float w1 = v * kd, w2 = v * W, ph = w1 - w2;
  const float w1d = a * kd;                                 // w1' along the drift
  const float w2d = a * W + v * Wp * ph;                    // w2'
  const float w2dd = 2.0f * a * Wp * ph - v * W * ph * ph + v * Wp * (w1d - w2d);   // w2''
  D.v0x = v * c1;  D.v0y = v * s1;
  D.vAx = w1 * e2x;  D.vAy = w1 * e2y;
  D.vBx = w2 * n2x;  D.vBy = w2 * n2y;
  D.a0x = a * c1 + v * w1 * e2x;  D.a0y = a * s1 + v * w1 * e2y;
  D.aAx = w1d * e2x - w1 * w1 * c1;  D.aAy = w1d * e2y - w1 * w1 * s1;
  D.aBx = w2d * n2x - w2 * w2 * D.f2x;  D.aBy = w2d * n2y - w2 * w2 * D.f2y;
  const float j1 = -v * w1 * w1, j2 = 2.0f * a * w1 + v * w1d;
  D.j0x = j1 * c1 + j2 * e2x;  D.j0y = j1 * s1 + j2 * e2y;
  const float jA1 = -3.0f * w1 * w1d, jA2 = -w1 * w1 * w1;
  D.jAx = jA1 * c1 + jA2 * e2x;  D.jAy = jA1 * s1 + jA2 * e2y;
  const float jB1 = -3.0f * w2 * w2d, jB2 = w2dd - w2 * w2 * w2;
  D.jBx = jB1 * D.f2x + jB2 * n2x;  D.jBy = jB1 * D.f2y + jB2 * n2y;
  D.gAx = v * dkd * e2x;  D.gAy = v * dkd * e2y;
  D.gBx = v * Wd * n2x;  D.gBy = v * Wd * n2y;
  D.ha0x = c1;  D.ha0y = s1;
  D.haAx = kd * e2x;  D.haAy = kd * e2y;
  D.haBx = W * n2x;  D.haBy = W * n2y;
  const float w2d_dl = a * Wd + v * Wpd * ph + v * Wp * (v * dkd - v * Wd);
  D.hd0x = v * v * dkd * e2x;  D.hd0y = v * v * dkd * e2y;
  D.hdAx = a * dkd * e2x - 2.0f * w1 * v * dkd * c1;  D.hdAy = a * dkd * e2y - 2.0f * w1 * v * dkd * s1;
  D.hdBx = w2d_dl * n2x - 2.0f * w2 * v * Wd * D.f2x;  D.hdBy = w2d_dl * n2y - 2.0f * w2 * v * Wd * D.f2y;
  return D;
}

// Row of an obstacle around a footprint disc (e = 2 or 4), eqs. (16)-(17), in
// the obstacle's scaled frame and the units of a step: h = sum y^e - 1 and its
// time derivatives along the drift from those of y = A (c - p_o); hhat = h + hd
// + hdd/2; Lf = d hhat/dt along the drift (obstacle motion included) = hd + hdd
// + hddd/2; the inputs reach hhat through c' (delta) and c'' (g1: G1 = Ts).
// The derivatives of y^e for e = 2 and 4 are one expression each in a = 1 or
// y^2 and the exponent's coefficients: no selects.
__device__ __forceinline__ ObsRow obstacle_row_disc(const ObsL& ob, const DiscBasis& D, float px, float py,
                                                    float c1, float s1, float tau) {
  const float A = ob.dA, B = ob.dB;
  const float dx = px + A * c1 - B * D.f2x - (ob.cx + ob.mx * tau);
  const float dy = py + A * s1 - B * D.f2y - (ob.cy + ob.my * tau);
  const float ux = D.v0x + A * D.vAx - B * D.vBx - ob.mx, uy = D.v0y + A * D.vAy - B * D.vBy - ob.my;
  const float wx = D.a0x + A * D.aAx - B * D.aBx, wy = D.a0y + A * D.aAy - B * D.aBy;
  const float zx = D.j0x + A * D.jAx - B * D.jBx, zy = D.j0y + A * D.jAy - B * D.jBy;
  const float gx = A * D.gAx - B * D.gBx, gy = A * D.gAy - B * D.gBy;
  const float hax = D.ha0x + A * D.haAx - B * D.haBx, hay = D.ha0y + A * D.haAy - B * D.haBy;
  const float hdx = D.hd0x + A * D.hdAx - B * D.hdBx, hdy = D.hd0y + A * D.hdAy - B * D.hdBy;
  const float e4 = ob.e4, ne4 = 1.0f - e4;
  const float n1 = fmaf(2.0f, e4, 2.0f), n2 = fmaf(10.0f, e4, 2.0f), n3 = 24.0f * e4;
  const float a0[2] = {ob.a00, ob.a10}, a1[2] = {ob.a01, ob.a11};
  float h = -1.0f, hd = 0.0f, hdd = 0.0f, hddd = 0.0f, da = 0.0f, dd1 = 0.0f, dd2 = 0.0f;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const float y = a0[i] * dx + a1[i] * dy, yd = a0[i] * ux + a1[i] * uy;
    const float ydd = a0[i] * wx + a1[i] * wy, yddd = a0[i] * zx + a1[i] * zy;
    const float ydl = a0[i] * gx + a1[i] * gy;          // d y_dot / d delta
    const float ya = a0[i] * hax + a1[i] * hay;         // d y_ddot / da
    const float yddl = a0[i] * hdx + a1[i] * hdy;       // d y_ddot / d delta
    const float yy = y * y;
    const float b = fmaf(yy, e4, ne4);                  // 1 or y^2
    const float f0 = yy * b, f1 = n1 * b * y, f2 = n2 * b, f3 = n3 * y;
    h += f0;
    hd += f1 * yd;
    hdd += f2 * yd * yd + f1 * ydd;
    hddd += f3 * yd * yd * yd + 3.0f * f2 * yd * ydd + f1 * yddd;
    da += f1 * ya;
    dd1 += f1 * ydl;
    dd2 += 2.0f * f2 * yd * ydl + f1 * yddl;
  }
  ObsRow R;
  R.hhat = h + hd + 0.5f * hdd;
  R.Lf = hd + hdd + 0.5f * hddd;
  R.g0 = 0.5f * da;
  R.g1 = dd1 + 0.5f * dd2;
  return R;
}

// the row of obstacle slot `ob`, by the instance's kind of rows
template <int ROWS>
__device__ __forceinline__ ObsRow obstacle_row_sel(const ObsL& ob, const DiscBasis& D, const StepGeom& g) {
  if constexpr (ROWS == kRowsDisc) {
    return obstacle_row_disc(ob, D, g.px, g.py, g.c1, g.s1, g.tau);
  } else if constexpr (ROWS == kRowsE4) {
    if (ob.e4 != 0.0f) return obstacle_row_e4(ob, g);
    return obstacle_row<true>(ob, g);
  } else {
    return obstacle_row<ROWS == kRowsMoving>(ob, g);
  }
}

// value held by lane Q of each G-lane group, broadcast to the group (DPP quad
// permute; G = 2 or 4 divides a quad, G = 8 groups hold two quads that each
// carry the value)
template <int G, int Q>
__device__ __forceinline__ float group_bcast(float x) {
  if constexpr (G == 1) {
    return x;
  } else {
    constexpr int ctrl = (G >= 4) ? (Q * 0x55) : ((Q) | (Q << 2) | ((2 + Q) << 4) | ((2 + Q) << 6));
    // every lane reads an in-range lane of its own quad: no "old" value needed
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), ctrl, 0xF, 0xF, true));
  }
}

// DPP controls of the three butterfly levels over 8 lanes: lane i reads lane
// i ^ 1, i ^ 2 (quad permutes), then 7 - i (half-row mirror: the other quad)
constexpr int kDppXor1 = 0xB1;
constexpr int kDppXor2 = 0x4E;
constexpr int kDppHalfMirror = 0x141;

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  const int lo = __double2loint(x), hi = __double2hiint(x);
  const int lo2 = __builtin_amdgcn_mov_dpp(lo, CTRL, 0xF, 0xF, true);
  const int hi2 = __builtin_amdgcn_mov_dpp(hi, CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi2, lo2);
}

template <int CTRL>
__device__ __forceinline__ Acc5 acc_partner_add(const Acc5& a) {
  return acc_add(a, Acc5{dpp_f64<CTRL>(a.PP), dpp_f64<CTRL>(a.PQ), dpp_f64<CTRL>(a.QQ), dpp_f64<CTRL>(a.Ps),
                         dpp_f64<CTRL>(a.Qs)});
}

// Canonical accumulation order of the projection rows, independent of the
// number G of lanes per sample: row r belongs to virtual lane v(r) (hitch row
// k -> v = k, obstacle o -> v = o mod 8); a virtual lane sums its rows from
// zero in row order (hitch row first, then obstacles v, v + 8, ...); the 8
// virtual sums are added by a fixed binary tree (v ^ 4, then v ^ 2, then v ^ 1).
// A group's lane of index q owns virtual lanes q + G i, so the levels inside a
// lane come first and only log2 G levels cross lanes, as DPP butterflies (IEEE
// addition commutes, so both partners hold the same bits).  With eight lanes
// the first level is the half-row mirror (lane i reads lane 7 - i), so lanes 4
// to 7 take the indices 7 to 4 (lane_index).
template <int G>
__device__ __forceinline__ int lane_index(int g) {
  return G == 8 && g >= 4 ? 11 - g : g;
}
template <int G>
__device__ __forceinline__ Acc5 cross_lane_levels(Acc5 a) {
  if constexpr (G >= 8) a = acc_partner_add<kDppHalfMirror>(a);
  if constexpr (G >= 4) a = acc_partner_add<kDppXor2>(a);
  if constexpr (G >= 2) a = acc_partner_add<kDppXor1>(a);
  return a;
}

// Collision-penalty baseline (the paper's second MPPI baseline, Sec. V; its
// form is not given): sum over the obstacle rows of max(0, -h)^2 with h the
// obstacle function of eq. (16) (e = 2 or 4) at the row's point (the rear
// axle, or its footprint disc centre) and the current time, in row order
// (every lane of a group sums all rows of its own step).
template <int ROWS>
__device__ __forceinline__ float collision_pen(const ObsL* __restrict__ sobs, int n_obs, float px, float py,
                                               float th1, float th2, float tau) {
  float c1 = 0.0f, s1 = 0.0f, c2 = 0.0f, s2 = 0.0f;
  if constexpr (ROWS == kRowsDisc) {
    sincospif(2.0f * th1, &s1, &c1);
    sincospif(2.0f * th2, &s2, &c2);
  }
  float pen = 0.0f;
  // four obstacles' LDS reads at a time (3 instances of 2000 samples in a batch, 40 steps,
  // 24 obstacles: one at a time 147 us, 101)
#pragma unroll 4
  for (int o = 0; o < n_obs; ++o) {
    const ObsL ob = sobs[o];
    float qx = px, qy = py;
    if constexpr (ROWS == kRowsDisc) {
      qx = px + ob.dA * c1 - ob.dB * c2;
      qy = py + ob.dA * s1 - ob.dB * s2;
    }
    const float dx = fmaf(-ob.mx, tau, qx - ob.cx), dy = fmaf(-ob.my, tau, qy - ob.cy);
    float h;
    if constexpr (ROWS >= kRowsE4) {
      const float y0 = ob.a00 * dx + ob.a01 * dy, y1 = ob.a10 * dx + ob.a11 * dy;
      const float z0 = y0 * y0, z1 = y1 * y1;
      const float b = 1.0f - ob.e4;
      h = z0 * fmaf(z0, ob.e4, b) + z1 * fmaf(z1, ob.e4, b) - 1.0f;
    } else {
      h = dx * (ob.q11 * dx + ob.q12 * dy) + dy * (ob.q12 * dx + ob.q22 * dy) - 1.0f;
    }
    h = fminf(h, 0.0f);
    pen = fmaf(h, h, pen);
  }
  return pen;
}

// sine and cosine of the three angles a step needs (th1, th1 - th2, delta), one
// pair per lane for G >= 4 (lane masks ma, mb, mc pick the angle: exact, as one
// of them is 1 or -1 and the others 0), then broadcast.
struct StepTrig {
  float s1, c1, sp, cp, tn;
};
struct TrigMask {
  float m1, m2, md;
};
template <int G>
__device__ __forceinline__ TrigMask trig_mask(int g) {
  const int q = g & 3;
  return TrigMask{q < 2 ? 1.0f : 0.0f, q == 1 ? -1.0f : 0.0f, q >= 2 ? 1.0f : 0.0f};
}

template <int G>
__device__ __forceinline__ StepTrig step_trig(const TrigMask& M, float th1, float th2, float dl) {
  StepTrig t;
  if constexpr (G < 4) {
    float sd, cd;
    sincos_rev(th1, &t.s1, &t.c1);
    sincos_rev(th1 - th2, &t.sp, &t.cp);
    sincos_rev(dl, &sd, &cd);
    t.tn = sd * rcp(cd);      // |delta| stays far from pi/2: cos > 0
  } else {
    const float a = fmaf(M.md, dl, fmaf(M.m2, th2, M.m1 * th1));
    float sa, ca;
    sincos_rev(a, &sa, &ca);
    const float ta = sa * rcp(ca);
    t.s1 = group_bcast<G, 0>(sa);
    t.c1 = group_bcast<G, 0>(ca);
    t.sp = group_bcast<G, 1>(sa);
    t.cp = group_bcast<G, 1>(ca);
    t.tn = group_bcast<G, 2>(ta);
  }
  return t;
}

// weights of the stage cost, headings in revolutions
struct CostConst {
  float Qc, Ql, Q1, Q2, Rj, Rw, mu, nu_bar;
};

// Tracking part of eq. (13): contour (14), lag (15) and heading errors, with
// the reference heading's sine and cosine given.
__device__ __forceinline__ float tracking_cost(const CostConst& C, const RefPoint& rf, float sr, float cr,
                                               float px, float py, float th1, float th2) {
  const float ex = px - rf.x, ey = py - rf.y;
  const float ec = fmaf(sr, ex, -(cr * ey));
  const float el = fmaf(cr, ex, sr * ey);
  const float e1 = wrap_rev(th1 - rf.th1);
  const float e2 = wrap_rev(th2 - rf.th2);
  return fmaf(C.Q2 * e2, e2, fmaf(C.Q1 * e1, e1, fmaf(C.Ql * el, el, C.Qc * ec * ec)));
}

// Stage cost r(x, u*, psi) of eq. (13): tracking terms, effort on (j, omega)
// and the progress term mu (nu_bar - nu)^2.
__device__ __forceinline__ float stage_cost(const CostConst& C, const RefPoint& rf, float px, float py, float th1,
                                            float th2, float uj, float uw, float unu) {
  float sr, cr;
  sincos_rev(rf.th1, &sr, &cr);
  const float prog = C.nu_bar - unu;
  return fmaf(C.mu * prog, prog,
              fmaf(C.Rw * uw, uw, fmaf(C.Rj * uj, uj, tracking_cost(C, rf, sr, cr, px, py, th1, th2))));
}

// value held by lane Q of each G-lane group, correct in the group's lane 0
// (G = 8: lanes 4..7 hold it after a quad permute, and lane 0 reads lane 7
// through the half-row mirror)
template <int G, int Q>
__device__ __forceinline__ float lane_value(float x) {
  if constexpr (G < 8 || Q < 4) {
    return group_bcast<G, Q>(x);
  } else {
    const float y = group_bcast<4, Q - 4>(x);
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(y), kDppHalfMirror, 0xF, 0xF, true));
  }
}

// J += the costs of lanes FIRST .. G - 1 of the group, in lane order
template <int G, int FIRST>
__device__ __forceinline__ void add_lane_costs(double& J, float rc) {
  if constexpr (FIRST < G) {
    J += (double)lane_value<G, FIRST>(rc);
    add_lane_costs<G, FIRST + 1>(J, rc);
  }
}
// the same for a last, partial run of n steps
template <int G, int FIRST>
__device__ __forceinline__ void add_lane_costs_n(double& J, float rc, uint32_t n) {
  if constexpr (FIRST < G) {
    if (n > (uint32_t)FIRST) {
      J += (double)lane_value<G, FIRST>(rc);
      add_lane_costs_n<G, FIRST + 1>(J, rc, n);
    }
  }
}

// Philox blocks of four normals that a step of the kernel's largest instance needs
template <int NOB, bool GUIDED>
constexpr int philox_blocks() {
  return GUIDED ? (5 + NOB + 3) / 4 : 1;
}

// Where a rollout's normals come from: drawn by its own lanes, read from the
// buffer of the noise kernel, or read from LDS, where the block draws those of a
// run of steps at a time (k_rollout_drawn)
enum NoiseFrom : int { kOwnDraw = 0, kBuffer = 1, kRuns = 2 };

// floats of a sample and step in a run (16 bytes of padding, as below)
template <int NOB, bool GUIDED>
constexpr int run_stride() {
  return 4 * philox_blocks<NOB, GUIDED>() + 4;
}

// Normals drawn in the kernel for samples shared by G lanes: lane g draws the
// blocks g, g + G, ..., and the lanes read what they need from the sample's
// place in LDS (in floats; 16 bytes of padding spread the samples over the banks)
template <int NOB, int G>
constexpr int coop_stride() {
  return 4 * G * ((philox_blocks<NOB, true>() + G - 1) / G) + 4;
}

// One sample's rollout over T steps, run by the G lanes of its group (lane g).
// Rows: every lane computes the hitch row g mod 2 (G = 1: both), obstacle o is
// computed by the lane of index o mod G in its slot o / G.  After the projection every lane
// holds the same inputs, state and cost.
// s_u / s_J (fused epilogue): the tile's applied inputs [3T][lds_stride] and
// costs in LDS, at column t_local.
// kRuns: the steps before run_end are drawn; next_run(run_end) draws the next
// ones and gives their end.
template <int NOB, bool GUIDED, int G, int NOISE, int ROWS, typename NextRun>
__device__ __forceinline__ void rollout_sample(const SolveDesc& d, uint32_t s, bool store, int g, const float* x0,
                                               const ObsL* __restrict__ sobs, const float4* __restrict__ spath,
                                               const float4* __restrict__ s_un, int w0, int nw, int k0, float phi0,
                                               float* s_u, uint32_t lds_stride, uint32_t t_local, float* s_J,
                                               float* s_nrm, uint32_t run_end, NextRun next_run) {
  static_assert(G == 1 || G == 2 || G == 4 || G == 8, "lanes per sample");
  constexpr int NSL = GUIDED ? (NOB + G - 1) / G : 1;   // obstacle slots of this lane
  constexpr int NV = 8 / G;                            // virtual lanes of this lane
  constexpr int kLeaves = NSL > (G == 1 ? 2 : 1) ? (NSL < NV ? NSL : NV) : (G == 1 ? 2 : 1);   // of them with rows
  constexpr int NH = (G == 1) ? 2 : 1;                 // hitch rows computed by this lane
  constexpr int NBMAX = philox_blocks<NOB, GUIDED>();    // Philox blocks of a step
  // normals drawn in the kernel and shared by the sample's lanes through LDS
  constexpr bool PRE = NOISE == kBuffer;
  constexpr bool kCoop = NOISE == kOwnDraw && G > 1;
  constexpr bool kFromRun = NOISE == kRuns;
  const brmppi_params& P = d.prm;
  const uint32_t T = d.T;
  const int n_obs = (int)d.n_obs;
  const bool hitch = !(d.flags & BRMPPI_HITCH_OFF);
  const bool penalty = (d.flags & BRMPPI_COLLISION_PENALTY) != 0;
  const int nb = GUIDED ? (5 + n_obs + 3) / 4 : 1;
  if constexpr (NOISE == kOwnDraw) {
    // uniform in the block: to scalar registers in the forms whose vector registers
    // spill (64 instances 707 -> 685 us)
    k0 = __builtin_amdgcn_readfirstlane(k0);
    w0 = __builtin_amdgcn_readfirstlane(w0);
    nw = __builtin_amdgcn_readfirstlane(nw);
  }
  const float4* __restrict__ gpath = d.path;
  const int n_path = (int)d.n_path;
  const int hk0 = (G == 1) ? 0 : (g & 1);    // first hitch row of this lane
  const int gi = lane_index<G>(g);           // its obstacles are gi + G j

  // constants of the step.  Held in vector registers (an empty asm makes each a
  // per-lane value): an instruction with a scalar operand takes 4 cycles of
  // its SIMD where the same on vector registers takes 2, and the eight-lane
  // form has too few scalar registers for them.
  const float Ts = P.Ts;
  float sj = P.sigma_j, sw = P.sigma_w, sn = P.sigma_nu;
  float inv_l1 = 1.0f / P.l1, inv_l2 = 1.0f / P.l2, ch = P.lh / P.l1;
  float chl = P.lh / P.l2;                   // ch l1 / l2
  float dmax = P.dtheta_max, kap = P.kappa / Ts;
  float h_eps = P.h_eps;
  // soft-bound projection, eq. (11): M = W + rho I, p = W z_des + rho/2 (lo + hi).
  // A row's auxiliary input: s = L + alpha + abar with abar = (W_a at + rho (amid
  // - alpha)) / Ma, at = sigma_a e, is L + nz + ka beta with beta = -alpha and
  // nz = ke e + kc.
  const float Ma = P.W_a + P.rho;
  float ke = P.W_a * P.sigma_a / Ma, kc = 0.5f * P.rho * (P.alpha_lo + P.alpha_hi) / Ma, ka = -(P.W_a / Ma);
  float Wj = P.W_j, Ww = P.W_w;
  float pj0 = 0.5f * P.rho * (P.j_lo + P.j_hi), pw0 = 0.5f * P.rho * (P.w_lo + P.w_hi);
  float G0 = Ts * Ts * Ts;
  float G1k = ROWS == kRowsDisc ? Ts : Ts * inv_l1;
  const double MG0 = (double)Ma * (double)G0, K00 = MG0 * (double)G0;
  const double NJ = (double)(P.W_j + P.rho), NW = (double)(P.W_w + P.rho), Mad = (double)Ma;
  float tsn = Ts, ddl = Ts * kInvTurn;
  const float inv_ds = d.inv_ds;
  CostConst C;
  C.Qc = P.Qc; C.Ql = P.Ql; C.Q1 = P.Qth1 * (kTurn * kTurn); C.Q2 = P.Qth2 * (kTurn * kTurn);
  C.Rj = P.R_j; C.Rw = P.R_w; C.mu = P.mu; C.nu_bar = P.nu_bar;
  const float w_col = P.w_col;
  {
    auto vpin = [](float& x) { asm volatile("" : "+v"(x)); };
    vpin(sj); vpin(sw); vpin(sn); vpin(tsn); vpin(ddl); vpin(inv_l1); vpin(inv_l2); vpin(ch);
    if constexpr (GUIDED) {
      vpin(chl); vpin(dmax); vpin(kap); vpin(h_eps); vpin(ke); vpin(kc); vpin(ka);
      vpin(Wj); vpin(Ww); vpin(pj0); vpin(pw0); vpin(G0); vpin(G1k);
    }
    vpin(C.Qc); vpin(C.Ql); vpin(C.Q1); vpin(C.Q2); vpin(C.Rj); vpin(C.Rw); vpin(C.mu); vpin(C.nu_bar);
  }

  float px = 0.0f, py = 0.0f, vh = Ts * x0[2], ah = Ts * Ts * x0[3];
  const Frame F = frame_at(x0[0], x0[1], x0[4]);
  float th1 = into_frame(F, x0[4]), th2 = into_frame(F, x0[5]), dl = x0[6] * kInvTurn, psi = 0.0f;
  // barrier rates, negated: beta = -alpha
  float bt_h[NH];
#pragma unroll
  for (int k = 0; k < NH; ++k) bt_h[k] = -P.alpha0;
  float bt_o[NSL];
#pragma unroll
  for (int j = 0; j < NSL; ++j) bt_o[j] = -P.alpha0;
  double J = 0.0;
  const uint32_t S_pad = d.S_pad;
  // Stage costs.  One lane per sample evaluates the cost of every step.  With
  // several lanes an unguided sample splits nothing but these (5000 samples, 120
  // steps, one -> eight lanes: 81 -> 66 us; with the penalty over eight
  // super-ellipses, every lane summing the rows of its own step, 159 -> 77 us).
  // With
  // G > 1 lanes the cost is not repeated on every lane: lane g keeps the cost
  // inputs of the steps tau with tau % G == g (state, progress and applied
  // inputs), and once per G steps each lane evaluates the cost of its kept
  // step, reference lookup included; lane 0 then adds the G costs to J in step
  // order.  J therefore receives the same terms in the same order as in the
  // one-lane form, and only lane 0 (the lane that stores) holds it.
  constexpr bool kBatchCost = (G > 1);
  float k_px = 0.0f, k_py = 0.0f, k_th1 = 0.0f, k_th2 = 0.0f, k_psi = 0.0f, k_uj = 0.0f, k_uw = 0.0f, k_unu = 0.0f;
  constexpr uint64_t kGroupMask = G == 8 ? 0x0101010101010101ull
                                  : G == 4 ? 0x1111111111111111ull
                                  : G == 2 ? 0x5555555555555555ull : ~0ull;
  // the hitch rows: signs +1, -1; with G > 1 they are owned by lanes 0 and 1,
  // and the others zero their copy by these factors (P = Q = 0 makes every
  // term of the row's sums an exact zero)
  float hs[NH], hp[NH], hq[NH];
#pragma unroll
  for (int k = 0; k < NH; ++k) {
    const bool own = G == 1 || (hitch && g < 2);
    hs[k] = (hk0 + k) == 0 ? 1.0f : -1.0f;
    hp[k] = own ? -kap : 0.0f;
    hq[k] = own ? hs[k] : 0.0f;
  }
  const TrigMask TM = trig_mask<G>(g);
  // a lane's own obstacles stay in registers when it has few
  constexpr bool kObsRegs = GUIDED && G > 1 && NSL <= 4 && ROWS != kRowsDisc;
  ObsL ob_r[kObsRegs ? NSL : 1];
  if constexpr (kObsRegs) {
#pragma unroll
    for (int j = 0; j < NSL; ++j) ob_r[j] = sobs[gi + G * j];
  }

  // Precomputed normals are loaded two steps ahead into a queue of two slots:
  // step tau reads slot tau % 2 and refills it with step tau + 2.  The loop is
  // unrolled by two so that the slot is a compile-time index (no register
  // moves, which would wait for the loads in flight).  Every load is in range
  // (the last step's rows are loaded again past the end, row indices are
  // clamped), so none needs a branch; rows past the instance's own (obstacles o
  // >= n_obs, unguided instances) feed only rows whose terms are zeroed or
  // unused.  A load is a buffer load: the noise buffer (at most 2 GiB), a lane
  // offset per row and a scalar offset advanced once a step, with no address
  // arithmetic per load.
  static_assert(!PRE || kNoisePrefetch == 2, "two queue slots");
  constexpr int PF = PRE ? 2 : 1;
  float nx_in[PF][3], nx_h[PF][NH], nx_o[PF][NSL];   // (from LDS: the next step's)
  uint32_t off_in[3], off_h[NH], off_o[NSL];
  const uint32_t step_bytes = d.n_normals * S_pad * (uint32_t)sizeof(float);
  const uint32_t last_bytes = step_bytes * (T - 1);
  uint32_t at_bytes = 0;                       // the step that the next load reads
  const __amdgpu_buffer_rsrc_t noise_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(d.noise, 0, PRE ? (int)(last_bytes + step_bytes) : 0, 0x00020000);
  if constexpr (PRE) {
    const uint32_t n_rows = d.n_normals;
#pragma unroll
    for (uint32_t k = 0; k < 3; ++k) off_in[k] = 4u * (k * S_pad + s);
#pragma unroll
    for (int k = 0; k < NH; ++k) off_h[k] = 4u * (min((uint32_t)(3 + hk0 + k), n_rows - 1) * S_pad + s);
#pragma unroll
    for (int j = 0; j < NSL; ++j) off_o[j] = 4u * (min((uint32_t)(5 + gi + G * j), n_rows - 1) * S_pad + s);
  }
  auto load_normals = [&](int q) __attribute__((always_inline)) {
    if constexpr (PRE) {
      auto ld = [&](uint32_t off) {
        return __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(noise_rsrc, (int)off, (int)at_bytes, 0));
      };
#pragma unroll
      for (int k = 0; k < 3; ++k) nx_in[q][k] = ld(off_in[k]);
      if constexpr (GUIDED) {
#pragma unroll
        for (int k = 0; k < NH; ++k) nx_h[q][k] = ld(off_h[k]);
#pragma unroll
        for (int j = 0; j < NSL; ++j) nx_o[q][j] = ld(off_o[j]);
      }
      at_bytes = min(at_bytes + step_bytes, last_bytes);
    }
  };
  if constexpr (PRE) {
    // slot 0 before slot 1, in this order, as inside the loop
    load_normals(0);
    __builtin_amdgcn_sched_barrier(0);
    load_normals(1);
    __builtin_amdgcn_sched_barrier(0);
  }
  // kCoop: the step's blocks into the sample's place in LDS, and this lane's
  // normals from it.  The lanes of a sample are lanes of one wave, whose LDS
  // operations execute in order: the fences only keep the compiler from
  // reordering them.  A normal past the drawn blocks (rows past the last
  // obstacle) is read from the last drawn one.
  // kFromRun: the same from the sample's place in the run of steps in LDS.
  const float* nrm = s_nrm + t_local * (kCoop ? coop_stride<NOB, G>() : run_stride<NOB, GUIDED>());
  uint32_t nrm_o[NSL];
  if constexpr (kCoop || kFromRun) {
#pragma unroll
    for (int j = 0; j < NSL; ++j) nrm_o[j] = min((uint32_t)(5 + gi + G * j), (uint32_t)(4 * nb - 1));
  }
  auto coop_draw = [&](uint32_t tau) __attribute__((always_inline)) {
    if constexpr (kCoop) {
      asm volatile("" ::: "memory");
#pragma unroll
      for (int i = 0; i * G < NBMAX; ++i) {
        if (i * G < nb) {
          uint32_t r[4];
          float e[4];
          philox4x32_10(s, tau, (uint32_t)(g + G * i), d.instance, d.seed_lo, d.seed_hi, r);
          box_muller4(r, e);
          lds_put(reinterpret_cast<float4*>(s_nrm + t_local * coop_stride<NOB, G>()) + g + G * i,
                  make_float4(e[0], e[1], e[2], e[3]));
        }
      }
      asm volatile("" ::: "memory");
    }
    if constexpr (kCoop || kFromRun) {
      const float* at = nrm;
      const Vec3 in = lds3(reinterpret_cast<const float4*>(at));
      nx_in[0][0] = in.x;
      nx_in[0][1] = in.y;
      nx_in[0][2] = in.z;
      if constexpr (GUIDED) {
#pragma unroll
        for (int k = 0; k < NH; ++k) nx_h[0][k] = lds(at + min(3 + hk0 + k, 4 * nb - 1));
#pragma unroll
        for (int j = 0; j < NSL; ++j) nx_o[0][j] = lds(at + nrm_o[j]);
      }
    }
    if constexpr (kFromRun) nrm += kDrawnTile * run_stride<NOB, GUIDED>();
  };
  coop_draw(0);
  Vec3 un = lds3(s_un);                        // nominal inputs, read a step ahead
  // uniform switches, tested as scalar integers each step (as conditions they
  // would be kept as lane masks and cost twice the instructions)
  const int to_hbm = __builtin_amdgcn_readfirstlane((int)d.ustar_global);
  const int to_lds = __builtin_amdgcn_readfirstlane((int)(s_u != nullptr));
  float* su = s_u + t_local;                   // this step's place in the tile's inputs
  float* ug = d.u_star + s;

  auto step = [&](const uint32_t tau, auto SLOT) __attribute__((always_inline)) {
    constexpr int q = decltype(SLOT)::value;
    // --- noise: normals 0..2 perturb the inputs, 3 and 4 the hitch rows'
    // auxiliary inputs, 5 + o obstacle o's ---
    float uj, uw, unu, nz_h[NH], nz_o[NSL];
    if constexpr (PRE || kCoop || kFromRun) {
      uj = fmaf(sj, nx_in[q][0], un.x);
      uw = fmaf(sw, nx_in[q][1], un.y);
      unu = fmaf(sn, nx_in[q][2], un.z);
      if constexpr (GUIDED) {
#pragma unroll
        for (int k = 0; k < NH; ++k) nz_h[k] = fmaf(ke, nx_h[q][k], kc);
#pragma unroll
        for (int j = 0; j < NSL; ++j) nz_o[j] = fmaf(ke, nx_o[q][j], kc);
      }
    } else {
      float eps[4 * NBMAX];
#pragma unroll
      for (int b = 0; b < NBMAX; ++b) {
        if (b < nb) {
          uint32_t r[4];
          philox4x32_10(s, tau, (uint32_t)b, d.instance, d.seed_lo, d.seed_hi, r);
          box_muller4(r, &eps[4 * b]);
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) eps[4 * b + k] = 0.0f;
        }
      }
      uj = fmaf(sj, eps[0], un.x);
      uw = fmaf(sw, eps[1], un.y);
      unu = fmaf(sn, eps[2], un.z);
      if constexpr (GUIDED) {
#pragma unroll
        for (int k = 0; k < NH; ++k) nz_h[k] = fmaf(ke, eps[3 + k], kc);
#pragma unroll
        for (int j = 0; j < NSL; ++j) nz_o[j] = fmaf(ke, eps[5 + j], kc);   // G == 1: slot j is obstacle j
      }
    }
    if constexpr (kCoop) coop_draw(tau + 1);   // (step T's are unused)
    un = lds3(s_un + (tau + 1));   // (past the last step: the staged array's extra entry, unused)
    RefPoint rf{};
    if constexpr (!kBatchCost) rf = reference(fmaf(psi, inv_ds, phi0), k0, n_path, spath, w0, nw, gpath);
    const StepTrig tg = step_trig<G>(TM, th1, th2, dl);
    const float s1 = tg.s1, c1 = tg.c1, sp = tg.sp, cp = tg.cp, tn = tg.tn;
    const float kd = tn * inv_l1;
    const float w = vh * kd;                   // th1 increment of the step [rad]
    const float W2 = inv_l2 * fmaf(-(ch * cp), tn, sp);
    const float w2 = vh * W2;                  // th2 increment
    const float vc = vh * c1, vs = vh * s1;    // position increment
    // Refill the queue slot with step tau + 2 only now, after the last use of
    // its values: a refill hoisted above a use needs a second register, and the
    // copy back into the slot's register at the loop's back edge would wait
    // for every load in flight (the prefetch lost).  The empty asm pins the
    // normals' products here (the compiler would otherwise sink them to their
    // uses in the rows, past the refill) and the scheduling barrier keeps the
    // refill below them.
    if constexpr (PRE || kFromRun) {
      asm volatile("" : "+v"(uj), "+v"(uw), "+v"(unu));
      if constexpr (GUIDED) {
#pragma unroll
        for (int k = 0; k < NH; ++k) asm volatile("" : "+v"(nz_h[k]));
#pragma unroll
        for (int j = 0; j < NSL; ++j) asm volatile("" : "+v"(nz_o[j]));
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (PRE) load_normals(q);
      else coop_draw(tau + 1);
    }

    float U0 = 0.0f;
    if constexpr (GUIDED) {
      const float sec2 = fmaf(tn, tn, 1.0f);
      const StepGeom geo = step_geom<ROWS != kRowsStatic>(px, py, c1, s1, vc, vs, vh, ah, kd, w, (float)tau);
      DiscBasis DB;
      if constexpr (ROWS == kRowsDisc) DB = disc_basis(vh, ah, c1, s1, cp, sp, tn, sec2, inv_l1, inv_l2, ch);
      // Ts d hhat / d delta = G1 g1
      const float G1 = ROWS == kRowsDisc ? G1k : G1k * (vh * sec2);

      // hitch rows, eq. (18) split into h_s = dth_max - kappa v + s (th1 - th2),
      // first-order expansion hhat = h + Ts hd = base + s (phi - Dh)
      // (with G > 1 lanes the rows are formed whether the instance has them or
      // not, and zeroed by hp, hq: no branch in the step)
      RowTerms H[NH];
      if (G > 1 || hitch) {
        const float Dh = w2 - w;
        const float Dphi = vh * (inv_l2 * fmaf(ch * sp, tn, cp));
        const float base = fmaf(-kap, vh + ah, dmax);
        const float sg = fmaf(kTurn, th1 - th2, -Dh);
        const float lsum = fmaf(W2 - kd, ah, fmaf(-Dphi, Dh, Dh));
        const float lb = -kap * ah;
        float qh = fmaf(cp, chl, 1.0f);
        if constexpr (ROWS == kRowsDisc) qh *= inv_l1 * (vh * sec2);
#pragma unroll
        for (int k = 0; k < NH; ++k) {
          const float ih = barrier_rcp(fmaf(hs[k], sg, base), h_eps);
          H[k].L = fmaf(-hs[k], lsum, lb) * ih;
          H[k].P = hp[k] * ih;
          H[k].Q = hq[k] * qh * ih;
        }
      }
      // rows of virtual lane g + G i: its hitch row, then obstacles in order
      RowTerms O[NSL];
      auto obs_row = [&](int j, const ObsL& ob, Acc5& A) __attribute__((always_inline)) {
        const ObsRow R = obstacle_row_sel<ROWS>(ob, DB, geo);
        const float ih = barrier_rcp(R.hhat, h_eps);
        O[j].L = R.Lf * ih;
        O[j].P = R.g0 * ih;
        O[j].Q = R.g1 * ih;
        acc_row(A, O[j], O[j].L + fmaf(ka, bt_o[j], nz_o[j]));
      };
      // Rows two slots at a time, so that one branch and one wait for the
      // obstacles' LDS reads serve two rows; no branch where every instance of
      // the kernel's bucket has the first of them.  A row past the last
      // obstacle reads a staged blank one (Q = A = 0: hhat = -1, Lf = g = +-0)
      // and a finite normal, so it adds exact zeros to the sums (an accumulator
      // is never -0, so x + 0 keeps its bits), without divergent branches or
      // selects.
      constexpr int kMinRows = NOB == 32 ? 17 : (NOB == 16 ? 9 : (NOB == 8 ? 3 : 0));
      Acc5 A[NV];
#pragma unroll
      for (int i = 0; i < NV; ++i) A[i] = acc_zero();
      if constexpr (G == 1) {
        if (hitch) {
          acc_row(A[0], H[0], H[0].L + fmaf(ka, bt_h[0], nz_h[0]));
          acc_row(A[1], H[1], H[1].L + fmaf(ka, bt_h[1], nz_h[1]));
        }
      } else {
        // lanes 0 and 1 hold the hitch rows; the others add exact zeros
        acc_row(A[0], H[0], H[0].L + fmaf(ka, bt_h[0], nz_h[0]));
      }
      // A footprint's rows on one lane go one by one: two at a time they spill (16
      // instances of 32768 samples, 60 steps, two obstacles around two discs in a batch:
      // 1335 us, 1040; with four lanes pairs are 4 % faster).
      constexpr bool kPairs = ROWS != kRowsDisc || G > 1;
      if constexpr (kPairs) {
#pragma unroll
        for (int j = 0; j < NSL; j += 2) {
          if (G * j < kMinRows || G * j < n_obs) {
            ObsL oa, ob;
            if constexpr (kObsRegs) oa = ob_r[j];
            else oa = sobs[gi + G * j];
            if (j + 1 < NSL) {
              if constexpr (kObsRegs) ob = ob_r[j + 1 < NSL ? j + 1 : 0];
              else ob = sobs[gi + G * (j + 1)];
            }
            obs_row(j, oa, A[j % NV]);
            if (j + 1 < NSL) obs_row(j + 1, ob, A[(j + 1) % NV]);
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < NSL; ++j)
          if (G * j < n_obs) obs_row(j, sobs[gi + G * j], A[j % NV]);
      }
#pragma unroll
      for (int n = NV / 2; n >= 1; n /= 2) {
#pragma unroll
        for (int i = 0; i < n; ++i)
          if (i + n < kLeaves) A[i] = acc_add(A[i], A[i + n]);
      }
      const Acc5 S8 = cross_lane_levels<G>(A[0]);
      const double G1d = (double)G1, MG1 = Mad * G1d;
      const double N00 = fma(K00, S8.PP, NJ), N01 = (MG0 * G1d) * S8.PQ, N11 = fma(MG1 * G1d, S8.QQ, NW);
      const double y0 = fma(-MG0, S8.Ps, (double)fmaf(Wj, uj, pj0));
      const double y1 = fma(-MG1, S8.Qs, (double)fmaf(Ww, uw, pw0));
      const double det = fma(N00, N11, -(N01 * N01));
      // det > 0 (N is the diagonal W + rho I plus positive semidefinite rank-one
      // terms): the hardware reciprocal and one Newton step square its relative
      // error, far below the FP32 rounding of the result (3 instructions
      // instead of the IEEE division's 12)
      double idet = __builtin_amdgcn_rcp(det);
      idet = fma(fma(-det, idet, 1.0), idet, idet);
      uj = (float)(fma(N11, y0, -(N01 * y1)) * idet);
      uw = (float)(fma(N00, y1, -(N01 * y0)) * idet);
      U0 = G0 * uj;
      const float U1 = G1 * uw;
      // next barrier rates: alpha + u^alpha = -(L + P U0 + Q U1) (eq. (9) holds exactly)
      if (G > 1 || hitch) {
#pragma unroll
        for (int k = 0; k < NH; ++k) {
          // (H[k].P and H[k].Q are zero on lanes that do not own the row: their rate is unused)
          bt_h[k] = fmaf(H[k].Q, U1, fmaf(H[k].P, U0, H[k].L));
        }
      }
#pragma unroll
      for (int j = 0; j < NSL; ++j) {
        const int row = G * (kPairs ? j & ~1 : j);
        if ((kPairs && row < kMinRows) || row < n_obs) bt_o[j] = fmaf(O[j].Q, U1, fmaf(O[j].P, U0, O[j].L));
      }
    } else {
      U0 = G0 * uj;
    }

    // --- stage cost r(x_tau, u*_tau, psi_tau), eq. (13) ---
    if constexpr (!kBatchCost) {
      float rc = stage_cost(C, rf, px, py, th1, th2, uj, uw, unu);
      if (penalty) rc = fmaf(w_col, collision_pen<ROWS>(sobs, n_obs, px, py, th1, th2, (float)tau), rc);
      J += (double)rc;
    } else {
      const uint64_t mine = kGroupMask << (tau & (G - 1));
      k_px = sel_mask(mine, px, k_px);
      k_py = sel_mask(mine, py, k_py);
      k_th1 = sel_mask(mine, th1, k_th1);
      k_th2 = sel_mask(mine, th2, k_th2);
      k_psi = sel_mask(mine, psi, k_psi);
      k_uj = sel_mask(mine, uj, k_uj);
      k_uw = sel_mask(mine, uw, k_uw);
      k_unu = sel_mask(mine, unu, k_unu);
    }

    // --- applied inputs: [3T][S_pad] in HBM and/or the tile's LDS ---
    int hbm = to_hbm, in_lds = to_lds;
    if constexpr (G > 1) asm volatile("" : "+s"(hbm), "+s"(in_lds));
    if (hbm) {
      if (store) {
        gst(ug, uj);
        gst(ug + S_pad, uw);
        gst(ug + 2 * (size_t)S_pad, unu);
      }
      ug += 3 * (size_t)S_pad;
    }
    if (in_lds) {
      // the reads made ahead are awaited before the writes, not with them
      asm volatile("" : "+v"(un.x), "+v"(un.y), "+v"(un.z));
      if constexpr (kFromRun) {
#pragma unroll
        for (int k = 0; k < 3; ++k) asm volatile("" : "+v"(nx_in[0][k]));
        if constexpr (GUIDED) {
#pragma unroll
          for (int k = 0; k < NH; ++k) asm volatile("" : "+v"(nx_h[0][k]));
#pragma unroll
          for (int j = 0; j < NSL; ++j) asm volatile("" : "+v"(nx_o[0][j]));
        }
      }
      // every lane of the sample writes the same values to its column; the
      // column of a sample past S is never weighted
      lds_put(su, uj);
      lds_put(su + lds_stride, uw);
      lds_put(su + 2 * lds_stride, unu);
      su += 3 * lds_stride;
    }

    // --- explicit Euler, eq. (6), plus psi_dot = nu ---
    px += vc;
    py += vs;
    vh += ah;
    ah += U0;
    th1 = fmaf(w, kInvTurn, th1);
    th2 = fmaf(w2, kInvTurn, th2);
    dl = fmaf(ddl, uw, dl);
    psi = fmaf(tsn, unu, psi);
  };
  // costs of the kept steps tau0 .. tau0 + n - 1 (lane g: step tau0 + g)
  auto kept_cost = [&](uint32_t tau0) __attribute__((always_inline)) -> float {
    const RefPoint r = reference(fmaf(k_psi, inv_ds, phi0), k0, n_path, spath, w0, nw, gpath);
    float rc = stage_cost(C, r, k_px, k_py, k_th1, k_th2, k_uj, k_uw, k_unu);
    if (penalty)
      rc = fmaf(w_col, collision_pen<ROWS>(sobs, n_obs, k_px, k_py, k_th1, k_th2, (float)(tau0 + (uint32_t)g)), rc);
    return rc;
  };
  uint32_t tau = 0;
  if constexpr (PRE || kFromRun) {
    // whole pairs, then an odd last step: every pass of the loop issues both
    // slots' refills, so a step's wait for its own slot leaves the other
    // slot's loads in flight; G is even, so only the pair's second step can
    // complete a run of G kept steps (and a run of drawn steps is even too)
    // (tested at the bottom: with the test at the top the compiler keeps two
    // copies of the state and moves one into the other in every pass)
    const uint32_t T2 = T & ~1u;
    if (T2 != 0) {
      do {
        step(tau, std::integral_constant<int, 0>{});
        step(tau + 1, std::integral_constant<int, PF - 1>{});
        tau += 2;
        if constexpr (kFromRun) {
          // the next run (what was read ahead past the end of one, from the path
          // window, is unused)
          if (tau == run_end && tau != T) {
            run_end = next_run(tau);
            nrm = s_nrm + t_local * run_stride<NOB, GUIDED>();
            coop_draw(tau);
          }
        }
        if constexpr (kBatchCost) {
          if ((tau & (G - 1)) == 0) {
            const float rc = kept_cost(tau - G);
            add_lane_costs<G, 0>(J, rc);
          }
        }
      } while (tau != T2);
    }
    if (T & 1u) step(tau, std::integral_constant<int, 0>{});
    if constexpr (kBatchCost) {
      const uint32_t n = T & (G - 1);
      if (n != 0) {
        const float rc = kept_cost(T - n);
        add_lane_costs_n<G, 0>(J, rc, n);
      }
    }
  } else {
    do {
      step(tau, std::integral_constant<int, 0>{});
      ++tau;
      if constexpr (kBatchCost) {
        if ((tau & (G - 1)) == 0) {
          const float rc = kept_cost(tau - G);
          add_lane_costs<G, 0>(J, rc);
        }
      }
    } while (tau != T);
    if constexpr (kBatchCost) {
      const uint32_t n = T & (G - 1);
      if (n != 0) {
        const float rc = kept_cost(T - n);
        add_lane_costs_n<G, 0>(J, rc, n);
      }
    }
  }
  // the reference at psi_T; its heading's sine and cosine by the library (within 5.1e-8,
  // the hardware's within 1.3e-7: once a sample, not once a step)
  const RefPoint rT = reference(fmaf(psi, inv_ds, phi0), k0, n_path, spath, w0, nw, gpath);
  float sr, cr;
  sincospif(2.0f * rT.th1, &sr, &cr);
  float rN = tracking_cost(C, rT, sr, cr, px, py, th1, th2);
  if (penalty) rN = fmaf(w_col, collision_pen<ROWS>(sobs, n_obs, px, py, th1, th2, (float)T), rN);
  J += (double)rN;
  float Jf = (float)J;
  if (!isfinite(Jf)) Jf = INFINITY;
  if (store) {
    d.J[s] = Jf;
    if (s_J) s_J[t_local] = Jf;
  }
}


// ---------------------------------------------------------------------------
// Noise: every (four consecutive samples, step) in parallel, all their Philox
// blocks in one thread (independent chains the scheduler interleaves) ->
// [tau][k][S_pad], one 16-byte store per lane and row
// ---------------------------------------------------------------------------
constexpr int kMaxPhiloxBlocks = (5 + BRMPPI_MAX_OBS + 3) / 4;

// Inputs of an update (descriptor, zeroed counters, nominal sequence), read from
// pinned host memory by the launch that precedes the rollout on its stream, and
// its results written there by the rollout.  Bounded by the host link's latency
// (a few KB): as copy commands of their own, before the noise and after the
// rollout, they took 6 us more (8192 samples, 50 steps, 8 obstacles: 68.2 -> 62.0 us; with 20011
// costs fetched 155 -> 141 us).
__global__ __launch_bounds__(256) void k_upload(Upload up) {
  const uint4* __restrict__ src = static_cast<const uint4*>(up.src);
  uint4* __restrict__ dst = static_cast<uint4*>(up.dst);
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < up.n; i += (size_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

__global__ __launch_bounds__(256) void k_noise(NoiseArgs a, uint32_t nb, Upload up) {
  // blockIdx.z = update u of a run of consecutive updates; a thread draws
  // four consecutive samples at step blockIdx.y and stores each row of normals
  // with one 16-byte store (samples from S up to S_pad get the normals of
  // their own indices, which nothing reads)
  // The first blocks carry the upload, a unit a thread: read before the draws,
  // which hide the latency of the host's memory, and written after them.
  const size_t nt = (size_t)gridDim.x * gridDim.y * gridDim.z * blockDim.x;
  const size_t me = (blockIdx.x + (size_t)gridDim.x * (blockIdx.y + (size_t)gridDim.y * blockIdx.z)) * blockDim.x + threadIdx.x;
  const uint4* __restrict__ src = static_cast<const uint4*>(up.src);
  uint4* __restrict__ dst = static_cast<uint4*>(up.dst);
  uint4 in = make_uint4(0, 0, 0, 0);
  if (me < up.n) in = src[me];
  const uint32_t s0 = 4 * (blockIdx.x * blockDim.x + threadIdx.x);
  const uint32_t tau = blockIdx.y;
  const uint64_t seed = a.seed + blockIdx.z;
  const uint32_t seed_lo = (uint32_t)seed, seed_hi = (uint32_t)(seed >> 32);
  float* __restrict__ out = a.noise + blockIdx.z * a.stride + (size_t)tau * a.n_normals * a.S_pad + s0;
  const uint32_t n_draw = s0 < a.S_pad ? a.n_normals : 0u;
#pragma unroll
  for (int b = 0; b < kMaxPhiloxBlocks; ++b) {
    if ((uint32_t)b < nb && n_draw) {
      float e[4][4];
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i) {
        uint32_t r[4];
        philox4x32_10(s0 + i, tau, (uint32_t)b, a.instance, seed_lo, seed_hi, r);
        box_muller4(r, e[i]);
      }
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        const uint32_t kk = 4 * (uint32_t)b + k;
        if (kk < n_draw)
          gst4(reinterpret_cast<float4*>(out + (size_t)kk * a.S_pad), make_float4(e[0][k], e[1][k], e[2][k], e[3][k]));
      }
    }
  }
  if (me < up.n) dst[me] = in;
  for (size_t i = me + nt; i < up.n; i += nt) dst[i] = src[i];
}

// ---------------------------------------------------------------------------
// Block reductions (deterministic: fixed butterfly, fixed wave order)
// ---------------------------------------------------------------------------
__device__ __forceinline__ float wave_min(float v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v = fminf(v, __shfl_xor(v, m, 64));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}

// Hand-off of partial results between blocks (the "last block" patterns).
// The partials are written and read only as device-scope relaxed atomics:
// such a store writes through its XCD's L2 and such a load does not take a
// stale line from the reader's L2, so each partial is coherent across the
// XCDs by itself.  A publisher then needs only every wave's stores complete
// (vmcnt drained) before the block's counter increment, and the block that
// sees the last increment reads with those loads after it.  A release fence
// at device scope would instead write back every dirty line of the XCD's L2
// (and an acquire invalidate it), which stalls every block on that XCD: one
// such write-back per work item cost the batched reduce a quarter of its
// time.
typedef __attribute__((address_space(1))) float glb_float;
__device__ __forceinline__ void pub_st(float* p, float v) {
  __hip_atomic_store((glb_float*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void pub_st4(float4* p, float4 v) {
  pub_st(&p->x, v.x);
  pub_st(&p->y, v.y);
  pub_st(&p->z, v.z);
  pub_st(&p->w, v.w);
}
__device__ __forceinline__ float pub_ld(const float* p) {
  return __hip_atomic_load((const glb_float*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float4 pub_ld4(const float4* p) {
  return make_float4(pub_ld(&p->x), pub_ld(&p->y), pub_ld(&p->z), pub_ld(&p->w));
}
// this wave's stores complete; also a compiler barrier, so that no store
// moves past it
__device__ __forceinline__ void pub_complete() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// the block's next work item.  Persistent launch (grid <= items): the first
// item of block b is item b, the later ones come from the queue, past the
// grid's first round (so that the whole grid does not start on one contended
// atomic).  Direct launch: item blockIdx.x only.
__device__ __forceinline__ bool next_item(uint32_t it, uint32_t n_items, uint32_t* ctr_next, uint32_t* s_slot,
                                          uint32_t& ix) {
  if (ctr_next) {
    if (it == 0) {
      ix = blockIdx.x;
    } else {
      if (threadIdx.x == 0) *s_slot = gridDim.x + atomicAdd(ctr_next, 1u);
      __syncthreads();
      ix = *s_slot;
    }
  } else {
    if (it > 0) return false;
    ix = blockIdx.x;
  }
  ix = __builtin_amdgcn_readfirstlane(ix);
  return ix < n_items;
}

// The last block to finish resets the queue for the next launch (a graph
// replay).  Only the two counters take part: a block increments done after
// its last grab of next has returned, so no fence is needed.
__device__ __forceinline__ void finish_persistent(uint32_t* next, uint32_t* done) {
  if (threadIdx.x == 0) {
    const uint32_t k = atomicAdd(done, 1u);
    if (k == gridDim.x - 1) {
      atomicExch(next, 0u);
      atomicExch(done, 0u);
    }
  }
}

// ---------------------------------------------------------------------------
// Weights, weighted reduction and update (Sec. III-B weights, eq. (5))
// ---------------------------------------------------------------------------
// The weights exp(-(J_s - m)/lambda) and the weighted average of the applied
// inputs are formed in a fixed structure so that the result never depends on
// the launch shape: a unit of 32 samples takes weights relative to its own
// minimum, a group of 32 units rescales them to the group minimum, and the
// last block of the instance rescales the groups to the global minimum
// (log-sum-exp merges) and writes U_new, the receding-horizon shift and, when
// asked, the closed-loop plant step.

// FP64 plant step of the closed loop (Sec. II model, inputs clipped to the
// hard bounds), in two halves so that only the last few operations wait for
// the merge.  s_plant: [0..5] sin/cos of th1, delta, th1 - th2; [6..13] the
// state; [14..16] the applied input U_new[0].
constexpr int kPlantLds = 17;
// first half (no barrier): lanes 0..7 load the state, lanes 0..2 one sincos each
__device__ __forceinline__ void plant_prep(const SolveDesc& d, double* s_plant) {
  const uint32_t t = threadIdx.x;
  const double* x = d.plant_x;
  if (t < 8) lds_put(s_plant + 6 + t, x[t]);
  if (t < 3) {
    const double ang = t == 0 ? x[4] : (t == 1 ? x[6] : x[4] - x[5]);
    double sn, cs;
    sincos(ang, &sn, &cs);
    lds_put(s_plant + 2 * t, sn);
    lds_put(s_plant + 2 * t + 1, cs);
  }
}
// Hitch-angle stabiliser (Sec. IV-D, eq. (19)) in FP64: (j, w) <- argmin of
// q_j (j - j_ref)^2 + q_w (w - w_ref)^2 over the input box subject to
// Lf + g u >= -alpha_h hhat for both hitch rows (the first-order expanded
// barrier of the rollouts).  The optimum of this strictly convex 2-D problem
// is the reference, the projection onto one constraint line, or a vertex of
// two: every candidate is formed and the feasible one with the least cost
// kept.  No feasible input: the reference clipped to the box.
__device__ bool hitch_qp(const brmppi_params& P, const double x[8], const double* s_plant, double& j, double& w) {
  const double Ts = P.Ts, l1 = P.l1, l2 = P.l2;
  const double v = x[2], a = x[3], phi = x[4] - x[5];
  const double sp = s_plant[4], cp = s_plant[5];
  const double tn = s_plant[2] / s_plant[3], sec2 = 1.0 + tn * tn;
  const double ch = (double)P.lh / l1, kd = tn / l1;
  const double Aw2 = sp - ch * cp * tn;
  const double D = v / l2 * Aw2 - v * kd;
  const double D_v = Aw2 / l2 - kd;
  const double D_phi = v / l2 * (cp + ch * sp * tn);
  const double D_dl = -v * sec2 * (ch * cp / l2 + 1.0 / l1);
  double A[6][2], c[6];
  for (int k = 0; k < 2; ++k) {
    const double sg = k == 0 ? 1.0 : -1.0;
    const double h = (double)P.dtheta_max - (double)P.kappa * v + sg * phi;
    const double hd = -(double)P.kappa * a - sg * D;
    const double hv = -(double)P.kappa - sg * Ts * D_v;
    const double Lf = Ts * (hv * a - sg * (1.0 - Ts * D_phi) * D);
    A[k][0] = -(double)P.kappa * Ts * Ts;
    A[k][1] = -sg * Ts * Ts * D_dl;
    c[k] = -(double)P.alpha_h * (h + Ts * hd) - Lf;
  }
  A[2][0] = 1.0;  A[2][1] = 0.0;  c[2] = P.j_lo;
  A[3][0] = -1.0; A[3][1] = 0.0;  c[3] = -(double)P.j_hi;
  A[4][0] = 0.0;  A[4][1] = 1.0;  c[4] = P.w_lo;
  A[5][0] = 0.0;  A[5][1] = -1.0; c[5] = -(double)P.w_hi;
  const double q0 = P.qh_j, q1 = P.qh_w;
  const double r0 = j, r1 = w;
  double best = INFINITY, b0 = 0.0, b1 = 0.0;
  auto consider = [&](double u0, double u1) {
    for (int i = 0; i < 6; ++i) {
      const double lhs = A[i][0] * u0 + A[i][1] * u1;
      const double scale = fabs(c[i]) + fabs(A[i][0] * u0) + fabs(A[i][1] * u1) + 1e-300;
      if (lhs - c[i] < -1e-10 * scale) return;
    }
    const double e0 = u0 - r0, e1 = u1 - r1;
    const double obj = q0 * e0 * e0 + q1 * e1 * e1;
    if (obj < best) {
      best = obj;
      b0 = u0;
      b1 = u1;
    }
  };
  consider(r0, r1);
  for (int i = 0; i < 6; ++i) {
    const double aQa = A[i][0] * A[i][0] / q0 + A[i][1] * A[i][1] / q1;
    if (!(aQa > 0.0)) continue;
    const double lam = (c[i] - (A[i][0] * r0 + A[i][1] * r1)) / aQa;
    consider(r0 + A[i][0] / q0 * lam, r1 + A[i][1] / q1 * lam);
  }
  for (int i = 0; i < 6; ++i) {
    for (int k = i + 1; k < 6; ++k) {
      const double det = A[i][0] * A[k][1] - A[i][1] * A[k][0];
      const double nrm = fabs(A[i][0] * A[k][1]) + fabs(A[i][1] * A[k][0]);
      if (!(fabs(det) > 1e-14 * nrm)) continue;
      consider((c[i] * A[k][1] - c[k] * A[i][1]) / det, (A[i][0] * c[k] - A[k][0] * c[i]) / det);
    }
  }
  if (!(best < INFINITY)) return false;
  j = b0;
  w = b1;
  return true;
}

// second half, one thread, after a barrier
__device__ __forceinline__ void plant_finish(const SolveDesc& d, const double* s_plant) {
  const brmppi_params& P = d.prm;
  double x[8];
  for (int k = 0; k < 8; ++k) x[k] = lds(s_plant + 6 + k);
  double j = lds(s_plant + 14), w = lds(s_plant + 15);
  const double nu = lds(s_plant + 16);
  const bool stabilised = (d.flags & BRMPPI_HITCH_QP) && hitch_qp(P, x, s_plant, j, w);
  if (!stabilised) {   // hard input bounds on the applied input
    j = fmin(fmax(j, (double)P.j_lo), (double)P.j_hi);
    w = fmin(fmax(w, (double)P.w_lo), (double)P.w_hi);
  }
  const double Ts = P.Ts, l1 = P.l1, l2 = P.l2, lh = P.lh;
  const double v = x[2], a = x[3];
  const double s1 = lds(s_plant + 0), c1 = lds(s_plant + 1);
  const double tan_dl = lds(s_plant + 2) / lds(s_plant + 3);
  const double s12 = lds(s_plant + 4), c12 = lds(s_plant + 5);
  double xn[8];
  xn[0] = x[0] + Ts * v * c1;
  xn[1] = x[1] + Ts * v * s1;
  xn[2] = v + Ts * a;
  xn[3] = a + Ts * j;
  xn[4] = x[4] + Ts * v / l1 * tan_dl;
  xn[5] = x[5] + Ts * v / l2 * (s12 - lh / l1 * c12 * tan_dl);
  xn[6] = x[6] + Ts * w;
  xn[7] = x[7] + Ts * nu;
  for (int k = 0; k < 8; ++k) d.plant_x[k] = xn[k];
  // closed loop: the state after the update and the averaged first input
  if (d.log) {
    for (int k = 0; k < 8; ++k) d.log[k] = xn[k];
    float* u = reinterpret_cast<float*>(d.log + 8);
    for (int k = 0; k < 3; ++k) u[k] = (float)lds(s_plant + 14 + k);
  }
}

// block-wide reductions in a fixed order (thread stride, wave butterfly, waves
// in index order): the same inputs give the same bits on every launch
__device__ __forceinline__ float block_min(float v, float* s_red) {
  v = wave_min(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) lds_put(s_red + (threadIdx.x >> 6), v);
  __syncthreads();
  float r = lds(s_red);
  for (uint32_t w = 1; w < blockDim.x / 64; ++w) r = fminf(r, lds(s_red + w));
  return r;
}
// two sums with one pair of barriers (s_red: two floats per wave), each in the same
// order as a single block sum
__device__ __forceinline__ void block_sum2(float& a, float& b, float* s_red) {
  const uint32_t nw = blockDim.x / 64;
  a = wave_sum(a);
  b = wave_sum(b);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) {
    lds_put(s_red + (threadIdx.x >> 6), a);
    lds_put(s_red + nw + (threadIdx.x >> 6), b);
  }
  __syncthreads();
  float ra = lds(s_red), rb = lds(s_red + nw);
  for (uint32_t w = 1; w < nw; ++w) {
    ra += lds(s_red + w);
    rb += lds(s_red + nw + w);
  }
  a = ra;
  b = rb;
}

// One row of the result: the new nominal sequence, the log and plant step of its
// first input, and the receding-horizon shift U_nom <- [U[1:], U[T-1]]
__device__ __forceinline__ void put_result(const SolveDesc& d, uint32_t r, uint32_t R, float U, bool plant,
                                           double* s_plant) {
  gst(d.u_new + r, U);
  if (plant && r < 3) lds_put(s_plant + 14 + r, (double)U);
  if (r >= 3) gst(d.u_nom_out + r - 3, U);
  if (r + 3 >= R) gst(d.u_nom_out + r, U);
}
__device__ __forceinline__ const float* nominal_in(const SolveDesc& d) {
  return d.u_nom_in ? d.u_nom_in : reinterpret_cast<const float*>(&d + 1);
}
// every cost non-finite: return the nominal sequence, keep the warm start
__device__ __forceinline__ void put_nominal(const SolveDesc& d, uint32_t R, bool plant, double* s_plant) {
  for (uint32_t r = threadIdx.x; r < R; r += blockDim.x) {
    const float U = gld(nominal_in(d) + r);
    gst(d.u_new + r, U);
    if (plant && r < 3) lds_put(s_plant + 14 + r, (double)U);
  }
}
// statistics, plant step and its logs
__device__ __forceinline__ void finish_instance(const SolveDesc& d, float m, float Z, float Z2, bool ok, bool plant,
                                                double* s_plant) {
  if (threadIdx.x == 0) {
    d.stats[0] = m;
    d.stats[1] = Z;
    d.stats[2] = ok ? Z * Z / Z2 : 0.0f;
    d.stats[3] = ok ? (float)BRMPPI_OK : (float)BRMPPI_ENONFINITE;
  }
  if (plant) {
    __syncthreads();                 // U_new[0] from threads 0..2, the state and sines
    if (threadIdx.x == 0) plant_finish(d, s_plant);
  }
}

// Merge of the group partials (a group = 1024 samples) by the last block of an
// instance: global min m = min_c m_c, group scale exp(-(m_c - m)/lambda), Z
// and sum of squared weights, then U = sum_c scale_c rpart[c] / Z per row
// (eq. (5)).  Every load is issued by a different thread or unrolled, so the
// merge costs a few memory latencies, not one per group.
__device__ void finalize_instance(const SolveDesc& d, float* s_scale, float* s_red, double* s_plant) {
  const uint32_t nW = d.n_wchunk;
  const uint32_t R = 3 * d.T;
  const uint32_t nt = blockDim.x;
  const bool plant = (d.flags & BRMPPI_ADVANCE_PLANT) != 0;
  if (plant) plant_prep(d, s_plant);   // overlaps the merge
  // the first 8 group partials of this thread's first row, loaded before the
  // merge's barriers so that their latency overlaps them
  constexpr int kPre = 8;
  const uint32_t r0 = threadIdx.x;
  float pre[kPre];
#pragma unroll
  for (int k = 0; k < kPre; ++k) pre[k] = (r0 < R && (uint32_t)k < nW) ? pub_ld(d.rpart + (size_t)k * R + r0) : 0.0f;
  // this thread's first group partial is loaded once, for the minimum and the sums
  const float4 w_first = threadIdx.x < nW ? pub_ld4(d.wpart + threadIdx.x) : make_float4(INFINITY, 0.0f, 0.0f, 0.0f);
  float mloc = w_first.x;
  for (uint32_t c = threadIdx.x + nt; c < nW; c += nt) {
    mloc = fminf(mloc, pub_ld(&d.wpart[c].x));
  }
  const float m = block_min(mloc, s_red);
  float zl = 0.0f, z2l = 0.0f;
  for (uint32_t c = threadIdx.x; c < nW; c += nt) {
    const float4 w = c == threadIdx.x ? w_first : pub_ld4(d.wpart + c);
    const float sc = (m < INFINITY && w.x < INFINITY) ? expf(-(w.x - m) * d.inv_lambda) : 0.0f;
    lds_put(s_scale + c, sc);
    zl += sc * w.y;
    z2l += sc * sc * w.z;
  }
  block_sum2(zl, z2l, s_red);   // also orders the s_scale stores before the reads below
  const float Z = zl, Z2 = z2l;
  const bool ok = (m < INFINITY) && (Z > 0.0f);
  if (ok) {
    const float iZ = 1.0f / Z;
    for (uint32_t r = threadIdx.x; r < R; r += nt) {
      const float* __restrict__ col = d.rpart + r;
      float acc = 0.0f;
      uint32_t c = 0;
      for (; c + kPre <= nW; c += kPre) {
        const bool use_pre = (c == 0) && (r == r0);
        float v[kPre];
#pragma unroll
        for (int k = 0; k < kPre; ++k) v[k] = use_pre ? pre[k] : pub_ld(col + (size_t)(c + k) * R);
#pragma unroll
        for (int k = 0; k < kPre; ++k) acc += lds(s_scale + c + k) * v[k];
      }
#pragma unroll
      for (int k = 0; k < kPre; ++k) {
        if (c + k < nW) {
          const float vk = (c == 0 && r == r0) ? pre[k] : pub_ld(col + (size_t)(c + k) * R);
          acc += lds(s_scale + c + k) * vk;
        }
      }
      put_result(d, r, R, acc * iZ, plant, s_plant);
    }
  } else {
    put_nominal(d, R, plant, s_plant);
  }
  finish_instance(d, m, Z, Z2, ok, plant, s_plant);
}

// ---------------------------------------------------------------------------
// Canonical reduction primitives (Sec. III-B weights and eq. (5)).  The fused
// rollout epilogue and k_reduce both call exactly these, so a unit's or a
// group's partial has the same bits whichever kernel computes it.
// ---------------------------------------------------------------------------
// weight of a sample relative to its unit's minimum m (0 for non-finite costs
// and samples past S, which carry J = +inf)
__device__ __forceinline__ float unit_weight(float j, float m, float inv_lambda) {
  return (m < INFINITY && j < INFINITY) ? expf(-(j - m) * inv_lambda) : 0.0f;
}
// Z_u and the sum of squared weights over the unit's samples, in sample order
__device__ __forceinline__ void unit_sums(const float* gam, float& z, float& z2) {
  z = 0.0f;
  z2 = 0.0f;
#pragma unroll
  for (int i = 0; i < kUnit; ++i) {
    const float gm = lds(gam + i);
    z = z + gm;
    z2 = fmaf(gm, gm, z2);
  }
}
// one term of a unit's row sum: zero weights leave the sum as it is (samples
// past S hold no data)
__device__ __forceinline__ float unit_row_term(float acc, float gm, float u) {
  return gm != 0.0f ? fmaf(gm, u, acc) : acc;
}
// scale of a unit (or group) with minimum m inside a merge with minimum mg
__device__ __forceinline__ float merge_scale(float m, float mg, float inv_lambda) {
  return (mg < INFINITY && m < INFINITY) ? expf(-(m - mg) * inv_lambda) : 0.0f;
}
// group (Z, Z2) from its units' (m_u, Z_u, Z2_u) and scales, in unit order
// (entries are read kChunk at a time, in bounds, before any of them is used,
// so that the reads are not serialised behind the per-unit condition)
constexpr int kChunk = 8;
__device__ __forceinline__ void group_sums(const float4* up, const float* sig, uint32_t nu, float& z, float& z2) {
  z = 0.0f;
  z2 = 0.0f;
#pragma unroll
  for (int c = 0; c < kGroupUnits; c += kChunk) {
    float sc[kChunk];
    float4 q[kChunk];
#pragma unroll
    for (int k = 0; k < kChunk; ++k) {
      q[k] = lds(up + c + k);
      sc[k] = lds(sig + c + k);
    }
#pragma unroll
    for (int k = 0; k < kChunk; ++k) {
      if ((uint32_t)(c + k) < nu) {
        z = fmaf(sc[k], q[k].y, z);
        z2 = fmaf(sc[k] * sc[k], q[k].z, z2);
      }
    }
  }
}

// Group merge by the last tile of the group: m_g, unit scales, (Z_g, Z2_g)
// and the group row sums from the units' partials.
// put_part(m_g, Z_g, Z2_g) runs on one thread, put_row(r, sum) on the row's.
template <typename PutPart, typename PutRow>
__device__ __forceinline__ void group_merge(const SolveDesc& d, uint32_t gu0, uint32_t nu_g, float* s_sig,
                                            float4* s_up, float* s_red, PutPart put_part, PutRow put_row) {
  const uint32_t t = threadIdx.x, nt = blockDim.x, R = 3 * d.T;
  // this thread's first row: all the group's unit sums, loaded before the
  // minimum (they do not depend on it)
  // (units past nu_g read the group's last unit, in range; only terms of units
  // below nu_g are ever used)
  float v0[kGroupUnits];
  {
    const float* __restrict__ col = d.urow + (size_t)gu0 * R + (t < R ? t : 0);
#pragma unroll
    for (int u = 0; u < kGroupUnits; ++u) v0[u] = pub_ld(col + (size_t)min((uint32_t)u, nu_g - 1) * R);
  }
  float4 up = make_float4(INFINITY, 0.0f, 0.0f, 0.0f);
  if (t < nu_g) up = pub_ld4(d.upart + gu0 + t);
  const float mg = block_min(up.x, s_red);
  if (t < nu_g) {
    lds_put(s_up + t, up);
    lds_put(s_sig + t, merge_scale(up.x, mg, d.inv_lambda));
  }
  __syncthreads();
  // the group's (Z, Z2), on the first thread of a wave without a row when there
  // is one, so that it overlaps the row sums instead of preceding them
  const uint32_t tz = ((R + 63u) & ~63u) < nt ? ((R + 63u) & ~63u) : 0u;
  if (t == tz) {
    float z, z2;
    group_sums(s_up, s_sig, nu_g, z, z2);
    put_part(mg, z, z2);
  }
  // one row: its unit sums in v, the scales read kChunk at a time (in bounds,
  // before any of them is used)
  auto row_sum = [&](uint32_t r, const float* v) __attribute__((always_inline)) {
    float acc = 0.0f;
#pragma unroll
    for (int c = 0; c < kGroupUnits; c += kChunk) {
      float sg[kChunk];
#pragma unroll
      for (int k = 0; k < kChunk; ++k) sg[k] = lds(s_sig + c + k);
#pragma unroll
      for (int k = 0; k < kChunk; ++k)
        if ((uint32_t)(c + k) < nu_g) acc = unit_row_term(acc, sg[k], v[c + k]);
    }
    put_row(r, acc);
  };
  if (t < R) row_sum(t, v0);
  for (uint32_t r = t + nt; r < R; r += nt) {
    // all the group's unit sums of this row are loaded at once: one latency
    const float* __restrict__ col = d.urow + (size_t)gu0 * R + r;
    float v[kGroupUnits];
#pragma unroll
    for (int u = 0; u < kGroupUnits; ++u) v[u] = pub_ld(col + (size_t)min((uint32_t)u, nu_g - 1) * R);
    row_sum(r, v);
  }
}

// Waves per SIMD the register allocation must leave room for.  Up to 16
// obstacle slots every launch shape is held to two waves, and so are the four- and
// eight-lane forms with 32 slots (a lane holds 8 or 4 obstacle rows).  The forms that
// the default shape takes spill 0 to 20 values there (58 with 16 slots on two lanes that
// draw), which still pays: at one wave per SIMD nothing hides the step's latency.  Of the
// others, one lane with precomputed normals spills 176 (8 slots) and 632 (16), one lane
// that draws 208 (16 slots).  The one- and two-lane forms with 32 slots keep the whole
// register file (112 spilled with one lane and precomputed normals, none otherwise).
template <int NOB, int G>
constexpr int rollout_waves_per_simd() {
  return (NOB <= 16 || G >= 4) ? 2 : 1;
}
// Waves per SIMD that the schedule may assume.  Without rows the registers are the
// instance merge's 134, three waves; scheduled for four, the penalty's loop over
// obstacles waits for each one's LDS reads (60000 samples, 90 steps, 24 obstacles, four
// lanes: 207 us against 187).
template <int NOB>
constexpr int rollout_waves_max() {
  return NOB == 0 ? 3 : 8;
}

// Fused reduction of one tile (its samples' costs and applied inputs are in
// LDS): unit weights, unit partials to HBM; the last tile of each group merges
// the group, the last group the instance (U_new, shift, plant step).
// Inlined into the kernel: as a function call, every lane saved and restored
// its callee-saved registers around it (tens of bytes of scratch per lane).
__device__ __forceinline__ void tile_epilogue(const SolveDesc& d, uint32_t s0, uint32_t per_tile, float* s_u, uint32_t lds_stride,
                              const float* s_J, float* s_gam, float* s_mu, float* s_sig, float4* s_up,
                              float* s_red, double* s_trig, uint32_t* s_flag) {
  const uint32_t t = threadIdx.x, nt = blockDim.x, R = 3 * d.T;
  const uint32_t k_units = per_tile / kUnit;
  const uint32_t u0 = s0 / kUnit;
  const uint32_t nu_tile = min(k_units, d.n_units - u0);
  // unit minimum (exact in any order) and weights; a unit is half a wave
  if (t < per_tile) {
    const float j = lds(s_J + t);
    float m = j;
#pragma unroll
    for (int o = kUnit / 2; o >= 1; o >>= 1) m = fminf(m, __shfl_xor(m, o, 64));
    lds_put(s_gam + t, unit_weight(j, m, d.inv_lambda));
    if ((t & (kUnit - 1)) == 0) lds_put(s_mu + t / kUnit, m);
  }
  __syncthreads();
  if (t < nu_tile) {
    float z, z2;
    unit_sums(s_gam + kUnit * t, z, z2);
    pub_st4(d.upart + u0 + t, make_float4(lds(s_mu + t), z, z2, 0.0f));
  }
  for (uint32_t it = t; it < nu_tile * R; it += nt) {
    const uint32_t j = it / R, r = it - j * R;
    const float* gam = s_gam + kUnit * j;
    const float* u = s_u + r * lds_stride + kUnit * j;
    float acc = 0.0f;
#pragma unroll
    for (int c = 0; c < kUnit; c += kChunk) {
      float g8[kChunk], u8[kChunk];
#pragma unroll
      for (int k = 0; k < kChunk; ++k) {
        g8[k] = lds(gam + c + k);
        u8[k] = lds(u + c + k);
      }
#pragma unroll
      for (int k = 0; k < kChunk; ++k) acc = unit_row_term(acc, g8[k], u8[k]);
    }
    pub_st(d.urow + (size_t)(u0 + j) * R + r, acc);
  }
  // publish the tile's units; the last tile of the group merges it
  const uint32_t grp = u0 / kGroupUnits, gu0 = grp * kGroupUnits;
  const uint32_t nu_g = min((uint32_t)kGroupUnits, d.n_units - gu0);
  const uint32_t tiles_g = (nu_g + k_units - 1) / k_units;
  pub_complete();
  __syncthreads();
  if (t == 0) *s_flag = (atomicAdd(&d.gctr[grp * kCtrStride], 1u) == tiles_g - 1) ? 1u : 0u;
  __syncthreads();
  if (*s_flag == 0u) return;
  if (t == 0) atomicExch(&d.gctr[grp * kCtrStride], 0u);
  group_merge(
      d, gu0, nu_g, s_sig, s_up, s_red,
      [&](float m, float z, float z2) { pub_st4(d.wpart + grp, make_float4(m, z, z2, 0.0f)); },
      [&](uint32_t r, float sum) { pub_st(d.rpart + (size_t)grp * R + r, sum); });
  // publish the group; the last group merges the instance
  pub_complete();
  __syncthreads();
  if (d.n_wchunk > 1) {
    if (t == 0) {
      const bool last = atomicAdd(d.counter, 1u) == d.n_wchunk - 1;
      if (last) atomicExch(d.counter, 0u);
      *s_flag = last ? 1u : 0u;
    }
    __syncthreads();
    if (*s_flag == 0u) return;
  }
  finalize_instance(d, s_u, s_red, s_trig);   // the inputs' LDS is free: merge scales
}

// Where a tile's instance starts: the start state, the path index of its start
// progress (k0 + phi0) and the window of the path staged in LDS (nw waypoints
// from w0)
struct TileStart {
  float x0[8];
  int k0, w0, nw;
  float phi0;
};

// Where a tile's instance starts, from its descriptor
__device__ __forceinline__ void tile_start(const SolveDesc& d, TileStart& st) {
  float (&x0)[8] = st.x0;
  if (d.x0_resident) {
#pragma unroll
    for (int k = 0; k < 8; ++k) x0[k] = (float)d.plant_x[k];
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k) x0[k] = d.x0[k];
  }
  // progress origin: f0 = psi0/ds = k0 + phi0
  const double f0 = (double)x0[7] / (double)d.ds;
  double fk = floor(f0);
  fk = fmin(fmax(fk, -1.0e9), 1.0e9);
  const int k0 = (int)fk;
  st.k0 = k0;
  st.phi0 = (float)(f0 - fk);
  const int n_path = (int)d.n_path;
  int w0 = k0 - kPathBack;
  if (w0 < 0) w0 = 0;
  if (w0 > n_path - 2) w0 = n_path - 2;
  int nw = n_path - w0;
  if (nw > kPathWin) nw = kPathWin;
  st.w0 = w0;
  st.nw = nw;
}

// Stages a tile's instance into LDS by the block's first bd threads (at least
// 64): the path window, the nominal inputs and the obstacle rows.  The caller's
// barrier completes it.
__device__ __forceinline__ void stage_tile(const SolveDesc& d, float4* s_path, float4* s_unom, ObsL* s_obs,
                                           const TileStart& st, int bd) {
  const Frame F = frame_at(st.x0[0], st.x0[1], st.x0[4]);
  const int w0 = st.w0, nw = st.nw;
  // stage the obstacle rows (row r: obstacle r % n_objects around footprint
  // disc r / n_objects) and the path window
  if (threadIdx.x < d.n_obs) {
    const uint32_t oi = threadIdx.x % d.n_objects;
    const brmppi_obstacle o = d.obs[oi];
    const float ax = o.mx + d.prm.r_disc, ay = o.my + d.prm.r_disc;
    const float iax = 1.0f / (ax * ax), iay = 1.0f / (ay * ay);
    float so, co;
    sincosf(o.heading, &so, &co);
    into_frame(F, co, so);
    ObsL L;
    L.cx = fmaf(o.vx, d.t0, o.cx - F.ox);
    L.cy = fmaf(o.vy, d.t0, o.cy - F.oy);
    into_frame(F, L.cx, L.cy);
    L.mx = d.prm.Ts * o.vx;
    L.my = d.prm.Ts * o.vy;
    into_frame(F, L.mx, L.my);
    L.q11 = co * co * iax + so * so * iay;
    L.q12 = co * so * (iax - iay);
    L.q22 = so * so * iax + co * co * iay;
    L.qa = 0.5f * (iax + iay);
    L.qd = 0.5f * (iax - iay) * (co * co - so * so);
    L.rx = fmaf(L.q12, L.my, L.q11 * L.mx);
    L.ry = fmaf(L.q22, L.my, L.q12 * L.mx);
    L.rr = fmaf(L.ry, L.my, L.rx * L.mx);
    L.e4 = (o.e == 4.0f) ? 1.0f : 0.0f;
    L.a00 = co / ax;
    L.a01 = so / ax;
    L.a10 = -so / ay;
    L.a11 = co / ay;
    L.pad = 0.0f;
    disc_ab(d.prm, threadIdx.x / d.n_objects, L.dA, L.dB);
    s_obs[threadIdx.x] = L;
  } else if (threadIdx.x < BRMPPI_MAX_OBS) {
    // blank slots (Q = A = 0, at rest): the rows of lanes past the last
    // obstacle row
    s_obs[threadIdx.x] = ObsL{};
  }
  // the path window and the nominal inputs, their
  // first loads all issued before the first store (the window's 4 per thread
  // at 256 threads): one memory latency, not one per value a thread stages
  const int Ti = (int)d.T, tx = (int)threadIdx.x;
  const float* un_in = nominal_in(d);
  auto load_un = [&](int tau) __attribute__((always_inline)) {
    const float* p = un_in + 3 * min(tau, Ti - 1);
    return make_float4(gld(p), gld(p + 1), gld(p + 2), 0.0f);
  };
  const float4 un0 = load_un(tx);
  for (int j0 = 0; j0 < nw; j0 += 4 * bd) {
    float4 w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = d.path[w0 + min(j0 + k * bd + tx, nw - 1)];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int j = j0 + k * bd + tx;
      if (j < nw) s_path[j] = into_frame(F, w[k]);
    }
  }
  if (tx == 0) {   // the frame, for the points outside of the window
    s_path[kPathWin] = make_float4(F.ox, F.oy, F.turn, F.c);
    s_path[kPathWin + 1].x = F.s;
  }
  if (tx < Ti) s_unom[tx] = un0;
  for (int tau = tx + bd; tau < Ti; tau += bd) s_unom[tau] = load_un(tau);
}

// The rollouts of a staged tile from sample s0 on, G threads each.  Every lane
// runs (lanes past S repeat the last sample and do not store), so the
// group-wide DPP broadcasts always read active lanes.
struct NoRun {
  __device__ __forceinline__ uint32_t operator()(uint32_t) const { return 0; }
};
template <int NOB, bool GUIDED, int G, int NOISE, typename NextRun = NoRun>
__device__ __forceinline__ void tile_rollout(const SolveDesc& d, uint32_t s0, const TileStart& st,
                                             const float4* s_path, const float4* s_unom, const ObsL* s_obs,
                                             float* s_u, uint32_t lds_stride, float* s_J, float* s_nrm,
                                             uint32_t run_end = 0, NextRun next_run = NextRun{}) {
  const uint32_t t_local = threadIdx.x / G;
  const uint32_t s_raw = s0 + t_local;
  const int g = (int)(threadIdx.x % G);
  const bool valid = s_raw < d.S;
  const uint32_t s = valid ? s_raw : d.S - 1;
  auto rollout = [&](auto ROWS) __attribute__((always_inline)) {
    rollout_sample<NOB, GUIDED, G, NOISE, decltype(ROWS)::value>(d, s, valid && g == 0, g, st.x0, s_obs, s_path, s_unom,
                                                              st.w0, st.nw, st.k0, st.phi0, s_u, lds_stride, t_local,
                                                              s_J, s_nrm, run_end, next_run);
  };
  if constexpr (GUIDED) {
    if (d.row_kind == kRowsDisc) rollout(std::integral_constant<int, kRowsDisc>{});
    else if (d.row_kind == kRowsE4) rollout(std::integral_constant<int, kRowsE4>{});
    else if (d.row_kind == kRowsMoving) rollout(std::integral_constant<int, kRowsMoving>{});
    else rollout(std::integral_constant<int, kRowsStatic>{});
  } else {
    // no rows: the kinds matter to the collision penalty alone
    if (d.row_kind == kRowsDisc) rollout(std::integral_constant<int, kRowsDisc>{});
    else rollout(std::integral_constant<int, kRowsE4>{});
  }
}

// Rollout of one instance (a direct launch, a tile per block).
template <int NOB, bool GUIDED, int G, bool PRE>
__global__ __launch_bounds__(kMaxBlock) __attribute__((amdgpu_waves_per_eu(rollout_waves_per_simd<NOB, G>(), rollout_waves_max<NOB>())))
void k_rollout(const SolveDesc* __restrict__ desc) {
  __shared__ float4 s_path[kPathLds];
  __shared__ float4 s_unom[BRMPPI_MAX_T + 1];
  __shared__ ObsL s_obs[BRMPPI_MAX_OBS];
  __shared__ uint32_t s_flag;
  __shared__ float s_red[2 * (kMaxBlock / 64)];
  __shared__ double s_trig[kPlantLds];
  constexpr bool kCoop = !PRE && G > 1;
  __shared__ float4 s_nrm[kCoop ? kMaxBlock / G * coop_stride<NOB, G>() / 4 : 1];
  extern __shared__ float s_dyn[];            // fused epilogue only
  const uint32_t per_tile = blockDim.x / G;   // samples per tile
  const uint32_t lds_stride = per_tile + 1;
  const uint32_t s0 = blockIdx.x * per_tile;
  const SolveDesc& d = *desc;
  TileStart st;
  tile_start(d, st);
  stage_tile(d, s_path, s_unom, s_obs, st, (int)blockDim.x);
  // fused epilogue: LDS for the tile's applied inputs, costs (+inf where no
  // sample stores), weights, units
  const bool fused = d.fused != 0;
  float *s_u = nullptr, *s_J = nullptr, *s_gam = nullptr, *s_mu = nullptr, *s_sig = nullptr;
  float4* s_up = nullptr;
  if (fused) {
    s_u = s_dyn;
    s_J = s_dyn + fused_lds_region(per_tile, d.T, d.n_wchunk);
    s_gam = s_J + per_tile;
    s_mu = s_gam + per_tile;
    s_sig = s_mu + kGroupUnits;
    s_up = reinterpret_cast<float4*>(s_sig + kGroupUnits);
    for (uint32_t i = threadIdx.x; i < per_tile; i += blockDim.x) s_J[i] = INFINITY;
  }
  __syncthreads();
  tile_rollout<NOB, GUIDED, G, PRE ? kBuffer : kOwnDraw>(d, s0, st, s_path, s_unom, s_obs, s_u, lds_stride, s_J,
                                                         reinterpret_cast<float*>(s_nrm));
  if (!fused) return;
  __syncthreads();
  tile_epilogue(d, s0, per_tile, s_u, lds_stride, s_J, s_gam, s_mu, s_sig, s_up, s_red, s_trig, &s_flag);
}

// Rollout of one instance of up to one block per CU: eight lanes per sample on
// the block's first four waves, one on each SIMD.  The normals of a run of steps
// (as many as LDS holds: 50 steps of 8 rows in two runs, 162 of 32 in 14) are drawn by all eight
// waves before the first four take the steps: two waves on a SIMD draw in half
// the time of one, which issues an instruction every 4 cycles where most take 2 of
// the pipe.  (Four waves that draw while the others take the steps cost the
// steps more than the draws take apart from them: 49.2 us against 47.2, 8192
// samples, 50 steps, 8 obstacles.)  The inputs are the launch's arguments, so that
// an update is one launch.  Measured against the noise kernel's launch and then
// the rollout's: that update 62.7 -> 57.2 us, 512 samples of 20 steps 40.9 -> 37.8,
// 5000 of 120 steps without guidance 61.2 -> 54.2, with 8 obstacles 124.0 -> 119.6,
// 4096 of 60 steps and 32 rows 140 on both sides (its normals take three runs; drawn_fits
// has the limit of that).
// What bounds it is the chain of steps, 0.6 us each, at one wave a SIMD.
template <int NOB, bool GUIDED>
__global__ __launch_bounds__(2 * kMaxBlock) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_rollout_drawn(const SolveArgs) {
  __shared__ float4 s_unom[kInlineSteps + 1];
  __shared__ ObsL s_obs[BRMPPI_MAX_OBS];
  __shared__ uint32_t s_flag;
  __shared__ float s_red[2 * (2 * kMaxBlock / 64)];
  __shared__ double s_trig[kPlantLds];
  extern __shared__ float4 s_drawn[];         // as drawn_lds lays it out
  static_assert(sizeof(s_unom) + sizeof(s_obs) + sizeof(s_flag) + sizeof(s_red) + sizeof(s_trig) + 64 <= kDrawnStatic,
                "with padding");
  constexpr int G = 8, kStride = run_stride<NOB, GUIDED>();
  constexpr uint32_t kAhead = 32;             // a multiple of kMaxBlock / kDrawnTile
  const uint32_t per_tile = kDrawnTile, lds_stride = per_tile + 1;
  const uint32_t s0 = blockIdx.x * per_tile;
  // the argument itself, not a copy of it
  const SolveArgs& a = *(const SolveArgs*)__builtin_amdgcn_kernarg_segment_ptr();
  const SolveDesc& d = a.d;
  const uint32_t T = d.T, run = a.run;
  float* s_nrm = reinterpret_cast<float*>(s_drawn);
  static_assert(4 * kDrawnTile * kStride == drawn_slot(NOB), "a slot of the run");
  float4* s_path = reinterpret_cast<float4*>(s_nrm + run * (per_tile * kStride));
  float* s_u = reinterpret_cast<float*>(s_path + kPathLds);
  float* s_J = s_u + fused_lds_region(per_tile, T, d.n_wchunk);
  float* s_gam = s_J + per_tile;
  float* s_mu = s_gam + per_tile;
  float* s_sig = s_mu + kGroupUnits;
  float4* s_up = reinterpret_cast<float4*>(s_sig + kGroupUnits);
  if (threadIdx.x < per_tile) s_J[threadIdx.x] = INFINITY;
  // the first four waves stage the tile, its loads in flight while the others
  // begin to draw
  const bool rolls = __builtin_amdgcn_readfirstlane(threadIdx.x) < kMaxBlock;
  TileStart st;
  if (rolls) {
    tile_start(d, st);
    stage_tile(d, s_path, s_unom, s_obs, st, kMaxBlock);
  }
  // a run's blocks of four normals, 32 samples each: (step, block) q.  The last
  // four waves take the first `ahead` of them (8 at a time), then all eight go on.
  const uint32_t nb = GUIDED ? (5 + d.n_obs + 3) / 4 : 1u, inv_nb = 65536u / nb + 1u;
  auto draw = [&](uint32_t tau0, uint32_t ahead) __attribute__((always_inline)) -> uint32_t {
    const uint32_t end = min(tau0 + run, T), n = (end - tau0) * nb;
    const uint32_t j = threadIdx.x % per_tile, s = min(s0 + j, d.S - 1);
    constexpr uint32_t kHalf = kMaxBlock / kDrawnTile;
    uint32_t q = threadIdx.x / per_tile;
    q = rolls ? ahead + kHalf + q : q - kHalf;
    // two at a time: their chains of dependent instructions overlap (past the
    // last one, that one again)
    while (q < n) {
      const uint32_t q1 = q + (q < ahead ? kHalf : 2 * kHalf);
      float e[2][4];
      uint32_t at[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const uint32_t qk = min(k ? q1 : q, n - 1);
        const uint32_t i = (qk * inv_nb) >> 16, b = qk - i * nb;   // qk / nb, exact: qk < 10 * 162
        uint32_t r[4];
        philox4x32_10(s, tau0 + i, b, d.instance, d.seed_lo, d.seed_hi, r);
        box_muller4(r, e[k]);
        at[k] = (i * per_tile + j) * kStride + 4 * b;
      }
#pragma unroll
      for (int k = 0; k < 2; ++k)
        lds_put(reinterpret_cast<float4*>(s_nrm + at[k]), make_float4(e[k][0], e[k][1], e[k][2], e[k][3]));
      q = q1 + (q1 < ahead ? kHalf : 2 * kHalf);
    }
    __syncthreads();
    return end;
  };
  uint32_t end = draw(0, kAhead);
  if (rolls) {
    tile_rollout<NOB, GUIDED, G, kRuns>(d, s0, st, s_path, s_unom, s_obs, s_u, lds_stride, s_J, s_nrm, end,
                                        [&](uint32_t tau) __attribute__((always_inline)) {
                                          __syncthreads();   // the run's normals have been read
                                          return draw(tau, 0);
                                        });
  } else {
    while (end != T) {
      __syncthreads();
      end = draw(end, 0);
    }
  }
  __syncthreads();
  tile_epilogue(d, s0, per_tile, s_u, lds_stride, s_J, s_gam, s_mu, s_sig, s_up, s_red, s_trig, &s_flag);
}

// Rollouts of a batch: one persistent launch over the tiles of all its
// instances, longest first, each tile in the in-kernel-noise form of its
// instance's constraint bucket (d.bucket): one lane per sample up to eight
// rows, two up to 16, four up to 32.  One launch per bucket, one after the
// other, left the device to the last tiles of each; a bucket too small for a
// launch of its own ran in the next heavier kernel.  The forms are held to the 256
// registers of two waves per SIMD; 106 of their values spill.  What bounds it is the vector pipe: at two
// waves per SIMD about 2700 of its cycles a wave and step (2 per FP32
// instruction on vector registers, 4 per FP64, comparison or scalar-operand
// one, 8 per transcendental), 80 % of the launch.  Measured, launch per bucket
// -> this: 64 instances (1024 to 16384 samples, 20 to 80 steps, up to 16
// obstacles) 765 -> 745 us a call (685 since), 48 served requests (up to 32768
// samples, 100 steps, 32 obstacles) 2813 -> 2125 us (2030 since).
// A batch without guidance has a kernel of its own (GUIDED false): 120 registers and
// less LDS, four waves per SIMD where the common one has two (16 instances of 32768
// samples, 60 steps: 296 -> 270 us, with the penalty over 24 obstacles 720 -> 542).
template <bool GUIDED>
__global__ __launch_bounds__(kMaxBlock) __attribute__((amdgpu_waves_per_eu(2, GUIDED ? 8 : 4)))
void k_rollout_batch(const SolveDesc* __restrict__ descs, const Tile* __restrict__ tiles, uint32_t n_tiles,
                     BatchCounters* __restrict__ ctr) {
  __shared__ float4 s_path[kPathLds];
  __shared__ float4 s_unom[BRMPPI_MAX_T + 1];
  __shared__ ObsL s_obs[BRMPPI_MAX_OBS];
  __shared__ uint32_t s_tile;
  constexpr int kNrm2 = kMaxBlock / 2 * coop_stride<16, 2>() / 4, kNrm4 = kMaxBlock / 4 * coop_stride<32, 4>() / 4;
  __shared__ float4 s_nrm4[!GUIDED ? 1 : (kNrm2 > kNrm4 ? kNrm2 : kNrm4)];
  float* s_nrm = reinterpret_cast<float*>(s_nrm4);
  for (uint32_t it = 0;; ++it) {
    uint32_t tix;
    if (!next_item(it, n_tiles, &ctr->tile_next, &s_tile, tix)) break;
    const Tile tl = tiles[tix];
    const SolveDesc& d = descs[__builtin_amdgcn_readfirstlane(tl.inst)];
    TileStart st;
    tile_start(d, st);
    stage_tile(d, s_path, s_unom, s_obs, st, (int)blockDim.x);
    __syncthreads();
    auto run = [&](auto NOB, auto GD, auto G) __attribute__((always_inline)) {
      tile_rollout<decltype(NOB)::value, decltype(GD)::value, decltype(G)::value, kOwnDraw>(
          d, tl.s0, st, s_path, s_unom, s_obs, nullptr, 0, nullptr, s_nrm);
    };
    using std::integral_constant;
    if constexpr (!GUIDED) {
      run(integral_constant<int, 0>{}, std::false_type{}, integral_constant<int, 1>{});
    } else {
      switch (d.bucket) {
        case 0: run(integral_constant<int, 0>{}, std::false_type{}, integral_constant<int, 1>{}); break;
        case 2: run(integral_constant<int, 2>{}, std::true_type{}, integral_constant<int, 1>{}); break;
        case 8: run(integral_constant<int, 8>{}, std::true_type{}, integral_constant<int, 1>{}); break;
        case 16: run(integral_constant<int, 16>{}, std::true_type{}, integral_constant<int, 2>{}); break;
        default: run(integral_constant<int, 32>{}, std::true_type{}, integral_constant<int, 4>{}); break;
      }
    }
    __syncthreads();
  }
  finish_persistent(&ctr->tile_next, &ctr->tile_done);
}

constexpr uint32_t kMaxWChunks = BRMPPI_MAX_S / kWChunk;
static_assert(kRowsPerPass == 2 * (kWThreads / 64), "two rows per wave and pass");
static_assert(kMaxRowsPerItem % kRowsPerPass == 0 && kMaxRowsPerItem <= kWThreads, "whole passes");
static_assert(kWChunk == 4 * kWThreads, "four samples per thread");
static_assert(kUnit == 32 && kGroupUnits == 32, "a unit is half a wave; a group's units fit one wave");

// Reduction from the applied inputs in HBM (batched launches and tiles that
// are not whole units), with the same canonical structure as the fused
// epilogue.  Work item = (group of 1024 samples, d.rows_item rows, up to
// 256): the group's unit weights are recomputed from its 4 KB of costs (same
// code: same values), the first row block also stores the group's (m_g, Z_g,
// Z2_g).  Wave w owns the group's samples 256 w .. 256 w + 255 (units 8 w ..
// 8 w + 7) and takes the item's rows 8 at a time: each row is read with one
// coalesced 16-byte load per lane, the 8 rows go through a padded LDS tile of
// the wave, and lane l then sums unit l % 8 of row l / 8 over its 32 samples
// in sample order (the weights of its unit are held in registers).  The next
// two passes' loads are in flight meanwhile.  The unit sums go to LDS and are
// merged in unit order by one thread per row; the item is published once.
// The last block of the instance merges the groups, with the group scales in
// the tiles' LDS.  Two blocks share a CU (LDS).
constexpr int kRedRows = 8;                          // rows per wave and pass
constexpr int kRedUnitStride = kUnit + 4;            // floats per unit segment in the tile (16 B pad)
constexpr int kRedRowStride = 8 * kRedUnitStride;    // floats per row of a wave's tile
static_assert(kRedRows * 8 == 64, "one (row, unit) pair per lane");

__global__ __launch_bounds__(kWThreads) void k_reduce(const SolveDesc* __restrict__ descs,
                                                     const Item* __restrict__ items, uint32_t n_items,
                                                     BatchCounters* __restrict__ ctr) {
  __shared__ float4 s_gam4[kWChunk / 4];
  __shared__ float s_mu[kGroupUnits], s_sig[kGroupUnits];
  __shared__ float4 s_up[kGroupUnits];
  __shared__ float s_R[kMaxRowsPerItem][kGroupUnits + 1];   // +1: row-wise reads hit distinct banks
  __shared__ float4 s_T4[(kWThreads / 64) * kRedRows * kRedRowStride / 4];
  __shared__ float s_red[2 * (kWThreads / 64)];
  __shared__ double s_trig[kPlantLds];
  __shared__ uint32_t s_slot, s_last;
  const uint32_t t = threadIdx.x;
  const int lane = t & 63, wid = t >> 6;
  const float* s_gam = reinterpret_cast<const float*>(s_gam4);
  float* s_T = reinterpret_cast<float*>(s_T4) + wid * (kRedRows * kRedRowStride);
  // the instance merge's group scales use the tiles' LDS (free by then)
  float* s_scale = reinterpret_cast<float*>(s_T4);
  static_assert(sizeof(s_T4) >= kMaxWChunks * sizeof(float), "group scales fit the tiles");
  // this lane's place in the wave's tile when storing (sample 4 lane of each
  // row) and when summing (unit lu of row lr)
  const uint32_t st_off = (uint32_t)(lane >> 3) * kRedUnitStride + 4 * (uint32_t)(lane & 7);
  const uint32_t lu = (uint32_t)lane & 7u, lr = (uint32_t)lane >> 3;
  for (uint32_t it = 0;; ++it) {
    uint32_t ix;
    if (!next_item(it, n_items, ctr ? &ctr->r_next : nullptr, &s_slot, ix)) break;
    Item item;
    if (items) {
      item = items[ix];
    } else {
      item.inst = 0;
      item.idx = ix;
    }
    const SolveDesc& d = descs[__builtin_amdgcn_readfirstlane(item.inst)];
    const uint32_t grp = item.idx / d.n_rgroup, rg = item.idx % d.n_rgroup;
    const uint32_t base = grp * kWChunk;
    const uint32_t R = 3 * d.T;
    const uint32_t S = d.S;
    const uint32_t gu0 = grp * kGroupUnits;
    const uint32_t nu_g = min((uint32_t)kGroupUnits, d.n_units - gu0);
    const uint32_t r0 = rg * d.rows_item;
    const uint32_t nrow = min(d.rows_item, R - r0);

    // thread t: samples 4t .. 4t + 3 of the group (unit t / 8); S_pad is a
    // multiple of 256, so a wave's samples are all inside the buffer or none.
    // Every load below is unconditional (a wave past S_pad reads the row's
    // last 16 bytes and gets weight 0), so that a wait for one pass's rows
    // can leave the next pass's loads in flight.
    const uint32_t s4 = base + 4 * t;
    const bool sv = s4 < d.S_pad;
    const uint32_t s4c = sv ? s4 : d.S_pad - 4;
    const float* __restrict__ colp = d.u_star + s4c;
    // the costs first: waiting for them does not wait for the rows
    const float4 jc = gld4(reinterpret_cast<const float4*>(d.J + s4c));
    // two passes of 8 rows in flight: pass p (p / 8 even) in slot 0, the next
    // in slot 1; a slot is refilled with the pass 16 rows on as soon as its
    // rows are in the tile.  Rows past nrow repeat the item's last row (cache
    // hits; their sums are not stored): with no branch around a load, the
    // wait for one slot never drains the other.
    float4 q[2][kRedRows];
    auto load_rows = [&](uint32_t p, auto SLOT) __attribute__((always_inline)) {
      constexpr int sl = decltype(SLOT)::value;
#pragma unroll
      for (int j = 0; j < kRedRows; ++j) {
        const uint32_t rr = min(p + (uint32_t)j, nrow - 1);
        // global-space loads: a flat load would also count against the LDS wait
        // counter, and the tile's LDS reads would wait for the next rows' loads
        q[sl][j] = gld4(reinterpret_cast<const float4*>(colp + (size_t)(r0 + rr) * d.S_pad));
      }
    };
    using Slot0 = std::integral_constant<int, 0>;
    using Slot1 = std::integral_constant<int, 1>;
    load_rows(0u, Slot0{});    // in flight while the weights are formed
    load_rows((uint32_t)kRedRows, Slot1{});

    // costs and unit weights
    float jv[4] = {jc.x, jc.y, jc.z, jc.w};
    float m = INFINITY;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (!(s4 + k < S) || !(jv[k] < INFINITY)) jv[k] = INFINITY;  // past S (or S_pad) or NaN -> weight 0
      m = fminf(m, jv[k]);
    }
    m = fminf(m, __shfl_xor(m, 1, 64));
    m = fminf(m, __shfl_xor(m, 2, 64));
    m = fminf(m, __shfl_xor(m, 4, 64));
    s_gam4[t] = make_float4(unit_weight(jv[0], m, d.inv_lambda), unit_weight(jv[1], m, d.inv_lambda),
                            unit_weight(jv[2], m, d.inv_lambda), unit_weight(jv[3], m, d.inv_lambda));
    if ((t & 7) == 0) s_mu[t >> 3] = m;
    __syncthreads();
    // group minimum and unit scales
    if (wid == 0) {
      float mg = (lane < (int)nu_g) ? s_mu[lane] : INFINITY;
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) mg = fminf(mg, __shfl_xor(mg, o, 64));
      if (lane < (int)nu_g) {
        s_sig[lane] = merge_scale(s_mu[lane], mg, d.inv_lambda);
        if (rg == 0) {
          float z, z2;
          unit_sums(s_gam + kUnit * lane, z, z2);
          s_up[lane] = make_float4(s_mu[lane], z, z2, 0.0f);
        }
      }
      if (lane == 0) s_red[0] = mg;
    }
    // the weights of the unit this lane sums
    float gw[kUnit];
    {
      const float4* g4 = s_gam4 + (kUnit / 4) * (8 * (uint32_t)wid + lu);
#pragma unroll
      for (int k = 0; k < kUnit / 4; ++k) {
        const float4 w = g4[k];
        gw[4 * k + 0] = w.x;
        gw[4 * k + 1] = w.y;
        gw[4 * k + 2] = w.z;
        gw[4 * k + 3] = w.w;
      }
    }
    // unit row sums, in sample order, 8 rows per pass
    auto pass = [&](uint32_t p, auto SLOT) __attribute__((always_inline)) {
      constexpr int sl = decltype(SLOT)::value;
#pragma unroll
      for (int j = 0; j < kRedRows; ++j)
        *reinterpret_cast<float4*>(s_T + j * kRedRowStride + st_off) = q[sl][j];
      load_rows(p + 2 * kRedRows, SLOT);
      __builtin_amdgcn_wave_barrier();
      const float4* u4 = reinterpret_cast<const float4*>(s_T + lr * kRedRowStride + lu * kRedUnitStride);
      float acc = 0.0f;
#pragma unroll
      for (int k = 0; k < kUnit / 4; ++k) {
        const float4 u = u4[k];
        acc = unit_row_term(acc, gw[4 * k + 0], u.x);
        acc = unit_row_term(acc, gw[4 * k + 1], u.y);
        acc = unit_row_term(acc, gw[4 * k + 2], u.z);
        acc = unit_row_term(acc, gw[4 * k + 3], u.w);
      }
      if (p + lr < nrow) s_R[p + lr][8 * wid + lu] = acc;
      __builtin_amdgcn_wave_barrier();
    };
    for (uint32_t p = 0; p < nrow; p += 2 * kRedRows) {
      pass(p, Slot0{});
      pass(p + kRedRows, Slot1{});
    }
    __syncthreads();
    if (rg == 0 && t == kWThreads - 1) {   // a thread without a row: overlaps the row merges
      float z, z2;
      group_sums(s_up, s_sig, nu_g, z, z2);
      pub_st4(d.wpart + grp, make_float4(s_red[0], z, z2, 0.0f));
    }
    // group row sums, in unit order
    if (t < nrow) {
      float acc = 0.0f;
      for (uint32_t v = 0; v < nu_g; ++v) acc = unit_row_term(acc, s_sig[v], s_R[t][v]);
      pub_st(d.rpart + (size_t)grp * R + r0 + t, acc);
    }
    // publish: the barrier completes every wave's stores, one release by
    // thread 0 then makes them visible to the block that finishes the instance
    pub_complete();
    __syncthreads();
    if (t == 0) {
      const uint32_t k = atomicAdd(d.counter, 1u);
      s_last = (k == d.n_ritems - 1) ? 1u : 0u;
    }
    __syncthreads();
    if (s_last) {
      finalize_instance(d, s_scale, s_red, s_trig);
      if (t == 0) atomicExch(d.counter, 0u);
    }
    __syncthreads();
  }
  if (ctr) finish_persistent(&ctr->r_next, &ctr->r_done);
}

// ---------------------------------------------------------------------------
// Debug: raw Philox blocks and the normals a rollout draws
// ---------------------------------------------------------------------------
__global__ void k_philox_dump(const uint32_t* __restrict__ ctr, uint32_t k0, uint32_t k1, uint32_t n,
                              uint32_t* __restrict__ out) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint32_t r[4];
  philox4x32_10(ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3], k0, k1, r);
  for (int k = 0; k < 4; ++k) out[4 * i + k] = r[k];
}

__global__ void k_normals_dump(uint32_t seed_lo, uint32_t seed_hi, uint32_t instance,
                               const uint32_t* __restrict__ s_tau, uint32_t n, uint32_t K,
                               float* __restrict__ out) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t s = s_tau[2 * i], tau = s_tau[2 * i + 1];
  for (uint32_t b = 0; 4 * b < K; ++b) {
    uint32_t r[4];
    float e[4];
    philox4x32_10(s, tau, b, instance, seed_lo, seed_hi, r);
    box_muller4(r, e);
    for (uint32_t k = 0; k < 4 && 4 * b + k < K; ++k) out[(size_t)i * K + 4 * b + k] = e[k];
  }
}

// the radius and the two angle factors of box_muller4 for raw words r
__global__ void k_box_muller_dump(const uint32_t* __restrict__ r, uint32_t n, float* __restrict__ out) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float u = unif23(r[i]);
  out[3 * (size_t)i] = bm_radius(u);
  out[3 * (size_t)i + 1] = __builtin_amdgcn_cosf(u);
  out[3 * (size_t)i + 2] = __builtin_amdgcn_sinf(u);
}

__global__ void k_fill_u32(uint32_t* __restrict__ p, uint32_t value, size_t n) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = value;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <int NOB, bool GD, int G, bool PRE>
static hipError_t launch_rollout_t(const SolveDesc* desc, uint32_t grid, uint32_t block, size_t lds,
                                   hipStream_t stream) {
  hipLaunchKernelGGL((k_rollout<NOB, GD, G, PRE>), dim3(grid), dim3(block), lds, stream, desc);
  return hipGetLastError();
}

template <int NOB, bool GD>
static hipError_t launch_variant(int variant, const SolveDesc* desc, uint32_t grid, uint32_t block, size_t lds,
                                 hipStream_t stream) {
  switch (variant) {
    case 0: return launch_rollout_t<NOB, GD, 1, false>(desc, grid, block, lds, stream);
    case 1: return launch_rollout_t<NOB, GD, 1, true>(desc, grid, block, lds, stream);
    case 2: return launch_rollout_t<NOB, GD, 2, true>(desc, grid, block, lds, stream);
    case 3: return launch_rollout_t<NOB, GD, 4, true>(desc, grid, block, lds, stream);
    case 4: return launch_rollout_t<NOB, GD, 8, true>(desc, grid, block, lds, stream);
    case 5:
      if constexpr (NOB == 16) return launch_rollout_t<NOB, GD, 2, false>(desc, grid, block, lds, stream);
      return hipErrorInvalidValue;
    case 6:
      if constexpr (NOB == 32) return launch_rollout_t<NOB, GD, 4, false>(desc, grid, block, lds, stream);
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_rollout(int bucket, int variant, const SolveDesc* desc, uint32_t grid, uint32_t block, size_t lds,
                          hipStream_t stream) {
  if (block == 0 || block > (uint32_t)kMaxBlock || (block % 64) != 0) return hipErrorInvalidValue;
  switch (bucket) {
    case 0: return launch_variant<0, false>(variant, desc, grid, block, lds, stream);
    case 2: return launch_variant<2, true>(variant, desc, grid, block, lds, stream);
    case 8: return launch_variant<8, true>(variant, desc, grid, block, lds, stream);
    case 16: return launch_variant<16, true>(variant, desc, grid, block, lds, stream);
    case 32: return launch_variant<32, true>(variant, desc, grid, block, lds, stream);
    default: return hipErrorInvalidValue;
  }
}

template <int NOB, bool GD>
static hipError_t launch_drawn_t(const SolveArgs& args, uint32_t grid, size_t lds, hipStream_t stream) {
  hipLaunchKernelGGL((k_rollout_drawn<NOB, GD>), dim3(grid), dim3(2 * kMaxBlock), lds, stream, args);
  return hipGetLastError();
}

hipError_t launch_rollout_drawn(int bucket, SolveArgs& args, uint32_t grid, size_t lds, hipStream_t stream) {
  if (args.d.T > kInlineSteps || args.d.S > grid * kDrawnTile || lds > kFusedLdsMax || !args.d.fused)
    return hipErrorInvalidValue;
  const DrawnLds l = drawn_lds(bucket, args.d.T, lds);
  args.run = l.run;
  lds = l.bytes;
  switch (bucket) {
    case 0: return launch_drawn_t<0, false>(args, grid, lds, stream);
    case 2: return launch_drawn_t<2, true>(args, grid, lds, stream);
    case 8: return launch_drawn_t<8, true>(args, grid, lds, stream);
    case 16: return launch_drawn_t<16, true>(args, grid, lds, stream);
    case 32: return launch_drawn_t<32, true>(args, grid, lds, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_rollout_batch(const SolveDesc* descs, const Tile* tiles, uint32_t n_tiles, BatchCounters* ctr,
                                uint32_t grid, uint32_t block, bool guided, hipStream_t stream) {
  if (block == 0 || block > (uint32_t)kMaxBlock || (block % 64) != 0) return hipErrorInvalidValue;
  if (guided) hipLaunchKernelGGL(k_rollout_batch<true>, dim3(grid), dim3(block), 0, stream, descs, tiles, n_tiles, ctr);
  else hipLaunchKernelGGL(k_rollout_batch<false>, dim3(grid), dim3(block), 0, stream, descs, tiles, n_tiles, ctr);
  return hipGetLastError();
}

int rollout_batch_blocks_per_cu(uint32_t block, bool guided) {
  int nb = 0;
  const hipError_t e = guided ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_rollout_batch<true>, (int)block, 0)
                              : hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_rollout_batch<false>, (int)block, 0);
  return e == hipSuccess && nb > 0 ? nb : 1;
}

hipError_t launch_noise(const NoiseArgs& a, uint32_t count, uint32_t T, const Upload& up, hipStream_t stream) {
  const uint32_t nb = (a.n_normals + 3) / 4;
  if (count == 0 || nb == 0 || nb > (uint32_t)kMaxPhiloxBlocks) return hipErrorInvalidValue;
  const dim3 grid((a.S_pad + 1023) / 1024, T, count);
  hipLaunchKernelGGL(k_noise, grid, dim3(256), 0, stream, a, nb, up);
  return hipGetLastError();
}

hipError_t launch_upload(const Upload& up, hipStream_t stream) {
  const uint32_t grid = (uint32_t)std::min<size_t>((up.n + 255) / 256, 1024);
  hipLaunchKernelGGL(k_upload, dim3(grid), dim3(256), 0, stream, up);
  return hipGetLastError();
}

hipError_t launch_reduce(const SolveDesc* descs, const Item* items, uint32_t n_items, BatchCounters* ctr,
                         uint32_t grid, hipStream_t stream) {
  hipLaunchKernelGGL(k_reduce, dim3(grid), dim3(kWThreads), 0, stream, descs, items, n_items, ctr);
  return hipGetLastError();
}



hipError_t launch_philox_dump(const uint32_t* ctr, uint32_t k0, uint32_t k1, uint32_t n, uint32_t* out,
                              hipStream_t stream) {
  const uint32_t b = 256, g = (n + b - 1) / b;
  if (g == 0) return hipSuccess;
  hipLaunchKernelGGL(k_philox_dump, dim3(g), dim3(b), 0, stream, ctr, k0, k1, n, out);
  return hipGetLastError();
}

hipError_t launch_normals_dump(uint32_t seed_lo, uint32_t seed_hi, uint32_t instance, const uint32_t* s_tau,
                               uint32_t n, uint32_t K, float* out, hipStream_t stream) {
  const uint32_t b = 256, g = (n + b - 1) / b;
  if (g == 0) return hipSuccess;
  hipLaunchKernelGGL(k_normals_dump, dim3(g), dim3(b), 0, stream, seed_lo, seed_hi, instance, s_tau, n, K, out);
  return hipGetLastError();
}

hipError_t launch_box_muller_dump(const uint32_t* r, uint32_t n, float* out, hipStream_t stream) {
  const uint32_t b = 256, g = (n + b - 1) / b;
  if (g == 0) return hipSuccess;
  hipLaunchKernelGGL(k_box_muller_dump, dim3(g), dim3(b), 0, stream, r, n, out);
  return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t value, size_t n, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  const uint32_t b = 256;
  const size_t g = (n + b - 1) / b;
  hipLaunchKernelGGL(k_fill_u32, dim3((uint32_t)g), dim3(b), 0, stream, p, value, n);
  return hipGetLastError();
}

}  // namespace brm
