// Device-side ideal GLM-MHD arithmetic for gfx950 (register-resident, fully
// unrolled; the face direction is a template parameter so component
// selection costs nothing).  Face arithmetic is templated on the real type:
// double on the FP64 path, float on the FP32-mixed path (where the
// conserved-to-primitive step and the pressure recovery stay in double).
//
// Scheme (MPI-AMRVAC 3.0, arXiv 2303.03026): conservative finite volumes
// ("Schemes and limiters for HD and MHD"), 'vanleer' slopes on primitive
// variables (Table t:limiters), HLL fluxes (Table tab:schemes_space), 'glm'
// divergence control after Dedner et al. 2002 (Table t:divb), small-value
// checks on entry to conserved->primitive ("Bootstrapping" section).
#pragma once

#include <hip/hip_runtime.h>

namespace amrvac {

constexpr int NV = 9;
// conserved slots; primitives reuse them with v in 1..3 and p in 4
enum { I_RHO = 0, I_MX = 1, I_MY = 2, I_MZ = 3, I_EN = 4, I_BX = 5, I_BY = 6, I_BZ = 7, I_PSI = 8 };
enum { F_SMALL_RHO = 1, F_SMALL_P = 2, F_BAD_DT = 4 };

// Per-launch physical constants (by value in kernel arguments).
struct PhysConst {
  double gamma;
  double gm1;      // gamma - 1
  double inv_gm1;  // 1 / (gamma - 1)
  double small_rho;
  double small_p;
  int fix;
  int limiter;  // LIM_* (the fused stage takes it as a template argument)
  int flux;     // FLUX_HLL, FLUX_HLLD or FLUX_HLLC (likewise)
};

// Library-owned device status record.
struct DevStatus {
  unsigned int flags;
  unsigned int cfl_nan;  // a NaN rate was met by the running CFL reduction
  unsigned long long nfix;
  unsigned long long rate_bits;  // max CFL rate (non-negative double bits)
  double last_dt;
};

// ---------------------------------------------------------------------------
// Lean reciprocal, quotient and square root for the normal-range operands of
// this scheme (no denormal or overflow scaling).  FP64: a hardware seed
// (v_rcp_f64 / v_rsq_f64, measured on gfx950 to about 2^-24 relative) refined
// by Newton steps; the reciprocal takes two (about one ulp), the quotient one
// step plus a residual correction of the product (about one ulp).  FP32: the
// single-instruction v_rcp_f32 / v_sqrt_f32 (about one ulp).

__device__ __forceinline__ double rcp_(double x) {
  double r = __builtin_amdgcn_rcp(x);
  double e = fma(-x, r, 1.0);
  r = fma(e, r, r);
  e = fma(-x, r, 1.0);
  return fma(e, r, r);
}
__device__ __forceinline__ float rcp_(float x) { return __builtin_amdgcn_rcpf(x); }

__device__ __forceinline__ double div_(double a, double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = fma(fma(-b, r, 1.0), r, r);  // ~2^-48 relative
  const double q = a * r;
  return fma(fma(-b, q, a), r, q);
}
__device__ __forceinline__ float div_(float a, float b) { return a * __builtin_amdgcn_rcpf(b); }

// Third-order refinement of the seed: with e = 1 - x r, 1/x = r (1 + e + e^2
// + ...), so two multiply-adds give r (1 + e + e^2), e^3 ~ 2^-73 off: one
// operation less than two Newton steps and a shorter chain.
__device__ __forceinline__ double rcp3_(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
__device__ __forceinline__ float rcp3_(float x) { return __builtin_amdgcn_rcpf(x); }

// 1/x and 1/y.  FP64: from one reciprocal of the product (the seed and its
// refinement are the costly part: 4 of the 12 issue slots of a quotient are
// the quarter-rate v_rcp_f64 alone), for operands whose product neither
// overflows nor underflows.  Half an ulp worse than two reciprocals, and an
// infinity on one side is one on both: for the sound speeds and the slopes,
// where it does not show, not for the star states (HLLC at Mach numbers of
// 0.01 lost a quarter, 4.8 to 5.7 roundings, and ran no faster).
__device__ __forceinline__ void rcp_pair(double x, double y, double& ix, double& iy) {
  const double r = rcp3_(x * y);
  ix = r * y;
  iy = r * x;
}
__device__ __forceinline__ void rcp_pair(float x, float y, float& ix, float& iy) {
  ix = __builtin_amdgcn_rcpf(x);
  iy = __builtin_amdgcn_rcpf(y);
}

// Square root of max(x, 0) (of 1e-300 in FP64, where the seed needs a
// positive operand: no square root is below 1e-150); a NaN gives 0 as well.  FP64: with y the seed, g = x y
// and e = 1 - g y, sqrt(x) = g (1 - e)^(-1/2) = g (1 + e/2 + 3/8 e^2), e^3
// ~ 2^-72 off.
__device__ __forceinline__ double sqrt_pos(double x) {
  x = fmax(x, 1e-300);
  const double y = __builtin_amdgcn_rsq(x);
  const double g = x * y;
  const double e = fma(-g, y, 1.0);
  return fma(g, e * fma(e, 0.375, 0.5), g);
}
__device__ __forceinline__ float sqrt_pos(float x) { return __builtin_amdgcn_sqrtf(fmaxf(x, 0.0f)); }

// The same and its reciprocal (two operations more).
__device__ __forceinline__ double sqrt_rsqrt_pos(double x, double& inv) {
  x = fmax(x, 1e-300);
  const double y = __builtin_amdgcn_rsq(x);
  const double g = x * y;
  const double e = fma(-g, y, 1.0);
  const double t = e * fma(e, 0.375, 0.5);
  inv = fma(y, t, y);
  return fma(g, t, g);
}
__device__ __forceinline__ float sqrt_rsqrt_pos(float x, float& inv) {
  const float r = __builtin_amdgcn_sqrtf(fmaxf(x, 0.0f));
  inv = __builtin_amdgcn_rcpf(r);
  return r;
}

// A square root up to this size stands for 0.
template <class R>
constexpr R kZeroSpeed = sizeof(R) == sizeof(double) ? R(1e-140) : R(0);

__device__ __forceinline__ double sqrt_(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  const double r = fma(-g, h, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  g = fma(fma(-g, g, x), h, g);
  return x > 0.0 ? g : 0.0;
}
__device__ __forceinline__ float sqrt_(float x) { return x > 0.0f ? __builtin_amdgcn_sqrtf(x) : 0.0f; }

// ---------------------------------------------------------------------------
// conserved -> primitive; returns the small-value bits of this cell.  The
// conserved input is double (the FP64 energy and the promoted FP32 rest on
// the mixed path) and the pressure recovery e - m^2/2rho - B^2/2 is done in
// double; the primitive is then rounded to R.  With the fix on, density is
// floored first (velocity uses the floored value), then pressure; conserved
// values and B are never changed.
template <class R>
__device__ __forceinline__ int cons_to_prim(const double u[NV], R w[NV], const PhysConst& P) {
  int bad = 0;
  double rho = u[I_RHO];
  if (!(rho > P.small_rho)) {
    bad |= F_SMALL_RHO;
    if (P.fix) rho = P.small_rho;
  }
  const double ri = rcp_(rho);
  w[I_RHO] = (R)rho;
  w[1] = (R)(u[I_MX] * ri);
  w[2] = (R)(u[I_MY] * ri);
  w[3] = (R)(u[I_MZ] * ri);
  const double m2 = u[I_MX] * u[I_MX] + u[I_MY] * u[I_MY] + u[I_MZ] * u[I_MZ];
  const double b2 = u[I_BX] * u[I_BX] + u[I_BY] * u[I_BY] + u[I_BZ] * u[I_BZ];
  double p = P.gm1 * (u[I_EN] - 0.5 * m2 * ri - 0.5 * b2);
  if (!(p > P.small_p)) {
    bad |= F_SMALL_P;
    if (P.fix) p = P.small_p;
  }
  w[4] = (R)p;
  w[I_BX] = (R)u[I_BX];
  w[I_BY] = (R)u[I_BY];
  w[I_BZ] = (R)u[I_BZ];
  w[I_PSI] = (R)u[I_PSI];
  return bad;
}

__device__ __forceinline__ void prim_to_cons(const double w[NV], double u[NV], const PhysConst& P) {
  const double rho = w[I_RHO];
  u[I_RHO] = rho;
  u[I_MX] = rho * w[1];
  u[I_MY] = rho * w[2];
  u[I_MZ] = rho * w[3];
  const double v2 = w[1] * w[1] + w[2] * w[2] + w[3] * w[3];
  const double b2 = w[I_BX] * w[I_BX] + w[I_BY] * w[I_BY] + w[I_BZ] * w[I_BZ];
  u[I_EN] = w[4] * P.inv_gm1 + 0.5 * rho * v2 + 0.5 * b2;
  u[I_BX] = w[I_BX];
  u[I_BY] = w[I_BY];
  u[I_BZ] = w[I_BZ];
  u[I_PSI] = w[I_PSI];
}

// Limiters of Table t:limiters that work on the 2-ghost-cell stencil.  With
// d- = w_i - w_(i-1) and d+ = w_(i+1) - w_i, cell i's face values are
//   right face:  w_i + lim(d+, d-) / 2,    left face:  w_i - lim(d-, d+) / 2,
// lim(near, far) being the limited difference across the face (odd in its
// arguments).  van Leer's is symmetric: lim(d+, d-) = lim(d-, d+) = the
// harmonic slope 2 d- d+ / (d- + d+), zero where d- d+ <= 0.  Koren's and
// Cada-Torrilhon's third-order ones are not; written division-free with
// s = sign(near), b = |near|, a = s far, they are
//   koren:  s max(0, min(2a, (2b + a)/3, 2b))
//   cada3:  s max(0, min((2b + a)/3, max(-a/2, min(2a, (2b + a)/3, 1.6 b))))
// (the unlimited third-order value (2b + a)/3 in smooth monotone regions).
// The functions below give half of them, the quantity a face value takes.
enum { LIM_VANLEER = 0, LIM_KOREN = 1, LIM_CADA3 = 2, LIM_WENO5 = 3, LIM_WENOZ5 = 4, LIM_MP5 = 5, LIM_WENOZP5 = 6 };

// v with its sign flipped where that of s is set, without a multiplication
__device__ __forceinline__ double flip_sign(double v, double s) {
  const long long m = __double_as_longlong(s) & (long long)0x8000000000000000ull;
  return __longlong_as_double(__double_as_longlong(v) ^ m);
}
__device__ __forceinline__ float flip_sign(float v, float s) {
  return __int_as_float(__float_as_int(v) ^ (__float_as_int(s) & (int)0x80000000));
}

// Koren's and Cada and Torrilhon's, one side.  (Koren's two sides share the
// smaller of |d-| and |d+|, but an evaluation of both at once holds more
// values: in FP64 with HLLD it spilled 55 against 19 registers and a 96^3
// step took 0.41 against 0.28 ms.)
template <class R>
__device__ __forceinline__ R koren_half(R near, R far) {
  const R b = fabs(near), a = flip_sign(far, near);
  const R p3 = (R(2) * b + a) * R(1.0 / 6.0);
  return flip_sign(fmax(R(0), fmin(fmin(a, p3), b)), near);
}
template <class R>
__device__ __forceinline__ R cada3_half(R near, R far) {
  const R b = fabs(near), a = flip_sign(far, near);
  const R p3 = (R(2) * b + a) * R(1.0 / 6.0);
  return flip_sign(fmax(R(0), fmin(p3, fmax(R(-0.25) * a, fmin(fmin(a, p3), R(0.8) * b)))), near);
}

// van Leer's half slope d- d+ / (d- + d+) of two variables of a cell.
// FP64: one reciprocal serves both quotients (9 against 15 issue slots per
// slope with a quotient and a select each); the product is clamped at zero
// instead of selecting, and the sums are kept off zero by 1e-150 (the range
// of the products is that of d- d+ itself, about 1e-150 to 1e150).  FP32:
// the reciprocal is one instruction and the range too short for products.
constexpr double kSlopeTiny = 1e-150;
__device__ __forceinline__ void vl_half2(double dm1, double dp1, double dm2, double dp2, double& h1, double& h2) {
  const double s1 = (dm1 + dp1) + kSlopeTiny, s2 = (dm2 + dp2) + kSlopeTiny;
  const double q1 = fmax(dm1 * dp1, 0.0), q2 = fmax(dm2 * dp2, 0.0);
  double i1, i2;
  rcp_pair(s1, s2, i1, i2);
  h1 = q1 * i1;
  h2 = q2 * i2;
}
__device__ __forceinline__ double vl_half(double dm, double dp) {
  return fmax(dm * dp, 0.0) * rcp3_((dm + dp) + kSlopeTiny);
}
__device__ __forceinline__ float vl_half(float dm, float dp) {
  const float q = dm * dp;
  const float v = div_(q, dm + dp);
  return q > 0.0f ? v : 0.0f;
}
__device__ __forceinline__ void vl_half2(float dm1, float dp1, float dm2, float dp2, float& h1, float& h2) {
  h1 = vl_half(dm1, dp1);
  h2 = vl_half(dm2, dp2);
}

// Half the limited differences of a variable (a pair of variables) of a
// cell, for its right (r) and left (l) face values w + r and w - l.
template <int LIM, class R>
__device__ __forceinline__ void half_increments1(R dm, R dp, R& r, R& l) {
  if (LIM == LIM_VANLEER) {
    r = vl_half(dm, dp);
    l = r;
  } else if (LIM == LIM_KOREN) {
    r = koren_half(dp, dm);
    l = koren_half(dm, dp);
  } else {
    r = cada3_half(dp, dm);
    l = cada3_half(dm, dp);
  }
}
template <int LIM, class R>
__device__ __forceinline__ void half_increments2(R dm1, R dp1, R dm2, R dp2, R& r1, R& l1, R& r2, R& l2) {
  if (LIM == LIM_VANLEER) {
    vl_half2(dm1, dp1, dm2, dp2, r1, r2);
    l1 = r1;
    l2 = r2;
  } else {
    half_increments1<LIM>(dm1, dp1, r1, l1);
    half_increments1<LIM>(dm2, dp2, r2, l2);
  }
}

// The pairs of variables that share a reciprocal: (rho, p), (v_x, v_y),
// (v_z, psi), (B_x, B_y); B_z is on its own.  They are the same in every
// direction and map onto themselves when x and y are exchanged, so that a
// cell's face values do not depend on where they are evaluated.
constexpr int kPairs = 5;
__host__ __device__ constexpr int pair_a(int u) { return (0x75310 >> (4 * u)) & 15; }
__host__ __device__ constexpr int pair_b(int u) { return (0x76824 >> (4 * u)) & 15; }

// For every variable q of a cell: f(q, w, r, l) with the cell's value w and
// its half increments; get(q, m, w, p) gives the cell and its neighbours.
// (pair by pair, so that few of the operands are live at a time)
template <int LIM, class R, class Get, class F>
__device__ __forceinline__ void for_increments(Get get, F f) {
#pragma unroll
  for (int u = 0; u < kPairs; ++u) {
    const int a = pair_a(u), b = pair_b(u);
    R m1, w1, p1, r1, l1;
    get(a, m1, w1, p1);
    if (u < kPairs - 1) {
      R m2, w2, p2, r2, l2;
      get(b, m2, w2, p2);
      half_increments2<LIM>(w1 - m1, p1 - w1, w2 - m2, p2 - w2, r1, l1, r2, l2);
      f(b, w2, r2, l2);
    } else {
      half_increments1<LIM>(w1 - m1, p1 - w1, r1, l1);
    }
    f(a, w1, r1, l1);
  }
}

__device__ __forceinline__ double minmod2(double a, double b) {
  return a * b > 0.0 ? (fabs(a) < fabs(b) ? a : b) : 0.0;
}

// Fast magnetosonic speed along D from a primitive state (1/rho given).
template <int D, class R>
__device__ __forceinline__ R cfast(const R w[NV], R ri, R b2, R gamma) {
  const R a2 = gamma * w[4] * ri;
  const R bb = b2 * ri;
  const R bn2 = w[I_BX + D] * w[I_BX + D] * ri;
  const R s = a2 + bb;
  R disc = s * s - R(4) * a2 * bn2;
  disc = disc < R(0) ? R(0) : disc;
  return sqrt_(R(0.5) * (s + sqrt_(disc)));
}

// CFL rate of one cell from its conserved state (always FP64): the sum over
// directions of (|v_d| + c_fast,d) / dx_d, after the small-value check of the
// conserved-to-primitive step (its bits are or-ed into bad).  The time-step
// pass and the fused last stage both use this, so they agree bit for bit.
template <int NDIM>
__device__ __forceinline__ double cell_rate(const double u[NV], const PhysConst& P, double ix, double iy, double iz,
                                            int& bad) {
  double w[NV];
  bad |= cons_to_prim(u, w, P);
  const double ri = rcp_(w[I_RHO]);
  const double b2 = w[I_BX] * w[I_BX] + w[I_BY] * w[I_BY] + w[I_BZ] * w[I_BZ];
  double rate = (fabs(w[1]) + cfast<0>(w, ri, b2, P.gamma)) * ix;
  rate = rate + (fabs(w[2]) + cfast<1>(w, ri, b2, P.gamma)) * iy;
  if (NDIM == 3) rate = rate + (fabs(w[3]) + cfast<2>(w, ri, b2, P.gamma)) * iz;
  return rate;
}

// Axes transverse to D.  The fluxes below write every sum over components in
// the order normal, first, second transverse axis, so that a y face
// evaluated as an x face with x and y exchanged gives the same bits.
template <int D>
struct Transverse {
  static constexpr int T1 = D == 0 ? 1 : 0, T2 = D == 2 ? 1 : 2;
};

// Fast speeds along the normal on both sides of a face with the common
// normal field (bn2 = B_n^2, t2 = |B_t|^2): c_f^2 = (S + sqrt(S^2 - 4 gamma p
// B_n^2)) / (2 rho), S = gamma p + B^2, with the radicand written as the sum
// of squares (gamma p - B^2)^2 + 4 gamma p B_t^2, which does not cancel.
// FP64: the two 1/rho come from one reciprocal.  FP32 divides by rho first:
// the square of a pressure leaves its range from 1e19 up and from 1e-19 down,
// whatever the speeds are.
template <class R>
__device__ __forceinline__ void cfast_faces(R rl, R rr, R pl, R pr, R t2l, R t2r, R bn2, R gamma, R& cl, R& cr) {
  R il, ir;
  rcp_pair(rl, rr, il, ir);
  constexpr bool kScale = sizeof(R) < sizeof(double);
  const R gl = kScale ? gamma * pl * il : gamma * pl, gr = kScale ? gamma * pr * ir : gamma * pr;
  const R tl = kScale ? t2l * il : t2l, tr = kScale ? t2r * ir : t2r;
  const R b2l = (kScale ? bn2 * il : bn2) + tl, b2r = (kScale ? bn2 * ir : bn2) + tr;
  const R ml = gl - b2l, mr = gr - b2r;
  const R dl = ml * ml + (R(4) * gl) * tl, dr = mr * mr + (R(4) * gr) * tr;
  cl = sqrt_pos(((gl + b2l) + sqrt_pos(dl)) * (kScale ? R(0.5) : R(0.5) * il));
  cr = sqrt_pos(((gr + b2r) + sqrt_pos(dr)) * (kScale ? R(0.5) : R(0.5) * ir));
}

// Interface flux along D from reconstructed left/right primitive states:
// GLM interface values of (B_n, psi) from the exact solution of the linear
// subsystem, then HLL (Davis bounds) on rho, m, e and the tangential B,
// with B_n replaced on both sides.  half_inv_ch = 0.5 / c_h.
// With a = min(S_L, 0), b = max(S_R, 0) and the weights k_l = b / (b - a) and
// k_r = -a / (b - a) of the two sides, HLL's (b F_l - a F_r + a b (U_r -
// U_l)) / (b - a) is, for the advected part F = U v_n, k_l (v_n,l - a) U_l +
// k_r (v_n,r - b) U_r, and for the rest its weighted mean.  It is written from
// one side o, with the differences to the other side, q, taken first: U_o v^ +
// k_q (v_n,q - s) (U_q - U_o), where x^ = x_o + k_q (x_q - x_o) and s is q's
// bound of a and b.  That is half the operations of forming both sides'
// fluxes and U_r - U_l per component.  (The pressure term keeps the two
// products: where nothing but the density varies it then rounds as the
// quotient does.)  Side o is the left one, and the right one where its weight
// is above 3/5: written from the other side, if that is the heavier state, the
// flux would be what is left over of products that cancel (with density ratios
// of 1000, some 1000 roundings).  From 1/2 on, symmetrically, errors are the
// same and the exchange costs a 32^3 step 3% more, its waves then all having
// such faces.  Where every wave moves one way k_q = 0 and F = F_o.
template <int D, class R>
__device__ __forceinline__ void hll_glm_flux(R wl[NV], R wr[NV], R ch, R half_inv_ch, R gamma, R inv_gm1,
                                             R F[NV]) {
  constexpr int N = I_BX + D, VN = 1 + D;
  constexpr int T1 = Transverse<D>::T1, T2 = Transverse<D>::T2;
  const R bn = R(0.5) * (wl[N] + wr[N]) - (wr[I_PSI] - wl[I_PSI]) * half_inv_ch;
  const R ps = R(0.5) * (wl[I_PSI] + wr[I_PSI]) - R(0.5) * ch * (wr[N] - wl[N]);
  const R bn2 = bn * bn;
  // sides o and q
  R ro = wl[I_RHO], rq = wr[I_RHO], po = wl[4], pq = wr[4], vno = wl[VN], vnq = wr[VN];
  R u1o = wl[1 + T1], u1q = wr[1 + T1], u2o = wl[1 + T2], u2q = wr[1 + T2];
  R b1o = wl[I_BX + T1], b1q = wr[I_BX + T1], c1o = wl[I_BX + T2], c1q = wr[I_BX + T2];
  const R t2l = b1o * b1o + c1o * c1o, t2r = b1q * b1q + c1q * c1q;
  R b2o = bn2 + t2l, b2q = bn2 + t2r;
  R cl, cr;
  cfast_faces(ro, rq, po, pq, t2l, t2r, bn2, gamma, cl, cr);
  const R a = fmin(fmin(vno - cl, vnq - cr), R(0));
  const R b = fmax(fmax(vno + cl, vnq + cr), R(0));
  const R inv = rcp3_(b - a);
  R ko = b * inv, kq = -a * inv, s = b;
  const bool turn = R(2) * a + R(3) * b < R(0);
  const bool one_way = a >= -kZeroSpeed<R> || b <= kZeroSpeed<R>;
  if (__any(turn || one_way)) {
    asm volatile("");  // keeps the branch wave-uniform
    if (turn) {
      auto swap = [](R& x, R& y) {
        const R z = x;
        x = y;
        y = z;
      };
      swap(ro, rq), swap(po, pq), swap(vno, vnq), swap(u1o, u1q), swap(u2o, u2q);
      swap(b1o, b1q), swap(c1o, c1q), swap(b2o, b2q), swap(ko, kq);
      s = a;
    }
    if (one_way) {  // (b - a may be zero)
      ko = R(1);
      kq = R(0);
    }
  }
  const R dvn = vnq - vno;
  const R vh = vno + kq * dvn;  // v_n^
  const R g = kq * (vnq - s);   // weight of U_q - U_o
  // mass
  const R fm = ro * vh + g * (rq - ro);
  F[I_RHO] = fm;
  const R rg = rq * g;  // rho_o (v_n^ - g) v_o + rho_q g v_q = fm v_o + rg (v_q - v_o)
  // normal momentum and energy
  const R pto = po + R(0.5) * b2o, ptq = pq + R(0.5) * b2q;
  F[VN] = ko * (pto - bn2) + kq * (ptq - bn2) + (fm * vno + rg * dvn);
  {
    const R v2o = vno * vno + u1o * u1o + u2o * u2o;
    const R v2q = vnq * vnq + u1q * u1q + u2q * u2q;
    const R eo = po * inv_gm1 + R(0.5) * (ro * v2o + b2o);
    const R eq = pq * inv_gm1 + R(0.5) * (rq * v2q + b2q);
    const R vbo = vno * bn + u1o * b1o + u2o * c1o;
    const R vbq = vnq * bn + u1q * b1q + u2q * c1q;
    const R ho = pto * vno - bn * vbo, hq = ptq * vnq - bn * vbq;
    F[I_EN] = eo * vh + g * (eq - eo) + (ho + kq * (hq - ho));
    // tangential momentum and field
    const R dv1 = u1q - u1o, dv2 = u2q - u2o, db1 = b1q - b1o, db2 = c1q - c1o;
    F[1 + T1] = fm * u1o + rg * dv1 - bn * (b1o + kq * db1);
    F[1 + T2] = fm * u2o + rg * dv2 - bn * (c1o + kq * db2);
    F[I_BX + T1] = b1o * vh + g * db1 - bn * (u1o + kq * dv1);
    F[I_BX + T2] = c1o * vh + g * db2 - bn * (u2o + kq * dv2);
  }
  F[N] = ps;
  F[I_PSI] = ch * ch * bn;
}

// HLLD (Miyoshi and Kusano 2005) with the same GLM interface values as
// hll_glm_flux: B_n := B_n* on both sides, F(B_n) = psi*, F(psi) = c_h^2 B_n*,
// and HLLD on the other seven components.  S_L, S_R bracket both fast speeds
// around both normal velocities; S_M is the contact speed and p_T* the total
// pressure of the star region; the single-star states follow from the jump
// conditions across S_L / S_R (their tangential parts unchanged where
// rho (S - u)(S - S_M) - B_n^2 vanishes), the Alfven waves sit at
// S_M -/+ |B_n| / sqrt(rho*), and the double-star states between them and the
// contact.  Only the side of the contact that the interface lies on is
// assembled: F = F_a + S_a (U*_a - U_a) [+ S*_a (U**_a - U*_a) between the
// Alfven wave and the contact].
template <int D, class R>
__device__ __forceinline__ void hlld_glm_flux(R wl[NV], R wr[NV], R ch, R half_inv_ch, R gamma, R inv_gm1,
                                              R F[NV]) {
  constexpr int N = I_BX + D;
  constexpr int T1 = Transverse<D>::T1, T2 = Transverse<D>::T2;
  const R bn = R(0.5) * (wl[N] + wr[N]) - (wr[I_PSI] - wl[I_PSI]) * half_inv_ch;
  const R ps = R(0.5) * (wl[I_PSI] + wr[I_PSI]) - R(0.5) * ch * (wr[N] - wl[N]);
  wl[N] = bn;
  wr[N] = bn;
  const R rl = wl[I_RHO], rr = wr[I_RHO];
  const R ul = wl[1 + D], ur = wr[1 + D];
  const R bn2 = bn * bn;
  const R t2l = wl[I_BX + T1] * wl[I_BX + T1] + wl[I_BX + T2] * wl[I_BX + T2];
  const R t2r = wr[I_BX + T1] * wr[I_BX + T1] + wr[I_BX + T2] * wr[I_BX + T2];
  const R b2l = bn2 + t2l, b2r = bn2 + t2r;
  const R ptl = wl[4] + R(0.5) * b2l, ptr = wr[4] + R(0.5) * b2r;
  R cl, cr;
  cfast_faces(rl, rr, wl[4], wr[4], t2l, t2r, bn2, gamma, cl, cr);
  const R cfm = fmax(cl, cr);
  const R sl = fmin(ul, ur) - cfm, sr = fmax(ul, ur) + cfm;
  const R dl = (sl - ul) * rl, dr = (sr - ur) * rr;
  const R idd = rcp3_(dr - dl);
  R sm = (dr * ur - dl * ul - ptr + ptl) * idd;
  const R pts = (dr * ptl - dl * ptr + dl * dr * (ur - ul)) * idd;
  // single-star density and tangential parts, both sides.  With n = rho
  // (S - u)^2 - B_n^2 the denominator of the jump conditions is n - rho
  // (S - u)(S_M - u), so that the cancellation in n enters both terms of
  // their quotient alike.
  R isb[2] = {rcp3_(sl - sm), rcp3_(sr - sm)}, iden[2], num[2], den[2];
  num[0] = dl * (sl - ul) - bn2;
  num[1] = dr * (sr - ur) - bn2;
  den[0] = num[0] - dl * (sm - ul);
  den[1] = num[1] - dr * (sm - ur);
  iden[0] = rcp3_(den[0]);
  iden[1] = rcp3_(den[1]);
  const R rs0 = dl * isb[0], rs1 = dr * isb[1];
  R f1[2], f2[2];
  f1[0] = bn * (sm - ul) * iden[0];
  f1[1] = bn * (sm - ur) * iden[1];
  f2[0] = num[0] * iden[0];
  f2[1] = num[1] * iden[1];
  // the degenerate case is rare: its selects run only in waves that have it
  const bool deg0 = !(fabs(den[0]) > R(1e-12) * (dl * (sl - ul))), deg1 = !(fabs(den[1]) > R(1e-12) * (dr * (sr - ur)));
  if (__any(deg0 || deg1)) {
    asm volatile("");  // keeps the branch wave-uniform
    f1[0] = deg0 ? R(0) : f1[0];
    f1[1] = deg1 ? R(0) : f1[1];
    f2[0] = deg0 ? R(1) : f2[0];
    f2[1] = deg1 ? R(1) : f2[1];
  }
  const R v10 = wl[1 + T1] - f1[0] * wl[I_BX + T1], v11 = wr[1 + T1] - f1[1] * wr[I_BX + T1];
  const R v20 = wl[1 + T2] - f1[0] * wl[I_BX + T2], v21 = wr[1 + T2] - f1[1] * wr[I_BX + T2];
  const R b10 = f2[0] * wl[I_BX + T1], b11 = f2[1] * wr[I_BX + T1];
  const R b20 = f2[0] * wl[I_BX + T2], b21 = f2[1] * wr[I_BX + T2];
  // double-star tangential parts
  R isql, isqr;
  const R sql = sqrt_rsqrt_pos(rs0, isql), sqr = sqrt_rsqrt_pos(rs1, isqr);
  const R isum = rcp3_(sql + sqr);
  const R sg = bn > R(0) ? R(1) : (bn < R(0) ? R(-1) : R(0));
  const R sgq = sql * sqr * sg;
  R vss1 = (sql * v10 + sqr * v11 + (b11 - b10) * sg) * isum;
  R vss2 = (sql * v20 + sqr * v21 + (b21 - b20) * sg) * isum;
  R bss1 = (sql * b11 + sqr * b10 + sgq * (v11 - v10)) * isum;
  R bss2 = (sql * b21 + sqr * b20 + sgq * (v21 - v20)) * isum;
  // the side a of the contact the interface lies on, and its states
  const bool right = sr < R(0) || (!(sl > R(0)) && sm < R(0));
  const R rho = right ? rr : rl, u = right ? ur : ul, pt = right ? ptr : ptl, p = right ? wr[4] : wl[4];
  const R u1 = right ? wr[1 + T1] : wl[1 + T1], u2 = right ? wr[1 + T2] : wl[1 + T2];
  const R c1 = right ? wr[I_BX + T1] : wl[I_BX + T1], c2 = right ? wr[I_BX + T2] : wl[I_BX + T2];
  const R S = right ? sr : sl, sa = S - u;
  const R isba = right ? isb[1] : isb[0];
  R rsa = right ? rs1 : rs0;
  R vs1a = right ? v11 : v10, vs2a = right ? v21 : v20;
  R bs1a = right ? b11 : b10, bs2a = right ? b21 : b20;
  const R b2 = bn2 + (c1 * c1 + c2 * c2);
  const R v2 = u * u + u1 * u1 + u2 * u2;
  const R e = p * inv_gm1 + R(0.5) * rho * v2 + R(0.5) * b2;
  const R vb = u * bn + u1 * c1 + u2 * c2;
  const R vbs = sm * bn + vs1a * bs1a + vs2a * bs2a;
  R es = (sa * e - pt * u + pts * sm + bn * (vb - vbs)) * isba;
  const R vbss = sm * bn + vss1 * bss1 + vss2 * bss2;
  const R sqa = right ? sqr : -sql;  // with the sign of the side
  R des = sqa * (vbs - vbss) * sg;  // e** - e*
  const R sas = sm + fabs(bn) * (right ? isqr : -isql);  // S*_a
  const bool super = sl > R(0) || sr < R(0);                        // every wave moves one way: F = F_a
  const bool inner = !super && (right ? sas : -sas) > R(0);          // between the Alfven wave and the contact
  // F = F_a + S (U* - U_a) + S* (U** - U*): the terms of waves that do not
  // reach the interface drop by their factor, once their states are finite.
  // They are not where the fast speed is lost in rounding beside u (S = u on
  // both sides leaves S_M undefined) or a pressure is not positive; es + des
  // shows it, since every quotient above enters it.
  const bool finite = isfinite(es + des);
  if (__any(!finite)) {
    asm volatile("");  // keeps the branch wave-uniform
    if (!finite) {
      if (super) {
        rsa = rho, sm = u, es = e;
        vs1a = u1, vs2a = u2, bs1a = c1, bs2a = c2;
      }
      if (!inner) {
        vss1 = vs1a, vss2 = vs2a, bss1 = bs1a, bss2 = bs2a;
        des = R(0);
      }
    }
  }
  const R s1 = super ? R(0) : S, s2 = inner ? sas : R(0);
  const R ru = rho * u, m1 = rho * u1, m2 = rho * u2;
  F[I_RHO] = ru + s1 * (rsa - rho);
  F[1 + D] = ru * u + pt - bn2 + s1 * (rsa * sm - ru);
  F[1 + T1] = m1 * u - c1 * bn + s1 * (rsa * vs1a - m1) + s2 * (rsa * (vss1 - vs1a));
  F[1 + T2] = m2 * u - c2 * bn + s1 * (rsa * vs2a - m2) + s2 * (rsa * (vss2 - vs2a));
  F[I_EN] = (e + pt) * u - bn * vb + s1 * (es - e) + s2 * des;
  F[I_BX + T1] = u * c1 - bn * u1 + s1 * (bs1a - c1) + s2 * (bss1 - bs1a);
  F[I_BX + T2] = u * c2 - bn * u2 + s1 * (bs2a - c2) + s2 * (bss2 - bs2a);
  F[N] = ps;
  F[I_PSI] = ch * ch * bn;
}

// HLLC for MHD (Li 2005) with the same GLM interface values: Davis bounds
// S_L, S_R as for HLL, contact speed S_M, star-region total pressure
// pT* = rho_L (S_L - u_L)(S_M - u_L) + pT_L; both star states take the
// tangential field and velocity of the HLL average state, and their density,
// momentum and energy from the jump conditions across S_L or S_R.  Only the
// side of the contact the interface lies on is assembled.
template <int D, class R>
__device__ __forceinline__ void hllc_glm_flux(R wl[NV], R wr[NV], R ch, R half_inv_ch, R gamma, R inv_gm1,
                                              R F[NV]) {
  constexpr int N = I_BX + D;
  constexpr int T1 = Transverse<D>::T1, T2 = Transverse<D>::T2;
  const R bn = R(0.5) * (wl[N] + wr[N]) - (wr[I_PSI] - wl[I_PSI]) * half_inv_ch;
  const R ps = R(0.5) * (wl[I_PSI] + wr[I_PSI]) - R(0.5) * ch * (wr[N] - wl[N]);
  wl[N] = bn;
  wr[N] = bn;
  const R rl = wl[I_RHO], rr = wr[I_RHO];
  const R ul = wl[1 + D], ur = wr[1 + D];
  const R bn2 = bn * bn;
  const R t2l = wl[I_BX + T1] * wl[I_BX + T1] + wl[I_BX + T2] * wl[I_BX + T2];
  const R t2r = wr[I_BX + T1] * wr[I_BX + T1] + wr[I_BX + T2] * wr[I_BX + T2];
  const R b2l = bn2 + t2l, b2r = bn2 + t2r;
  const R ptl = wl[4] + R(0.5) * b2l, ptr = wr[4] + R(0.5) * b2r;
  R cl, cr;
  cfast_faces(rl, rr, wl[4], wr[4], t2l, t2r, bn2, gamma, cl, cr);
  const R sl = fmin(ul - cl, ur - cr), sr = fmax(ul + cl, ur + cr);
  // HLL average of density and of the tangential momentum and field
  const R dl = (sl - ul) * rl, dr = (sr - ur) * rr;
  const R isr = rcp3_(sr - sl), idd = rcp3_(dr - dl);
  auto havg = [&](R ql, R qr, R fql, R fqr) { return (sr * qr - sl * ql - (fqr - fql)) * isr; };
  const R rh = havg(rl, rr, rl * ul, rr * ur);
  const R m1h = havg(rl * wl[1 + T1], rr * wr[1 + T1], rl * wl[1 + T1] * ul - wl[I_BX + T1] * bn,
                     rr * wr[1 + T1] * ur - wr[I_BX + T1] * bn);
  const R m2h = havg(rl * wl[1 + T2], rr * wr[1 + T2], rl * wl[1 + T2] * ul - wl[I_BX + T2] * bn,
                     rr * wr[1 + T2] * ur - wr[I_BX + T2] * bn);
  R b1h = havg(wl[I_BX + T1], wr[I_BX + T1], ul * wl[I_BX + T1] - bn * wl[1 + T1],
                     ur * wr[I_BX + T1] - bn * wr[1 + T1]);
  R b2h = havg(wl[I_BX + T2], wr[I_BX + T2], ul * wl[I_BX + T2] - bn * wl[1 + T2],
                     ur * wr[I_BX + T2] - bn * wr[1 + T2]);
  R sm = (dr * ur - dl * ul + ptl - ptr) * idd;
  const R pts = dl * (sm - ul) + ptl;
  // the side of the contact the interface lies on
  const bool left = sl >= -kZeroSpeed<R>, super = left || sr <= kZeroSpeed<R>;
  const bool right = !left && (super || sm < R(0));
  const R rho = right ? rr : rl, u = right ? ur : ul, pt = right ? ptr : ptl, p = right ? wr[4] : wl[4];
  const R u1 = right ? wr[1 + T1] : wl[1 + T1], u2 = right ? wr[1 + T2] : wl[1 + T2];
  const R c1 = right ? wr[I_BX + T1] : wl[I_BX + T1], c2 = right ? wr[I_BX + T2] : wl[I_BX + T2];
  const R S = right ? sr : sl, sa = S - u;
  const R irh = rcp3_(rh), isb = rcp3_(S - sm);
  const R vs1 = m1h * irh, vs2 = m2h * irh;
  const R vbs = sm * bn + vs1 * b1h + vs2 * b2h;
  const R b2 = bn2 + (c1 * c1 + c2 * c2);
  const R v2 = u * u + u1 * u1 + u2 * u2;
  const R e = p * inv_gm1 + R(0.5) * rho * v2 + R(0.5) * b2;
  const R vb = u * bn + u1 * c1 + u2 * c2;
  const R m1 = rho * u1, m2 = rho * u2, ru = rho * u;
  R rs = rho * sa * isb;
  R ms1 = (m1 * sa + bn * (c1 - b1h)) * isb;
  R ms2 = (m2 * sa + bn * (c2 - b2h)) * isb;
  R es = (e * sa - pt * u + pts * sm + bn * (vb - vbs)) * isb;
  // (a factor of zero drops only finite star states: see HLLD)
  const bool finite = isfinite(es);
  if (__any(!finite)) {
    asm volatile("");  // keeps the branch wave-uniform
    if (!finite && super) {
      rs = rho, sm = u, es = e;
      ms1 = m1, ms2 = m2, b1h = c1, b2h = c2;
    }
  }
  const R s1 = super ? R(0) : S;  // F = F_a + S (U* - U_a), F_a when every wave moves one way
  F[I_RHO] = ru + s1 * (rs - rho);
  F[1 + D] = ru * u + pt - bn2 + s1 * (rs * sm - ru);
  F[1 + T1] = m1 * u - c1 * bn + s1 * (ms1 - m1);
  F[1 + T2] = m2 * u - c2 * bn + s1 * (ms2 - m2);
  F[I_EN] = (e + pt) * u - bn * vb + s1 * (es - e);
  F[I_BX + T1] = u * c1 - bn * u1 + s1 * (b1h - c1);
  F[I_BX + T2] = u * c2 - bn * u2 + s1 * (b2h - c2);
  F[N] = ps;
  F[I_PSI] = ch * ch * bn;
}

enum { FLUX_HLL = 0, FLUX_HLLD = 1, FLUX_HLLC = 2 };

// interface flux of the scheme chosen at compile time
template <int FLX, int D, class R>
__device__ __forceinline__ void face_flux(R wl[NV], R wr[NV], R ch, R half_inv_ch, R gamma, R inv_gm1, R F[NV]) {
  if (FLX == FLUX_HLLD)
    hlld_glm_flux<D, R>(wl, wr, ch, half_inv_ch, gamma, inv_gm1, F);
  else if (FLX == FLUX_HLLC)
    hllc_glm_flux<D, R>(wl, wr, ch, half_inv_ch, gamma, inv_gm1, F);
  else
    hll_glm_flux<D, R>(wl, wr, ch, half_inv_ch, gamma, inv_gm1, F);
}

// ... and at run time (the per-kernel path)
template <int D, class R>
__device__ __forceinline__ void face_flux_rt(int flux, R wl[NV], R wr[NV], R ch, R half_inv_ch, R gamma, R inv_gm1,
                                             R F[NV]) {
  if (flux == FLUX_HLLD)
    hlld_glm_flux<D, R>(wl, wr, ch, half_inv_ch, gamma, inv_gm1, F);
  else if (flux == FLUX_HLLC)
    hllc_glm_flux<D, R>(wl, wr, ch, half_inv_ch, gamma, inv_gm1, F);
  else
    hll_glm_flux<D, R>(wl, wr, ch, half_inv_ch, gamma, inv_gm1, F);
}

// First-order fallback at a face: where rho or p of either reconstructed
// state is not positive, both states become the two cell states (cl, cr).
// It is rare, so the selects run only in waves where some lane needs them
// (a wave-uniform branch on the vote).
template <class R>
__device__ __forceinline__ void positivity_fallback(R wl[NV], R wr[NV], const R cl[NV], const R cr[NV]) {
  const bool bad = !((wl[I_RHO] > R(0)) && (wl[4] > R(0)) && (wr[I_RHO] > R(0)) && (wr[4] > R(0)));
  if (__any(bad)) {
    asm volatile("");  // keeps the branch: the compiler would otherwise select unconditionally
    if (bad) {
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        wl[q] = cl[q];
        wr[q] = cr[q];
      }
    }
  }
}

// Fifth-order WENO face values of cell i (cells i-2 .. i+2; 3 ghost layers)
// on its right and its left: candidate polynomials q_k, smoothness indicators
// beta_k, optimal weights (0.1, 0.6, 0.3).  Weights by limiter: 'weno5'
// (Jiang-Shu) d_k / (1e-6 + beta_k)^2; 'wenoz5' (Borges et al.) d_k (1 +
// tau5 / (beta_k + 1e-40)) with tau5 = |beta_0 - beta_2|; 'wenozp5' (Acker et
// al.) d_k (1 + (tau5 / (beta_k + 1e-40))^2 + lambda (beta_k + 1e-40) /
// (tau5 + 1e-40)) with lambda = dx^(2/3).
//
// The two sides share the beta_k and the unweighted factors of the weights:
// the left one exchanges the optimal weights of the first and the third
// stencil.  About 93 issue slots for both against 2 x 82 for each by itself.
// Everything is written in the differences of neighbouring cells, q_k as v0
// plus a correction, and every step is symmetric under reversing the cells,
// so that the left value is bit for bit the right value of the reversed
// cells.  The beta_k are four times the published ones, and so are the
// constants added to them (the weights keep their ratios).
__device__ __forceinline__ void weno5_sides(double vm2, double vm1, double v0, double vp1, double vp2, int lim,
                                            double lambda, double& right, double& left) {
  const double d0 = vm1 - vm2, d1 = v0 - vm1, d2 = vp1 - v0, d3 = vp2 - vp1;
  const double a0 = d1 - d0, a1 = d2 - d1, a2 = d3 - d2;
  auto beta = [](double a, double b) { return (13.0 / 3.0) * a * a + b * b; };
  const double be0 = beta(a0, 3.0 * d1 - d0), be1 = beta(a1, d1 + d2), be2 = beta(a2, 3.0 * d2 - d3);
  // the three reciprocals of the weights come from one reciprocal of their
  // product (the refined hardware reciprocal is the costly operation here);
  // the factors are at least 4e-40 (1.6e-11 for 'weno5'), so the product does
  // not underflow.  It is of the sixth power of the differences (the twelfth
  // for 'weno5') and overflows for values beyond about 1e50 (1e25).
  auto rcp_three = [](double x0, double x1, double x2, double& r0, double& r1, double& r2) {
    const double x02 = x0 * x2;
    const double r = rcp3_(x02 * x1);
    const double t = r * x1;
    r0 = t * x2;
    r1 = r * x02;
    r2 = t * x0;
  };
  double g0, g1, g2;
  if (lim == LIM_WENOZ5 || lim == LIM_WENOZP5) {
    const double tau5 = fabs(be0 - be2);
    const double e0 = be0 + 4e-40, e1 = be1 + 4e-40, e2 = be2 + 4e-40;
    double i0, i1, i2;
    rcp_three(e0, e1, e2, i0, i1, i2);
    const double r0 = tau5 * i0, r1 = tau5 * i1, r2 = tau5 * i2;
    if (lim == LIM_WENOZ5) {
      g0 = 1.0 + r0;
      g1 = 1.0 + r1;
      g2 = 1.0 + r2;
    } else {
      // the weights times tau5 + 1e-40 (their ratios are what counts), which
      // takes the quotient lambda / (tau5 + 1e-40) out
      const double tp = tau5 + 4e-40;
      g0 = tp + (tp * r0) * r0 + lambda * e0;
      g1 = tp + (tp * r1) * r1 + lambda * e1;
      g2 = tp + (tp * r2) * r2 + lambda * e2;
    }
  } else {
    const double e0 = 4e-6 + be0, e1 = 4e-6 + be1, e2 = 4e-6 + be2;
    rcp_three(e0 * e0, e1 * e1, e2 * e2, g0, g1, g2);
  }
  // v0 + (al0 c0 + al1 c1 + al2 c2) / (6 (al0 + al1 + al2)), c_k = 6 (q_k - v0)
  auto value = [&](double ga, double gb, double gc, double ca, double cb, double cc) {
    const double al0 = 0.1 * ga, al1 = 0.6 * gb, al2 = 0.3 * gc;
    const double den = al0 + al1 + al2;
    const double num = (al0 * ca + al1 * cb + al2 * cc) * (1.0 / 6.0);
    const double r = __builtin_amdgcn_rcp(den);
    const double e = fma(-den, r, 1.0);
    const double q = num * r;
    return v0 + fma(q, fma(e, e, e), q);
  };
  right = value(g0, g1, g2, 2.0 * a0 + 3.0 * d1, 3.0 * d2 - a1, 3.0 * d2 - a2);
  left = value(g2, g1, g0, 2.0 * a2 - 3.0 * d2, -3.0 * d1 - a1, -3.0 * d1 - a0);
}

__device__ __forceinline__ double mm2(double a, double b) {
  return (a > 0.0 && b > 0.0) ? fmin(a, b) : ((a < 0.0 && b < 0.0) ? fmax(a, b) : 0.0);
}

__device__ __forceinline__ double mm4(double a, double b, double c, double d) {
  const double lo = fmin(fmin(a, b), fmin(c, d)), hi = fmax(fmax(a, b), fmax(c, d));
  return lo > 0.0 ? lo : (hi < 0.0 ? hi : 0.0);
}

// Monotonicity-preserving fifth-order face value ('mp5', Suresh and Huynh):
// the fifth-order interpolant unless it leaves the interval between u_i and
// u_i + minmod(u_{i+1} - u_i, 4 (u_i - u_{i-1})); then its median with the
// bounds u_min, u_max built from curvature-limited second differences.
__device__ __forceinline__ double mp5_face(double vm2, double vm1, double v0, double vp1, double vp2) {
  const double u_or = (2.0 * vm2 - 13.0 * vm1 + 47.0 * v0 + 27.0 * vp1 - 3.0 * vp2) * (1.0 / 60.0);
  const double back = v0 - vm1;
  const double u_mp = v0 + mm2(vp1 - v0, 4.0 * back);
  if ((u_or - v0) * (u_or - u_mp) <= 0.0) return u_or;
  const double dm1 = vm2 - 2.0 * vm1 + v0, d0 = vm1 - 2.0 * v0 + vp1, dp1 = v0 - 2.0 * vp1 + vp2;
  const double cp = mm4(4.0 * d0 - dp1, 4.0 * dp1 - d0, d0, dp1);
  const double cm = mm4(4.0 * d0 - dm1, 4.0 * dm1 - d0, d0, dm1);
  const double u_ul = v0 + 4.0 * back;
  const double u_md = 0.5 * (v0 + vp1) - 0.5 * cp;
  const double u_lc = v0 + 0.5 * back + (4.0 / 3.0) * cm;
  const double u_min = fmax(fmin(fmin(v0, vp1), u_md), fmin(fmin(v0, u_ul), u_lc));
  const double u_max = fmin(fmax(fmax(v0, vp1), u_md), fmax(fmax(v0, u_ul), u_lc));
  return u_or + mm2(u_min - u_or, u_max - u_or);
}

// The five-cell face values of a cell at face precision R: the stored (R)
// cell values are promoted and the values computed in FP64, then rounded to R.
// (In FP32 the WENO-Z+ term (tau5 / (beta + 1e-40))^2 overflows and 1e-40
// is not representable, so the nonlinear weights stay FP64 on the mixed
// path too.)
template <class R>
__device__ __forceinline__ void five_cell_sides(int lim, R vm2, R vm1, R v0, R vp1, R vp2, double lambda, R& right,
                                                R& left) {
  double r, l;
  if (lim == LIM_MP5) {
    r = mp5_face((double)vm2, (double)vm1, (double)v0, (double)vp1, (double)vp2);
    l = mp5_face((double)vp2, (double)vp1, (double)v0, (double)vm1, (double)vm2);
  } else {
    weno5_sides((double)vm2, (double)vm1, (double)v0, (double)vp1, (double)vp2, lim, lambda, r, l);
  }
  right = (R)r;
  left = (R)l;
}

// Face states from the six cells c[0..5] around the face between c[2] and
// c[3] (3 ghost layers) by a five-cell reconstruction (lambda = dx^(2/3) of
// the block), with the first-order fallback.
template <class R>
__device__ __forceinline__ void reconstruct_face6(int lim, const R c[6][NV], double lambda, R wl[NV], R wr[NV]) {
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    R unused;
    five_cell_sides(lim, c[0][q], c[1][q], c[2][q], c[3][q], c[4][q], lambda, wl[q], unused);
    five_cell_sides(lim, c[1][q], c[2][q], c[3][q], c[4][q], c[5][q], lambda, unused, wr[q]);
  }
  positivity_fallback(wl, wr, c[2], c[3]);
}

// ---------------------------------------------------------------------------
// Slot storage policies.  A slot is [block][...] with pc padded cells per
// block.  FP64: 9 double arrays.  Mixed: 8 float arrays (rho, m_x, m_y, m_z,
// B_x, B_y, B_z, psi) then one double array (e).  Values move as double.

// Address of element `off` bytes into the array at base, a wave-uniform
// address, for the scalar-base form of the global loads and stores (a scalar
// pair and one 32-bit lane offset).  The empty asm keeps the two apart: the
// compiler would otherwise add the lane offset first and form a 64-bit lane
// address for every variable (two VALU additions per access in FP64, where
// the variables of a block lie 64 KB apart, beyond the immediate offsets).
template <class T>
__device__ __forceinline__ T __attribute__((address_space(1))) * lane_ptr(const char* base, unsigned off) {
  auto* p = (__attribute__((address_space(1))) char*)base;
  asm("" : "+s"(p));
  return (T __attribute__((address_space(1)))*)(p + (size_t)off);
}

// A wave-uniform address the compiler takes as new, so that what is added to
// it is not formed once before a loop (a block's variables times its slots
// are more scalar registers than there are).
__device__ __forceinline__ const void* fresh(const void* p) {
  asm volatile("" : "+s"(p));
  return p;
}

struct StoreF64 {
  using R = double;  // face arithmetic type
  static constexpr int kBytesPerCell = 72;
  static constexpr int kWavesPerEU = 2;  // fused-stage occupancy target
  __device__ static double ld(const void* blk, int q, long c, long pc) {
    return static_cast<const double*>(blk)[q * pc + c];
  }
  __device__ static void st(void* blk, int q, long c, long pc, double v) {
    static_cast<double*>(blk)[q * pc + c] = v;
  }
  // the same at cell c of a block whose address is wave-uniform: the
  // variable's address stays scalar and one 32-bit byte offset per lane
  // serves all variables
  __device__ static double ld_at(const void* blk, int q, unsigned c, long pc) {
    return *lane_ptr<double>(static_cast<const char*>(blk) + q * pc * 8, c * 8u);
  }
  __device__ static void st_at(void* blk, int q, unsigned c, long pc, double v) {
    *lane_ptr<double>(static_cast<const char*>(blk) + q * pc * 8, c * 8u) = v;
  }
  // the value a later load of variable q returns after st(v)
  __device__ static double as_stored(int, double v) { return v; }
};

struct StoreMixed {
  using R = float;
  static constexpr int kBytesPerCell = 40;
  static constexpr int kWavesPerEU = 3;
  __device__ static int fidx(int q) { return q < I_EN ? q : q - 1; }
  __device__ static double ld(const void* blk, int q, long c, long pc) {
    if (q == I_EN) return reinterpret_cast<const double*>(static_cast<const char*>(blk) + 32 * pc)[c];
    return (double)static_cast<const float*>(blk)[fidx(q) * pc + c];
  }
  __device__ static void st(void* blk, int q, long c, long pc, double v) {
    if (q == I_EN)
      reinterpret_cast<double*>(static_cast<char*>(blk) + 32 * pc)[c] = v;
    else
      static_cast<float*>(blk)[fidx(q) * pc + c] = (float)v;
  }
  __device__ static double ld_at(const void* blk, int q, unsigned c, long pc) {
    const char* p = static_cast<const char*>(blk);
    if (q == I_EN) return *lane_ptr<double>(p + 32 * pc, c * 8u);
    return (double)*lane_ptr<float>(p + fidx(q) * pc * 4, c * 4u);
  }
  __device__ static void st_at(void* blk, int q, unsigned c, long pc, double v) {
    const char* p = static_cast<const char*>(blk);
    if (q == I_EN)
      *lane_ptr<double>(p + 32 * pc, c * 8u) = v;
    else
      *lane_ptr<float>(p + fidx(q) * pc * 4, c * 4u) = (float)v;
  }
  __device__ static double as_stored(int q, double v) { return q == I_EN ? v : (double)(float)v; }
};

template <class SP>
__device__ __forceinline__ const void* block_ptr(const void* slot, long b, long pc) {
  return static_cast<const char*>(slot) + b * pc * SP::kBytesPerCell;
}
template <class SP>
__device__ __forceinline__ void* block_ptr(void* slot, long b, long pc) {
  return static_cast<char*>(slot) + b * pc * SP::kBytesPerCell;
}

}  // namespace amrvac
