// One Lanczos step in one pass: the window's dot products on the matrix cores
// and the scalar recurrence.  Internal; the one-block sweeps share the products and
// the small exponential.
//
// u_i are the stored (unnormalised) basis vectors, y_i = H u_i, and the pass
// of step k forms
//   u_k = sig w'_{k-1} - c_{k-1} u_{k-1},  y_k = sig H w'_{k-1} - c_{k-1} y_{k-1}
//   w'_k = s_k y_k - sum_{i < k in the window} c^(k)_i u_i
// (w'_0 = y_0, sig = s_0 in step 1 and 1 after).  The newest coefficient
// c_k = s_k <u_k|y_k> / ||u_k||^2 needs a sum over the whole vector of this
// step's own H v, so its subtraction is deferred to the next pass; H is
// linear, so y follows w' without another H v (within limits: see kMaxGrowth).  The
// pass measures
//   A_i = <u_i|y_k>, G_i = <u_i|u_k> for the window,
//   <u_k|y_k>, ||u_k||^2, ||y_k||^2,
// from which step_scalars derives everything the next pass needs.  s_k only
// keeps the vectors' scale (it estimates 1/||u_k|| before u_k exists); the
// tridiagonal matrix takes the measured norms.
#pragma once

#include "kg_device.h"

namespace kg {
namespace {

// A wavefront takes a unit of 64 amplitudes against four vectors at a time:
// lane l holds vector 4g + (l & 3) at amplitudes 16 t + (l >> 2), t = 0..3.  In
// that layout a vector's components are the A operand of v_mfma_f64_4x4x4
// (row l & 3, 16 inner amplitudes over the lane's quads) and
// (yr, yi, xr, xi) the B operand (column l & 3), so the four real dots of every
// vector accumulate over the amplitudes in one register per four vectors and
// two lane exchanges finish them.  The update sum_i c_i u_i is four FMA per
// amplitude on the vector unit; its quad sum is taken once per unit.
__device__ __forceinline__ uint32_t unit_amp(int t, uint32_t a) { return 16u * (uint32_t)t + a; }

// Makes this wavefront's LDS writes visible to its other lanes.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The B operands of one amplitude: v = (yr, yi, xr, xi)[l & 3], and
// (yi, -yr, xi, -xr)[l & 3] for the imaginary parts: conj(q) y = qr B + qi B'.
__device__ __forceinline__ double turned(double v) {
  const double p = dpp_f64<0xB1>(v);   // quad_perm [1,0,3,2]
  return (threadIdx.x & 1u) ? -p : p;
}

// Four amplitudes of four vectors: dots into d0 + d1.
template <typename V>
__device__ __forceinline__ void unit_mfma(const V (&q)[4], const double (&b)[4],
                                          const double (&bp)[4], double& d0, double& d1) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const double qr = q[t].x, qi = q[t].y;
    d0 = __builtin_amdgcn_mfma_f64_4x4x4f64(qr, b[t], d0, 0, 0, 0);
    d1 = __builtin_amdgcn_mfma_f64_4x4x4f64(qi, bp[t], d1, 0, 0, 0);
  }
}

// The same with the update into zr, zi.
template <typename V>
__device__ __forceinline__ void unit_rows(const V (&q)[4], const double (&b)[4],
                                          const double (&bp)[4], cplx_d w, double (&zr)[4],
                                          double (&zi)[4], double& d0, double& d1) {
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const double qr = q[t].x, qi = q[t].y;
    d0 = __builtin_amdgcn_mfma_f64_4x4x4f64(qr, b[t], d0, 0, 0, 0);
    d1 = __builtin_amdgcn_mfma_f64_4x4x4f64(qi, bp[t], d1, 0, 0, 0);
    zr[t] += w.re * qr - w.im * qi;
    zi[t] += w.re * qi + w.im * qr;
  }
}

// The dots of four vectors over the unit from their two accumulators: every lane of
// row l >> 4 (the vector) holds the total of column l & 3.  A v_mfma_f64_4x4x4 result
// may be read by the vector unit after six wait states; the wait is written out here,
// since hipcc 7.2 leaves it out where a branch ends between the two (the sums then
// held the registers' old values).
__device__ __forceinline__ double unit_dots(double d0, double d1) {
  asm volatile("s_nop 7" : "+v"(d0), "+v"(d1));
  double v = d0 + d1;
  v += dpp_f64<0x124>(v);   // row_ror:4 and :8: the instruction's four blocks
  v += dpp_f64<0x128>(v);
  return v;
}

// Sums the lanes' parts of z over the quad; the lane keeps the sum for its
// amplitude unit_amp(l & 3, l >> 2).
__device__ __forceinline__ double quad_z(const double (&z)[4]) {
  const bool hi = (threadIdx.x & 2u) != 0, lo = (threadIdx.x & 1u) != 0;
  const double s0 = hi ? z[0] : z[2], s1 = hi ? z[1] : z[3];
  const double k0 = (hi ? z[2] : z[0]) + dpp_f64<0x4E>(s0);   // quad_perm [2,3,0,1]
  const double k1 = (hi ? z[3] : z[1]) + dpp_f64<0x4E>(s1);
  return (lo ? k1 : k0) + dpp_f64<0xB1>(lo ? k0 : k1);
}

// ---------------------------------------------------------------------- scalars

// The recurrence's scalars, vector i in lane i of a wavefront.
struct LzLane {
  double al = 0.0, of = 0.0;    // diagonal and off-diagonal (with i-1) of T
  double G = 0.0, sc = 0.0;     // ||u_i||^2, 1/||u_i||
  double sh = 0.0, ish = 0.0;   // the scale s_i used in w'_i, and 1/s_i
  cplx_d cd{0.0, 0.0};          // c^(i)_i
  cplx_d cs{0.0, 0.0};          // c^(i)_{i-1}
  cplx_d cw{0.0, 0.0};          // c^(k)_i of the step to come, zero outside its window
  cplx_d gp{0.0, 0.0};          // <u_i|u_{k-1}> of the step before
};

// The same in LDS, where the registers are wanted for the pass between two
// steps' scalars.
struct LzStore {
  double v[14][64];
};

__device__ __forceinline__ void put_lane(LzStore& o, const LzLane& s) {
  const int l = threadIdx.x & 63;
  const double v[14] = {s.al, s.of, s.G, s.sc, s.sh, s.ish, s.cd.re, s.cd.im, s.cs.re, s.cs.im,
                        s.cw.re, s.cw.im, s.gp.re, s.gp.im};
#pragma unroll
  for (int i = 0; i < 14; ++i) o.v[i][l] = v[i];
}

__device__ __forceinline__ void get_lane(const LzStore& o, LzLane& s) {
  const int l = threadIdx.x & 63;
  s.al = o.v[0][l];
  s.of = o.v[1][l];
  s.G = o.v[2][l];
  s.sc = o.v[3][l];
  s.sh = o.v[4][l];
  s.ish = o.v[5][l];
  s.cd = cplx_d{o.v[6][l], o.v[7][l]};
  s.cs = cplx_d{o.v[8][l], o.v[9][l]};
  s.cw = cplx_d{o.v[10][l], o.v[11][l]};
  s.gp = cplx_d{o.v[12][l], o.v[13][l]};
}

struct LzRun {
  double normT = 0.0;           // max (|alpha_i| + offd_i) so far
  double beta0 = 0.0;           // ||u_0||
  double sk = 0.0;              // s_k of the step to come
  double rp = 0.0;              // 1/(s_{k-1} ||u_{k-1}||)
  double gp = 0.0, ig = 0.0;    // ||u_{k-1}||^2 and its inverse
  // Bound of ||y_k - H u_k|| in roundings of ||H|| ||u_k||: 1 where y_k = H u_k was
  // formed, and r (g + 1) + 1 after a step of the recurrence, r = |c_k| ||u_k|| /
  // ||u_{k+1}|| (|alpha_k| / beta_{k+1}).
  double g = 1.0;
  int m_eff = 0;
};

// Where the recurrence would lose accuracy, the next pass forms y = H u itself and takes
// the remainder d of the coefficient on u_{k-1} out of u_{k+1} too: c_{k-1} was derived
// with an estimate of ||u_k||^2, made before u_k was rounded, and is measured now.
// That is when g, or |d| ||u_{k-1}|| / ||u_{k+1}|| in units of the vectors' roundoff
// (complex128: of 2^-50, what FP64 sums of a few terms leave of the estimate), exceeds
// this limit.  With couplings and controls of order one and random states g stays below
// 3.5 and d below 1 / sqrt(D).  Of 2,000 random calls (complex64 and complex128, L =
// 5..8) the errors were 1.01 (complex64) and 0.98 (complex128) times those of two passes
// a step in the geometric mean with strong fields and product states, where r reaches
// 200, and 1.03 and 1.07 with ordinary ones; without this 1.5 and 1.2 with the strong
// ones, and up to 5,000 times in single calls.  Limits of 4 to 16 differ by 5 %.
constexpr double kMaxGrowth = 8.0;

// sqrt(v) and its inverse, both to the last bit or nearly: the library's rsqrt alone
// leaves 1 to 2 units in their product, which scale every slice's state the same way
// (30 slices at D = 256, complex128: state error 2.9e-15, this 1.0e-15).  NaN and 0 as sqrt
// and 1 / sqrt give them.
__device__ __forceinline__ void norm_and_inverse(double v, double& n, double& inv) {
  inv = rsqrt(v);
  n = v > 0.0 ? v * inv : v;
  if (v > 0.0) {
    n = fma(fma(-n, n, v), 0.5 * inv, n);
    inv = fma(fma(-n, inv, 1.0), inv, inv);
  }
}

__device__ __forceinline__ cplx_d lane_cplx(const cplx_d& v, int l) {
  return cplx_d{lane_value(v.re, l), lane_value(v.im, l)};
}

__device__ __forceinline__ int window_first(int k, int m, int reorth) {
  return k == m - 1 ? k : (reorth ? 0 : (k > 0 ? k - 1 : 0));
}

// What a step hands to the next one.
struct StepNext {
  cplx_d c;     // the deferred coefficient c_k
  double sig;   // scale of w'_k in u_{k+1}
  double s;     // scale of y_{k+1} in w'_{k+1}
  cplx_d d;     // the remainder on u_{k-1}
  double fresh; // 1: y_{k+1} = H u_{k+1} is formed, and d applies; else 0
};

// The scalars after the pass of step k, on one wavefront.  A, Gm: lane i in
// [i0, k) holds A_i, G_i; akk = <u_k|y_k>, gkk = ||u_k||^2, yy = ||y_k||^2 the
// same in every lane.  Returns true when the basis goes on; then s.cw holds
// the window coefficients of step k+1.  `unit`: the vectors' unit roundoff.  False at the last step or when the
// basis ends before u_k (a breakdown: ||u_k|| small against ||T||, an
// invariant space of dimension k; a zero or non-finite input): r.m_eff is its
// dimension.
//
// Window dots of step k+1, d_i = <u_i|H u_{k+1}> = <y_i|u_{k+1}>, from what the
// pass measured (H is Hermitian): with w'_i's definition
//   d_i = (e_{i+1} + conj(c^(i)_i) e_i + conj(c^(i)_{i-1}) e_{i-1}) / s_i,
//   e_j = <u_j|u_{k+1}> = s_k A_j - c_k G_{j,k} - c_{k-1} G_{j,k-1} - c_j ||u_j||^2,
// e_{k+1} = ||u_{k+1}||^2 = ||s_k y_k - c_k u_k - c_{k-1} u_{k-1}||^2; products
// of two terms of the order of the rounding error (the Gram entries and
// coefficients beyond the three-term window) are dropped.
__device__ __forceinline__ bool step_scalars(LzLane& s, LzRun& r, int k, int m, int reorth, double tol,
                                             double unit, cplx_d A, cplx_d Gm, cplx_d akk, double gkk, double yy,
                                             StepNext& nx) {
  const int lane = threadIdx.x & 63;
  if (k == 0 && !(gkk > 0.0)) {
    // a zero input gives a zero output; a non-finite one a NaN output
    r.beta0 = gkk == 0.0 ? 0.0 : NAN;
    r.m_eff = gkk == 0.0 ? 0 : 1;
    s.al = 0.0;
    s.sc = 1.0;
    return false;
  }
  double nrm, inv;                                  // u_k = 0 is a breakdown
  norm_and_inverse(gkk, nrm, inv);
  const int km = k > 0 ? k - 1 : 0;
  // ||u_k|| / (s_{k-1} ||u_{k-1}||): the off-diagonal entry
  const double off = k > 0 ? nrm * r.rp : 0.0;
  if (k > 0 && off <= tol * fmax(1.0, r.normT)) {
    r.m_eff = k;
    return false;
  }
  if (k == 0) r.beta0 = nrm;
  const double inv2 = inv * inv;
  const double alpha = akk.re * inv2;
  r.normT = fmax(r.normT, fabs(alpha) + off);
  const bool top = lane == k;
  if (top) {
    s.al = alpha;
    s.of = off;
    s.G = gkk;
    s.sc = inv;
    if (k == 0) {
      s.sh = inv;
      s.ish = nrm;
    }
  }
  if (k == m - 1) {
    r.m_eff = m;
    return false;
  }
  const double sk = k == 0 ? inv : r.sk;
  const cplx_d ck{akk.re * sk * inv2, akk.im * sk * inv2};
  if (top) s.cd = ck;
  const int i0 = window_first(k, m, reorth), kn = k + 1, i0n = window_first(kn, m, reorth);
  // ||u_{k+1}||^2, kept away from zero; the coefficient on u_{k-1} as measured
  double big = sk * sk * yy;
  double b2 = big - sk * (ck.re * akk.re + ck.im * akk.im);
  const bool prev = k > 0 && km >= i0;
  cplx_d cp{0.0, 0.0}, gk{0.0, 0.0}, d{0.0, 0.0};
  if (prev) {
    const cplx_d ap = lane_cplx(A, km), used = lane_cplx(s.cw, km);
    gk = lane_cplx(Gm, km);
    const double f = sk * r.ig;
    cp = cplx_d{f * ap.re, f * ap.im};
    d = cplx_d{cp.re - used.re, cp.im - used.im};
    b2 += (cp.re * cp.re + cp.im * cp.im) * r.gp - 2.0 * sk * (cp.re * ap.re + cp.im * ap.im) +
          2.0 * ((cp.re * ck.re + cp.im * ck.im) * gk.re - (cp.re * ck.im - cp.im * ck.re) * gk.im);
  }
  b2 = fmax(b2, 1e-28 * big + 1e-300);
  double bn, sn;
  norm_and_inverse(b2, bn, sn);
  const double lim = kMaxGrowth * fmax(unit, 0x1p-50);
  // a bound: single precision will do
  const double ratio = (double)__builtin_sqrtf((float)((ck.re * ck.re + ck.im * ck.im) * gkk * (sn * sn)));
  const double g1 = ratio * (r.g + 1.0) + 1.0;
  const bool fresh = g1 > kMaxGrowth || (d.re * d.re + d.im * d.im) * r.gp > lim * lim * b2;
  if (!fresh) {
    cp = cplx_d{cp.re - d.re, cp.im - d.im};
    d = cplx_d{0.0, 0.0};
  }
  double er = 0.0, ei = 0.0;
  const bool in = lane >= i0 && lane <= k;
  {
    const cplx_d a = top ? akk : A;
    const cplx_d g = top ? cplx_d{gkk, 0.0} : Gm;
    er = sk * a.re - (ck.re * g.re - ck.im * g.im);
    ei = sk * a.im - (ck.re * g.im + ck.im * g.re);
  }
  if (prev) {
    const cplx_d g = top ? cplx_d{gk.re, -gk.im} : (lane == km ? cplx_d{s.G, 0.0} : s.gp);
    er -= cp.re * g.re - cp.im * g.im;
    ei -= cp.re * g.im + cp.im * g.re;
    if (lane < km) {
      er -= s.cw.re * s.G;
      ei -= s.cw.im * s.G;
    }
    if (top) s.cs = cp;
  }
  if (!in) {
    er = lane == kn ? b2 : 0.0;
    ei = 0.0;
  }
  const double e1r = dpp_f64<0x130>(er), e1i = dpp_f64<0x130>(ei);   // lane i + 1
  const double emr = dpp_f64<0x138>(er), emi = dpp_f64<0x138>(ei);   // lane i - 1
  cplx_d cw{0.0, 0.0};
  if (lane >= i0n && lane <= k) {
    double dr = e1r + s.cd.re * er + s.cd.im * ei;
    double di = e1i + s.cd.re * ei - s.cd.im * er;
    if (lane > i0) {
      dr += s.cs.re * emr + s.cs.im * emi;
      di += s.cs.re * emi - s.cs.im * emr;
    }
    const double f = sn * (s.sc * s.sc * s.ish);
    cw = cplx_d{dr * f, di * f};
  }
  const double csr = dpp_f64<0x138>(cw.re), csi = dpp_f64<0x138>(cw.im);
  if (lane == kn) {
    s.sh = sn;
    s.ish = bn;
    s.cs = cplx_d{csr, csi};
  }
  // 1/(s_k ||u_k||); s_0 is 1/||u_0|| itself
  r.rp = k == 0 ? 1.0 : inv * lane_value(s.ish, k);
  r.gp = gkk;
  r.ig = inv2;
  r.sk = sn;
  s.cw = cw;
  s.gp = (lane >= i0 && lane < k) ? Gm : cplx_d{0.0, 0.0};
  nx.c = ck;
  nx.sig = k == 0 ? sk : 1.0;
  nx.s = sn;
  nx.d = d;
  nx.fresh = fresh ? 1.0 : 0.0;
  r.g = fresh ? 1.0 : g1;
  return true;
}

// exp(-i t T) e_1 from the lanes' rows, times beta0 / ||u_i||: the combination
// coefficient of stored vector i in lane i (zero past m_eff).
__device__ __forceinline__ cplx_d comb_coef(const LzLane& s, const LzRun& r, double t) {
  const int i = threadIdx.x & 63;
  const bool in = i < r.m_eff;
  const double ai = in ? s.al : 0.0;
  const double lo = (in && i > 0) ? s.of : 0.0;
  const double up = dpp_f64<0x130>(s.of);
  const double hi = (i + 1 < r.m_eff) ? up : 0.0;
  double cr, ci;
  tri_exp_wave(ai, lo, hi, t, cr, ci);
  const double f = r.beta0 * s.sc;
  return in ? cplx_d{f * cr, f * ci} : cplx_d{0.0, 0.0};
}

}  // namespace
}  // namespace kg
