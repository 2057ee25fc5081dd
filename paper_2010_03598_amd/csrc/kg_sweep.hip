// Short vectors: a block runs a whole sweep of Krylov calls.
//
// For D <= 1024 amplitudes whose basis fits in LDS, one block carries a chain
// of Krylov calls (Algorithm 2, the small exponential of Eqs. A2-A3 and the
// combination; each call's output is the next one's input) without leaving the
// compute unit: no launch, no global round trip and one barrier per Lanczos
// step.  Independent sweeps (the forward states and the costates of a
// gradient, the columns of an operator) are the blocks of one launch.
//
// Such a step is a serial chain on one compute unit: H v from LDS, the window's
// dots, the sums over the block, the scalars, the update.  It is bound by that
// chain's latency, so it is kept short: one amplitude per thread with its neighbour
// list in registers; the dots by MFMA, ||u_k||^2 among them; and every wavefront
// computes the scalars itself, which saves a barrier and a round trip through LDS.
//
// Every dot is taken with y_k = H u_k itself, and w_k is complete in FP64 before it
// is rounded: the single-pass step of kg_step.h (one barrier a step here) defers a
// subtraction of the size of alpha_k past that rounding, and its accuracy falls with
// |alpha_k| / beta_{k+1}.
//
// Measured against one launch per call with two block-wide sums and three barriers per
// step, in complex128: the gradient of 50 slices at D = 256, m = 10 takes 0.91 ms
// (2.88), the centred one of 584 slices at D = 146 10.9 ms (45.2), one call alone at
// D = 256 20.1 us (29.5), at D = 512 and m = 12 37.3 us (42.0).  The single-pass step
// took 1.18 ms, 14.2 ms, 25.5 us and 39.3 us: its scalars are a longer chain than the
// second barrier.
//
// LDS: slot i (stride DS) holds u_i, then one slot of y in units of wavefronts.

#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include "kg_device.h"
#include "kg_internal.h"
#include "kg_step.h"

namespace kg {
namespace {

constexpr int kSweepNbr = 12;             // neighbours per row held in registers
constexpr size_t kSweepLds = 160u << 10;  // LDS of a compute unit
constexpr int kSweepThreads = 512;        // largest block

struct SweepBatch {
  SweepJob job[kSweepJobs];
};

// Vector stride in LDS: padded so that the four vectors a wavefront reads at
// once start 64 bytes apart modulo the 256 bytes of the banks.
template <typename R>
__host__ __device__ inline uint32_t slot_stride(uint32_t D) {
  const uint32_t unit = sizeof(R) == 4 ? 32u : 16u, want = unit / 4u;
  return D + ((want + unit - (D % unit)) % unit);
}

// Rows per thread: one up to eight wavefronts; beyond, two (16 wavefronts of
// one row would run four to a SIMD and repeat the per-wavefront work).
inline int sweep_rows(uint32_t D) { return D <= (uint32_t)kSweepThreads ? 1 : 2; }

template <typename R>
inline size_t sweep_lds_bytes(uint32_t D, int m) {
  const size_t na = sweep_rows(D), nw = (D + 64 * na - 1) / (64 * na);
  const size_t vecs = ((size_t)m * slot_stride<R>(D) + na * nw * 64) * sizeof(typename VT<R>::T);
  const size_t meas = nw * (size_t)(4 * m) * sizeof(double);
  const size_t coef = nw * kMaxM * sizeof(cplx_d);
  return ((vecs + 15) / 16) * 16 + meas + coef;
}

// Address of call q's output.
template <typename V>
__device__ __forceinline__ V* sweep_out(const SweepJob& J, int q, int j) {
  size_t at;
  if (!J.states) {
    at = (size_t)q;
  } else if (J.c == 0) {
    at = (size_t)(j - 1);
  } else {
    const int seg = (j - 1) / J.c;
    if (j % J.c == 0 && seg < J.nseg - 1) {
      at = (size_t)seg;
    } else {
      const int b = J.nbuf == 2 ? (seg & 1) : 0;
      at = (size_t)(J.nseg - 1 + b * J.c + (j - seg * J.c - 1));
    }
  }
  return reinterpret_cast<V*>(J.out + at * J.vb);
}

// NA: rows per thread, blockDim apart.  TH: largest block.  PE: the reduced basis.
template <typename R, int NA, int TH, bool PE>
__global__ void __launch_bounds__(TH) k_sweep(SweepBatch Bt) {
  using V = typename VT<R>::T;
  const SweepJob& J = Bt.job[blockIdx.x];
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, T = blockDim.x;
  const uint32_t wv = uniform_u32(tid >> 6), nwv = T >> 6;
  const uint32_t c = lane & 3u, a = lane >> 2;
  const uint32_t D = J.D, DS = slot_stride<R>(D);
  const int m = J.m;
  V* ub = reinterpret_cast<V*>(smem_raw);
  V* yst = ub + (size_t)m * DS;
  const uint32_t vecs = (uint32_t)m * DS + NA * T;
  double* wred = reinterpret_cast<double*>(smem_raw + (((size_t)vecs * sizeof(V) + 15) / 16) * 16);
  const uint32_t rowlen = 4u * (uint32_t)m;
  cplx_d* cfs = reinterpret_cast<cplx_d*>(wred + nwv * rowlen) + wv * (uint32_t)kMaxM;

  // rows past D (and the padding that whole units read) stay finite
  if (D != NA * T)
    for (uint32_t i = tid; i < vecs; i += T) ub[i] = V{(R)0, (R)0};

  // this thread's rows: diagonal d0 + u dz, neighbours and their weights
  const int L = J.hv.L;
  const bool sx = J.hv.hc_kind == 0;
  const int slots = J.nbr;
  uint32_t nb[NA][kSweepNbr], flip[NA];
  R wt[NA][kSweepNbr], d0[NA], dz[NA];
  bool in[NA];
  uint32_t row[NA];
#pragma unroll
  for (int n = 0; n < NA; ++n) {
    in[n] = tid + n * T < D;
    row[n] = in[n] ? tid + n * T : 0u;
    dz[n] = (R)0;
#pragma unroll
    for (int i = 0; i < kSweepNbr; ++i) {
      nb[n][i] = row[n];
      wt[n][i] = (R)0;
    }
    const R hJ = (R)J.hv.half_J;
    const uint32_t bondmask = (L >= 2) ? ((1u << (L - 1)) - 1u) : 0u;
    const uint32_t r = PE ? J.pe.reps[row[n]] : row[n];
    const uint32_t anti = (r ^ (r >> 1)) & bondmask;
    d0[n] = (R)J.hv.c_zz * (R)(L - 1 - 2 * (int)__popc(anti));
    if (!sx) dz[n] = (R)(0.5 * J.hv.sz_count) - (R)__popc(r & J.hv.sz_mask);
    if constexpr (!PE) {
#pragma unroll
      for (int i = 0; i < kSweepNbr; ++i) {
        if ((anti >> i) & 1u) {
          nb[n][i] = r ^ (3u << i);
          wt[n][i] = hJ;
        }
      }
    } else {
      uint32_t act = anti;
      const uint32_t full = (L == 32) ? 0xFFFFFFFFu : ((1u << L) - 1u);
      const uint32_t rank = J.pe.ranks[row[n]];
      const bool nb2 = (__brev(r) >> (32 - L)) != r;
      bool bad = rank >= J.pe.nsec;
#pragma unroll
      for (int i = 0; i < kSweepNbr; ++i) {
        if (i < slots && act && !bad) {
          const int q = __builtin_ctz(act);
          act &= act - 1u;
          const uint32_t s2 = r ^ (3u << q);
          // the orbit through the combinatorial rank over the zero bits
          const uint32_t dl = J.pe.binom[q * kPeBinom + __popc(~r & full & ((1u << q) - 1u))];
          const uint32_t rk = (((r >> q) & 1u) == 0u) ? rank + dl : rank - dl;
          const int32_t ai = (rk < J.pe.nsec) ? J.pe.index[rk] : -1;
          const bool ok = (uint32_t)ai < D;
          bad = bad || !ok;
          const bool na2 = (__brev(s2) >> (32 - L)) != s2;
          nb[n][i] = ok ? (uint32_t)ai : row[n];
          wt[n][i] = hJ * ((nb2 == na2) ? (R)1 : (nb2 ? (R)1.4142135623730951 : (R)0.70710678118654752));
        }
      }
      // a table entry out of range turns the row into NaN, never a stray read
      if (bad) d0[n] = (R)NAN;
    }
    if (!in[n]) {
      d0[n] = dz[n] = (R)0;
#pragma unroll
      for (int i = 0; i < kSweepNbr; ++i) wt[n][i] = (R)0;
    }
    flip[n] = sx ? (row[n] ^ (1u << J.hv.hc_bit)) : row[n];
  }

  V xin[NA];
#pragma unroll
  for (int n = 0; n < NA; ++n)
    xin[n] = in[n] ? reinterpret_cast<const V*>(J.in)[row[n]] : V{(R)0, (R)0};
  double unext = J.u ? J.u[J.j0 - 1] : J.hv.u_val;
  for (int q = 0; q < J.n; ++q) {
    const int j = J.j0 + q * J.dj;
    const double u = unext;
    if (J.u && q + 1 < J.n) unext = J.u[j + J.dj - 1];
    const R cu = sx ? (R)(0.5 * u) : (R)0;
    // the recurrence's scalars, vector i in lane i of every wavefront
    double al = 0.0, of = 0.0, sc = 0.0;
    double normT = 0.0, beta0 = 0.0;
    int me = m;
#pragma unroll
    for (int n = 0; n < NA; ++n)
      if (in[n]) ub[row[n]] = xin[n];
    __syncthreads();
    for (int k = 0; k < m; ++k) {
      const bool last = k == m - 1;
      const int i0 = window_first(k, m, J.reorth), nrows = k - i0 + 1;
      const V* uk = ub + (size_t)k * DS;
      R hr[NA], hi[NA];
#pragma unroll
      for (int n = 0; n < NA; ++n) {
        // ---- y = H u_k on this row, in the vector type
        const V xs = uk[row[n]], xf = uk[flip[n]];
        const R diag = d0[n] + (R)u * dz[n];
        R yr = diag * xs.x, yi = diag * xs.y;
        // four neighbours' reads in flight together; unused slots have weight 0
#pragma unroll
        for (int i = 0; i < kSweepNbr; i += 4) {
          if (i < slots) {
            V x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = uk[nb[n][i + e]];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              yr += wt[n][i + e] * x[e].x;
              yi += wt[n][i + e] * x[e].y;
            }
          }
        }
        yr += cu * xf.x;
        yi += cu * xf.y;
        hr[n] = in[n] ? yr : (R)0;
        hi[n] = in[n] ? yi : (R)0;
        yst[tid + n * T] = V{hr[n], hi[n]};
      }
      wave_lds_fence();
      // ---- rows [i0, k] against (y, u_k), a unit of 64 per n
      double b[NA][4], bp[NA][4];
#pragma unroll
      for (int n = 0; n < NA; ++n) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const uint32_t sa = ((wv + nwv * n) << 6) + unit_amp(t, a);
          const R v = reinterpret_cast<const R*>((c < 2u ? yst : uk) + sa)[c & 1u];
          b[n][t] = sa < D ? (double)v : 0.0;
          bp[n][t] = turned(b[n][t]);
        }
      }
      double* wrow = wred + wv * rowlen;
      for (int r0 = 0; r0 < nrows; r0 += 8) {
        const bool two = r0 + 4 < nrows;
        const auto at = [&](int r) { return ub + (size_t)(i0 + min(r, nrows - 1)) * DS; };
        const V* p0 = at(r0 + (int)c);
        const V* p1 = at(r0 + 4 + (int)c);
        double e0 = 0.0, e1 = 0.0, f0 = 0.0, f1 = 0.0;
#pragma unroll
        for (int n = 0; n < NA; ++n) {
          const uint32_t s0 = (wv + nwv * n) << 6;
          V q0[4], q1[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) q0[t] = p0[s0 + unit_amp(t, a)];
          if (two) {
#pragma unroll
            for (int t = 0; t < 4; ++t) q1[t] = p1[s0 + unit_amp(t, a)];
          }
          unit_mfma(q0, b[n], bp[n], e0, e1);
          if (two) unit_mfma(q1, b[n], bp[n], f0, f1);
        }
        const int r = r0 + (int)(lane >> 4);
        const double e = unit_dots(e0, e1);
        if ((lane & 12u) == 0u && r < nrows) wrow[4 * r + (int)c] = e;
        if (two) {
          const double f = unit_dots(f0, f1);
          if ((lane & 12u) == 0u && r + 4 < nrows) wrow[4 * (r + 4) + (int)c] = f;
        }
      }
      __syncthreads();
      // ---- totals over the wavefronts, in order, and the scalars
      const int r = (int)lane - i0;
      double tr = 0.0, ti = 0.0, tg = 0.0;   // <u_i|y>, Re <u_i|u_k>
      if (r >= 0 && r < nrows) {
        const double* p = wred + 4 * r;
        for (uint32_t w0 = 0; w0 < nwv; w0 += 4) {
          double2 x[4];
          double g[4];
#pragma unroll
          for (uint32_t e = 0; e < 4; ++e) {
            const double* pw = p + min(w0 + e, nwv - 1u) * rowlen;
            x[e] = *reinterpret_cast<const double2*>(pw);
            g[e] = pw[2];
          }
#pragma unroll
          for (uint32_t e = 0; e < 4; ++e) {
            if (w0 + e < nwv) {
              tr += x[e].x;
              ti += x[e].y;
              tg += g[e];
            }
          }
        }
      }
      const double gkk = lane_value(tg, k), akk = lane_value(tr, k);
      if (k == 0 && !(gkk > 0.0)) {
        // a zero input gives a zero output; a non-finite one a NaN output
        me = gkk == 0.0 ? 0 : 1;
        beta0 = NAN;
        break;
      }
      double nrm, sk;                                  // u_k = 0 is a breakdown
      norm_and_inverse(gkk, nrm, sk);
      const double off = k > 0 ? nrm : 0.0;
      if (k == 0) beta0 = nrm;
      // ||u_k|| small against ||T||: an invariant Krylov space of dimension k
      if (k > 0 && off <= J.tol * fmax(1.0, normT)) {
        me = k;
        break;
      }
      const double alpha = sk * sk * akk;
      normT = fmax(normT, fabs(alpha) + off);
      if ((int)lane == k) {
        al = alpha;
        of = off;
        sc = sk;
      }
      if (last) break;
      // ---- w = s_k y - sum_i c_i u_i, c_i = s_i^2 s_k <u_i|y>, stored as u_{k+1}
      const double f = sc * sc * sk;
      cfs[lane] = cplx_d{f * tr, f * ti};
      wave_lds_fence();
      double wr[NA], wi[NA];
#pragma unroll
      for (int n = 0; n < NA; ++n) {
        wr[n] = sk * (double)hr[n];
        wi[n] = sk * (double)hi[n];
      }
#pragma unroll 4
      for (int i = i0; i <= k; ++i) {
        const cplx_d d = cfs[i];
#pragma unroll
        for (int n = 0; n < NA; ++n) {
          const V x = ub[(size_t)i * DS + row[n]];
          wr[n] -= d.re * x.x - d.im * x.y;
          wi[n] -= d.re * x.y + d.im * x.x;
        }
      }
#pragma unroll
      for (int n = 0; n < NA; ++n)
        if (in[n]) ub[(size_t)(k + 1) * DS + row[n]] = V{(R)wr[n], (R)wi[n]};
      __syncthreads();
    }
    // ---- exp(-itT) e_1 and the combination
    LzLane s;
    LzRun run;
    s.al = al;
    s.of = of;
    s.sc = sc;
    run.beta0 = beta0;
    run.m_eff = me;
    cfs[lane] = comb_coef(s, run, J.t);
    wave_lds_fence();
    double orr[NA], oi[NA];
#pragma unroll
    for (int n = 0; n < NA; ++n) orr[n] = oi[n] = 0.0;
#pragma unroll 4
    for (int i = 0; i < me; ++i) {
      const cplx_d d = cfs[i];
#pragma unroll
      for (int n = 0; n < NA; ++n) {
        const V x = ub[(size_t)i * DS + row[n]];
        orr[n] += d.re * x.x - d.im * x.y;
        oi[n] += d.re * x.y + d.im * x.x;
      }
    }
#pragma unroll
    for (int n = 0; n < NA; ++n) {
      xin[n].x = in[n] ? (R)orr[n] : (R)0;
      xin[n].y = in[n] ? (R)oi[n] : (R)0;
      if (in[n]) sweep_out<V>(J, q, j)[row[n]] = xin[n];
    }
    if (J.m_eff_out && tid == 0) *J.m_eff_out = me;
  }
}

template <typename R, int NA, int TH, bool PE>
hipError_t launch_sweep_t(const SweepBatch& b, int n, size_t lds, uint32_t threads, hipStream_t s) {
  static std::atomic<uint64_t> raised{0};
  const hipError_t e = allow_lds(&k_sweep<R, NA, TH, PE>, lds, kSweepLds, raised);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_sweep<R, NA, TH, PE>), dim3(n), dim3(threads), lds, s, b);
  return hipGetLastError();
}

template <typename R, bool PE>
hipError_t launch_sweep_r(const SweepBatch& b, int n, hipStream_t s) {
  const uint32_t D = b.job[0].D;
  const int na = sweep_rows(D);
  const uint32_t threads = (D + 64u * na - 1u) / (64u * na) * 64u;
  const size_t lds = sweep_lds_bytes<R>(D, b.job[0].m);
  if (na == 1)
    return threads <= 256u ? launch_sweep_t<R, 1, 256, PE>(b, n, lds, threads, s)
                           : launch_sweep_t<R, 1, kSweepThreads, PE>(b, n, lds, threads, s);
  return launch_sweep_t<R, 2, kSweepThreads, PE>(b, n, lds, threads, s);
}

// The brackets of a run of slices, one block each: block b takes slice
// j = jhi - b with costate b - with0 of `lams` (with0: block 0 takes lam0) and
// writes g_j = 2 cr Im(conj(beta) <lambda_j|Hc|psi_j>) (added with
// `accumulate`); slice 0 goes to *g0.
template <typename R>
__global__ void __launch_bounds__(256) k_brackets(BracketRun r, const double* beta, int accumulate) {
  using V = typename VT<R>::T;
  __shared__ double part[2][4];
  const int b = blockIdx.x, j = r.jhi - b;
  const V* lam = reinterpret_cast<const V*>(
      (r.lam0 && b == 0) ? static_cast<const char*>(r.lam0) : r.lams + (size_t)(b - (r.lam0 ? 1 : 0)) * r.states.vb);
  const V* psi = j == 0 ? reinterpret_cast<const V*>(r.psi0) : sweep_out<V>(r.states, 0, j);
  const HvArgs& a = r.states.hv;
  const uint32_t D = r.states.D;
  const uint32_t* reps = r.states.has_pe ? r.states.pe.reps : nullptr;
  const uint32_t flip = (a.hc_kind == 0) ? (1u << a.hc_bit) : 0u;
  double sr = 0.0, si = 0.0;
  for (uint32_t s = threadIdx.x; s < D; s += 256u) {
    const V l = lam[s], p = psi[s ^ flip];
    const uint32_t pat = reps ? reps[s] : s;
    const double hc = (a.hc_kind == 0) ? 0.5 : 0.5 * a.sz_count - (double)__popc(pat & a.sz_mask);
    const double pr = hc * (double)p.x, pi = hc * (double)p.y;
    const double lr = l.x, li = l.y;
    sr += lr * pr + li * pi;
    si += lr * pi - li * pr;
  }
  sr = wave_sum(sr);
  si = wave_sum(si);
  if ((threadIdx.x & 63u) == 0) {
    part[0][threadIdx.x >> 6] = sr;
    part[1][threadIdx.x >> 6] = si;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double Br = ((part[0][0] + part[0][1]) + part[0][2]) + part[0][3];
    const double Bi = ((part[1][0] + part[1][1]) + part[1][2]) + part[1][3];
    const double g = 2.0 * r.cr * (beta[0] * Bi - beta[1] * Br);
    double* out = j == 0 ? r.g0 : r.grad + (j - 1);
    *out = accumulate ? *out + g : g;
  }
}

}  // namespace

hipError_t launch_brackets(int prec, const BracketRun& r, int n, const double* beta, bool accumulate,
                           hipStream_t s) {
  if (n < 1) return hipSuccess;
  if (prec == 0)
    hipLaunchKernelGGL(k_brackets<double>, dim3(n), dim3(256), 0, s, r, beta, accumulate ? 1 : 0);
  else
    hipLaunchKernelGGL(k_brackets<float>, dim3(n), dim3(256), 0, s, r, beta, accumulate ? 1 : 0);
  return hipGetLastError();
}

int sweep_neighbours(const PeArgs* pe, int L) {
  if (!pe) return L - 1;
  const int up = pe->K < pe->L - pe->K ? pe->K : pe->L - pe->K;
  return 2 * up < pe->L - 1 ? 2 * up : pe->L - 1;
}

bool sweep_fits(int prec, uint32_t D, int m, int nbr) {
  if (D < 1 || D > kSweepMaxD || nbr > kSweepNbr) return false;
  const size_t need = prec == 0 ? sweep_lds_bytes<double>(D, m) : sweep_lds_bytes<float>(D, m);
  return need <= kSweepLds;
}

bool passes_forced() {
  const char* tb = getenv("KG_TILE_BITS");
  const char* nf = getenv("KG_NO_FUSED");
  return (tb && *tb) || (nf && *nf && strcmp(nf, "0") != 0);
}

// The one-block form applies when its vectors fit in LDS.
bool sweep_applies(const KrylovCall& c) {
  return sweep_fits(c.prec, c.geo.D, c.m, sweep_neighbours(c.pe, c.hv.L)) && !passes_forced();
}

SweepJob sweep_job(const KrylovCall& c) {
  SweepJob j;
  memset(static_cast<void*>(&j), 0, sizeof(j));
  j.hv = c.hv;
  if (c.pe) j.pe = *c.pe;
  j.has_pe = c.pe ? 1 : 0;
  j.nbr = sweep_neighbours(c.pe, c.hv.L);
  j.D = c.geo.D;
  j.m = c.m;
  j.reorth = c.reorth;
  j.t = c.t;
  j.tol = c.tol;
  j.u = c.hv.u_ptr;
  j.in = c.v_in;
  j.n = 1;
  j.j0 = 1;
  j.dj = 1;
  j.out = static_cast<char*>(c.v_out);
  j.vb = (size_t)c.geo.D * (c.prec == 0 ? 16 : 8);
  j.m_eff_out = c.m_eff_out;
  return j;
}

hipError_t launch_sweeps(int prec, const SweepJob* jobs, int n, hipStream_t s) {
  SweepBatch b;
  memset(static_cast<void*>(&b), 0, sizeof(b));
  for (int at = 0; at < n; at += kSweepJobs) {
    const int cnt = n - at < kSweepJobs ? n - at : kSweepJobs;
    for (int i = 0; i < cnt; ++i) b.job[i] = jobs[at + i];
    const bool pe = b.job[0].has_pe != 0;
    const hipError_t e =
        prec == 0 ? (pe ? launch_sweep_r<double, true>(b, cnt, s) : launch_sweep_r<double, false>(b, cnt, s))
                  : (pe ? launch_sweep_r<float, true>(b, cnt, s) : launch_sweep_r<float, false>(b, cnt, s));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace kg
