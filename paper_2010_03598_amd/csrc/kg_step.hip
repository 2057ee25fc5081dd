// One launch per Lanczos step.
//
// Vectors between those a single block holds and those that fill the chip are
// bound by the latency of a chain of launches, about 7 us each whatever they
// move.  The step as pass A (H v and its dots), then pass B (the update) takes
// two; in the single-pass form of kg_step.h it takes one: the launch of step k
// reads the measurements of step k - 1, derives the coefficients, forms u_k,
// y_k and w'_k and measures.  A Krylov call is m such launches and the
// combination, whose blocks run the last scalars themselves.
//
// A block is NW wavefronts of tile work and one more for the scalars.  Every
// wavefront sums a share of the previous step's rows (one row of values per
// block, read in one round trip beside the tile's loads); the extra wavefront
// turns the totals into coefficients while the others apply H to w'_{k-1},
// which needs none of them.  All blocks compute the same scalars from the same
// sums in the same order; block 0 keeps them for the next launch.
//
// w'_k is rounded before its largest part, c_k u_k, is subtracted, and y_k follows a
// recurrence; both lose |alpha_k| / beta_{k+1}.  In complex64 the rounding's remainder
// is therefore kept beside w'_k (lo: two vectors by the parity of the step) and
// enters u_{k+1}; and past the limit kMaxGrowth all blocks agree, from the same
// scalars, to form y_k = H u_k in that launch, each partner's u_k from w'_{k-1}, lo,
// u_{k-1} and u_{k-2}, which nobody writes meanwhile.  L=12, m=30, S^z field of 100,
// complex64: error 6.5e-8; without it 2.3e-4, two passes 1.8e-7.
//
// A launch is about 6.0 us at L = 13 (two passes: 14.4): the gap between launches, a
// chain of two trips to memory, the scalars (0.8) and the block's sums.  One that forms y
// takes 8 to 9.  Calls at m = 16, complex64, two passes, this form, and this form with y
// formed in every step: L=13 231, 103, 148 us; L=15 232, 118, 166; L=16 234, 138, 192;
// L=17 239, 164, 221; L=18 265, 219, 357; complex128 L=13 230, 102, 133; L=16 239, 145,
// 174; L=18 322, 256, 388.  Strong fields and product states form it in a third of the
// steps.

#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <string.h>

#include "kg_device.h"
#include "kg_internal.h"
#include "kg_step.h"

namespace kg {
namespace {

constexpr int kStepJobs = 2;

// Scalars between launches, in the partials table of the workspace (by the
// parity of the step: a launch reads one copy and writes the other), and the
// final ones of a basis that ended early.
struct StepState {
  LzStore lz[2];
  LzStore fin;
  double run[2][7];       // normT, beta0, sk, rp, gp, g, ig
  double fin_beta0;
  int32_t fin_m_eff;
  int32_t done;
};

struct StepArgs {
  HvArgs hv;
  Geo geo;
  const void* slot0;
  void* basis;            // slots 1..m
  void* y;
  void* lo;               // complex64: w'_k less its stored value, [2][D] by k & 1
  StepState* st;
  cplx_d* rows;           // [2][kStepRows][kStepCols]
  int32_t k, m, reorth;
  int32_t pad_;
  double tol, t;
  void* out;              // combination
  int32_t* m_eff_out;
  PeArgs pe;              // reduced basis: its neighbour table
};

constexpr int kStepFar = 4;               // far partners per round trip
constexpr int kStepRows = 512;            // blocks of a step
constexpr int kStepCols = 2 * kMaxM + 2;  // values of a row, in pairs

struct StepBatch {
  StepArgs job[kStepJobs];
};

template <typename R>
constexpr double kUnit = sizeof(R) == 4 ? 0x1p-24 : 0x1p-53;

template <typename V>
__device__ __forceinline__ V* step_slot(const StepArgs& a, int i) {
  return i == 0 ? reinterpret_cast<V*>(const_cast<void*>(a.slot0))
                : reinterpret_cast<V*>(a.basis) + (size_t)(i - 1) * a.geo.D;
}

__device__ __forceinline__ void get_run(const StepState& st, int b, LzRun& r) {
  r.normT = st.run[b][0];
  r.beta0 = st.run[b][1];
  r.sk = st.run[b][2];
  r.rp = st.run[b][3];
  r.gp = st.run[b][4];
  r.g = st.run[b][5];
  r.ig = st.run[b][6];
}

// The scalars of step k on one wavefront from its totals (LDS: window vector w
// at 2w, 2w + 1, then <u_k|y_k> and (||u_k||^2, ||y_k||^2)).
__device__ bool run_scalars(const StepArgs& a, double unit, int k, const cplx_d* tot, LzLane& s, LzRun& r,
                            StepNext& nx) {
  const int lane = threadIdx.x & 63;
  const int i0 = window_first(k, a.m, a.reorth), nw = k - i0;
  const int w = lane - i0;
  cplx_d A{0.0, 0.0}, G{0.0, 0.0};
  if (w >= 0 && w < nw) {
    A = tot[2 * w];
    G = tot[2 * w + 1];
  }
  const cplx_d akk = tot[2 * nw], x = tot[2 * nw + 1];
  return step_scalars(s, r, k, a.m, a.reorth, a.tol, unit, A, G, akk, x.re, x.im, nx);
}

// The arguments in registers after one wait: read where they are used, each
// cache line of them costs the launch another trip to memory (L=13: 4 us of a call).
__device__ __forceinline__ void hold_args(const StepArgs& a) {
  asm volatile("" ::"s"(a.hv.L), "s"(a.hv.hc_kind), "s"(a.hv.hc_bit), "s"(a.hv.sz_count),
               "s"(a.hv.sz_mask), "s"(a.hv.half_J), "s"(a.hv.c_zz), "s"(a.hv.u_ptr), "s"(a.hv.u_val),
               "s"(a.geo.D), "s"(a.geo.TB), "s"(a.geo.ntiles), "s"(a.slot0), "s"(a.basis), "s"(a.y), "s"(a.lo),
               "s"(a.st), "s"(a.rows), "s"(a.k), "s"(a.m), "s"(a.reorth), "s"(a.tol));
}

// The previous step's rows: wavefront wv of nwv sums a share of them.  A lane
// takes a pair of values (column); short rows go several to a load.  The
// first loads are requested by the constructor and summed by sum(), so that
// the tile's loads go out between the two.
struct RowGather {
  static constexpr uint32_t kFetch = 4;
  const cplx_d* rows;
  uint32_t G, nc, lg, rsub, first, step, col;
  cplx_d v0[kFetch];

  __device__ __forceinline__ void fetch(uint32_t c, uint32_t r0, cplx_d (&v)[kFetch]) const {
#pragma unroll
    for (uint32_t e = 0; e < kFetch; ++e)
      v[e] = rows[min(r0 + e * step, G - 1u) * (uint32_t)kStepCols + min(c, nc - 1u)];
  }
  __device__ __forceinline__ void add(uint32_t r0, const cplx_d (&v)[kFetch], cplx_d& t) const {
#pragma unroll
    for (uint32_t e = 0; e < kFetch; ++e) {
      const bool in = r0 + e * step < G;
      t.re += in ? v[e].re : 0.0;
      t.im += in ? v[e].im : 0.0;
    }
  }
  __device__ __forceinline__ RowGather(const cplx_d* p, uint32_t rows_n, uint32_t cols, uint32_t wv,
                                       uint32_t nwv)
      : rows(p), G(rows_n), nc(cols) {
    const uint32_t lane = threadIdx.x & 63u;
    lg = nc <= 8 ? 3u : (nc <= 16 ? 4u : (nc <= 32 ? 5u : 6u));
    rsub = lane >> lg;
    step = nwv << (6u - lg);
    first = (wv << (6u - lg)) + rsub;
    col = lane & ((1u << lg) - 1u);
    fetch(col, first, v0);
  }
  // totals of this wavefront's rows into part[0, nc)
  __device__ __forceinline__ void sum(cplx_d* part) const {
    cplx_d t{0.0, 0.0};
    add(first, v0, t);
    for (uint32_t r0 = first + kFetch * step; r0 < G + rsub; r0 += kFetch * step) {
      cplx_d v[kFetch];
      fetch(col, r0, v);
      add(r0, v, t);
    }
    if (lg <= 3u) {
      t.re += dpp_f64<0x128>(t.re);   // row_ror:8
      t.im += dpp_f64<0x128>(t.im);
    }
    if (lg <= 4u) {
      t.re += xor_lanes_16(t.re);
      t.im += xor_lanes_16(t.im);
    }
    if (lg <= 5u) {
      t.re += xor_lanes_32(t.re);
      t.im += xor_lanes_32(t.im);
    }
    if (col < nc) part[col] = t;
    for (uint32_t c = col + 64u; c < nc; c += 64u) {   // rows of more than 64 pairs
      cplx_d q{0.0, 0.0};
      for (uint32_t r0 = first; r0 < G; r0 += kFetch * step) {
        cplx_d v[kFetch];
        fetch(c, r0, v);
        add(r0, v, q);
      }
      part[c] = q;
    }
  }
};

// The extra wavefront: the previous step's totals, the coefficients for the
// others, and (in block 0) the scalars for the next launch.
template <typename R, bool FIRST, bool PE>
__device__ __forceinline__ void step_scalar_wave(const StepArgs& a, uint32_t bl, uint32_t G, uint32_t NW,
                                                 cplx_d* part, cplx_d* tot, cplx_d* cf, StepNext* nxs,
                                                 int* gos) {
  const uint32_t lane = threadIdx.x & 63u;
  const int k = a.k;
  StepState& ss = *a.st;
  if constexpr (FIRST) {
    cf[lane] = cplx_d{0.0, 0.0};
    if (lane < 8u) cf[64 + lane] = cplx_d{0.0, 0.0};
    if (lane == 0) {
      *nxs = StepNext{cplx_d{0.0, 0.0}, 1.0, 1.0, cplx_d{0.0, 0.0}, 0.0};
      *gos = 1;
    }
    __syncthreads();
    __syncthreads();
    if (bl == 0 && lane == 0) ss.done = 0;
    __syncthreads();
    return;
  }
  LzLane s;
  LzRun r;
  const int ip = window_first(k - 1, a.m, a.reorth);
  const uint32_t nc = 2u * (uint32_t)(k - 1 - ip) + 2u;
  RowGather rg(a.rows + (size_t)((k - 1) & 1) * kStepRows * kStepCols, G, nc, NW, NW + 1u);
  const int done = ss.done;
  get_lane(ss.lz[(k - 1) & 1], s);
  get_run(ss, (k - 1) & 1, r);
  rg.sum(part + NW * kStepCols);
  if (k == 1) {   // nothing kept yet
    s = LzLane();
    r = LzRun();
  }
  __syncthreads();
  for (uint32_t col = lane; col < nc; col += 64u) {
    double re = 0.0, im = 0.0;
    for (uint32_t w0 = 0; w0 <= NW; w0 += 5) {
      cplx_d v[5];
#pragma unroll
      for (uint32_t e = 0; e < 5; ++e) v[e] = part[min(w0 + e, NW) * kStepCols + col];
#pragma unroll
      for (uint32_t e = 0; e < 5; ++e) {
        re += w0 + e <= NW ? v[e].re : 0.0;
        im += w0 + e <= NW ? v[e].im : 0.0;
      }
    }
    tot[col] = cplx_d{re, im};
  }
  wave_lds_fence();
  StepNext nx{cplx_d{0.0, 0.0}, 1.0, 1.0, cplx_d{0.0, 0.0}, 0.0};
  const bool go = done == 0 && run_scalars(a, kUnit<R>, k - 1, tot, s, r, nx);
  cf[lane] = s.cw;
  if (lane < 8u) cf[64 + lane] = cplx_d{0.0, 0.0};
  if (lane == 0) {
    *nxs = nx;
    *gos = go ? 1 : 0;
  }
  // the others go on; then the scalars are kept for the next launch
  __syncthreads();
  if (bl == 0) {
    if (go) {
      put_lane(ss.lz[k & 1], s);
      if (lane == 0) {
        const double v[7] = {r.normT, r.beta0, r.sk, r.rp, r.gp, r.g, r.ig};
#pragma unroll
        for (int e = 0; e < 7; ++e) ss.run[k & 1][e] = v[e];
      }
    } else if (done == 0) {
      put_lane(ss.fin, s);
      if (lane == 0) {
        ss.fin_beta0 = r.beta0;
        ss.fin_m_eff = r.m_eff;
        ss.done = 1;
      }
    }
  }
  if (go) {
    if (!PE && nx.fresh != 0.0) __syncthreads();   // the fresh tile's
    __syncthreads();
  }
}

__device__ __forceinline__ void hold_pe_args(const PeArgs& p) {
  asm volatile("" ::"s"(p.reps), "s"(p.scnt), "s"(p.nbr), "s"(p.nbr_slots), "s"(p.L), "s"(p.dim));
}

// u_k at one amplitude from w'_{k-1} (x, and lo in complex64) and u_{k-1} (p), rounded
// as stored.
template <typename V>
__device__ __forceinline__ V next_u(const StepNext& nx, V x, V lo, V p) {
  using R = decltype(x.x);
  double xr = x.x, xi = x.y;
  if constexpr (sizeof(R) == 4) {
    xr += (double)lo.x;
    xi += (double)lo.y;
  }
  const double ar = nx.sig * xr, ai = nx.sig * xi;
  return V{(R)(ar - (nx.c.re * (double)p.x - nx.c.im * (double)p.y)),
           (R)(ai - (nx.c.re * (double)p.y + nx.c.im * (double)p.x))};
}

// The same with the remainder d on u_{k-2} (p2).  Written with fma, so that every place
// forms the same value.
template <typename V>
__device__ __forceinline__ V next_u(const StepNext& nx, V x, V lo, V p, V p2) {
  using R = decltype(x.x);
  double ar = nx.sig * ((double)x.x + (double)lo.x), ai = nx.sig * ((double)x.y + (double)lo.y);
  ar = fma(nx.c.im, (double)p.y, fma(-nx.c.re, (double)p.x, ar));
  ai = fma(-nx.c.im, (double)p.x, fma(-nx.c.re, (double)p.y, ai));
  ar = fma(nx.d.im, (double)p2.y, fma(-nx.d.re, (double)p2.x, ar));
  ai = fma(-nx.d.im, (double)p2.x, fma(-nx.d.re, (double)p2.y, ai));
  return V{(R)ar, (R)ai};
}

// RAG: the last tile reaches past the vector.  FIRST: step 0.  PE: the reduced
// basis, H v gathered through its neighbour table (a wavefront's unit of 64
// rows is a slice of the table).  One tile per block.
template <typename R, int RB, bool RAG, bool FIRST, bool PE>
__device__ __forceinline__ void step_body(const StepArgs a, uint32_t bl, uint32_t G) {
  using V = typename VT<R>::T;
  constexpr int NR = 1 << RB;
  hold_args(a);
  if constexpr (PE) hold_pe_args(a.pe);
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ cplx_d cf[kMaxM + 8];
  __shared__ cplx_d tot[kStepCols];
  __shared__ StepNext nxs;
  __shared__ int gos;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wv = uniform_u32(threadIdx.x >> 6);
  Geo g = a.geo;
  // a full-space tile is never longer than the vector; known here, hv_tile's loads
  // have no masked alternative to wait for
  if constexpr (!RAG) g.small = 0;
  const uint32_t NW = 1u << g.WB;
  const uint32_t c = lane & 3u, aa = lane >> 2;
  const uint32_t D = g.D;
  const int k = FIRST ? 0 : a.k, m = a.m;
  const bool last = k == m - 1;
  const int i0 = window_first(k, m, a.reorth), nw = k - i0;
  const uint32_t nv = 4u * (uint32_t)nw + 4u;                   // values of this step's row
  V* lds = reinterpret_cast<V*>(smem_raw);
  R* stage = reinterpret_cast<R*>(smem_raw + ((size_t)sizeof(V) << g.TB));
  double* meas = reinterpret_cast<double*>(stage + NW * 256u);
  cplx_d* part = reinterpret_cast<cplx_d*>(meas + NW * nv);
  if (wv == NW) {
    step_scalar_wave<R, FIRST, PE>(a, bl, G, NW, part, tot, cf, &nxs, &gos);
    return;
  }
  const int ip = window_first(FIRST ? 0 : k - 1, m, a.reorth);
  const V* src = FIRST ? step_slot<const V>(a, 0) : step_slot<const V>(a, k + 1);
  V* yb = reinterpret_cast<V*>(a.y);
  constexpr bool kLo = sizeof(R) == 4;   // w'_0 = y_0 has no remainder
  const V* lo_in = reinterpret_cast<const V*>(a.lo) + (size_t)((k - 1) & 1) * D;
  V* lo_out = reinterpret_cast<V*>(a.lo) + (size_t)(k & 1) * D;
  const uint32_t tile = tile_of(g, 0, bl, G);
  const uint32_t base = tile << g.TB;
  const uint32_t sw = base | (wv << (6 + RB));                  // this wavefront's amplitudes
  Tile<R, RB> T;
  V up[NR], yp[NR], lo[NR];
  V w0q[2][4];   // the first window vectors of the first unit, in flight beside the scalars
  const auto load = [&](uint32_t s0, int w, V (&q)[4]) {
    const V* p = step_slot<const V>(a, min(i0 + w, k - 1));
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const uint32_t s = s0 | unit_amp(t, aa);
      q[t] = RAG ? ld_masked(p, s, s < D) : p[s];
    }
  };
  const double u = control_value(a.hv);
  const auto window_first_loads = [&] {
    if (nw > 0) {
      load(sw, (int)c, w0q[0]);
      load(sw, (int)c + 4, w0q[1]);
    }
  };
  // H v, with one barrier of the block on the way
  const auto apply_h = [&](auto before) {
    if constexpr (PE) {
      const uint32_t ns = (D + 63u) >> 6;
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const uint32_t sl = min((sw >> 6) + r, ns - 1u), b = min((sl << 6) | lane, D - 1u);
        bool bad;
        pe_row_nbr<R>(a.hv, a.pe, u, sl, b, lane, [&](uint32_t i) { return src[i]; }, T.yr[r], T.yi[r],
                      bad);
        const V x = src[b];
        T.xr[r] = x.x;
        T.xi[r] = x.y;
        if (bad) T.yr[r] = T.yi[r] = (R)NAN;
      }
      before();
      __syncthreads();
    } else {
      hv_tile<R, RB, false, kStepFar>(T, a.hv, g, tile, src, lds, u, before);
    }
  };
  if constexpr (FIRST) {
    apply_h(NoWork());
  } else {
    RowGather rg(a.rows + (size_t)((k - 1) & 1) * kStepRows * kStepCols, G,
                 2u * (uint32_t)(k - 1 - ip) + 2u, wv, NW + 1u);
    load_slots<V, NR>(step_slot<const V>(a, k - 1), sw | lane, !RAG, D, up);
    load_slots<V, NR>(yb, sw | lane, !RAG, D, yp);
    if constexpr (kLo) load_slots<V, NR>(lo_in, sw | lane, !RAG, D, lo);   // not used at k = 1
    apply_h([&] {
      window_first_loads();
      rg.sum(part + wv * kStepCols);
    });
  }
  __syncthreads();
  const int go = gos;
  const StepNext nx = nxs;   // both in one trip to LDS
  if (!go) return;
  V* uk = FIRST ? nullptr : step_slot<V>(a, k);
  V* wk = last ? nullptr : step_slot<V>(a, k + 2);
  R* st = stage + wv * 256u;
  double* row = meas + wv * nv;
  double kr = 0.0, ki = 0.0, kk = 0.0, yy = 0.0;
  const bool fresh = !FIRST && uniform_u32((uint32_t)(nx.fresh != 0.0));
  if (__builtin_expect(!FIRST && fresh, 0)) {   // out of the ordinary path's way
    const V* pu = step_slot<const V>(a, k - 1);
    const V* pu2 = step_slot<const V>(a, max(k - 2, 0));   // k = 1: d is 0
    const auto u_at = [&](uint32_t i) {
      return next_u<V>(nx, src[i], (kLo && k >= 2) ? lo_in[i] : V{(R)0, (R)0}, pu[i], pu2[i]);
    };
    if constexpr (PE) {
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const uint32_t sl = min((sw >> 6) + r, ((D + 63u) >> 6) - 1u), b = min((sl << 6) | lane, D - 1u);
        bool bad;
        pe_row_nbr<R>(a.hv, a.pe, u, sl, b, lane, u_at, T.yr[r], T.yi[r], bad);
        if (bad) T.yr[r] = T.yi[r] = (R)NAN;
        const V x = u_at(b);
        T.xr[r] = x.x;
        T.xi[r] = x.y;
      }
    } else {
      // the tile in LDS has served its turn; the scalar wavefront joins the barrier
      hv_tile_of<R, RB, false, kStepFar>(T, a.hv, g, tile, u_at, lds, u, NoWork());
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const uint32_t s0 = sw | ((uint32_t)r << 6), sl = s0 | lane;
    const bool in = !RAG || sl < D;
    // u_k and y_k, rounded as stored
    V uo, yo;
    if constexpr (FIRST) {
      uo = V{T.xr[r], T.xi[r]};
      yo = V{T.yr[r], T.yi[r]};
    } else {
      uo = next_u<V>(nx, V{T.xr[r], T.xi[r]}, (kLo && k >= 2) ? lo[r] : V{(R)0, (R)0}, up[r]);
      yo.x = (R)(nx.sig * (double)T.yr[r] - (nx.c.re * (double)yp[r].x - nx.c.im * (double)yp[r].y));
      yo.y = (R)(nx.sig * (double)T.yi[r] - (nx.c.re * (double)yp[r].y + nx.c.im * (double)yp[r].x));
      if (fresh) {   // both formed above
        uo = V{T.xr[r], T.xi[r]};
        yo = V{T.yr[r], T.yi[r]};
      }
      if (in) uk[sl] = uo;
    }
    if (RAG && !in) uo = yo = V{(R)0, (R)0};
    {
      const double xr = uo.x, xi = uo.y, yr = yo.x, yi = yo.y;
      kr += xr * yr + xi * yi;
      ki += xr * yi - xi * yr;
      kk += xr * xr + xi * xi;
      yy += yr * yr + yi * yi;
    }
    if (last) continue;
    if (in) yb[sl] = yo;
    if (FIRST || nw == 0) {
      if (in) wk[sl] = V{(R)(nx.s * (double)yo.x), (R)(nx.s * (double)yo.y)};
      continue;
    }
    // ---- the window
    if constexpr (sizeof(R) == 4) {
      reinterpret_cast<float4*>(st)[lane] = float4{yo.x, yo.y, uo.x, uo.y};
    } else {
      reinterpret_cast<double2*>(st)[2 * lane] = double2{yo.x, yo.y};
      reinterpret_cast<double2*>(st)[2 * lane + 1] = double2{uo.x, uo.y};
    }
    wave_lds_fence();
    double b[4], bp[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      b[t] = (double)st[unit_amp(t, aa) * 4u + c];
      bp[t] = turned(b[t]);
    }
    double zr[4] = {0.0, 0.0, 0.0, 0.0}, zi[4] = {0.0, 0.0, 0.0, 0.0};
    // two groups of four vectors; the next ones are requested before these are used
    V q[2][4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      q[0][t] = w0q[0][t];
      q[1][t] = w0q[1][t];
    }
    if (r > 0) {
      load(s0, (int)c, q[0]);
      load(s0, (int)c + 4, q[1]);
    }
    for (int w0 = 0; w0 < nw; w0 += 8) {
      const bool two = w0 + 4 < nw, more = w0 + 8 < nw;
      V n[2][4];
      if (more) {
        load(s0, w0 + 8 + (int)c, n[0]);
        load(s0, w0 + 12 + (int)c, n[1]);
      }
      double e0 = 0.0, e1 = 0.0, f0 = 0.0, f1 = 0.0;
      unit_rows(q[0], b, bp, cf[i0 + w0 + (int)c], zr, zi, e0, e1);
      if (two) unit_rows(q[1], b, bp, cf[i0 + w0 + 4 + (int)c], zr, zi, f0, f1);
      const auto put = [&](int w, double d0, double d1) {
        const double e = unit_dots(d0, d1);
        if ((lane & 12u) == 0u && w < nw) {
          double& d = row[4 * w + (int)c];
          d = r == 0 ? e : d + e;
        }
      };
      put(w0 + (int)(lane >> 4), e0, e1);
      if (two) put(w0 + 4 + (int)(lane >> 4), f0, f1);
      if (more) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          q[0][t] = n[0][t];
          q[1][t] = n[1][t];
        }
      }
    }
    {
      const uint32_t s = s0 | unit_amp((int)c, aa);
      const R* o = st + unit_amp((int)c, aa) * 4u;
      const double wr = nx.s * (double)o[0] - quad_z(zr), wi = nx.s * (double)o[1] - quad_z(zi);
      const V w{(R)wr, (R)wi};
      if (!RAG || s < D) {
        wk[s] = w;
        if (kLo) lo_out[s] = V{(R)(wr - (double)w.x), (R)(wi - (double)w.y)};
      }
    }
    wave_lds_fence();
  }
  // ---- this block's row of measurements
  const double e4 = quad_sums_swap(kr, ki, kk, yy);
  if (lane < 4u) row[4 * nw + (int)lane] = e4;
  __syncthreads();
  double* dst = reinterpret_cast<double*>(a.rows + ((size_t)(k & 1) * kStepRows + bl) * kStepCols);
  for (uint32_t v = threadIdx.x; v < nv; v += NW * 64u) {
    double e = 0.0;
    for (uint32_t w0 = 0; w0 < NW; w0 += 4) {
      double x[4];
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) x[q] = meas[min(w0 + q, NW - 1u) * nv + v];
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) e += w0 + q < NW ? x[q] : 0.0;
    }
    dst[v] = e;
  }
}

// Blocks of up to four wavefronts of tile work (TH 320) get the registers of
// two wavefronts per SIMD.
template <typename R, int RB, bool RAG, int TH, bool FIRST, bool PE = false>
__global__ void __launch_bounds__(TH) k_step(StepBatch B) {
  const uint32_t G = B.job[0].geo.grid;
  const uint32_t j = blockIdx.x < G ? 0u : 1u;
  step_body<R, RB, RAG, FIRST, PE>(B.job[j], blockIdx.x - j * G, G);
}

constexpr int kCombBlock = 256;

// v_out = sum_j d_j u_j (FP64 accumulation).  Every block first runs the last
// step's scalars and the small exponential on wavefront 0 (a basis that ended
// early has its own); four vectors per round trip after that.
template <typename R>
__global__ void __launch_bounds__(kCombBlock) k_step_combine(StepBatch B, uint32_t grid) {
  using V = typename VT<R>::T;
  __shared__ cplx_d tot[2];
  __shared__ cplx_d cs[kMaxM];
  __shared__ int mes;
  const uint32_t j = blockIdx.x < grid ? 0u : 1u;
  const StepArgs& a = B.job[j];
  const uint32_t bl = blockIdx.x - j * grid, lane = threadIdx.x & 63u;
  if (threadIdx.x < 64) {
    const StepState& ss = *a.st;
    const int k = a.m - 1;
    LzLane s;
    LzRun r;
    const int done = k > 0 ? ss.done : 0;
    if (k > 0) {
      get_lane(ss.lz[k & 1], s);
      get_run(ss, k & 1, r);
    }
    double e[4] = {0.0, 0.0, 0.0, 0.0};
    const uint32_t G = a.geo.grid;
    for (uint32_t q = lane; q < G; q += 64) {
      const cplx_d* p = a.rows + ((size_t)(k & 1) * kStepRows + q) * kStepCols;
      const cplx_d x = p[0], y = p[1];
      e[0] += x.re;
      e[1] += x.im;
      e[2] += y.re;
      e[3] += y.im;
    }
    if (done == 0) {
      const cplx_d t0{wave_sum(e[0]), wave_sum(e[1])}, t1{wave_sum(e[2]), 0.0};
      if (lane == 0) {
        tot[0] = t0;
        tot[1] = t1;
      }
      wave_lds_fence();
      StepNext nx;
      (void)run_scalars(a, kUnit<R>, k, tot, s, r, nx);
    } else {
      get_lane(ss.fin, s);
      r.beta0 = ss.fin_beta0;
      r.m_eff = ss.fin_m_eff;
    }
    cs[lane] = comb_coef(s, r, a.t);
    if (lane == 0) {
      mes = r.m_eff;
      if (bl == 0 && a.m_eff_out) *a.m_eff_out = r.m_eff;
    }
  }
  __syncthreads();
  const int me = mes;
  const uint32_t D = a.geo.D, stride = grid * kCombBlock;
  V* out = reinterpret_cast<V*>(a.out);
  for (uint32_t s0 = bl * kCombBlock + threadIdx.x; s0 < D; s0 += stride) {
    double ar = 0.0, ai = 0.0;
    for (int i0 = 0; i0 < me; i0 += 8) {
      V v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = step_slot<const V>(a, min(i0 + e, me - 1))[s0];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (i0 + e < me) {
          const cplx_d d = cs[i0 + e];
          const double vr = v[e].x, vi = v[e].y;
          ar += d.re * vr - d.im * vi;
          ai += d.re * vi + d.im * vr;
        }
      }
    }
    out[s0] = V{(R)ar, (R)ai};
  }
}

// The most dynamic LDS of a launch: 68 KB at 2^10 tiles, complex128, m = 64.
constexpr size_t kStepLds = 80u << 10;

template <typename R, int RB, bool RAG, int TH, bool PE>
hipError_t launch_step_t(const StepBatch& b, int n, size_t lds, hipStream_t s) {
  const Geo& g = b.job[0].geo;
  const dim3 grid(g.grid * n), block(64u * ((1u << g.WB) + 1u));
  static std::atomic<uint64_t> raised[2];
  const int later = b.job[0].k == 0 ? 0 : 1;
  const auto kernel = later ? k_step<R, RB, RAG, TH, false, PE> : k_step<R, RB, RAG, TH, true, PE>;
  const hipError_t e = allow_lds(kernel, lds, kStepLds, raised[later]);
  if (e != hipSuccess) return e;
  kg_launch(kernel, grid, block, lds, s, b);
  return hipGetLastError();
}

template <typename R, int RB>
hipError_t launch_step_rb(const StepBatch& b, int n, size_t lds, hipStream_t s) {
  const Geo& g = b.job[0].geo;
  if (b.job[0].pe.nbr)
    return g.WB <= 2 ? launch_step_t<R, RB, true, 320, true>(b, n, lds, s)
                     : launch_step_t<R, RB, true, 576, true>(b, n, lds, s);
  return g.WB <= 2 ? launch_step_t<R, RB, false, 320, false>(b, n, lds, s)
                   : launch_step_t<R, RB, false, 576, false>(b, n, lds, s);
}

template <typename R>
size_t step_lds(const Geo& g, int k, int m, int reorth) {
  using V = typename VT<R>::T;
  const size_t NW = (size_t)1 << g.WB;
  const int i0 = k == m - 1 ? k : (reorth ? 0 : (k > 0 ? k - 1 : 0));
  const size_t nv = (size_t)(4 * (k - i0) + 4);
  return (sizeof(V) << g.TB) + NW * 256 * sizeof(R) + NW * nv * sizeof(double) +
         (NW + 1) * kStepCols * sizeof(cplx_d);
}

template <typename R>
hipError_t launch_krylov_steps_r(const KrylovCall* calls, const Workspace* const* wss, int n,
                                 hipStream_t s) {
  StepBatch b;
  memset(static_cast<void*>(&b), 0, sizeof(b));
  for (int j = 0; j < n; ++j) {
    const KrylovCall& c = calls[j];
    StepArgs& a = b.job[j];
    a.hv = c.hv;
    a.geo = c.step;
    a.slot0 = c.v_in;
    a.basis = wss[j]->basis;
    a.y = wss[j]->yk;
    a.lo = static_cast<char*>(wss[j]->basis) + (size_t)c.m * c.step.D * sizeof(typename VT<R>::T);
    a.rows = wss[j]->partials;
    a.st = reinterpret_cast<StepState*>(wss[j]->partials + 2 * (size_t)kStepRows * kStepCols);
    a.m = c.m;
    a.reorth = c.reorth;
    a.tol = c.tol;
    a.t = c.t;
    a.out = c.v_out;
    a.m_eff_out = c.m_eff_out;
    if (c.pe) a.pe = *c.pe;
  }
  const Geo& g = b.job[0].geo;
  hipError_t e = hipSuccess;
  Profiler* prof = profiler_for_call();
  const int m = calls[0].m;
  const double vb = (double)g.D * sizeof(typename VT<R>::T) * n;
  for (int k = 0; k < m; ++k) {
    for (int j = 0; j < n; ++j) b.job[j].k = k;
    if (prof) profiler_start(prof, s);
    const size_t lds = step_lds<R>(g, k, calls[0].m, calls[0].reorth);
    e = g.RB == 0 ? launch_step_rb<R, 0>(b, n, lds, s) : launch_step_rb<R, 1>(b, n, lds, s);
    if (e != hipSuccess) return e;
    // as a pass A (v_k read, y written but in the last step) and, before the
    // last step, a pass B (y and the window read, v_{k+1} written); lo is not counted
    const int i0 = k == m - 1 ? k : (calls[0].reorth ? 0 : (k > 0 ? k - 1 : 0));
    if (prof && calls[0].pe)
      profiler_stop(prof, s, kProfHv, n * pe_gather_bytes(*calls[0].pe, vb / n), kProfPassB,
                    (k < m - 1 ? k - i0 + 3 : 1) * vb);
    else if (prof && k < m - 1)
      profiler_stop(prof, s, kProfPassA, 2 * vb, kProfPassB, (k - i0 + 3) * vb);
    else if (prof)
      profiler_stop(prof, s, kProfPassA, vb);
  }
  uint32_t grid = (g.D + kCombBlock - 1) / kCombBlock;
  if (grid > 1024u) grid = 1024u;
  if (prof) profiler_start(prof, s);
  kg_launch(k_step_combine<R>, dim3(grid * n), dim3(kCombBlock), 0, s, b, grid);
  e = hipGetLastError();
  if (prof) profiler_stop(prof, s, kProfCombine, (m + 1) * vb);
  return e;
}

}  // namespace

static_assert(2 * kStepRows * kStepCols + (sizeof(StepState) + sizeof(cplx_d) - 1) / sizeof(cplx_d) <=
                  (size_t)kPartialRows * kMaxScal,
              "the rows and the scalars fit in the partials table");

size_t step_table_pairs() {
  return 2 * (size_t)kStepRows * kStepCols + (sizeof(StepState) + sizeof(cplx_d) - 1) / sizeof(cplx_d);
}

hipError_t launch_krylov_steps(const KrylovCall* calls, const Workspace* const* wss, int n,
                               hipStream_t s) {
  return calls[0].prec == 0 ? launch_krylov_steps_r<double>(calls, wss, n, s)
                            : launch_krylov_steps_r<float>(calls, wss, n, s);
}

}  // namespace kg
