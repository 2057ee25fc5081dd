// HIP kernels of the K-GRAPE hot path for gfx950 (MI355X).
//
// Memory-bound throughout, so without MFMA (only the forms of short vectors take
// their dots on the matrix cores, kg_step.h): every kernel streams state
// vectors through HBM (or the Infinity Cache) once per pass and keeps the arithmetic in
// registers.  Layout: a state vector is D = 2^L interleaved complex amplitudes.
//
// H v (Sec. III.A, Eqs. 6 and 10).  A block stages a tile of 2^TB consecutive
// amplitudes in LDS.  Inside the tile, amplitude index bits are assigned as
//   bits 0..5           lane of the wavefront,
//   bits 6..6+RB-1      register slot r of the thread (2^RB amplitudes per thread),
//   bits 6+RB..TB-1     wavefront of the block,
// so global loads are fully coalesced (a wavefront reads 64 consecutive
// amplitudes per slot).  The hopping term of bond p couples s and s^(3<<p)
// when bits p and p+1 of s differ.  Bonds between two register bits are
// resolved in registers with compile-time predicates; bonds inside the tile
// read the partner from LDS; bonds reaching bit TB or above read the partner
// tile from global memory (L2/Infinity Cache), with a predicate that is
// uniform across the wavefront, so the loads stay coalesced and inactive bonds
// cost one scalar branch.  The diagonal S^z S^z term is one popcount.
//
// Lanczos (App. A, Algorithm 2 with the full re-orthonormalisation it
// describes).  Vectors of more than 2^18 amplitudes (shorter ones take a launch
// per step or a block per call, kg_step.hip and kg_sweep.hip; these passes serve
// them too when KG_TILE_BITS forces a tile size or KG_NO_FUSED is set).  With full re-orthonormalisation two
// steps share one pass over the basis (pass C and pass P, described there); the
// plain two-vector window takes two passes a step:
//   pass A(k): x = stored v_k; y = H x, stored (the H v vector); each block
//              writes its parts of <x|y> and ||x||^2 and ends (no grid-wide
//              reduction); helper wavefronts sum the earlier pass's
//              measurement columns over the grid;
//   pass B(k): every block first runs the scalar update of step k on the same
//              sums (breakdown test, window dots, projection coefficients),
//              then w = s_k y - sum_i c_i v_i is stored unnormalised as
//              v_{k+1}, with the blocks' parts of ||w||^2 and of the dots the
//              next step derives its window dots from; a streaming pass over y
//              and the window.
// The scalar update costs each block of a streaming pass one memory round trip and a few
// hundred FP64 instructions on one wavefront, instead of a serial tail in
// which the last block of pass A waits for every partial and then computes
// alone.  Storing y costs one vector write and read; recomputing it in pass B
// would repeat the partner-tile reads of the far hopping bonds, which cost
// more.  Stored vectors are not rescaled: scale_k = 1/||stored_k|| lives in
// device memory and is folded into the coefficients.  Every sum is
// deterministic in FP64 (fixed order, no floating-point atomics).  After the
// last pass A, one wavefront runs the last step's update and evaluates
// exp(-itT) e_1 in FP64, and a streaming pass forms
// v_out = beta0 V^T exp(-itT) e_1 with FP64 accumulation.
//
// Blocks of the tiled kernels are mapped to tiles XCD by XCD: block b runs on
// XCD b%8, and the tiles of one XCD form one contiguous range, so partner tiles
// of the lower hopping bonds are read from the same L2.

#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>
#include <string.h>
#include <stdlib.h>

#include <atomic>

#include "kg_device.h"
#include "kg_internal.h"

namespace kg {

namespace {

// ---------------------------------------------------------------------- xxz_apply

// Store y of a pair-layout tile (hv_tile_pairs): 16 bytes per pair.
template <int RB>
__device__ __forceinline__ void store_pairs(const Tile<float, RB>& T, float2* out, uint32_t base) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wb = uniform_u32(threadIdx.x >> 6) << (6 + RB);
#pragma unroll
  for (int q = 0; q < (1 << RB) / 2; ++q) {
    const uint32_t e = (lane << 1) | ((uint32_t)q << 7) | wb;
    reinterpret_cast<float4*>(out)[(base | e) >> 1] =
        float4{T.yr[2 * q], T.yi[2 * q], T.yr[2 * q + 1], T.yi[2 * q + 1]};
  }
}

// kPairs: complex64 in the pair layout (hv_tile_pairs), 16-byte accesses.
template <typename R, int RB, bool kPairs = false>
__global__ void __launch_bounds__((RB >= 3 && sizeof(R) == 8) ? 512 : 1024) k_hv(HvArgs a, Geo g, const typename VT<R>::T* __restrict__ v,
                                            typename VT<R>::T* __restrict__ w) {
  using V = typename VT<R>::T;
  extern __shared__ unsigned char smem_raw[];
  V* lds = reinterpret_cast<V*>(smem_raw);
  const double u = control_value(a);
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wv = uniform_u32(threadIdx.x >> 6);
  const uint32_t eb = lane | (wv << (6 + RB));
  const uint32_t iters = g.ntiles / gridDim.x;
  Tile<R, RB> T;
  for (uint32_t it = 0; it < iters; ++it) {
    const uint32_t tile = tile_of(g, it, blockIdx.x, gridDim.x);
    if (it) __syncthreads();
    const uint32_t base = tile << g.TB;
    if constexpr (kPairs) {
      hv_tile_pairs<RB>(T, a, g, tile, v, lds, u);
      store_pairs<RB>(T, w, base);
      continue;
    }
    hv_tile<R, RB>(T, a, g, tile, v, lds, u);
#pragma unroll
    for (int r = 0; r < (1 << RB); ++r) {
      const uint32_t s = base | eb | ((uint32_t)r << 6);
      if (!g.small || s < g.D) {
        V o;
        o.x = T.yr[r];
        o.y = T.yi[r];
        w[s] = o;
      }
    }
  }
}

// ---------------------------------------------------------------------- H v, reduced basis

// y = (H0 + u Hc) x in the fixed-excitation, parity-even basis (Sec. III.A),
// one output amplitude per thread.  With r the orbit label of output b and
// n = 1 or 2 the orbit sizes,
//   y_b = d(r) x_b + (J/2) sum_{antiparallel bonds p of r} sqrt(n_b / n_a) x_a,
// a the orbit of r with bits p, p+1 exchanged.  a is found through the
// combinatorial rank of the sector state over its zero bits (up spins):
// rank(s) = sum_i C(z_i, i) for zero positions z_1 < z_2 < ...; exchanging a
// zero at p with a one at p+1 (or back) changes the rank by C(p, j) with j the
// zeros below p.  The S^z control is diagonal; the amplitudes x_a are gathered.
//
// The gathers are latency-bound (index, then amplitude, per bond), so the
// bonds of a row go kPeHops at a time: their ranks first, then all index
// loads, then all amplitude loads, each group in flight together.  Slots past
// a row's last bond load the row's own entries (cached) with weight 0.  The
// binomial table is staged in LDS; the label's own rank comes from the tables.
constexpr int kPeHops = 8;

// One output of the reduced-basis H v: row b, with the binomials in LDS (sb)
// and xat(i) the amplitude of orbit i.  Sets `bad` when a table entry is out
// of range (the output is then NaN, never a stray load).
template <typename R, typename XAt>
__device__ __forceinline__ void pe_row(const HvArgs& a, const PeArgs& p, const uint32_t* sb, double u,
                                       uint32_t b, XAt xat, R& yr, R& yi, bool& bad) {
  using V = typename VT<R>::T;
  const int L = p.L;
  const uint32_t full = (L == 32) ? 0xFFFFFFFFu : ((1u << L) - 1u);
  const uint32_t bondmask = (L >= 2) ? ((1u << (L - 1)) - 1u) : 0u;
  const R hJ = (R)a.half_J, czz = (R)a.c_zz, uR = (R)u;
  const R rt2 = (R)1.4142135623730951, irt2 = (R)0.70710678118654752;
  const uint32_t r = p.reps[b];
  const uint32_t rank = p.ranks[b];
  const uint32_t zeros = ~r & full;
  const bool nb2 = (__brev(r) >> (32 - L)) != r;
  const int n_anti = (int)__popc((r ^ (r >> 1)) & bondmask);   // __popc is unsigned
  R d = czz * (R)(L - 1 - 2 * n_anti);
  if (a.hc_kind == 1) d += uR * ((R)(0.5 * a.sz_count) - (R)__popc(r & a.sz_mask));
  const V xb = xat(b);
  yr = d * xb.x;
  yi = d * xb.y;
  bad = rank >= p.nsec;
  uint32_t act = bad ? 0u : ((r ^ (r >> 1)) & bondmask);
  while (act) {
    uint32_t rk[kPeHops];
    R w[kPeHops];
#pragma unroll
    for (int j = 0; j < kPeHops; ++j) {
      const bool on = act != 0u;
      const int q = on ? __builtin_ctz(act) : 0;
      act &= act - 1u;
      const uint32_t dl = sb[q * kPeBinom + __popc(zeros & ((1u << q) - 1u))];
      const uint32_t s2 = r ^ (3u << q);
      const bool na2 = (__brev(s2) >> (32 - L)) != s2;
      rk[j] = on ? ((((r >> q) & 1u) == 0u) ? rank + dl : rank - dl) : rank;
      w[j] = on ? ((nb2 == na2) ? (R)1 : (nb2 ? rt2 : irt2)) : (R)0;
    }
    int32_t ai[kPeHops];
#pragma unroll
    for (int j = 0; j < kPeHops; ++j) ai[j] = (rk[j] < p.nsec) ? p.index[rk[j]] : -1;
#pragma unroll
    for (int j = 0; j < kPeHops; ++j) {
      const bool ok = (uint32_t)ai[j] < p.dim;
      bad = bad || !ok;
      const V xa = xat(ok ? (uint32_t)ai[j] : b);
      yr += hJ * w[j] * xa.x;
      yi += hJ * w[j] * xa.y;
    }
  }
}

template <typename R>
__global__ void __launch_bounds__(256) k_hv_pe(HvArgs a, PeArgs p,
                                               const typename VT<R>::T* __restrict__ x,
                                               typename VT<R>::T* __restrict__ y) {
  using V = typename VT<R>::T;
  __shared__ uint32_t sb[kPeBinom * kPeBinom];
  for (int i = threadIdx.x; i < kPeBinom * kPeBinom; i += blockDim.x) sb[i] = p.binom[i];
  __syncthreads();
  const double u = control_value(a);
  uint32_t lo = 0, hi = p.dim, b0 = blockIdx.x * blockDim.x + threadIdx.x,
           stride = gridDim.x * blockDim.x;
  if ((gridDim.x & 7u) == 0u) {
    // contiguous rows per XCD (blocks are dealt to the 8 XCDs round robin)
    const uint32_t chunk = (p.dim + 7u) >> 3;
    lo = (blockIdx.x & 7u) * chunk;
    hi = min(lo + chunk, p.dim);
    b0 = lo + (blockIdx.x >> 3) * blockDim.x + threadIdx.x;
    stride = (gridDim.x >> 3) * blockDim.x;
  }
  for (uint32_t b = b0; b < hi; b += stride) {
    R yr, yi;
    bool bad;
    pe_row<R>(a, p, sb, u, b, [&](uint32_t i) { return x[i]; }, yr, yi, bad);
    V o;
    o.x = bad ? (R)NAN : yr;
    o.y = bad ? (R)NAN : yi;
    y[b] = o;
  }
}

// The same H v from the neighbour table built with the basis: a wavefront takes
// the 64 rows of a slice, reads the slice's slot count (one scalar load), then
// its rows' entries slot by slot (256 contiguous bytes per slot) and gathers
// the amplitudes they name, kPeNbrHops slots at a time.  The entries of a row
// follow its bonds in ascending order, so the sums are those of pe_row, bit
// for bit.  Slices are dealt to the XCDs in contiguous ranges, so that the
// near neighbours of low bonds are in the XCD's own L2.
template <typename R>
__global__ void __launch_bounds__(512) k_hv_pe_nbr(HvArgs a, PeArgs p,
                                                   const typename VT<R>::T* __restrict__ x,
                                                   typename VT<R>::T* __restrict__ y) {
  using V = typename VT<R>::T;
  const double u = control_value(a);
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wv = uniform_u32(threadIdx.x >> 6);
  const uint32_t ns = (p.dim + 63u) >> 6;
  const uint32_t nwv = blockDim.x >> 6;
  uint32_t hi = ns, s0 = blockIdx.x * nwv + wv, stride = gridDim.x * nwv;
  if ((gridDim.x & 7u) == 0u) {
    // contiguous slices per XCD (blocks are dealt to the 8 XCDs round robin)
    const uint32_t chunk = (ns + 7u) >> 3;
    const uint32_t lo = (blockIdx.x & 7u) * chunk;
    hi = min(lo + chunk, ns);
    s0 = lo + (blockIdx.x >> 3) * nwv + wv;
    stride = (gridDim.x >> 3) * nwv;
  }
  for (uint32_t s = s0; s < hi; s += stride) {
    const uint32_t b = (s << 6) | lane;
    const bool in = b < p.dim;
    R yr, yi;
    bool bad;
    pe_row_nbr<R>(a, p, u, s, in ? b : p.dim - 1u, lane, [&](uint32_t i) { return x[i]; }, yr, yi,
                  bad);
    if (in) {
      V o;
      o.x = bad ? (R)NAN : yr;
      o.y = bad ? (R)NAN : yi;
      y[b] = o;
    }
  }
}

// ---------------------------------------------------------------------- Lanczos passes

struct LzArgs {
  HvArgs hv;
  Geo geo;
  const void* slot0;  // stored vector 0: the input of the Krylov call
  void* basis;        // stored vectors 1..m-1
  void* yk;           // y_k = H v_k: written by pass A(k), read by pass B(k)
  int32_t k;          // basis step
  int32_t i0;         // first index of the projection window [i0, k]
  int32_t m;
  int32_t i0n;        // first index of the next step's window
  int32_t i0p;        // first index of the previous step's window
  int32_t alone;      // pass C: a step by itself, not the first of a pair
  double t;
  double tol;
  KState* st;
  cplx_d* partials;
};

constexpr int kMaxJobs = 2;

// Columns of the partials table (column major, one row per block).  Pass B(k)
// writes its measurements <u_j|y_k> in columns [0, nb) and <u_j|u_k> in
// [nb, 2nb) (window order) and its part of ||w||^2 in kNormCol; pass A(k)
// writes its parts of <v_k|y_k> and (||v_k||^2, ||y_k||^2) in kACol and kACol + 1, which
// no pass B writes.
constexpr int kACol = 2 * kMaxM;
constexpr int kNormCol = kMaxScal - 1;
static_assert(kACol + 2 == kNormCol, "partials columns");
static_assert(kMaxM <= 64, "a window is held one vector per lane of a wavefront");

// Independent Krylov calls of the same shape advanced by the same launches:
// blocks [j*G, (j+1)*G) serve job j.
struct LzBatch {
  LzArgs job[kMaxJobs];
};

template <typename V>
__device__ __forceinline__ const V* slot_ptr(const LzArgs& a, int i) {
  return i == 0 ? reinterpret_cast<const V*>(a.slot0)
                : reinterpret_cast<const V*>(a.basis) + (size_t)(i - 1) * a.geo.D;
}

// One lane's share of FinScalars.  Plain doubles, assigned one by one, so that
// they stay in registers while the loads are in flight.
struct FinRegs {
  double alpha = 0.0, offd = 0.0, scale = 0.0, normT = 0.0, beta0 = 0.0;
  double coef_re = 0.0, coef_im = 0.0, gprev_re = 0.0, gprev_im = 0.0;
  double cdiag_re = 0.0, cdiag_im = 0.0, csub_re = 0.0, csub_im = 0.0;
};

__device__ __forceinline__ void load_fin(const LzArgs& a, FinRegs& r) {
  const KState* st = a.st;
  const int l = threadIdx.x & 63;
  const int pk = (a.k - 1) & 1;   // step k-1's copies
  r.alpha = st->alpha[l];
  r.offd = st->offd[l];
  r.scale = st->scale[l];
  r.normT = st->normT[pk];
  r.beta0 = st->beta0;
  r.coef_re = st->coef[pk][l].re;
  r.coef_im = st->coef[pk][l].im;
  r.gprev_re = st->gcol[a.k & 1][l].re;
  r.gprev_im = st->gcol[a.k & 1][l].im;
  r.cdiag_re = st->cdiag[l].re;
  r.cdiag_im = st->cdiag[l].im;
  r.csub_re = st->csub[l].re;
  r.csub_im = st->csub[l].im;
}

// Wavefront 0 puts the fetched scalars in LDS.
__device__ __forceinline__ void stage_fin(const FinRegs& r, FinScalars& fs) {
  if (threadIdx.x >= 64) return;
  const int l = threadIdx.x;
  fs.alpha[l] = r.alpha;
  fs.offd[l] = r.offd;
  fs.scale[l] = r.scale;
  fs.coef[l] = cplx_d{r.coef_re, r.coef_im};
  fs.gprev[l] = cplx_d{r.gprev_re, r.gprev_im};
  fs.cdiag[l] = cplx_d{r.cdiag_re, r.cdiag_im};
  fs.csub[l] = cplx_d{r.csub_re, r.csub_im};
  if (l == 0) {
    fs.normT = r.normT;
    fs.beta0 = r.beta0;
  }
}

// Column `col` of a partials table summed over rows [0, G): lane l adds rows l,
// l + 64, ... in order (eight rows a lane in flight together), then a fixed
// butterfly.  The same value in every lane.
__device__ __forceinline__ cplx_d column_total(const cplx_d* col, uint32_t G) {
  const uint32_t lane = threadIdx.x & 63u;
  double re = 0.0, im = 0.0;
  for (uint32_t b0 = 0; b0 < G; b0 += 8u * 64u) {
    cplx_d v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = col[min(b0 + q * 64u + lane, G - 1u)];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const bool in = b0 + q * 64u + lane < G;
      re += in ? v[q].re : 0.0;
      im += in ? v[q].im : 0.0;
    }
  }
  return cplx_d{wave_sum(re), wave_sum(im)};
}

// Scalar tail of a basis: exp(-itT) e_1 on wavefront 0 and the combination
// coefficients beta0 c_j scale_j, into `dc` (LDS, nullable) and, with
// `writer`, into the state with m_eff.  Before the last step (a breakdown
// found in a pass B) the writer also sets the done flag, which stops the
// later launches of the call.  The combination never sets it: its other
// blocks read the flag to learn whether the basis ended before the last step.  `fresh_alpha`
// replaces alpha[m_eff-1], `fresh_b0`/`fresh_s0` beta0 and scale_0 (NaN: from
// fs), and for step kf >= 1 the pair (`off_kf`, `scale_kf`) replaces offd[kf]
// and scale[kf] (kf < 0: none): values of the running step, not in fs.
__device__ void finish_basis(const LzArgs& a, const FinScalars& fs, int m_eff, double fresh_alpha,
                             double fresh_b0, double fresh_s0, int kf, double off_kf,
                             double scale_kf, cplx_d* dc, bool writer, int* me) {
  KState* st = a.st;
  const int i = threadIdx.x & 63;
  double ai = 0.0, lo = 0.0, hi = 0.0, sc = 0.0;
  if (i < m_eff) {
    ai = (i == m_eff - 1 && !isnan(fresh_alpha)) ? fresh_alpha : fs.alpha[i];
    lo = (i > 0) ? (i == kf ? off_kf : fs.offd[i]) : 0.0;
    hi = (i + 1 < m_eff) ? (i + 1 == kf ? off_kf : fs.offd[i + 1]) : 0.0;
    sc = (i == 0 && !isnan(fresh_s0)) ? fresh_s0 : (i == kf ? scale_kf : fs.scale[i]);
  }
  const double b0 = isnan(fresh_b0) ? fs.beta0 : fresh_b0;
  double cr, ci;
  tri_exp_wave(ai, lo, hi, a.t, cr, ci);
  if (i < m_eff) {
    const cplx_d d{b0 * cr * sc, b0 * ci * sc};
    if (dc) dc[i] = d;
    if (writer) st->dcomb[i] = d;
  }
  if (i == 0) {
    if (me) *me = m_eff;
    if (writer) {
      st->m_eff = m_eff;
      if (a.k < a.m - 1) st->done = 1;
    }
  }
}

template <typename R, int RB>
__device__ __forceinline__ void store_y(const Tile<R, RB>& T, typename VT<R>::T* yk, uint32_t base,
                                        uint32_t eb, const Geo& g) {
  using V = typename VT<R>::T;
#pragma unroll
  for (int r = 0; r < (1 << RB); ++r) {
    const uint32_t s = base | eb | ((uint32_t)r << 6);
    if (!g.small || s < g.D) {
      V o;
      o.x = T.yr[r];
      o.y = T.yi[r];
      yk[s] = o;
    }
  }
}

// The reduced sums of step k into `tot` (LDS) and the earlier steps' scalars
// into `fs` (LDS), in the layout the scalar update reads:
//   tot[0, 2nb)   pass B(k-1)'s measurement totals (window dots of step k),
//   tot[2nb]      <v_k|y_k>,  tot[2nb + 1] = (||v_k||^2, ||y_k||^2)  (with `norm` only),
//   tot[2nb + 2]  ||w||^2 of pass B(k-1), the square of the next off-diagonal.
// The totals of pass B(k-1)'s columns come from pass A(k)'s helper
// wavefronts (KState::colsum); pass A(k)'s own columns are summed here over
// its G rows.  Every wavefront issues its loads before it waits.  Ends with a
// barrier; false (in every thread) when the basis ended in an earlier step.
__device__ bool gather_step(const LzArgs& a, uint32_t G, int nb, bool norm, FinScalars& fs,
                            cplx_d* tot) {
  __shared__ int ended;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wv = uniform_u32(threadIdx.x >> 6);
  const uint32_t nw = blockDim.x >> 6;
  const int k = a.k;
  const int ca = 2 * nb, ns = ca + 2;
  const KState* st = a.st;
  // wavefronts that sum the A columns: kACol always, kACol + 1 with `norm`
  const uint32_t wa0 = nw >= 2 ? 1u : 0u;
  const uint32_t wa1 = nw >= 3 ? 2u : wa0;
  if (wv == 0) {
    FinRegs fr;
    int d = 0;
    cplx_d c0{0.0, 0.0}, c1{0.0, 0.0};
    if (k > 0) {
      d = st->done;
      load_fin(a, fr);
      c0 = st->colsum[lane];
      c1 = st->colsum[lane + 64u];
    }
    if (wa0 == 0) {
      const cplx_d t = column_total(a.partials + (size_t)kACol * kPartialRows, G);
      if (lane == 0) tot[ca] = t;
      if (norm) {
        const cplx_d t1 = column_total(a.partials + (size_t)(kACol + 1) * kPartialRows, G);
        if (lane == 0) tot[ca + 1] = t1;
      }
    }
    if (k > 0) {
      stage_fin(fr, fs);
      const int nc = 2 * nb + 1;
      if ((int)lane < nc) tot[(int)lane < ca ? (int)lane : ns] = c0;
      if ((int)lane + 64 < nc) tot[(int)lane + 64 < ca ? (int)lane + 64 : ns] = c1;
    }
    if (lane == 0) ended = d;
  } else {
    if (wv == wa0) {
      const cplx_d t = column_total(a.partials + (size_t)kACol * kPartialRows, G);
      if (lane == 0) tot[ca] = t;
    }
    if (norm && wv == wa1) {
      const cplx_d t = column_total(a.partials + (size_t)(kACol + 1) * kPartialRows, G);
      if (lane == 0) tot[ca + 1] = t;
    }
  }
  __syncthreads();
  return ended == 0;
}

// The scalar update of step k on wavefront 0, from gather_step's sums: the
// breakdown test (or, at k = 0, the input norm), the window dots, the
// projection coefficients c^(k) into `cf` (LDS, window order; nullable) and
// 1/||v_k|| into *sk_out (nullable), alpha_k and the running ||T||.  Every block of a launch runs it on the same
// values, so all of them get the same coefficients; the one with `writer`
// keeps the scalars in the state for the later steps.  Returns true when the
// basis goes on.  At the last step (k = m-1), or when it ends here (a zero or
// non-finite input, a breakdown), it returns false after the combination
// coefficients went to `dc`/*me (nullable) and, with `writer`, to the state.
// kLocal: the first step of a pair, whose window is v_k alone: *cf is c_k, and no
// window dots are formed.
template <bool kLocal = false>
__device__ bool step_update(const LzArgs& a, const FinScalars& fs, const cplx_d* tot, int nb,
                            bool writer, cplx_d* cf, double* sk_out, cplx_d* dc, int* me,
                            double* sk_all = nullptr, double* bk_all = nullptr) {
  KState* st = a.st;
  const int lane = threadIdx.x;
  const int k = a.k;
  const int ca = 2 * nb, ns = ca + 2;
  const int nwin = k - a.i0 + 1;
  double sk, b0 = NAN, s0 = NAN, bk = 0.0;
  if (k == 0) {
    const double nn = tot[ca + 1].re;
    if (!(nn > 0.0)) {
      // a zero input gives a zero output; a non-finite one a NaN output
      const bool zero = nn == 0.0;
      if (lane == 0) {
        if (writer) {
          st->beta0 = zero ? 0.0 : NAN;
          st->m_eff = zero ? 0 : 1;
          st->dcomb[0] = cplx_d{NAN, NAN};
          if (a.m > 1) st->done = 1;
        }
        if (dc) dc[0] = cplx_d{NAN, NAN};
        if (me) *me = zero ? 0 : 1;
      }
      return false;
    }
    b0 = sqrt(nn);
    sk = 1.0 / b0;
    s0 = sk;
    if (writer && lane == 0) {
      st->beta0 = b0;
      st->scale[0] = sk;
      st->offd[0] = 0.0;
      st->done = 0;
    }
  } else {
    // ||w|| of pass B(k-1): the off-diagonal entry of step k, or a breakdown
    // (an invariant Krylov space of dimension k)
    bk = sqrt(tot[ns].re);
    if (bk <= a.tol * fmax(1.0, fs.normT)) {
      if (writer || dc) finish_basis(a, fs, k, NAN, NAN, NAN, -1, 0.0, 0.0, dc, writer, me);
      return false;
    }
    sk = 1.0 / bk;
    if (writer && lane == 0) {
      st->offd[k] = bk;
      st->scale[k] = sk;
    }
  }
  // lane l: window index i0 + l (a window holds at most kMaxM <= 64 vectors)
  const cplx_d d = (!kLocal && nb > 0) ? window_dots(k, a.i0, a.i0p, fs, tot, nb, tot[ns].re,
                                          writer ? st->gcol[(k - 1) & 1] : nullptr)
                             : cplx_d{0.0, 0.0};
  if (kLocal) {
    if (cf && lane == 0) cf[0] = cplx_d{tot[ca].re * sk * sk * sk, tot[ca].im * sk * sk * sk};
  } else if (lane < nwin) {
    const int i = a.i0 + lane;
    const double si = (i == k) ? sk : fs.scale[i];
    const double f = si * sk;
    const cplx_d t = (i == k) ? tot[ca] : d;
    const cplx_d c{t.re * f * si, t.im * f * si};
    if (cf) cf[lane] = c;
    if (writer) {
      st->coef[k & 1][lane] = c;
      if (i == k) st->cdiag[k] = c;
      if (i == k - 1) st->csub[k] = c;
    }
  }
  const double alpha = tot[ca].re * sk * sk;
  const double offk = (k == 0) ? 0.0 : bk;
  const double prevT = (k == 0) ? 0.0 : fs.normT;
  const double normT = fmax(prevT, fabs(alpha) + offk);
  if (writer && lane == 0) {
    st->alpha[k] = alpha;
    st->normT[k & 1] = normT;
  }
  if (k == a.m - 1) {
    finish_basis(a, fs, a.m, alpha, b0, s0, k, bk, sk, dc, writer, me);
    return false;
  }
  if (sk_out && lane == 0) *sk_out = sk;
  if (sk_all) {   // every lane's own
    *sk_all = sk;
    *bk_all = bk;
  }
  return true;
}

// Pass A(k): y = H v_k, stored as y_k (not at the last step), and this block's
// parts of <v_k|y>, ||v_k||^2 and ||y||^2 (row bl of the A columns).  No grid-wide
// reduction: the scalar update of step k runs in the prologue of pass B(k)
// (of the combination at the last step), in every block.  Helper wavefronts
// (wavefront w of block b takes column b + w G) sum pass B(k-1)'s measurement
// and norm columns over the grid into KState::colsum, so that pass B(k) reads
// 2nb + 1 totals instead of the whole table.
// kYIn: y_k was written by a separate H v kernel (the reduced basis); the pass
// then loads it instead of forming it on the tile.
template <typename R, int RB, bool kYIn = false, bool kPairs = false>
__device__ __forceinline__ void pass_a_body(const LzArgs& a, uint32_t bl, uint32_t G) {
  using V = typename VT<R>::T;
  constexpr int NR = 1 << RB;
  extern __shared__ unsigned char smem_raw[];
  V* lds = reinterpret_cast<V*>(smem_raw);
  __shared__ double wsum[16][4];

  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wv = uniform_u32(threadIdx.x >> 6);
  const uint32_t nw = blockDim.x >> 6;
  const uint32_t eb = lane | (wv << (6 + RB));
  // this wavefront's totals: lane 0 Re<v_k|y>, lane 1 Im<v_k|y>, lane 2 ||v_k||^2,
  // lane 3 ||y||^2
  double acc = 0.0;

  const double u = control_value(a.hv);
  const V* x = slot_ptr<V>(a, a.k);
  V* yk = reinterpret_cast<V*>(a.yk);
  const uint32_t iters = a.geo.ntiles / G;
  // a finished basis (breakdown in an earlier step): the flag is read here
  // and tested after the tile work, so its load waits on nothing
  const bool finished = a.k > 0 && a.st->done != 0;
  Tile<R, RB> T;
  for (uint32_t it = 0; it < iters; ++it) {
    const uint32_t tile = tile_of(a.geo, it, bl, G);
    if (it) __syncthreads();
    const uint32_t base = tile << a.geo.TB;
    if constexpr (kYIn) {
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const uint32_t s = base | eb | ((uint32_t)r << 6);
        const bool ok = s < a.geo.D;
        const V xv = ld_masked(x, s, ok);
        const V yy = ld_masked(yk, s, ok);
        T.xr[r] = xv.x;
        T.xi[r] = xv.y;
        T.yr[r] = yy.x;
        T.yi[r] = yy.y;
      }
    } else if constexpr (kPairs) {
      hv_tile_pairs<RB>(T, a.hv, a.geo, tile, x, lds, u);
      if (a.k + 1 < a.m) store_pairs<RB>(T, yk, base);
    } else {
      hv_tile<R, RB>(T, a.hv, a.geo, tile, x, lds, u);
      if (a.k + 1 < a.m) store_y<R, RB>(T, yk, base, eb, a.geo);
    }
    // <v_k|y>, ||v_k||^2 and ||y||^2 from registers
    double sr = 0.0, si = 0.0, nn = 0.0, yy = 0.0;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const double vr = T.xr[r], vi = T.xi[r], yr = T.yr[r], yi = T.yi[r];
      sr += vr * yr + vi * yi;
      si += vr * yi - vi * yr;
      nn += vr * vr + vi * vi;
      yy += yr * yr + yi * yi;
    }
    acc += quad_sums(sr, si, nn, yy);
  }
  if (finished) return;
  // this block's row of the A columns, the wavefronts summed in order
  if (lane < 4u) wsum[wv][lane] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double sr = 0.0, si = 0.0, nn = 0.0, yy = 0.0;
    for (uint32_t q = 0; q < nw; ++q) {
      sr += wsum[q][0];
      si += wsum[q][1];
      nn += wsum[q][2];
      yy += wsum[q][3];
    }
    a.partials[(size_t)kACol * kPartialRows + bl] = cplx_d{sr, si};
    a.partials[(size_t)(kACol + 1) * kPartialRows + bl] = cplx_d{nn, yy};
  }
  // helpers: totals of pass B(k-1)'s columns (written by the previous launch)
  const int nb = (a.k > 0 && a.i0 < a.k) ? a.k - a.i0p : 0;
  const int nh = (a.k > 0) ? 2 * nb + 1 : 0;
  for (int c = (int)bl + (int)(G * wv); c < nh; c += (int)(G * nw)) {
    const int src = (c < 2 * nb) ? c : kNormCol;
    const cplx_d t = column_total(a.partials + (size_t)src * kPartialRows, G);
    if (lane == 0) a.st->colsum[c] = t;
  }
}

template <typename R, int RB, bool kPairs = false>
__global__ void __launch_bounds__(RB >= 3 ? 512 : 1024) k_pass_a(LzBatch B) {
  const uint32_t G = B.job[0].geo.grid;
  if (blockIdx.x < G) {
    pass_a_body<R, RB, false, kPairs>(B.job[0], blockIdx.x, G);
  } else {
    pass_a_body<R, RB, false, kPairs>(B.job[1], blockIdx.x - G, G);
  }
}

// Pass A of the reduced basis: y given (complex64 and complex128 with four
// amplitudes per thread).
template <typename R>
__global__ void __launch_bounds__(1024) k_pass_a_y(LzBatch B) {
  const uint32_t G = B.job[0].geo.grid;
  if (blockIdx.x < G) {
    pass_a_body<R, 2, true>(B.job[0], blockIdx.x, G);
  } else {
    pass_a_body<R, 2, true>(B.job[1], blockIdx.x - G, G);
  }
}

// Pass B(k): the scalar update of step k in its prologue (every block, on the
// same sums: gather_step, step_update), then w = s_k y_k - sum_i c_i v_i over
// the window [i0, k], i0 = k - 1 or k (FP64), stored unnormalised as v_{k+1}, with this block's
// part of ||w||^2 (column kNormCol) and, when step k+1 has window dots, of
// <v_i|y_k> (columns [0, nb)) and <v_i|v_k> (columns [nb, 2nb)) for i in the
// window: the operands are already in registers for the update, and step k+1
// derives its dots from them.
// Placement of a thread's NR amplitudes in pass B's tile.  Pass B couples no
// neighbours, so any placement that covers the tile will do.  kBPairs (whole
// tiles, complex64): amplitude r = 2p + h at base | wv << (6+RB) | p << 7 |
// lane << 1 | h, so that every load and store moves two amplitudes (16 bytes).
// kBSlots / kBMasked: pass A's slots base | lane | wv << (6+RB) | r << 6, the
// masked form for a vector shorter than its tile.
enum BMode { kBPairs = 0, kBSlots = 1, kBMasked = 2 };

template <int MODE, int RB>
__device__ __forceinline__ uint32_t bpos(uint32_t base, uint32_t lane, uint32_t wv, int r) {
  if constexpr (MODE == kBPairs) {
    return base | (wv << (6 + RB)) | ((uint32_t)(r >> 1) << 7) | (lane << 1) | (uint32_t)(r & 1);
  } else {
    return base | lane | (wv << (6 + RB)) | ((uint32_t)r << 6);
  }
}

// NT: nontemporal loads (whole tiles only; see ld_stream).
template <int MODE, int RB, bool NT = false, typename V, int NR>
__device__ __forceinline__ void bload(const V* __restrict__ p, uint32_t base, uint32_t lane, uint32_t wv,
                                      uint32_t D, V (&o)[NR]) {
  if constexpr (MODE == kBPairs) {
    static_assert(sizeof(V) == 8 && NR % 2 == 0, "pairs of complex64 amplitudes");
#pragma unroll
    for (int q = 0; q < NR / 2; ++q) {
      const float4* a = reinterpret_cast<const float4*>(p + bpos<MODE, RB>(base, lane, wv, 2 * q));
      const float4 v = NT ? ld_stream4(a) : *a;
      o[2 * q] = V{v.x, v.y};
      o[2 * q + 1] = V{v.z, v.w};
    }
  } else {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const uint32_t s = bpos<MODE, RB>(base, lane, wv, r);
      if constexpr (MODE == kBSlots) {
        o[r] = NT ? ld_stream(p + s) : p[s];
      } else {
        o[r] = ld_masked(p, s, s < D);
      }
    }
  }
}

// NT streams the vectors with nontemporal loads.
template <typename R, int RB, int MODE, bool NT = false>
__device__ __forceinline__ void pass_b_body(const LzArgs& a, uint32_t bl, uint32_t G) {
  using V = typename VT<R>::T;
  constexpr int NR = 1 << RB;
  extern __shared__ unsigned char smem_raw[];
  __shared__ cplx_d tot[kMaxScal];
  __shared__ FinScalars fs;
  __shared__ cplx_d cf[kMaxM];
  __shared__ double sk_s;
  __shared__ int go;

  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wv = uniform_u32(threadIdx.x >> 6);

  // ---- the scalar update of step k (window dots of pass B(k-1)'s measurements)
  const int nb_in = (a.k > 0 && a.i0 < a.k) ? a.k - a.i0p : 0;
  if (!gather_step(a, G, nb_in, a.k == 0, fs, tot)) return;
  if (wv == 0) {
    const bool cont = step_update(a, fs, tot, nb_in, bl == 0, cf, &sk_s, nullptr, nullptr);
    if (lane == 0) go = cont ? 1 : 0;
  }
  __syncthreads();
  if (!go) return;

  const int nb = (a.i0n <= a.k) ? a.k - a.i0 + 1 : 0;
  double acc_nn = 0.0;
  // this wavefront's measurements accumulate in its row of wacc: <v_i|y_k>
  // in column i - i0, <v_i|v_k> in column nb + i - i0
  cplx_d* wacc = reinterpret_cast<cplx_d*>(smem_raw);
  cplx_d* wrow = wacc + wv * kMaxScal;
  for (int j = (int)lane; j < 2 * nb; j += 64) wrow[j] = cplx_d{0.0, 0.0};
  // lanes 0..3 hold the totals of quad_sums: column w's re and im parts of the
  // first dot, then of the second
  const auto add_quad = [&](int w, double t) {
    if (lane < 4u) {
      cplx_d& d = wrow[(lane < 2u ? 0 : nb) + w];
      if (lane & 1u) {
        d.im += t;
      } else {
        d.re += t;
      }
    }
  };

  // the streaming part stores only v_{k+1}, so the vectors it reads cannot
  // alias its stores
  const V* __restrict__ x = slot_ptr<V>(a, a.k);
  const V* __restrict__ yv = reinterpret_cast<const V*>(a.yk);
  V* __restrict__ out = reinterpret_cast<V*>(a.basis) + (size_t)a.k * a.geo.D;
  const uint32_t iters = a.geo.ntiles / G;
  const double sk = sk_s;
  const uint32_t D = a.geo.D;
  // same block-to-tile map as pass A, so y is read back from the L2 that wrote it
  for (uint32_t it = 0; it < iters; ++it) {
    const uint32_t base = tile_of(a.geo, it, bl, G) << a.geo.TB;
    V yo[NR], xo[NR];
    bload<MODE, RB, NT>(yv, base, lane, wv, D, yo);
    bload<MODE, RB, NT>(x, base, lane, wv, D, xo);
    double zr[NR], zi[NR];
    {
      const cplx_d c = cf[a.k - a.i0];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const double vr = xo[r].x, vi = xo[r].y;
        zr[r] = sk * (double)yo[r].x - (c.re * vr - c.im * vi);
        zi[r] = sk * (double)yo[r].y - (c.re * vi + c.im * vr);
      }
    }
    if (nb) {
      // <v_k|y_k> and ||v_k||^2
      double sr = 0.0, si = 0.0, gr = 0.0;
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const double vr = xo[r].x, vi = xo[r].y, yr = yo[r].x, yi = yo[r].y;
        sr += vr * yr + vi * yi;
        si += vr * yi - vi * yr;
        gr += vr * vr + vi * vi;
      }
      add_quad(a.k - a.i0, quad_sums(sr, si, gr, 0.0));
    }
    if (a.i0 < a.k) {
      V q[NR];
      bload<MODE, RB, NT>(slot_ptr<V>(a, a.i0), base, lane, wv, D, q);
      const cplx_d c = cf[0];
      double sr = 0.0, si = 0.0, gr = 0.0, gi = 0.0;
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const double vr = q[r].x, vi = q[r].y;
        zr[r] -= c.re * vr - c.im * vi;
        zi[r] -= c.re * vi + c.im * vr;
        const double yr = yo[r].x, yi = yo[r].y, xr = xo[r].x, xi = xo[r].y;
        sr += vr * yr + vi * yi;
        si += vr * yi - vi * yr;
        gr += vr * xr + vi * xi;
        gi += vr * xi - vi * xr;
      }
      if (nb) add_quad(0, quad_sums(sr, si, gr, gi));
    }
    // store w; its norm from the stored (rounded) values
    double nn = 0.0;
    if constexpr (MODE == kBPairs) {
#pragma unroll
      for (int q = 0; q < NR / 2; ++q) {
        const float4 o{(float)zr[2 * q], (float)zi[2 * q], (float)zr[2 * q + 1], (float)zi[2 * q + 1]};
        *reinterpret_cast<float4*>(out + bpos<MODE, RB>(base, lane, wv, 2 * q)) = o;
        nn += (double)o.x * o.x + (double)o.y * o.y + (double)o.z * o.z + (double)o.w * o.w;
      }
    } else {
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const uint32_t s = bpos<MODE, RB>(base, lane, wv, r);
        V o;
        o.x = (R)zr[r];
        o.y = (R)zi[r];
        if (MODE == kBSlots || s < D) {
          out[s] = o;
          const double wr = o.x, wi = o.y;
          nn += wr * wr + wi * wi;
        }
      }
    }
    acc_nn += wave_sum(nn);
  }
  if (lane == 0) wrow[2 * nb] = cplx_d{acc_nn, 0.0};
  __syncthreads();
  block_totals(wacc, 2 * nb + 1, tot);
  // this block's row: the measurements, and its part of ||w||^2 for step k+1
  for (int j = threadIdx.x; j < 2 * nb; j += blockDim.x) a.partials[(size_t)j * kPartialRows + bl] = tot[j];
  if (threadIdx.x == 0) a.partials[(size_t)kNormCol * kPartialRows + bl] = cplx_d{tot[2 * nb].re, 0.0};
}

template <typename R, int RB, int MODE, bool NT = false>
__global__ void __launch_bounds__(RB >= 3 ? 512 : 1024) k_pass_b(LzBatch B) {
  const uint32_t G = B.job[0].geo.grid;
  if (blockIdx.x < G) {
    pass_b_body<R, RB, MODE, NT>(B.job[0], blockIdx.x, G);
  } else {
    pass_b_body<R, RB, MODE, NT>(B.job[1], blockIdx.x - G, G);
  }
}

// Two Lanczos steps per pass over the window (full re-orthogonalisation).  A pass
// B(k) is bound by the stream of v_0..v_k; here one stream serves two steps:
//   pass A(b), pass C(b):      v_{b+1} = p = s_b y - alpha_b v_b - beta_b v_{b-1}, the
//                              three-term step, and - sum E_i v_i where p's overlaps
//                              E_i = <v_i|p> with the window matter;
//   pass A(b+1), pass P(b):    with y = H p: w_{b+2} = H v_{b+1} - alpha v_{b+1}
//                              - beta v_b - (overlaps).
// What <v_i|p> is follows, as in pass B, from the overlaps of v_b and v_{b-1} that
// pass P(b-2) measured and H's tridiagonal form, before p is formed.  While every
// |E_i| / ||p|| is below a few units of roundoff of the stored vectors (random states:
// about one over sqrt(D)), or E_i is what FP64 sums leave of ||T|| anyway, p reads three
// vectors; then the overlaps enter w_{b+2} alone.  (Limits of 1 to 64 units gave the
// same errors within 3 % over 1,600 random calls; the projections cost 8 % of a call at
// L=20 in complex128 when FP64's own noise counted.)  Otherwise p is projected on the whole
// window like pass B's vectors, before it is rounded and before its norm is tested: near
// the end of a basis p is rounding noise, whose overlaps are of its own size, and a
// correction after the fact ended in NaN.  w_{b+2} is always corrected.  Per pair the
// vectors moved fall from 2b + 7 to b + 8 (2b + 7 again where p is projected).
// A vector that overlaps an earlier one by more than a half is no new direction: the
// invariant space is exhausted in the vectors' precision though the breakdown test,
// whose tolerance is a few units of roundoff of ||T||, let noise through; the basis ends
// before it.  (The measured overlaps say so two steps later: the last two vectors of a
// basis go unchecked.)
//
// In normalised vectors, with g_i = <v_i|v_b>, h_i = <v_i|v_{b-1}> and
// beta = ||p||:
//   E_i = beta_{i+1} g_{i+1} + (alpha_i - alpha_b) g_i + beta_i g_{i-1}
//         - beta_b h_i                           (i < b; the exact 1s cancel),
//   E_b = -beta_b conj(g_{b-1}),   e_i = E_i / beta, or 0 where p was projected,
//   alpha    = <p|Hp> / beta^2,
//   f_i      = beta_i e_{i-1} + (alpha_i - alpha) e_i + beta_{i+1} e_{i+1} - beta g_i,
//   w_{b+2}  = (H p - alpha p) / beta - beta v_b - sum f_i v_i.
// Pass P measures <v_i|p>, <v_i|Hp> and, from its output, <v_{b+1}|w_{b+2}> and
// ||w_{b+2}||^2; pass C(b+2) turns them into the next g and h.

// The overlaps of a pair's p, on wavefront 0 of every block of pass C(b) (b = a.k, sb =
// 1/||v_b||, bb = ||v_b||, 0 at b = 0): g and h from pass P(b-2)'s totals (nb = b columns a set), then E_i.  Returns
// kPairProject when p is projected; then ec[i] holds E_i on the stored vectors, i in [0, b].
// ||p||^2 comes from ||y||^2 less the two coefficients; where these cancel to where the
// estimate means little, any overlap counts.  kPairEnd: v_{b-1} or v_b is no new direction.
// State, with `writer`: g, and E in csub (0 if p is projected), or the finished basis.
enum { kPairPlain, kPairProject, kPairEnd };
__device__ int pair_overlaps(const LzArgs& a, const FinScalars& fs, const cplx_d* tot, double sb,
                             double bb, double unit, bool writer, cplx_d* ec) {
  const int i = threadIdx.x, b = a.k;
  const cplx_d zero{0.0, 0.0};
  cplx_d g = zero, h = zero;
  if (i < b) {
    const double s1 = fs.scale[b - 1];
    if (i == b - 1) {
      g = cplx_d{tot[i].re * s1 * sb, tot[i].im * s1 * sb};
    } else {
      const double f = fs.scale[i] * s1;
      h = cplx_d{tot[b + i].re * f, tot[b + i].im * f};
      const cplx_d N{tot[i].re * f, tot[i].im * f}, S = fs.cdiag[i];
      const double al = fs.alpha[b - 1];
      g = cplx_d{(N.re - al * h.re - S.re) * sb, (N.im - al * h.im - S.im) * sb};
    }
  }
  const bool old_h = __any(h.re * h.re + h.im * h.im > 0.25);
  if (old_h || __any(g.re * g.re + g.im * g.im > 0.25)) {
    if (writer) finish_basis(a, fs, old_h ? b - 1 : b, NAN, NAN, NAN, -1, 0.0, 0.0, nullptr, true, nullptr);
    return kPairEnd;
  }
  const cplx_d gm{__shfl_up(g.re, 1, 64), __shfl_up(g.im, 1, 64)};
  const cplx_d gp{__shfl_down(g.re, 1, 64), __shfl_down(g.im, 1, 64)};   // 0 from lane b on
  const double ab = tot[2 * b].re * sb * sb;
  cplx_d E = zero;
  if (i < b) {
    const double ai = fs.alpha[i] - ab, bi = i > 0 ? fs.offd[i] : 0.0;
    const double bn = i + 1 < b ? fs.offd[i + 1] : 0.0;
    E.re = bn * gp.re + ai * g.re + (i > 0 ? bi * gm.re : 0.0) - bb * h.re;
    E.im = bn * gp.im + ai * g.im + (i > 0 ? bi * gm.im : 0.0) - bb * h.im;
  } else if (i == b && b > 0) {
    E.re = -bb * gm.re;
    E.im = bb * gm.im;
  }
  const double normT = fmax(b > 0 ? fs.normT : 0.0, fabs(ab) + bb);
  const double b2 = sb * sb * tot[2 * b + 1].im - ab * ab - bb * bb;
  // FP64 sums leave an E of a few of their own roundings of ||T||, whatever the overlap
  const double own = (32 * 0x1p-53) * normT;
  const double lim = b2 > 1e-10 * normT * normT ? fmax(16.0 * unit * unit * b2, own * own) : 0.0;
  const bool corr = __any(E.re * E.re > lim || E.im * E.im > lim);
  if (i <= b) {
    const double si = i < b ? fs.scale[i] : sb;
    ec[i] = cplx_d{E.re * si, E.im * si};
  }
  if (writer && i <= b) {
    a.st->csub[i] = corr ? zero : E;
    if (i < b) a.st->gcol[(b + 1) & 1][i] = g;
  }
  return corr ? kPairProject : kPairPlain;
}

// The scalars of pass P on wavefront 0 (a.k = b + 1; tot[0] = <p|Hp>, tot[1].re =
// ||p||^2; fs.gprev holds g and fs.csub E): the coefficients of w_{b+2} on the stored
// window vectors into fc, alpha and 1/||p||.  State, with `writer`: cdiag[i], the part of
// <v_i|w_{b+2}> known before the stream.  False after a breakdown.
__device__ bool pair_update(const LzArgs& a, const FinScalars& fs, const cplx_d* tot, bool writer,
                            cplx_d* fc, double* alpha_out, double* sp_out) {
  KState* st = a.st;
  const int i = threadIdx.x;
  const int k = a.k, b = k - 1;
  const double bk = sqrt(tot[1].re);
  if (bk <= a.tol * fmax(1.0, fs.normT)) {
    finish_basis(a, fs, k, NAN, NAN, NAN, -1, 0.0, 0.0, nullptr, writer, nullptr);
    return false;
  }
  const double sp = 1.0 / bk;
  const cplx_d zero{0.0, 0.0};
  const bool in = i <= b;
  const double ai = in ? fs.alpha[i] : 0.0, bi = (in && i > 0) ? fs.offd[i] : 0.0;
  const double bn = i < b ? fs.offd[i + 1] : 0.0, si = in ? fs.scale[i] : 0.0;
  const cplx_d g = i < b ? fs.gprev[i] : zero;
  const cplx_d E = in ? fs.csub[i] : zero;
  const cplx_d e{E.re * sp, E.im * sp};
  const cplx_d em{__shfl_up(e.re, 1, 64), __shfl_up(e.im, 1, 64)};
  const cplx_d ep{__shfl_down(e.re, 1, 64), __shfl_down(e.im, 1, 64)};
  const double alpha = tot[0].re * sp * sp;
  // beta_0 = 0 and beta_{i+1} of lane b = 0 end the three-term sums
  cplx_d S{(i > 0 ? bi * em.re : 0.0) + (ai - alpha) * e.re + bn * ep.re,
           (i > 0 ? bi * em.im : 0.0) + (ai - alpha) * e.im + bn * ep.im};
  cplx_d F{S.re - bk * g.re, S.im - bk * g.im};
  if (i == b) {
    S.re += bk;
    F.re += bk;
  }
  if (in) fc[i] = cplx_d{F.re * si, F.im * si};
  if (i == 0) {
    *alpha_out = alpha;
    *sp_out = sp;
  }
  if (writer) {
    if (in) st->cdiag[i] = S;
    if (i == 0) {
      st->alpha[k] = alpha;
      st->offd[k] = bk;
      st->scale[k] = sp;
      st->normT[k & 1] = fmax(fs.normT, fabs(alpha) + bk);
    }
  }
  return true;
}

template <int MODE, int RB, typename V, int NR>
__device__ __forceinline__ void bstore(V* __restrict__ p, uint32_t base, uint32_t lane, uint32_t wv,
                                       uint32_t D, const V (&o)[NR]) {
  if constexpr (MODE == kBPairs) {
#pragma unroll
    for (int q = 0; q < NR / 2; ++q)
      *reinterpret_cast<float4*>(p + bpos<MODE, RB>(base, lane, wv, 2 * q)) =
          float4{o[2 * q].x, o[2 * q].y, o[2 * q + 1].x, o[2 * q + 1].y};
  } else {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const uint32_t s = bpos<MODE, RB>(base, lane, wv, r);
      if (MODE == kBSlots || s < D) p[s] = o[r];
    }
  }
}

// Pass C(b), b = a.k: the scalar update of step b, then the three-term step.  Three
// vectors read, one written; b - 1 more read where p is projected on the window.
// `alone` (b = 0, m even): the step stands for itself, so its norm and overlap with
// v_0 are measured.
template <typename R, int RB, int MODE, int NW, bool NT>
__device__ __forceinline__ void pass_c_body(const LzArgs& a, uint32_t bl, uint32_t G) {
  using V = typename VT<R>::T;
  constexpr int NR = 1 << RB;
  // one row a wavefront; static arrays alone would let the compiler put the scalar
  // update's temporaries into 64 KB of LDS, and one block fit on a CU (20 us for 8)
  extern __shared__ unsigned char smem_raw[];
  double* wsum = reinterpret_cast<double*>(smem_raw);
  __shared__ cplx_d tot[kMaxScal];
  __shared__ FinScalars fs;
  __shared__ cplx_d ec[kMaxM];
  __shared__ cplx_d cf;
  __shared__ double sk_s;
  __shared__ int go, corr_s;

  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wv = uniform_u32(threadIdx.x >> 6);
  const int b = a.k;
  if (!gather_step(a, G, b, true, fs, tot)) return;
  if (wv == 0) {
    double sb, bb;
    const bool cont = step_update<true>(a, fs, tot, b, bl == 0, &cf, &sk_s, nullptr, nullptr, &sb, &bb);
    const int pair = cont ? pair_overlaps(a, fs, tot, sb, bb, sizeof(R) == 4 ? 0x1p-24 : 0x1p-53, bl == 0, ec)
                          : kPairEnd;
    if (lane == 0) {
      go = pair != kPairEnd ? 1 : 0;
      corr_s = pair == kPairProject ? 1 : 0;
    }
  }
  __syncthreads();
  if (!go) return;
  const double sk = sk_s;
  const bool corr = uniform_u32((uint32_t)corr_s) != 0;
  cplx_d c = cf, c1{b > 0 ? fs.scale[b - 1] / sk : 0.0, 0.0};
  if (corr) {
    c = cplx_d{c.re + ec[b].re, c.im + ec[b].im};
    c1 = cplx_d{c1.re + ec[b - 1].re, ec[b - 1].im};
  }
  const V* __restrict__ x = slot_ptr<V>(a, b);
  const V* __restrict__ x1 = slot_ptr<V>(a, b > 0 ? b - 1 : 0);
  const V* __restrict__ yv = reinterpret_cast<const V*>(a.yk);
  V* __restrict__ out = reinterpret_cast<V*>(a.basis) + (size_t)b * a.geo.D;
  const uint32_t iters = a.geo.ntiles / G;
  const uint32_t D = a.geo.D;
  double acc = 0.0;
  for (uint32_t it = 0; it < iters; ++it) {
    const uint32_t base = tile_of(a.geo, it, bl, G) << a.geo.TB;
    V yo[NR], xo[NR], xm[NR], o[NR];
    bload<MODE, RB, NT>(yv, base, lane, wv, D, yo);
    bload<MODE, RB, NT>(x, base, lane, wv, D, xo);
    bload<MODE, RB, NT>(x1, base, lane, wv, D, xm);  // b = 0: v_0 again, times 0
    double zr[NR], zi[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const double vr = xo[r].x, vi = xo[r].y, ur = xm[r].x, ui = xm[r].y;
      zr[r] = sk * (double)yo[r].x - (c.re * vr - c.im * vi) - (c1.re * ur - c1.im * ui);
      zi[r] = sk * (double)yo[r].y - (c.re * vi + c.im * vr) - (c1.re * ui + c1.im * ur);
    }
    if (corr) {
      for (int i = 0; i < b - 1; i += NW) {
        V q[NW][NR];
#pragma unroll
        for (int j = 0; j < NW; ++j) {
          if (i + j < b - 1) bload<MODE, RB, NT>(slot_ptr<V>(a, i + j), base, lane, wv, D, q[j]);
        }
#pragma unroll
        for (int j = 0; j < NW; ++j) {
          if (i + j < b - 1) {
            const cplx_d e = ec[i + j];
#pragma unroll
            for (int r = 0; r < NR; ++r) {
              const double vr = q[j][r].x, vi = q[j][r].y;
              zr[r] -= e.re * vr - e.im * vi;
              zi[r] -= e.re * vi + e.im * vr;
            }
          }
        }
      }
    }
    double sr = 0.0, si = 0.0, nn = 0.0;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const double vr = xo[r].x, vi = xo[r].y;
      o[r].x = (R)zr[r];
      o[r].y = (R)zi[r];
      const double wr = o[r].x, wi = o[r].y;
      sr += vr * wr + vi * wi;
      si += vr * wi - vi * wr;
      nn += wr * wr + wi * wi;
    }
    bstore<MODE, RB>(out, base, lane, wv, D, o);
    if (a.alone) acc += quad_sums(sr, si, nn, 0.0);
  }
  if (!a.alone) return;
  if (lane < 3u) wsum[3u * wv + lane] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double sr = 0.0, si = 0.0, nn = 0.0;
    for (uint32_t q = 0; q < (blockDim.x >> 6); ++q) {
      sr += wsum[3 * q];
      si += wsum[3 * q + 1];
      nn += wsum[3 * q + 2];
    }
    a.partials[bl] = cplx_d{sr, si};
    a.partials[kPartialRows + bl] = cplx_d{0.0, 0.0};
    a.partials[(size_t)kNormCol * kPartialRows + bl] = cplx_d{nn, 0.0};
  }
}

template <typename R, int RB, int MODE, int NW, bool NT = false>
__global__ void __launch_bounds__(RB >= 3 ? 512 : 1024) k_pass_c(LzBatch B) {
  const uint32_t G = B.job[0].geo.grid;
  if (blockIdx.x < G) {
    pass_c_body<R, RB, MODE, NW, NT>(B.job[0], blockIdx.x, G);
  } else {
    pass_c_body<R, RB, MODE, NW, NT>(B.job[1], blockIdx.x - G, G);
  }
}

// Pass P(b), a.k = b + 1: w_{b+2} in one pass over v_0..v_b.  Bound
// by the stream: at L=20 complex64 1.4 us per window vector of 8.4 MB (6 TB/s) on 11
// us of prologue, two vectors and stores; pass C takes 8 us.  A call at m = 20 613 ->
// 502 us, at L=24, m = 24 11.4 -> 8.75 ms (pass B streamed as fast, twice as much).
// Columns of its measurements: <v_i|Hp> in [0, b + 1), <v_{b+1}|w_{b+2}> in b + 1,
// <v_i|p> from b + 2, ||w_{b+2}||^2 in kNormCol.
template <typename R, int RB, int MODE, int NW, bool NT>
__device__ __forceinline__ void pass_p_body(const LzArgs& a, uint32_t bl, uint32_t G) {
  using V = typename VT<R>::T;
  constexpr int NR = 1 << RB;
  extern __shared__ unsigned char smem_raw[];
  __shared__ cplx_d tot[kMaxScal];
  __shared__ FinScalars fs;
  __shared__ cplx_d fc[kMaxM];
  __shared__ double alpha_s, sp_s;
  __shared__ int go;

  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wv = uniform_u32(threadIdx.x >> 6);
  if (!gather_step(a, G, 0, true, fs, tot)) return;
  if (wv == 0) {
    const bool cont = pair_update(a, fs, tot, bl == 0, fc, &alpha_s, &sp_s);
    if (lane == 0) go = cont ? 1 : 0;
  }
  __syncthreads();
  if (!go) return;

  const int nwin = a.k;        // window vectors 0..b
  const int nb = a.k + 1;
  cplx_d* wacc = reinterpret_cast<cplx_d*>(smem_raw);
  cplx_d* wrow = wacc + wv * kMaxScal;
  for (int j = (int)lane; j <= 2 * nb; j += 64) wrow[j] = cplx_d{0.0, 0.0};
  const auto add_quad = [&](int w, double t) {
    if (lane < 4u) {
      cplx_d& d = wrow[(lane < 2u ? 0 : nb) + w];
      if (lane & 1u) {
        d.im += t;
      } else {
        d.re += t;
      }
    }
  };
  const double sp = sp_s, kp = alpha_s * sp;
  const V* __restrict__ yv = reinterpret_cast<const V*>(a.yk);
  const V* __restrict__ pv = slot_ptr<V>(a, a.k);
  V* __restrict__ out = reinterpret_cast<V*>(a.basis) + (size_t)a.k * a.geo.D;
  const uint32_t iters = a.geo.ntiles / G;
  const uint32_t D = a.geo.D;
  for (uint32_t it = 0; it < iters; ++it) {
    const uint32_t base = tile_of(a.geo, it, bl, G) << a.geo.TB;
    V yo[NR], xo[NR];
    bload<MODE, RB, NT>(yv, base, lane, wv, D, yo);
    bload<MODE, RB, NT>(pv, base, lane, wv, D, xo);
    double zr[NR], zi[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      zr[r] = sp * (double)yo[r].x - kp * (double)xo[r].x;
      zi[r] = sp * (double)yo[r].y - kp * (double)xo[r].y;
    }
    for (int i = 0; i < nwin; i += NW) {
      V q[NW][NR];
#pragma unroll
      for (int j = 0; j < NW; ++j) {
        if (i + j < nwin) bload<MODE, RB, NT>(slot_ptr<V>(a, i + j), base, lane, wv, D, q[j]);
      }
#pragma unroll
      for (int j = 0; j < NW; ++j) {
        if (i + j < nwin) {
          const cplx_d f = fc[i + j];
          double sr = 0.0, si = 0.0, gr = 0.0, gi = 0.0;
#pragma unroll
          for (int r = 0; r < NR; ++r) {
            const double vr = q[j][r].x, vi = q[j][r].y;
            zr[r] -= f.re * vr - f.im * vi;
            zi[r] -= f.re * vi + f.im * vr;
            // p and Hp stay in their own precision: converted once, ahead of the loop,
            // complex64 pairs would take 16 registers more and spill
            if constexpr (sizeof(R) == 4)
              asm("" : "+v"(yo[r].x), "+v"(yo[r].y), "+v"(xo[r].x), "+v"(xo[r].y));
            const double yr = yo[r].x, yi = yo[r].y, xr = xo[r].x, xi = xo[r].y;
            sr += vr * yr + vi * yi;
            si += vr * yi - vi * yr;
            gr += vr * xr + vi * xi;
            gi += vr * xi - vi * xr;
          }
          add_quad(i + j, quad_sums(sr, si, gr, gi));
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    // store w; its overlap with v_{b+1} and its norm from the stored (rounded) values
    V o[NR];
    double sr = 0.0, si = 0.0, nn = 0.0;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      o[r].x = (R)zr[r];
      o[r].y = (R)zi[r];
      const double vr = xo[r].x, vi = xo[r].y, wr = o[r].x, wi = o[r].y;
      sr += vr * wr + vi * wi;
      si += vr * wi - vi * wr;
      nn += wr * wr + wi * wi;
    }
    bstore<MODE, RB>(out, base, lane, wv, D, o);
    const double t = quad_sums(sr, si, nn, 0.0);
    if (lane < 2u) {
      cplx_d& d = wrow[nb - 1];
      if (lane & 1u) {
        d.im += t;
      } else {
        d.re += t;
      }
    } else if (lane == 2u) {
      wrow[2 * nb].re += t;
    }
  }
  __syncthreads();
  block_totals(wacc, 2 * nb + 1, tot);
  for (int j = threadIdx.x; j < 2 * nb; j += blockDim.x) a.partials[(size_t)j * kPartialRows + bl] = tot[j];
  if (threadIdx.x == 0) a.partials[(size_t)kNormCol * kPartialRows + bl] = cplx_d{tot[2 * nb].re, 0.0};
}

template <typename R, int RB, int MODE, int NW, bool NT = false>
__global__ void __launch_bounds__(RB >= 3 ? 512 : 1024) k_pass_p(LzBatch B) {
  const uint32_t G = B.job[0].geo.grid;
  if (blockIdx.x < G) {
    pass_p_body<R, RB, MODE, NW, NT>(B.job[0], blockIdx.x, G);
  } else {
    pass_p_body<R, RB, MODE, NW, NT>(B.job[1], blockIdx.x - G, G);
  }
}

// The scalar update of the last step (alpha_{m-1}, or a breakdown there) and
// exp(-itT) e_1: one wavefront per Krylov call, writing the combination
// coefficients and m_eff to the state for k_combine.  A basis that ended in
// an earlier step (a breakdown found by a pass B) already has them.
__global__ void __launch_bounds__(64) k_finish(LzBatch B) {
  __shared__ cplx_d tot[kMaxScal];
  __shared__ FinScalars fs;
  const LzArgs& a = B.job[blockIdx.x];
  if (gather_step(a, a.geo.grid, 0, a.k == 0, fs, tot))
    step_update(a, fs, tot, 0, true, nullptr, nullptr, nullptr, nullptr);
}

// ---------------------------------------------------------------------- streaming kernels

constexpr int kStreamBlock = 256;
constexpr int kStreamUnroll = 4;

struct CombJob {
  const KState* st;
  const void* slot0;
  const void* basis;
  void* out;
  int32_t* m_eff_out;
};

struct CombBatch {
  CombJob job[kMaxJobs];
  uint32_t D;
  uint32_t grid;  // blocks per job
};

// One chunk of the combination: kStreamUnroll elements per thread, spaced `stride`
// apart from s0.  FULL: every element exists, so no load or store is masked (kept
// apart from the masked form so that the two never share a load's registers).
template <typename R, bool FULL, bool NT = false>
__device__ __forceinline__ void combine_chunk(const typename VT<R>::T* __restrict__ slot0,
                                              const typename VT<R>::T* __restrict__ basis,
                                              typename VT<R>::T* __restrict__ out, const cplx_d* cs,
                                              int me, uint32_t s0, uint32_t stride, uint32_t D) {
  using V = typename VT<R>::T;
  constexpr int NJ = 4;  // basis vectors per round trip
  double ar[kStreamUnroll], ai[kStreamUnroll];
#pragma unroll
  for (int q = 0; q < kStreamUnroll; ++q) {
    ar[q] = 0.0;
    ai[q] = 0.0;
  }
  for (int j0 = 0; j0 < me; j0 += NJ) {
    V v[NJ][kStreamUnroll];
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
      const int j = j0 + jj;
      if (j < me) {
        const V* vj = (j == 0) ? slot0 : basis + (size_t)(j - 1) * D;
#pragma unroll
        for (int q = 0; q < kStreamUnroll; ++q) {
          const uint32_t s = s0 + q * stride;
          v[jj][q] = FULL ? (NT ? ld_stream(vj + s) : vj[s]) : ld_masked(vj, s, s < D);
        }
      }
    }
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
      const int j = j0 + jj;
      if (j < me) {
        const cplx_d c = cs[j];
#pragma unroll
        for (int q = 0; q < kStreamUnroll; ++q) {
          const double vr = v[jj][q].x, vi = v[jj][q].y;
          ar[q] += c.re * vr - c.im * vi;
          ai[q] += c.re * vi + c.im * vr;
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < kStreamUnroll; ++q) {
    const uint32_t s = s0 + q * stride;
    if (FULL || s < D) {
      V o;
      o.x = (R)ar[q];
      o.y = (R)ai[q];
      out[s] = o;
    }
  }
}

template <typename R, bool NT = false>
__device__ __forceinline__ void combine_body(const CombJob& cj, uint32_t D, uint32_t bl, uint32_t G) {
  using V = typename VT<R>::T;
  __shared__ cplx_d cs[kMaxM];
  const KState* __restrict__ st = cj.st;
  const V* slot0 = reinterpret_cast<const V*>(cj.slot0);
  const V* basis = reinterpret_cast<const V*>(cj.basis);
  V* out = reinterpret_cast<V*>(cj.out);
  const int me = st->m_eff;
  // the coefficients once per block, so that the streaming loop waits on vector loads only
  if ((int)threadIdx.x < me) cs[threadIdx.x] = st->dcomb[threadIdx.x];
  __syncthreads();
  const uint32_t stride = G * kStreamBlock;
  for (uint32_t c0 = bl * kStreamBlock; c0 < D; c0 += stride * kStreamUnroll) {
    // block-uniform: every element of the block's chunk exists
    if (c0 + (kStreamBlock - 1) + (kStreamUnroll - 1) * stride < D) {
      combine_chunk<R, true, NT>(slot0, basis, out, cs, me, c0 + threadIdx.x, stride, D);
    } else {
      combine_chunk<R, false>(slot0, basis, out, cs, me, c0 + threadIdx.x, stride, D);
    }
  }
  if (cj.m_eff_out && bl == 0 && threadIdx.x == 0) *cj.m_eff_out = me;
}

template <typename R, bool NT = false>
__global__ void __launch_bounds__(kStreamBlock) k_combine(CombBatch B) {
  if (blockIdx.x < B.grid) {
    combine_body<R, NT>(B.job[0], B.D, blockIdx.x, B.grid);
  } else {
    combine_body<R, NT>(B.job[1], B.D, blockIdx.x - B.grid, B.grid);
  }
}

// Elements per thread and round trip of the reducing streaming kernels.
template <typename R>
struct RedChunk {
  static constexpr int n = (sizeof(R) == 4) ? 16 : 8;
};

// beta = <f|psi> (Eq. 2); the last block writes beta, F = |beta|^2.
template <typename R>
__global__ void __launch_bounds__(kStreamBlock)
    k_overlap(uint32_t D, const typename VT<R>::T* __restrict__ f, const typename VT<R>::T* __restrict__ psi,
              KState* st, cplx_d* partials, double* F_dev, double* beta_dev) {
  using V = typename VT<R>::T;
  constexpr int E = RedChunk<R>::n;
  __shared__ cplx_d wacc[(kStreamBlock / 64) * kMaxScal];
  __shared__ cplx_d tot[kMaxScal];
  const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
  const uint32_t T = gridDim.x * kStreamBlock;
  const uint32_t tid = blockIdx.x * kStreamBlock + threadIdx.x;
  double sr = 0.0, si = 0.0;
  for (uint32_t base = 0; base < D; base += T * E) {
    V a[E], b[E];
    if (base + E * T <= D) {  // the whole chunk exists (block-uniform test)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        a[e] = f[base + e * T + tid];
        b[e] = psi[base + e * T + tid];
      }
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const uint32_t s = base + e * T + tid;
        a[e] = ld_masked(f, s, s < D);
        b[e] = ld_masked(psi, s, s < D);
      }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const double fr = a[e].x, fi = a[e].y, pr = b[e].x, pi = b[e].y;
      sr += fr * pr + fi * pi;
      si += fr * pi - fi * pr;
    }
  }
  sr = wave_sum(sr);
  si = wave_sum(si);
  if (lane == 0) wacc[wv * kMaxScal] = cplx_d{sr, si};
  __syncthreads();
  block_totals(wacc, 1, tot);
  if (!grid_reduce(tot, 1, partials, st->counters, blockIdx.x, gridDim.x)) return;
  if (threadIdx.x == 0) {
    const cplx_d b = tot[0];
    st->overlap = b;
    st->fid = b.re * b.re + b.im * b.im;
    if (beta_dev) {
      beta_dev[0] = b.re;
      beta_dev[1] = b.im;
    }
    if (F_dev) *F_dev = b.re * b.re + b.im * b.im;
  }
}

// This thread's share of <lambda|Hc|psi>; with `keep` psi is also copied there
// (lambda's amplitudes are read first, by the same thread, so keep may be lam).
template <typename R>
__device__ __forceinline__ void bracket_sum(const HvArgs& a, uint32_t D, const typename VT<R>::T* lam,
                                            const typename VT<R>::T* __restrict__ psi,
                                            typename VT<R>::T* keep,
                                            const uint32_t* __restrict__ pe_reps, uint32_t T, uint32_t tid,
                                            double& sr, double& si) {
  using V = typename VT<R>::T;
  constexpr int E = RedChunk<R>::n;
  const uint32_t flip = (a.hc_kind == 0) ? (1u << a.hc_bit) : 0u;
  sr = si = 0.0;
  for (uint32_t base = 0; base < D; base += T * E) {
    V l[E], p[E];
    if (base + E * T <= D) {  // the whole chunk exists (block-uniform test)
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const uint32_t s = base + e * T + tid;
        l[e] = lam[s];
        p[e] = psi[s ^ flip];
      }
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const uint32_t s = base + e * T + tid;
        l[e] = ld_masked(lam, s, s < D);
        p[e] = ld_masked(psi, s ^ flip, s < D);
      }
    }
    if (keep) {
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const uint32_t s = base + e * T + tid;
        if (s < D) keep[s] = psi[s];
      }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const uint32_t s = base + e * T + tid;
      // (Hc psi)[s]: S^x flips one bit with amplitude 1/2; sum of S^z is diagonal
      // (in the reduced basis, of the orbit label's bit pattern)
      const uint32_t pat = pe_reps ? pe_reps[s < D ? s : 0u] : s;
      const double hc = (a.hc_kind == 0) ? 0.5 : 0.5 * a.sz_count - (double)__popc(pat & a.sz_mask);
      const double pr = hc * (double)p[e].x, pi = hc * (double)p[e].y;
      const double lr = l[e].x, li = l[e].y;
      sr += lr * pr + li * pi;
      si += lr * pi - li * pr;
    }
  }
}

// g_j = 2 Im(conj(beta) c <lambda|Hc|psi>) with c = (cr, ci); c = dt gives Eq. 5
// (chi = beta lambda, sign of dF).  Written to *grad_slot, or added to it with
// `accumulate` (quadrature nodes, hierarchy terms).
template <typename R>
__global__ void __launch_bounds__(kStreamBlock)
    k_bracket(HvArgs a, uint32_t D, const typename VT<R>::T* __restrict__ lam,
              const typename VT<R>::T* __restrict__ psi, double cr, double ci,
              const double* beta_dev, KState* st, cplx_d* partials, double* grad_slot,
              int accumulate, const uint32_t* __restrict__ pe_reps) {
  __shared__ cplx_d wacc[(kStreamBlock / 64) * kMaxScal];
  __shared__ cplx_d tot[kMaxScal];
  const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
  const uint32_t T = gridDim.x * kStreamBlock;
  const uint32_t tid = blockIdx.x * kStreamBlock + threadIdx.x;
  double sr, si;
  bracket_sum<R>(a, D, lam, psi, nullptr, pe_reps, T, tid, sr, si);
  sr = wave_sum(sr);
  si = wave_sum(si);
  if (lane == 0) wacc[wv * kMaxScal] = cplx_d{sr, si};
  __syncthreads();
  block_totals(wacc, 1, tot);
  if (!grid_reduce(tot, 1, partials, st->counters, blockIdx.x, gridDim.x)) return;
  if (threadIdx.x == 0) {
    const double br = beta_dev[0], bi = beta_dev[1];
    const cplx_d B = tot[0];
    double g;
    if (ci == 0.0) {
      g = 2.0 * cr * (br * B.im - bi * B.re);
    } else {
      const double zr = cr * B.re - ci * B.im, zi = cr * B.im + ci * B.re;
      g = 2.0 * (br * zi - bi * zr);
    }
    *grad_slot = accumulate ? *grad_slot + g : g;
  }
}

// The bracket <lambda|Hc|psi> itself, of one or two pairs of vectors
// (blockIdx.y).
template <typename R>
__global__ void __launch_bounds__(kStreamBlock) k_bracket_raw(HvArgs a, uint32_t D, RawBracketPair p,
                                                              const uint32_t* __restrict__ pe_reps) {
  using V = typename VT<R>::T;
  __shared__ cplx_d wacc[(kStreamBlock / 64) * kMaxScal];
  __shared__ cplx_d tot[kMaxScal];
  const RawBracket& q = p.job[blockIdx.y];
  const uint32_t lane = threadIdx.x & 63u, wv = threadIdx.x >> 6;
  const uint32_t T = gridDim.x * kStreamBlock;
  const uint32_t tid = blockIdx.x * kStreamBlock + threadIdx.x;
  double sr, si;
  bracket_sum<R>(a, D, reinterpret_cast<const V*>(q.lam), reinterpret_cast<const V*>(q.psi),
                 reinterpret_cast<V*>(q.keep), pe_reps, T, tid, sr, si);
  sr = wave_sum(sr);
  si = wave_sum(si);
  if (lane == 0) wacc[wv * kMaxScal] = cplx_d{sr, si};
  __syncthreads();
  block_totals(wacc, 1, tot);
  if (!grid_reduce(tot, 1, q.partials, q.st->counters, blockIdx.x, gridDim.x)) return;
  if (threadIdx.x == 0) *q.out = tot[0];
}

// The brackets' share of the gradient once beta is known (k_bracket's formula).
__global__ void __launch_bounds__(256)
    k_scale_brackets(const cplx_d* raw, int n, double c, const double* beta, double* g, int accumulate) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const cplx_d B = raw[i];
  const double v = 2.0 * c * (beta[0] * B.im - beta[1] * B.re);
  g[i] = accumulate ? g[i] + v : v;
}

// u <- u + eta g / max|g| in one block (deterministic max).
__global__ void __launch_bounds__(1024) k_ascent(double* u, const double* g, int N, double eta) {
  __shared__ double wmax[16];
  double m = 0.0;
  for (int j = threadIdx.x; j < N; j += blockDim.x) m = fmax(m, fabs(g[j]));
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
  __syncthreads();
  double gm = 0.0;
  for (int q = 0; q < (int)(blockDim.x >> 6); ++q) gm = fmax(gm, wmax[q]);
  if (gm == 0.0) return;
  const double f = eta / gm;
  for (int j = threadIdx.x; j < N; j += blockDim.x) u[j] += f * g[j];
}

// Centred gradient from the end-point brackets, in place: on entry g[j-1] holds
// the bracket at the end of slice j (j = 1..N) and *g0 the one at the start of
// slice 1; on exit g[j-1] = (bracket at the start + bracket at the end) / 2.
// One block walks the array from the top, 1024 entries at a time: every
// thread reads its two inputs before any thread of the chunk writes, and the
// chunk below has not been written yet.
__global__ void __launch_bounds__(1024) k_centre(double* g, int N, const double* g0) {
  for (int top = N; top > 0; top -= (int)blockDim.x) {
    const int j = top - 1 - (int)threadIdx.x;   // 0-based slice index
    double mid = 0.0;
    if (j >= 0) {
      const double lo = (j == 0) ? *g0 : g[j - 1];
      mid = 0.5 * (lo + g[j]);
    }
    __syncthreads();
    if (j >= 0) g[j] = mid;
    __syncthreads();
  }
}

// beta = (1/n) sum_c beta_c (columns in order, one thread: deterministic), F = |beta|^2
__global__ void k_mean_overlap(const double* beta_cols, int n, double* beta, double* F) {
  if (threadIdx.x != 0) return;
  double re = 0.0, im = 0.0;
  for (int c = 0; c < n; ++c) {
    re += beta_cols[2 * c];
    im += beta_cols[2 * c + 1];
  }
  re /= n;
  im /= n;
  beta[0] = re;
  beta[1] = im;
  if (F) *F = re * re + im * im;
}

__global__ void k_index_map(int L, uint32_t s0, uint32_t count, int32_t* n_anti, uint32_t* pmask) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const uint32_t s = s0 + i;
  const uint32_t m = (s ^ (s >> 1)) & ((1u << (L - 1)) - 1u);
  n_anti[i] = __popc(m);
  pmask[i] = m;
}

__global__ void k_init_state(KState* st) {
  const int i = threadIdx.x;
  if (i < kMaxGrid / 64 + 4) st->counters[i] = 0u;
  if (i == 0) {
    st->done = 0;
    st->m_eff = 0;
    st->normT[0] = 0.0;
    st->normT[1] = 0.0;
  }
}

// ---------------------------------------------------------------------- launch helpers

template <typename R>
size_t lds_bytes(const Geo& g) {
  const size_t tile = ((size_t)1 << g.TB) * sizeof(typename VT<R>::T);
  const size_t red = ((size_t)1 << g.WB) * kMaxScal * sizeof(cplx_d);
  return tile > red ? tile : red;
}

template <typename R, int RB>
hipError_t launch_hv_t(const HvArgs& a, const Geo& g, const void* v, void* w, hipStream_t s) {
  using V = typename VT<R>::T;
  // complex64 whole tiles in pairs when both vectors are 16-byte aligned
  const bool pairs = sizeof(R) == 4 && RB >= 2 && pairs_tiling(g) &&
                     (((uintptr_t)v | (uintptr_t)w) % 16) == 0;
  if constexpr (sizeof(R) == 4 && RB >= 2) {
    if (pairs) {
      kg_launch((k_hv<R, RB, true>), dim3(g.grid), dim3(64 << g.WB), lds_bytes<R>(g), s, a,
                         g, reinterpret_cast<const V*>(v), reinterpret_cast<V*>(w));
      return hipGetLastError();
    }
  }
  kg_launch((k_hv<R, RB>), dim3(g.grid), dim3(64 << g.WB), lds_bytes<R>(g), s, a, g,
                     reinterpret_cast<const V*>(v), reinterpret_cast<V*>(w));
  return hipGetLastError();
}

template <typename R>
hipError_t launch_hv_pe_t(const HvArgs& a, const PeArgs& p, const void* v, void* w, hipStream_t s) {
  using V = typename VT<R>::T;
  if (p.nbr) {
    // one slice per wavefront: blocks of eight (the L=25, K=12 centred
    // gradient 629 -> 624 ms against blocks of four, the gather alone the
    // same), a multiple of 8 blocks for the XCD split
    const uint32_t ns = (p.dim + 63u) >> 6;
    uint32_t blocks = ((ns + 7u) / 8u + 7u) & ~7u;
    if (blocks < 64u) blocks = (ns + 7u) / 8u;
    kg_launch((k_hv_pe_nbr<R>), dim3(blocks), dim3(512), 0, s, a, p, reinterpret_cast<const V*>(v),
              reinterpret_cast<V*>(w));
    return hipGetLastError();
  }
  uint32_t blocks = (p.dim + 255u) / 256u;
  // grid-stride beyond 8192 blocks (the binomials are staged per block); at
  // 2.6 million rows 8192 blocks were 6 % faster than 2048
  if (blocks > 8192u) blocks = 8192u;
  if (blocks < 1u) blocks = 1u;
  if (blocks >= 64u) blocks = (blocks + 7u) & ~7u;
  kg_launch((k_hv_pe<R>), dim3(blocks), dim3(256), 0, s, a, p, reinterpret_cast<const V*>(v),
                     reinterpret_cast<V*>(w));
  return hipGetLastError();
}

template <typename R>
hipError_t launch_hv_r(const HvArgs& a, const Geo& g, const void* v, void* w, hipStream_t s) {
  switch (g.RB) {
    case 0: return launch_hv_t<R, 0>(a, g, v, w, s);
    case 1: return launch_hv_t<R, 1>(a, g, v, w, s);
    case 2: return launch_hv_t<R, 2>(a, g, v, w, s);
    default: return launch_hv_t<R, 3>(a, g, v, w, s);
  }
}

// The launches of a Lanczos step: pass A, pass B, or a pair's pass C and pass P.
enum Pass { kPassA, kPassB, kPassC, kPassP };

template <typename R, int RB, int MODE, bool NT>
hipError_t launch_stream_pass(Pass which, const LzBatch& lb, int njobs, hipStream_t s) {
  const Geo& g = lb.job[0].geo;
  const dim3 grid(g.grid * njobs), block(64 << g.WB);
  // window vectors per round trip: 32 bytes a thread, two complex64 vectors at the
  // 2^11 tiles (one: L=22, m=20 1751 -> 1770 us, L=23 3476 -> 3543, L=20 the same;
  // four spill)
  constexpr int units = 8 / ((1 << RB) * (int)(sizeof(R) / 4));
  constexpr int NW = units < 1 ? 1 : units;
  const size_t red = ((size_t)1 << g.WB) * kMaxScal * sizeof(cplx_d);
  if (which == kPassB) {
    kg_launch((k_pass_b<R, RB, MODE, NT>), grid, block, red, s, lb);
  } else if (which == kPassC) {
    kg_launch((k_pass_c<R, RB, MODE, NW, NT>), grid, block, 3 * sizeof(double) << g.WB, s, lb);
  } else {
    kg_launch((k_pass_p<R, RB, MODE, NW, NT>), grid, block, red, s, lb);
  }
  return hipGetLastError();
}

template <typename R, int RB>
hipError_t launch_pass(Pass which, const LzBatch& lb, int njobs, hipStream_t s) {
  const Geo& g = lb.job[0].geo;
  const dim3 grid(g.grid * njobs), block(64 << g.WB);
  if (which == kPassA) {
    bool pairs = sizeof(R) == 4 && RB >= 2 && pairs_tiling(g);
    for (int j = 0; j < njobs; ++j) {
      const LzArgs& q = lb.job[j];
      if (((uintptr_t)q.slot0 | (uintptr_t)q.basis | (uintptr_t)q.yk) % 16) pairs = false;
    }
    if constexpr (sizeof(R) == 4 && RB >= 2) {
      if (pairs) {
        kg_launch((k_pass_a<R, RB, true>), grid, block, lds_bytes<R>(g), s, lb);
        return hipGetLastError();
      }
    }
    kg_launch((k_pass_a<R, RB>), grid, block, lds_bytes<R>(g), s, lb);
  } else {
    // 16-byte pairs need whole tiles and 16-byte aligned vectors (the boundary
    // requires the alignment; checked again here, since a misaligned pair is
    // not an option)
    bool pairs = sizeof(R) == 4 && RB >= 1 && !g.small;
    for (int j = 0; j < njobs; ++j) {
      const LzArgs& q = lb.job[j];
      if (((uintptr_t)q.slot0 | (uintptr_t)q.basis | (uintptr_t)q.yk) % 16) pairs = false;
    }
    // a basis larger than the Infinity Cache is streamed with nontemporal loads
    const bool nt = streamed_past_cache(lb.job[0].m, g.D, sizeof(typename VT<R>::T));
    constexpr int PM = (sizeof(R) == 4 && RB >= 1) ? kBPairs : kBSlots;
    if (g.small) return launch_stream_pass<R, RB, kBMasked, false>(which, lb, njobs, s);
    if (pairs)
      return nt ? launch_stream_pass<R, RB, PM, true>(which, lb, njobs, s)
                : launch_stream_pass<R, RB, PM, false>(which, lb, njobs, s);
    return nt ? launch_stream_pass<R, RB, kBSlots, true>(which, lb, njobs, s)
              : launch_stream_pass<R, RB, kBSlots, false>(which, lb, njobs, s);
  }
  return hipGetLastError();
}

template <typename R>
hipError_t launch_pass_r(Pass which, const LzBatch& lb, int njobs, hipStream_t s) {
  switch (lb.job[0].geo.RB) {
    case 0: return launch_pass<R, 0>(which, lb, njobs, s);
    case 1: return launch_pass<R, 1>(which, lb, njobs, s);
    case 2: return launch_pass<R, 2>(which, lb, njobs, s);
    default: return launch_pass<R, 3>(which, lb, njobs, s);
  }
}

// Advance n (1 or 2) independent Krylov calls of one shape (same L, m,
// reorth, precision) through the same launches.
template <typename R>
hipError_t launch_krylov_t(const KrylovCall* calls, const Workspace* const* wss, int n, hipStream_t s) {
  using V = typename VT<R>::T;
  const KrylovCall& c0 = calls[0];
  if (sweep_applies(c0)) {
    SweepJob jobs[kMaxJobs];
    for (int j = 0; j < n; ++j) jobs[j] = sweep_job(calls[j]);
    return launch_sweeps(c0.prec, jobs, n, s);
  }
  // one launch per step; vectors that fit the one-block form but do not take it (the
  // passes are forced, or more neighbours than it holds) have no room for the steps
  const bool steps = c0.geo.D <= kStepMaxD && (!c0.pe || c0.pe->nbr) && !passes_forced();
  if (steps && !sweep_fits(c0.prec, c0.geo.D, c0.m, 0)) {
    KrylovCall c[kMaxJobs];
    for (int j = 0; j < n; ++j) {
      c[j] = calls[j];
      c[j].step = c0.pe ? make_geo_step_pe(c0.hv.L, c0.geo.D)
                        : make_geo_step(c0.hv.L);
    }
    return launch_krylov_steps(c, wss, n, s);
  }
  LzBatch lb;
  CombBatch cb;
  memset(&lb, 0, sizeof(lb));
  memset(&cb, 0, sizeof(cb));
  for (int j = 0; j < n; ++j) {
    LzArgs& la = lb.job[j];
    la.hv = calls[j].hv;
    la.geo = calls[j].geo;
    la.slot0 = calls[j].v_in;
    la.basis = wss[j]->basis;
    la.yk = wss[j]->yk;
    la.m = calls[j].m;
    la.t = calls[j].t;
    la.tol = calls[j].tol;
    la.st = wss[j]->st;
    la.partials = wss[j]->partials;
    cb.job[j] = CombJob{wss[j]->st, calls[j].v_in, wss[j]->basis, calls[j].v_out, calls[j].m_eff_out};
  }
  Profiler* prof = profiler_for_call();
  const double vb = (double)c0.geo.D * sizeof(V) * n;
  hipError_t e;
  // windows: all stored vectors (full re-orthogonalisation) or the last two;
  // the last step only forms alpha
  int i0p = 0;
  // full windows two steps at a time, whatever m; an even m leaves the first step by
  // itself (against a pass B per step, both timed, m = 4 / 8 / 24: complex64 L=20 81 -> 80,
  // 184 -> 169, 783 -> 619 us; complex128 L=22 442 -> 438, 1125 -> 1068, 5361 -> 4210)
  const bool paired = c0.reorth != 0;
  const int first = (c0.m - 1) & 1;
  for (int k = 0; k < c0.m; ++k) {
    const bool last = (k == c0.m - 1);
    const Pass second = !paired ? kPassB : (k < first || !((k - first) & 1)) ? kPassC : kPassP;
    // pass A sums the measurements that pass C reads; pass P needs none
    const int i0 = (last || second == kPassP) ? k : (c0.reorth ? 0 : (k > 0 ? k - 1 : 0));
    const int i0n = (k + 1 == c0.m - 1) ? k + 1 : (c0.reorth ? 0 : k);
    for (int j = 0; j < n; ++j) {
      lb.job[j].k = k;
      lb.job[j].i0 = i0;
      lb.job[j].i0n = i0n;
      lb.job[j].i0p = paired ? 0 : i0p;
      lb.job[j].alone = k < first;
    }
    i0p = i0;
    if (c0.pe) {
      // reduced basis: y = H v_k by the gather kernel, then pass A on the given y
      for (int j = 0; j < n; ++j) {
        const char* xk = (k == 0) ? static_cast<const char*>(calls[j].v_in)
                                  : static_cast<const char*>(wss[j]->basis) +
                                        (size_t)(k - 1) * c0.geo.D * sizeof(V);
        void* yk = wss[j]->yk;
        if (prof) profiler_start(prof, s);
        if ((e = launch_hv_pe_t<R>(lb.job[j].hv, *calls[j].pe, xk, yk, s)) != hipSuccess)
          return e;
        if (prof) profiler_stop(prof, s, kProfHv, pe_gather_bytes(*calls[j].pe, vb / n));
      }
    }
    if (prof) profiler_start(prof, s);
    if (c0.pe) {
      const Geo& g = c0.geo;
      const size_t red = ((size_t)1 << g.WB) * kMaxScal * sizeof(cplx_d);
      kg_launch((k_pass_a_y<R>), dim3(g.grid * n), dim3(64 << g.WB), red, s, lb);
      if ((e = hipGetLastError()) != hipSuccess) return e;
    } else if ((e = launch_pass_r<R>(kPassA, lb, n, s)) != hipSuccess) {
      return e;
    }
    // algorithmic bytes: v_k is read and y = H v_k is written (not in the
    // last step; the reduced basis reads the given y instead)
    if (prof) profiler_stop(prof, s, kProfPassA, (1 + ((last && !c0.pe) ? 0 : 1)) * vb);
    if (!last) {
      if (prof) profiler_start(prof, s);
      if ((e = launch_pass_r<R>(second, lb, n, s)) != hipSuccess) return e;
      // pass B: y_k and the window are read, v_{k+1} is written; pass C: y, v_k and
      // v_{k-1} (the window too where p is projected); pass P: y, p and the window
      const int moved = second == kPassC ? (k > 0 ? 4 : 3)
                        : second == kPassP ? k + 3 : k - i0 + 3;
      if (prof) profiler_stop(prof, s, kProfPassB, moved * vb);
    }
  }
  // the last step's scalar update and the small exponential
  hipLaunchKernelGGL(k_finish, dim3(n), dim3(64), 0, s, lb);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const uint32_t D = c0.geo.D;
  cb.D = D;
  cb.grid = (uint32_t)stream_grid(D);
  if (prof) profiler_start(prof, s);
  if (streamed_past_cache(c0.m, D, sizeof(V)))
    kg_launch((k_combine<R, true>), dim3(cb.grid * n), dim3(kStreamBlock), 0, s, cb);
  else
    kg_launch((k_combine<R>), dim3(cb.grid * n), dim3(kStreamBlock), 0, s, cb);
  e = hipGetLastError();
  // m basis vectors read (fewer after a breakdown), v_out written
  if (prof) profiler_stop(prof, s, kProfCombine, (c0.m + 1) * vb);
  return e;
}

}  // namespace

// ---------------------------------------------------------------------- public launchers

int stream_grid(uint32_t D) {
  const uint64_t per = (uint64_t)kStreamBlock * kStreamUnroll;
  uint64_t g = (D + per - 1) / per;
  if (g < 1) g = 1;
  if (g > (uint64_t)kMaxGrid) g = kMaxGrid;
  return (int)g;
}

hipError_t launch_init(KState* st, hipStream_t s) {
  hipLaunchKernelGGL(k_init_state, dim3(1), dim3(128), 0, s, st);
  return hipGetLastError();
}

hipError_t launch_hv(int prec, const HvArgs& a, const Geo& g, const void* v, void* w, hipStream_t s) {
  return prec == 0 ? launch_hv_r<double>(a, g, v, w, s) : launch_hv_r<float>(a, g, v, w, s);
}

hipError_t launch_hv_pe(int prec, const HvArgs& a, const PeArgs& p, const void* v, void* w,
                        hipStream_t s) {
  return prec == 0 ? launch_hv_pe_t<double>(a, p, v, w, s) : launch_hv_pe_t<float>(a, p, v, w, s);
}

hipError_t launch_krylov(const KrylovCall& c, const Workspace& ws, hipStream_t s) {
  const Workspace* w[1] = {&ws};
  return c.prec == 0 ? launch_krylov_t<double>(&c, w, 1, s) : launch_krylov_t<float>(&c, w, 1, s);
}

hipError_t launch_krylov_pair(const KrylovCall& c0, const Workspace& w0, const KrylovCall& c1,
                              const Workspace& w1, hipStream_t s) {
  const KrylovCall c[2] = {c0, c1};
  const Workspace* w[2] = {&w0, &w1};
  return c0.prec == 0 ? launch_krylov_t<double>(c, w, 2, s) : launch_krylov_t<float>(c, w, 2, s);
}

int reduce_grid(uint32_t D, int prec) {
  const uint64_t per = (uint64_t)kStreamBlock * (prec == 0 ? RedChunk<double>::n : RedChunk<float>::n);
  uint64_t g = (D + per - 1) / per;
  if (g < 1) g = 1;
  if (g > 256) g = 256;
  return (int)g;
}

hipError_t launch_overlap(int prec, uint32_t D, const void* f, const void* psi, const Workspace& ws,
                          double* F_dev, double* beta_dev, hipStream_t s) {
  const int grid = reduce_grid(D, prec);
  if (prec == 0) {
    kg_launch(k_overlap<double>, dim3(grid), dim3(kStreamBlock), 0, s, D,
                       reinterpret_cast<const double2*>(f), reinterpret_cast<const double2*>(psi),
                       ws.st, ws.partials, F_dev, beta_dev);
  } else {
    kg_launch(k_overlap<float>, dim3(grid), dim3(kStreamBlock), 0, s, D,
                       reinterpret_cast<const float2*>(f), reinterpret_cast<const float2*>(psi),
                       ws.st, ws.partials, F_dev, beta_dev);
  }
  return hipGetLastError();
}

hipError_t launch_bracket(int prec, const HvArgs& a, uint32_t D, const void* lam, const void* psi,
                          double dt, const double* beta_dev, const Workspace& ws, double* grad_slot,
                          hipStream_t s, bool accumulate, double coef_im,
                          const uint32_t* pe_reps) {
  const int grid = reduce_grid(D, prec);
  const int acc = accumulate ? 1 : 0;
  if (prec == 0) {
    kg_launch(k_bracket<double>, dim3(grid), dim3(kStreamBlock), 0, s, a, D,
                       reinterpret_cast<const double2*>(lam), reinterpret_cast<const double2*>(psi),
                       dt, coef_im, beta_dev, ws.st, ws.partials, grad_slot, acc, pe_reps);
  } else {
    kg_launch(k_bracket<float>, dim3(grid), dim3(kStreamBlock), 0, s, a, D,
                       reinterpret_cast<const float2*>(lam), reinterpret_cast<const float2*>(psi),
                       dt, coef_im, beta_dev, ws.st, ws.partials, grad_slot, acc, pe_reps);
  }
  return hipGetLastError();
}

hipError_t launch_bracket_raw(int prec, const HvArgs& a, uint32_t D, const RawBracket* jobs, int n,
                              hipStream_t s, const uint32_t* pe_reps) {
  const int grid = reduce_grid(D, prec);
  RawBracketPair p;
  memset(static_cast<void*>(&p), 0, sizeof(p));
  for (int i = 0; i < n; ++i) p.job[i] = jobs[i];
  if (prec == 0)
    kg_launch(k_bracket_raw<double>, dim3(grid, n), dim3(kStreamBlock), 0, s, a, D, p, pe_reps);
  else
    kg_launch(k_bracket_raw<float>, dim3(grid, n), dim3(kStreamBlock), 0, s, a, D, p, pe_reps);
  return hipGetLastError();
}

hipError_t launch_scale_brackets(const cplx_d* raw, int n, double c, const double* beta, double* g,
                                 bool accumulate, hipStream_t s) {
  hipLaunchKernelGGL(k_scale_brackets, dim3((n + 255) / 256), dim3(256), 0, s, raw, n, c, beta, g,
                     accumulate ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_ascent(double* u, const double* g, int N, double eta, hipStream_t s) {
  hipLaunchKernelGGL(k_ascent, dim3(1), dim3(1024), 0, s, u, g, N, eta);
  return hipGetLastError();
}

hipError_t launch_centre(double* g, int N, const double* g0, hipStream_t s) {
  hipLaunchKernelGGL(k_centre, dim3(1), dim3(1024), 0, s, g, N, g0);
  return hipGetLastError();
}

hipError_t launch_mean_overlap(const double* beta_cols, int n, double* beta, double* F,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_mean_overlap, dim3(1), dim3(64), 0, s, beta_cols, n, beta, F);
  return hipGetLastError();
}

hipError_t launch_index_map(int L, uint32_t s0, uint32_t count, int32_t* n_anti, uint32_t* pmask,
                            hipStream_t s) {
  const uint32_t blocks = (count + 255) / 256;
  hipLaunchKernelGGL(k_index_map, dim3(blocks), dim3(256), 0, s, L, s0, count, n_anti, pmask);
  return hipGetLastError();
}

}  // namespace kg
