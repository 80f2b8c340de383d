// fit_kernels.h -- kernels of the fixed-lambda fit and the lambda path
// (Sec. 2: Lemma 1 per (j, k) segment, Algorithm 1 objective and argmin).
#pragma once

#include "device_common.h"

#include <l1line.h>

enum : int {
  COL_NONFINITE = 1,   // a NaN or an infinity in the column
  COL_WIDE = 2,        // nonzero magnitudes too spread for 128-bit sums
};

enum : int {
  SEG_INTERNAL = 1,    // a selection exceeded its round bound
};

struct ColInfo {
  u128 wfix;    // exact sum of |x_ij| / 2^e0 over the column
  double W;     // R64 sum of |x_ij| (column mass)
  int e0;       // exponent of the lowest set bit over nonzero |x_ij|
  int nnz;      // nonzeros
  int zeros;    // exact zeros
  int flags;    // COL_*
  int bemin;    // smallest biased exponent field over nonzero entries
  int bemax;    // largest biased exponent field over nonzero entries
  double unit;  // the weights are whole multiples of it and their FP64 sums safe (column_unit), or 0
};

// One problem of a batch, as the kernels see it.  Workspace offsets are in
// elements of the batch-wide arrays.
struct ProbDesc {
  const double *X;      // n x m, column-major
  long long ld;
  int n, m, L;
  int lam_off;          // first penalty in the flat penalty array
  int col_off;          // first column in ColInfo / segflags
  int out_off;          // first (problem, lambda) slot: sum of L over earlier problems
  long long ws_off;     // first element of this problem's L*m*m block in V / E / R
  long long z_off;      // first element of this problem's L*m block in Z / zflag
  long long pair_off;   // first element of this problem's m*m block of sign sums
  long long mask_off;   // first word of this problem's zero-segment mask (mj ceil(m / 64) words)
  double *Vout;         // L*m
  long long *Jout;      // L
  double *OBJout;       // L
  int *ROWout;          // L*m or null
  double *ZALLout;      // L*m or null
  int *status;          // 1 or null
};

// A workgroup's unit of work: problem b, preserved column j, k in [kbeg, kend).
struct WorkItem {
  int b, j, kbeg, kend;
};

// first index i in [0, count) with prefix[i + 1] > g (prefix has count + 1 entries)
__device__ __forceinline__ int find_owner(const int *__restrict__ prefix, int count, long long g) {
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (prefix[mid] <= g) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// ------------------------------------------------------------------ columns
constexpr int SAMPLE_ROWS = 128;    // rows of column j drawn for the key windows

// A unit of a column's weights in which sums of them come out near enough to
// tell whole numbers apart: 2^e0 for weights with a sum below 2^50 of them (whole
// numbers: every FP64 sum is exact), or the magnitude that all its nonzeros share
// (two-valued data: a sum of n <= 65535 equal weights is off by less than 2^-20
// of one); else 0.  amin, amax: least and largest nonzero magnitude.
__device__ __forceinline__ double column_unit(u128 wfix, int e0, int nnz, double amin, double amax) {
  if (nnz == 0) return 1.0;
  if (amin >= 0x1p-300 && wfix < ((u128)1 << 50)) return ldexp(1.0, e0);
  return amin == amax && amin >= 0x1p-900 && amax <= 0x1p900 ? amin : 0.0;
}

// One workgroup of kW waves per column: finiteness, counts, the fixed-point
// exponent e0, the range check, the exact fixed-point mass, the R64 column
// mass and (smp not null) a systematic sample of SAMPLE_ROWS rows with
// probability ~ |x_ij|.  The exponent e0 and the mass are needed before the
// exact sum and the sample, so the column is gone through twice.
//   kLds, 4 waves   up to PREP_LDS_MAX rows: the column stays in LDS between
//   4 waves         longer columns, too few to fill the chip with one wave
//                   each: a wave takes a quarter of the 64-row slots, wave 0
//                   also the R64 mass (its order is one chain of adds a lane)
//   1 wave          many columns: the four-wave form's extra pass and
//                   reductions cost more than they hide
// (one wave per column and one load in flight before, and no sample: 2000 x
// 2000 32 us, now 23; 20011 x 151 212 us, now 83; 10000 x 4000 213 us, now 146)
// The sample's cumulative weight runs wave by wave and lane by lane (a lane's
// rows in turn, from the scan of the lanes' masses): sample r is the row whose
// weight interval holds (r + 1/2) step.  A row stores itself at its first
// sample only; the ones after it, and those that no row took (rounding), are
// filled in at the end from the nearest sample before, else from the column's
// first nonzero row (a store per sample was a serial loop where a few rows
// hold most of the weight: counts of up to 150 rows 14.9 us, now 5.5).  Any
// rows serve: they only place windows.
template <int CB, class F>
__device__ __forceinline__ void for_rows_batch(const double *__restrict__ x, int n, int i0, F f) {
  double v[CB];
#pragma unroll
  for (int q = 0; q < CB; ++q) v[q] = i0 + 64 * q < n ? gld(x + i0 + 64 * q) : 0.0;
#pragma unroll
  for (int q = 0; q < CB; ++q) f(v[q], i0 + 64 * q);
}
// the rows lane + 64 t, t in [t0, t1), of a column, loads 8 slots at a time
// (rows past n give 0)
template <class F>
__device__ __forceinline__ void for_rows(const double *__restrict__ x, int n, int t0, int t1, int lane, F f) {
  int t = t0;
  for (; t + 6 < t1; t += 8) for_rows_batch<8>(x, min(n, 64 * t1), 64 * t + lane, f);
  for (; t < t1; t += 2) for_rows_batch<2>(x, min(n, 64 * t1), 64 * t + lane, f);
}

constexpr int PREP_WAVES = 4, PREP_LDS_MAX = 4096;   // (a 32 KB copy leaves room for five workgroups per CU)
struct PrepShared {
  unsigned short smp[SAMPLE_ROWS];
  double mass[PREP_WAVES], amin[PREP_WAVES], amax[PREP_WAVES];
  int nbad[PREP_WAVES], nnz[PREP_WAVES], lsb[PREP_WAVES], first[PREP_WAVES];
  u128 fix[PREP_WAVES];
};

__device__ __forceinline__ double wave_min_dbl_x(double x) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) x = fmin(x, xswapd(x, d));
  return readlane_dbl(x, 0);
}
__device__ __forceinline__ double wave_max_dbl_x(double x) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) x = fmax(x, xswapd(x, d));
  return readlane_dbl(x, 0);
}

template <int kW, bool kLds>
__device__ __forceinline__ void colprep_block(const double *__restrict__ x, int n, ColInfo *__restrict__ out,
                                              unsigned short *__restrict__ smp, PrepShared &sh, double *col) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int T = (n + 63) >> 6, Tq = (T + kW - 1) / kW, t0 = min(T, wave * Tq), t1 = min(T, t0 + Tq);
  int nbad = 0, nnz = 0, lsb = 1 << 20, first = 1 << 30;
  double mine = 0.0, amin = __builtin_inf(), amax = 0.0;
  for_rows(x, n, t0, t1, lane, [&](double v, int i) {
    const double a = fabs(v);
    if (kLds && i < min(n, 64 * t1)) col[i] = a;
    mine = mine + a;
    const uint64_t ab = (uint64_t)__double_as_longlong(a);
    const uint32_t lo = (uint32_t)ab, hi = (uint32_t)(ab >> 32), be = hi >> 20;
    const bool fin = be != 0x7ff, nz = fin && ab != 0;
    nbad += fin ? 0 : 1;
    nnz += nz ? 1 : 0;
    // lowest set bit of the magnitude (the implicit bit included)
    const uint32_t hm = (hi & 0xFFFFFu) | (be ? 1u << 20 : 0u);
    const int tz = lo ? __builtin_ctz(lo) : 32 + __builtin_ctz(hm | (1u << 21));
    lsb = nz ? min(lsb, (int)max(be, 1u) - 1075 + tz) : lsb;
    first = nz ? min(first, i) : first;
    amin = nz ? fmin(amin, a) : amin;
    amax = nz ? fmax(amax, a) : amax;
  });
  const double scan = wave_incl_scan_dbl_x(mine, lane), all = readlane_dbl(scan, 63);
  nbad = wave_sum_int(nbad);
  nnz = wave_sum_int(nnz);
  lsb = wave_min_int(lsb);
  first = wave_min_int(first);
  amin = wave_min_dbl_x(amin);
  amax = wave_max_dbl_x(amax);
  if (lane == 0) {
    sh.mass[wave] = all;
    sh.amin[wave] = amin;
    sh.amax[wave] = amax;
    sh.nbad[wave] = nbad;
    sh.nnz[wave] = nnz;
    sh.lsb[wave] = lsb;
    sh.first[wave] = first;
  }
  // the rows again, from where they are now
  auto again = [&](int ta, int tb, auto f) {
    if constexpr (kLds) {
      for (int i = 64 * ta + lane; i < min(n, 64 * tb); i += 64) f(col[i], i);
    } else {
      for_rows(x, n, ta, tb, lane, f);
    }
  };
  __syncthreads();
  double before = 0.0, total = 0.0;
  nbad = nnz = 0;
#pragma unroll
  for (int w = 0; w < kW; ++w) {
    before = w < wave ? before + sh.mass[w] : before;
    total = total + sh.mass[w];
    nbad += sh.nbad[w];
    nnz += sh.nnz[w];
    lsb = min(lsb, sh.lsb[w]);
    first = min(first, sh.first[w]);
    amin = fmin(amin, sh.amin[w]);
    amax = fmax(amax, sh.amax[w]);
  }
  int flags = nbad ? COL_NONFINITE : 0;
  const int e0 = nnz ? lsb : 0;
  if (!nbad && nnz) {
    const int bl = 32 - __builtin_clz((unsigned)nnz);
    if ((highest_bit_exp(amax) - e0 + 1) + bl > 124) flags |= COL_WIDE;
  }
  const bool sample = smp != nullptr && flags == 0 && nnz > 0;
  if (wave == 0) {
    ((unsigned *)sh.smp)[lane] = 0xFFFFFFFFu;
  }
  __syncthreads();
  u128 s = 0;
  if (!flags) {
    const bool chunks = n <= L1LINE_MAX_N;        // (chunk sums exact below 2^16 nonzeros)
    double c0s = 0.0, c1s = 0.0, c2s = 0.0;
    const double step = total / SAMPLE_ROWS, inv = SAMPLE_ROWS / total;
    double cum = before + (scan - mine);
    int r = sample ? max((int)ceil(cum / step - 0.5), 0) : SAMPLE_ROWS;
    double next = r < SAMPLE_ROWS ? (r + 0.5) * step : __builtin_inf();
    again(t0, t1, [&](double v, int i) {
      const double a = fabs(v);
      if (chunks) {
        double c0, c1, c2;
        weight_chunks(a, e0, c0, c1, c2);
        c0s = c0s + c0;
        c1s = c1s + c1;
        c2s = c2s + c2;
      } else {
        s += a != 0.0 ? fixed_of(a, e0) : (u128)0;
      }
      cum = cum + a;
      if (cum > next && a != 0.0) {
        sh.smp[r] = (unsigned short)i;
        r = (int)fmin(fmax(ceil(cum * inv - 0.5), r + 1.0), (double)SAMPLE_ROWS);
        next = r < SAMPLE_ROWS ? (r + 0.5) * step : __builtin_inf();
      }
    });
    s = chunks ? chunks_to_u128(wave_sum_dbl_x(c0s), wave_sum_dbl_x(c1s), wave_sum_dbl_x(c2s)) : wave_sum_u128(s);
    if (lane == 0) sh.fix[wave] = s;
  }
  double part = mine;
  if (wave == 0) {
    if constexpr (kW > 1) {
      part = 0.0;
      again(0, T, [&](double v, int) { part = part + fabs(v); });   // (rows past n add +0)
    }
    part = wave_r64_tree_x(part);
  }
  __syncthreads();
  if (wave != 0) return;
  if (smp) {
    const uint32_t two = ((const unsigned *)sh.smp)[lane];
    const bool has0 = (two & 0xFFFFu) != 0xFFFFu, has1 = two >> 16 != 0xFFFFu;
    // the lanes at or below that hold a sample, and each one's last
    const uint64_t m = __ballot(has0 || has1), below = m & ((1ull << lane) - 1ull);
    const uint32_t last = has1 ? two >> 16 : two & 0xFFFFu;
    const uint32_t prev = (uint32_t)__shfl((int)last, below ? 63 - __builtin_clzll(below) : 0);
    const uint32_t f = sample ? (uint32_t)first : 0u;   // (without a sample no segment uses it)
    const uint32_t s0 = has0 ? two & 0xFFFFu : below ? prev : f, s1 = has1 ? two >> 16 : s0;
    ((unsigned *)smp)[lane] = s0 | (s1 << 16);
  }
  if (lane == 0) {
    ColInfo c;
    c.wfix = 0;
    if (!flags)
      for (int w = 0; w < kW; ++w) c.wfix += sh.fix[w];
    c.W = part;
    c.e0 = e0;
    c.nnz = nnz;
    c.zeros = n - nnz - nbad;
    c.flags = flags;
    c.bemin = nnz ? (int)((uint64_t)__double_as_longlong(amin) >> 52) : 4096;
    c.bemax = nbad ? 0x7ff : nnz ? (int)((uint64_t)__double_as_longlong(amax) >> 52) : -1;
    c.unit = flags ? 0.0 : column_unit(c.wfix, e0, nnz, amin, amax);
    *out = c;
  }
}

// smp (optional): SAMPLE_ROWS row ids per column.  kLds: the launch has n
// doubles of dynamic LDS.
template <int kW, bool kLds>
__global__ void __launch_bounds__(64 * kW)
k_colprep(const double *__restrict__ X, int n, int m, long long ld, ColInfo *__restrict__ ci,
          unsigned short *__restrict__ smp) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ __attribute__((aligned(16))) PrepShared sh;
  const int col = blockIdx.x;
  colprep_block<kW, kLds>(X + (long long)col * ld, n, ci + col, smp ? smp + (long long)col * SAMPLE_ROWS : nullptr, sh,
                      (double *)smem);
}

// every column of every problem: colstart[b] = first column of problem b.
// kLds: the launch has room for the longest problem's column.  counters: the
// call's SEG_COUNTERS counters, cleared here for the launches that follow (a
// launch of its own took 4 of the 107 us of 4 matrices of up to 150 x 30).
constexpr int SEG_COUNTERS = 16;
template <int kW, bool kLds>
__global__ void __launch_bounds__(64 * kW)
k_colprep_batch(const ProbDesc *__restrict__ P, const int *__restrict__ colstart, int B,
                ColInfo *__restrict__ ci, unsigned short *__restrict__ smp, int *__restrict__ segflags,
                const int *__restrict__ gate, int gate_on, int *__restrict__ counters) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ __attribute__((aligned(16))) PrepShared sh;
  const int g = blockIdx.x;
  if (gate && *gate != gate_on) return;
  if (g == 0 && threadIdx.x < SEG_COUNTERS) counters[threadIdx.x] = 0;
  const int b = find_owner(colstart, B, g);
  const ProbDesc d = P[b];
  const int col = g - colstart[b];
  colprep_block<kW, kLds>(d.X + (long long)col * d.ld, d.n, ci + g, smp + (long long)g * SAMPLE_ROWS, sh, (double *)smem);
  if (threadIdx.x == 0) segflags[g] = 0;
}

// ----------------------------------------------------------- segment access
// One wave streams over the rows of segment (j, k); row i = lane + 64 t for
// slot t < T.  Column j sits in LDS, column k is read from global memory
// (it stays in L2/MALL across the concurrent workgroups).  Nothing per row
// is kept in registers: every pass recomputes the ratio it needs, which keeps
// the register count low and the occupancy high.
struct SegIO {
  const double *__restrict__ xk;   // column k (device memory)
  const double *__restrict__ sxj;  // column j (LDS when lds, else device memory)
  int n, T, e0, lane;              // rows, slots, fixed-point exponent
  bool lds;                        // a compile-time constant at every construction
};

// x_ij of row i, through the address space column j lives in
__device__ __forceinline__ double sxj_at(const SegIO &s, int i) {
  return s.lds ? s.sxj[i] : gld(s.sxj + i);
}

// x_ij of row i < 64 T, 0 past row n: the zero-padded LDS copy, or the
// column in device memory through its range-checked descriptor rj
__device__ __forceinline__ double sxj_pad(const SegIO &s, __amdgpu_buffer_rsrc_t rj, int i) {
  return s.lds ? s.sxj[i] : col_ld(rj, i * 8);
}

// key of fl(x_ik / x_ij) + 0.0; KEY_NONE outside the matrix or where x_ij = 0
__device__ __forceinline__ uint64_t seg_key(const SegIO &s, int i) {
  const bool in = i < s.n;
  const int ic = in ? i : 0;
  const double a = sxj_at(s, ic), b = gld(s.xk + ic);
  double r = b / a;
  r = r + 0.0;
  return (in && a != 0.0) ? key_of(r) : KEY_NONE;
}

// the same key from x_ij = a and x_ik = b already loaded (in: the row is
// inside the matrix); branch-free, so that loads of the next slot issued
// before it stay in flight across the divide
__device__ __forceinline__ uint64_t key_of_pair(bool in, double a, double b) {
  const bool ok = in && a != 0.0;
  double r = b / (ok ? a : 1.0);
  r = r + 0.0;
  return ok ? key_of(r) : KEY_NONE;
}

// The top 32 bits of the key of row i's ratio, estimated with the hardware
// reciprocal inv of x_ij (not 0 at sample rows).  Sample keys only place window
// bounds and pivots, and any keys are valid there (every element is decided
// exactly against them), so neither the IEEE divide nor the low 32 bits of
// the key are needed: a bound derived from a prefix p is p 2^32 (lower) or
// p 2^32 + 2^32 - 1 (upper), at most 2^-20 relative off the sample's ratio.
__device__ __forceinline__ uint32_t sample_key32(const SegIO &s, int i, double inv) {
  double r = gld(s.xk + i) * inv;
  r = r + 0.0;
  return (uint32_t)(key_of(r) >> 32);
}

// exact weight |x_ij| / 2^e0 of row i, 0 where !valid
__device__ __forceinline__ u128 seg_weight(const SegIO &s, int i, bool valid) {
  const double a = sxj_at(s, valid ? i : 0);
  return valid ? fixed_of_col(a, s.e0) : (u128)0;
}

__device__ __forceinline__ void take_sample(bool c, int pri, uint64_t key, int t, int &bp, uint64_t &bk,
                                            int &bt) {
  const bool better = c && pri < bp;
  bp = better ? pri : bp;
  bk = better ? key : bk;
  bt = better ? t : bt;
}

// Per-wave LDS of the exact kernel: the <= 64 final candidates of the
// selection rounds, and the window list (keys and rows; WIN_CAP for single
// penalties, PATH_CAP for several).
constexpr int WIN_CAP = 512;
constexpr int PATH_CAP = 1024;
// (the LDS sort pads a list to the next power of two, which must stay
// inside the wave's area)
static_assert((WIN_CAP & (WIN_CAP - 1)) == 0 && (PATH_CAP & (PATH_CAP - 1)) == 0,
              "window list capacities must be powers of two");
struct WaveScratch {
  uint64_t ckey[64];
  int crow[64];
  // bisection of a window too full for the list: lower end and element
  // count of the part that holds the target, probe passes so far (kept here,
  // off the registers of the window pass)
  uint64_t blo;
  int bcnt, steps;
};

// Element source of the exact selection: every row of the column, the ratio
// recomputed.  Slot t of lane l is element l + 64 t (increasing row order).
// sbase / cbase: weight and count of elements below them.
struct ColSrc {
  const SegIO &s;
  u128 sbase;
  int cbase;
  __device__ __forceinline__ int slots() const { return s.T; }
  __device__ __forceinline__ void at(int t, uint64_t &key, int &row) const {
    row = s.lane + 64 * t;
    key = seg_key(s, row);
  }
};

// ------------------------------------------------- finishing <= 64 candidates
// Candidates are the elements with klo < key <= khi (count <= 64); Slo is the
// exact weight of all elements with key <= klo.  Compact them to LDS, sort by
// (key, row) across the lanes, scan their exact weights from Slo and take the
// first whose prefix reaches tau.
template <class Src>
__device__ __forceinline__ void wave_finish(const SegIO &s, const Src &src, uint64_t klo, uint64_t khi, int count,
                                            u128 Slo, u128 tau, WaveScratch *ws, uint64_t &okey, int &orow,
                                            int &err) {
  const int lane = s.lane;
  int base = 0;
  const int ns = src.slots();
#pragma unroll 2
  for (int t = 0; t < ns; ++t) {
    uint64_t key;
    int row;
    src.at(t, key, row);
    const bool c = key > klo && key <= khi;
    const uint64_t mask = __ballot(c);
    const int pos = base + __builtin_popcountll(mask & ((1ull << lane) - 1ull));
    if (c && pos < 64) {
      ws->ckey[pos] = key;
      ws->crow[pos] = row;
    }
    base += __builtin_popcountll(mask);
  }
  wave_lds_sync();
  uint64_t ck = lane < count ? ws->ckey[lane] : KEY_NONE;
  int cr = lane < count ? ws->crow[lane] : 0x7fffffff;
  wave_lds_sync();
  wave_sort_key_row(ck, cr, lane);
  const u128 w = seg_weight(s, lane < count ? cr : 0, lane < count);
  const u128 S = wave_incl_scan_u128(w, lane) + Slo;
  const uint64_t hit = __ballot(lane < count && S >= tau);
  if (!hit || base != count) {
    err |= SEG_INTERNAL;
    okey = KEY_NONE;
    orow = -1;
    return;
  }
  const int srcl = __builtin_ctzll(hit);
  okey = uni_u64(shfl_u64(ck, srcl));
  orow = uni_int(__shfl(cr, srcl));
}

// ----------------------------------------------------------- selection rounds
// Exact selection: find the first element, in (ratio, row) order, whose
// inclusive prefix weight reaches tau.  Candidates are the elements with
// klo < key <= khi; Slo/Clo (Shi/Chi) are the exact weight and count of ALL
// elements with key <= klo (<= khi).  Rounds take two pivots from a weighted
// sample of the candidates and count exactly; a round without progress
// switches to key-space bisection; a single repeated key falls back to row
// order.
template <class Src>
__device__ __forceinline__ void wave_select_rounds(const SegIO &s, const Src &src, uint64_t klo, uint64_t khi,
                                                   u128 Slo, u128 Shi, int Clo, int Chi, u128 tau,
                                                   WaveScratch *ws, uint64_t &okey, int &orow, int &err) {
  constexpr double DELTA = 0.15;
  const int lane = s.lane;
  const int ns = src.slots();
  int nsp = 1;
  while (nsp < ns) nsp <<= 1;
  int count = Chi - Clo;
  bool bisect = false, single_key = false;
  int rounds = 0;
  uint64_t sk = KEY_NONE;
  int sr = 0;
  okey = KEY_NONE;
  orow = -1;
  while (count > 64) {
    if (++rounds > 160) {
      err |= SEG_INTERNAL;
      return;
    }
    uint64_t plo, phi;
    if (!bisect) {
      double sw = (sk != KEY_NONE) ? fabs(sxj_at(s, sr)) : 0.0;
      wave_sort_key_dbl(sk, sw, lane);
      const double cw = wave_incl_scan_dbl(sw, lane);
      const double tot = __shfl(cw, 63);
      const double f = u128_to_double_approx(tau - Slo) / u128_to_double_approx(Shi - Slo);
      const double flo = (f - DELTA) * tot, fhi = (f + DELTA) * tot;
      const uint64_t mlo = __ballot(sk != KEY_NONE && cw <= flo);
      const uint64_t mhi = __ballot(sk != KEY_NONE && cw >= fhi);
      plo = mlo ? uni_u64(shfl_u64(sk, 63 - __builtin_clzll(mlo))) : klo;
      phi = mhi ? uni_u64(shfl_u64(sk, __builtin_ctzll(mhi))) : khi;
      if (phi < plo) phi = plo;
    } else {
      uint64_t cmin = KEY_NONE, cmax = 0;
#pragma unroll 2
      for (int t = 0; t < ns; ++t) {
        uint64_t key;
        int row;
        src.at(t, key, row);
        const bool c = key > klo && key <= khi;
        cmin = (c && key < cmin) ? key : cmin;
        cmax = (c && key > cmax) ? key : cmax;
      }
      cmin = wave_min_u64(cmin);
      cmax = wave_max_u64(cmax);
      if (cmin == cmax) {
        single_key = true;
        khi = cmax;
        break;
      }
      plo = phi = cmin + ((cmax - cmin) >> 1);
    }
    // exact weights and counts at or below each pivot, and one sample per
    // lane from each of the three sub-intervals
    u128 s1 = 0, s2 = 0;
    int c1 = 0, c2 = 0;
    uint64_t ka = KEY_NONE, kb = KEY_NONE, kc = KEY_NONE;
    int pa = nsp, pb = nsp, pc = nsp, ra = 0, rb = 0, rc = 0;
    const int start = (lane * 11 + rounds * 5) & (nsp - 1);
#pragma unroll 2
    for (int t = 0; t < ns; ++t) {
      uint64_t key;
      int row;
      src.at(t, key, row);
      const bool valid = key != KEY_NONE;
      const u128 w = seg_weight(s, row, valid);
      const bool le1 = valid && key <= plo, le2 = valid && key <= phi;
      s1 += le1 ? w : (u128)0;
      s2 += le2 ? w : (u128)0;
      c1 += le1 ? 1 : 0;
      c2 += le2 ? 1 : 0;
      const int pri = (t - start) & (nsp - 1);
      take_sample(key > klo && le1, pri, key, row, pa, ka, ra);
      take_sample(key > plo && le2, pri, key, row, pb, kb, rb);
      take_sample(key > phi && key <= khi, pri, key, row, pc, kc, rc);
    }
    s1 = wave_sum_u128(s1) + src.sbase;
    s2 = wave_sum_u128(s2) + src.sbase;
    c1 = wave_sum_int(c1) + src.cbase;
    c2 = wave_sum_int(c2) + src.cbase;
    if (s1 >= tau) {
      khi = plo; Shi = s1; Chi = c1;
      sk = ka; sr = ra;
    } else if (s2 >= tau) {
      klo = plo; Slo = s1; Clo = c1;
      khi = phi; Shi = s2; Chi = c2;
      sk = kb; sr = rb;
    } else {
      klo = phi; Slo = s2; Clo = c2;
      sk = kc; sr = rc;
    }
    const int ncount = Chi - Clo;
    bisect = (ncount == count);
    count = ncount;
  }
  if (!single_key) {
    wave_finish(s, src, klo, khi, count, Slo, tau, ws, okey, orow, err);
    return;
  }
  // every candidate has the same key K: (key, row) order is enumeration order
  const uint64_t K = khi;
  u128 S = Slo;
  for (int t = 0; t < ns; ++t) {
    uint64_t key;
    int row;
    src.at(t, key, row);
    const bool c = key == K;
    const u128 w = seg_weight(s, row, c);
    const u128 sc = wave_incl_scan_u128(w, lane) + S;
    const uint64_t hit = __ballot(c && sc >= tau);
    if (hit) {
      const int sl = __builtin_ctzll(hit);
      okey = K;
      orow = uni_int(__shfl(row, sl));
      return;
    }
    S = uni_u128(shfl_u128(sc, 63));
  }
  err |= SEG_INTERNAL;
}

// --------------------------------------------------- sorting the window list
// The window list (nlist entries, row order) is padded to a power of two
// N >= 64 with KEY_NONE and sorted by (key, row) with a bitonic network in
// LDS (each lane handles N/128 compare-exchanges per stage).  Returns N.
__device__ __forceinline__ int wave_sort_lds(uint64_t *lk, unsigned short *lr, int nlist, int lane) {
  int N = 64;
  while (N < nlist) N <<= 1;
  for (int e = nlist + lane; e < N; e += 64) {
    lk[e] = KEY_NONE;
    lr[e] = 0xFFFF;
  }
  wave_lds_sync();
  for (int size = 2; size <= N; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int pidx = lane; pidx < (N >> 1); pidx += 64) {
        const int e = ((pidx & ~(stride - 1)) << 1) | (pidx & (stride - 1));
        const int f = e + stride;
        const uint64_t ke = lk[e], kf = lk[f];
        const unsigned re = lr[e], rf = lr[f];
        const bool up = (e & size) == 0;
        const bool gt = ke > kf || (ke == kf && re > rf);
        const bool lt = ke < kf || (ke == kf && re < rf);
        if (up ? gt : lt) {
          lk[e] = kf;
          lk[f] = ke;
          lr[e] = (unsigned short)rf;
          lr[f] = (unsigned short)re;
        }
      }
      wave_lds_sync();
    }
  }
  return N;
}

// Exact weights of the sorted list: lane l owns the E = N/64 consecutive
// entries [E l, E l + E); tot = their exact weight, incl = inclusive scan of
// tot over the lanes.
__device__ __forceinline__ void wave_list_sums(const SegIO &s, const uint64_t *lk, const unsigned short *lr, int E,
                                               u128 &tot, u128 &incl) {
  tot = 0;
  for (int q = 0; q < E; ++q) {
    const int e = E * s.lane + q;
    const bool valid = lk[e] != KEY_NONE;
    tot += seg_weight(s, valid ? (int)lr[e] : 0, valid);
  }
  incl = wave_incl_scan_u128_x(tot, s.lane);
}

// Lane-parallel resolution: every lane with a target (active) finds the first
// list entry whose exact prefix weight, counted from Slo (the weight of every
// element below the list), reaches its tau.  A binary search over the lanes'
// inclusive sums finds the owning lane, a walk over its entries the element.
// hit = false when tau lies outside (Slo, Slo + weight of the list].
__device__ __forceinline__ void wave_resolve(const SegIO &s, const uint64_t *lk, const unsigned short *lr, int E,
                                             u128 Slo, u128 tot, u128 incl, bool active, u128 tau,
                                             uint64_t &okey, int &orow, bool &hit) {
  const u128 wall = readlane_u128(incl, 63);
  const bool inwin = active && tau > Slo && tau <= Slo + wall;
  int lo = 0, hi = 63;
#pragma unroll
  for (int it = 0; it < 6; ++it) {
    const int mid = (lo + hi) >> 1;
    const u128 im = shfl_u128(incl, mid);
    if (Slo + im >= tau) hi = mid;
    else lo = mid + 1;
  }
  const u128 totc = shfl_u128(tot, lo), inclc = shfl_u128(incl, lo);
  hit = false;
  if (inwin) {
    u128 run = Slo + inclc - totc;
    for (int q = 0; q < E; ++q) {
      const int e = E * lo + q;
      const uint64_t key = lk[e];
      const bool valid = key != KEY_NONE;
      run += seg_weight(s, valid ? (int)lr[e] : 0, valid);
      if (valid && run >= tau) {
        okey = key;
        orow = (int)lr[e];
        hit = true;
        break;
      }
    }
  }
}

// e_jk = R64 over i of |x_ik - fl(v x_ij)| (result in lane 0).
__device__ __forceinline__ double wave_residual(const SegIO &s, double v) {
  // column k in batches of RB loads issued back to back (the sum is still
  // taken slot by slot in increasing order)
  constexpr int RB = 8;
  double p = 0.0;
  if (__builtin_isfinite(v)) {
    // rows past n read 0 from both columns and add |0 - v 0| = +0, which
    // leaves the lane's partial as it is: no per-row masks or clamps
    const __amdgpu_buffer_rsrc_t rk = col_rsrc(s.xk, s.n), rj = col_rsrc(s.lds ? s.xk : s.sxj, s.n);
    int t0 = 0;
    for (; t0 + RB <= s.T; t0 += RB) {
      double xk[RB], xj[RB];
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        xk[r] = col_ld(rk, (s.lane + 64 * (t0 + r)) * 8);
        xj[r] = sxj_pad(s, rj, s.lane + 64 * (t0 + r));
      }
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        const double prod = v * xj[r];
        const double d = xk[r] - prod;
        p = p + fabs(d);
      }
    }
    for (; t0 < s.T; ++t0) {
      const int i = s.lane + 64 * t0;
      const double prod = v * sxj_pad(s, rj, i);
      const double d = col_ld(rk, i * 8) - prod;
      p = p + fabs(d);
    }
    return wave_r64_tree_x(p);
  }
  // (an infinite ratio: v 0 is NaN, so the rows past n are masked)
  for (int t0 = 0; t0 < s.T; t0 += RB) {
    double xk[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const int i = s.lane + 64 * (t0 + r);
      xk[r] = gld(s.xk + (i < s.n ? i : 0));
    }
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const int i = s.lane + 64 * (t0 + r);
      const bool in = i < s.n;
      const double prod = v * sxj_at(s, in ? i : 0);
      const double d = xk[r] - prod;
      p = p + (in ? fabs(d) : 0.0);
    }
  }
  return wave_r64_tree_x(p);
}

// Bitonic sort of 128 32-bit keys held two per lane (element 2 lane + r),
// ascending, through VALU lane exchanges.
__device__ __forceinline__ void wave_sort2_u32_x(uint32_t &a, uint32_t &b, int lane) {
#pragma unroll
  for (int size = 2; size <= 128; size <<= 1) {
#pragma unroll
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      const bool up = ((2 * lane) & size) == 0;
      if (stride == 1) {
        const uint32_t lo = min(a, b), hi = max(a, b);
        a = up ? lo : hi;
        b = up ? hi : lo;
      } else {
        const int ls = stride >> 1;
        const uint32_t oa = xswap32(a, ls), ob = xswap32(b, ls);
        const bool keep_min = (((2 * lane) & stride) == 0) == up;
        a = keep_min ? min(oa, a) : max(oa, a);
        b = keep_min ? min(ob, b) : max(ob, b);
      }
    }
  }
}

// Bitonic sort of 128 (key, row) pairs held two per lane (element
// 2 lane + r), ascending in (key, row).
__device__ __forceinline__ void wave_sort2_kr_x(uint64_t &ka, int &ra, uint64_t &kb, int &rb, int lane) {
#pragma unroll
  for (int size = 2; size <= 128; size <<= 1) {
#pragma unroll
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      const bool up = ((2 * lane) & size) == 0;
      if (stride == 1) {
        const bool sw = (kb < ka || (kb == ka && rb < ra)) == up;
        const uint64_t tk = ka;
        const int tr = ra;
        ka = sw ? kb : ka;
        ra = sw ? rb : ra;
        kb = sw ? tk : kb;
        rb = sw ? tr : rb;
      } else {
        const int ls = stride >> 1;
        const bool keep_min = (((2 * lane) & stride) == 0) == up;
        const uint64_t oka = xswap64(ka, ls), okb = xswap64(kb, ls);
        const int ora = (int)xswap32((uint32_t)ra, ls), orb = (int)xswap32((uint32_t)rb, ls);
        const bool la = oka < ka || (oka == ka && ora < ra), lb = okb < kb || (okb == kb && orb < rb);
        ka = la == keep_min ? oka : ka;
        ra = la == keep_min ? ora : ra;
        kb = lb == keep_min ? okb : kb;
        rb = lb == keep_min ? orb : rb;
      }
    }
  }
}

// The same network over 256 entries, four per lane (entry 4 lane + q in
// slot q): strides 1 and 2 pair slots of one lane, longer strides pair slot q
// with slot q of lane (lane ^ stride / 4).
__device__ __forceinline__ void wave_sort4_kr_x(uint64_t (&k)[4], int (&r)[4], int lane) {
#pragma unroll
  for (int size = 2; size <= 256; size <<= 1) {
#pragma unroll
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      if (stride < 4) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (q & stride) continue;
          const int p = q | stride;
          const bool up = ((4 * lane + q) & size) == 0;
          const bool sw = (k[p] < k[q] || (k[p] == k[q] && r[p] < r[q])) == up;
          const uint64_t tk = k[q];
          const int tr = r[q];
          k[q] = sw ? k[p] : k[q];
          r[q] = sw ? r[p] : r[q];
          k[p] = sw ? tk : k[p];
          r[p] = sw ? tr : r[p];
        }
      } else {
        const int ls = stride >> 2;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const bool up = ((4 * lane + q) & size) == 0;
          const bool keep_min = ((lane & ls) == 0) == up;
          const uint64_t ok = xswap64(k[q], ls);
          const int orow = (int)xswap32((uint32_t)r[q], ls);
          const bool lt = ok < k[q] || (ok == k[q] && orow < r[q]);
          k[q] = lt == keep_min ? ok : k[q];
          r[q] = lt == keep_min ? orow : r[q];
        }
      }
    }
  }
}

// Sorts the window list lk/lr[0, nlist) ascending in (key, row) and pads it
// with (KEY_NONE, 0xFFFF) to N = the returned power of two (>= 64).  Lists of
// up to 256 are sorted in registers (VALU lane exchanges, no LDS round trips
// per stage) and written back; longer ones by the LDS network.
__device__ __forceinline__ int wave_sort_list(uint64_t *lk, unsigned short *lr, int nlist, int lane) {
  if (nlist > 256) return wave_sort_lds(lk, lr, nlist, lane);
  if (nlist > 128) {
    uint64_t k[4];
    int r[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = 4 * lane + q;
      k[q] = e < nlist ? lk[e] : KEY_NONE;
      r[q] = e < nlist ? (int)lr[e] : 0xFFFF;
    }
    wave_sort4_kr_x(k, r, lane);
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      lk[4 * lane + q] = k[q];
      lr[4 * lane + q] = (unsigned short)r[q];
    }
    wave_lds_sync();
    return 256;
  }
  if (nlist <= 64) {
    uint64_t k = lane < nlist ? lk[lane] : KEY_NONE;
    int r = lane < nlist ? (int)lr[lane] : 0xFFFF;
    wave_sort_key_row_x(k, r, lane);
    wave_lds_sync();
    lk[lane] = k;
    lr[lane] = (unsigned short)r;
    wave_lds_sync();
    return 64;
  }
  const int e = 2 * lane;
  uint64_t ka = e < nlist ? lk[e] : KEY_NONE, kb = e + 1 < nlist ? lk[e + 1] : KEY_NONE;
  int ra = e < nlist ? (int)lr[e] : 0xFFFF, rb = e + 1 < nlist ? (int)lr[e + 1] : 0xFFFF;
  wave_sort2_kr_x(ka, ra, kb, rb, lane);
  wave_lds_sync();
  lk[e] = ka;
  lr[e] = (unsigned short)ra;
  lk[e + 1] = kb;
  lr[e + 1] = (unsigned short)rb;
  wave_lds_sync();
  return 128;
}

// --------------------------------------------------------------- sign sums
// For the pair (j, k) the ratio of row i, x_ik / x_ij, is positive, negative
// or zero with the signs of x_ik and x_ij (barring underflow, checked per
// segment).  Its weight is |x_ij|, so
//   D_jk  = sum_i x_ij sgn(x_ik)        = (weight of positive ratios) - (negative)
//   Zr_jk = sum_i |x_ij| [x_ik == 0]    = weight of the zero ratios
// and 0 minimises g_jk exactly when |D_jk| <= lambda + Zr_jk (Lemma 1 at the
// point 0).  Both are dense contractions over the rows: X^T sgn(X) and
// |X|^T [X == 0], computed here for all pairs with FP64 MFMA (16x16x4).
// Their rounding error (at most about n 2^-52 of the column mass) is far
// below the decision margin the segment kernel applies.
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int SS_TILE = 64;     // 64 (j) x 64 (k) outputs per workgroup, 4 waves of 16 x 64
constexpr int SS_ROWS = 16;     // rows i per LDS stage
constexpr int SS_LD = SS_TILE + 2;

// Fragment layout of v_mfma_f64_16x16x4f64 (wave64, measured on gfx950):
// lane l holds A[l & 15][l >> 4], B[l >> 4][l & 15] and D[(l >> 4) + 4 q][l & 15],
// q = 0..3 (unlike the FP32-output forms, the row index steps by 4 per
// register).
__device__ __forceinline__ f64x4 mfma_f64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// One 64 x 64 output tile of the sign sums of a column-major matrix; rows j of
// the tile are j0.. j0 + 63 of the candidate list (cand) or of 0..m-1.
// out[j m + k] = (D_jk, Zr_jk).  Every thread of the 256-wide block calls it.
__device__ __forceinline__ void signsum_tile(const double *__restrict__ X, int ilo, int ihi, int m, long long ld,
                                             const int *__restrict__ cand, int mj, int j0, int k0,
                                             double2 *__restrict__ out, bool by_index) {
  __shared__ double sA[SS_ROWS * SS_LD];
  __shared__ double sB[SS_ROWS * SS_LD];
  __shared__ int sj[SS_TILE];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  if (tid < SS_TILE) {
    const int jj = j0 + tid;
    sj[tid] = jj < mj ? (cand ? cand[jj] : jj) : -1;
  }
  __syncthreads();
  f64x4 accD[4], accZ[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    accD[t] = (f64x4){0.0, 0.0, 0.0, 0.0};
    accZ[t] = (f64x4){0.0, 0.0, 0.0, 0.0};
  }
  // rows in stages of SS_ROWS: each thread loads its PER + PER elements of
  // the next stage into registers while the current one is multiplied, and
  // stores column k's elements as their signs (computed once per element,
  // not once per wave that reads them)
  constexpr int PER = SS_ROWS * SS_TILE / 256;
  double pa[PER], pb[PER];
  auto load = [&](int i0) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int e = tid + 256 * q;
      const int c = e / SS_ROWS, r = e % SS_ROWS, i = i0 + r;
      const int jc = sj[c], kc = k0 + c;
      pa[q] = (i < ihi && jc >= 0) ? X[(long long)jc * ld + i] : 0.0;
      pb[q] = (i < ihi && kc < m) ? X[(long long)kc * ld + i] : 0.0;
    }
  };
  load(ilo);
  for (int i0 = ilo; i0 < ihi; i0 += SS_ROWS) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int e = tid + 256 * q;
      const int c = e / SS_ROWS, r = e % SS_ROWS;
      const double x = pb[q];
      sA[r * SS_LD + c] = pa[q];
      sB[r * SS_LD + c] = x > 0.0 ? 1.0 : (x < 0.0 ? -1.0 : 0.0);
    }
    __syncthreads();
    if (i0 + SS_ROWS < ihi) load(i0 + SS_ROWS);
#pragma unroll 2
    for (int kk = 0; kk < SS_ROWS / 4; ++kk) {
      const int r = 4 * kk + (lane >> 4);
      const double a = sA[r * SS_LD + 16 * wave + (lane & 15)];
      const double aa = fabs(a);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const double sg = sB[r * SS_LD + 16 * t + (lane & 15)];
        accD[t] = mfma_f64(a, sg, accD[t]);
        // exact zeros are rare: skip the product when this 4 x 16 block has none
        if (__ballot(sg == 0.0)) accZ[t] = mfma_f64(aa, sg == 0.0 ? 1.0 : 0.0, accZ[t]);
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int k = k0 + 16 * t + (lane & 15);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int jl = 16 * wave + (lane >> 4) + 4 * q, j = sj[jl];
      if (j >= 0 && k < m) out[(long long)(by_index ? j0 + jl : j) * m + k] = make_double2(accD[t][q], accZ[t][q]);
    }
  }
}

// tstart[b] = first tile of problem b; problem b has ceil(mj / 64) x
// ceil(m / 64) tiles with mj = ncand when cand is given (problem 0 only),
// else m.  DZ[pair_off + j m + k] = (D_jk, Zr_jk).
// split > 1: block g sums tile g / split over the rows of part g % split
// (whole LDS stages) into part[(g % split) per + e], e the pair's place in DZ
// (with a candidate list jj m + k, jj the candidate's index);
// k_zero_segments adds the parts in order and writes DZ.
// One block takes about 2 us per 16-row stage when it has a CU to itself
// (load latency and the FP64 matrix rate), so a matrix of few columns, whose
// tiles leave most of the CUs idle, is bound by the length of its row loop:
// 1003 x 517 (81 tiles) 123 us in one part, the fit 742 -> 661 in several;
// 20011 x 151 (9 tiles) 2344 us, the fit 5016 -> 2791.  2000 x 2000 (1024
// tiles, one part) runs at 0.6 of the FP64 matrix rate, 0.56 ms.
__global__ void __launch_bounds__(256)
k_signsum_batch(const ProbDesc *__restrict__ P, const int *__restrict__ tstart, int B,
                const int *__restrict__ cand, int ncand, double2 *__restrict__ DZ,
                const int *__restrict__ gate, int gate_on, int split, double2 *__restrict__ part, long long per) {
  if (gate && *gate != gate_on) return;
  const int g = blockIdx.x / split, sp = blockIdx.x % split;
  const int b = find_owner(tstart, B, g);
  const ProbDesc d = P[b];
  const int mj = cand ? ncand : d.m;
  const int tk_count = (d.m + SS_TILE - 1) / SS_TILE;
  const int tloc = g - tstart[b];
  const int rows = ((d.n + split - 1) / split + SS_ROWS - 1) / SS_ROWS * SS_ROWS;
  const int ilo = min(d.n, sp * rows), ihi = min(d.n, ilo + rows);
  double2 *out = split > 1 ? part + sp * per + (cand ? 0 : d.pair_off) : DZ + d.pair_off;
  signsum_tile(d.X, ilo, ihi, d.m, d.ld, cand, mj, (tloc / tk_count) * SS_TILE, (tloc % tk_count) * SS_TILE, out,
               split > 1);
}

// ---------------------------------------------------------------- segments
// For every (j, k) and lambda_t:  V[(t m + j) m + k] = v_k,  E[...] = e_jk,
// R[...] = median row (-1 for 0).
//  1. The sign sums D_jk, Zr_jk (k_signsum_batch) decide, with a rigorous
//     error margin, whether 0 minimises g_jk -- then v_k = 0 and e_jk is the
//     R64 column mass of k (|x_ik - fl(0 x_ij)| = |x_ik|): k_zero_segments --
//     or on which side of 0 the minimiser lies.
//  2. The ratios of 128 rows drawn once per j with probability proportional
//     to |x_ij| estimate where the weighted median lies: a window.  k_seg_fast
//     (one penalty) and k_seg_path (several) list its rows in one pass without
//     a division per row and select among them in FP64 with a rigorous margin.
//     Workgroup = (preserved column j, one part of the k range); its waves take
//     the next k from an LDS counter.
//  3. What the margin does not settle is left to k_seg_rest: exact 128-bit
//     sums and general rounds.
constexpr int SEG_WAVES = 4;        // waves per workgroup of k_seg_rest
constexpr int SEG_WAVES_MAX = 8;    // at most, of k_seg_fast and k_seg_path (4 or 8)
constexpr int SXJ_LDS_MAX = 4096;   // longest column j copied to LDS (32 KB)
constexpr int SEG_MASK_WORDS = 64;  // zero-segment mask words an item holds (one per lane: 4096 k)

__host__ __device__ constexpr size_t seg_sxj_bytes(int n) {
  return ((size_t)((n + 63) / 64) * 64 * 8 + 15) / 16 * 16;
}
__host__ __device__ constexpr size_t rest_wave_bytes(int L, int lcap) {
  return (size_t)L * 16 + sizeof(WaveScratch) + (size_t)lcap * (sizeof(uint64_t) + sizeof(unsigned short));
}

// The division-free path takes the columns k whose nonzero magnitudes keep every
// ratio to column j in 2^+-981 (normal, and between FAST_ZERO and FAST_OPEN);
// column j in 2^+-901, so that its sums and 2^-38 of them are normal too.  The
// exponents of column k that it takes with column j: none if !ok.
constexpr int FAST_RATIO = 980, FAST_COLUMN = 900;
struct FastRange {
  int lo, hi;
  __device__ __forceinline__ FastRange(const ColInfo &cj, bool ok) {
    ok = ok && (cj.nnz == 0 || (cj.bemin >= 1023 - FAST_COLUMN && cj.bemax <= 1023 + FAST_COLUMN));
    lo = ok ? max(1, cj.bemax - FAST_RATIO) : 1 << 20;
    hi = min(cj.bemin + FAST_RATIO, 0x7fe);
  }
  // (an empty column k: bemin 4096, bemax -1; one that is not finite: bemax 0x7ff,
  // since a bound of its samples may be NaN, and padding rows would be listed)
  __device__ __forceinline__ bool has(const ColInfo &ck) const { return ck.bemin >= lo && ck.bemax <= hi; }
};

// Probe point of a window (plo, phi] that holds more elements than the
// list: the middle one of the sample keys inside it, or with none inside the
// key halfway between its ends (when both are keys of finite ratios).  Any
// key inside the window serves: it only steers where the next exact listing
// pass looks.
// The sorted sample (128 top-32-bit keys, packed in pairs) is read from smp
// in LDS.
// false: no key strictly inside the window was found.
// sample key ix (top 32 bits, times 2^32) of a sorted sample stored as
// packed pairs: entry l holds keys 2 l (low half) and 2 l + 1 (high half)
__device__ __forceinline__ uint64_t sample_key(const uint64_t *smp, int ix) {
  const uint64_t w = smp[ix >> 1];
  return (ix & 1) ? (w & 0xFFFFFFFF00000000ull) : (w << 32);
}

__device__ __forceinline__ int sample_count(const uint64_t *smp, uint64_t bound, bool strict) {
  // sample keys at or below bound (strict: below); the keys ascend
  int lo = 0;
#pragma unroll
  for (int step = 64; step >= 1; step >>= 1) {
    const uint64_t k = sample_key(smp, lo + step - 1);
    if (strict ? k < bound : k <= bound) lo += step;
  }
  return lo;
}

__device__ __forceinline__ bool window_midpoint(const uint64_t *smp, uint64_t plo, uint64_t phi, uint64_t &mid) {
  const int i0 = sample_count(smp, plo, false), i1 = sample_count(smp, phi, true);
  if (i1 > i0) {
    mid = sample_key(smp, (i0 + i1) >> 1);
    return true;
  }
  // the keys of the finite doubles form one interval, [key(-inf), key(+inf)]
  constexpr uint64_t KEY_NEG_INF = 0x000FFFFFFFFFFFFFull, KEY_POS_INF = 0xFFF0000000000000ull;
  if (plo < KEY_NEG_INF || phi > KEY_POS_INF) return false;
  mid = plo + ((phi - plo) >> 1);
  return mid > plo;
}

// The penalty to compare with.  A weight sum of a column with a unit compared
// with a penalty is an integer compared with a real: the outcome is the one of
// the integer part, or of anything up to the next integer.  So it is taken in the
// middle between two whole ones, a quarter of a unit from the target of every
// prefix weight and half from the sides' sums, and neither ties (count data at
// whole penalties tie in most segments, which the exact kernel then had).  From
// 2^50 units on a penalty is above every weight sum as it is.
__device__ __forceinline__ double between_units(double lam, double unit) {
  const double l = lam * __builtin_amdgcn_rcp(unit);
  double q = floor(l);                             // off by one at most
  const double r = fma(-q, unit, lam);
  q = r < 0.0 ? q - 1.0 : r >= unit ? q + 1.0 : q;
  return unit > 0.0 && l < 0x1p50 ? (q + 0.5) * unit : lam;
}

// The side of the minimiser of segment (j, k) at penalty lam (between_units)
// from the sign sums dz = (D_jk, Zr_jk): 0 when 0 minimises g_jk, 1 negative, 2
// positive, 3 undecided (the exact pass decides).  Decision margin 2^-32 (W_j +
// lam): far above the rounding error of the sign sums (at most ~n 2^-52 of W_j,
// plus n 2^-1022 should the matrix unit flush subnormal terms: hence the floor
// on the margin); with a unit an eighth of it will do.
// unc: the sums cannot be trusted for this segment.
__device__ __forceinline__ int sign_sum_side(double2 dz, double lam, double Wj, double unit, bool unc) {
  const double M = unit > 0.0 ? 0.125 * unit : 0x1p-32 * (Wj + lam);
  const double d1 = lam + dz.y + dz.x;               // >= 0  <=>  2A <= W + lambda
  const double d2 = lam + dz.y - dz.x;               // >= 0  <=>  W <= 2B + lambda
  if (unc || !(M >= 0x1p-1000)) return 3;
  if (d1 > M && d2 > M) return 0;
  if (d1 < -M) return 1;
  if (d2 < -M) return 2;
  return 3;
}

// The sign sums cannot decide segment (j, k) when a ratio could underflow to
// 0 (exponent fields more than 1000 apart) or a sum is not finite.
__device__ __forceinline__ bool sign_sums_unsure(const ColInfo &cj, const ColInfo &ck, double2 dz) {
  const bool maybe_tiny = ck.nnz > 0 && cj.nnz > 0 && ck.bemin - cj.bemax < -1000;
  return maybe_tiny || !isfinite(dz.x) || !isfinite(dz.y);
}

// Where the division-free kernels leave what they cannot settle: a bit per
// segment, and a list of the words' parts: part p of a word is its left segments
// of rank rest_rank(p) to rest_rank(p + 1) - 1.  An append to the list takes about
// 6 ns, one after the other, so a full word has ten parts, not one per segment;
// the first of a word are short, since what is left clusters (the 2859 segments
// of the 2000 x 2000 path are close together in few columns; a word to a wave took
// 5.3 ms).
constexpr int REST_PARTS = 10;      // of a word, at most
__host__ __device__ constexpr int rest_rank(int p) { return p < 3 ? 2 * p : 8 * (p - 2); }
// parts of a word with `count` segments left
__host__ __device__ constexpr int rest_parts(int count) { return count <= 4 ? (count + 1) / 2 : (count + 23) / 8; }
struct TodoPart {
  int word, part;
};
struct TodoList {
  unsigned long long *bits;
  TodoPart *list;
  int *count;
};
__device__ __forceinline__ void leave_segment(const TodoList &td, long long word, int bit) {
  const unsigned long long old = atomicOr(td.bits + word, 1ull << bit);
  const int c = __builtin_popcountll(old), p = rest_parts(c);
  if (!((old >> bit) & 1ull) && rest_parts(c + 1) > p) td.list[atomicAdd(td.count, 1)] = TodoPart{(int)word, p};
}

// Segments settled by the sign sums alone.  One thread per pair (j, k), one
// wave per 64 consecutive k of a preserved column: where every penalty of the
// problem has 0 as a minimiser (sign_sum_side, the segment kernels' own test),
// sets bit k & 63 of mask word (jj, k >> 6); the segment kernel skips such
// segments.  They have v_k = 0, e_jk = the R64 mass of column k and row -1 for
// every penalty: written here for a problem of one penalty (Algorithm 2 reads
// them), taken from the mask by the kernels that follow for one of several
// (2000 x 2000 with 64: 2.0 ms of scattered stores).  wstart[b] = first mask
// word of problem b (mj ceil(m / 64) words, mj = ncand with a candidate list,
// problem 0 only, else m).
// Pairs outside the division-free range are left to the exact kernel here, a word
// at a time (one by one by the segment kernels 49 x 438 subnormal data took 1390 us,
// now 1060); `done` has them and the mask's bits: what the segment kernels skip.
__global__ void __launch_bounds__(256)
k_zero_segments(const ProbDesc *__restrict__ P, const int *__restrict__ wstart, int B, int total_words,
                const double *__restrict__ lam_all, const ColInfo *__restrict__ ci,
                double2 *__restrict__ DZ, double *__restrict__ V, double *__restrict__ E,
                int *__restrict__ R, unsigned long long *__restrict__ mask, unsigned long long *__restrict__ done, TodoList td,
                const int *__restrict__ cand, const int *__restrict__ gate, int gate_on, int split, const double2 *__restrict__ part,
                long long per) {
  const int w = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (w >= total_words) return;
  if (gate && *gate != gate_on) return;
  const int b = find_owner(wstart, B, w);
  const ProbDesc d = P[b];
  const int wpr = (d.m + 63) >> 6;
  const int wl = w - wstart[b];
  const int jj = wl / wpr, k = (wl - jj * wpr) * 64 + lane;
  const int j = cand ? cand[jj] : jj;
  bool skip = false, left = false;
  if (k < d.m && k != j) {
    const long long pair = d.pair_off + (long long)j * d.m + k;
    double2 dz;
    if (split > 1) {
      const double2 *pp = part + (cand ? (long long)jj * d.m + k : pair);
      dz = pp[0];
      for (int sp = 1; sp < split; ++sp) {
        const double2 x = pp[sp * per];
        dz.x = dz.x + x.x;
        dz.y = dz.y + x.y;
      }
      DZ[pair] = dz;
    } else {
      dz = DZ[pair];
    }
    const ColInfo cj = ci[d.col_off + j], ck = ci[d.col_off + k];
    if (!cj.flags && !ck.flags) {
      const bool unc = sign_sums_unsure(cj, ck, dz);
      const double *lam = lam_all + d.lam_off;
      const double unit = cj.unit;
      skip = true;
      for (int t = 0; t < d.L && skip; ++t)
        skip = sign_sum_side(dz, between_units(lam[t], unit), cj.W, unit, unc) == 0;
      if (skip && d.L == 1) {
        const long long base = d.ws_off + (long long)j * d.m + k;
        V[base] = 0.0;
        E[base] = ck.W;
        R[base] = -1;
      }
      left = !skip && !FastRange(cj, true).has(ck);
    }
  }
  const unsigned long long bits = __ballot(skip), rest = __ballot(left);
  if (lane == 0) {
    mask[d.mask_off + wl] = bits;
    done[d.mask_off + wl] = bits | rest;
    td.bits[d.mask_off + wl] = rest;
  }
  if (rest) {
    const int parts = rest_parts(__builtin_popcountll(rest));
    int at = 0;
    if (lane == 0) at = atomicAdd(td.count, parts);
    at = __builtin_amdgcn_readfirstlane(at);
    if (lane < parts) td.list[at + lane] = TodoPart{(int)(d.mask_off + wl), lane};
  }
}

// exact A (negative ratios), B (non-positive), counts, one sample per side
struct ExactSides {
  u128 A, B;
  int N, Z, NV;
};

__device__ __forceinline__ ExactSides exact_sides(const SegIO &s) {
  u128 a128 = 0, z128 = 0;
  int cN = 0, cZ = 0, cV = 0;
#pragma unroll 2
  for (int tt = 0; tt < s.T; ++tt) {
    const int i = s.lane + 64 * tt;
    const uint64_t key = seg_key(s, i);
    const bool valid = key != KEY_NONE;
    const u128 w = seg_weight(s, i, valid);
    const bool neg = key < KEY_ZERO, zer = key == KEY_ZERO;
    a128 += neg ? w : (u128)0;
    z128 += zer ? w : (u128)0;
    cN += neg ? 1 : 0;
    cZ += zer ? 1 : 0;
    cV += valid ? 1 : 0;
  }
  ExactSides e;
  e.A = wave_sum_u128(a128);
  e.B = e.A + wave_sum_u128(z128);
  e.N = wave_sum_int(cN);
  e.Z = wave_sum_int(cZ);
  e.NV = wave_sum_int(cV);
  return e;
}

// ------------------------------------------------- division-free segments
// One segment (j, k) at one penalty by one wave, without a division per row
// and without a sort.  With a = x_ij, b = x_ik the sign of the fused d =
// fma(-t, a, b) is the exact sign of b - t a (one rounding of the exact value,
// which keeps its sign when it overflows or underflows), so it says on which
// side of t the ratio b / a lies: below where d and a differ in sign.
//  window_pass  over the rows: T = sum of |a| sgn(b/a - lo) (a with its sign
//               flipped by d's: no comparison, no select), which is W - 2 S
//               for the weight S below lo; the rows between lo and hi are
//               those where the two signs differ, one bit per row shifted
//               into a word per lane (v_alignbit) and expanded to a list of
//               rows once per 32 slots;
//  select_listed  the listed rows' ratios (one IEEE divide each) go to 64
//               bins of the window, whose weights (LDS adds) are scanned; the
//               target's bin holds a few rows, ranked by counting.
// The target, counted from lo, is D = (T + lambda) / 2 on the negative side and
// (T - lambda) / 2 on the positive one (first prefix sum reaching D).  Sums
// run in FP64: every value compared is a sum of nonnegative weights of column j
// or a difference of such sums, at most W_j, and a rounding is at most u W_j (u =
// 2^-53).  For 65535 rows T takes 1024 adds a lane and a scan, D two more: 1040.
// The bins add up to 512 weights in turn, a scan and two for the new D, at up to
// eight levels, and the ranking 64: 4240 (select_listed).  A tie's rows take 1024
// slots' totals and scans: 1040 (tie_rows), a sorted list 30 (fast_path).  So two
// sides of a comparison are off by less than 2^13 u W_j together, and one whose
// operands differ by more than tol = 2^-38 W_j (2^15 u W_j) has the exact
// comparison's outcome; closer ones, a selected ratio equal to lo or hi (a row
// whose rounded ratio meets the bound may be on either side of it) and whatever
// else is unsettled leave the segment to k_seg_rest, which is exact.
constexpr int FAST_CAP = 512;       // rows a window may list
constexpr double FAST_ZERO = 0x1p-1000, FAST_OPEN = 0x1p1000;   // next to 0, beyond every ratio

// what two weight sums of column j may be off in a comparison; with a unit they
// differ from every target by a quarter of it at least
__device__ __forceinline__ double segment_tol(double Wj, double unit) { return unit > 0.0 ? 0.125 * unit : 0x1p-38 * Wj; }

struct FastScratch {
  uint32_t list[FAST_CAP];          // row, then row | bin << 16
  double bin[64];                   // bin weights, then the target bin's rows
};

// The rows of a segment in batches of FB slots, the next batch's loads issued
// while f(a, b) runs on the current one; rows past n give (0, 0).
// f is called for the slots [t0, t1) in order, in multiples of FB.
template <int FB, class LdJ, class LdK, class F>
__device__ __forceinline__ void for_row_pairs(const SegIO &s, LdJ ldj, LdK ldk, int t0, int t1, F f) {
  auto load = [&](int t, double *av, double *bv) {
    if (t + FB <= s.T) {
#pragma unroll
      for (int r = 0; r < FB; ++r) {
        av[r] = ldj(s.lane + 64 * (t + r));
        bv[r] = ldk(s.lane + 64 * (t + r));
      }
    } else {
#pragma unroll
      for (int r = 0; r < FB; ++r) {
        const bool in = t + r < s.T;
        av[r] = in ? ldj(s.lane + 64 * (t + r)) : 0.0;
        bv[r] = in ? ldk(s.lane + 64 * (t + r)) : 0.0;
      }
    }
  };
  // (two buffers in turn: no copies)
  double a0[FB], b0[FB], a1[FB], b1[FB];
  load(t0, a0, b0);
  for (int t = t0;; t += 2 * FB) {
    const bool more = t + FB < t1;
    if (more) load(t + FB, a1, b1);
#pragma unroll
    for (int r = 0; r < FB; ++r) f(a0[r], b0[r]);
    if (!more) break;
    const bool more2 = t + 2 * FB < t1;
    if (more2) load(t + 2 * FB, a0, b0);
#pragma unroll
    for (int r = 0; r < FB; ++r) f(a1[r], b1[r]);
    if (!more2) break;
  }
}

template <class LdJ, class LdK>
__device__ __forceinline__ void window_pass(const SegIO &s, LdJ ldj, LdK ldk, double lo, double hi, uint32_t *list,
                                            int cap, double &Tsum, int &count, int &listed) {
  double S = 0.0;
  int c = 0;
  listed = 0;
  for (int t0 = 0; t0 < s.T; t0 += 32) {
    uint32_t m = 0;
    const int t1 = min(s.T, t0 + 32);
    for_row_pairs<4>(s, ldj, ldk, t0, t1, [&](double a, double b) {
      const double dl = fma(-lo, a, b), dh = fma(-hi, a, b);
      S = S + flip_sign(a, dl);
      m = __builtin_amdgcn_alignbit(m, hi32(dl) ^ hi32(dh), 31);
    });
    // slot t0 + i at bit 31 - i
    m <<= 32 - ((t1 - t0 + 3) & ~3);
    const int pc = __builtin_popcount(m), incl = wave_scan_int(pc);
    const int tot = __builtin_amdgcn_readlane(incl, 63);
    if (c < cap) {
      // (past the list's end nothing is written; the count goes on)
      int pos = c + incl - pc;
      const uint64_t fit = __ballot(c + incl <= cap);   // (the lanes up to one)
      listed = c + (fit ? __builtin_amdgcn_readlane(incl, __builtin_popcountll(fit) - 1) : 0);
      m = c + incl <= cap ? m : 0;
      while (__ballot(m != 0)) {
        if (m) {
          const int i = __builtin_clz(m);
          list[pos++] = (uint32_t)(s.lane + 64 * (t0 + i));
          m ^= 0x80000000u >> i;
        }
      }
    }
    c += tot;
  }
  wave_lds_sync();
  Tsum = wave_total_dbl(S);
  count = c;
}

// T at three bounds in one pass, nothing listed
template <class LdJ, class LdK>
__device__ __forceinline__ void probe_pass(const SegIO &s, LdJ ldj, LdK ldk, const double (&t)[3], double (&T)[3]) {
  double S[3] = {0.0, 0.0, 0.0};
  for_row_pairs<4>(s, ldj, ldk, 0, s.T, [&](double a, double b) {
#pragma unroll
    for (int q = 0; q < 3; ++q) S[q] = S[q] + flip_sign(a, fma(-t[q], a, b));
  });
#pragma unroll
  for (int q = 0; q < 3; ++q) T[q] = wave_total_dbl(S[q]);
}

// A window that overflows the list although its samples promised fewer rows
// holds many equal ratios (whole numbers in long columns).  The most common
// ratio of three of the listed rows, and bounds just around it.
__device__ __forceinline__ bool tied_ratio(const SegIO &s, const uint32_t *list, int count, double &K, double &klo,
                                           double &khi) {
  if (count < 64) return false;                    // (too few were listed before the overflow)
  const int r = (int)list[s.lane];
  const double q = gld(s.xk + r) / sxj_at(s, r);
  int best = -1;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const double x = readlane_dbl(q, 21 * c);
    const int n = __builtin_popcountll(__ballot(q == x));
    K = n > best ? x : K;
    best = max(best, n);
  }
  klo = K - fabs(K) * 0x1p-44;
  khi = K + fabs(K) * 0x1p-44;
  return best > 1;
}

// The targets D (counted from klo, on the lanes of pend) among the rows
// between klo and khi when every one of their ratios rounds to K: the order is
// then the rows' order.  One pass finds each target's 64-row slot, a look at
// that slot its row.  false: another ratio lies there, or too close to call.
template <class LdJ, class LdK>
__device__ __forceinline__ bool tie_rows(const SegIO &s, LdJ ldj, LdK ldk, double K, double klo, double khi,
                                         uint64_t pend, double D, double tol, int &row) {
  const bool mine = ((pend >> s.lane) & 1ull) != 0;
  auto weight = [&](double a, double b, bool &bad) {
    const bool in = ((hi32(fma(-klo, a, b)) ^ hi32(fma(-khi, a, b))) >> 31) != 0;
    bad = bad || (in && b / a != K);
    return in ? fabs(a) : 0.0;
  };
  double run = 0.0, base = 0.0;
  int t = 0, slot = -1;
  bool bad = false;
  for_row_pairs<4>(s, ldj, ldk, 0, s.T, [&](double a, double b) {
    const double w = weight(a, b, bad);
    if (__ballot(w != 0.0)) {
      const double to = run + wave_total_dbl(w);
      const bool here = mine && D > run && D <= to;
      slot = here ? t : slot;
      base = here ? run : base;
      bad = bad || (mine && fabs(to - D) <= tol);
      run = to;
    }
    ++t;
  });
  if (__ballot(bad || (mine && slot < 0))) return false;
  for (; pend; pend &= pend - 1) {
    const int l = __builtin_ctzll(pend), ts = __builtin_amdgcn_readlane(slot, l);
    const double d = readlane_dbl(D, l) - readlane_dbl(base, l);
    const double w = weight(ldj(s.lane + 64 * ts), ldk(s.lane + 64 * ts), bad), incl = wave_scan_dbl(w);
    const uint64_t m = __ballot(w != 0.0 && incl >= d);
    if (m == 0 || __ballot(w != 0.0 && fabs(incl - d) <= tol)) return false;
    if (s.lane == l) row = 64 * ts + __builtin_ctzll(m);
  }
  return true;
}

// lanes (as a 64-bit mask) that keep the larger word of a bitonic stage over
// E words per lane: element E lane + q, partner lane ^ ls
template <int E>
constexpr uint64_t keep_max_mask(int size, int ls) {
  uint64_t m = 0;
  for (int l = 0; l < 64; ++l) {
    const bool up = ((E * l) & size) == 0, lower = (l & ls) == 0;
    if (up != lower) m |= 1ull << l;
  }
  return m;
}
__device__ __forceinline__ uint32_t pick(uint64_t keep_max, uint32_t x, uint32_t o) {
  return ((o < x) != __builtin_amdgcn_inverse_ballot_w64(keep_max)) ? o : x;
}
// compare-exchange of x with lane ^ ls (equal words are interchangeable)
__device__ __forceinline__ uint32_t cmpx_lane(uint32_t x, int ls, uint64_t keep_max) {
  if (ls >= 16) {
    // the swap leaves the pair's lower word in p[0] and its upper one in p[1]
    // on both lanes
    const auto p = ls == 16 ? __builtin_amdgcn_permlane16_swap(x, x, false, false)
                            : __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return ((p[1] < p[0]) != __builtin_amdgcn_inverse_ballot_w64(keep_max)) ? p[1] : p[0];
  }
  return pick(keep_max, x, xswap32(x, ls));
}

// Bitonic sort of 64 E words, element E lane + q, ascending.
template <int E>
__device__ __forceinline__ void wave_sort_u32(uint32_t (&x)[E]) {
#pragma unroll
  for (int size = 2; size <= 64 * E; size <<= 1) {
#pragma unroll
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      if (stride < E) {
#pragma unroll
        for (int q = 0; q < E; ++q) {
          if (q & stride) continue;
          const uint32_t a = x[q], b = x[q | stride];
          if (size < E) {
            const bool up = (q & size) == 0;
            x[q] = up ? min(a, b) : max(a, b);
            x[q | stride] = up ? max(a, b) : min(a, b);
            continue;
          }
          const uint64_t down = keep_max_mask<E>(size, 0);   // lanes whose block descends
          const bool sw = (b < a) != __builtin_amdgcn_inverse_ballot_w64(down);
          x[q] = sw ? b : a;
          x[q | stride] = sw ? a : b;
        }
      } else {
        const int ls = stride / E;
        const uint64_t km = keep_max_mask<E>(size, ls);
#pragma unroll
        for (int q = 0; q < E; ++q) x[q] = cmpx_lane(x[q], ls, km);
      }
    }
  }
}

enum : int { FAST_HIT, FAST_ABOVE, FAST_UNSURE };

// The first listed row, in (ratio, row) order, whose prefix weight reaches D
// (> tol): FAST_HIT with its ratio and row; FAST_ABOVE when the whole list
// weighs less than D; FAST_UNSURE when it is too close to call.  [blo, bhi]:
// the range the bins divide.  A target bin of more than 64 rows is divided
// again: over the range of its ratios, or, where they are all the same (whole
// numbers tie often), over the rows.
__device__ __forceinline__ int select_listed(const SegIO &s, FastScratch *fs, int count, double blo, double bhi,
                                             double D, double tol, double &v, int &row) {
  const int lane = s.lane;
  double scale = 64.0 / (bhi - blo);
  scale = bhi > blo && scale < 0x1p1000 ? scale : 0.0;
  const uint32_t OUT = 0xFFu << 16;               // a row outside the bin being divided
  bool by_row = false;
  for (int level = 0; level < 8; ++level) {
    fs->bin[lane] = 0.0;
    wave_lds_sync();
    constexpr int GB = 2;
    for (int e0 = 0; e0 < count; e0 += 64 * GB) {
      uint32_t x[GB];
      double av[GB], bv[GB];
#pragma unroll
      for (int q = 0; q < GB; ++q) {
        const int e = e0 + 64 * q + lane;
        x[q] = e < count ? fs->list[e] : OUT;
      }
#pragma unroll
      for (int q = 0; q < GB; ++q) {
        const int r = (int)(x[q] & 0xFFFFu);
        av[q] = sxj_at(s, r);
        bv[q] = gld(s.xk + r);
      }
#pragma unroll
      for (int q = 0; q < GB; ++q) {
        if (e0 + 64 * q >= count) break;
        const double r = by_row ? (double)(x[q] & 0xFFFFu) : bv[q] / av[q];
        const int bi = (int)min((uint32_t)fmax((r - blo) * scale, 0.0), 63u);
        if (x[q] < OUT) {
          fs->list[e0 + 64 * q + lane] = (x[q] & 0xFFFFu) | ((uint32_t)bi << 16);
          unsafeAtomicAdd(&fs->bin[bi], fabs(av[q]));
        }
      }
    }
    wave_lds_sync();
    const double w = fs->bin[lane], incl = wave_scan_dbl(w);
    if (__ballot(fabs(incl - D) <= tol)) return FAST_UNSURE;
    const uint64_t reach = __ballot(incl >= D);
    if (reach == 0) return level == 0 ? FAST_ABOVE : FAST_UNSURE;
    const int bt = __builtin_ctzll(reach);
    D = D - (readlane_dbl(incl, bt) - readlane_dbl(w, bt));
    // the target bin's rows, one per lane
    uint32_t *cr = (uint32_t *)fs->bin;
    int nc = 0;
    wave_lds_sync();
    for (int e0 = 0; e0 < count; e0 += 64) {
      const int e = e0 + lane;
      const uint32_t y = e < count ? fs->list[e] : OUT;
      const bool in = (y >> 16) == (uint32_t)bt;
      const uint64_t m = __ballot(in);
      const int pos = nc + lanes_below(m);
      nc += __builtin_popcountll(m);
      if (in && pos < 64) cr[pos] = y & 0xFFFFu;
    }
    nc = uni_int(nc);
    wave_lds_sync();
    if (nc <= 64) {
      const int myrow = lane < nc ? (int)cr[lane] : 0;
      const double a = sxj_at(s, myrow), r = gld(s.xk + myrow) / a, wa = fabs(a);
      if (nc > 24 && __ballot(lane < nc && r != readlane_dbl(r, 0)) == 0) {
        // equal ratios: sorted by row (87 x 657 of two values 1531 us by counting
        // among up to 64 rows, now 877)
        uint32_t x[1] = {lane < nc ? ((uint32_t)myrow << 6) | (uint32_t)lane : ~0u};
        wave_sort_u32<1>(x);
        const double ws = __shfl(wa, (int)(x[0] & 63u)), sum = wave_scan_dbl(lane < nc ? ws : 0.0);
        if (__ballot(lane < nc && fabs(sum - D) <= tol)) return FAST_UNSURE;
        const uint64_t at = __ballot(lane < nc && sum >= D);
        if (at == 0) return FAST_UNSURE;
        v = readlane_dbl(r, 0);
        row = (int)((uint32_t)__builtin_amdgcn_readlane((int)x[0], __builtin_ctzll(at)) >> 6);
        return FAST_HIT;
      }
      double run = 0.0;
      for (int i = 0; i < nc; ++i) {
        const double ri = readlane_dbl(r, i), wi = readlane_dbl(wa, i);
        const int rowi = __builtin_amdgcn_readlane(myrow, i);
        run = run + ((ri < r || (ri == r && rowi <= myrow)) ? wi : 0.0);
      }
      const bool mine = lane < nc;
      if (__ballot(mine && fabs(run - D) <= tol)) return FAST_UNSURE;
      const uint64_t sel = __ballot(mine && run >= D && run - wa < D);
      if (__builtin_popcountll(sel) != 1) return FAST_UNSURE;
      const int l = __builtin_ctzll(sel);
      v = readlane_dbl(r, l);
      row = __builtin_amdgcn_readlane(myrow, l);
      return FAST_HIT;
    }
    // too many: only the bin's rows stay, over the range of their ratios
    double rmin = __builtin_inf(), rmax = -__builtin_inf();
    for (int e = lane; e < count; e += 64) {
      const uint32_t y = fs->list[e];
      const int r = (int)(y & 0xFFFFu);
      const bool in = (y >> 16) == (uint32_t)bt;
      const double ra = by_row ? (double)r : gld(s.xk + r) / sxj_at(s, r);
      rmin = in ? fmin(rmin, ra) : rmin;
      rmax = in ? fmax(rmax, ra) : rmax;
      if (!in) fs->list[e] = (uint32_t)r | OUT;
    }
    blo = wave_min_dbl_x(rmin);
    bhi = wave_max_dbl_x(rmax);
    if (!by_row && !(bhi > blo)) {
      by_row = true;
      blo = 0.0;
      bhi = (double)s.n;
    }
    scale = 64.0 / (bhi - blo);
    scale = scale < 0x1p1000 ? scale : 0.0;
    wave_lds_sync();
  }
  return FAST_UNSURE;
}

// The minimiser of segment s at one penalty (between_units), on side neg; tol:
// what a comparison of weight sums may be off (segment_tol); sa, sb: the sorted
// sample (top 32 bits of the keys; index 2 l + c in lane l), c0 the target's
// expected place in it.  false: unsettled.
// The window starts WDELTA of the weight either side of the target's place
// in the sample (which is off by about 0.044, one sigma); a target outside it
// moves it on.  Windows whose samples promise more rows than the list holds
// (from about 2500 rows) are first cut by probe passes at three sample keys,
// two or three apart as the bracket shrinks, and inside one sample's gap
// (from about 26000 rows) at quarters of its range.
template <class LdJ, class LdK>
__device__ __forceinline__ bool fast_one(const SegIO &s, LdJ ldj, LdK ldk, bool neg, double lam, double Wd,
                                         double tol, uint32_t sa, uint32_t sb, double c0, FastScratch *fs, double &v, int &row) {
  constexpr double WDELTA = 0.06;
  // sample values with low bits no simple fraction has: a ratio equal to a
  // bound cannot be settled here.  `out`: a step of the keys' top 32 bits, for
  // bounds that have the sample's own row inside (a row that weighs more than
  // the window lies between two equal samples: 434 x 291 of heavy tails took 4.7
  // passes a segment, one now)
  auto value = [&](int ix, int out) {
    const uint32_t p = (uint32_t)__builtin_amdgcn_readlane((int)((ix & 1) ? sb : sa), ix >> 1) + (uint32_t)out;
    return ratio_of_key(((uint64_t)p << 32) | 0x9E3779B1u);
  };
  // samples on the target's side: [first, last)
  const uint32_t kz = (uint32_t)(key_of(neg ? -FAST_ZERO : FAST_ZERO) >> 32);
  const int nb = __builtin_popcountll(__ballot(sa < kz)) + __builtin_popcountll(__ballot(sb < kz));
  const int lmin = neg ? -1 : nb - 1, rmax = neg ? nb : SAMPLE_ROWS;
  auto bound = [&](int ix, int out) {
    return ix <= lmin ? (neg ? -FAST_OPEN : FAST_ZERO) : ix >= rmax ? (neg ? -FAST_ZERO : FAST_OPEN) : value(ix, out);
  };
  auto target = [&](double T) { return 0.5 * (neg ? T + lam : T - lam); };
  double c = c0;
  int il = max((int)floor(c - WDELTA * SAMPLE_ROWS) - 1, lmin), ir = min((int)ceil(c + WDELTA * SAMPLE_ROWS), rmax);
  if (neg) il = max(min(il, rmax - 3), lmin);
  else ir = min(max(ir, lmin + 3), rmax);
  double lo = bound(il, -1), hi = bound(ir, 1);
  double est = (double)(ir - il) * s.n * (1.0 / SAMPLE_ROWS);   // rows the window may list
  for (int it = 0; it < 12; ++it) {
    if (est > 0.8 * FAST_CAP) {
      // cut the bracket at three points
      double t[3], T[3];
      int ix[3];
      const bool by_sample = ir - il >= 2;
      if (by_sample) {
        const int h = max(1, (ir - il + 2) / 6), mid = min(max((int)rint(c), il + 1), ir - 1);
        ix[0] = max(mid - h, il + 1);
        ix[1] = mid;
        ix[2] = min(mid + h, ir - 1);
#pragma unroll
        for (int q = 0; q < 3; ++q) t[q] = value(ix[q], 0);
      } else {
#pragma unroll
        for (int q = 0; q < 3; ++q) t[q] = lo + (hi - lo) * (0.25 * (q + 1));
      }
      probe_pass(s, ldj, ldk, t, T);
      double dl = 0.0, dr = 0.0;
      bool hl = false, hr = false;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const double d = target(T[q]);
        if (fabs(d) <= tol) return false;
        if (d > 0.0) {
          lo = t[q];
          dl = d;
          hl = true;
          if (by_sample) il = ix[q];
        }
      }
#pragma unroll
      for (int q = 2; q >= 0; --q) {
        const double d = target(T[q]);
        if (d < 0.0) {
          hi = t[q];
          dr = d;
          hr = true;
          if (by_sample) ir = ix[q];
        }
      }
      if (by_sample) {
        const double per = Wd * (1.0 / SAMPLE_ROWS);
        c = hl && hr ? il + (ir - il) * (dl / (dl - dr)) : hl ? il + dl / per : ir + dr / per;
        est = (double)(ir - il) * s.n * (1.0 / SAMPLE_ROWS);
      } else {
        est *= 0.25;
      }
      continue;
    }
    double T;
    int count, listed;
    window_pass(s, ldj, ldk, lo, hi, fs->list, FAST_CAP, T, count, listed);
    const double D = target(T);
    if (fabs(D) <= tol) return false;
    if (D < 0.0) {
      // the target lies at or below lo
      if (il <= lmin) return false;
      hi = lo;
      ir = il;
      il = max(il - 12, lmin);
      lo = bound(il, -1);
      c = 0.5 * (il + ir);
      est = (double)(ir - il) * s.n * (1.0 / SAMPLE_ROWS);
      continue;
    }
    if (count > FAST_CAP) {
      est = count;
      double t[3], Tq[3], K = 0.0;
      if (tied_ratio(s, fs->list, listed, K, t[0], t[2]) && t[0] > lo && t[2] < hi) {
        t[1] = t[2];
        probe_pass(s, ldj, ldk, t, Tq);
        const double dl = target(Tq[0]), dr = target(Tq[2]);
        if (fabs(dl) <= tol || fabs(dr) <= tol) return false;
        if (dl > 0.0 && dr < 0.0) {
          v = K;
          const bool ok = tie_rows(s, ldj, ldk, K, t[0], t[2], 1ull, dl, tol, row);
          row = __builtin_amdgcn_readfirstlane(row);
          return ok;
        }
        lo = dr > 0.0 ? t[2] : lo;
        hi = dl < 0.0 ? t[0] : hi;
      }
      continue;
    }
    const double blo = il <= lmin && neg ? value(0, 0) : lo, bhi = ir >= rmax && !neg ? value(SAMPLE_ROWS - 1, 0) : hi;
    const int got = select_listed(s, fs, count, blo, bhi, D, tol, v, row);
    if (got == FAST_HIT) return v > lo && v < hi;
    if (got == FAST_UNSURE || ir >= rmax) return false;
    il = ir;
    lo = hi;
    ir = min(ir + 12, rmax);
    hi = bound(ir, 1);
    c = 0.5 * (il + ir);
    est = (double)(ir - il) * s.n * (1.0 / SAMPLE_ROWS);
  }
  return false;
}

// ------------------------------------------- several penalties, one segment
// The same pass with one target per lane (penalties in groups of 64): a window
// that holds every target's place in the sample is listed once, its rows are
// sorted once and every lane finds its target by a search over the prefix
// weights.  A window whose samples promise more rows than the list holds is
// taken in parts from its lower end, each part's pass serving the targets that
// lie in it (at 5918 rows and 43 penalties up to 43 passes, one per penalty,
// before).
//  The sort is of one 32-bit word per row: the place of its ratio in the
// window in 23 to 26 bits (a monotone function of the ratio) and its index in
// the list, 9 to 6 bits: one exchange, one comparison and one select per
// stage.  Neighbours in the sorted order are then checked against their exact
// ratios and rows; where they are out of order (equal ratios, or different ones
// that share a word) the rows are sorted again by further words.
// 2000 x 2000 with 64 penalties 52.2 -> 23.1 ms, 128 uneven matrices with 16
// 100 -> 40.
struct PathScratch {
  double val[FAST_CAP];             // ratios in list order, then prefix weights in sorted order
  uint32_t list[FAST_CAP];          // rows in list order, then in sorted order
};

// The listed rows in (ratio, row) order: ps->list the rows, ps->val the
// inclusive prefix weights, 64 E entries (the last repeated past count).
// [blo, bhi]: the range the words divide.  Sorts after the first keep the order
// that they find among equal words: by the rows' numbers and the place again,
// for equal ratios, and, where different ratios share a place (decimal fractions
// differ in the last bits only), by their keys' bits, lowest first, which settles
// every order (left to the exact kernel, 1200 x 300 one-decimal data at 33
// penalties took 12.0 ms, now 2.2).
template <int E>
__device__ __forceinline__ void sort_listed(const SegIO &s, PathScratch *ps, int count, double blo, double bhi) {
  constexpr int N = 64 * E, IB = E == 1 ? 6 : E == 2 ? 7 : E == 4 ? 8 : 9;
  const int lane = s.lane;
  double scale = (double)(1u << (32 - IB)) / (bhi - blo);
  scale = bhi > blo && scale < 0x1p1000 ? scale : 0.0;
  {
    int rw[E];
    double av[E], bv[E];
#pragma unroll
    for (int q = 0; q < E; ++q) rw[q] = 64 * q + lane < count ? (int)ps->list[64 * q + lane] : 0;
#pragma unroll
    for (int q = 0; q < E; ++q) {
      av[q] = sxj_at(s, rw[q]);
      bv[q] = gld(s.xk + rw[q]);
    }
#pragma unroll
    for (int q = 0; q < E; ++q) ps->val[64 * q + lane] = bv[q] / av[q];
  }
  uint32_t rw[E];
  double r[E];
#pragma unroll 1
  for (int phase = 0; phase < 6; ++phase) {
    uint32_t x[E];
#pragma unroll
    for (int q = 0; q < E; ++q) {
      const int e = 64 * q + lane;
      const uint64_t key = key_of(ps->val[e]);
      const uint32_t w = phase == 1 ? ps->list[e]
                         : phase > 2 ? (uint32_t)(key >> (23 * (phase - 3))) & 0x7FFFFFu
                                     : min((uint32_t)fmax((ps->val[e] - blo) * scale, 0.0), (1u << (32 - IB)) - 1u);
      x[q] = e < count ? (w << IB) | (uint32_t)e : ~0u;
    }
    wave_sort_u32<E>(x);
    wave_lds_sync();
    // the entries E lane + q in this order
#pragma unroll
    for (int q = 0; q < E; ++q) {
      const int id = E * lane + q < count ? (int)(x[q] & (N - 1)) : 0;
      rw[q] = ps->list[id];
      r[q] = ps->val[id];
    }
    wave_lds_sync();
    if (phase == 5) break;
    if (phase == 0 || phase == 2) {
      const double nr = __shfl_down(r[0], 1);
      const uint32_t nw = (uint32_t)__shfl_down((int)rw[0], 1);
      bool bad = false;
#pragma unroll
      for (int q = 0; q < E; ++q) {
        const double rn = q + 1 < E ? r[q + 1 < E ? q + 1 : 0] : nr;
        const uint32_t wn = q + 1 < E ? rw[q + 1 < E ? q + 1 : 0] : nw;
        bad = bad || (E * lane + q + 1 < count && !(r[q] < rn || (r[q] == rn && rw[q] < wn)));
      }
      if (__ballot(bad) == 0) break;
      if (phase == 0) continue;
    }
    // the next sort keeps this order among its equal words
#pragma unroll
    for (int q = 0; q < E; ++q)
      if (E * lane + q < count) {
        ps->list[E * lane + q] = rw[q];
        ps->val[E * lane + q] = r[q];
      }
    wave_lds_sync();
  }
  double w[E], tot = 0.0;
#pragma unroll
  for (int q = 0; q < E; ++q) {
    const bool in = E * lane + q < count;
    w[q] = in ? fabs(sxj_at(s, (int)rw[q])) : 0.0;
    tot = tot + w[q];
  }
  double run = wave_scan_dbl(tot) - tot;
  wave_lds_sync();
#pragma unroll
  for (int q = 0; q < E; ++q) {
    run = run + w[q];
    ps->val[E * lane + q] = run;
    ps->list[E * lane + q] = rw[q];
  }
  wave_lds_sync();
}

// The minimisers of segment s for the penalties of the lanes with act (lam the
// lane's penalty, between_units; tol as in fast_one; c its target's expected
// place in the sample sa, sb); v and
// row on those lanes.  false: some target is unsettled.
template <class LdJ, class LdK>
__device__ __forceinline__ bool fast_path(const SegIO &s, LdJ ldj, LdK ldk, bool neg, bool act, double lam, const double &tol,
                                          uint32_t sa, uint32_t sb, double c, PathScratch *ps, double &v, int &row) {
  constexpr double WDELTA = 0.06;
  const int lane = s.lane;
  auto value = [&](int ix, int out) {
    const uint32_t p = (uint32_t)__builtin_amdgcn_readlane((int)((ix & 1) ? sb : sa), ix >> 1) + (uint32_t)out;
    return ratio_of_key(((uint64_t)p << 32) | 0x9E3779B1u);
  };
  const uint32_t kz = (uint32_t)(key_of(neg ? -FAST_ZERO : FAST_ZERO) >> 32);
  const int nb = __builtin_popcountll(__ballot(sa < kz)) + __builtin_popcountll(__ballot(sb < kz));
  const int lmin = neg ? -1 : nb - 1, rmax = neg ? nb : SAMPLE_ROWS;
  auto bound = [&](int ix, int out) {
    return ix <= lmin ? (neg ? -FAST_OPEN : FAST_ZERO) : ix >= rmax ? (neg ? -FAST_ZERO : FAST_OPEN) : value(ix, out);
  };
  const int cl = (int)floor(c - WDELTA * SAMPLE_ROWS) - 1, cr = (int)ceil(c + WDELTA * SAMPLE_ROWS);
  const double per = (double)s.n * (1.0 / SAMPLE_ROWS);   // rows a sample stands for
  const int step = max(1, (int)(0.8 * FAST_CAP / per));   // samples a window may span
  uint64_t pend = __ballot(act), low = 0;
  // [il, iend): what the pending targets' windows span
  int il = max(min(wave_min_int_x(act ? cl : SAMPLE_ROWS), neg ? rmax - 3 : SAMPLE_ROWS), lmin);
  int iend = min(max(wave_max_int_x(act ? cr : -1), neg ? -1 : lmin + 3), rmax);
  double lo = bound(il, -1);
  int shrink = 0, start = il;
  bool jump = true;
  for (int it = 0; it < 160 && (pend | low); ++it) {
    if (pend == 0) {
      // (after a listed window or a tie's rows) targets below the first window,
      // or in a part passed over: again from further down, part by part
      if (start <= lmin && !jump) return false;
      pend = low;
      low = 0;
      jump = false;
      iend = rmax;
      il = start = max(start - 13, lmin);
      lo = bound(il, -1);
      shrink = 0;
    }
    // the next window: [lo, hi), hi at sample ir or (shrink) inside a gap
    int ir = min(il + step, max(iend, il + 1));
    ir = min(ir, rmax);
    if (ir <= il) return false;
    double hi = bound(ir, 1);
    int again = 0;                                 // shrink of the next window if this one is listed
    if (shrink > 0) {
      const int whole = 31 - __builtin_clz((unsigned)(ir - il));   // from here on one sample's gap
      if (shrink <= whole) {
        ir = il + ((ir - il) >> shrink);
        hi = bound(ir, 1);
      } else {
        // a quarter of what is left of the gap, and so on (not towards an open
        // end); the next window is the rest of it.  (A cut by what all shrinks
        // had reached, and the shrinks again for each, settled 310 of 380
        // segments of 5030 x 20 with 39 penalties in 24 passes each; now all
        // in 5.6.)
        if (shrink > whole + 12 || (neg ? il <= lmin : il + 1 >= rmax)) return false;
        hi = lo + (bound(il + 1, 1) - lo) * ldexp(1.0, 2 * (whole - shrink));
        ir = il;                                   // (the window ends inside the gap)
        again = whole;
      }
    }
    double T;
    int count, listed;
    window_pass(s, ldj, ldk, lo, hi, ps->list, FAST_CAP, T, count, listed);
    const bool mine = ((pend >> lane) & 1ull) != 0;
    if (count > FAST_CAP) {
      ++shrink;
      double t[3], Tq[3], K = 0.0;
      if (tied_ratio(s, ps->list, listed, K, t[0], t[2]) && t[0] > lo && t[2] < hi) {
        // the targets among the equal ratios, now; the window then ends before them
        t[1] = t[2];
        probe_pass(s, ldj, ldk, t, Tq);
        const double dl = 0.5 * (neg ? Tq[0] + lam : Tq[0] - lam), dr = 0.5 * (neg ? Tq[2] + lam : Tq[2] - lam);
        if (__ballot(mine && (fabs(dl) <= tol || fabs(dr) <= tol))) return false;
        const uint64_t tied = __ballot(mine && dl > 0.0 && dr < 0.0);
        if (tied) {
          int rr = 0;
          if (!tie_rows(s, ldj, ldk, K, t[0], t[2], tied, dl, tol, rr)) return false;
          if ((tied >> lane) & 1ull) {
            v = K;
            row = rr;
          }
          pend &= ~tied;
        }
        // nothing below the tie is wanted: go on above it
        if (__ballot(((pend >> lane) & 1ull) && dl < 0.0) == 0) {
          lo = t[2];
          shrink = 0;
        }
      }
      continue;
    }
    const double D = 0.5 * (neg ? T + lam : T - lam);
    if (__ballot(mine && fabs(D) <= tol)) return false;
    low |= __ballot(mine && D < 0.0);
    pend &= ~low;
    if (pend && count > 0) {
      const double blo = il <= lmin && neg ? value(0, 0) : lo, bhi = ir >= rmax && !neg ? value(SAMPLE_ROWS - 1, 0) : hi;
      if (count <= 64) sort_listed<1>(s, ps, count, blo, bhi);
      else if (count <= 128) sort_listed<2>(s, ps, count, blo, bhi);
      else if (count <= 256) sort_listed<4>(s, ps, count, blo, bhi);
      else sort_listed<8>(s, ps, count, blo, bhi);
      // first entry whose prefix weight reaches D
      int p = 0;
      for (int h = count <= 64 ? 32 : count <= 128 ? 64 : count <= 256 ? 128 : 256; h; h >>= 1)
        if (ps->val[p + h - 1] < D) p += h;
      const double at = ps->val[p], before = p > 0 ? ps->val[p - 1] : 0.0;
      const bool here = mine && D > 0.0;
      const bool hit = here && at >= D;
      const int rr = (int)ps->list[p];
      const double vv = gld(s.xk + rr) / sxj_at(s, rr);
      if (__ballot(here && (fabs(at - D) <= tol || fabs(before - D) <= tol)) ||
          __ballot(hit && !(vv > lo && vv < hi)))
        return false;
      if (hit) {
        v = vv;
        row = rr;
      }
      pend &= ~__ballot(hit);
      wave_lds_sync();
    }
    shrink = again;
    lo = hi;
    il = ir;
    if (pend) {
      // (nothing is expected before the pending targets' windows)
      const int nx = min(wave_min_int_x(((pend >> lane) & 1ull) ? cl : SAMPLE_ROWS), rmax - 1);
      if (jump && nx > il) {
        il = nx;
        lo = bound(il, -1);
      }
      iend = max(iend, il + 12);
    }
  }
  return (pend | low) == 0;
}

// RJ residuals in one pass over the rows (the sums of wave_residual, RJ at a
// time); the lanes of the first RJ bits of jm (v_l: the lane's ratio) receive
// theirs in e_l, and the bits are cleared.  The R64 trees are folded: at each
// level two trees trade halves and go on as one, the lower one on the lower
// lanes, so the adds and their pairing are those of RJ separate trees.
__device__ __forceinline__ double fold32(double a, double b, bool wide) {
  const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
  const auto l = wide ? __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false)
                      : __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
  const auto h = wide ? __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false)
                      : __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
  return __longlong_as_double((long long)(((uint64_t)h[0] << 32) | l[0])) +
         __longlong_as_double((long long)(((uint64_t)h[1] << 32) | l[1]));
}
__device__ __forceinline__ double add_down(double p, int d) {
  const uint64_t b = (uint64_t)__double_as_longlong(p);
  return p + __longlong_as_double((long long)(((uint64_t)xdown32((uint32_t)(b >> 32), d) << 32) | xdown32((uint32_t)b, d)));
}
template <int RJ, class LdJ, class LdK>
__device__ __forceinline__ void run_jobs(const SegIO &s, LdJ ldj, LdK ldk, uint64_t &jm, double v_l, double &e_l) {
  const uint64_t all = jm;
  double jv[RJ], p[RJ];
#pragma unroll
  for (int r = 0; r < RJ; ++r) {
    jv[r] = jm ? readlane_dbl(v_l, __builtin_ctzll(jm)) : 0.0;
    jm &= jm ? jm - 1 : 0;
    p[r] = 0.0;
  }
  for_row_pairs<4>(s, ldj, ldk, 0, s.T, [&](double a, double b) {
#pragma unroll
    for (int r = 0; r < RJ; ++r) {
      const double prod = jv[r] * a;
      const double d = b - prod;
      p[r] = p[r] + fabs(d);
    }
  });
  double x;
  int src;                                         // where job i ends: its bits on lane bits 5, 4 (, 3)
  const int i = lanes_below(all);
  if constexpr (RJ > 4) {
    auto at = [&](int r) { return r < RJ ? p[r] : 0.0; };
    const double q0 = fold32(fold32(p[0], p[4], true), fold32(p[2], at(6), true), false);
    const double q1 = fold32(fold32(p[1], at(5), true), fold32(p[3], at(7), true), false);
    const bool up = (threadIdx.x & 8) != 0;
    const double keep = up ? q1 : q0, send = up ? q0 : q1;
    const uint64_t sb = (uint64_t)__double_as_longlong(send);
    x = keep + __longlong_as_double((long long)(((uint64_t)xswap32((uint32_t)(sb >> 32), 8) << 32) | xswap32((uint32_t)sb, 8)));
    src = ((i & 4) << 3) | ((i & 2) << 3) | ((i & 1) << 3);
  } else if constexpr (RJ > 2) {
    x = add_down(fold32(fold32(p[0], p[2], true), fold32(p[1], p[3], true), false), 8);
    src = ((i & 2) << 4) | ((i & 1) << 4);
  } else {
    x = add_down(add_down(fold32(p[0], p[1], true), 16), 8);
    src = (i & 1) << 5;
  }
  x = add_down(add_down(add_down(x, 4), 2), 1);
  const double got = __shfl(x, src);
  if (((all >> (threadIdx.x & 63)) & 1ull) && i < RJ) e_l = got;
}

// residuals of the lanes of jm (v_l finite), up to eight per pass over the rows
template <class LdJ, class LdK>
__device__ __forceinline__ void run_all_jobs(const SegIO &s, LdJ ldj, LdK ldk, uint64_t jm, double v_l, double &e_l) {
  while (jm) {
    const int c = __builtin_popcountll(jm);
    if (c > 6) run_jobs<8>(s, ldj, ldk, jm, v_l, e_l);
    else if (c > 4) run_jobs<6>(s, ldj, ldk, jm, v_l, e_l);
    else if (c > 2) run_jobs<4>(s, ldj, ldk, jm, v_l, e_l);
    else run_jobs<2>(s, ldj, ldk, jm, v_l, e_l);
  }
}

// ------------------------------------------------- segments left to the end
// One segment by one wave with exact 128-bit sums and the general rounds:
// what the division-free kernels leave (pairs outside their range, sums too
// close to call, windows that missed).  Any number of penalties.
//  1. the sign sums dz decide the side of every penalty, the exact pass
//     where they cannot;
//  2. a key window from the row sample is listed with the exact weight below
//     it, sorted and scanned exactly;
//  3. whatever the window does not settle goes to the general rounds.
__device__ __forceinline__ void seg_exact(const SegIO &s, const ColInfo &cj, const ColInfo &ck,
                                          const unsigned short *__restrict__ smp, const double *__restrict__ lam, int L,
                                          double2 dz, const u128 *slam, WaveScratch *ws, uint64_t *lk,
                                          unsigned short *lr, int lcap, double *__restrict__ V,
                                          double *__restrict__ E, int *__restrict__ R, long long base, long long mm,
                                          int &err) {
  const int lane = s.lane, n = s.n, T = s.T;
  const double Wd = cj.W;
  const double Wk = ck.W;

  // 1. sign sums.  |x_ik / x_ij| can underflow to 0 only if the exponent
  // fields differ by more than 1000: the column ranges rule that out for the
  // whole segment in the usual case, else the exact pass decides.
    const bool unc = sign_sums_unsure(cj, ck, dz);

  bool have_exact = false;
  ExactSides ex;
  const u128 W = cj.wfix;
  // (a) the side of every penalty: v_k = 0, or the minimiser is negative
  // (1) or positive (2).  A <= B makes the nonzero side the same for every
  // penalty of the segment.
  uint64_t nz0 = 0, nz1 = 0;                     // bit t: v_k != 0 at penalty t
  int sd = 0;
  // one penalty per lane, in groups of 64
  for (int g0 = 0; g0 < L; g0 += 64) {
    const int t = g0 + lane;
    const bool in = t < L;
    int side = 0;
    if (in) side = sign_sum_side(dz, lam[t], Wd, 0.0, unc);
    if (__ballot(side == 3)) {
      if (!have_exact) {
        ex = exact_sides(s);
        have_exact = true;
      }
      if (side == 3) {
        const u128 lamf = slam[t], WpL = W + lamf;
        side = ((ex.A << 1) <= WpL && W <= (ex.B << 1) + lamf) ? 0 : ((ex.A << 1) > WpL ? 1 : 2);
      }
    }
    const uint64_t nzm = __ballot(side != 0);
    if (g0 == 0) nz0 = nzm;
    else nz1 = nzm;
    // every nonzero penalty has the same side (A <= B)
    if (nzm) sd = __builtin_amdgcn_readlane(side, __builtin_ctzll(nzm));
  }
  if ((nz0 | nz1) == 0) {
    // v_k = 0 at every penalty: e_jk = R64 sum of |x_ik|
    for (int t = lane; t < L; t += 64) {
      V[t * mm + base] = 0.0;
      E[t * mm + base] = Wk;
      R[t * mm + base] = -1;
    }
    return;
  }
  const bool neg = sd == 1;
  const uint64_t klo0 = neg ? 0ull : KEY_ZERO, khi0 = neg ? KEY_ZERO - 1 : KEY_NONE - 1;
  // the sample's keys (top 32 bits), sorted across the wave
  const int sr0 = smp[lane], sr1 = smp[64 + lane];
  uint32_t sa = sample_key32(s, sr0, __builtin_amdgcn_rcp(sxj_at(s, sr0))),
           sb = sample_key32(s, sr1, __builtin_amdgcn_rcp(sxj_at(s, sr1)));
  wave_sort2_u32_x(sa, sb, lane);
  // sample position ix as a lower or upper key bound
  auto sample_lo = [&](int ix) { return sample_key(ws->ckey, ix); };
  auto sample_hi = [&](int ix) { return sample_lo(ix) | 0xFFFFFFFFull; };
  int prev_row = -2;
  double prev_e = 0.0;
  // penalties in groups of 64, lane l holding the target of penalty 64 g + l
  for (int g = 0; 64 * g < L; ++g) {
    const uint64_t nzg = g ? nz1 : nz0;
    const int tl = 64 * g + lane;
    const bool act = ((nzg >> lane) & 1ull) != 0;
    // negative side: first S_p > (W + lambda)/2; positive: first S_p >= (W - lambda)/2
    double q = 2.0;
    if (act) {
      const double lamt = lam[tl];
      q = (neg ? 0.5 * (Wd + lamt) : 0.5 * (Wd - lamt)) / Wd;
    }
    // window bounds on the targets' weight fractions (positive doubles
    // order as their bit patterns)
    const double qmin = __longlong_as_double((long long)wave_min_u64_x((uint64_t)__double_as_longlong(fmax(q, 0.0))));
    const double qmax =
        __longlong_as_double((long long)wave_max_u64_x((uint64_t)__double_as_longlong(act ? fmax(q, 0.0) : 0.0)));
    // the sorted sample (index 2 l + c in lane l) in the wave's LDS scratch,
    // which the rounds of an earlier group may have used
    ws->ckey[lane] = ((uint64_t)sb << 32) | sa;
    wave_lds_sync();
    uint64_t okey = KEY_NONE;
    int orow = -1;
    bool hit = false;
    // the ratios of the weighted row sample bracket the targets: a key
    // window; one exact pass lists the window's elements, one sort serves
    // every penalty.  A window too wide for the list is retried per penalty.
    for (int pass = 0; nzg && pass <= 64; ++pass) {
      double wlo = qmin, whi = qmax;
      bool mine = act;
      if (pass > 0) {
        const int t = pass - 1;
        if (!((nzg >> t) & 1ull) || __builtin_amdgcn_readlane((int)hit, t)) continue;
        wlo = whi = readlane_dbl(q, t);
        mine = lane == t;
      }
      constexpr double WDELTA = 0.08;
      const int ilo = (int)floor((wlo - WDELTA) * SAMPLE_ROWS) - 1;
      const int ihi = (int)ceil((whi + WDELTA) * SAMPLE_ROWS);
      uint64_t plo = klo0, phi = khi0;
      if (ilo >= 0 && ilo < SAMPLE_ROWS) {
        const uint64_t v = sample_lo(ilo);
        plo = v > plo ? v : plo;
      }
      if (ihi >= 0 && ihi < SAMPLE_ROWS) {
        const uint64_t v = sample_hi(ihi);
        phi = v < phi ? v : phi;
      }
      if (plo > khi0) plo = khi0;
      if (phi < plo) phi = plo;

      bool ovf = false;
      bool probe = false;
      ws->steps = 0;
      while (true) {
        int nwin = 0;
        u128 Slw;
        {
          // exact pass: weight at or below the window; the window's
          // elements go to the LDS list (in row order).  The weight below
          // the window in three FP64 sums of 37-bit chunks (whole numbers
          // below 2^53: every add is exact)
          double c0s = 0.0, c1s = 0.0, c2s = 0.0;
          // columns j and k are read one slot ahead so the loads overlap
          // the divide; the weight reuses x_ij
          auto ldj = [&](int i) { return sxj_at(s, i < n ? i : 0); };
          auto ldk = [&](int i) { return gld(s.xk + (i < n ? i : 0)); };
          double anext = ldj(lane), bnext = ldk(lane);
          for (int tt = 0; tt < T; ++tt) {
            const int i = lane + 64 * tt;
            const double a = anext, b = bnext;
            if (tt + 1 < T) {
              anext = ldj(i + 64);
              bnext = ldk(i + 64);
            }
            const uint64_t key = key_of_pair(i < n, a, b);
            const bool valid = key != KEY_NONE;
            const bool le_lo = valid && key <= plo;
            const bool inwin = valid && key > plo && key <= phi;
            {
              double c0, c1, c2;
              weight_chunks(a, s.e0, c0, c1, c2);
              // masked adds as fma with a 0/1 factor: the same exact sums
              // (whole numbers below 2^53; c 0 adds +0), one op each
              const double fl = le_lo ? 1.0 : 0.0;
              c0s = fma(c0, fl, c0s);
              c1s = fma(c1, fl, c1s);
              c2s = fma(c2, fl, c2s);
            }
            const uint64_t wm = __ballot(inwin);
            const int pos = nwin + lanes_below(wm);
            nwin += __builtin_popcountll(wm);
            if (inwin && pos < lcap) {
              lk[pos] = key;
              lr[pos] = (unsigned short)i;
            }
          }
          Slw = chunks_to_u128(wave_sum_dbl_x(c0s), wave_sum_dbl_x(c1s), wave_sum_dbl_x(c2s));
          nwin = uni_int(nwin);
          wave_lds_sync();
        }
        const u128 lamf = act ? slam[tl] : (u128)0;
        const u128 tau = neg ? ((W + lamf) >> 1) + 1 : (W - lamf + 1) >> 1;
        if (probe || nwin > lcap) {
          // one target: a window too full for the list is bisected.  (blo,
          // phi] holds the target and about bcnt elements; a probe pass
          // over (plo, phi], plo inside it, gives the weight at or below
          // plo, which names the half.
          const uint64_t tm = __ballot(mine && !hit);
          if (__builtin_popcountll(tm) == 1 && ws->steps < 12) {
            const bool at_or_below = readlane_u128(tau, __builtin_ctzll(tm)) <= Slw;
            bool more = true;
            if (!probe) {
              // the window itself: the target at or below it is a miss
              if (at_or_below) {
                ovf = true;
                break;
              }
              ws->blo = plo;
              ws->bcnt = nwin;
            } else if (at_or_below) {
              // at or below the probe point: (blo, plo], not listed yet
              ws->bcnt -= nwin;
              phi = plo;
              plo = ws->blo;
            } else {
              ws->blo = plo;
              ws->bcnt = nwin;
              more = nwin > lcap;
            }
            probe = false;
            if (more) {
              ws->steps += 1;
              if (ws->bcnt <= lcap) continue;      // list (blo, phi] in one pass
              uint64_t mid;
              if (!window_midpoint(ws->ckey, plo, phi, mid)) {
                ovf = true;
                break;
              }
              plo = mid;
              probe = true;
              continue;
            }
          }
          probe = false;
        }
        if (nwin > lcap) {
          ovf = true;
          break;
        }
        const bool want = mine && !hit;
        const uint64_t wantm = __ballot(want);
        u128 Slo = Slw;
        if (__builtin_popcountll(wantm) == 1 && nwin > 128) {
          // one target: only the quarter of the window that holds it is
          // sorted.  Three sample keys around the target split the list;
          // the exact weights below them pick the part (a contiguous range
          // of the sorted order), which is compacted to the list's front.
          const u128 tau1 = uni_u128(shfl_u128(tau, __builtin_ctzll(wantm)));
          uint64_t piv[3];
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            int ix = (int)floor((wlo + 0.04 * (c - 1)) * SAMPLE_ROWS);
            ix = ix < 0 ? 0 : (ix >= SAMPLE_ROWS ? SAMPLE_ROWS - 1 : ix);
            piv[c] = sample_lo(ix);
          }
          piv[1] = piv[1] < piv[0] ? piv[0] : piv[1];
          piv[2] = piv[2] < piv[1] ? piv[1] : piv[2];
          u128 a0 = 0, a1 = 0, a2 = 0;
          for (int e = lane; e < nwin; e += 64) {
            const uint64_t key = lk[e];
            const u128 w = fixed_of_col(sxj_at(s, lr[e]), s.e0);
            a0 += key < piv[0] ? w : (u128)0;
            a1 += key < piv[1] ? w : (u128)0;
            a2 += key < piv[2] ? w : (u128)0;
          }
          a0 = wave_sum_u128_x(a0);
          a1 = wave_sum_u128_x(a1);
          a2 = wave_sum_u128_x(a2);
          const int c = (Slw + a0 < tau1 ? 1 : 0) + (Slw + a1 < tau1 ? 1 : 0) + (Slw + a2 < tau1 ? 1 : 0);
          const uint64_t plo2 = c == 0 ? 0 : piv[c - 1], phi2 = c == 3 ? KEY_NONE : piv[c];
          Slo = Slw + (c == 0 ? (u128)0 : (c == 1 ? a0 : (c == 2 ? a1 : a2)));
          {
            // stable in-place compaction: an element never moves above its
            // own slot, so slots not yet read are never overwritten
            int kept = 0;
            for (int e0 = 0; e0 < nwin; e0 += 64) {
              const int e = e0 + lane;
              const bool in = e < nwin;
              const uint64_t key = in ? lk[e] : 0;
              const unsigned short row = in ? lr[e] : 0;
              const bool keep = in && (c == 0 || key >= plo2) && (c == 3 || key < phi2);
              const uint64_t km = __ballot(keep);
              const int d = kept + lanes_below(km);
              kept += __builtin_popcountll(km);
              if (keep) {
                lk[d] = key;
                lr[d] = row;
              }
            }
            nwin = uni_int(kept);
            wave_lds_sync();
          }
        }
        const int N = wave_sort_list(lk, lr, nwin, lane);
        u128 tot, incl;
        wave_list_sums(s, lk, lr, N >> 6, tot, incl);
        uint64_t k2 = KEY_NONE;
        int r2 = -1;
        bool h2 = false;
        wave_resolve(s, lk, lr, N >> 6, Slo, tot, incl, want, tau, k2, r2, h2);
        if (h2) {
          okey = k2;
          orow = r2;
          hit = true;
        }
        wave_lds_sync();
        break;
      }
      if (ovf) {
        // the list cannot hold the window: after the shared window, retry
        // each penalty with its own; a single penalty goes to the rounds
        if (pass == 0 && __builtin_popcountll(nzg) == 1) break;
        continue;
      }
      // the shared window held: the targets it missed go to the rounds
      if (pass == 0) break;
    }

    // targets the windows missed: rounds over the whole side
    uint64_t left = __ballot(act && !hit);
    while (left) {
      const int t = __builtin_ctzll(left);
      left &= left - 1;
      if (!have_exact) {
        ex = exact_sides(s);
        have_exact = true;
      }
      const u128 lamf = slam[64 * g + t];
      const u128 tau = neg ? ((W + lamf) >> 1) + 1 : (W - lamf + 1) >> 1;
      uint64_t k2 = KEY_NONE;
      int r2 = -1;
      const ColSrc cs{s, (u128)0, 0};
      wave_select_rounds(s, cs, klo0, khi0, neg ? (u128)0 : ex.B, neg ? ex.A : W, neg ? 0 : ex.N + ex.Z,
                         neg ? ex.N : ex.NV, tau, ws, k2, r2, err);
      if (lane == t) {
        okey = k2;
        orow = r2;
      }
    }

    // residuals, reused while the selected row repeats: the group's targets
    // whose row differs from the previous target's are the jobs, scored up to
    // eight at a time in one pass over the rows (2000 x 1000
    // through this kernel with 16 penalties 19.5 ms a pass each, now 17.1); one job,
    // or an infinite ratio, takes a pass of its own
    const int tend = min(L, 64 * g + 64);
    const int cnt = tend - 64 * g;
    int orw_l = -1;
    double v_l = 0.0;
    if (lane < cnt && ((nzg >> lane) & 1ull)) {
      orw_l = orow;
      v_l = ratio_of_key(okey);
    }
    int prv = __shfl_up(orw_l, 1);
    if (lane == 0) prv = prev_row;
    const bool need = lane < cnt && orw_l >= 0 && orw_l != prv;
    const uint64_t needm = __ballot(need);
    double e_l = 0.0;
    uint64_t many = __ballot(need && __builtin_isfinite(v_l));
    many = __builtin_popcountll(many) > 1 ? many : 0;
    if (many) {
      const __amdgpu_buffer_rsrc_t rk = col_rsrc(s.xk, n), rj = col_rsrc(s.sxj, n);
      run_all_jobs(s, [&](int i) { return col_ld(rj, i * 8); }, [&](int i) { return col_ld(rk, i * 8); }, many, v_l, e_l);
    }
    for (uint64_t jm = needm & ~many; jm; jm &= jm - 1) {
      const int jl = __builtin_ctzll(jm);
      const double e1 = readlane_dbl(wave_residual(s, readlane_dbl(v_l, jl)), 0);
      if (lane == jl) e_l = e1;
    }
    // each target takes the e of the last job at or before it (or the
    // previous group's last e when its row continues from there)
    double e_t;
    if (orw_l < 0) {
      e_t = Wk;                                    // R64 sum of |x_ik|
    } else {
      const uint64_t upto = needm & (lane == 63 ? ~0ull : ((2ull << lane) - 1ull));
      const double ej = __shfl(e_l, upto ? 63 - __builtin_clzll(upto) : 0);
      e_t = upto ? ej : prev_e;
    }
    if (lane < cnt) {
      const int t = 64 * g + lane;
      V[t * mm + base] = orw_l >= 0 ? v_l : 0.0;
      E[t * mm + base] = e_t;
      R[t * mm + base] = orw_l;
    }
    prev_row = __builtin_amdgcn_readlane(orw_l, cnt - 1);
    prev_e = readlane_dbl(e_t, cnt - 1);
  }
}

// The parts that the division-free kernels listed, cut into 2^cut pieces (every
// 2^cut-th segment) as long as four pieces per wave are not reached: few segments
// go one to a wave (20000 x 40 with 8 penalties by two and by eight 39 and 120
// ms), and the waves take the pieces in turn, since many are empty and a claim of
// each, about 6 ns one after the other, costs more than it evens out (150 x 600
// one-decimal data 1.00 ms, in turn 0.70).  Longer lists go part by part, by claims
// from *next (49 x 438 of subnormals 0.89 ms, in turn 1.02), and so do the pieces of
// long_segments (rows times penalties: 6727 x 133 of subnormals with 61 penalties
// 342 ms, in turn 499).  The list is final: it belongs to earlier kernels.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4)))
k_seg_rest(const ProbDesc *__restrict__ P, const int *__restrict__ wstart, int B, const double *__restrict__ lam_all,
           const ColInfo *__restrict__ ci, const unsigned short *__restrict__ smp, const double2 *__restrict__ DZ,
           double *__restrict__ V, double *__restrict__ E, int *__restrict__ R, int *__restrict__ segflags,
           const int *__restrict__ cand, const int *__restrict__ gate, int gate_on,
           TodoList td, int *__restrict__ next, int Lmax, int lcap, bool long_segments) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  if (gate && *gate != gate_on) return;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  u128 *slam = (u128 *)(smem + wave * rest_wave_bytes(Lmax, lcap));
  WaveScratch *ws = (WaveScratch *)(slam + Lmax);
  uint64_t *lk = (uint64_t *)(ws + 1);
  unsigned short *lr = (unsigned short *)(lk + lcap);
  const int count = *td.count, waves = (int)gridDim.x * SEG_WAVES;
  int cut = 0;
  while (cut < 3 && ((long long)count << cut) < 4ll * waves) ++cut;
  const int pieces = count << cut;
  const bool claims = (cut == 0 || long_segments) && pieces > waves;
  for (int e = blockIdx.x * SEG_WAVES + wave, next_e; e < pieces; e = next_e) {
    const TodoPart part = td.list[e % count];
    const int w = uni_int(part.word), p = uni_int(part.part), piece = e / count;
    uint64_t bits = td.bits[w];
    next_e = e + waves;
    if (claims) {
      int c = 0;
      if (lane == 0) c = atomicAdd(next, 1);
      next_e = waves + uni_int(c);
    }
    for (int q = rest_rank(p); q > 0; --q) bits &= bits - 1;
    int size = min(rest_rank(p + 1) - rest_rank(p), __builtin_popcountll(bits));
    if (size <= piece) continue;
    const int b = find_owner(wstart, B, w);
    const ProbDesc d = P[b];
    const int wpr = (d.m + 63) >> 6, wl = w - wstart[b], jj = wl / wpr, k0 = (wl - jj * wpr) * 64;
    const int j = cand ? cand[jj] : jj;
    const ColInfo cj = ci[d.col_off + j];
    const double *lam = lam_all + d.lam_off;
    const int T = (d.n + 63) >> 6;
    int err = 0;
    wave_lds_sync();
    for (int t = lane; t < d.L; t += 64) slam[t] = lambda_fixed(lam[t], cj.e0);
    wave_lds_sync();
    for (int q = 0; q < size; ++q, bits &= bits - 1) {
      if ((q & ((1 << cut) - 1)) != piece) continue;
      const int k = k0 + __builtin_ctzll(bits);
      const SegIO s{d.X + (long long)k * d.ld, d.X + (long long)j * d.ld, d.n, T, cj.e0, lane, false};
      seg_exact(s, cj, ci[d.col_off + k], smp + (long long)(d.col_off + j) * SAMPLE_ROWS, lam, d.L,
                DZ[d.pair_off + (long long)j * d.m + k], slam, ws, lk, lr, lcap, V + d.ws_off, E + d.ws_off,
                R + d.ws_off, (long long)j * d.m + k, (long long)d.m * d.m, err);
    }
    if (err && lane == 0) atomicOr(segflags + d.col_off + j, err);
  }
}

// The items of the segment kernels.  Every workgroup pulls work items from
// the counter of its XCD until none is left.  Explicit items (a batch) come in
// one list per XCD, [xstart[x], xstart[x + 1]).  With items == nullptr the
// items of problem 0 are implicit and routed by XCD: its k range is cut into
// SEG_XCDS * chunks equal parts, XCD x owns parts [x chunks, (x + 1) chunks)
// and enumerates them part by part, every preserved column j (or cand[jj])
// within a part, so the columns k that the workgroups of one XCD stream stay
// in its L2.  Workgroups are dispatched to the XCDs round-robin (blockIdx mod
// 8); one whose XCD has no item left takes items of the next XCDs (the
// routing only affects where data is cached, never the results).  nitems =
// items per XCD (implicit) or in total (explicit).
constexpr int SEG_XCDS = 8;
struct ItemQueue {
  const WorkItem *items;
  int nitems, chunks;
  int *counter;
  const int *xstart;
};

// The next item of the workgroup (every thread calls it): false when none is
// left.  jj: the item's row in the masks; near: 0 before the first call.
__device__ __forceinline__ bool next_item(const ItemQueue &q, const ProbDesc *__restrict__ P,
                                          const int *__restrict__ cand, int ncand, int *s_item, WorkItem &it, int &jj, int &near) {
  while (true) {
    if (threadIdx.x < 64) {
      // the XCD of the last item (lane near's) is tried at once; when it has
      // none left, lanes 0 .. 7 look at the counters together (trying them one
      // atomic after the other cost every workgroup about 6 us at its end) and
      // the nearest XCD at or after home with items left is tried
      int g = -1;
      const int lane = threadIdx.x, x = (blockIdx.x + lane) % SEG_XCDS;
      int begin = 0, have = 0;
      if (lane < SEG_XCDS) {
        begin = q.items ? q.xstart[x] : x * q.nitems;
        have = q.items ? q.xstart[x + 1] - begin : q.nitems;
      }
      uint64_t open = __ballot(have > 0);
      open = (open >> near) & 1ull ? 1ull << near : open;
      while (open != 0) {
        const int l = __builtin_ctzll(open);
        int c = 0;
        if (lane == l) c = atomicAdd(q.counter + x, 1);
        c = __builtin_amdgcn_readlane(c, l);
        if (c < __builtin_amdgcn_readlane(have, l)) {
          g = __builtin_amdgcn_readlane(begin, l) + c;
          near = l;
          break;
        }
        const int seen = lane < SEG_XCDS ? __hip_atomic_load(q.counter + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        open = __ballot(lane < SEG_XCDS && seen < have);
      }
      if (lane == 0) *s_item = g;
    }
    __syncthreads();
    const int g = uni_int(*s_item);
    __syncthreads();
    if (g < 0) return false;
    if (q.items) {
      it = q.items[g];
      jj = it.j;
      return true;
    }
    const int m0 = P[0].m, mj = cand ? ncand : m0;
    const int x = g / q.nitems, c = g % q.nitems;
    const int part = x * q.chunks + c / mj;
    jj = c % mj;
    const int kchunk = (m0 + SEG_XCDS * q.chunks - 1) / (SEG_XCDS * q.chunks);
    it.b = 0;
    it.j = cand ? cand[jj] : jj;
    it.kbeg = min(m0, part * kchunk);
    it.kend = min(m0, it.kbeg + kchunk);
    if (it.kbeg < it.kend) return true;            // (else an empty part of a narrow matrix)
  }
}

// The live segments of an item: k in [kbeg, kend) not settled by
// k_zero_segments.  Lane l holds word l of the item's mask inverted (bit b:
// segment 64 (w0 + l) + b is live) and the live count of the words below it;
// the waves claim live segments by their rank, so settled ones cost no claim.
// An item of more than SEG_MASK_WORDS words counts every segment as live.
struct LiveSegs {
  uint64_t live;
  int kpre, nlive, w0, nwords, kbeg;
  bool use_mask;
  __device__ __forceinline__ LiveSegs(const unsigned long long *__restrict__ maskrow, int kbeg_, int kend, int lane) {
    kbeg = kbeg_;
    w0 = kbeg >> 6;
    nwords = kend > kbeg ? ((kend - 1) >> 6) - w0 + 1 : 0;
    use_mask = nwords <= SEG_MASK_WORDS;
    live = 0;
    kpre = 0;
    nlive = kend - kbeg;
    if (use_mask) {
      if (lane < nwords) {
        const int lo = max(kbeg - 64 * (w0 + lane), 0), hi = min(kend - 64 * (w0 + lane), 64);
        const uint64_t range = (hi == 64 ? ~0ull : (1ull << hi) - 1ull) & ~((1ull << lo) - 1ull);
        live = ~maskrow[w0 + lane] & range;
      }
      const int cnt = __builtin_popcountll(live), incl = wave_scan_int(cnt);
      kpre = incl - cnt;
      nlive = __builtin_amdgcn_readlane(incl, 63);
    }
  }
  // the c-th live segment: the last word whose live prefix is <= c, then the
  // (c - prefix)-th set bit of that word
  __device__ __forceinline__ int at(int c, int lane) const {
    if (!use_mask) return kbeg + c;
    const int w = __builtin_popcountll(__ballot(lane < nwords && kpre <= c)) - 1;
    const uint64_t lw = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(live >> 32), w) << 32) |
                        (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)live, w);
    const int r = c - __builtin_amdgcn_readlane(kpre, w);
    return 64 * (w0 + w) + __builtin_ctzll(__ballot(((lw >> lane) & 1ull) && lanes_below(lw) == r));
  }
};

// One penalty per problem: every live segment by the division-free path, one
// wave per segment.  kLdsJ: every problem's column j fits the launch's LDS
// copy (sxj_rows rows), else it is read from global memory (it stays in L2
// across the item's k).  gate (optional): the kernel does nothing unless
// *gate == gate_on.
// Bound by VALU issue: about 1150 instructions per live segment of 2000 rows,
// 0.68 of the issue slots (2600 and 0.89 with a guarded window test, IEEE
// divisions and 64-bit sorts).  Four waves per SIMD: with five or six the
// registers spill or gain nothing (3.9 to 4.6 ms).  2000 x 2000 6.25 -> 3.57
// ms; 10000 x 4000 49.0 -> 31.4 ms, 32 of its columns 3.03 -> 0.85.
template <bool kLdsJ>
__global__ void __launch_bounds__(64 * SEG_WAVES_MAX) __attribute__((amdgpu_waves_per_eu(4)))
k_seg_fast(const ProbDesc *__restrict__ P, ItemQueue queue, const double *__restrict__ lam_all,
           const ColInfo *__restrict__ ci, const unsigned short *__restrict__ smp, const double2 *__restrict__ DZ,
           double *__restrict__ V, double *__restrict__ E, int *__restrict__ R, const int *__restrict__ cand, int ncand,
           const int *__restrict__ gate, int gate_on, const unsigned long long *__restrict__ segmask, TodoList td,
           int sxj_rows) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int s_item, knext;
  if (gate && *gate != gate_on) return;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double *sxj_lds = (double *)smem;
  FastScratch *fs = (FastScratch *)(smem + (kLdsJ ? seg_sxj_bytes(sxj_rows) : 0)) + wave;
  WorkItem it;
  int jj, near = 0;
  while (next_item(queue, P, cand, ncand, &s_item, it, jj, near)) {
    const ProbDesc d = P[it.b];
    const int n = d.n, m = d.m, T = (n + 63) >> 6, j = it.j;
    const ColInfo *cis = ci + d.col_off;
    const ColInfo cj = cis[j];
    const double *xjg = d.X + (long long)j * d.ld;
    if constexpr (kLdsJ)
      for (int i = threadIdx.x; i < T * 64; i += blockDim.x) sxj_lds[i] = i < n ? xjg[i] : 0.0;
    const double *__restrict__ sxj = kLdsJ ? (const double *)sxj_lds : xjg;
    if (threadIdx.x == 0) knext = 0;
    __syncthreads();
    const long long word0 = d.mask_off + (long long)jj * ((m + 63) >> 6);
    const LiveSegs segs(segmask + word0, it.kbeg, it.kend, lane);
    // the sample of column j: two rows per lane, and the reciprocals of their
    // x_ij (sample keys need neither an exact quotient nor one per segment)
    const unsigned short *sm = smp + (long long)(d.col_off + j) * SAMPLE_ROWS;
    const int sr0 = sm[lane], sr1 = sm[64 + lane];
    const double sv0 = __builtin_amdgcn_rcp(sxj[sr0]), sv1 = __builtin_amdgcn_rcp(sxj[sr1]);
    const double Wd = cj.W, unit = cj.unit, tol = segment_tol(Wd, unit);
    const double lam = between_units(lam_all[d.lam_off], unit);
    // the targets' places in the sample
    const double cneg = 0.5 * SAMPLE_ROWS * (Wd + lam) / Wd, cpos = 0.5 * SAMPLE_ROWS * (Wd - lam) / Wd;
    const FastRange fast(cj, !cj.flags);
    const double2 *DZj = DZ + d.pair_off + (long long)j * m;
    // claims are taken one segment ahead, and the next segment's sign sums and
    // sample are loaded before the current one's residual
    int claim = 0;
    if (lane == 0) claim = atomicAdd(&knext, 1);
    int c = __builtin_amdgcn_readlane(claim, 0);
    if (lane == 0) claim = atomicAdd(&knext, 1);
    int k = c < segs.nlive ? segs.at(c, lane) : it.kbeg;
    double2 dz = DZj[k];
    double b0 = gld(d.X + (long long)k * d.ld + sr0), b1 = gld(d.X + (long long)k * d.ld + sr1);
    while (c < segs.nlive) {
      const SegIO s{d.X + (long long)k * d.ld, sxj, n, T, cj.e0, lane, kLdsJ};
      const ColInfo ck = cis[k];
      double v = 0.0, e = ck.W;
      int row = -1;
      bool left = false;
      if (k == j || cj.flags) {
        v = k == j ? 1.0 : __longlong_as_double(0x7ff8000000000000ll);
        e = 0.0;
      } else {
        const int side = sign_sum_side(dz, lam, Wd, unit, sign_sums_unsure(cj, ck, dz));
        left = side == 3 || (side != 0 && !fast.has(ck));
        if (side != 0 && !left) {
          const bool neg = side == 1;
          uint32_t sx[2] = {(uint32_t)(key_of(b0 * sv0 + 0.0) >> 32), (uint32_t)(key_of(b1 * sv1 + 0.0) >> 32)};
          wave_sort_u32<2>(sx);
          const __amdgpu_buffer_rsrc_t rk = col_rsrc(s.xk, n), rj = col_rsrc(kLdsJ ? s.xk : s.sxj, n);
          auto ldj = [&](int i) { return sxj_pad(s, rj, i); };
          auto ldk = [&](int i) { return col_ld(rk, i * 8); };
          left = !fast_one(s, ldj, ldk, neg, lam, Wd, tol, sx[0], sx[1], neg ? cneg : cpos, fs, v, row);
        }
      }
      const long long base = d.ws_off + (long long)j * m + k;
      const int kc = k;
      c = __builtin_amdgcn_readlane(claim, 0);
      if (lane == 0) claim = atomicAdd(&knext, 1);
      k = c < segs.nlive ? segs.at(c, lane) : it.kbeg;
      dz = DZj[k];
      b0 = gld(d.X + (long long)k * d.ld + sr0);
      b1 = gld(d.X + (long long)k * d.ld + sr1);
      if (left) {
        if (lane == 0) leave_segment(td, word0 + (kc >> 6), kc & 63);
        continue;
      }
      if (row >= 0) e = wave_residual(s, v);
      if (lane == 0) {
        V[base] = v;
        E[base] = e;
        R[base] = row;
      }
    }
    __syncthreads();   // the LDS is reused by the next item
  }
}

// Several penalties per problem: every live segment, one wave per segment, a
// penalty per lane in groups of 64: the window pass and the sort once per segment,
// then a residual per distinct row (7 of 64 penalties on average at 2000 x 2000; up
// to eight per pass over the rows).  There, with 64 penalties, it takes 0.63 of the
// VALU issue slots (8.9e9 instructions, 23.1 ms) and moves 75 GB, 25 of them
// stores: a segment's results lie 8 m^2 bytes apart, each in a line of its own.
template <bool kLdsJ>
__global__ void __launch_bounds__(64 * SEG_WAVES_MAX) __attribute__((amdgpu_waves_per_eu(4)))
k_seg_path(const ProbDesc *__restrict__ P, ItemQueue queue, const double *__restrict__ lam_all,
           const ColInfo *__restrict__ ci, const unsigned short *__restrict__ smp, const double2 *__restrict__ DZ,
           double *__restrict__ V, double *__restrict__ E, int *__restrict__ R, const int *__restrict__ cand, int ncand,
           const int *__restrict__ gate, int gate_on, const unsigned long long *__restrict__ segmask, TodoList td,
           int sxj_rows) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ int s_item, knext;
  __shared__ double s_unit, s_tol;
  if (gate && *gate != gate_on) return;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  double *sxj_lds = (double *)smem;
  PathScratch *ps = (PathScratch *)(smem + (kLdsJ ? seg_sxj_bytes(sxj_rows) : 0)) + wave;
  WorkItem it;
  int jj, near = 0;
  while (next_item(queue, P, cand, ncand, &s_item, it, jj, near)) {
    const ProbDesc d = P[it.b];
    const int n = d.n, m = d.m, L = d.L, T = (n + 63) >> 6, j = it.j;
    const ColInfo *cis = ci + d.col_off;
    const ColInfo cj = cis[j];
    const double *xjg = d.X + (long long)j * d.ld;
    if constexpr (kLdsJ)
      for (int i = threadIdx.x; i < T * 64; i += blockDim.x) sxj_lds[i] = i < n ? xjg[i] : 0.0;
    const double *__restrict__ sxj = kLdsJ ? (const double *)sxj_lds : xjg;
    if (threadIdx.x == 0) {
      knext = 0;
      s_unit = cj.unit;
      s_tol = segment_tol(cj.W, cj.unit);
    }
    __syncthreads();
    const long long word0 = d.mask_off + (long long)jj * ((m + 63) >> 6), mm = (long long)m * m;
    const LiveSegs segs(segmask + word0, it.kbeg, it.kend, lane);
    const unsigned short *sm = smp + (long long)(d.col_off + j) * SAMPLE_ROWS;
    const int sr0 = sm[lane], sr1 = sm[64 + lane];
    const double sv0 = __builtin_amdgcn_rcp(sxj[sr0]), sv1 = __builtin_amdgcn_rcp(sxj[sr1]);
    const double *lams = lam_all + d.lam_off;
    const double Wd = cj.W;
    const FastRange fast(cj, !cj.flags);
    const double2 *DZj = DZ + d.pair_off + (long long)j * m;
    int claim = 0;
    if (lane == 0) claim = atomicAdd(&knext, 1);
    while (true) {
      const int cq = __builtin_amdgcn_readlane(claim, 0);
      if (cq >= segs.nlive) break;
      if (lane == 0) claim = atomicAdd(&knext, 1);
      const int k = segs.at(cq, lane);
      const long long base = d.ws_off + (long long)j * m + k;
      const SegIO s{d.X + (long long)k * d.ld, sxj, n, T, cj.e0, lane, kLdsJ};
      const ColInfo ck = cis[k];
      const double2 dz = DZj[k];
      const bool unc = sign_sums_unsure(cj, ck, dz), plain = k == j || cj.flags;
      bool left = false, sorted = false;
      uint32_t sa = 0, sb = 0;
      int prev_row = -2;
      double prev_e = 0.0;
      const __amdgpu_buffer_rsrc_t rk = col_rsrc(s.xk, n), rj = col_rsrc(kLdsJ ? s.xk : s.sxj, n);
      auto ldj = [&](int i) { return sxj_pad(s, rj, i); };
      auto ldk = [&](int i) { return col_ld(rk, i * 8); };
      for (int t0 = 0; t0 < L && !left; t0 += 64) {
        const int t = t0 + lane;
        const double unit = s_unit, lam = between_units(t < L ? lams[t] : 0.0, unit);
        double v = plain ? (k == j ? 1.0 : __longlong_as_double(0x7ff8000000000000ll)) : 0.0, e = plain ? 0.0 : ck.W;
        int row = -1;
        const int side = t < L && !plain ? sign_sum_side(dz, lam, Wd, unit, unc) : 0;
        const uint64_t nz = __ballot(side != 0);
        left = __ballot(side == 3) != 0 || (nz && !fast.has(ck));
        if (nz && !left) {
          // (every penalty of a segment has the minimiser on the same side)
          const bool neg = __builtin_amdgcn_readlane(side, __builtin_ctzll(nz)) == 1;
          if (!sorted) {
            uint32_t x[2] = {(uint32_t)(key_of(gld(s.xk + sr0) * sv0 + 0.0) >> 32),
                             (uint32_t)(key_of(gld(s.xk + sr1) * sv1 + 0.0) >> 32)};
            wave_sort_u32<2>(x);
            sa = x[0];
            sb = x[1];
            sorted = true;
          }
          const double u = 0.5 * SAMPLE_ROWS * lam / Wd;
          left = !fast_path(s, ldj, ldk, neg, side != 0, lam, s_tol, sa, sb, 0.5 * SAMPLE_ROWS + (neg ? u : -u), ps, v, row);
          if (!left) {
            // residuals, reused while the selected row repeats: the targets whose
            // row differs from the previous target's are the jobs
            int prv = __shfl_up(row, 1);
            if (lane == 0) prv = prev_row;
            const uint64_t needm = __ballot(row >= 0 && row != prv);
            double e_l = 0.0;
            run_all_jobs(s, ldj, ldk, needm, v, e_l);
            // each target takes the e of the last job at or before it (or the
            // previous group's last e when its row continues from there)
            const uint64_t upto = needm & (lane == 63 ? ~0ull : ((2ull << lane) - 1ull));
            const double ej = __shfl(e_l, upto ? 63 - __builtin_clzll(upto) : 0);
            e = row < 0 ? ck.W : upto ? ej : prev_e;
          }
        }
        if (!left) {
          if (t < L) {
            V[t * mm + base] = v;
            E[t * mm + base] = e;
            R[t * mm + base] = row;
          }
          prev_row = __builtin_amdgcn_readlane(row, 63);
          prev_e = readlane_dbl(e, 63);
        }
      }
      if (left && lane == 0) leave_segment(td, word0 + (k >> 6), k & 63);
    }
    __syncthreads();   // the LDS is reused by the next item
  }
}

// ------------------------------------------------------------ per-j objective
// One wave per (problem, lambda_t, j): E_j = R64_k e_jk, P_j = R64_k |v_k|,
// z_j = E_j + fl(lambda P_j).  zflag marks an infinite or NaN v_k.
// zstart[b] = first (t, j) slot of problem b (sum of L m over earlier ones).
__global__ void __launch_bounds__(64)
k_reduce_batch(const ProbDesc *__restrict__ P, const int *__restrict__ zstart, int B,
               const double *__restrict__ lam_all, const double *__restrict__ V, const double *__restrict__ E,
               double *__restrict__ Z, int *__restrict__ zflag, const int *__restrict__ jmask,
               const int *__restrict__ gate, int gate_on, const unsigned long long *__restrict__ segmask,
               const ColInfo *__restrict__ ci) {
  if (gate && *gate != gate_on) return;
  const long long g = blockIdx.x;
  const int lane = threadIdx.x;
  const int b = find_owner(zstart, B, g);
  const ProbDesc d = P[b];
  const int local = (int)(g - zstart[b]);
  const int t = local / d.m, j = local % d.m;
  if (jmask && !jmask[j]) {
    // not a candidate (problem 0 only): never the argmin
    if (lane == 0) {
      Z[d.z_off + (long long)t * d.m + j] = __longlong_as_double(0x7ff0000000000000ll);
      zflag[d.z_off + (long long)t * d.m + j] = 0;
    }
    return;
  }
  const long long off = d.ws_off + ((long long)t * d.m + j) * d.m;
  double pe = 0.0, pv = 0.0;
  int bad = 0;
  // (several penalties: the segments of the mask are not in V and E)
  const unsigned long long *zero = d.L > 1 ? segmask + d.mask_off + (long long)j * ((d.m + 63) >> 6) : nullptr;
  for (int k = lane; k < d.m; k += 64) {
    const bool z = zero && ((zero[k >> 6] >> lane) & 1ull);
    pe = pe + (z ? ci[d.col_off + k].W : E[off + k]);
    const double a = z ? 0.0 : fabs(V[off + k]);
    pv = pv + a;
    bad |= !isfinite(a);
  }
  pe = wave_r64_tree(pe);
  pv = wave_r64_tree(pv);
  bad = wave_max_int(bad);
  if (lane == 0) {
    const double pen = lam_all[d.lam_off + t] * pv;
    const double z = pe + pen;
    Z[d.z_off + (long long)t * d.m + j] = z;
    zflag[d.z_off + (long long)t * d.m + j] = bad;
  }
}

// -------------------------------------------------------------- argmin/gather
// One workgroup per (problem, lambda_t): j* = lexicographic argmin of
// (z_j, j); gathers v*, rows, z_all.  The workgroup of t = 0 also folds the
// problem's flags into its status word.  ostart[b] = sum of L over earlier
// problems.
__global__ void __launch_bounds__(256)
k_argmin_batch(const ProbDesc *__restrict__ P, const int *__restrict__ ostart, int B,
               const double *__restrict__ V, const int *__restrict__ R, const double *__restrict__ Z,
               const int *__restrict__ zflag, const ColInfo *__restrict__ ci, const int *__restrict__ segflags,
               const int *__restrict__ jmask, const int *__restrict__ gate, int gate_on, int *__restrict__ sticky,
               const unsigned long long *__restrict__ segmask) {
  __shared__ double sz[256];
  __shared__ int sj[256];
  __shared__ int sflag[256];
  if (gate && *gate != gate_on) return;
  const int g = blockIdx.x, tid = threadIdx.x;
  const int b = find_owner(ostart, B, g);
  const ProbDesc d = P[b];
  const int t = g - ostart[b];
  const int m = d.m;
  const double *z = Z + d.z_off + (long long)t * m;
  double bz = 0.0;
  int bj = -1;
  for (int j = tid; j < m; j += blockDim.x) {
    double v = z[j];
    if (isnan(v)) v = __longlong_as_double(0x7ff0000000000000ll);
    if (bj < 0 || v < bz) { bz = v; bj = j; }
  }
  sz[tid] = bz;
  sj[tid] = bj;
  __syncthreads();
  for (int s = blockDim.x >> 1; s > 0; s >>= 1) {
    if (tid < s) {
      const int oj = sj[tid + s];
      const double oz = sz[tid + s];
      if (oj >= 0 && (sj[tid] < 0 || oz < sz[tid] || (oz == sz[tid] && oj < sj[tid]))) {
        sz[tid] = oz;
        sj[tid] = oj;
      }
    }
    __syncthreads();
  }
  const int js = sj[0];
  const long long src = d.ws_off + ((long long)t * m + js) * m;
  const unsigned long long *zero = d.L > 1 ? segmask + d.mask_off + (long long)js * ((m + 63) >> 6) : nullptr;
  for (int k = tid; k < m; k += blockDim.x) {
    const bool zk = zero && ((zero[k >> 6] >> (k & 63)) & 1ull);
    d.Vout[(long long)t * m + k] = zk ? 0.0 : V[src + k];
    if (d.ROWout) d.ROWout[(long long)t * m + k] = zk ? -1 : R[src + k];
    if (d.ZALLout) d.ZALLout[(long long)t * m + k] = z[k];
  }
  if (tid == 0) {
    d.Jout[t] = js;
    d.OBJout[t] = z[js];
  }
  if (t == 0 && (d.status || sticky)) {
    // condition bits; the status is the first that applies of: non-finite
    // input, too-wide column, selection bound, overflowed ratio
    int f = 0;
    for (int j = tid; j < m; j += blockDim.x) {
      const int cf = ci[d.col_off + j].flags;
      if (cf & COL_NONFINITE) f |= 1;
      if (cf & COL_WIDE) f |= 2;
      if (segflags[d.col_off + j] && (!jmask || jmask[j])) f |= 4;
    }
    for (long long q = tid; q < (long long)d.L * m; q += blockDim.x)
      if (zflag[d.z_off + q]) f |= 8;
    sflag[tid] = f;
    __syncthreads();
    for (int s = blockDim.x >> 1; s > 0; s >>= 1) {
      if (tid < s) sflag[tid] |= sflag[tid + s];
      __syncthreads();
    }
    if (tid == 0) {
      const int bb = sflag[0];
      const int st = (bb & 1) ? L1LINE_ENONFINITE : (bb & 2) ? L1LINE_EWIDE : (bb & 4) ? L1LINE_EINTERNAL
                   : (bb & 8) ? L1LINE_ERANGE : L1LINE_OK;
      if (d.status) *d.status = st;
      // the context's sticky error keeps the first data-dependent error
      if (sticky && st != L1LINE_OK) atomicCAS(sticky, 0, st);
    }
  }
}

// Column statistics to user buffers.
__global__ void k_colstats_out(const ColInfo *__restrict__ ci, int m, double *__restrict__ W,
                               int *__restrict__ zeros, int *__restrict__ status) {
  __shared__ int sflag[256];
  int f = 0;
  for (int j = threadIdx.x; j < m; j += blockDim.x) {
    ColInfo c = ci[j];
    if (W) W[j] = c.W;
    if (zeros) zeros[j] = c.zeros;
    if (c.flags & COL_NONFINITE) f = L1LINE_ENONFINITE;
  }
  sflag[threadIdx.x] = f;
  __syncthreads();
  for (int s = blockDim.x >> 1; s > 0; s >>= 1) {
    if (threadIdx.x < s) sflag[threadIdx.x] = min(sflag[threadIdx.x], sflag[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0 && status) *status = sflag[0];
}
