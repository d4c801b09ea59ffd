// Whole-cube and single-region kernels: moments, histogram, radix-select
// median, and the fused two-pass trio.
#include <math.h>

#include <mutex>
#include <vector>

#include "tsa_internal.hpp"

namespace tsa {

// ---------------------------------------------------------------------------
// small utility kernels
// ---------------------------------------------------------------------------
// Several disjoint ranges filled by one launch: on a small cube the gaps
// between dependent launches, not the bytes, set the time of the clears.
struct FillRange {
  uint32_t* p;
  uint64_t n;
  uint32_t v, pad;
};
constexpr int kMaxFills = 6;
// The selection states of a call are set in the same launch (st: where, null
// for none).
struct FillSet {
  FillRange r[kMaxFills];
  int count, pad;
  SelState* st[2];
  SelState init[2];
};
__global__ void k_fill_set(FillSet f) {
  if (blockIdx.x == 0 && threadIdx.x < 2 && f.st[threadIdx.x]) *f.st[threadIdx.x] = f.init[threadIdx.x];
  const uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (uint64_t)gridDim.x * blockDim.x;
  for (int k = 0; k < f.count; ++k)
    for (uint64_t i = i0; i < f.r[k].n; i += stride) f.r[k].p[i] = f.r[k].v;
}

// ---------------------------------------------------------------------------
// moments pass: one Partial per block
// ---------------------------------------------------------------------------
// float32 lanes sum about a shift of their own and the partials hold
// (n, mean, M2); int16 partials hold exact integer sums.  float32 runs and tiles (ROWS)
// are kernels of their own: see ShiftMomVecAcc.
template <int DT, int VEC, bool NT, bool ROWS>
__global__ __launch_bounds__(1024) void k_moments(Geom g, Partial* __restrict__ parts) {
  using Acc = std::conditional_t<DT == 1, MomAcc<1>, std::conditional_t<ROWS, ShiftMomAcc, ShiftMomVecAcc>>;
  __shared__ MomShared sm;
  Acc acc;
  if constexpr (DT == 1) {
    walk<DT, VEC, kUnrollOf<DT, VEC>, NT>(g, acc);
    block_store_partial(acc, sm, parts + blockIdx.x);
  } else {
    if constexpr (ROWS)
      walk_tiles<DT, VEC, kUnrollOf<DT, VEC>, NT>(g, acc);
    else
      walk_run<DT, VEC, kUnrollOf<DT, VEC>, NT>(g, acc);
    block_store_centered(acc, sm, parts + blockIdx.x);
  }
}

// ---------------------------------------------------------------------------
// fixed-range histogram pass (Section 4.1)
// ---------------------------------------------------------------------------
template <int DT, int VEC, bool NT>
__global__ __launch_bounds__(1024) void k_hist(Geom g, float lo, float hi, float scale, int32_t nbins,
                                               uint32_t rshift, uint64_t* __restrict__ counts,
                                               uint64_t* __restrict__ outl) {
  extern __shared__ uint32_t lds[];
  __shared__ uint32_t osm[32];
  lds_zero(lds, ((uint32_t)nbins << rshift) + kTrash);
  __syncthreads();
  HistAcc<DT> h(lds, lo, hi, scale, nbins, rshift);
  walk<DT, VEC, kUnrollOf<DT, VEC>, NT>(g, h);
  __syncthreads();
  lds_flush(lds, (uint32_t)nbins, rshift, counts);
  block_add_outliers(h.below, h.above, outl, osm);
}

// ---------------------------------------------------------------------------
// histograms of more bins than one LDS copy holds (the standalone call)
// ---------------------------------------------------------------------------
// Where the window of kWinBins 32-bit LDS counters goes: 65536 voxels spread
// evenly over the region are binned (the stated formula) and counted per group
// of nbins/256 bins; the block that ends last writes the first bin of the run
// of groups that holds the most.  Only the placement depends on the sample;
// k_hist_win counts every voxel exactly wherever the window is.  Bound by the
// latency of the scattered loads, so one per lane over 64 blocks (one block
// with 64 per lane took 85 to 150 us).
constexpr int kPlaceThreads = 1024, kPlaceBlocks = 64, kPlaceGroups = 256;

template <int DT>
__global__ __launch_bounds__(kPlaceThreads) void k_hist_place(const void* base, int64_t nx, int64_t ny, tsa_region b,
                                                              float lo, float hi, float scale, int32_t nbins,
                                                              uint32_t* __restrict__ groups, Arrive* arrive,
                                                              int32_t* __restrict__ w0_out) {
  using T = typename Ty<DT>::T;
  __shared__ uint32_t coarse[kPlaceGroups], below[kPlaceGroups + 1];
  __shared__ uint64_t best;
  const int t = threadIdx.x;
  uint32_t gshift = 0;  // bins per group: 2^gshift, at most kPlaceGroups groups
  while (((uint32_t)(nbins - 1) >> gshift) >= (uint32_t)kPlaceGroups) ++gshift;
  if (t < kPlaceGroups) coarse[t] = 0u;
  __syncthreads();
  const int64_t lx = b.x1 - b.x0, ly = b.y1 - b.y0, lz = b.z1 - b.z0;
  const uint64_t vol = (uint64_t)lx * (uint64_t)ly * (uint64_t)lz;
  const uint64_t ns = (uint64_t)kPlaceThreads * kPlaceBlocks, s = (uint64_t)blockIdx.x * kPlaceThreads + t;
  const uint64_t i = (uint64_t)(((unsigned __int128)s * vol) / ns);  // < vol
  const int64_t x = (int64_t)(i % (uint64_t)lx), r = (int64_t)(i / (uint64_t)lx);
  const int64_t y = r % ly, z = r / ly;
  const float v = (float)((const T*)base)[(b.z0 + z) * nx * ny + (b.y0 + y) * nx + (b.x0 + x)];
  if (v >= lo && v <= hi) {
    const int32_t bin = min(max((int32_t)((v - lo) * scale), 0), nbins - 1);
    atomicAdd(&coarse[(uint32_t)bin >> gshift], 1u);
  }
  __syncthreads();
  if (t < kPlaceGroups && coarse[t]) atomicAdd(groups + t, coarse[t]);
  if (!last_block(arrive)) return;
  if (t == 0) {
    best = 0;
    below[0] = 0;
  }
  if (t < kPlaceGroups) coarse[t] = groups[t];
  __syncthreads();
  if (t < kWave) {  // below[g]: samples in groups before g
    uint32_t c[kPlaceGroups / kWave], sum = 0;
#pragma unroll
    for (int k = 0; k < kPlaceGroups / kWave; ++k) {
      sum += coarse[t * (kPlaceGroups / kWave) + k];
      c[k] = sum;
    }
    const uint32_t before = wave_scan_incl_u32(sum) - sum;
#pragma unroll
    for (int k = 0; k < kPlaceGroups / kWave; ++k) below[t * (kPlaceGroups / kWave) + k + 1] = before + c[k];
  }
  __syncthreads();
  const int32_t ngroups = (int32_t)(((uint32_t)(nbins - 1) >> gshift) + 1);
  const int32_t wg = min((int32_t)(kWinBins >> gshift), ngroups);  // groups the window spans
  if (t + wg <= ngroups)  // the fullest run, the first of equals
    atomicMax((unsigned long long*)&best, ((unsigned long long)(below[t + wg] - below[t]) << 32) | (uint32_t)(kPlaceGroups - t));
  __syncthreads();
  if (t == 0) {
    int32_t w0 = (kPlaceGroups - (int32_t)(uint32_t)best) << gshift;
    if (w0 > nbins - (int32_t)kWinBins) w0 = max(nbins - (int32_t)kWinBins, 0);
    *w0_out = w0;
  }
}

template <int DT, int VEC, bool NT>
__global__ __launch_bounds__(1024) void k_hist_win(Geom g, float lo, float hi, float scale, int32_t nbins,
                                                   const int32_t* __restrict__ w0p, uint64_t* __restrict__ counts,
                                                   uint64_t* __restrict__ outl) {
  extern __shared__ uint32_t lds[];  // kWinBins window counters
  __shared__ uint32_t osm[32];
  const int32_t w0 = *w0p;
  lds_zero(lds, kWinBins);
  __syncthreads();
  HistWinOutAcc<DT> h{lds, lo, hi, scale, nbins - 1, w0, counts};
  walk<DT, VEC, kUnrollOf<DT, VEC>, NT>(g, h);
  __syncthreads();
  const uint32_t nw = (uint32_t)min((int32_t)kWinBins, nbins - w0);
  for (uint32_t i = threadIdx.x; i < nw; i += blockDim.x) {
    const uint32_t c = lds[i];
    if (c) atomicAdd((unsigned long long*)(counts + w0 + i), (unsigned long long)c);
  }
  block_add_outliers(h.below, h.above, outl, osm);
}

// ---------------------------------------------------------------------------
// digit selection (one block)
// ---------------------------------------------------------------------------
TSA_DEV double value_of_key(uint32_t k, int dtype) {
  return dtype == 0 ? (double)__uint_as_float(f32bits_of_key(k)) : (double)i16_of_key(k);
}

struct SelectShared {
  uint64_t wsum[16];
  uint32_t found;
};

// Whole block: choose the digit of the current level from its histogram.
// Level 1 also fixes n and the rank k = floor((n-1)/2) of the lower median.
// When the key is complete, writes the median (and, if write_counts, the
// count fields) to *out.
// With qout != NULL the finished selection goes to qout[0..2] = (value, width of
// the bucket it came from (0 when all digits were selected), count) instead of
// out->median.  st->rank_mode / q / levels select the rank and an early stop.
TSA_DEV void select_level(int level, const uint64_t* __restrict__ hist, SelState* st, int dtype, uint64_t volume,
                          tsa_result* out, bool write_counts, SelectShared& sm, double* qout = nullptr) {
  if (st->done) return;
  const int nb = level == 3 ? kBins3 : kBins1;
  const int shift = level == 1 ? kShift1 : level == 2 ? kShift2 : 0;
  const int t = threadIdx.x, bs = blockDim.x;
  const int per = (nb + bs - 1) / bs;  // at most 16: blocks have 256 threads or more
  const int b0 = t * per;
  uint64_t h[16], local = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) h[i] = (i < per && b0 + i < nb) ? hist[b0 + i] : 0;  // all in flight at once
#pragma unroll
  for (int i = 0; i < 16; ++i) local += h[i];
  // block exclusive scan of `local`
  const int lane = t % kWave, w = t / kWave;
  const uint64_t inc = wave_scan_incl_u64(local);
  if (lane == kWave - 1) sm.wsum[w] = inc;
  if (t == 0) sm.found = 0;
  __syncthreads();
  uint64_t base = inc - local, total = 0;
  for (int i = 0; i < bs / kWave; ++i) {
    if (i < w) base += sm.wsum[i];
    total += sm.wsum[i];
  }
  uint64_t n = level == 1 ? total : st->n;
  if (level == 1 && n == 0) {
    __syncthreads();
    if (t == 0) {
      st->n = 0;
      st->done = 1;
      if (qout) {
        qout[0] = qout[1] = __builtin_nan("");
        qout[2] = 0.0;
      }
      out->median = __builtin_nan("");
      if (write_counts) {
        out->count = 0;
        out->nan_count = volume;
        out->status = TSA_OK;
      }
    }
    return;
  }
  uint64_t k = st->k;
  if (level == 1) {
    if (st->rank_mode) {
      const double kk = floor(st->q * (double)(n - 1));
      k = kk <= 0.0 ? 0 : kk >= (double)(n - 1) ? n - 1 : (uint64_t)kk;
    } else {
      k = (n - 1) / 2;
    }
  }
  __syncthreads();  // every thread has read st before it changes
  if (local > 0 && k >= base && k < base + local) {
    uint64_t cum = base, bucket = 0, below = base;
    int d = b0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {  // the last bin that starts at or below k and is not empty
      if (h[i] && k >= below) {
        d = b0 + i;
        cum = below;
        bucket = h[i];
      }
      below += h[i];
    }
    const uint32_t prefix = (level == 1 ? 0u : st->prefix) | ((uint32_t)d << shift);
    st->n = n;
    st->k = k - cum;
    st->bucket_n = bucket;
    st->prefix = prefix;
    st->level = level;
    if (level == 1) st->compact = bucket <= st->cand_cap ? 1u : 0u;
    const bool exact = level == 3 || (dtype == 1 && level == 2);
    const bool complete = exact || (st->levels >= 1 && (uint32_t)level >= st->levels);
    if (complete) {
      st->done = 1;
      st->result_key = prefix;
      if (qout) {
        // the bucket [prefix, prefix | rest] holds the rank: its smallest value
        // and its width bound the early answer
        uint32_t rest = level == 1 ? 0x000FFFFFu : level == 2 ? 0xFFu : 0u;
        if (dtype == 1) rest &= 0xFFFF0000u;
        double lo = value_of_key(prefix, dtype), hi = value_of_key(prefix | rest, dtype);
        if (lo != lo) lo = -__builtin_inf();
        if (hi != hi) hi = __builtin_inf();
        qout[0] = lo;
        qout[1] = exact ? 0.0 : hi - lo;
        qout[2] = (double)n;
      }
      out->median = value_of_key(prefix, dtype);
      if (write_counts) {
        out->count = n;
        out->nan_count = volume - n;
        out->status = TSA_OK;
      }
    }
    sm.found = 1;
  }
  __syncthreads();
  if (t == 0 && !sm.found) {  // inconsistent histogram: never expected
    st->done = 1;
    out->median = __builtin_nan("");
    out->status = TSA_EDEVICE;
  }
}

// What the last block of a digit pass needs to choose the digit.
struct Tail {
  tsa_result* out;
  double* qout;
  uint64_t volume;
  Arrive* arrive;  // by digit; null: the pass goes out in several launches, the digit is chosen by k_select
  int32_t dtype, write_counts;
};
TSA_DEV void select_tail(int level, const uint64_t* hist, SelState* st, const Tail& tl) {
  __shared__ SelectShared sm;
  if (!tl.arrive || !last_block(tl.arrive + (level - 1))) return;
  select_level(level, hist, st, tl.dtype, tl.volume, tl.out, tl.write_counts != 0, sm, tl.qout);
}

// ---------------------------------------------------------------------------
// radix selection: level passes over the cube
// ---------------------------------------------------------------------------
template <int DT, int VEC, bool NT>
__global__ __launch_bounds__(1024) void k_level1(Geom g, uint32_t rshift, SelState* __restrict__ st,
                                                 uint64_t* __restrict__ hist1, Tail tl) {
  extern __shared__ uint32_t lds[];
  if (st->done) return;
  lds_zero(lds, ((uint32_t)kBins1 << rshift) + kTrash);
  __syncthreads();
  Digit1Acc<DT> d(lds, rshift);
  walk<DT, VEC, kUnrollOf<DT, VEC>, NT>(g, d);
  __syncthreads();
  lds_flush_digits<DT>(lds, rshift, hist1);
  select_tail(1, hist1, st, tl);
}

template <int DT, int VEC, bool NT>
__global__ __launch_bounds__(1024) void k_level2(Geom g, SelState* __restrict__ st, uint64_t* __restrict__ hist2,
                                                 uint32_t* __restrict__ cand, Tail tl) {
  __shared__ uint32_t lds[kBins2];
  __shared__ CandShared cs;
  if (st->done) return;
  lds_zero(lds, kBins2);
  __syncthreads();
  Level2Acc<DT> a(lds, st->prefix, true, st->compact != 0, cand_sink(cs, cand, &st->ncand, st->cand_cap));
  walk<DT, VEC, kUnrollOf<DT, VEC>, NT>(g, a);
  a.finish();
  __syncthreads();
  lds_flush(lds, kBins2, 0, hist2);
  select_tail(2, hist2, st, tl);
}

// Level 3 reads the candidate list when level 2 made one, else the cube.
// first = 0: one more slab of a scan cut into slabs (the candidates, when
// there are any, were counted with the first).  hc: pass B's histogram copies
// to add up (none for a selection alone); the launch's blocks share the bins.
struct HistCopies {
  const uint64_t* copies;
  uint64_t* counts;
  int32_t nbins;
};
template <int DT, int VEC, bool NT>
__global__ __launch_bounds__(1024) void k_level3(Geom g, SelState* __restrict__ st, uint64_t* __restrict__ hist3,
                                                 const uint32_t* __restrict__ cand, int first, Tail tl,
                                                 HistCopies hc) {
  __shared__ uint32_t lds[kBins3];
  if (hc.copies) {
    for (uint32_t b = blockIdx.x * blockDim.x + threadIdx.x; b < (uint32_t)hc.nbins; b += gridDim.x * blockDim.x) {
      uint64_t c = 0;
#pragma unroll
      for (int k = 0; k < kHistCopies; ++k) c += hc.copies[(size_t)k * (uint32_t)hc.nbins + b];
      hc.counts[b] = c;
    }
  }
  if (st->done || (st->compact && !first)) return;
  lds_zero(lds, kBins3);
  __syncthreads();
  const uint32_t p2 = st->prefix >> kShift2;
  if (st->compact) {
    const uint32_t n = min(st->ncand, st->cand_cap);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
      const uint32_t key = cand[i];
      if ((key >> kShift2) == p2) lds_inc(lds, key & 0xFFu);
    }
  } else {
    Level3Acc<DT> a{lds, p2};
    walk<DT, VEC, kUnrollOf<DT, VEC>, NT>(g, a);
  }
  __syncthreads();
  lds_flush(lds, kBins3, 0, hist3);
  select_tail(3, hist3, st, tl);
}

// ---------------------------------------------------------------------------
// epilogues of one block: moments merge and digit selection
// ---------------------------------------------------------------------------

// Per-thread arrays of a block's merge (32 bytes a thread).
struct MergeScratch {
  double *n, *m, *q;
  uint32_t *kmin, *kmax;
};
TSA_DEV MergeScratch merge_scratch(double* d) {
  const uint32_t bs = blockDim.x;
  uint32_t* u = (uint32_t*)(d + 3 * bs);
  return MergeScratch{d, d + bs, d + 2 * bs, u, u + bs};
}

// Whole block: merge np partials in a fixed order (each thread a strided
// sequence, then a pairwise tree) and write the moments fields of *out.
// Returns (in every thread) the global count and min/max keys.
// centered: the partials hold (mean about ref, M2) (k_moments' float32
// lanes); they are merged about one reference, the ref of the first partial
// with a finite mean, which the mean gets back at the end.
TSA_DEV void merge_moments(const Partial* __restrict__ parts, int np, int dtype, uint64_t volume, tsa_result* out,
                           const MergeScratch& sm, uint64_t& n_out, uint32_t& kmin_out, uint32_t& kmax_out,
                           bool centered = false) {
  __shared__ int first;
  const int t = threadIdx.x, bs = blockDim.x;
  double ref0 = 0.0;
  if (centered) {
    if (t == 0) first = np;
    __syncthreads();
    for (int i = t; i < np; i += bs) {
      const Partial& p = parts[i];
      if (p.n && __builtin_isfinite(p.s)) {
        atomicMin(&first, i);
        break;
      }
    }
    __syncthreads();
    if (first < np) ref0 = parts[first].ref;
  }
  double n = 0.0, m = 0.0, q = 0.0;
  uint32_t mn = 0xFFFFFFFFu, mx = 0u;
  for (int i = t; i < np; i += bs) {
    const Partial p = parts[i];
    double pn, pm, pq;
    partial_stats(p, dtype, pn, pm, pq, centered, ref0);
    chan_merge(n, m, q, pn, pm, pq);
    if (p.n) {
      mn = min(mn, p.kmin);
      mx = max(mx, p.kmax);
    }
  }
  sm.n[t] = n;
  sm.m[t] = m;
  sm.q[t] = q;
  sm.kmin[t] = mn;
  sm.kmax[t] = mx;
  __syncthreads();
  for (int s = bs / 2; s > 0; s >>= 1) {
    if (t < s) {
      double a = sm.n[t], b = sm.m[t], c = sm.q[t];
      chan_merge(a, b, c, sm.n[t + s], sm.m[t + s], sm.q[t + s]);
      sm.n[t] = a;
      sm.m[t] = b;
      sm.q[t] = c;
      sm.kmin[t] = min(sm.kmin[t], sm.kmin[t + s]);
      sm.kmax[t] = max(sm.kmax[t], sm.kmax[t + s]);
    }
    __syncthreads();
  }
  const double N = sm.n[0];
  const uint64_t cnt = (uint64_t)N;
  n_out = cnt;
  kmin_out = sm.kmin[0];
  kmax_out = sm.kmax[0];
  if (t == 0) {
    out->count = cnt;
    out->nan_count = volume - cnt;
    out->status = TSA_OK;
    if (cnt == 0) {
      out->mean = out->m2 = out->std = out->min = out->max = __builtin_nan("");
    } else {
      const double vmin = value_of_key(sm.kmin[0], dtype), vmax = value_of_key(sm.kmax[0], dtype);
      out->min = vmin;
      out->max = vmax;
      if (sm.kmin[0] == sm.kmax[0]) {  // every valid voxel holds the same value
        out->mean = vmin;
        out->m2 = 0.0;
        out->std = 0.0;
      } else {
        const double m2 = sm.q[0] < 0.0 ? 0.0 : sm.q[0];  // NaN (infinite values) stays
        out->mean = ref0 + sm.m[0];
        out->m2 = m2;
        out->std = sqrt(m2 / N);
      }
    }
  }
  __syncthreads();
}

__global__ __launch_bounds__(1024) void k_moments_merge(const Partial* __restrict__ parts, int np, int dtype,
                                                        uint64_t volume, tsa_result* out) {
  __shared__ double sm[4 * 1024];
  uint64_t n;
  uint32_t a, b;
  merge_moments(parts, np, dtype, volume, out, merge_scratch(sm), n, a, b, dtype == 0);
}

__global__ __launch_bounds__(1024) void k_select(int level, const uint64_t* __restrict__ hist, SelState* st,
                                                 int dtype, uint64_t volume, tsa_result* out, int write_counts,
                                                 double* qout) {
  __shared__ SelectShared sm;
  select_level(level, hist, st, dtype, volume, out, write_counts != 0, sm, qout);
}

// ---------------------------------------------------------------------------
// median absolute deviation: the radix passes over d = |x - m|
// ---------------------------------------------------------------------------
template <int DT>
TSA_DEV void median_of_state(const SelState* med, float& mf, int32_t& mi) {
  const uint32_t k = med->result_key;
  mf = __uint_as_float(f32bits_of_key(k));
  mi = i16_of_key(k);
}

template <int DT, int VEC, bool NT>
__global__ __launch_bounds__(1024) void k_mlevel1(Geom g, uint32_t rshift, const SelState* __restrict__ med,
                                                  SelState* __restrict__ st, uint64_t* __restrict__ hist1, Tail tl) {
  extern __shared__ uint32_t lds[];
  if (!med->done || med->n == 0 || st->done) return;  // no value: st is left unfinished
  lds_zero(lds, ((uint32_t)kBins1 << rshift) + kTrash);
  __syncthreads();
  float mf;
  int32_t mi;
  median_of_state<DT>(med, mf, mi);
  AbsDev<DT, Digit1Acc<0>> a{Digit1Acc<0>(lds, rshift), mf, mi};
  walk<DT, VEC, kUnrollOf<DT, VEC>, NT>(g, a);
  __syncthreads();
  lds_flush_digits<0>(lds, rshift, hist1);
  select_tail(1, hist1, st, tl);
}

template <int DT, int VEC, bool NT>
__global__ __launch_bounds__(1024) void k_mlevel2(Geom g, const SelState* __restrict__ med, SelState* __restrict__ st,
                                                  uint64_t* __restrict__ hist2, uint32_t* __restrict__ cand, Tail tl) {
  __shared__ uint32_t lds[kBins2];
  __shared__ CandShared cs;
  if (st->level != 1 || st->done) return;
  lds_zero(lds, kBins2);
  __syncthreads();
  float mf;
  int32_t mi;
  median_of_state<DT>(med, mf, mi);
  AbsDev<DT, Level2Acc<0>> a{
      Level2Acc<0>(lds, st->prefix, true, st->compact != 0, cand_sink(cs, cand, &st->ncand, st->cand_cap)), mf, mi};
  walk<DT, VEC, kUnrollOf<DT, VEC>, NT>(g, a);
  a.inner.finish();
  __syncthreads();
  lds_flush(lds, kBins2, 0, hist2);
  select_tail(2, hist2, st, tl);
}

// out[0..2] = (median, MAD, count); NaN, NaN, 0 without a valid voxel.
TSA_DEV void mad_finish(const SelState* med, const SelState* st, int dtype, double* out) {
  if (med->n == 0 || !med->done || !st->done) {
    out[0] = out[1] = __builtin_nan("");
    out[2] = (double)med->n;
    return;
  }
  out[0] = value_of_key(med->result_key, dtype);
  out[1] = (double)__uint_as_float(f32bits_of_key(st->result_key));
  out[2] = (double)med->n;
}

template <int DT, int VEC, bool NT>
__global__ __launch_bounds__(1024) void k_mlevel3(Geom g, const SelState* __restrict__ med, SelState* __restrict__ st,
                                                  uint64_t* __restrict__ hist3, const uint32_t* __restrict__ cand,
                                                  Tail tl, int med_dtype, double* __restrict__ out) {
  __shared__ uint32_t lds[kBins3];
  __shared__ SelectShared ssm;
  if (st->level != 2 || st->done) {  // the same for every block: the state was left by earlier launches
    if (blockIdx.x == 0 && threadIdx.x == 0) mad_finish(med, st, med_dtype, out);
    return;
  }
  lds_zero(lds, kBins3);
  __syncthreads();
  const uint32_t p2 = st->prefix >> kShift2;
  if (st->compact) {
    const uint32_t n = min(st->ncand, st->cand_cap);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
      const uint32_t key = cand[i];
      if ((key >> kShift2) == p2) lds_inc(lds, key & 0xFFu);
    }
  } else {
    float mf;
    int32_t mi;
    median_of_state<DT>(med, mf, mi);
    AbsDev<DT, Level3Acc<0>> a{Level3Acc<0>{lds, p2}, mf, mi};
    walk<DT, VEC, kUnrollOf<DT, VEC>, NT>(g, a);
  }
  __syncthreads();
  lds_flush(lds, kBins3, 0, hist3);
  if (!last_block(tl.arrive + 2)) return;
  select_level(3, hist3, st, tl.dtype, tl.volume, tl.out, false, ssm);
  __syncthreads();
  if (threadIdx.x == 0) mad_finish(med, st, med_dtype, out);
}

// ---------------------------------------------------------------------------
// fused trio: pass A (moments + digit 1), mid (merge + select 1 + range),
// pass B (histogram over [min, max] + level 2)
// ---------------------------------------------------------------------------
// Pass A's last block: merges the moments, fixes the histogram's range and the
// shift of the second moment, and chooses the first digit.  lds: 8 kBins1
// bytes and 32 a thread (the larger).
TSA_DEV void mid_tail(const Partial* parts, int np, int dtype, uint64_t volume, int32_t nbins,
                      const uint64_t* __restrict__ hist1, SelState* st, tsa_result* out, uint64_t* lds) {
  __shared__ SelectShared ssm;
  uint64_t n;
  uint32_t kmin, kmax;
  merge_moments(parts, np, dtype, volume, out, merge_scratch((double*)lds), n, kmin, kmax);
  if (threadIdx.x == 0) {
    uint32_t ok = 0;
    float lo = 0.f, hi = 0.f, scale = 0.f;
    if (n > 0) {
      lo = (float)value_of_key(kmin, dtype);
      hi = (float)value_of_key(kmax, dtype);
      ok = own_range(lo, hi, nbins, scale) ? 1u : 0u;
    }
    st->hist_ok = ok;
    st->lo = lo;
    st->hi = hi;
    st->scale = scale;
    // pass B recomputes M2 about c = fl32(mean) when the values differ (float32 cubes)
    const double mean = out->mean;
    const bool von = dtype == 0 && n > 0 && kmin != kmax && isfinite(mean) &&
                     one_pass_m2_at_risk(mean, out->m2 / (double)n);
    st->shift = von ? (float)mean : 0.0f;
    st->var_on = von ? 1u : 0u;
    out->flags = ok ? 0 : TSA_FLAG_HIST_SKIPPED;
    out->median = __builtin_nan("");
  }
  // pass A's blocks added into kHistCopies copies of the first-digit counts: summed here
  static_assert(kBins1 % 1024 == 0, "blocks of 256, 512 or 1024 threads share the bins evenly");
  for (uint32_t b = threadIdx.x; b < (uint32_t)kBins1; b += 4 * blockDim.x) {
    uint64_t c[4][kHistCopies];  // every load issued before the first add
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int k = 0; k < kHistCopies; ++k) c[j][k] = hist1[(size_t)k * kBins1 + b + j * blockDim.x];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint64_t x = 0;
#pragma unroll
      for (int k = 0; k < kHistCopies; ++k) x += c[j][k];
      lds[b + j * blockDim.x] = x;
    }
  }
  __syncthreads();
  select_level(1, lds, st, dtype, volume, out, false, ssm);
  __syncthreads();
  if (threadIdx.x == 0) {
    // many bins: pass B counts the kWinBins bins around the median's first-digit
    // bucket in LDS (where noise-dominated cubes put nearly every value)
    int32_t w0 = 0;
    if (st->hist_ok && nbins > (int32_t)kWinBins) {
      double bm = ((double)(float)value_of_key(st->prefix, dtype) - (double)st->lo) * (double)st->scale;
      if (!(bm >= 0.0)) bm = 0.0;
      if (bm > (double)(nbins - 1)) bm = (double)(nbins - 1);
      w0 = (int32_t)bm - (int32_t)(kWinBins / 2);
      if (w0 > nbins - (int32_t)kWinBins) w0 = nbins - (int32_t)kWinBins;
      if (w0 < 0) w0 = 0;
    }
    st->win0 = w0;
  }
}

// Bound by HBM: 1024x1024x1280 voxels (5.4 GB) 0.86 ms, 6.2 TB/s, which a launch
// with only the loads takes too (two blocks per compute unit; with three, or
// with loads issued a chunk ahead, 0.89 to 0.91).
template <int DT, int VEC, bool NT>
__global__ __launch_bounds__(1024) void k_pass_a(Geom g, uint32_t rshift, Partial* __restrict__ parts,
                                                 uint64_t* __restrict__ hist1, uint64_t* __restrict__ hcopy,
                                                 uint32_t hcopy_n, SelState* __restrict__ st,
                                                 tsa_result* __restrict__ out, uint64_t volume, int32_t nbins,
                                                 Arrive* arrive) {
  extern __shared__ __align__(16) uint32_t lds[];
  __shared__ MomShared sm;
  __shared__ Partial sm_part;
  // pass B's histogram copies start at zero (cleared here, not by a launch of their own)
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < hcopy_n; i += gridDim.x * blockDim.x) hcopy[i] = 0ull;
  lds_zero(lds, ((uint32_t)kBins1 << rshift) + kTrash);
  __syncthreads();
  Pass1Acc<DT> a(lds, rshift);
  walk<DT, VEC, kUnrollOf<DT, VEC>, NT>(g, a);
  // every valid value incremented one first-digit counter: the block's count
  // is their total (each lane adds a strided share; the partial sums them)
  __syncthreads();
  uint32_t c = 0;
  for (uint32_t i = threadIdx.x; i < ((uint32_t)kBins1 << rshift); i += blockDim.x) c += lds[i];
  a.mom.cnt = c;
  block_store_partial(a.mom, sm, &sm_part);  // thread 0's
  if (threadIdx.x == 0) publish_partial(sm_part, parts + blockIdx.x);
  __syncthreads();
  lds_flush_digits<DT>(lds, rshift, hist1 + (size_t)(blockIdx.x % kHistCopies) * kBins1);
  if (last_block(arrive))
    mid_tail(parts, (int)gridDim.x, DT, volume, nbins, hist1, st, out, (uint64_t*)lds);
}

// Pass B's last block: M2 about the shift c, M2 = sum (x-c)^2 - n (mean - c)^2,
// the block partials added in a fixed order (strided per thread, then a
// pairwise tree; sq: 8 bytes a thread), and the second digit.
TSA_DEV void pass_b_tail(const Partial* parts2, SelState* st, const uint64_t* hist2, bool var_on, double* sq,
                         const Tail& tl) {
  __shared__ SelectShared ssm;
  if (!last_block(tl.arrive + 1)) return;
  if (var_on) {
    const int t = threadIdx.x, bs = blockDim.x;
    double q = 0.0;
    for (int i = t; i < (int)gridDim.x; i += bs) q += parts2[i].q;
    sq[t] = q;
    __syncthreads();
    for (int s2 = bs / 2; s2 > 0; s2 >>= 1) {
      if (t < s2) sq[t] += sq[t + s2];
      __syncthreads();
    }
    if (t == 0) {
      const double n = (double)tl.out->count;
      const double dm = tl.out->mean - (double)st->shift;
      double m2 = sq[0] - n * dm * dm;
      if (m2 < 0.0) m2 = 0.0;  // rounding below zero; NaN (infinite values) stays
      tl.out->m2 = m2;
      tl.out->std = sqrt(m2 / n);
    }
  }
  select_level(2, hist2, st, tl.dtype, tl.volume, tl.out, false, ssm);
}

template <int DT, int VEC, bool NT>
__global__ __launch_bounds__(1024) void k_pass_b(Geom g, int32_t nbins, uint32_t rshift, uint32_t stage,
                                                 SelState* __restrict__ st,
                                                 uint64_t* __restrict__ counts,
                                                 uint64_t* __restrict__ hist2, uint32_t* __restrict__ cand,
                                                 Partial* __restrict__ parts2, Tail tl) {
  // dynamic LDS: [nbins << rshift] histogram, [kBins2] level-2 digits, then the
  // candidate staging of the block's waves
  extern __shared__ __align__(16) uint32_t lds[];
  __shared__ MomShared sm;
  __shared__ Partial sm_part;
  const uint32_t hsize = ((uint32_t)nbins << rshift) + kTrash;
  uint32_t* l2 = lds + hsize;
  const bool hist_on = st->hist_ok != 0;
  const bool sel_on = st->done == 0;
  const bool var_on = DT == 0 && st->var_on != 0;
  if (!hist_on && !sel_on && !var_on) return;
  lds_zero(lds, hsize + kBins2);
  const CandSink<> sink = cand_sink_lds(l2 + kBins2, stage, cand, &st->ncand, st->cand_cap);
  __syncthreads();
  Pass2Acc<DT, HistOwnAcc> b{HistOwnAcc(lds, st->lo, st->scale, nbins, rshift),
                             Level2Acc<DT>(l2, st->prefix, sel_on, st->compact != 0, sink), VarAcc{st->shift},
                             hist_on, sel_on, var_on};
  walk<DT, VEC, kUnrollOf<DT, VEC>, NT>(g, b);
  b.l2.finish();
  __syncthreads();
  // into one of kHistCopies copies (counts holds them nbins apart), summed by k_level3
  if (hist_on)
    lds_flush(lds, (uint32_t)nbins, rshift, counts + (size_t)(blockIdx.x % kHistCopies) * (uint32_t)nbins);
  if (sel_on) lds_flush(l2, kBins2, 0, hist2);
  // values lie in their own [min, max]: the outlier counters keep their zeros
  if (var_on) {
    block_store_var(b.var, sm, &sm_part);  // thread 0's
    if (threadIdx.x == 0) publish_partial(sm_part, parts2 + blockIdx.x);
  }
  pass_b_tail(parts2, st, hist2, var_on, (double*)lds, tl);
}

// Pass B with a window of kWinBins 32-bit LDS counters (more bins than fit):
// one 1024-lane block per compute unit; values outside the window go straight
// to the global bins.
template <int DT, int VEC, bool NT>
__global__ __launch_bounds__(1024) void k_pass_bwin(Geom g, int32_t nbins, SelState* __restrict__ st,
                                                    uint64_t* __restrict__ counts, uint64_t* __restrict__ hist2,
                                                    uint32_t* __restrict__ cand, Partial* __restrict__ parts2,
                                                    Tail tl) {
  // dynamic LDS: [kWinBins] window counters, [kBins2] level-2 digits, candidate staging
  extern __shared__ __align__(16) uint32_t lds[];
  __shared__ MomShared sm;
  __shared__ Partial sm_part;
  uint32_t* l2 = lds + kWinBins;
  const bool hist_on = st->hist_ok != 0;
  const bool sel_on = st->done == 0;
  const bool var_on = DT == 0 && st->var_on != 0;
  if (!hist_on && !sel_on && !var_on) return;
  lds_zero(lds, kWinBins + kBins2);
  const CandSink<> sink = cand_sink_lds(l2 + kBins2, kWaveStage, cand, &st->ncand, st->cand_cap);
  __syncthreads();
  const int32_t w0 = st->win0;
  Pass2Acc<DT, HistWinAcc> b{HistWinAcc{lds, st->lo, st->scale, nbins - 1, w0, counts},
                             Level2Acc<DT>(l2, st->prefix, sel_on, st->compact != 0, sink), VarAcc{st->shift},
                             hist_on, sel_on, var_on};
  walk<DT, VEC, kUnrollOf<DT, VEC>, NT>(g, b);
  b.l2.finish();
  __syncthreads();
  if (hist_on) {
    const uint32_t nw = (uint32_t)min((int32_t)kWinBins, nbins - w0);
    for (uint32_t i = threadIdx.x; i < nw; i += blockDim.x) {
      const uint32_t c = lds[i];
      if (c) atomicAdd((unsigned long long*)(counts + w0 + i), (unsigned long long)c);
    }
  }
  if (sel_on) lds_flush(l2, kBins2, 0, hist2);
  if (var_on) {
    block_store_var(b.var, sm, &sm_part);  // thread 0's
    if (threadIdx.x == 0) publish_partial(sm_part, parts2 + blockIdx.x);
  }
  pass_b_tail(parts2, st, hist2, var_on, (double*)lds, tl);
}

// ---------------------------------------------------------------------------
// host side: argument checks, geometry, workspace layout, launches
// ---------------------------------------------------------------------------

static const Tuning& tuning() {
  static Tuning t = [] {
    Tuning x;
    if (const char* s = getenv("TSA_BLOCK")) x.block = atoi(s);
    if (const char* s = getenv("TSA_BPC")) x.bpc = atoi(s);
    if (const char* s = getenv("TSA_NT")) x.nt = atoi(s) != 0;
    if (const char* s = getenv("TSA_REP")) x.rep_shift = atoi(s);
    if (x.block != 256 && x.block != 512 && x.block != 1024) x.block = 512;
    if (x.bpc < 1 || x.bpc > 16) x.bpc = 0;
    if (x.rep_shift < 0 || x.rep_shift > 3) x.rep_shift = -1;
    return x;
  }();
  return t;
}

int device_info(DevInfo* out) {
  static DevInfo cache[64];
  static bool have[64] = {false};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return TSA_EDEVICE;
  if (!have[dev]) {
    hipDeviceProp_t p;
    if (hipGetDeviceProperties(&p, dev) != hipSuccess) return TSA_EDEVICE;
    if (strncmp(p.gcnArchName, "gfx950", 6) != 0) return TSA_ENOTSUP;
    cache[dev].cus = p.multiProcessorCount;
    cache[dev].lds_per_block = p.sharedMemPerBlock;
    have[dev] = true;
  }
  *out = cache[dev];
  return TSA_OK;
}

Magic make_magic(uint32_t d) {
  uint32_t l = 0;
  while ((1ull << l) < (uint64_t)d) ++l;
  Magic g;
  g.m = (uint32_t)((((1ull << 32) * ((1ull << l) - (uint64_t)d)) / (uint64_t)d) + 1ull);
  g.s1 = l ? 1u : 0u;
  g.s2 = l ? l - 1u : 0u;
  return g;
}

int check_cube(const tsa_cube* c) {
  if (!c || !c->data) return TSA_EINVAL;
  if (c->dtype != TSA_F32 && c->dtype != TSA_I16) return TSA_ENOTSUP;
  if (c->reserved != 0) return TSA_EINVAL;
  if (c->nx < 1 || c->ny < 1 || c->nz < 1) return TSA_EINVAL;
  if (c->nx > (1ll << 31) || c->ny > (1ll << 31) || c->nz > (1ll << 31)) return TSA_EINVAL;
  const double n = (double)c->nx * (double)c->ny * (double)c->nz;
  if (n > (double)(1ll << 46)) return TSA_EINVAL;
  return TSA_OK;
}

int region_box(const tsa_cube* c, const tsa_region* r, tsa_region* b) {
  if (!r) {
    b->x0 = b->y0 = b->z0 = 0;
    b->x1 = c->nx;
    b->y1 = c->ny;
    b->z1 = c->nz;
    return TSA_OK;
  }
  if (r->x0 < 0 || r->y0 < 0 || r->z0 < 0 || r->x1 > c->nx || r->y1 > c->ny || r->z1 > c->nz) return TSA_EINVAL;
  if (r->x0 >= r->x1 || r->y0 >= r->y1 || r->z0 >= r->z1) return TSA_EINVAL;
  *b = *r;
  return TSA_OK;
}

int row_mode(const tsa_cube* c) {
  const int64_t esz = c->dtype == TSA_F32 ? 4 : 2;
  if ((uintptr_t)c->data % esz) return 0;
  return (uintptr_t)c->data % 16 == 0 && c->nx % (16 / esz) == 0 ? 1 : 2;
}

// Rows of tiles of `units` vectors.
static void cut_rows(Geom* g, uint32_t units) {
  uint32_t rpt = units / g->vpr;
  if (rpt < 1) rpt = 1;
  while ((uint64_t)rpt * g->vpr > (1ull << 30) && rpt > 1) rpt >>= 1;
  g->rpt = rpt;
  g->ntiles = (g->nrows + rpt - 1) / rpt;
}

// Tiles of a box read at any element boundary, for blocks that take `step` vectors
// at a time, on `cus` compute units: of the whole steps up to kTileUnits, those that
// leave each the least to do, a tile costing a fifth of a step to begin.  A thousand tiles of
// whatever size ended in steps that were mostly empty, some blocks with one tile more
// than others: the histogram of a 249x195x193 int16 box 23.5 -> 20.1 us, the trio of
// 295x293x297 float32 voxels 83.6 -> 78.3.
static void cut_whole_steps(Geom* g, uint32_t step, int cus) {
  uint32_t best = step;
  uint64_t least = UINT64_MAX;
  for (uint32_t k = 1; k * step <= kTileUnits; ++k) {
    cut_rows(g, k * step);
    const uint64_t cost = ((uint64_t)g->ntiles + cus - 1) / cus * (5 * k + 1);
    if (cost < least) {
      least = cost;
      best = k * step;
    }
  }
  cut_rows(g, best);
}

// Build the walk geometry of box b for a device of `cus` compute units.
int make_geom(const tsa_cube* c, const tsa_region& b, int cus, Geom* g, int* vec, int64_t* volume) {
  const int64_t esz = c->dtype == TSA_F32 ? 4 : 2;
  const int64_t epv = 16 / esz;
  const int64_t lx = b.x1 - b.x0, ly = b.y1 - b.y0, lz = b.z1 - b.z0;
  *volume = lx * ly * lz;
  memset(g, 0, sizeof(*g));
  g->base = c->data;
  int64_t e0 = b.x0 + c->nx * (b.y0 + c->ny * b.z0);
  const bool contig = (lx == c->nx && (ly == c->ny || lz == 1)) || (ly == 1 && lz == 1);
  *vec = row_mode(c);
  if (contig) {
    g->mode = 0;
    if (*vec) {
      // vectors from the aligned address at or below the cube's; those that
      // begin before the run are not visited
      const int64_t mis = (int64_t)((uintptr_t)c->data % 16) / esz;
      g->base = (const char*)c->data - mis * esz;
      e0 += mis;
      *vec = 1;
    }
    const int64_t e1 = e0 + *volume;
    if (*vec) {
      int64_t v0 = (e0 + epv - 1) / epv, v1 = e1 / epv;
      if (v0 >= v1) {
        g->v0 = g->v1 = 0;
        g->h0 = e0;
        g->h1 = e1;
        g->t0 = g->t1 = 0;
      } else {
        g->v0 = v0;
        g->v1 = v1;
        g->h0 = e0;
        g->h1 = v0 * epv;
        g->t0 = v1 * epv;
        g->t1 = e1;
      }
    } else {
      g->v0 = e0;
      g->v1 = e1;
    }
    return TSA_OK;
  }
  g->mode = 1;
  if ((uint64_t)ly * (uint64_t)lz > 0xFFFFFFFFull) return TSA_EINVAL;
  g->nrows = (uint32_t)(ly * lz);
  g->ly = (uint32_t)ly;
  if (*vec == 1) {
    const int64_t c0 = b.x0 / epv, c1 = (b.x1 + epv - 1) / epv;
    g->v_origin = (b.x0 / epv) + (c->nx / epv) * (b.y0 + c->ny * b.z0);
    g->v_ystride = c->nx / epv;
    g->v_zstride = (c->nx / epv) * c->ny;
    g->vpr = (uint32_t)(c1 - c0);
    g->head_skip = (uint32_t)(b.x0 % epv);
    g->last_valid = (uint32_t)(b.x1 - (c1 - 1) * epv);
  } else {
    g->v_origin = e0;
    g->v_ystride = c->nx;
    g->v_zstride = c->nx * c->ny;
    if (*vec == 2) {
      g->vpr = (uint32_t)((lx + epv - 1) / epv);
      g->head_skip = lx < epv ? 0u : (uint32_t)(g->vpr * epv - lx);
      g->last_valid = (uint32_t)(lx < epv ? lx : epv);
    } else {
      g->vpr = (uint32_t)lx;
      g->head_skip = 0;
      g->last_valid = 1;
    }
  }
  if (*vec == 2)
    cut_whole_steps(g, kTileUnits / (uint32_t)epv, cus);  // 512 lanes of kUnrollOf vectors
  else
    cut_rows(g, kTileUnits);
  g->ly_m = make_magic(g->ly);
  g->vpr_m = make_magic(g->vpr);
  return TSA_OK;
}

// Blocks for a pass over geometry g.
static int pass_grid(const Geom& g, int vec, int block, int maxblocks) {
  int64_t want;
  if (g.mode == 0)
    want = vec ? (g.v1 - g.v0 + (int64_t)block * kUnroll - 1) / ((int64_t)block * kUnroll)
               : (g.v1 - g.v0 + block - 1) / block;
  else
    want = g.ntiles;
  if (want < 1) want = 1;
  if (want > maxblocks) want = maxblocks;
  return (int)want;
}

// Workspace layout of the single-region calls.
struct WsLayout {
  size_t partials, partials2, arrive, hist1, hist2, hist3, state, state2, result, outl, hcopy, cand, total;
  uint32_t cand_cap;
};

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

constexpr int kArrives = 6;  // launches of a call that end in one block's work, at most

// cand_limit: most candidate keys the layout may hold (the fixed scratch of
// tsa_stats_static); a median bucket above the capacity takes a third pass.
static WsLayout ws_layout(int64_t volume, int64_t cand_limit = INT64_MAX) {
  WsLayout L;
  size_t o = 0;
  L.partials = o;
  o = align256(o + sizeof(Partial) * kMaxBlocks);
  L.partials2 = o;
  o = align256(o + sizeof(Partial) * kMaxBlocks);
  L.arrive = o;
  o = align256(o + 2 * sizeof(Partial) * 256);  // room for Arrive[kArrives]
  static_assert(sizeof(Arrive) * kArrives <= 2 * sizeof(Partial) * 256, "arrival counters");
  L.hist1 = o;
  o = align256(o + 8 * (size_t)kBins1 * kHistCopies);
  L.hist2 = o;
  o = align256(o + 8 * kBins2);
  L.hist3 = o;
  o = align256(o + 8 * kBins3);
  L.state = o;
  o = align256(o + sizeof(SelState));
  L.state2 = o;
  o = align256(o + sizeof(SelState));
  L.result = o;
  o = align256(o + sizeof(tsa_result));
  L.outl = o;
  o = align256(o + 16);
  L.hcopy = o;
  o = align256(o + 8 * (size_t)kHistCopies * kCopyBinsMax);
  int64_t cap = volume / 64;
  if (cap < 65536) cap = 65536;
  if (cap > (1ll << 26)) cap = 1ll << 26;
  if (cap > volume) cap = volume;
  if (cap > cand_limit) cap = cand_limit;
  L.cand_cap = (uint32_t)cap;
  L.cand = o;
  o = align256(o + 4 * (size_t)cap);
  L.total = o;
  return L;
}

size_t single_ws_bytes(int64_t volume) { return ws_layout(volume).total; }

static int launch_ok() { return hipGetLastError() == hipSuccess ? TSA_OK : TSA_EDEVICE; }

// One launch for up to kMaxFills disjoint (words, value) ranges.
static void fill_set(std::initializer_list<FillRange> ranges, hipStream_t s, SelState* st = nullptr,
                     const SelState& init = SelState{}, SelState* st2 = nullptr,
                     const SelState& init2 = SelState{}) {
  FillSet f{};
  f.st[0] = st;
  f.init[0] = init;
  f.st[1] = st2;
  f.init[1] = init2;
  uint64_t most = 0;
  for (const FillRange& r : ranges) {
    if (r.n == 0) continue;
    f.r[f.count++] = r;  // callers pass at most kMaxFills
    if (r.n > most) most = r.n;
  }
  if (f.count == 0) return;
  int blocks = (int)((most + 255) / 256);
  if (blocks > 1024) blocks = 1024;
  TSA_TRACED("fill", s, hipLaunchKernelGGL(k_fill_set, dim3(blocks), dim3(256), 0, s, f));
}

// The expression with the kernel's template constants: the type, how rows are read, and
// whether loads are non-temporal (always for vectors at any element boundary).
#define TSA_DISPATCH_AS(D, V, N, ...) \
  {                                    \
    constexpr int DT = D, VEC = V;     \
    constexpr bool NT = N;             \
    __VA_ARGS__;                       \
  }
#define TSA_DISPATCH(DTV, VECV, NTV, ...)       \
  do {                                           \
    if ((DTV) == 0) {                            \
      if ((VECV) == 1 && (NTV))                  \
        TSA_DISPATCH_AS(0, 1, true, __VA_ARGS__)        \
      else if ((VECV) == 1)                      \
        TSA_DISPATCH_AS(0, 1, false, __VA_ARGS__)       \
      else if ((VECV) == 2)                      \
        TSA_DISPATCH_AS(0, 2, true, __VA_ARGS__)        \
      else                                       \
        TSA_DISPATCH_AS(0, 0, false, __VA_ARGS__)       \
    } else {                                     \
      if ((VECV) == 1 && (NTV))                  \
        TSA_DISPATCH_AS(1, 1, true, __VA_ARGS__)        \
      else if ((VECV) == 1)                      \
        TSA_DISPATCH_AS(1, 1, false, __VA_ARGS__)       \
      else if ((VECV) == 2)                      \
        TSA_DISPATCH_AS(1, 2, true, __VA_ARGS__)        \
      else                                       \
        TSA_DISPATCH_AS(1, 0, false, __VA_ARGS__)       \
    }                                            \
  } while (0)

// Common preparation of a single-region call.
struct Prep {
  DevInfo dev;
  tsa_region box;
  Geom g;
  int vec;
  int64_t volume;
  WsLayout L;
  char* ws;
  hipStream_t s;
  int block, grid, bpc;
};

// Blocks per compute unit of a call's passes: two, and of the trio and the moments three
// where rows are read one by one (two -> three: trio of a 1711x1711x246 box 595 + 673 ->
// 561 + 617 us, moments of a 995x997x244 box 204 -> 186; of whole cubes 1.73 -> 1.83 ms
// for the trio of 1024x1024x1280 float32 voxels, 169 -> 180 us for the moments of 640^3).
constexpr int kBpc = 2, kBpcRows = 3;

static int prepare(const tsa_cube* cube, const tsa_region* region, void* d_ws, size_t ws_bytes,
                   tsa_stream_t stream, Prep* P, int rows_bpc = kBpc, int64_t cand_limit = INT64_MAX) {
  int st = check_cube(cube);
  if (st) return st;
  if ((st = region_box(cube, region, &P->box))) return st;
  if ((st = device_info(&P->dev))) return st;
  if ((st = make_geom(cube, P->box, P->dev.cus, &P->g, &P->vec, &P->volume))) return st;
  P->L = ws_layout(P->volume, cand_limit);
  if (!d_ws || ws_bytes < P->L.total) return TSA_ENOMEM;
  P->ws = (char*)d_ws;
  P->s = (hipStream_t)stream;
  const Tuning& T = tuning();
  P->block = T.block;
  P->bpc = T.bpc ? T.bpc : P->g.mode == 1 ? rows_bpc : kBpc;
  int maxb = P->dev.cus * P->bpc;
  if (maxb > kMaxBlocks) maxb = kMaxBlocks;
  P->grid = pass_grid(P->g, P->vec, P->block, maxb);
  return TSA_OK;
}

// int16 regions large enough for it are answered from one count of their
// values; returns false when the call takes the passes by key digits.
static bool try_count16(const tsa_cube* cube, const Prep& P, const Count16Ask& ask, int* st) {
  if (cube->dtype != TSA_I16) return false;
  Geom g = P.g;
  const int blocks = count16_grid(P.volume, P.dev.cus);
  if (g.mode == 1 && P.vec == 2) cut_whole_steps(&g, kCount16Step, blocks);
  const int grid = pass_grid(g, P.vec, kCount16Step / kUnroll, blocks);
  const int mode = count16_mode(P.volume, grid, 4 * (size_t)P.L.cand_cap, ask);
  if (!mode) return false;
  *st = run_count16(g, P.vec, grid, mode, P.ws + P.L.hcopy, P.ws + P.L.partials, P.ws + P.L.cand, ask, P.s);
  return true;
}

static uint32_t rep_shift_for(int nbins, size_t lds_budget) {
  const Tuning& T = tuning();
  uint32_t r = 0;
  if (T.rep_shift >= 0)
    r = (uint32_t)T.rep_shift;
  else
    r = nbins <= 1024 ? 2u : nbins <= 4096 ? 1u : 0u;
  while (r > 0 && ((size_t)nbins << r) * 4 > lds_budget) --r;
  return r;
}

// The arrival counters of the call's launches from number `first` on.
static Arrive* arrive_of(const Prep& P, int first) { return (Arrive*)(P.ws + P.L.arrive) + first; }

// The selection state a call starts from: the lower median, or quantile q
// selected to `levels` digits.
static SelState first_state(const Prep& P) {
  SelState x{};
  x.cand_cap = P.L.cand_cap;
  return x;
}
static SelState first_state(const Prep& P, double q, int32_t levels) {
  SelState x = first_state(P);
  x.q = q;
  x.rank_mode = 1u;
  x.levels = (uint32_t)levels;
  return x;
}

// Zero the arrival counters and the level histograms, set the selection state, and clear the caller's
// output counters (d_counts: nbins u64, outl: 2 u64; null for none), all in
// one launch.
// (more: the words of a bracket's memory, from the histogram copies' place on.)
static void reset_select(const Prep& P, const SelState& init, uint64_t* d_counts = nullptr, int32_t nbins = 0,
                         uint64_t* outl = nullptr, size_t more = 0) {
  fill_set({FillRange{(uint32_t*)(P.ws + P.L.arrive), (uint64_t)(P.L.state - P.L.arrive) / 4, 0u, 0u},
            FillRange{(uint32_t*)d_counts, d_counts ? (uint64_t)nbins * 2 : 0u, 0u, 0u},
            FillRange{(uint32_t*)outl, outl ? 4u : 0u, 0u, 0u},
            FillRange{(uint32_t*)(P.ws + P.L.hcopy), more / 4, 0u, 0u}},
           P.s, (SelState*)(P.ws + P.L.state), init);
}

template <int DT, int VEC, bool NT>
static int launch_pass_bwin(const Prep& P, int block, int grid, size_t lds, int32_t nbins, SelState* stp,
                            uint64_t* d_counts, uint64_t* h2, uint32_t* cand, Partial* parts2, const Tail& tl) {
  if (hipFuncSetAttribute((const void*)k_pass_bwin<DT, VEC, NT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)lds) != hipSuccess)
    return TSA_EDEVICE;
  TSA_TRACED("pass_bwin", P.s,
             hipLaunchKernelGGL((k_pass_bwin<DT, VEC, NT>), dim3(grid), dim3(block), lds, P.s, P.g, nbins, stp,
                                d_counts, h2, cand, parts2, tl));
  return TSA_OK;
}

template <int DT, int VEC, bool NT>
static int launch_hist_win(const Prep& P, int grid, size_t lds, float lo, float hi, float scale, int32_t nbins,
                           const int32_t* w0p, uint64_t* d_counts, uint64_t* outl) {
  if (hipFuncSetAttribute((const void*)k_hist_win<DT, VEC, NT>, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)lds) != hipSuccess)
    return TSA_EDEVICE;
  TSA_TRACED("hist_win", P.s,
             hipLaunchKernelGGL((k_hist_win<DT, VEC, NT>), dim3(grid), dim3(1024), lds, P.s, P.g, lo, hi, scale,
                                nbins, w0p, d_counts, outl));
  return TSA_OK;
}

int run_moments(const tsa_cube* cube, const tsa_region* region, tsa_result* d_out, void* d_ws, size_t ws_bytes,
                tsa_stream_t stream) {
  if (!d_out) return TSA_EINVAL;
  Prep P;
  int st = prepare(cube, region, d_ws, ws_bytes, stream, &P, kBpcRows);
  if (st) return st;
  Partial* parts = (Partial*)(P.ws + P.L.partials);
  TSA_TRACED("moments", P.s,
    TSA_DISPATCH(cube->dtype, P.vec, tuning().nt,
                 if (DT == 1 || P.g.mode == 0)
                   hipLaunchKernelGGL((k_moments<DT, VEC, NT, false>), dim3(P.grid), dim3(P.block), 0, P.s, P.g, parts);
                 else
                   hipLaunchKernelGGL((k_moments<DT, VEC, NT, DT == 0>), dim3(P.grid), dim3(P.block), 0, P.s, P.g, parts)));
  TSA_TRACED("moments_merge", P.s,
             hipLaunchKernelGGL(k_moments_merge, dim3(1), dim3(1024), 0, P.s, parts, P.grid, cube->dtype,
                                (uint64_t)P.volume, d_out));
  return launch_ok();
}

int run_histogram(const tsa_cube* cube, const tsa_region* region, float lo, float hi, int32_t nbins,
                  uint64_t* d_counts, uint64_t* d_outliers, void* d_ws, size_t ws_bytes, tsa_stream_t stream) {
  if (!d_counts) return TSA_EINVAL;
  if (nbins < 1 || nbins > 65536) return TSA_EINVAL;
  if (!isfinite(lo) || !isfinite(hi) || lo > hi) return TSA_EINVAL;
  float scale = 0.0f;
  if (lo < hi) {
    volatile float width = hi - lo;
    if (!isfinite(width)) return TSA_EINVAL;
    volatile float sc = (float)nbins / width;
    if (!isfinite(sc) || sc == 0.0f) return TSA_EINVAL;
    scale = sc;
  }
  Prep P;
  int st = prepare(cube, region, d_ws, ws_bytes, stream, &P);
  if (st) return st;
  uint64_t* outl = d_outliers ? d_outliers : (uint64_t*)(P.ws + P.L.outl);
  const size_t budget = P.dev.lds_per_block < 65536 ? P.dev.lds_per_block : 65536;
  const uint32_t rs = rep_shift_for(nbins, budget);
  const size_t lds = (((size_t)nbins << rs) + kTrash) * 4;
  uint32_t* groups = (uint32_t*)(P.ws + P.L.hist1);  // of the window's placement
  fill_set({FillRange{(uint32_t*)d_counts, (uint64_t)nbins * 2, 0u, 0u}, FillRange{(uint32_t*)outl, 4u, 0u, 0u},
            FillRange{groups, lds <= budget ? 0u : (uint64_t)kPlaceGroups, 0u, 0u},
            FillRange{(uint32_t*)arrive_of(P, 0), lds <= budget ? 0u : sizeof(Arrive) / 4, 0u, 0u}},
           P.s);
  if (lds <= budget) {
    TSA_TRACED("hist", P.s,
    TSA_DISPATCH(cube->dtype, P.vec, tuning().nt,
                   hipLaunchKernelGGL((k_hist<DT, VEC, NT>), dim3(P.grid), dim3(P.block), lds, P.s, P.g, lo, hi, scale,
                                      nbins, rs, d_counts, outl)));
    return launch_ok();
  }
  // a window of 32-bit counters where a sample of the region puts most values,
  // one 1024-lane block per compute unit; else (not on gfx950) 16-bit counters in epochs
  const size_t lds_win = (size_t)kWinBins * 4;
  if (lds_win + 1024 <= P.dev.lds_per_block) {
    int32_t* w0p = (int32_t*)(P.ws + P.L.state + offsetof(SelState, win0));
    if (cube->dtype == TSA_F32)
      TSA_TRACED("hist_place", P.s,
                 hipLaunchKernelGGL(k_hist_place<0>, dim3(kPlaceBlocks), dim3(kPlaceThreads), 0, P.s, cube->data,
                                    cube->nx, cube->ny, P.box, lo, hi, scale, nbins, groups, arrive_of(P, 0), w0p));
    else
      TSA_TRACED("hist_place", P.s,
                 hipLaunchKernelGGL(k_hist_place<1>, dim3(kPlaceBlocks), dim3(kPlaceThreads), 0, P.s, cube->data,
                                    cube->nx, cube->ny, P.box, lo, hi, scale, nbins, groups, arrive_of(P, 0), w0p));
    int grid = P.dev.cus;
    if (grid > P.grid) grid = P.grid;
    int stw = TSA_OK;
    TSA_DISPATCH(cube->dtype, P.vec, tuning().nt,
                 stw = (launch_hist_win<DT, VEC, NT>(P, grid, lds_win, lo, hi, scale, nbins, w0p, d_counts, outl)));
    if (stw) return stw;
    return launch_ok();
  }
  return run_histogram_wide(cube, P.g, P.vec, P.grid, P.block, lo, hi, scale, nbins, d_counts, outl, P.s);
}

// Voxels to sample when the region's ranks are bracketed first (0: they are not).
static uint32_t bracket_of(const tsa_cube* cube, const Prep& P) {
  return cube->dtype == TSA_F32 ? bracket_samples(P.volume, P.L.cand_cap) : 0u;
}
// The bracket of the rank that st holds (of the deviations from *med, where given), its memory at `mem`.
static int launch_bracket_of(const tsa_cube* cube, const Prep& P, uint32_t ns, char* mem, SelState* st,
                             const SelState* med, const Tail& tl) {
  return run_bracket(cube, P.box, P.g, P.vec, tuning().nt, P.grid, P.block, mem, ns, (uint32_t*)(P.ws + P.L.cand),
                     P.L.cand_cap, P.ws + P.L.partials, st, med,
                     BracketAsk{tl.out, tl.qout, tl.volume, tl.write_counts}, P.s);
}

// The three passes of a selection over the region, each choosing its digit in
// its last block; they end at once when a bracket has found the value.
static int launch_selection(const tsa_cube* cube, const Prep& P, const Tail& tl) {
  SelState* stp = (SelState*)(P.ws + P.L.state);
  uint64_t* h1 = (uint64_t*)(P.ws + P.L.hist1);
  uint64_t* h2 = (uint64_t*)(P.ws + P.L.hist2);
  uint64_t* h3 = (uint64_t*)(P.ws + P.L.hist3);
  uint32_t* cand = (uint32_t*)(P.ws + P.L.cand);
  const uint32_t rs = rep_shift_for(kBins1, 32768);
  TSA_TRACED("level1", P.s,
    TSA_DISPATCH(cube->dtype, P.vec, tuning().nt,
                 hipLaunchKernelGGL((k_level1<DT, VEC, NT>), dim3(P.grid), dim3(P.block),
                                    (((size_t)kBins1 << rs) + kTrash) * 4, P.s, P.g, rs, stp, h1, tl)));
  TSA_TRACED("level2", P.s,
    TSA_DISPATCH(cube->dtype, P.vec, tuning().nt,
                 hipLaunchKernelGGL((k_level2<DT, VEC, NT>), dim3(P.grid), dim3(P.block), 0, P.s, P.g, stp, h2, cand,
                                    tl)));
  TSA_TRACED("level3", P.s,
    TSA_DISPATCH(cube->dtype, P.vec, tuning().nt,
                 hipLaunchKernelGGL((k_level3<DT, VEC, NT>), dim3(P.grid), dim3(P.block), 0, P.s, P.g, stp, h3,
                                    (const uint32_t*)cand, 1, tl, HistCopies{})));
  return launch_ok();
}

int run_median(const tsa_cube* cube, const tsa_region* region, tsa_result* d_out, void* d_ws, size_t ws_bytes,
               tsa_stream_t stream) {
  if (!d_out) return TSA_EINVAL;
  Prep P;
  int st = prepare(cube, region, d_ws, ws_bytes, stream, &P);
  if (st) return st;
  Count16Ask ask{};
  ask.out = d_out;
  ask.rank = 1;
  ask.write_counts = 1;
  if (try_count16(cube, P, ask, &st)) return st;
  const uint32_t ns = bracket_of(cube, P);
  const Tail tl{d_out, nullptr, (uint64_t)P.volume, arrive_of(P, 0), cube->dtype, 1};
  reset_select(P, first_state(P), nullptr, 0, nullptr, ns ? bracket_bytes() : 0);
  if (ns && (st = launch_bracket_of(cube, P, ns, P.ws + P.L.hcopy, (SelState*)(P.ws + P.L.state), nullptr, tl)))
    return st;
  return launch_selection(cube, P, tl);
}

// ---------------------------------------------------------------------------
// Whole-cube scans cut into z-slabs of at most chunk_voxels voxels: every
// pass over the data goes out as one launch per slab, so a device shared
// with other streams (the serving loop's region batches) can start their
// work between two launches of a long scan.  The same kernels accumulate
// their counters across the slabs, so the results are the same as one
// launch per pass gives.
// ---------------------------------------------------------------------------
struct Slab {
  Geom g;
  int vec;
  int grid;
};

static int slabs_of(const tsa_cube* cube, int64_t chunk_voxels, const Prep& P, std::vector<Slab>* out) {
  const int64_t plane = cube->nx * cube->ny;
  int64_t planes = chunk_voxels / plane;
  if (planes < 1) planes = 1;
  int maxb = P.dev.cus * P.bpc;
  if (maxb > kMaxBlocks) maxb = kMaxBlocks;
  for (int64_t z0 = 0; z0 < cube->nz; z0 += planes) {
    const tsa_region b{0, 0, z0, cube->nx, cube->ny, z0 + planes < cube->nz ? z0 + planes : cube->nz};
    Slab sl;
    int64_t vol = 0;
    const int st = make_geom(cube, b, P.dev.cus, &sl.g, &sl.vec, &vol);
    if (st) return st;
    sl.grid = pass_grid(sl.g, sl.vec, P.block, maxb);
    out->push_back(sl);
  }
  return TSA_OK;
}

int run_histogram_chunked(const tsa_cube* cube, float lo, float hi, int32_t nbins, uint64_t* d_counts,
                          uint64_t* d_outliers, void* d_ws, size_t ws_bytes, tsa_stream_t stream,
                          int64_t chunk_voxels) {
  if (!d_counts || chunk_voxels < 1) return TSA_EINVAL;
  if (nbins < 1 || nbins > 65536) return TSA_EINVAL;
  if (!isfinite(lo) || !isfinite(hi) || lo > hi) return TSA_EINVAL;
  float scale = 0.0f;
  if (lo < hi) {
    volatile float width = hi - lo;
    if (!isfinite(width)) return TSA_EINVAL;
    volatile float sc = (float)nbins / width;
    if (!isfinite(sc) || sc == 0.0f) return TSA_EINVAL;
    scale = sc;
  }
  Prep P;
  int st = prepare(cube, nullptr, d_ws, ws_bytes, stream, &P);
  if (st) return st;
  std::vector<Slab> slabs;
  if ((st = slabs_of(cube, chunk_voxels, P, &slabs))) return st;
  uint64_t* outl = d_outliers ? d_outliers : (uint64_t*)(P.ws + P.L.outl);
  fill_set({FillRange{(uint32_t*)d_counts, (uint64_t)nbins * 2, 0u, 0u}, FillRange{(uint32_t*)outl, 4u, 0u, 0u}},
           P.s);
  const size_t budget = P.dev.lds_per_block < 65536 ? P.dev.lds_per_block : 65536;
  const uint32_t rs = rep_shift_for(nbins, budget);
  const size_t lds = (((size_t)nbins << rs) + kTrash) * 4;
  for (const Slab& sl : slabs) {
    if (lds <= budget) {
      TSA_TRACED("hist", P.s,
        TSA_DISPATCH(cube->dtype, sl.vec, tuning().nt,
                     hipLaunchKernelGGL((k_hist<DT, VEC, NT>), dim3(sl.grid), dim3(P.block), lds, P.s, sl.g, lo, hi,
                                        scale, nbins, rs, d_counts, outl)));
    } else if ((st = run_histogram_wide(cube, sl.g, sl.vec, sl.grid, P.block, lo, hi, scale, nbins, d_counts, outl,
                                        P.s))) {
      return st;
    }
  }
  return launch_ok();
}

int run_median_chunked(const tsa_cube* cube, tsa_result* d_out, void* d_ws, size_t ws_bytes, tsa_stream_t stream,
                       int64_t chunk_voxels) {
  if (!d_out || chunk_voxels < 1) return TSA_EINVAL;
  Prep P;
  int st = prepare(cube, nullptr, d_ws, ws_bytes, stream, &P);
  if (st) return st;
  std::vector<Slab> slabs;
  if ((st = slabs_of(cube, chunk_voxels, P, &slabs))) return st;
  reset_select(P, first_state(P));
  const Tail tl{};  // a digit is chosen after its last slab
  SelState* stp = (SelState*)(P.ws + P.L.state);
  uint64_t* h1 = (uint64_t*)(P.ws + P.L.hist1);
  uint64_t* h2 = (uint64_t*)(P.ws + P.L.hist2);
  uint64_t* h3 = (uint64_t*)(P.ws + P.L.hist3);
  uint32_t* cand = (uint32_t*)(P.ws + P.L.cand);
  const uint32_t rs = rep_shift_for(kBins1, 32768);
  for (const Slab& sl : slabs)
    TSA_TRACED("level1", P.s,
      TSA_DISPATCH(cube->dtype, sl.vec, tuning().nt,
                   hipLaunchKernelGGL((k_level1<DT, VEC, NT>), dim3(sl.grid), dim3(P.block),
                                      (((size_t)kBins1 << rs) + kTrash) * 4, P.s, sl.g, rs, stp, h1, tl)));
  TSA_TRACED("select", P.s,
             hipLaunchKernelGGL(k_select, dim3(1), dim3(1024), 0, P.s, 1, (const uint64_t*)h1, stp, cube->dtype,
                                (uint64_t)P.volume, d_out, 1, (double*)nullptr));
  for (const Slab& sl : slabs)
    TSA_TRACED("level2", P.s,
      TSA_DISPATCH(cube->dtype, sl.vec, tuning().nt,
                   hipLaunchKernelGGL((k_level2<DT, VEC, NT>), dim3(sl.grid), dim3(P.block), 0, P.s, sl.g, stp, h2,
                                      cand, tl)));
  TSA_TRACED("select", P.s,
             hipLaunchKernelGGL(k_select, dim3(1), dim3(1024), 0, P.s, 2, (const uint64_t*)h2, stp, cube->dtype,
                                (uint64_t)P.volume, d_out, 1, (double*)nullptr));
  for (size_t i = 0; i < slabs.size(); ++i)
    TSA_TRACED("level3", P.s,
      TSA_DISPATCH(cube->dtype, slabs[i].vec, tuning().nt,
                   hipLaunchKernelGGL((k_level3<DT, VEC, NT>), dim3(slabs[i].grid), dim3(P.block), 0, P.s,
                                      slabs[i].g, stp, h3, (const uint32_t*)cand, i == 0 ? 1 : 0, tl,
                                      HistCopies{})));
  TSA_TRACED("select", P.s,
             hipLaunchKernelGGL(k_select, dim3(1), dim3(1024), 0, P.s, 3, (const uint64_t*)h3, stp, cube->dtype,
                                (uint64_t)P.volume, d_out, 1, (double*)nullptr));
  return launch_ok();
}

static int enqueue_stats(const tsa_cube* cube, const tsa_region* region, int32_t nbins, tsa_result* d_out,
                         uint64_t* d_counts, uint64_t* d_outliers, void* d_ws, size_t ws_bytes, tsa_stream_t stream,
                         int64_t cand_limit = INT64_MAX);

namespace {
struct StatsCall {
  const tsa_cube* cube;
  const tsa_region* region;
  int32_t nbins;
  tsa_result* d_out;
  uint64_t* d_counts;
  uint64_t* d_outliers;
  void* d_ws;
  size_t ws_bytes;
};
int enqueue_stats_call(void* ctx, hipStream_t s) {
  const StatsCall& c = *(const StatsCall*)ctx;
  return enqueue_stats(c.cube, c.region, c.nbins, c.d_out, c.d_counts, c.d_outliers, c.d_ws, c.ws_bytes, s);
}
}  // namespace

// The fused trio's launches go out as one replayed graph (keyed by every
// argument, the box's corners included), so the GPU does not wait on the host
// between its short kernels; traced calls launch directly.
int run_stats(const tsa_cube* cube, const tsa_region* region, int32_t nbins, tsa_result* d_out, uint64_t* d_counts,
              uint64_t* d_outliers, void* d_ws, size_t ws_bytes, tsa_stream_t stream) {
  // argument errors, tracing, and more bins than one LDS histogram holds (the
  // wide passes set kernel attributes at launch) take the direct launch
  int dev = 0;
  if (check_cube(cube) != TSA_OK || !d_out || !d_counts || nbins < 1 || nbins > 8192 || !d_ws ||
      !graphs_enabled() || trace_active() || hipGetDevice(&dev) != hipSuccess)
    return enqueue_stats(cube, region, nbins, d_out, d_counts, d_outliers, d_ws, ws_bytes, stream);
  GraphKey key;
  memset(&key, 0, sizeof(key));
  key.v[0] = 2;  // tsa_stats
  key.v[1] = (uintptr_t)cube->data;
  key.v[2] = (uintptr_t)cube->dtype;
  key.v[3] = (uintptr_t)cube->nx;
  key.v[4] = (uintptr_t)cube->ny;
  key.v[5] = (uintptr_t)cube->nz;
  key.v[6] = (uintptr_t)nbins;
  key.v[7] = (uintptr_t)d_out;
  key.v[8] = (uintptr_t)d_counts;
  key.v[9] = (uintptr_t)d_outliers;
  key.v[10] = (uintptr_t)d_ws;
  key.v[11] = (uintptr_t)ws_bytes;
  key.v[12] = (uintptr_t)dev;
  if (region) {
    key.v[13] = 1;
    key.v[14] = (uintptr_t)region->x0;
    key.v[15] = (uintptr_t)region->y0;
    key.v[16] = (uintptr_t)region->z0;
    key.v[17] = (uintptr_t)region->x1;
    key.v[18] = (uintptr_t)region->y1;
    key.v[19] = (uintptr_t)region->z1;
  }
  StatsCall c{cube, region, nbins, d_out, d_counts, d_outliers, d_ws, ws_bytes};
  return graph_run(key, (hipStream_t)stream, enqueue_stats_call, &c);
}

// ---------------------------------------------------------------------------
// tsa_stats_static: the fused trio on a fixed scratch array of the library's
// own, for callers that cannot allocate device memory.  The host never uses
// the array's name as an address: each device's copy is looked up once with
// hipGetSymbolAddress (with that device current) and that pointer is what
// the kernels get.  Every call on a device shares its copy; calls that
// overlap on one device race.  Each call clears what has to start at zero
// (selection state, level histograms, counts and outliers) with fill kernels.
// ---------------------------------------------------------------------------
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxScratchDevices = 64;
std::once_flag g_scratch_once[kMaxScratchDevices];
void* g_scratch_ptr[kMaxScratchDevices];
int g_scratch_status[kMaxScratchDevices];
}  // namespace

static int static_scratch(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxScratchDevices) return TSA_EDEVICE;
  std::call_once(g_scratch_once[dev], [dev] {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    g_scratch_ptr[dev] = e == hipSuccess ? p : nullptr;
    g_scratch_status[dev] = (e == hipSuccess && p) ? TSA_OK : TSA_EDEVICE;
  });
  *out = g_scratch_ptr[dev];
  return g_scratch_status[dev];
}

// Candidate keys the fixed scratch holds beside everything else of the call.
static int64_t static_cand_limit() {
  const size_t fixed = ws_layout(0, 0).total;
  return (int64_t)((kStaticScratchBytes - fixed) / 4) & ~(int64_t)63;
}

int run_stats_static(const tsa_cube* cube, const tsa_region* region, int32_t nbins, tsa_result* d_out,
                     uint64_t* d_counts, uint64_t* d_outliers, tsa_stream_t stream) {
  void* ws = nullptr;
  const int st = static_scratch(&ws);
  if (st) return st;
  // launched directly: a graph would be instantiated, and instantiation may allocate
  return enqueue_stats(cube, region, nbins, d_out, d_counts, d_outliers, ws, kStaticScratchBytes, stream,
                       static_cand_limit());
}

size_t stats_static_scratch_bytes() { return kStaticScratchBytes; }
int64_t stats_static_cand_keys() { return static_cand_limit(); }

// The trio's last launch: the third digit (over the candidates, rarely over the
// region again) and the sum of the histogram's copies.
static int launch_last_digit(const tsa_cube* cube, const Prep& P, const Tail& tl, const HistCopies& hc) {
  SelState* stp = (SelState*)(P.ws + P.L.state);
  uint64_t* h3 = (uint64_t*)(P.ws + P.L.hist3);
  const uint32_t* cand = (const uint32_t*)(P.ws + P.L.cand);
  TSA_TRACED("level3", P.s,
    TSA_DISPATCH(cube->dtype, P.vec, tuning().nt,
                 hipLaunchKernelGGL((k_level3<DT, VEC, NT>), dim3(P.grid), dim3(P.block), 0, P.s, P.g, stp, h3, cand,
                                    1, tl, hc)));
  return launch_ok();
}

static int enqueue_stats(const tsa_cube* cube, const tsa_region* region, int32_t nbins, tsa_result* d_out,
                         uint64_t* d_counts, uint64_t* d_outliers, void* d_ws, size_t ws_bytes, tsa_stream_t stream,
                         int64_t cand_limit) {
  if (!d_out || !d_counts) return TSA_EINVAL;
  if (nbins < 1 || nbins > 65536) return TSA_EINVAL;
  Prep P;
  int st = prepare(cube, region, d_ws, ws_bytes, stream, &P, kBpcRows, cand_limit);
  if (st) return st;
  const size_t budget = P.dev.lds_per_block < 65536 ? P.dev.lds_per_block : 65536;
  const size_t cand_small = (size_t)(P.block / kWave) * kWaveStage * 4;  // pass B's candidate staging
  const bool wide = ((size_t)nbins + kTrash + kBins2) * 4 + cand_small > budget;
  // more bins: one 1024-lane block per compute unit, a window of 32-bit counters
  const int win_block = 1024;
  const size_t lds_win = ((size_t)kWinBins + kBins2 + (win_block / kWave) * kWaveStage) * 4;
  if (wide && lds_win + sizeof(MomShared) + 1024 > P.dev.lds_per_block) return TSA_ENOTSUP;  // not on gfx950
  uint64_t* outl = d_outliers ? d_outliers : (uint64_t*)(P.ws + P.L.outl);
  Count16Ask ask{};
  ask.out = d_out;
  ask.counts = d_counts;
  ask.outl = outl;
  ask.nbins = nbins;
  ask.moments = 1;
  ask.rank = 1;
  if (try_count16(cube, P, ask, &st)) return st;
  reset_select(P, first_state(P), d_counts, nbins, outl);
  Partial* parts = (Partial*)(P.ws + P.L.partials);
  SelState* stp = (SelState*)(P.ws + P.L.state);
  uint64_t* h1 = (uint64_t*)(P.ws + P.L.hist1);
  uint64_t* h2 = (uint64_t*)(P.ws + P.L.hist2);
  uint32_t* cand = (uint32_t*)(P.ws + P.L.cand);
  uint64_t* hcopy = (uint64_t*)(P.ws + P.L.hcopy);
  if (!wide && nbins > (int32_t)kCopyBinsMax) return TSA_ENOTSUP;  // cannot happen: the LDS bounds nbins first
  const Tail tl{d_out, nullptr, (uint64_t)P.volume, arrive_of(P, 0), cube->dtype, 0};
  const uint32_t rs1 = rep_shift_for(kBins1, 32768);
  size_t lds_a = (((size_t)kBins1 << rs1) + kTrash) * 4;
  if (lds_a < 8 * (size_t)kBins1) lds_a = 8 * (size_t)kBins1;  // its last block's sums (32 bytes a thread fit too)
  TSA_TRACED("pass_a", P.s,
    TSA_DISPATCH(cube->dtype, P.vec, tuning().nt,
                 hipLaunchKernelGGL((k_pass_a<DT, VEC, NT>), dim3(P.grid), dim3(P.block), lds_a, P.s, P.g, rs1, parts,
                                    h1, hcopy, wide ? 0u : (uint32_t)kHistCopies * (uint32_t)nbins, stp, d_out,
                                    (uint64_t)P.volume, nbins, arrive_of(P, 0))));
  Partial* parts2 = (Partial*)(P.ws + P.L.partials2);
  if (!wide) {
    // replicas only as far as bpc blocks of pass B still share a compute unit
    // (its static LDS: candidate staging, moment reduction)
    const size_t per_block = P.dev.lds_per_block / (size_t)P.bpc;
    // (and within the 64 KB a launch takes without raising its LDS limit)
    const size_t cap_b = per_block < budget ? per_block : budget;
    auto fixed_of = [&](size_t cb) { return sizeof(MomShared) + cb + (kBins2 + kTrash) * 4 + 1024; };  // + slack
    // the deep candidate stage when one replica of every bin still fits beside it
    uint32_t stage = kWaveStageBig;
    size_t cand_b = (size_t)(P.block / kWave) * stage * 4;
    if (fixed_of(cand_b) + ((size_t)nbins + kTrash) * 4 > cap_b) {
      stage = kWaveStage;
      cand_b = cand_small;
    }
    const size_t fixed_b = fixed_of(cand_b);
    const size_t budget_b = cap_b > fixed_b ? cap_b - fixed_b : 0;
    uint32_t rsb = rep_shift_for(nbins, budget_b);
    const size_t ldsb = (((size_t)nbins << rsb) + kTrash + kBins2) * 4 + cand_b;
    TSA_TRACED("pass_b", P.s,
      TSA_DISPATCH(cube->dtype, P.vec, tuning().nt,
                   hipLaunchKernelGGL((k_pass_b<DT, VEC, NT>), dim3(P.grid), dim3(P.block), ldsb, P.s, P.g, nbins,
                                      rsb, stage, stp, hcopy, h2, cand, parts2, tl)));
  } else {
    const int grid = P.grid < P.dev.cus ? P.grid : P.dev.cus;
    int stw = TSA_OK;
    TSA_DISPATCH(cube->dtype, P.vec, tuning().nt,
                 stw = (launch_pass_bwin<DT, VEC, NT>(P, win_block, grid, lds_win, nbins, stp, d_counts, h2, cand,
                                                      parts2, tl)));
    if (stw) return stw;
  }
  return launch_last_digit(cube, P, tl, wide ? HistCopies{} : HistCopies{hcopy, d_counts, nbins});
}

int run_quantile(const tsa_cube* cube, const tsa_region* region, double q, int32_t digits, double* d_out,
                 void* d_ws, size_t ws_bytes, tsa_stream_t stream) {
  if (!d_out || !(q >= 0.0 && q <= 1.0) || digits < 1 || digits > 3) return TSA_EINVAL;
  Prep P;
  int st = prepare(cube, region, d_ws, ws_bytes, stream, &P);
  if (st) return st;
  Count16Ask ask{};
  ask.qout = d_out;
  ask.rank = 2;
  ask.q = q;
  ask.digits = digits;
  if (try_count16(cube, P, ask, &st)) return st;
  const uint32_t ns = digits == 3 ? bracket_of(cube, P) : 0u;
  reset_select(P, first_state(P, q, digits), nullptr, 0, nullptr, ns ? bracket_bytes() : 0);
  tsa_result* scratch = (tsa_result*)(P.ws + P.L.result);
  const Tail tl{scratch, d_out, (uint64_t)P.volume, arrive_of(P, 0), cube->dtype, 0};
  if (ns && (st = launch_bracket_of(cube, P, ns, P.ws + P.L.hcopy, (SelState*)(P.ws + P.L.state), nullptr, tl)))
    return st;
  return launch_selection(cube, P, tl);
}

int run_mad(const tsa_cube* cube, const tsa_region* region, double* d_out, void* d_ws, size_t ws_bytes,
            tsa_stream_t stream) {
  if (!d_out) return TSA_EINVAL;
  Prep P;
  int st = prepare(cube, region, d_ws, ws_bytes, stream, &P);
  if (st) return st;
  Count16Ask ask{};
  ask.qout = d_out;
  ask.rank = 1;
  ask.mad = 1;
  if (try_count16(cube, P, ask, &st)) return st;
  SelState* med = (SelState*)(P.ws + P.L.state);
  SelState* sb = (SelState*)(P.ws + P.L.state2);
  tsa_result* scratch = (tsa_result*)(P.ws + P.L.result);
  uint32_t* cand = (uint32_t*)(P.ws + P.L.cand);
  // the deviations' digit counts lie where the trio keeps its histogram copies
  uint64_t* m1 = (uint64_t*)(P.ws + P.L.hcopy);
  uint64_t* m2 = m1 + kBins1;
  uint64_t* m3 = m2 + kBins2;
  // and behind them the memory of the two brackets
  constexpr size_t kDigits = 8 * (size_t)(kBins1 + kBins2 + kBins3);
  const uint32_t ns = bracket_of(cube, P);
  char* mem = (char*)m1 + kDigits;
  const SelState init = first_state(P);
  fill_set({FillRange{(uint32_t*)(P.ws + P.L.arrive), (uint64_t)(P.L.state - P.L.arrive) / 4, 0u, 0u},
            FillRange{(uint32_t*)m1, (kDigits + (ns ? 2 * bracket_bytes() : 0)) / 4, 0u, 0u}},
           P.s, med, init, sb, init);
  // 1. the lower median m
  const Tail tlm{scratch, nullptr, (uint64_t)P.volume, arrive_of(P, 0), cube->dtype, 0};
  if (ns && (st = launch_bracket_of(cube, P, ns, mem, med, nullptr, tlm))) return st;
  st = launch_selection(cube, P, tlm);
  if (st) return st;
  // 2. the lower median of |x - m| (float keys whatever the cube's type)
  const Tail tl{scratch, nullptr, (uint64_t)P.volume, arrive_of(P, 3), 0, 0};
  if (ns && (st = launch_bracket_of(cube, P, ns, mem + bracket_bytes(), sb, med, tl))) return st;
  const uint32_t rs = rep_shift_for(kBins1, 32768);
  TSA_TRACED("mad_level1", P.s,
    TSA_DISPATCH(cube->dtype, P.vec, tuning().nt,
                 hipLaunchKernelGGL((k_mlevel1<DT, VEC, NT>), dim3(P.grid), dim3(P.block),
                                    (((size_t)kBins1 << rs) + kTrash) * 4, P.s, P.g, rs, (const SelState*)med, sb, m1,
                                    tl)));
  TSA_TRACED("mad_level2", P.s,
    TSA_DISPATCH(cube->dtype, P.vec, tuning().nt,
                 hipLaunchKernelGGL((k_mlevel2<DT, VEC, NT>), dim3(P.grid), dim3(P.block), 0, P.s, P.g,
                                    (const SelState*)med, sb, m2, cand, tl)));
  TSA_TRACED("mad_level3", P.s,
    TSA_DISPATCH(cube->dtype, P.vec, tuning().nt,
                 hipLaunchKernelGGL((k_mlevel3<DT, VEC, NT>), dim3(P.grid), dim3(P.block), 0, P.s, P.g,
                                    (const SelState*)med, sb, m3, (const uint32_t*)cand, tl, cube->dtype, d_out)));
  return launch_ok();
}

}  // namespace tsa
