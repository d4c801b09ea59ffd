// Per-element accumulators and block-level epilogues shared by the kernels.
#pragma once

#include <climits>
#include <type_traits>

#include "tsa_device.hpp"

namespace tsa {

// Accumulators take elements one at a time (operator(), masked by in_box and
// the NaN test) and, where they have it, whole 16-byte vectors (vec).  vec
// looks at its wave's values together first: where all are ordinary (no NaN,
// in range), as nearly all are, no lane mask, select or branch is spent on a
// single one; else the vector goes element by element.  The passes over the
// data are bound by vector instructions as much as by HBM (15 a voxel kept
// the SIMDs 70 % busy at 2 GHz), so vec is what sets their rate.

// ---- LDS words by byte address ------------------------------------------------
// The per-value increments add a shifted index to a base held in a register
// (one shift-and-add), and add a register holding 1: both values pass through
// an empty asm barrier so the compiler neither folds the base back into a
// constant it adds separately nor rebuilds the 1 before every increment.
typedef __attribute__((address_space(3))) uint32_t lds_word;
TSA_DEV uint32_t lds_byte_addr(uint32_t* p) { return (uint32_t)(uintptr_t)(lds_word*)p; }
TSA_DEV uint32_t in_register(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}
TSA_DEV void lds_add_at(uint32_t byte_addr, uint32_t v) {
  __hip_atomic_fetch_add((lds_word*)(uintptr_t)byte_addr, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The four values of a float32 vector.
struct Four {
  uint32_t u[4];
  float v[4];
  TSA_DEV explicit Four(const uint4& r)
      : u{r.x, r.y, r.z, r.w},
        v{__uint_as_float(r.x), __uint_as_float(r.y), __uint_as_float(r.z), __uint_as_float(r.w)} {}
  // whether some lane of the wave holds a NaN among its four (one compare tests two)
  TSA_DEV bool wave_has_nan() const {
    return __ballot(__builtin_isunordered(v[0], v[1]) || __builtin_isunordered(v[2], v[3])) != 0ull;
  }
};

// ---- validity and key of one element ---------------------------------------
template <int DT>
struct Elt;
template <>
struct Elt<0> {
  TSA_DEV static bool valid(float x, bool in) { return in && (x == x); }
  TSA_DEV static uint32_t key(float x) { return key_f32(__float_as_uint(x)); }
  TSA_DEV static float val(float x) { return x; }
};
template <>
struct Elt<1> {
  TSA_DEV static bool valid(int16_t, bool in) { return in; }
  TSA_DEV static uint32_t key(int16_t x) { return key_i16(x); }
  TSA_DEV static float val(int16_t x) { return (float)x; }
};

// ---- moments (Section 4.2): count, min/max keys, sum and sum of squares -------
// NaN and masked lanes add 0.  COUNT = false: the caller supplies the count (a
// pass that also builds the first-digit histogram of the valid values has it
// as the histogram's total).
template <int DT, bool COUNT = true>
struct MomAcc;

// totalOrder extremes of float32 bit patterns without forming keys: as signed
// integers the non-negative values keep their order (hi), as unsigned ones the
// negative values come above them, in reversed order (top, low).  One
// three-operand instruction takes two values.
struct RawRange {
  int32_t hi = INT_MIN;
  uint32_t top = 0u, low = 0xFFFFFFFFu;
  TSA_DEV void add(uint32_t u) {
    hi = max(hi, (int32_t)u);
    top = max(top, u);
    low = min(low, u);
  }
  TSA_DEV void add2(uint32_t a, uint32_t b) {
    hi = max(max((int32_t)a, (int32_t)b), hi);
    top = max(max(a, b), top);
    low = min(min(a, b), low);
  }
  // keys of the smallest and largest value (0xFFFFFFFF and 0 when none was added)
  TSA_DEV uint32_t kmin() const { return low > top ? 0xFFFFFFFFu : key_f32((top & 0x80000000u) ? top : low); }
  TSA_DEV uint32_t kmax() const { return low > top ? 0u : key_f32(hi >= 0 ? (uint32_t)hi : low); }
};

// float32: per-lane running sums in double.  Each value and its square are
// exact in double (a float32 square needs 48 significand bits and lies in
// [2^-298, 2^256]), so every step rounds once, with relative error 2^-53.
// gfx950 issues double adds and fused multiply-adds at the single-precision
// rate, which makes this both cheaper and more accurate than float pairs
// carrying their rounding errors (TwoSum and FMA splits).
template <bool COUNT>
struct MomAcc<0, COUNT> {
  double s = 0.0, q = 0.0;
  RawRange range;
  uint32_t cnt = 0u;
  TSA_DEV void sums(float x) {
    const double v = (double)x;
    s += v;
    q = __builtin_fma(v, v, q);
  }
  TSA_DEV void operator()(float x, bool in) {
    if (Elt<0>::valid(x, in)) {
      sums(x);
      range.add(__float_as_uint(x));
      if constexpr (COUNT) ++cnt;
    }
  }
  // None of them NaN.  Four values are summed before they meet the running
  // sums: a quarter of the roundings at the sums' size (1024x1024x1280 voxels,
  // two blocks per compute unit: error of the mean and M2 2.5e-15 -> 0.4e-15, with
  // three blocks one by one 1.5e-15; time 1.73 -> 1.735 ms).
  TSA_DEV void four(const Four& f) {
    const double v[4] = {(double)f.v[0], (double)f.v[1], (double)f.v[2], (double)f.v[3]};
    s += (v[0] + v[1]) + (v[2] + v[3]);
    q += __builtin_fma(v[1], v[1], v[0] * v[0]) + __builtin_fma(v[3], v[3], v[2] * v[2]);
    range.add2(f.u[0], f.u[1]);
    range.add2(f.u[2], f.u[3]);
    if constexpr (COUNT) cnt += 4u;
  }
  TSA_DEV uint32_t kmin() const { return range.kmin(); }
  TSA_DEV uint32_t kmax() const { return range.kmax(); }
  TSA_DEV void chunk() {}
};

// int16: exact integer sums (|x| <= 32768, x^2 <= 2^30).
template <bool COUNT>
struct MomAcc<1, COUNT> {
  int64_t s = 0;
  uint64_t q = 0;
  uint32_t mn = 0xFFFFFFFFu, mx = 0u, cnt = 0u;
  TSA_DEV void operator()(int16_t x, bool in) {
    const int32_t v = in ? (int32_t)x : 0;
    s += v;
    q += (uint32_t)(v * v);
    const uint32_t k = key_i16(x);
    mn = min(mn, in ? k : 0xFFFFFFFFu);
    mx = max(mx, in ? k : 0u);
    if constexpr (COUNT) cnt += in ? 1u : 0u;
  }
  TSA_DEV uint32_t kmin() const { return mn; }
  TSA_DEV uint32_t kmax() const { return mx; }
  TSA_DEV void chunk() {}
};

// Chan et al.'s pairwise update of (n, mean, M2) (the O(1) combine of
// Section 4.2's partial sums).  A partial whose mean is infinite (it holds
// infinities) makes the merged mean the sum of the two means (+inf, -inf, or
// NaN when both signs occur) and the spread undefined (NaN).
TSA_DEV void chan_merge(double& na, double& ma, double& qa, double nb, double mb, double qb) {
  if (nb == 0.0) return;
  if (na == 0.0) {
    na = nb;
    ma = mb;
    qa = qb;
    return;
  }
  const double n = na + nb;
  if (!__builtin_isfinite(ma) || !__builtin_isfinite(mb)) {
    ma = ma + mb;
    qa = __builtin_nan("");
    na = n;
    return;
  }
  const double d = mb - ma, f = nb / n;  // one division: a merge tree is a chain of them
  ma = ma + d * f;
  qa = qa + qb + d * d * (na * f);
  na = n;
}

// (n, mean, M2) of one block partial, in double.  centered: the partial holds
// M2 and its mean about p.ref (tsa_moments' shifted lanes), returned here as
// the mean about ref0; else float32 partials hold the sums S and Q, int16
// partials exact integer sums.
TSA_DEV void partial_stats(const Partial& p, int dtype, double& n, double& m, double& q, bool centered = false,
                           double ref0 = 0.0) {
  n = (double)p.n;
  if (p.n == 0) {
    m = q = 0.0;
    return;
  }
  if (dtype == 0) {
    if (centered) {
      m = p.s + (p.ref - ref0);  // ref - ref0: two float32 values, exact in double
      q = p.q;
    } else {
      m = p.s / n;
      q = p.q - p.s * m;
    }
  } else {
    // exact n*Q - S^2 in 128-bit integers, then one rounding to double
    const __int128 num = (__int128)p.qi * (__int128)p.n - (__int128)p.si * (__int128)p.si;
    const int64_t hi = (int64_t)(num >> 64);
    const uint64_t lo = (uint64_t)num;
    m = (double)p.si / n;
    q = ((double)hi * 18446744073709551616.0 + (double)lo) / n;
  }
}

// float32, one pass, for the moments alone: every lane subtracts a shift c,
// its first finite valid value, before summing, and keeps sum (x - c) and
// sum (x - c)^2 in double.  x - c is exact in double (or within 2^-53 when
// the exponents lie more than 29 apart), so the lane's
// M2 = sum (x-c)^2 - (sum (x-c))^2 / n loses only the digits that
// (mean - c)^2 / var costs, where c is one of the lane's own values, instead
// of the (mean / std)^2 that unshifted sums of x and x^2 lose.  Infinities
// seen before the first finite value add +-inf either way (c stays 0 until
// then), so the shift is the same for every finite value of the lane.
struct ShiftMomAcc {
  double c = 0.0, s = 0.0, q = 0.0;
  RawRange range;
  uint32_t cnt = 0u;
  bool have = false;
  TSA_DEV void sums(float x) {
    const double d = (double)x - c;
    s += d;
    q = __builtin_fma(d, d, q);
  }
  TSA_DEV void operator()(float x, bool in) {
    if (Elt<0>::valid(x, in)) {
      if (!have && __builtin_isfinite(x)) {
        c = (double)x;
        have = true;
      }
      sums(x);
      range.add(__float_as_uint(x));
      ++cnt;
    }
  }
  TSA_DEV uint32_t kmin() const { return range.kmin(); }
  TSA_DEV uint32_t kmax() const { return range.kmax(); }
  TSA_DEV void chunk() {}
};
// ... a vector at a time, its four values summed before they meet the running sums:
// for whole cubes (1024x1024x1024 voxels 680 -> 628 us, error of the mean and M2 3.8e-15
// -> 0.5e-15).  A NaN costs no branch: one in a vector of every sixth wave took 725 us.
// Boxes take the elements: their walk keeps so many registers that with these
// only two blocks share a compute unit (634x634x634 box: 182 -> 229 us).
struct ShiftMomVecAcc : ShiftMomAcc {
  TSA_DEV void vec(const uint4& r) {
    const Four f(r);
    if (__ballot(!have) == 0ull) {
      const float shift = (float)c;  // NaN: as the shift, a value that the lane holds
      float x[4];
      double d[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool ok = f.v[e] == f.v[e];
        x[e] = ok ? f.v[e] : shift;
        cnt += ok ? 1u : 0u;
        d[e] = (double)x[e] - c;
      }
      s += (d[0] + d[1]) + (d[2] + d[3]);
      q += __builtin_fma(d[1], d[1], d[0] * d[0]) + __builtin_fma(d[3], d[3], d[2] * d[2]);
      range.add2(__float_as_uint(x[0]), __float_as_uint(x[1]));
      range.add2(__float_as_uint(x[2]), __float_as_uint(x[3]));
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) (*this)(f.v[e], true);
    }
  }
};

// Stores a partial where another block of the same launch may read it
// (agent-scope atomic stores; see last_block).
TSA_DEV void publish_partial(const Partial& p, Partial* out) {
  const uint64_t* src = (const uint64_t*)&p;
#pragma unroll
  for (uint32_t i = 0; i < sizeof(Partial) / 8; ++i)
    __hip_atomic_store((uint64_t*)out + i, src[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Reduce a block's lanes (fixed order) and store one Partial.
struct alignas(16) MomShared {
  double s[16], q[16], ref[16];
  int64_t si[16];
  uint64_t qi[16];
  uint32_t kmin[16], kmax[16];
  uint64_t cnt[16];
};

template <bool COUNT>
TSA_DEV void block_store_partial(MomAcc<0, COUNT>& a, MomShared& sm, Partial* out) {
  const double s = wave_sum_f64(a.s), q = wave_sum_f64(a.q);
  const uint32_t kmin = wave_min_u32(a.kmin()), kmax = wave_max_u32(a.kmax());
  const uint64_t cnt = wave_sum_u64(a.cnt);
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  if (lane == 0) {
    sm.s[w] = s;
    sm.q[w] = q;
    sm.kmin[w] = kmin;
    sm.kmax[w] = kmax;
    sm.cnt[w] = cnt;
  }
  __syncthreads();
  if (w == 0) {  // the waves' sums by the first wave (a lane each, all read at once)
    const bool on = lane < (int)(blockDim.x / kWave);
    const int i = on ? lane : 0;
    Partial p;
    p.n = wave_sum_u64(on ? sm.cnt[i] : 0ull);
    p.kmin = wave_min_u32(sm.kmin[i]);
    p.kmax = wave_max_u32(sm.kmax[i]);
    p.s = wave_sum_f64(on ? sm.s[i] : 0.0);
    p.q = wave_sum_f64(on ? sm.q[i] : 0.0);
    p.si = 0;
    p.qi = 0;
    if (lane == 0) *out = p;
  }
}

template <bool COUNT>
TSA_DEV void block_store_partial(MomAcc<1, COUNT>& a, MomShared& sm, Partial* out) {
  const int64_t s = wave_sum_i64(a.s);
  const uint64_t q = wave_sum_u64(a.q);
  const uint32_t kmin = wave_min_u32(a.kmin()), kmax = wave_max_u32(a.kmax());
  const uint64_t cnt = wave_sum_u64(a.cnt);
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  if (lane == 0) {
    sm.si[w] = s;
    sm.qi[w] = q;
    sm.kmin[w] = kmin;
    sm.kmax[w] = kmax;
    sm.cnt[w] = cnt;
  }
  __syncthreads();
  if (w == 0) {
    const bool on = lane < (int)(blockDim.x / kWave);
    const int i = on ? lane : 0;
    Partial p;
    p.n = wave_sum_u64(on ? sm.cnt[i] : 0ull);
    p.kmin = wave_min_u32(sm.kmin[i]);
    p.kmax = wave_max_u32(sm.kmax[i]);
    p.si = wave_sum_i64(on ? sm.si[i] : 0ll);
    p.qi = wave_sum_u64(on ? sm.qi[i] : 0ull);
    p.s = p.q = 0.0;
    if (lane == 0) *out = p;
  }
}

// Lanes of ShiftMomAcc: each lane's (n, mean, M2), then Chan merges down a
// fixed tree (lane i takes lane i + o, o = 32 .. 1), the block's waves in
// order.  Means are carried about one reference value, the shift of the
// wave's (then the block's) first lane that has one, so the differences of
// means the merge forms are exact to the spread's scale, not the mean's:
// with mean/std = 1e7 a mean rounded to its own ulp would already cost 1e-9
// of the spread.  The Partial holds (n, mean about ref, M2, ref) ("centered")
// and the key extremes.
TSA_DEV void block_store_centered(ShiftMomAcc& a, MomShared& sm, Partial* out) {
  const uint64_t have = __ballot(a.have);
  const double ref_w = have ? __shfl(a.c, __builtin_ctzll(have)) : 0.0;
  double n = (double)a.cnt, m = 0.0, m2 = 0.0;
  if (a.cnt) {
    const double r = a.s / n;
    m = (a.c - ref_w) + r;  // a.c - ref_w: two float32 values (or 0), exact in double
    m2 = a.q - a.s * r;
    if (m2 < 0.0) m2 = 0.0;  // rounding below zero; NaN (infinite values) stays
  }
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    const double nb = __shfl_down(n, o), mb = __shfl_down(m, o), qb = __shfl_down(m2, o);
    if (lane < o) chan_merge(n, m, m2, nb, mb, qb);
  }
  const uint32_t kmin = wave_min_u32(a.kmin()), kmax = wave_max_u32(a.kmax());
  if (lane == 0) {
    sm.s[w] = m;
    sm.q[w] = m2;
    sm.ref[w] = have ? ref_w : __builtin_nan("");  // NaN: no finite value in the wave
    sm.cnt[w] = (uint64_t)n;
    sm.kmin[w] = kmin;
    sm.kmax[w] = kmax;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const int nw = blockDim.x / kWave;
    double ref = 0.0;
    for (int i = nw - 1; i >= 0; --i)
      if (sm.ref[i] == sm.ref[i]) ref = sm.ref[i];
    double bn = 0.0, bm = 0.0, bq = 0.0;
    uint32_t mn = 0xFFFFFFFFu, mx = 0u;
    for (int i = 0; i < nw; ++i) {
      // a wave without a finite value has a non-finite mean whatever its shift
      const double sh = sm.ref[i] == sm.ref[i] ? sm.ref[i] - ref : 0.0;
      chan_merge(bn, bm, bq, (double)sm.cnt[i], sm.s[i] + sh, sm.q[i]);
      mn = min(mn, sm.kmin[i]);
      mx = max(mx, sm.kmax[i]);
    }
    Partial p;
    p.n = (uint64_t)bn;
    p.kmin = mn;
    p.kmax = mx;
    p.s = bm;
    p.q = bq;
    p.ref = ref;
    p.qi = 0;
    *out = p;
  }
}

// ---- second moment about a shift (two-pass form, fused path) ----------------
// sum (x - c)^2 in double: the difference of two float32 values is formed in
// double (exact unless their exponents lie more than 29 apart, then within
// 2^-53), so the squares carry no cancellation however large the mean is
// against the spread, and they stay inside [2^-298, 2^258].
struct VarAcc {
  float c;
  double q = 0.0;
  TSA_DEV void operator()(float x, bool in) {
    const bool ok = in && (x == x);
    const double d = (double)(ok ? x : c) - (double)c;  // masked lanes: d = 0
    q = __builtin_fma(d, d, q);
  }
  TSA_DEV void four(const Four& f) {  // none of them NaN
    double d[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) d[e] = (double)f.v[e] - (double)c;
    q += __builtin_fma(d[1], d[1], d[0] * d[0]) + __builtin_fma(d[3], d[3], d[2] * d[2]);
  }
  TSA_DEV void chunk() {}
};

TSA_DEV void block_store_var(VarAcc& a, MomShared& sm, Partial* out) {
  const double q = wave_sum_f64(a.q);
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  if (lane == 0) sm.q[w] = q;
  __syncthreads();
  if (w == 0) {
    const bool on = lane < (int)(blockDim.x / kWave);
    Partial p;
    p.n = 0;
    p.kmin = p.kmax = 0;
    p.s = 0.0;
    p.q = wave_sum_f64(on ? sm.q[on ? lane : 0] : 0.0);
    p.si = 0;
    p.qi = 0;
    if (lane == 0) *out = p;
  }
}

// ---- |x - m| as the element (median absolute deviation) ----------------------
// Feeds an accumulator written for float elements with d = |x - m|: one IEEE
// single-precision subtraction for float32 cubes, exact for int16 cubes (the
// integer difference is at most 65535, exact in float).  A value equal to m
// deviates by +0, also when both are the same infinity (where the IEEE
// difference would be NaN), so every non-NaN voxel has a deviation.  NaN
// stays NaN.
template <int DT, class Inner>
struct AbsDev {
  Inner inner;
  float mf;
  int32_t mi;
  template <class T>
  TSA_DEV void operator()(T raw, bool in) {
    float d;
    if constexpr (DT == 0)
      d = ((float)raw == mf) ? 0.0f : fabsf((float)raw - mf);
    else
      d = (float)abs((int32_t)raw - mi);
    inner(d, in);
  }
  TSA_DEV void chunk() { inner.chunk(); }
};

// ---- LDS-privatised counters -------------------------------------------------
// Every LDS counter array is followed by kTrash spare words (one per lane of a
// wave) that branch-free increments of invalid lanes may hit; they are never read.
constexpr uint32_t kTrash = 64;

// Bin b, replica r lives at lds[(b << rshift) + r]; a lane uses replica
// (lane & (R-1)) so lanes of one wave that hit the same bin mostly touch
// different words.
TSA_DEV void lds_inc(uint32_t* lds, uint32_t idx) {
  __hip_atomic_fetch_add(lds + idx, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Increment for the lanes where m holds, rare across the wave: the wave skips
// the LDS instruction entirely when no lane needs it (an exec-masked LDS
// instruction with no active lane still takes an issue slot).
TSA_DEV void lds_inc_rare(uint32_t* lds, bool m, uint32_t idx) {
  if (__ballot(m) != 0ull) {
    if (m) lds_inc(lds, idx);
  }
}

TSA_DEV void lds_zero(uint32_t* lds, uint32_t n) {
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) lds[i] = 0u;
}

// Sum the replicas of each bin and add the non-zero ones to global counters.
TSA_DEV void lds_flush(const uint32_t* lds, uint32_t nbins, uint32_t rshift, uint64_t* g) {
  const uint32_t R = 1u << rshift;
  for (uint32_t b = threadIdx.x; b < nbins; b += blockDim.x) {
    uint32_t c = 0;
    for (uint32_t r = 0; r < R; ++r) c += lds[(b << rshift) + r];
    if (c) atomicAdd((unsigned long long*)(g + b), (unsigned long long)c);
  }
}

// Whether a histogram over the values' own extremes exists, and its scale (lo == hi,
// which both zeros are too: 0, every value in bin 0).  An infinite extreme or width
// makes the quotient 0 or NaN.
TSA_DEV bool own_range(float lo, float hi, int32_t nbins, float& scale) {
  const float s = (float)nbins / (hi - lo);
  const bool ok = __builtin_isfinite(s) && s != 0.0f;
  scale = ok ? s : 0.0f;
  return ok || (lo == hi && __builtin_isfinite(lo));
}

// ---- histogram (Section 4.1) ---------------------------------------------------
// LDS: (nbins << rshift) + kTrash words.  The vectors take the formula's minimum
// value by value: it costs no time (1024x1024x1280 voxels with it 1723 us, without
// 1726), and counting t == nbins past the last bin instead lengthens every flush
// (10000 bins of 8^3 voxels 7.8 -> 9.1 us) and puts the extremes of two-valued data
// into one LDS bank (640^3 voxels, 4096 bins: 1670 -> 1820 us).
template <int DT>
struct HistAcc {
  uint32_t* lds;
  float lo, hi, scale;
  int32_t nbm1;
  uint32_t rshift, rep;
  uint32_t base, one;  // byte address of bin 0's replica of the lane, a 1
  uint32_t below = 0, above = 0;
  TSA_DEV HistAcc(uint32_t* l, float lo_, float hi_, float scale_, int32_t nbins, uint32_t rshift_)
      : lds(l), lo(lo_), hi(hi_), scale(scale_), nbm1(nbins - 1), rshift(rshift_),
        rep(threadIdx.x & ((1u << rshift_) - 1u)), base(in_register(lds_byte_addr(l) + 4u * rep)),
        one(in_register(1u)) {}
  TSA_DEV void vec(const uint4& r) { some(r, 0xFFu); }
  template <int D = DT, class = std::enable_if_t<D == 1>>
  TSA_DEV void masked(const uint4& r, uint32_t mask) {
    some(r, mask);
  }
  TSA_DEV void some(const uint4& r, uint32_t mask) {  // mask: int16 only
    constexpr int N = Ty<DT>::EPV;
    float v[N];
    bool in = DT == 0 || mask == 0xFFu;
#pragma unroll
    for (int e = 0; e < N; ++e) {
      v[e] = (float)Ty<DT>::get(r, e);
      in = in && v[e] >= lo && v[e] <= hi;  // NaN fails both tests
    }
    if (__ballot(!in) == 0ull) {
#pragma unroll
      for (int e = 0; e < N; ++e)
        lds_add_at(((uint32_t)min((int32_t)((v[e] - lo) * scale), nbm1) << (rshift + 2u)) + base, one);
    } else {
#pragma unroll
      for (int e = 0; e < N; ++e) (*this)(v[e], DT == 0 || ((mask >> e) & 1u) != 0u);
    }
  }
  template <class T>
  TSA_DEV void operator()(T raw, bool in) {
    const float v = (float)raw;  // exact for int16
    below += (in && v < lo) ? 1u : 0u;
    above += (in && v > hi) ? 1u : 0u;
    if (in && v >= lo && v <= hi) {  // NaN fails both tests
      const float d = v - lo;
      const float t = d * scale;  // lo == hi: scale == 0 and t == 0
      const int32_t b = min(max((int32_t)t, 0), nbm1);
      lds_inc(lds, ((uint32_t)b << rshift) + rep);
    }
  }
  TSA_DEV void chunk() {}
};

// Histogram over the values' own [min, max] (lo and hi are the extremes of the
// same values, both finite): every valid value is in range, so only NaN needs a
// test, (v - lo) * scale is never negative, and there are no outliers.  Gives
// the same bins as HistAcc for such a range.
struct HistOwnAcc {
  uint32_t* lds;
  float lo, scale;
  int32_t nbm1;
  uint32_t rshift, rep;
  uint32_t base, one;  // byte address of bin 0's replica of the lane, a 1
  TSA_DEV HistOwnAcc(uint32_t* l, float lo_, float scale_, int32_t nbins, uint32_t rshift_)
      : lds(l), lo(lo_), scale(scale_), nbm1(nbins - 1), rshift(rshift_), rep(threadIdx.x & ((1u << rshift_) - 1u)),
        base(in_register(lds_byte_addr(l) + 4u * rep)), one(in_register(1u)) {}
  template <class T>
  TSA_DEV void operator()(T raw, bool in) {
    const float v = (float)raw;  // exact for int16
    if (in && v == v) {
      const float t = (v - lo) * scale;  // lo == hi: scale == 0 and t == 0
      const int32_t b = min((int32_t)t, nbm1);
      lds_inc(lds, ((uint32_t)b << rshift) + rep);
    }
  }
  TSA_DEV void four(const Four& f) {  // none of them NaN
#pragma unroll
    for (int e = 0; e < 4; ++e)
      lds_add_at(((uint32_t)min((int32_t)((f.v[e] - lo) * scale), nbm1) << (rshift + 2u)) + base, one);
  }
  TSA_DEV void chunk() {}
};

// Histogram over the values' own [min, max] with more bins than LDS holds as
// 32-bit counters: a window of kWinBins bins [w0, w0 + kWinBins) is counted in
// LDS, bins outside it directly in the global counters (exact for any data;
// fast when the window holds most values).  Same bins as HistOwnAcc.
constexpr uint32_t kWinBins = 32768;
struct HistWinAcc {
  uint32_t* lds;
  float lo, scale;
  int32_t nbm1, w0;
  uint64_t* counts;
  template <class T>
  TSA_DEV void operator()(T raw, bool in) {
    const float v = (float)raw;  // exact for int16
    if (in && v == v) {
      const float t = (v - lo) * scale;
      const int32_t b = min((int32_t)t, nbm1);
      const uint32_t rel = (uint32_t)(b - w0);
      if (rel < kWinBins)
        lds_inc(lds, rel);
      else
        atomicAdd((unsigned long long*)(counts + b), 1ull);
    }
  }
  TSA_DEV void four(const Four& f) {  // none of them NaN
    int32_t b[4];
    uint32_t far = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      b[e] = min((int32_t)((f.v[e] - lo) * scale), nbm1);
      far = max(far, (uint32_t)(b[e] - w0));
    }
    if (__ballot(far >= kWinBins) == 0ull) {
#pragma unroll
      for (int e = 0; e < 4; ++e) lds_inc(lds, (uint32_t)(b[e] - w0));
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) (*this)(f.v[e], true);
    }
  }
  TSA_DEV void chunk() {}
};

// HistWinAcc for a caller's range [lo, hi]: values below lo and above hi are
// counted apart (as HistAcc counts them), in-range values in the window
// [w0, w0 + kWinBins) go to the LDS counters, the other in-range values to
// the global bins.
template <int DT>
struct HistWinOutAcc {
  uint32_t* lds;
  float lo, hi, scale;
  int32_t nbm1, w0;
  uint64_t* counts;
  uint32_t below = 0, above = 0;
  TSA_DEV void vec(const uint4& r) { some(r, 0xFFu); }
  template <int D = DT, class = std::enable_if_t<D == 1>>
  TSA_DEV void masked(const uint4& r, uint32_t mask) {
    some(r, mask);
  }
  TSA_DEV void some(const uint4& r, uint32_t mask) {  // mask: int16 only
    constexpr int N = Ty<DT>::EPV;
    float v[N];
    uint32_t rel[N];
    bool in = DT == 0 || mask == 0xFFu;
#pragma unroll
    for (int e = 0; e < N; ++e) {
      v[e] = (float)Ty<DT>::get(r, e);
      rel[e] = (uint32_t)(min((int32_t)((v[e] - lo) * scale), nbm1) - w0);
      in = in && v[e] >= lo && v[e] <= hi && rel[e] < kWinBins;  // NaN fails
    }
    if (__ballot(!in) == 0ull) {
#pragma unroll
      for (int e = 0; e < N; ++e) lds_inc(lds, rel[e]);
    } else {
#pragma unroll
      for (int e = 0; e < N; ++e) (*this)(v[e], DT == 0 || ((mask >> e) & 1u) != 0u);
    }
  }
  template <class T>
  TSA_DEV void operator()(T raw, bool in) {
    const float v = (float)raw;  // exact for int16
    below += (in && v < lo) ? 1u : 0u;
    above += (in && v > hi) ? 1u : 0u;
    if (in && v >= lo && v <= hi) {  // NaN fails both tests
      const float t = (v - lo) * scale;  // lo == hi: scale == 0 and t == 0
      const int32_t b = min(max((int32_t)t, 0), nbm1);
      const uint32_t rel = (uint32_t)(b - w0);
      if (rel < kWinBins)
        lds_inc(lds, rel);
      else
        atomicAdd((unsigned long long*)(counts + b), 1ull);
    }
  }
  TSA_DEV void chunk() {}
};

// ---- histogram with 16-bit LDS counters (up to 65536 bins) ---------------------
// Bins [b0, b0+nb) live as 16-bit halves of LDS words; every `epoch` calls of
// chunk() the block adds its non-zero counters to the global uint64 bins and
// clears them, so no half can carry into its neighbour (the caller bounds the
// elements per epoch by 65535).
struct Hist16Acc {
  uint32_t* lds;
  float lo, hi, scale;
  int32_t nbm1, b0, nb;
  uint64_t* counts;
  uint32_t epoch, chunks;
  bool count_out;
  uint32_t below, above;

  template <class T>
  TSA_DEV void operator()(T raw, bool in) {
    const float v = (float)raw;
    if (count_out) {
      below += (in && v < lo) ? 1u : 0u;
      above += (in && v > hi) ? 1u : 0u;
    }
    if (in && v >= lo && v <= hi) {
      const float d = v - lo;
      const float t = d * scale;
      const int32_t b = min(max((int32_t)t, 0), nbm1);
      const uint32_t rel = (uint32_t)(b - b0);
      if (rel < (uint32_t)nb)
        __hip_atomic_fetch_add(lds + (rel >> 1), 1u << ((rel & 1u) * 16u), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
  TSA_DEV void flush() {
    __syncthreads();
    const uint32_t words = ((uint32_t)nb + 1u) >> 1;
    for (uint32_t w = threadIdx.x; w < words; w += blockDim.x) {
      const uint32_t x = lds[w];
      if (x) {
        const uint32_t c0 = x & 0xFFFFu, c1 = x >> 16;
        if (c0) atomicAdd((unsigned long long*)(counts + b0 + 2 * w), (unsigned long long)c0);
        if (c1) atomicAdd((unsigned long long*)(counts + b0 + 2 * w + 1), (unsigned long long)c1);
        lds[w] = 0u;
      }
    }
    __syncthreads();
  }
  TSA_DEV void chunk() {
    if (++chunks == epoch) {
      chunks = 0;
      flush();
    }
  }
};

TSA_DEV void block_add_outliers(uint32_t below, uint32_t above, uint64_t* g, uint32_t* sm) {
  below = wave_sum_u32(below);
  above = wave_sum_u32(above);
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  if (lane == 0) {
    sm[2 * w] = below;
    sm[2 * w + 1] = above;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t b = 0, a = 0;
    for (int i = 0; i < (int)(blockDim.x / kWave); ++i) {
      b += sm[2 * i];
      a += sm[2 * i + 1];
    }
    if (b) atomicAdd((unsigned long long*)g, (unsigned long long)b);
    if (a) atomicAdd((unsigned long long*)(g + 1), (unsigned long long)a);
  }
}

// ---- digit selection and moment merges (whole block / one thread) -----------
// Wave-wide inclusive prefix sum of 32-bit values: Hillis-Steele steps of 1,
// 2, 4 and 8 lanes inside each row of 16 (DPP row shifts; a lane with no
// source adds 0), then lane 15 of rows 0 and 2 added to rows 1 and 3, then
// lane 31 added to rows 2 and 3 (DPP row broadcasts).
TSA_DEV uint32_t wave_scan_incl_u32(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);  // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast:15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return v;
}

// Block-wide choice of the digit holding rank k in a histogram of nb bins whose total
// fits in 32 bits: DPP scans, and every wave total read at once.  Returns false when k
// is not inside the histogram.  SH provides wsum32[16] (16-byte aligned), found,
// sel_digit, sel_cum32 and sel_bucket32 in LDS; blockDim.x is at most 1024.
// at(i): where counter i lies.
struct InOrder {
  TSA_DEV uint32_t operator()(uint32_t i) const { return i; }
};
template <class SH, class AT = InOrder>
TSA_DEV bool block_select_small(const uint32_t* hist, int nb, uint32_t k, SH& sh, uint32_t* digit,
                                uint32_t* cum_before, uint32_t* bucket, AT at = AT{}) {
  const int t = threadIdx.x, bs = blockDim.x;
  const int per = (nb + bs - 1) / bs;
  const int b0 = t * per;
  uint32_t local = 0;
  if (per <= 8 && (per & (per - 1)) != 0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {  // every read in flight at once
      const uint32_t h = hist[at(min(b0 + i, nb - 1))];
      local += (i < per && b0 + i < nb) ? h : 0u;
    }
  } else if ((per & (per - 1)) == 0) {  // a power of two: each run read from an offset rotated by t / 8,
    // so lanes whose runs start in the same bank read different banks (8 a run: none shared)
    for (int i = 0; i < per; ++i) {
      const int j = b0 + ((i + (t >> 3)) & (per - 1));
      if (j < nb) local += hist[at(j)];
    }
  } else {
    for (int i = 0; i < per; ++i)
      if (b0 + i < nb) local += hist[at(b0 + i)];
  }
  const int lane = t % kWave, w = t / kWave;
  const uint32_t inc = wave_scan_incl_u32(local);
  if (lane == kWave - 1) sh.wsum32[w] = inc;
  if (t == 0) sh.found = 0;
  __syncthreads();
  uint32_t base = inc - local;
  const uint4* ws4 = reinterpret_cast<const uint4*>(sh.wsum32);  // 16-byte aligned in SH
#pragma unroll
  for (int i = 0; i < 4; ++i) {  // waves below this one, four totals a read
    const uint4 v = ws4[i];
    base += (4 * i < w ? v.x : 0u) + (4 * i + 1 < w ? v.y : 0u) + (4 * i + 2 < w ? v.z : 0u) +
            (4 * i + 3 < w ? v.w : 0u);
  }
  if (local > 0 && k >= base && k - base < local) {
    uint32_t cum = base, in = 0;
    int d = b0;
    if (per <= 8) {
      uint32_t h[8], below = base;
#pragma unroll
      for (int i = 0; i < 8; ++i) h[i] = hist[at(min(b0 + i, nb - 1))];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t c = (i < per && b0 + i < nb) ? h[i] : 0u;
        if (k >= below && k - below < c) {
          d = b0 + i;
          cum = below;
          in = c;
        }
        below += c;
      }
    } else {
      for (int i = 0; i < per; ++i) {
        in = (b0 + i < nb) ? hist[at(b0 + i)] : 0u;
        if (k - cum < in) {
          d = b0 + i;
          break;
        }
        cum += in;
      }
    }
    sh.sel_digit = (uint32_t)d;
    sh.sel_cum32 = cum;
    sh.sel_bucket32 = in;
    sh.found = 1;
  }
  __syncthreads();
  const bool found = sh.found != 0;
  *digit = sh.sel_digit;
  *cum_before = sh.sel_cum32;
  *bucket = sh.sel_bucket32;
  __syncthreads();
  return found;
}

TSA_DEV double bvalue_of_key(uint32_t k, int dtype) {
  return dtype == 0 ? (double)__uint_as_float(f32bits_of_key(k)) : (double)i16_of_key(k);
}

// Every wave waits until its own global stores and atomics are acknowledged
// (s_waitcnt vmcnt(0)) before the barrier after which one thread publishes
// the block's work with an agent-scope release: a workgroup barrier alone
// does not wait for other waves' writes to reach the L2 that the release
// writes back.
TSA_DEV void block_writes_done() {
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt 0; expcnt and lgkmcnt not waited for
  __syncthreads();
}

// The blocks of a launch count themselves as they end; true in every thread of
// the last one, which sees what all the others published.  One block's work on
// a pass's results so needs no launch of its own.  Published is what agent-scope
// atomics wrote (counters added to, publish_partial): they act at the device's
// point of coherence, and every wave waits until its own are acknowledged
// before its block counts itself, so no block pays an agent-scope release (each
// writes back a whole L2: 20 us over a pass of 768 blocks).  Plain stores are
// for the launches that follow.  Blocks that end together
// queue on one counter (12 ns each, 9 us for 768), so they count in
// kArriveGroups counters on lines of their own, and the last of each group in
// a root.  All zero before the launch.
constexpr uint32_t kArriveGroups = 16, kArriveLine = 32;  // words
struct Arrive {
  uint32_t word[(kArriveGroups + 1) * kArriveLine];
};
TSA_DEV bool last_block(Arrive* a) {
  __shared__ uint32_t last;
  block_writes_done();
  if (threadIdx.x == 0) {
    const uint32_t g = blockIdx.x % kArriveGroups, ng = gridDim.x < kArriveGroups ? gridDim.x : kArriveGroups;
    const uint32_t mine = (gridDim.x - g + kArriveGroups - 1u) / kArriveGroups;
    uint32_t r = 0;
    if (__hip_atomic_fetch_add(a->word + g * kArriveLine, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == mine)
      r = __hip_atomic_fetch_add(a->word + kArriveGroups * kArriveLine, 1u, __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT) + 1u == ng;
    if (r) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    last = r;
  }
  __syncthreads();
  return last != 0;
}

// ---- radix digits of the key (Section 4.3 replaced by radix selection) --------
// Counters by the top 12 bits of every valid element: of the key for int16, of
// the bit pattern for float32 (the key's digit is digit_slot's inverse, taken
// once per counter when they are read instead of once per value).
template <int DT>
TSA_DEV uint32_t digit_slot(uint32_t d) {
  return DT == 0 ? d ^ (d & 0x800u ? 0x800u : 0xFFFu) : d;
}
template <int DT>
struct Digit1Acc {
  uint32_t base, shift, one;  // byte address of digit 0's replica of the lane, log2 bytes per digit, a 1
  TSA_DEV Digit1Acc(uint32_t* lds, uint32_t rshift)
      : base(in_register(lds_byte_addr(lds) + 4u * (threadIdx.x & ((1u << rshift) - 1u)))), shift(rshift + 2u),
        one(in_register(1u)) {}
  TSA_DEV void add(uint32_t bits) { lds_add_at(((bits >> kShift1) << shift) + base, one); }
  template <class T>
  TSA_DEV void operator()(T raw, bool in) {
    if (Elt<DT>::valid(raw, in)) {
      if constexpr (DT == 0)
        add(__float_as_uint(raw));
      else
        add(Elt<DT>::key(raw));
    }
  }
  TSA_DEV void four(const Four& f) {  // none of them NaN
#pragma unroll
    for (int e = 0; e < 4; ++e) add(f.u[e]);
  }
  template <int D = DT, class = std::enable_if_t<D == 0>>
  TSA_DEV void vec(const uint4& r) {
    const Four f(r);
    if (!f.wave_has_nan()) {
      four(f);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) (*this)(f.v[e], true);
    }
  }
  TSA_DEV void chunk() {}
};

// As lds_flush for Digit1Acc's counters, in key order.
template <int DT>
TSA_DEV void lds_flush_digits(const uint32_t* lds, uint32_t rshift, uint64_t* g) {
  const uint32_t R = 1u << rshift;
  for (uint32_t d = threadIdx.x; d < (uint32_t)kBins1; d += blockDim.x) {
    uint32_t c = 0;
    for (uint32_t r = 0; r < R; ++r) c += lds[(digit_slot<DT>(d) << rshift) + r];
    if (c) atomicAdd((unsigned long long*)(g + d), (unsigned long long)c);
  }
}

// Moments and first digit together (the count is the digit counters' total).
template <int DT>
struct Pass1Acc {
  MomAcc<DT, false> mom;
  Digit1Acc<DT> d1;
  TSA_DEV Pass1Acc(uint32_t* lds, uint32_t rshift) : d1(lds, rshift) {}
  template <class T>
  TSA_DEV void operator()(T raw, bool in) {
    mom(raw, in);
    d1(raw, in);
  }
  template <int D = DT, class = std::enable_if_t<D == 0>>
  TSA_DEV void vec(const uint4& r) {
    const Four f(r);
    if (!f.wave_has_nan()) {
      mom.four(f);
      d1.four(f);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) (*this)(f.v[e], true);
    }
  }
  TSA_DEV void chunk() {}
};

// Candidate keys are staged per wave in LDS and copied to the global list in
// runs of up to kWaveStage keys, so the global counter sees one atomic per run
// instead of one per wave instruction.  Each wave owns its stage: no block
// barrier is needed, so the block's waves keep their loads in flight.  The
// walkers call every accumulator from all lanes at the same points, so the
// wave's fill count is an ordinary variable that every lane updates alike
// (kept in a register, no LDS round trip per append).
// A copy-out waits for its global atomic, so a deeper stage (fewer copy-outs)
// pays where the LDS allows it.
constexpr uint32_t kWaveStage = 128;     // staged keys per wave (default)
constexpr uint32_t kWaveStageBig = 512;  // where the LDS has room
constexpr int kMaxWaves = 16;

// Staging of a block of NW waves, S keys each.
template <int NW, uint32_t S = kWaveStage>
struct CandSharedN {
  uint32_t buf[NW][S];
};
using CandShared = CandSharedN<kMaxWaves>;

// PUBLISH: another block of the same launch reads the list (agent-scope stores).
template <bool PUBLISH = false>
struct CandSink {
  uint32_t* buf;      // `stage` staged keys per wave
  uint32_t* list;     // global list
  uint32_t* counter;  // global fill counter
  uint32_t cap;       // global capacity
  uint32_t stage;     // keys per wave the stage holds
  uint32_t fill;      // keys this wave has staged (equal in every lane)
};
template <bool PUBLISH>
TSA_DEV void cand_put(const CandSink<PUBLISH>& k, uint32_t at, uint32_t key) {
  if (at >= k.cap) return;
  if constexpr (PUBLISH)
    __hip_atomic_store(k.list + at, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    k.list[at] = key;
}

template <bool PUBLISH = false, int NW, uint32_t S>
TSA_DEV CandSink<PUBLISH> cand_sink(CandSharedN<NW, S>& cs, uint32_t* list, uint32_t* counter, uint32_t cap) {
  return CandSink<PUBLISH>{&cs.buf[0][0], list, counter, cap, S, 0u};
}

// Staging carved from dynamic LDS: `stage` words per wave of the block.
TSA_DEV CandSink<> cand_sink_lds(uint32_t* base, uint32_t stage, uint32_t* list, uint32_t* counter, uint32_t cap) {
  return CandSink<>{base, list, counter, cap, stage, 0u};
}

// The wave copies its `fill` staged keys out (one global atomic).  Whole wave.
template <bool PUBLISH>
TSA_DEV void cand_copy_out(const CandSink<PUBLISH>& k, uint32_t fill) {
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  __builtin_amdgcn_wave_barrier();  // the staged writes of every lane come first
  uint32_t g = 0;
  if (lane == 0) g = atomicAdd(k.counter, fill);
  g = __builtin_amdgcn_readfirstlane(g);  // lane 0's result, without an LDS permute
  for (uint32_t i = lane; i < fill; i += kWave) cand_put(k, g + i, k.buf[w * k.stage + i]);
  __builtin_amdgcn_wave_barrier();  // and the reads finish before the stage is refilled
}

// Wave-aggregated append of the lanes whose flag is set (bal = their ballot).
// Kept inline: an out-of-line call costs the element loops more than its
// code size saves (measured on the fused pass B).
template <bool PUBLISH>
TSA_DEV void cand_append_slow(bool m, uint32_t key, uint64_t bal, CandSink<PUBLISH>& k) {
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  const uint32_t n = (uint32_t)__popcll(bal);
  if (k.fill + n > k.stage) {
    cand_copy_out(k, k.fill);
    k.fill = 0;
  }
  const uint32_t off = (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
  if (m) k.buf[w * k.stage + k.fill + off] = key;
  k.fill += n;
}

// Whole block (blockDim.x at most 1024): every wave's still-staged keys
// copied out under one global reservation for the block.  One same-address
// atomic per block instead of one per wave: when a thousand blocks end
// together (a small cube, one unit of work each) their waves' reservations
// queued on the one counter for tens of microseconds.
template <bool PUBLISH>
TSA_DEV void cand_finish_block(CandSink<PUBLISH>& k) {
  __shared__ uint32_t fill_w[16];
  __shared__ uint32_t base_b;
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  const int nw = (blockDim.x + kWave - 1) / kWave;
  if (lane == 0) fill_w[w] = k.fill;
  __syncthreads();  // also orders every lane's staged writes before the copy
  if (threadIdx.x == 0) {
    uint32_t tot = 0;
    for (int i = 0; i < nw; ++i) tot += fill_w[i];
    base_b = tot ? atomicAdd(k.counter, tot) : 0u;
  }
  __syncthreads();
  uint32_t g = base_b;
  for (int i = 0; i < w; ++i) g += fill_w[i];
  for (uint32_t i = lane; i < k.fill; i += kWave) cand_put(k, g + i, k.buf[w * k.stage + i]);
  k.fill = 0;
  __syncthreads();  // fill_w and base_b read by every wave before a later call rewrites them
}

// A first digit's bucket as an interval [lo, lo + span] of float32 bit
// patterns, cut to non-NaN values.
struct BitRange {
  uint32_t lo, span;
};
TSA_DEV BitRange bits_of_bucket(uint32_t p1) {
  const uint32_t k0 = max(p1 << kShift1, 0x007FFFFFu), k1 = min((p1 << kShift1) | ((1u << kShift1) - 1u), 0xFF800000u);
  const uint32_t u0 = f32bits_of_key(k0), u1 = f32bits_of_key(k1);
  return BitRange{min(u0, u1), max(u0, u1) - min(u0, u1)};  // a bucket has one sign
}

template <int DT, bool PUBLISH = false>
struct Level2Acc {  // keys inside the level-1 bucket: next 12 bits, optional copy
  uint32_t* lds;
  uint32_t p1;
  bool compact;
  CandSink<PUBLISH> sink;
  BitRange br;  // p1's (float32)
  // on false: no member
  TSA_DEV Level2Acc(uint32_t* l, uint32_t prefix, bool on, bool compact_, const CandSink<PUBLISH>& k)
      : lds(l), p1(on ? prefix >> kShift1 : 0xFFFFFFFFu), compact(on && compact_), sink(k),
        br(on ? bits_of_bucket(prefix >> kShift1) : BitRange{0x7FFFFFFFu, 0u}) {}
  // One subtraction and compare per value, the rest only in waves that hold a
  // member of the bucket.
  template <int D = DT, class = std::enable_if_t<D == 0>>
  TSA_DEV void vec(const uint4& r) {
    const uint32_t u[4] = {r.x, r.y, r.z, r.w};
    bool m[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) m[e] = u[e] - br.lo <= br.span;
    if (__ballot(m[0] || m[1] || m[2] || m[3]) == 0ull) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint64_t bal = __ballot(m[e]);
      if (bal != 0ull) {
        const uint32_t key = key_f32(u[e]);
        if (m[e]) lds_inc(lds, (key >> kShift2) & 0xFFFu);
        if (compact) cand_append_slow(m[e], key, bal, sink);
      }
    }
  }
  template <class T>
  TSA_DEV void operator()(T raw, bool in) {
    const uint32_t key = Elt<DT>::key(raw);
    const bool m = Elt<DT>::valid(raw, in) && (key >> kShift1) == p1;
    const uint64_t bal = __ballot(m);
    if (bal != 0ull) {  // rare: most waves skip both the count and the copy
      if (m) lds_inc(lds, (key >> kShift2) & 0xFFFu);
      if (compact) cand_append_slow(m, key, bal, sink);
    }
  }
  TSA_DEV void chunk() {}
  // what every wave still holds, one reservation for the block (call with
  // every thread of the block; compact is the same across the block)
  TSA_DEV void finish() {
    if (compact) cand_finish_block(sink);
  }
};

// Histogram (counted by H), second digit and second moment together.
template <int DT, class H, bool PUBLISH = false>
struct Pass2Acc {
  H h;
  Level2Acc<DT, PUBLISH> l2;
  VarAcc var;
  bool hist_on, sel_on, var_on;
  template <class T>
  TSA_DEV void operator()(T raw, bool in) {
    if (hist_on) h(raw, in);
    l2(raw, in);
    if constexpr (DT == 0) {
      if (var_on) var(raw, in);
    }
  }
  template <int D = DT, class = std::enable_if_t<D == 0>>
  TSA_DEV void vec(const uint4& r) {
    const Four f(r);
    if (!f.wave_has_nan()) {
      if (hist_on) h.four(f);
      if (var_on) var.four(f);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (hist_on) h(f.v[e], true);
        if (var_on) var(f.v[e], true);
      }
    }
    if (sel_on) l2.vec(r);
  }
  TSA_DEV void chunk() {}
};

template <int DT>
struct Level3Acc {  // keys inside the level-2 bucket: last 8 bits
  uint32_t* lds;
  uint32_t p2;
  template <class T>
  TSA_DEV void operator()(T raw, bool in) {
    const uint32_t key = Elt<DT>::key(raw);
    lds_inc_rare(lds, Elt<DT>::valid(raw, in) && (key >> kShift2) == p2, key & 0xFFu);
  }
  TSA_DEV void chunk() {}
};

}  // namespace tsa
