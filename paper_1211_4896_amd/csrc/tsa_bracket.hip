// Ranks of large float32 regions in one pass over the data.
//
// A sample of the region brackets the wanted value between two of the sample's
// own values, lo <= x <= hi.  One pass counts the voxels below, at and above
// either bound and copies the few strictly between them to a list; those
// counts say whether the rank lies at lo, at hi or in the list, and the list
// is then searched by key digits.  The counts are exact, so the answer is; when
// they show that the rank lies outside the bounds, or the list overflowed, the
// state is left unfinished and the passes by key digits that follow every
// bracket do the work (else they end at once).
//
// The bounds are values that voxels hold, and only what lies strictly between
// them is copied: a value that many voxels share is counted, never listed.
#include <math.h>

#include "tsa_internal.hpp"

namespace tsa {
namespace {

constexpr uint32_t kDigit = 4096;
constexpr int kSampleThreads = 1024, kSampleBlocks = 256, kBoundsBlocks = 32;
constexpr int kRefineThreads = 512, kRefineBlocks = 256, kRefineLoads = 4;
constexpr double kSigmas = 4.0, kRanks = 12.0;  // the bounds' distance from the wanted rank of the sample
// The least voxels of a region that is bracketed: the launches around the pass
// take 95 us, so from 2^27 voxels on every call gains.  us, key digits ->
// bracket, of standard normal noise about 0 (the passes' best case: the first
// digit leaves few voxels), of noise of 0.1 about 100, and of one value:
//   2^26: median 103 -> 131, 220 -> 116, 579 -> 126; 0.9-quantile 147 -> 123; MAD 254 -> 254
//   2^27: median 178 -> 172, 401 -> 155, 1132 -> 165; 0.9-quantile 259 -> 166; MAD 439 -> 336
//   2^28: median 335 -> 255, 774 -> 236, 2233 -> 245; 0.9-quantile 493 -> 248; MAD 829 -> 504
// A region without a valid voxel pays for the launches (median of 2^27 voxels 93 ->
// 131): its first digit would have ended the call.
constexpr int64_t kBracketMin = 1ll << 27;
constexpr uint32_t kNoKey = 0xFFFFFFFFu;  // a sampled NaN (no value has this key)
constexpr uint32_t kKeyMinusInf = 0x007FFFFFu, kKeyPlusInf = 0xFF800000u;

struct Bracket {
  uint64_t k;        // rank still to find within the list
  uint64_t n;        // valid voxels
  float lo, hi;
  uint32_t klo, span;  // lo's key, hi's key - lo's
  unsigned long long nlist;  // voxels between the bounds (atomic; the list holds the first `cap`)
  uint32_t pending;  // 1: the rank lies in the list
  uint32_t prefix;   // top bits of (key - klo) found so far
};

// How the two bounds (0: lo, 1: hi) are found among the sampled keys.
struct Pick {
  uint32_t open[2];   // 1: the bound is infinite
  uint32_t prefix[2]; // the bound's digits found so far
  uint32_t rank[2];   // its rank among the keys that share them
};

// Everything here starts at zero.
struct BracketMem {
  Bracket b;
  Pick pick;
  Arrive arrive[7];
  uint32_t sample[kDigit];       // the sample by first digit
  uint32_t bound[2][2][kDigit];  // by second and last digit, around either bound
  uint32_t list[3][kDigit];      // the list by digit
};

struct PickShared {
  alignas(16) uint32_t wsum32[16];
  uint32_t found, sel_digit, sel_cum32, sel_bucket32, total;
};

TSA_DEV float dev_of(float x, float m) { return x == m ? 0.0f : fabsf(x - m); }
TSA_DEV uint32_t dev_key(uint32_t key, float m) {
  return key == kNoKey ? key : key_f32(__float_as_uint(dev_of(__uint_as_float(f32bits_of_key(key)), m)));
}
TSA_DEV float median_value(const SelState* med) { return __uint_as_float(f32bits_of_key(med->result_key)); }
TSA_DEV uint64_t rank_of(const SelState* st, uint64_t n) {  // n > 0
  if (!st->rank_mode) return (n - 1) / 2;
  const double kk = floor(st->q * (double)(n - 1));
  return kk <= 0.0 ? 0 : kk >= (double)(n - 1) ? n - 1 : (uint64_t)kk;
}

// ---------------------------------------------------------------------------
// the bounds
// ---------------------------------------------------------------------------
// One block: the ranks of the bounds among the sampled keys (whose counts by
// first digit are `first`) and their first digits.
TSA_DEV void choose_ranks(const uint32_t* first, const SelState* st, Pick* p, uint32_t* h) {
  __shared__ PickShared sh;
  const uint32_t t = threadIdx.x, bs = blockDim.x;
  if (t == 0) sh.total = 0;
  __syncthreads();
  uint32_t c = 0;
  for (uint32_t i = t; i < kDigit; i += bs) c += h[i] = first[i];
  c = wave_scan_incl_u32(c);
  if (t % kWave == kWave - 1) atomicAdd(&sh.total, c);
  __syncthreads();
  const uint32_t nv = sh.total;
  // 4 standard deviations of a sample rank to either side (and 12 ranks: the
  // tails of q near 0 and 1), 6 in 100000 to miss
  const double q = st->rank_mode ? st->q : 0.5, mid = q * ((double)nv - 1.0);
  const double half = kSigmas * sqrt((double)nv * q * (1.0 - q)) + kRanks;
  const double r[2] = {floor(mid - half), ceil(mid + half)};
  const bool open[2] = {!(r[0] >= 0.0), !(r[1] < (double)nv)};
  for (int j = 0; j < 2; ++j) {
    uint32_t digit = 0, below = 0, in = 0, rank = 0;
    if (!open[j]) {
      rank = (uint32_t)r[j];
      block_select_small(h, (int)kDigit, rank, sh, &digit, &below, &in);
    }
    if (t == 0) {
      p->open[j] = open[j] ? 1u : 0u;
      p->prefix[j] = digit;
      p->rank[j] = rank - below;
    }
  }
}

// ns voxels, one from each of ns equal runs of the region at a place that
// differs from run to run, or (DEV) the deviations of those voxels from the
// median, by first digit.  Bound by the latency of scattered loads (one a lane).
template <bool DEV>
__global__ __launch_bounds__(kSampleThreads) void k_sample(const float* __restrict__ base, int64_t nx, int64_t ny,
                                                           tsa_region box, uint32_t* __restrict__ keys, uint32_t ns,
                                                           BracketMem* m, const SelState* __restrict__ st,
                                                           const SelState* __restrict__ med) {
  __shared__ uint32_t h[kDigit];
  if (DEV && (!med->done || med->n == 0)) return;
  float mf = 0.0f;
  if constexpr (DEV) mf = median_value(med);
  const uint32_t t = threadIdx.x;
  lds_zero(h, kDigit);
  __syncthreads();
  const uint32_t stride = gridDim.x * blockDim.x;
  if constexpr (DEV) {
    for (uint32_t s = blockIdx.x * blockDim.x + t; s < ns; s += stride) {
      const uint32_t key = dev_key(keys[s], mf);
      if (key != kNoKey) lds_inc(h, key >> kShift1);
    }
  } else {
    const uint64_t lx = (uint64_t)(box.x1 - box.x0), ly = (uint64_t)(box.y1 - box.y0);
    const uint64_t run = lx * ly * (uint64_t)(box.z1 - box.z0) / ns;
    for (uint32_t s = blockIdx.x * blockDim.x + t; s < ns; s += stride) {
      const uint64_t i = s * run + ((run * (uint64_t)(s * 0x9E3779B1u)) >> 32);  // run < 2^32
      const uint64_t row = i / lx, x = i - row * lx, z = row / ly, y = row - z * ly;
      const float v = base[((box.z0 + (int64_t)z) * ny + (box.y0 + (int64_t)y)) * nx + box.x0 + (int64_t)x];
      const uint32_t key = v == v ? key_f32(__float_as_uint(v)) : kNoKey;
      if (v == v) lds_inc(h, key >> kShift1);
      keys[s] = key;
    }
  }
  __syncthreads();
  for (uint32_t i = t; i < kDigit; i += blockDim.x)
    if (h[i]) atomicAdd(m->sample + i, h[i]);
  if (!last_block(m->arrive + 0)) return;
  choose_ranks(m->sample, st, &m->pick, h);
}

// The bounds' second (level 2) and last digits, counted over the sampled keys
// that share the digits before; the last block picks.  Bound by launch latency.
template <bool DEV>
__global__ __launch_bounds__(kSampleThreads) void k_bounds(int level, const uint32_t* __restrict__ keys, uint32_t ns,
                                                           BracketMem* m, const SelState* __restrict__ med) {
  __shared__ uint32_t h[2][kDigit];
  __shared__ PickShared sh;
  if (DEV && (!med->done || med->n == 0)) return;
  float mf = 0.0f;
  if constexpr (DEV) mf = median_value(med);
  const uint32_t t = threadIdx.x, bs = blockDim.x;
  const Pick p = m->pick;
  const int above = level == 2 ? kShift1 : kShift2, shift = level == 2 ? kShift2 : 0;
  const uint32_t nd = level == 2 ? kBins2 : kBins3;
  lds_zero(h[0], 2 * kDigit);
  __syncthreads();
  const uint4* k4 = (const uint4*)keys;
  for (uint32_t i = blockIdx.x * bs + t; i < ns / 4; i += gridDim.x * bs) {
    const uint4 v = k4[i];
    const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t key = DEV ? dev_key(u[e], mf) : u[e];
#pragma unroll
      for (int j = 0; j < 2; ++j)
        if (!p.open[j] && (key >> above) == p.prefix[j]) lds_inc(h[j], (key >> shift) & (nd - 1u));
    }
  }
  __syncthreads();
  uint32_t* counts = m->bound[level - 2][0];
  for (uint32_t i = t; i < 2 * kDigit; i += bs)
    if (h[0][i]) atomicAdd(counts + i, h[0][i]);
  if (!last_block(m->arrive + level - 1)) return;
  for (uint32_t i = t; i < 2 * kDigit; i += bs) h[0][i] = counts[i];
  __syncthreads();
  uint32_t key[2] = {kKeyMinusInf, kKeyPlusInf};
  for (int j = 0; j < 2; ++j) {
    if (p.open[j]) continue;
    uint32_t d = 0, below = 0, in = 0;
    block_select_small(h[j], (int)nd, p.rank[j], sh, &d, &below, &in);
    key[j] = p.prefix[j] * nd + d;
    if (t == 0) {
      m->pick.prefix[j] = key[j];
      m->pick.rank[j] = p.rank[j] - below;
    }
  }
  if (t == 0 && level == 3) {
    Bracket& b = m->b;
    b.klo = key[0];
    b.span = key[1] - key[0];
    b.lo = __uint_as_float(f32bits_of_key(key[0]));
    b.hi = __uint_as_float(f32bits_of_key(key[1]));
  }
}

// ---------------------------------------------------------------------------
// the pass
// ---------------------------------------------------------------------------
// Every lane stages the values between the bounds in an LDS column of its own
// (two instructions a value, no ballots between elements); a wave whose fullest
// column nears its end copies all of them out under one reservation.
// Columns of 32 take 909 us over 5.4 GB, of 16 928, of 8 1448 (a wave's
// reservation is one atomic on one counter, 12 ns each over the whole chip).
constexpr size_t kStageBytes = 65536;  // of a block, what a launch takes without raising its LDS limit

template <bool DEV>
struct BracketAcc {
  float lo, hi, mf;
  bool zeros;  // a bound is zero: its two signs are told apart
  uint32_t lt = 0, le = 0, upto = 0, n = 0, minus0 = 0;
  uint32_t col, at, full;  // LDS byte addresses: the lane's column, its next free word, the first with less than four behind it
  uint32_t* list;
  unsigned long long* counter;
  uint32_t cap;
  TSA_DEV BracketAcc(uint32_t* lds, uint32_t depth, const Bracket& b, float m, uint32_t* l, unsigned long long* c,
                     uint32_t cap_)
      : lo(b.lo), hi(b.hi), mf(m), zeros(b.lo == 0.0f || b.hi == 0.0f),
        col(lds_byte_addr(lds) + 4u * ((threadIdx.x / kWave) * depth * kWave + threadIdx.x % kWave)), at(col),
        full(col + (depth - 4u) * 4u * kWave), list(l), counter(c), cap(cap_) {}
  TSA_DEV uint32_t staged() const { return (at - col) / (4u * kWave); }
  // reserve n places; the first, at most cap (what lies past cap is not kept)
  TSA_DEV uint32_t reserve(uint32_t n) const {
    const unsigned long long g = atomicAdd(counter, (unsigned long long)n);
    return g < cap ? (uint32_t)g : cap;
  }
  TSA_DEV void copy_out(uint32_t g) {
    for (uint32_t a = col; a < at; a += 4u * kWave, ++g)
      if (g < cap) list[g] = *(lds_word*)(uintptr_t)a;
    at = col;
  }
  TSA_DEV bool count(float v) {
    const bool low = v <= lo;
    lt += v < lo ? 1u : 0u;
    le += low ? 1u : 0u;
    upto += v <= hi ? 1u : 0u;
    n += v == v ? 1u : 0u;
    return v < hi && !low;
  }
  TSA_DEV void keep(float v) {
    *(lds_word*)(uintptr_t)at = __float_as_uint(v);
    at += 4u * kWave;
  }
  // room for four more in every column of the wave
  TSA_DEV void make_room() {
    if (__ballot(at > full) == 0ull) return;
    const uint32_t mine = staged(), upto_me = wave_scan_incl_u32(mine);
    const uint32_t all = __builtin_amdgcn_readlane(upto_me, kWave - 1);
    uint32_t g = 0;
    if (threadIdx.x % kWave == 0) g = reserve(all);
    copy_out(__builtin_amdgcn_readfirstlane(g) + upto_me - mine);
  }
  TSA_DEV void vec(const uint4& r) {
    const uint32_t u[4] = {r.x, r.y, r.z, r.w};
    float v[4];
    bool in[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = DEV ? dev_of(__uint_as_float(u[e]), mf) : __uint_as_float(u[e]);
      in[e] = count(v[e]);
    }
    if (!DEV && zeros) {
#pragma unroll
      for (int e = 0; e < 4; ++e) minus0 += u[e] == 0x80000000u ? 1u : 0u;
    }
    if (__ballot(in[0] || in[1] || in[2] || in[3]) == 0ull) return;
    make_room();
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (in[e]) keep(v[e]);
  }
  TSA_DEV void operator()(float x, bool in_box) {
    const float v = in_box ? (DEV ? dev_of(x, mf) : x) : __builtin_nanf("");
    const bool in = count(v);
    if (!DEV && zeros) minus0 += __float_as_uint(v) == 0x80000000u ? 1u : 0u;
    if (__ballot(in) == 0ull) return;
    make_room();
    if (in) keep(v);
  }
  TSA_DEV void chunk() {}
};

// The answer: key of rank k among n valid values.
TSA_DEV void finish(SelState* st, uint32_t key, uint64_t n, const BracketAsk& ask) {
  const double v = (double)__uint_as_float(f32bits_of_key(key));
  st->n = n;
  st->result_key = key;
  st->done = 1;
  if (ask.qout) {
    ask.qout[0] = v;
    ask.qout[1] = 0.0;
    ask.qout[2] = (double)n;
  }
  ask.out->median = v;
  if (ask.write_counts) {
    ask.out->count = n;
    ask.out->nan_count = ask.volume - n;
    ask.out->status = TSA_OK;
  }
}

// Bound by HBM: 1024x1024x1280 voxels (5.4 GB) 0.91 ms, 5.9 TB/s (deviations
// 0.96), two blocks per compute unit.  One block 1.13, three 0.98, loads a
// chunk ahead 0.94 and 1.12 for the deviations.  MAD and 0.9-quantile of those
// voxels: 6.55 -> 2.95 ms.
template <int VEC, bool NT, bool DEV>
__global__ __launch_bounds__(1024) void k_bracket(Geom g, uint32_t depth, BracketMem* m, uint32_t* __restrict__ list, uint32_t cap,
                                                  uint64_t* __restrict__ parts, SelState* __restrict__ st,
                                                  const SelState* __restrict__ med, BracketAsk ask) {
  extern __shared__ uint32_t lds[];  // [waves][depth][kWave] staged values
  __shared__ uint32_t wsum[5][16], staged[16], first;
  __shared__ unsigned long long total[5];
  if (DEV && (!med->done || med->n == 0)) return;
  const uint32_t t = threadIdx.x, w = t / kWave, nw = blockDim.x / kWave;
  const Bracket b = m->b;
  BracketAcc<DEV> a(lds, depth, b, DEV ? median_value(med) : 0.0f, list, &m->b.nlist, cap);
  walk<0, VEC, kUnroll, NT>(g, a);
  // what the waves still hold: one reservation for the block
  const uint32_t mine = a.staged(), upto_me = wave_scan_incl_u32(mine);
  const uint32_t c[5] = {wave_scan_incl_u32(a.lt), wave_scan_incl_u32(a.le), wave_scan_incl_u32(a.upto),
                         wave_scan_incl_u32(a.n), wave_scan_incl_u32(a.minus0)};
  if (t % kWave == kWave - 1) {
    staged[w] = upto_me;
#pragma unroll
    for (int j = 0; j < 5; ++j) wsum[j][w] = c[j];
  }
  __syncthreads();
  if (t == 0) {
    uint32_t all = 0;
    for (uint32_t i = 0; i < nw; ++i) all += staged[i];
    first = all ? a.reserve(all) : 0u;
  }
  if (t < 5) {
    uint64_t s = 0;
    for (uint32_t i = 0; i < nw; ++i) s += wsum[t][i];
    __hip_atomic_store(parts + 5 * (uint64_t)blockIdx.x + t, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    total[t] = 0;
  }
  __syncthreads();
  uint32_t at = first;
  for (uint32_t i = 0; i < w; ++i) at += staged[i];
  a.copy_out(at + upto_me - mine);
  if (!last_block(m->arrive + 3)) return;
  uint64_t s[5] = {0, 0, 0, 0, 0};
  for (uint32_t i = t; i < gridDim.x; i += blockDim.x)
#pragma unroll
    for (int j = 0; j < 5; ++j) s[j] += parts[5 * (uint64_t)i + j];
#pragma unroll
  for (int j = 0; j < 5; ++j) atomicAdd(&total[j], (unsigned long long)s[j]);
  __syncthreads();
  if (t != 0) return;
  const uint64_t below = total[0], upto_lo = total[1], upto_hi = total[2], n = total[3], minus0 = total[4];
  const uint64_t nlist = __hip_atomic_load(&m->b.nlist, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (n == 0) {
    st->n = 0;
    st->done = 1;
    if (ask.qout) {
      ask.qout[0] = ask.qout[1] = __builtin_nan("");
      ask.qout[2] = 0.0;
    }
    ask.out->median = __builtin_nan("");
    if (ask.write_counts) {
      ask.out->count = 0;
      ask.out->nan_count = ask.volume;
      ask.out->status = TSA_OK;
    }
    return;
  }
  const uint64_t k = rank_of(st, n);
  // the bound `x`, `at` voxels of its value (both zeros are one) below the rank
  auto bound = [&](float x, uint64_t at) {
    return x == 0.0f ? key_f32(at < minus0 ? 0x80000000u : 0u) : key_f32(__float_as_uint(x));
  };
  if (k < below || k >= upto_hi) return;  // outside the bounds
  if (k < upto_lo)
    finish(st, bound(b.lo, k - below), n, ask);
  else if (k - upto_lo >= nlist)
    finish(st, bound(b.hi, k - upto_lo - nlist), n, ask);
  else if (nlist <= cap) {
    m->b.n = n;
    m->b.k = k - upto_lo;
    m->b.pending = 1;
  }
}

// ---------------------------------------------------------------------------
// the list, by digits of (key - klo) from the top bit of the span: 12, 12, 8
// (10.5 million keys: 13 us a digit; twice the blocks 15, their counts' additions)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kRefineThreads) void k_refine(int level, BracketMem* m, const uint32_t* __restrict__ list,
                                                           SelState* __restrict__ st, BracketAsk ask) {
  __shared__ uint32_t h[kDigit];
  __shared__ PickShared sh;
  if (!m->b.pending) return;
  const uint32_t t = threadIdx.x, n = (uint32_t)m->b.nlist, klo = m->b.klo, prefix = m->b.prefix;
  const int top = 32 - __clz((int)m->b.span);
  const int s1 = max(top - 12, 0), s2 = max(s1 - 12, 0);
  const int above = level == 1 ? 31 : level == 2 ? s1 : s2, shift = level == 1 ? s1 : level == 2 ? s2 : 0;
  const uint32_t d0 = level == 1 ? 0u : prefix << (above - shift);
  lds_zero(h, kDigit);
  __syncthreads();
  auto add = [&](uint32_t u) {
    const uint32_t d = key_f32(u) - klo;
    if (level == 1 || (d >> above) == prefix) lds_inc(h, (d >> shift) - d0);
  };
  const uint4* l4 = (const uint4*)list;
  const uint32_t n4 = n / 4, stride = gridDim.x * blockDim.x;
  for (uint32_t i = blockIdx.x * blockDim.x + t; i < n4; i += kRefineLoads * stride) {
    uint4 v[kRefineLoads];
#pragma unroll
    for (int l = 0; l < kRefineLoads; ++l) v[l] = l4[min(i + l * stride, n4 - 1)];
#pragma unroll
    for (int l = 0; l < kRefineLoads; ++l)
      if (i + l * stride < n4) {
        add(v[l].x);
        add(v[l].y);
        add(v[l].z);
        add(v[l].w);
      }
  }
  if (blockIdx.x == 0 && t < n % 4) add(list[n / 4 * 4 + t]);
  __syncthreads();
  uint32_t* hist = m->list[level - 1];
  for (uint32_t i = t; i < kDigit; i += blockDim.x)
    if (h[i]) atomicAdd(hist + i, h[i]);
  if (!last_block(m->arrive + 3 + level)) return;
  const uint32_t k = (uint32_t)m->b.k;  // below nlist
  for (uint32_t i = t; i < kDigit; i += blockDim.x) h[i] = hist[i];
  __syncthreads();
  uint32_t digit = 0, below = 0, in = 0;
  const bool found = block_select_small(h, (int)kDigit, k, sh, &digit, &below, &in);
  if (t != 0) return;
  if (!found || shift == 0) m->b.pending = 0;
  if (!found) return;  // never expected; the passes by key digits answer
  m->b.k = k - below;
  m->b.prefix = d0 + digit;
  if (shift == 0) finish(st, klo + d0 + digit, m->b.n, ask);
}

template <int VEC, bool NT, bool DEV>
void launch_bracket(const Geom& g, int grid, int block, BracketMem* m, uint32_t* list, uint32_t cap, uint64_t* parts,
                    SelState* st, const SelState* med, const BracketAsk& ask, hipStream_t s) {
  const uint32_t depth = (uint32_t)(kStageBytes / 4 / (size_t)block);
  hipLaunchKernelGGL((k_bracket<VEC, NT, DEV>), dim3(grid), dim3(block), kStageBytes, s, g, depth, m, list, cap, parts,
                     st, med, ask);
}

}  // namespace

static_assert(8 * (kBins1 + kBins2 + kBins3) % 16 == 0 &&
                  8 * (kBins1 + kBins2 + kBins3) + 2 * (sizeof(BracketMem) + 255) <= 8 * (size_t)kHistCopies * kCopyBinsMax,
              "two brackets behind the deviations' digit counts");
size_t bracket_bytes() { return (sizeof(BracketMem) + 255) / 256 * 256; }

// Voxels to sample for a region of `volume` voxels whose list may hold cand_cap
// keys (the sample's own keys lie behind it); 0: by key digits.  With the 2^26 keys
// of the largest workspaces: 2^18 voxels up to 7.0e9, 2^20 up to 1.40e10, 2^22
// up to 2.676e10 (107 GB), above that none.
uint32_t bracket_samples(int64_t volume, uint32_t cand_cap) {
  if (volume < kBracketMin) return 0;
  for (uint32_t ns = kSampleBlocks * kSampleThreads; ns <= 1u << 22; ns *= 4) {
    const double share = (kSigmas * sqrt((double)ns) + 2.0 * kRanks) / ns;  // choose_ranks' widest
    if (cand_cap > ns && 1.2 * share * (double)volume <= (double)(cand_cap - ns)) return ns;
  }
  return 0;
}

int run_bracket(const tsa_cube* cube, const tsa_region& box, const Geom& g, int vec, bool nt, int grid, int block,
                void* mem, uint32_t ns, uint32_t* cand, uint32_t cand_cap, void* parts, SelState* st,
                const SelState* med, const BracketAsk& ask, hipStream_t s) {
  BracketMem* m = (BracketMem*)mem;
  const uint32_t cap = (cand_cap - ns) & ~3u;
  uint32_t* keys = cand + cap;
#define TSA_SAMPLE(DEV)                                                                                            \
  TSA_TRACED("sample", s,                                                                                          \
             hipLaunchKernelGGL(k_sample<DEV>, dim3(kSampleBlocks), dim3(kSampleThreads), 0, s,                    \
                                (const float*)cube->data, cube->nx, cube->ny, box, keys, ns, m,                    \
                                (const SelState*)st, med));                                                        \
  for (int level = 2; level <= 3; ++level)                                                                         \
    TSA_TRACED("bounds", s,                                                                                        \
               hipLaunchKernelGGL(k_bounds<DEV>, dim3(kBoundsBlocks), dim3(kSampleThreads), 0, s, level,           \
                                  (const uint32_t*)keys, ns, m, med))
  if (med) {
    TSA_SAMPLE(true);
  } else {
    TSA_SAMPLE(false);
  }
#undef TSA_SAMPLE
#define TSA_BRACKET(V, N)                                                                                       \
  TSA_TRACED("bracket", s,                                                                                      \
             med ? launch_bracket<V, N, true>(g, grid, block, m, cand, cap, (uint64_t*)parts, st, med, ask, s)  \
                 : launch_bracket<V, N, false>(g, grid, block, m, cand, cap, (uint64_t*)parts, st, med, ask, s))
  if (vec == 1 && nt)
    TSA_BRACKET(1, true);
  else if (vec == 1)
    TSA_BRACKET(1, false);
  else if (vec == 2)
    TSA_BRACKET(2, true);
  else
    TSA_BRACKET(0, false);
#undef TSA_BRACKET
  for (int level = 1; level <= 3; ++level)
    TSA_TRACED("refine", s,
               hipLaunchKernelGGL(k_refine, dim3(kRefineBlocks), dim3(kRefineThreads), 0, s, level, m,
                                  (const uint32_t*)cand, st, ask));
  return hipGetLastError() == hipSuccess ? TSA_OK : TSA_EDEVICE;
}

}  // namespace tsa
