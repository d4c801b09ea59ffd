// int16 cubes: every statistic from one count of the values.
//
// An int16 voxel holds one of 65536 values, so the number of voxels of each
// value is a complete summary: count, sums, extremes, any histogram, any rank
// and the median absolute deviation follow from it exactly.  One pass over
// the data counts the values in LDS; small kernels then read the answers from
// the counts, whatever their number.
//
// The count keeps all 65536 counters of a block as 16-bit halves of 32768 LDS
// words (128 KB, one 1024-lane block per compute unit): word i holds the
// value i in its low half and the value i - 32768 in its high half.  A half
// may wrap: the increments return the word they found, a wave takes the
// packed maximum of what came back, and only when some half was 65535 does a
// lane look at its own increments and count the wrap in global memory.  The
// sums are exact for any data and no barrier interrupts the loads.
//
// Bound: HBM reads (6.25 TB/s).  2048^3 voxels (17.2 GB), all three statistics:
// 7.64 ms in two passes that the vector ALU bounded (17 operations a voxel
// each, lane masks spilled) -> 2.66 ms.  One value in 2^29 voxels: 3.1 ms -> 0.26.
#include <math.h>

#include "tsa_internal.hpp"

namespace tsa {
namespace {

constexpr uint32_t kVals = 65536, kWords = 32768;
constexpr uint32_t kGroup = 1024, kGroups = kVals / kGroup;
constexpr int kCountThreads = kCount16Step / kUnroll;

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

TSA_DEV uint32_t lds_add_rtn(uint32_t byte_addr, uint32_t v) {
  return __hip_atomic_fetch_add((lds_word*)(uintptr_t)byte_addr, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
TSA_DEV uint32_t pk_max(uint32_t a, uint32_t b) {
  const u16x2 m = __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b));
  return __builtin_bit_cast(uint32_t, m);
}
TSA_DEV bool half_full(uint32_t m) { return (m & 0xFFFFu) == 0xFFFFu || m >= 0xFFFF0000u; }

// One 16-byte vector costs 5 VALU operations and one LDS increment a voxel.  A
// lane whose eight voxels are equal adds 8 at once: in runs of one value (sorted
// data, blanked parts) a wave's lanes meet on few words, and each increment of a
// shared word waits for the one before.
struct Count16Acc {
  uint32_t base;  // LDS byte address of the words
  uint64_t* adj;  // by key: what the wraps add (mod 2^64)
  // the increment `inc` of the word at byte offset `at` found `old`
  TSA_DEV void wrapped(uint32_t at, uint32_t inc, uint32_t old) {
    const uint32_t i = at >> 2;  // the high half's key; the low half's is i + 32768
    if ((old & 0xFFFFu) + (inc & 0xFFFFu) > 0xFFFFu) {  // the low half wrapped into the high one
      atomicAdd((unsigned long long*)(adj + kWords + i), 65536ull);
      atomicAdd((unsigned long long*)(adj + i), ~0ull);
    }
    if (old + inc < old) atomicAdd((unsigned long long*)(adj + i), 65536ull);  // the word wrapped
  }
  // whether some lane of the wave may hold eight equal voxels (none does in most waves of noise)
  TSA_DEV static bool may_run(const uint4& r) { return __ballot(r.x == r.w) != 0ull; }
  // The vectors of a chunk: one test for all of them (a test each: 2660 -> 2715 us over 2048^3 voxels).
  template <int U>
  TSA_DEV void vecs(const uint4 (&r)[U]) {
    if (may_run(r[0])) {
#pragma unroll
      for (int u = 0; u < U; ++u) vec(r[u]);
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) singles(r[u]);
    }
  }
  TSA_DEV void vec(const uint4& r) {
    if (may_run(r) && r.x == r.w && r.x == r.y && r.x == r.z && r.x >> 16 == (r.x & 0xFFFFu)) {
      const uint32_t at = (r.x << 2) & 0x1FFFCu, inc = (r.x & 0x8000u) ? 0x80000u : 8u;
      wrapped(at, inc, lds_add_rtn(base + at, inc));
    } else {
      singles(r);
    }
  }
  TSA_DEV void singles(const uint4& r) {
    const uint32_t w[4] = {r.x, r.y, r.z, r.w};
    uint32_t at[8], inc[8], old[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      at[2 * e] = (w[e] << 2) & 0x1FFFCu;
      at[2 * e + 1] = (w[e] >> 14) & 0x1FFFCu;
      inc[2 * e] = (w[e] & 0x8000u) ? 0x10000u : 1u;
      inc[2 * e + 1] = (w[e] & 0x80000000u) ? 0x10000u : 1u;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) old[e] = lds_add_rtn(base + at[e], inc[e]);
    uint32_t m = old[0];
#pragma unroll
    for (int e = 1; e < 8; ++e) m = pk_max(m, old[e]);
    if (half_full(m)) {
#pragma unroll
      for (int e = 0; e < 8; ++e) wrapped(at[e], inc[e], old[e]);
    }
  }
  TSA_DEV void operator()(int16_t x, bool in) {
    if (in) {
      const uint32_t at = ((uint32_t)x & 0x7FFFu) << 2, inc = x < 0 ? 0x10000u : 1u;
      const uint32_t old = lds_add_rtn(base + at, inc);
      if (half_full(old)) wrapped(at, inc, old);
    }
  }
  TSA_DEV void chunk() {}
};

// tables: one table of kWords per block; else (null) the counts are added to
// pk, word i as (low half, high half) of one 64-bit counter.
template <int VEC>
__global__ __launch_bounds__(kCountThreads) void k_count16(Geom g, uint32_t* __restrict__ tables,
                                                           uint64_t* __restrict__ pk, uint64_t* __restrict__ adj) {
  __shared__ __align__(16) uint32_t lds[kWords];
  for (uint32_t i = threadIdx.x; i < kWords / 4; i += blockDim.x) ((uint4*)lds)[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  Count16Acc a{lds_byte_addr(lds), adj};
  walk<1, VEC, kUnroll, true, true>(g, a);
  __syncthreads();
  if (tables) {
    uint4* t = (uint4*)(tables + (size_t)blockIdx.x * kWords);
    for (uint32_t i = threadIdx.x; i < kWords / 4; i += blockDim.x) t[i] = ((const uint4*)lds)[i];
  } else {
    // blocks start at different words: they end together, and would queue on the same counters
    const uint32_t first = (uint32_t)(((uint64_t)blockIdx.x * kWords) / gridDim.x) & ~63u;
    for (uint32_t j = threadIdx.x; j < kWords; j += blockDim.x) {
      const uint32_t i = (j + first) & (kWords - 1u), w = lds[i];
      if (w) atomicAdd((unsigned long long*)(pk + i), (unsigned long long)(w & 0xFFFFu) | ((unsigned long long)(w >> 16) << 32));
    }
  }
}

// The sum of v^2 over voxels as high 2^20 + low.  One value's count c is split
// at 2^20, so its parts are below 2^50 and (c < 2^46) 2^56, and the low parts of
// a group of 1024 values sum to less than 2^60; all 65536 values' would not fit
// 64 bits, so each group's low part is carried into its high part before groups
// are added.  The high part of everything is below 2^30 2^46 / 2^20.
struct Squares {
  uint64_t low, high;
};
__host__ __device__ __forceinline__ Squares squares_of(int64_t v, uint64_t c) {
  const uint64_t v2 = (uint64_t)(v * v);
  return Squares{v2 * (c & 0xFFFFFull), v2 * (c >> 20)};
}
__host__ __device__ __forceinline__ Squares carried(const Squares& q) {
  return Squares{q.low & 0xFFFFFull, q.high + (q.low >> 20)};
}

// Sums of one group of kGroup keys.
struct Group16 {
  uint64_t n;
  Squares q;  // carried
  int64_t s;
  uint32_t kmin, kmax;  // keys that occur (kmin > kmax: none)
  uint64_t pad;
};
static_assert(sizeof(Group16) == 48, "group layout");

// Exclusive prefix of v over the block's threads; total in *tot.
TSA_DEV uint64_t block_prefix_u64(uint64_t v, uint64_t* wsum, uint64_t* tot) {
  const int lane = threadIdx.x % kWave, w = threadIdx.x / kWave;
  uint64_t inc = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint64_t y = __shfl_up(inc, o);
    if (lane >= o) inc += y;
  }
  if (lane == kWave - 1) wsum[w] = inc;
  __syncthreads();
  uint64_t base = 0, total = 0;
  for (int i = 0; i < (int)(blockDim.x / kWave); ++i) {
    if (i < w) base += wsum[i];
    total += wsum[i];
  }
  *tot = total;
  return base + inc - v;
}

// Block b: the counts of keys [1024 b, 1024 b + 1024) -- one half of 1024
// words of every table -- into loc as prefix counts inside the group, and the
// group's sums.
__global__ __launch_bounds__(kGroup) void k_reduce16(const uint32_t* __restrict__ tables, int ntables,
                                                     const uint64_t* __restrict__ pk, uint64_t* __restrict__ adj_loc,
                                                     Group16* __restrict__ groups) {
  __shared__ uint64_t wsum[16], sq0[16], sq1[16];
  __shared__ int64_t ss[16];
  __shared__ uint32_t smn[16], smx[16];
  const uint32_t t = threadIdx.x, key = blockIdx.x * kGroup + t;
  const uint32_t i = key & (kWords - 1u), sh = key < kWords ? 16u : 0u;
  uint64_t c = adj_loc[key];
  if (tables) {
    int k = 0;
    for (; k + 16 <= ntables; k += 16) {
      uint32_t w[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) w[u] = tables[(size_t)(k + u) * kWords + i];
      uint32_t x = 0;
#pragma unroll
      for (int u = 0; u < 16; ++u) x += (w[u] >> sh) & 0xFFFFu;
      c += x;
    }
    for (; k < ntables; ++k) c += (tables[(size_t)k * kWords + i] >> sh) & 0xFFFFu;
  } else {
    c += sh ? pk[i] >> 32 : pk[i] & 0xFFFFFFFFull;
  }
  uint64_t tot;
  adj_loc[key] = block_prefix_u64(c, wsum, &tot);  // every thread read only its own entry
  const int64_t v = (int64_t)key - 32768;
  const Squares q = squares_of(v, c);
  const int64_t s = wave_sum_i64(v * (int64_t)c);
  const uint64_t q0 = wave_sum_u64(q.low), q1 = wave_sum_u64(q.high);
  const uint32_t mn = wave_min_u32(c ? key : 0xFFFFFFFFu), mx = wave_max_u32(c ? key : 0u);
  if (t % kWave == 0) {
    const uint32_t w = t / kWave;
    ss[w] = s;
    sq0[w] = q0;
    sq1[w] = q1;
    smn[w] = mn;
    smx[w] = mx;
  }
  __syncthreads();
  if (t == 0) {
    Group16 G{tot, {0, 0}, 0, 0xFFFFFFFFu, 0u, 0};
    for (int w = 0; w < 16; ++w) {
      G.s += ss[w];
      G.q.low += sq0[w];
      G.q.high += sq1[w];
      G.kmin = min(G.kmin, smn[w]);
      G.kmax = max(G.kmax, smx[w]);
    }
    G.q = carried(G.q);
    groups[blockIdx.x] = G;
  }
}

// What the histogram needs: the voxels below each group, and its range.
struct Fin16 {
  uint64_t base[kGroups + 1];
  float lo, scale;
  uint32_t kmin, kmax;
};

// Voxels whose key is below e (0 <= e <= 65536).
TSA_DEV uint64_t below_key(const uint64_t* loc, const uint64_t* base, uint32_t e) {
  return e >= kVals ? base[kGroups] : base[e / kGroup] + loc[e];
}

// Wave-wide: the smallest x in [0, n) with f(x) true (f is monotone and
// f(n - 1) holds), 64 probes a round.
template <class F>
TSA_DEV uint32_t wave_search(uint32_t n, F f) {
  const uint32_t lane = threadIdx.x % kWave;
  uint32_t lo = 0, hi = n - 1;  // the answer lies in [lo, hi]
  while (lo < hi) {
    const uint32_t step = (hi - lo + kWave - 1) / kWave;
    const uint32_t x = min(lo + lane * step, hi);
    const uint64_t yes = __ballot(f(x));
    if (yes == 0ull) {  // past the last probe
      lo = lo + (kWave - 1) * step + 1;
    } else {
      const uint32_t first = (uint32_t)__builtin_ctzll(yes);
      const uint32_t top = min(lo + first * step, hi);
      if (first) lo = lo + (first - 1) * step + 1;
      hi = top;
    }
  }
  return lo;
}

// x rounded once to double.
__host__ __device__ __forceinline__ double u128_to_f64(unsigned __int128 x) {
  const uint64_t hi = (uint64_t)(x >> 64);
  if (!hi) return (double)(uint64_t)x;
  const int sh = 64 - __builtin_clzll(hi);  // bits below the leading 64, kept as a sticky bit
  const uint64_t sticky = (uint64_t)x << (64 - sh) ? 1u : 0u;
  return ldexp((double)((uint64_t)(x >> sh) | sticky), sh);
}

// M2 of n voxels of sum S and sum of squares q: n Q - S^2 >= 0 in 128 bits
// (n <= 2^46, Q <= 2^76, |S| <= 2^61).
__host__ __device__ __forceinline__ double m2_of_sums(uint64_t n, int64_t S, const Squares& q) {
  const unsigned __int128 Q = ((unsigned __int128)q.high << 20) + q.low;
  return u128_to_f64(Q * n - (unsigned __int128)((__int128)S * S)) / (double)n;
}

// The scalar answers, by one wave.
__global__ __launch_bounds__(kWave) void k_fin16(const Group16* __restrict__ groups, const uint64_t* __restrict__ loc,
                                               Count16Ask ask, Fin16* __restrict__ fin) {
  __shared__ uint64_t base[kGroups + 1];
  static_assert(kGroups == kWave, "a lane per group");
  const uint32_t t = threadIdx.x;
  const Group16 g = groups[t];
  uint64_t inc = g.n;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint64_t y = __shfl_up(inc, o);
    if ((int)t >= o) inc += y;
  }
  base[t] = inc - g.n;
  if (t == kWave - 1) base[kGroups] = inc;
  const int64_t S = wave_sum_i64(g.s);
  const Squares q{wave_sum_u64(g.q.low), wave_sum_u64(g.q.high)};
  const uint32_t kmin = wave_min_u32(g.kmin), kmax = wave_max_u32(g.kmax);
  __syncthreads();
  const uint64_t n = __shfl(inc, kWave - 1);  // the region's volume: at least 1
  fin->base[t] = inc - g.n;
  const float lo = (float)((int32_t)kmin - 32768), hi = (float)((int32_t)kmax - 32768);
  if (t == 0) {
    fin->base[kGroups] = n;
    fin->kmin = kmin;
    fin->kmax = kmax;
    fin->lo = lo;
    fin->scale = lo == hi ? 0.0f : (float)ask.nbins / (hi - lo);
    if (ask.moments) {
      tsa_result* R = ask.out;
      R->count = n;
      R->nan_count = 0;
      R->min = (double)lo;
      R->max = (double)hi;
      R->status = TSA_OK;
      R->flags = 0;
      if (kmin == kmax) {
        R->mean = (double)lo;
        R->m2 = R->std = 0.0;
      } else {
        const double m2 = m2_of_sums(n, S, q);
        R->mean = (double)S / (double)n;
        R->m2 = m2;
        R->std = sqrt(m2 / (double)n);
      }
    }
  }
  uint64_t k;
  if (ask.rank == 2) {
    const double kk = floor(ask.q * (double)(n - 1));
    k = kk <= 0.0 ? 0 : kk >= (double)(n - 1) ? n - 1 : (uint64_t)kk;
  } else {
    k = (n - 1) / 2;
  }
  const uint32_t key = wave_search(kVals, [&](uint32_t e) { return below_key(loc, base, e + 1) > k; });
  if (ask.mad) {
    // deviations 0..65535 from the median: the smallest d whose interval holds more than k voxels
    const uint32_t d = wave_search(kVals, [&](uint32_t x) {
      const uint32_t e0 = x > key ? 0u : key - x, e1 = min(key + x + 1u, kVals);
      return below_key(loc, base, e1) - below_key(loc, base, e0) > k;
    });
    if (t == 0) {
      ask.qout[0] = (double)((int32_t)key - 32768);
      ask.qout[1] = (double)d;
      ask.qout[2] = (double)n;
    }
    return;
  }
  if (t != 0) return;
  if (ask.qout) {
    ask.qout[0] = (double)((int32_t)key - 32768);
    ask.qout[1] = 0.0;
    ask.qout[2] = (double)n;
  } else {
    ask.out->median = (double)((int32_t)key - 32768);
    if (ask.write_counts) {
      ask.out->count = n;
      ask.out->nan_count = 0;
      ask.out->status = TSA_OK;
    }
  }
}

// One lane per bin of the histogram over [min, max]: the bin formula is
// monotone in the value, so a bin is a run of keys, found by two binary
// searches of the formula itself.
__global__ __launch_bounds__(256) void k_bins16(const Fin16* __restrict__ fin, const uint64_t* __restrict__ loc,
                                                int32_t nbins, uint64_t* __restrict__ counts,
                                                uint64_t* __restrict__ outl) {
  const int32_t b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < 2) outl[b] = 0ull;
  if (b >= nbins) return;
  const float lo = fin->lo, scale = fin->scale;
  const uint32_t first = fin->kmin, end = fin->kmax + 1u;
  // the first key in [first, end) whose bin is at least x
  auto start = [&](int32_t x) {
    uint32_t a = first, z = end;
    while (a < z) {
      const uint32_t m = (a + z) >> 1;
      const float t = ((float)((int32_t)m - 32768) - lo) * scale;  // min == max: scale 0, bin 0
      if (min((int32_t)t, nbins - 1) >= x) z = m; else a = m + 1;
    }
    return a;
  };
  counts[b] = below_key(loc, fin->base, start(b + 1)) - below_key(loc, fin->base, start(b));
}

// Clears the words that the wraps and the packed counts are added to.
__global__ void k_clear16(uint64_t* __restrict__ p, uint32_t n) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0ull;
}

}  // namespace

// The least voxels of a region, by call, and of a block.  A block's counts
// leave it as up to 32768 additions to global memory (186 G/s over the chip:
// 45 us from 256 blocks of evenly spread values), so below 2^25 voxels fewer
// blocks of 2^17 voxels each are launched.  Ranks take this path from the size
// where it wins for every distribution tried (evenly spread, noise of 300 and of 3
// counts, one value); the others win at half their least sizes too.  us, key
// digits -> counts:
//   stats    2^24: spread 90 -> 58, noise 80 -> 38, one value 159 -> 40 (2^23: 69 -> 45, 61 -> 36, 97 -> 38)
//   MAD      2^23: spread 100 -> 35, noise 97 -> 25, one value 171 -> 30 (2^22: 80 -> 29, 76 -> 24, 117 -> 29)
//   median   2^27: spread 103 -> 100, noise 106 -> 59, one value 685 -> 74 (2^26: spread 69 -> 83)
// A quantile that stops after one digit stays with the digits: one pass either
// way, and the count is the longer one for spread values (2^27 voxels 57 -> 100, one
// value 236 -> 74; 2^29: spread 172 -> 192, noise 182 -> 192).
// The caller's-range histogram stays with its replicated bins: one pass either
// way (2^30 voxels, spread: 372 there, 352 here), and values that crowd on few
// words in random order are slow without replicas (two values: 699 there, 2054 here).
constexpr int64_t kCount16Stats = 1ll << 24, kCount16Mad = 1ll << 23, kCount16Rank = 1ll << 27;
constexpr int64_t kCount16Block = 1ll << 17;

size_t count16_scratch_bytes() { return 8 * ((size_t)kVals + kWords); }
size_t count16_small_bytes() { return sizeof(Group16) * kGroups + sizeof(Fin16); }

int count16_grid(int64_t volume, int blocks) {
  const int64_t most = (volume + kCount16Block - 1) / kCount16Block;
  return blocks < most ? blocks : (int)most;
}

// How the counts of a region of `volume` voxels leave the blocks: 1 in a
// table per block (grid * 128 KB of scratch), 2 added to 64-bit counters that
// hold two values each (their halves hold any count below 2^32), 0: the
// region is left to the passes by key digits.
int count16_mode(int64_t volume, int grid, size_t table_bytes, const Count16Ask& ask) {
  if (ask.rank == 2 && ask.digits == 1) return 0;
  if (volume < (ask.mad ? kCount16Mad : ask.moments ? kCount16Stats : kCount16Rank)) return 0;
  if ((size_t)grid * kWords * 4 <= table_bytes) return 1;
  return volume < (1ll << 32) ? 2 : 0;
}

int run_count16(const Geom& g, int vec, int grid, int mode, void* scratch, void* small, void* tables,
                const Count16Ask& ask, hipStream_t s) {
  uint64_t* adj = (uint64_t*)scratch;
  uint64_t* pk = adj + kVals;
  Group16* groups = (Group16*)small;
  Fin16* fin = (Fin16*)(groups + kGroups);
  uint32_t* tab = mode == 1 ? (uint32_t*)tables : nullptr;
  const uint32_t clear = mode == 1 ? kVals : kVals + kWords;
  TSA_TRACED("clear16", s, hipLaunchKernelGGL(k_clear16, dim3((clear + 255) / 256), dim3(256), 0, s, adj, clear));
#define TSA_COUNT16(V) \
  TSA_TRACED("count16", s, hipLaunchKernelGGL(k_count16<V>, dim3(grid), dim3(kCountThreads), 0, s, g, tab, pk, adj))
  if (vec == 1)
    TSA_COUNT16(1);
  else if (vec == 2)
    TSA_COUNT16(2);
  else
    TSA_COUNT16(0);
#undef TSA_COUNT16
  TSA_TRACED("reduce16", s,
             hipLaunchKernelGGL(k_reduce16, dim3(kGroups), dim3(kGroup), 0, s, (const uint32_t*)tab, grid,
                                (const uint64_t*)pk, adj, groups));
  TSA_TRACED("fin16", s,
             hipLaunchKernelGGL(k_fin16, dim3(1), dim3(kWave), 0, s, (const Group16*)groups, (const uint64_t*)adj, ask,
                                fin));
  if (ask.counts)
    TSA_TRACED("bins16", s,
               hipLaunchKernelGGL(k_bins16, dim3((ask.nbins + 255) / 256), dim3(256), 0, s, (const Fin16*)fin,
                                  (const uint64_t*)adj, ask.nbins, ask.counts, ask.outl));
  return hipGetLastError() == hipSuccess ? TSA_OK : TSA_EDEVICE;
}

}  // namespace tsa

// The moments the count gives, from the counts of the 65536 values (by key, value
// + 32768), summed on the host as the kernels sum them: a group of values at a
// time, then the groups.
extern "C" void tsa_internal_moments16(const uint64_t* counts, uint64_t* n, double* mean, double* m2) {
  using namespace tsa;
  uint64_t N = 0;
  int64_t S = 0;
  Squares q{0, 0};
  for (uint32_t g = 0; g < kGroups; ++g) {
    Squares gq{0, 0};
    for (uint32_t key = g * kGroup; key < (g + 1) * kGroup; ++key) {
      const int64_t v = (int64_t)key - 32768;
      const Squares x = squares_of(v, counts[key]);
      N += counts[key];
      S += v * (int64_t)counts[key];
      gq.low += x.low;
      gq.high += x.high;
    }
    gq = carried(gq);
    q.low += gq.low;
    q.high += gq.high;
  }
  *n = N;
  *mean = (double)S / (double)N;
  *m2 = m2_of_sums(N, S, q);
}
