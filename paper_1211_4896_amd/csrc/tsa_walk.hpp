// Visiting the voxels of a cube or of a box inside it, 16 bytes per lane.
//
// Two shapes of work:
//  * contiguous: the box is one run of memory (whole cube, whole planes, one
//    row).  Blocks stride over 16-byte vectors; U vector loads are issued per
//    lane before any is consumed, so each CU keeps many bytes in flight.  The
//    few elements before the first and after the last aligned vector are
//    visited one by one by block 0.
//  * rows: a general box is ly*lz rows of lx elements.  Rows are grouped into
//    tiles; a block flattens its tile's (row, vector) pairs so that narrow
//    boxes still fill every lane.
// How rows are read (the template parameter VEC):
//    1  aligned vectors: base and nx are multiples of the vector, so row starts
//       share one alignment offset and the first and last vector of every row
//       carry the same element masks;
//    2  vectors from the row's own first element, whatever its address; the
//       last one of a row is moved back to end with the row, and its elements
//       that the one before it held are masked.  No load leaves the row.
//       Rows narrower than a vector are read element by element.
//    0  elements: only for cubes not aligned to their own element size.
// 16-byte loads at any element boundary cost the extra line they may touch;
// element loads cost four times the instructions: the trio on a 1711x1711x246
// box of a 1721x1721x256 cube: 1.88 ms by elements, 1.07 ms by vectors.
//
// Slots without a voxel (masked elements, lanes past the end) reach a float32
// accumulator as NaN, which every one of them skips, with in_box true: no
// per-element lane masks.  int16 slots carry in_box false, or a clear bit where the
// accumulator takes a vector with a mask.
#pragma once

#include <type_traits>
#include <utility>

#include "tsa_device.hpp"

namespace tsa {

struct Geom {
  const void* base;
  int32_t mode;  // 0 contiguous, 1 rows
  int32_t pad0;
  // contiguous: vectors [v0, v1) plus single elements [h0, h1) and [t0, t1)
  int64_t v0, v1, h0, h1, t0, t1;
  // rows: units are vectors; origin and strides in vectors (VEC 1) or elements (VEC 0, 2)
  int64_t v_origin, v_ystride, v_zstride;
  uint32_t ly, nrows, vpr, rpt, ntiles;
  uint32_t head_skip, last_valid;
  uint32_t pad1;
  Magic ly_m, vpr_m;
};

// Rows [r0, r0 + nr) of a box (row r is y = r % ly, z = r / ly inside the
// box), flattened over (row, vector) so narrow rows still fill the lanes.
// Unit li (a vector, or an element on the scalar path) is column li % vpr of
// tile row li / vpr.  A lane finds its first U units with two divisions by
// invariant divisors, then steps every unit by bs*U units with constant
// increments and at most one carry per axis: no division and no 64-bit
// multiply inside the loop.
struct RowCursor {
  uint32_t j, ry, rz;  // column, y and z of the unit inside the box
  int64_t off;         // its index from the box origin, in units
};

// One whole vector: f.vec(uint4) where the accumulator has it, else its elements.
template <class F, class = void>
struct TakesVec : std::false_type {};
template <class F>
struct TakesVec<F, std::void_t<decltype(std::declval<F&>().vec(uint4{}))>> : std::true_type {};
template <int DT, class F>
TSA_DEV void visit_vec(const uint4& r, F& f) {
  if constexpr (TakesVec<F>::value) {
    f.vec(r);
  } else {
#pragma unroll
    for (int e = 0; e < Ty<DT>::EPV; ++e) f(Ty<DT>::get(r, e), true);
  }
}

// The vectors of a chunk: f.vecs where the accumulator has it, else one by one.
template <class F, int U, class = void>
struct TakesVecs : std::false_type {};
template <class F, int U>
struct TakesVecs<F, U, std::void_t<decltype(std::declval<F&>().vecs(std::declval<const uint4 (&)[U]>()))>>
    : std::true_type {};
template <int DT, int U, class F>
TSA_DEV void visit_vecs(const uint4 (&r)[U], F& f) {
  if constexpr (TakesVecs<F, U>::value) {
    f.vecs(r);
  } else {
#pragma unroll
    for (int u = 0; u < U; ++u) visit_vec<DT>(r[u], f);
  }
}

// Whether F takes int16 vectors with a bit for each element that is a voxel: one copy
// of its code then serves whole vectors and ends of rows (two copies: histogram of a
// 58x58x58 box 21.3 us against 18.7, of 1015x1013x503 369 against 332), another the
// whole and the last chunks of a cube (one mask for every vector there: 2048x2048x2048
// voxels 3.72 ms against 3.18).
template <class F, class = void>
struct TakesMask : std::false_type {};
template <class F>
struct TakesMask<F, std::void_t<decltype(std::declval<F&>().masked(uint4{}, 0u))>> : std::true_type {};

// What an empty slot holds.
constexpr uint32_t kNaNBits = 0x7FC00000u;
template <int DT>
TSA_DEV uint4 no_vec() {
  return DT == 0 ? make_uint4(kNaNBits, kNaNBits, kNaNBits, kNaNBits) : make_uint4(0u, 0u, 0u, 0u);
}
template <int DT>
TSA_DEV typename Ty<DT>::T no_elt() {
  if constexpr (DT == 0)
    return __uint_as_float(kNaNBits);
  else
    return (int16_t)0;
}

// 16 bytes from any element boundary.
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
template <int DT, bool NT>
TSA_DEV uint4 load16_any(const typename Ty<DT>::T* p) {
  const u32x4_any* q = (const u32x4_any*)p;
  u32x4 v;
  if constexpr (NT)
    v = __builtin_nontemporal_load(q);
  else
    v = *q;
  return make_uint4(v.x, v.y, v.z, v.w);
}
// The first n (1 to a vector's less one) elements from p.  float32: the rest empty.
// int16: any values past n; four and more by two loads of four that overlap
// in the row, two and three by two of two (an element a load: moments of
// 7x250x250 voxels 12.2 -> 10.4 us).
typedef uint64_t u64_any __attribute__((aligned(2)));
typedef uint32_t u32_any __attribute__((aligned(2)));
template <int DT>
TSA_DEV uint4 load_narrow(const typename Ty<DT>::T* p, uint32_t n) {
  uint4 r = no_vec<DT>();
  if constexpr (DT == 0) {
    if (n > 0) r.x = __float_as_uint(p[0]);
    if (n > 1) r.y = __float_as_uint(p[1]);
    if (n > 2) r.z = __float_as_uint(p[2]);
  } else if (n >= 4) {
    const uint64_t a = *(const u64_any*)p, b = *(const u64_any*)(p + (n - 4)) >> (16 * (8 - n) & 63);
    r = make_uint4((uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32));
  } else if (n >= 2) {
    r.x = *(const u32_any*)p;
    r.y = *(const u32_any*)(p + (n - 2)) >> (16 * (4 - n) & 31);
  } else {
    r.x = (uint32_t)(uint16_t)p[0];
  }
  return r;
}

// The elements of one vector of a row (column j of vpr): the first vector's
// first head_skip elements and what the last vector holds past last_valid (or,
// VEC 2, its first head_skip) are no voxels of the row; ok false: none is.
template <int DT, int VEC, class F>
TSA_DEV void visit_row_vec(uint4 r, uint32_t j, uint32_t vpr, uint32_t head_skip, uint32_t last_valid, bool ok,
                           F& f) {
  using TT = Ty<DT>;
  const bool first = j == 0, last = j == vpr - 1;
  const bool skips = VEC == 2 ? last : first;  // where head_skip applies
  if constexpr (DT == 0) {
    // empty slots hold NaN already; the whole wave passes where no lane is at an end of a row
    if (__ballot(VEC == 2 ? skips && head_skip != 0u : (first && head_skip != 0u) || (last && last_valid < 4u))) {
      uint32_t* w[4] = {&r.x, &r.y, &r.z, &r.w};
#pragma unroll
      for (uint32_t e = 0; e < 4; ++e) {
        if (e < 3 && skips && e < head_skip) *w[e] = kNaNBits;
        if (VEC == 1 && e > 0 && last && e >= last_valid) *w[e] = kNaNBits;
      }
    }
    visit_vec<DT>(r, f);
  } else if constexpr (TakesMask<F>::value) {
    uint32_t mask = ok ? 0xFFu : 0u;
    if (skips) mask &= 0xFFu << head_skip;
    if (last) mask &= 0xFFu >> (8u - last_valid);
    f.masked(r, mask);
  } else if (__ballot(!ok || (skips && head_skip != 0u) || (last && last_valid < (uint32_t)TT::EPV)) == 0ull) {
    visit_vec<DT>(r, f);
  } else {
#pragma unroll
    for (int e = 0; e < TT::EPV; ++e)
      f(TT::get(r, e), ok && (!skips || (uint32_t)e >= head_skip) && (!last || (uint32_t)e < last_valid));
  }
}

template <int DT, int VEC, int U, bool NT, class F>
TSA_DEV void walk_rows(const void* base, int64_t v_origin, int64_t v_ystride, int64_t v_zstride, uint32_t ly,
                       const Magic& ly_m, uint32_t vpr, const Magic& vpr_m, uint32_t head_skip, uint32_t last_valid,
                       uint32_t r0, uint32_t nr, F& f) {
  using TT = Ty<DT>;
  using T = typename TT::T;
  constexpr uint32_t C = VEC == 2 ? TT::EPV : 1;  // index units of a column
  const uint32_t bs = blockDim.x;
  const uint32_t cnt = nr * vpr;
  if (cnt == 0) return;
  // the step of bs*U units as (rows, columns), the rows as (planes, y)
  const uint32_t step = bs * U;
  const uint32_t dq = mdiv(step, vpr_m), dr = step - dq * vpr;
  const uint32_t dqz = mdiv(dq, ly_m), dqy = dq - dqz * ly;
  const int64_t dstep = (int64_t)dqz * v_zstride + (int64_t)dqy * v_ystride + dr * C;
  RowCursor c[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t li = u * bs + threadIdx.x;
    const uint32_t lr = mdiv(li, vpr_m);
    c[u].j = li - lr * vpr;
    const uint32_t row = r0 + lr;
    c[u].rz = mdiv(row, ly_m);
    c[u].ry = row - c[u].rz * ly;
    c[u].off = (int64_t)c[u].rz * v_zstride + (int64_t)c[u].ry * v_ystride + (int64_t)c[u].j * C;
  }
  const uint4* vb = (const uint4*)base + v_origin;
  const T* sb = (const T*)base + v_origin;
  const bool narrow = VEC == 2 && last_valid < (uint32_t)TT::EPV;
  auto load = [&](const RowCursor& k) -> uint4 {
    if constexpr (VEC == 1) {
      return load16<NT>(vb + k.off);
    } else {
      if (narrow) return load_narrow<DT>(sb + k.off, last_valid);
      return load16_any<DT, NT>(sb + k.off - (k.j == vpr - 1 ? head_skip : 0u));
    }
  };
  for (uint32_t li0 = 0; li0 < cnt; li0 += step) {
    // a full step needs no test per unit; in the last, partial one units past
    // the tile load nothing, so every lane still calls f at the same points
    const bool full = li0 + step <= cnt;
    bool ok[U];
    if constexpr (VEC != 0) {
      uint4 r[U];
      if (full) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          ok[u] = true;
          r[u] = load(c[u]);
        }
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          ok[u] = li0 + u * bs + threadIdx.x < cnt;
          r[u] = no_vec<DT>();
          if (ok[u]) r[u] = load(c[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        visit_row_vec<DT, VEC>(r[u], c[u].j, vpr, head_skip, last_valid, ok[u], f);
    } else {
      T v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        ok[u] = full || li0 + u * bs + threadIdx.x < cnt;
        v[u] = no_elt<DT>();
        if (ok[u]) v[u] = sb[c[u].off];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) f(v[u], DT == 0 || ok[u]);
    }
    // advance every cursor by step units
#pragma unroll
    for (int u = 0; u < U; ++u) {
      RowCursor& k = c[u];
      k.j += dr;
      k.ry += dqy;
      k.rz += dqz;
      k.off += dstep;
      if (k.j >= vpr) {  // carry from the column into the row
        k.j -= vpr;
        k.ry += 1;
        k.off += v_ystride - (int64_t)(vpr * C);
      }
      if (k.ry >= ly) {  // carry from y into z (ry < 2 ly here)
        k.ry -= ly;
        k.rz += 1;
        k.off += v_zstride - (int64_t)ly * v_ystride;
      }
    }
    f.chunk();
  }
}

// f(T value, bool in_box) is called once per element slot (see above for
// slots without a voxel), or f.vec(uint4), f.masked(uint4, bits) once per vector or
// f.vecs once per chunk where f has them.  Every lane of the block calls f at the same points (never from
// divergent code), so f may use wave-wide operations that need every lane.
// f.chunk() is called by every thread of the block at the same points, after
// at most blockDim.x * U vectors have been visited since the previous call,
// so it may synchronise the block.
// The contiguous geometry: AHEAD: the next chunk's loads are issued before
// the present one is consumed, so a wave's processing never leaves it without
// loads in flight (U more vectors of registers).
template <int DT, int VEC, int U, bool NT, bool AHEAD = false, class F>
TSA_DEV void walk_run(const Geom& g, F& f) {
  using TT = Ty<DT>;
  using T = typename TT::T;
  const T* sb = (const T*)g.base;
  const int64_t bs = blockDim.x;
  if constexpr (VEC != 0) {
    const uint4* vb = (const uint4*)g.base;
    const int64_t chunk = bs * U;
    const int64_t stride = chunk * gridDim.x;
    auto load = [&](int64_t cb, uint4(&r)[U]) {
      const int64_t i = cb + threadIdx.x;
      if (cb + chunk <= g.v1) {
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] = load16<NT>(vb + i + u * bs);
      } else {  // the last, partial chunk of a block
#pragma unroll
        for (int u = 0; u < U; ++u) {
          r[u] = no_vec<DT>();
          if (i + u * bs < g.v1) r[u] = load16<NT>(vb + i + u * bs);
        }
      }
    };
    auto consume = [&](int64_t cb, const uint4(&r)[U]) {
      if (DT == 0 || cb + chunk <= g.v1) {
        visit_vecs<DT>(r, f);
      } else if constexpr (TakesMask<F>::value) {
#pragma unroll
        for (int u = 0; u < U; ++u) f.masked(r[u], cb + threadIdx.x + u * bs < g.v1 ? 0xFFu : 0u);
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int e = 0; e < TT::EPV; ++e) f(TT::get(r[u], e), cb + threadIdx.x + u * bs < g.v1);
      }
      f.chunk();
    };
    int64_t cb = g.v0 + (int64_t)blockIdx.x * chunk;
    uint4 r[U];
    if constexpr (AHEAD) {
      if (cb < g.v1) {
        load(cb, r);
        for (;;) {
          const int64_t nb = cb + stride;
          uint4 n[U];
          if (nb < g.v1) load(nb, n);
          consume(cb, r);
          if (nb >= g.v1) break;
#pragma unroll
          for (int u = 0; u < U; ++u) r[u] = n[u];
          cb = nb;
        }
      }
    } else {
      for (; cb < g.v1; cb += stride) {
        load(cb, r);
        consume(cb, r);
      }
    }
    // the elements outside the vectors: fewer than two vectors' worth
    if (blockIdx.x == 0) {
      const int64_t nh = g.h1 - g.h0, t = threadIdx.x, e = t < nh ? g.h0 + t : g.t0 + (t - nh);
      const bool ok = e < (t < nh ? g.h1 : g.t1);
      T v = no_elt<DT>();
      if (ok) v = sb[e];
      f(v, DT == 0 || ok);
    }
  } else {
    const int64_t chunk = bs * U;
    const int64_t stride = chunk * gridDim.x;
    for (int64_t cb = g.v0 + (int64_t)blockIdx.x * chunk; cb < g.v1; cb += stride) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t j = cb + u * bs + threadIdx.x;
        const bool ok = j < g.v1;
        T v = no_elt<DT>();
        if (ok) v = sb[j];
        f(v, DT == 0 || ok);
      }
      f.chunk();
    }
  }
}
// The tiles of a box.
template <int DT, int VEC, int U, bool NT, class F>
TSA_DEV void walk_tiles(const Geom& g, F& f) {
  for (uint32_t t = blockIdx.x; t < g.ntiles; t += gridDim.x) {
    const uint32_t r0 = t * g.rpt;
    walk_rows<DT, VEC, U, NT>(g.base, g.v_origin, g.v_ystride, g.v_zstride, g.ly, g.ly_m, g.vpr, g.vpr_m,
                              g.head_skip, g.last_valid, r0, min(g.rpt, g.nrows - r0), f);
  }
}
// Either, by the geometry.
template <int DT, int VEC, int U, bool NT, bool AHEAD = false, class F>
TSA_DEV void walk(const Geom& g, F& f) {
  if (g.mode == 0)
    walk_run<DT, VEC, U, NT, AHEAD>(g, f);
  else
    walk_tiles<DT, VEC, U, NT>(g, f);
}

}  // namespace tsa
