// HIP kernels for gfx950 (CDNA4): the rectangle mover used by the pack,
// unpack-transform and direct paths, and the grid-overlay volume kernel.
//
// All of them are bound by HBM bandwidth: per element they read at most two
// values and write one, with at most a few flops (Section 5 eq:costa).  The
// movers are therefore built from one-shot workgroups: each takes one task
// from the plan's task table -- 256 or 512 consecutive 16-byte units (or
// elements) of a rectangle walked along its rows, four wave tasks of a stack
// of short rectangles that follow one another along a local column, or one
// LDS tile of a rectangle whose source and destination run in different
// directions -- moves it with coalesced 64-lane accesses and exits, so the
// workgroups in flight sweep the buffers in task order.  A launch whose
// tasks are all alike may hand each XCD (one L2) a contiguous range of them.
#include <hip/hip_runtime.h>

#include <cstring>
#include <type_traits>

#include "index_math.hpp"

// Products and sums are rounded one by one, never fused into an FMA, so the
// results are reproducible bit for bit.
#pragma clang fp contract(off)

namespace costa {
namespace {

// Tuning switches (compile-time; the defaults are the measured best).
#ifndef COSTA_NT_LOADS
#define COSTA_NT_LOADS 1  // row walks: each source line is read once
#endif
#ifndef COSTA_NT_LOADS_MAX_ES
#define COSTA_NT_LOADS_MAX_ES 8  // ...for element sizes up to this (measured: helps fp64, hurts complex128)
#endif
#ifndef COSTA_NT_STORES
#define COSTA_NT_STORES 1
#endif
#ifndef COSTA_NT_ALOADS
#define COSTA_NT_ALOADS 0  // loads of A in row walks (measured: 1 makes the scaled transpose's unpack 29% slower)
#endif
// Runs (bytes) from which a tile's loads are non-temporal although its runs
// end inside 128-byte lines that a neighbouring tile reads too; below it such
// tiles use plain loads, and the neighbour finds the line in L2 or in the
// Infinity Cache.  Measured on MI355X, plain against non-temporal:
//   source columns of 12 floats 251 against 412 us, 22 floats 236 - 318, 22
//   doubles 173 - 206, 59 floats 141 - 150, 32 doubles (pdtran) 830 - 858, 59
//   doubles 131 - 129; whole lines (32 and 48 doubles) 121 - 111;
//   rows of A (in launches that hand an XCD runs of tiles) 22 floats
//   247 - 277, 22 doubles 221 - 231, 59 doubles 199 - 181; whole lines
//   189 - 159.
constexpr int kShortTileColumn = 384, kShortTileRow = 256;

constexpr int kThreads = kThreadsPerTask;

template <typename S, int N>
struct alignas(sizeof(S) * N) Vec {
  S v[N];
};

// Raw integer vector of a given size, for loads and stores with an optional
// non-temporal hint (streaming data that is touched exactly once).
template <int BYTES>
struct Raw;
template <>
struct Raw<4> {
  using T = uint32_t;
};
template <>
struct Raw<8> {
  typedef uint32_t T __attribute__((ext_vector_type(2)));
};
template <>
struct Raw<16> {
  typedef uint32_t T __attribute__((ext_vector_type(4)));
};

// The buffers reach the kernels through a pointer table, so the compiler
// cannot see that they are global memory; the casts below make it emit global
// (not flat) loads and stores, which do not share a wait counter with LDS.
#define COSTA_GLOBAL __attribute__((address_space(1)))

// The call's table (CallTable), read with scalar loads from the kernel's own
// arguments (ArgTable is the first parameter of every mover, so it starts the
// argument segment) or from device memory; `device` is the same for every
// lane.
#define COSTA_CONST __attribute__((address_space(4)))
using Bufs = void* const COSTA_CONST*;
using Items = const ItemParam COSTA_CONST*;
__device__ __forceinline__ const char COSTA_CONST* call_table(const void* device) {
  return device ? (const char COSTA_CONST*)device : (const char COSTA_CONST*)__builtin_amdgcn_kernarg_segment_ptr();
}

template <bool NT = COSTA_NT_LOADS, typename U>
__device__ __forceinline__ U load(const U* p) {
  using R = typename Raw<sizeof(U)>::T;
  const COSTA_GLOBAL R* g = (const COSTA_GLOBAL R*)(p);
  R r;
  if constexpr (NT) r = __builtin_nontemporal_load(g);
  else r = *g;
  U u;
  __builtin_memcpy(&u, &r, sizeof(U));
  return u;
}

template <typename U>
__device__ __forceinline__ void store(U* p, const U& u) {
  using R = typename Raw<sizeof(U)>::T;
  COSTA_GLOBAL R* g = (COSTA_GLOBAL R*)(p);
  R r;
  __builtin_memcpy(&r, &u, sizeof(U));
  if constexpr (COSTA_NT_STORES) __builtin_nontemporal_store(r, g);
  else *g = r;
}

// Element arithmetic for a vector of NU scalars (pairs of them for complex).
template <typename S, int NU, bool CPLX, int MODE, bool CONJ>
__device__ __forceinline__ Vec<S, NU> combine(const Vec<S, NU>& b, const Vec<S, NU>& a, S ar, S ai, S br, S bi) {
  Vec<S, NU> o;
  if constexpr (CPLX) {
#pragma unroll
    for (int k = 0; k < NU; k += 2) {
      const S xr = b.v[k];
      const S xi = CONJ ? -b.v[k + 1] : b.v[k + 1];
      if constexpr (MODE == MODE_COPY) {
        o.v[k] = xr;
        o.v[k + 1] = xi;
      } else {
        const S p1 = ar * xr, p2 = ai * xi, p3 = ar * xi, p4 = ai * xr;
        S t1r = p1 - p2, t1i = p3 + p4;
        if constexpr (MODE == MODE_AXPBY) {
          const S q1 = br * a.v[k], q2 = bi * a.v[k + 1], q3 = br * a.v[k + 1], q4 = bi * a.v[k];
          const S t2r = q1 - q2, t2i = q3 + q4;
          t1r = t1r + t2r;
          t1i = t1i + t2i;
        }
        o.v[k] = t1r;
        o.v[k + 1] = t1i;
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < NU; ++k) {
      if constexpr (MODE == MODE_COPY) {
        o.v[k] = b.v[k];
      } else if constexpr (MODE == MODE_SCALE) {
        o.v[k] = ar * b.v[k];
      } else {
        const S t1 = ar * b.v[k];
        const S t2 = br * a.v[k];
        o.v[k] = t1 + t2;
      }
    }
  }
  return o;
}

template <typename S, bool CPLX>
struct TypeTraits {
  static constexpr int NS = CPLX ? 2 : 1;         // scalars per element
  static constexpr int ES = (int)sizeof(S) * NS;  // bytes per element
  static constexpr int WIDE_NEL = wide_elems(ES); // elements per 16-byte unit
  static constexpr bool NT_WALK = COSTA_NT_LOADS && ES <= COSTA_NT_LOADS_MAX_ES;
};

// Row walk: dst[y*dst_ld + x] = f(src[y*src_ld + x]).  The task starts at
// unit u0 of rectangle pi (a unit is a 16-byte vector for PIECE_WIDE
// rectangles, else one element; the flattened (y, x) index of a rectangle
// numbers its units) and covers the next UL*kThreads units: lane l takes
// units u0 + l + k*kThreads, k < UL.  A run of small rectangles
// (PIECE_GROUP_NEXT) is flattened the same way, its units one rectangle after
// another.  A lane issues all its loads (and those of A when it is read)
// before its stores.
template <typename S, bool CPLX, int MODE, bool CONJ, int UL>
__device__ __forceinline__ void move_walk(const Piece* __restrict__ pieces, int32_t pi, int32_t u0,
                                          Bufs bufs, int32_t allow_wide, S ar, S ai, S br,
                                          S bi) {
  using TT = TypeTraits<S, CPLX>;
  using E = Vec<S, TT::NS>;
  constexpr int W = TT::WIDE_NEL;
  const Piece& p0 = pieces[pi];
  const bool wide = (p0.flags & PIECE_WIDE) != 0;  // the same over a run
  const int32_t epu = wide ? W : 1;                // elements per unit
  const S* __restrict__ srcs[UL];
  S* __restrict__ dsts[UL];
  int64_t soffs[UL], doffs[UL];
  const int32_t nxu0 = wide ? p0.nx / W : p0.nx;
  const int32_t units0 = nxu0 * p0.ny;
  if (u0 + UL * kThreads <= units0) {
    // the whole task lies in rectangle pi: its fields are the same for every lane
    const S* src = reinterpret_cast<const S*>(bufs[p0.src_buf]);
    S* dst = reinterpret_cast<S*>(bufs[p0.dst_buf]);
#pragma unroll
    for (int k = 0; k < UL; ++k) {
      int32_t y, x;
      divmod(u0 + k * kThreads + (int32_t)threadIdx.x, nxu0, y, x);
      soffs[k] = p0.src_off + (int64_t)y * p0.src_ld + (int64_t)x * epu;
      doffs[k] = p0.dst_off + (int64_t)y * p0.dst_ld + (int64_t)x * epu;
      srcs[k] = src;
      dsts[k] = dst;
    }
  } else {
    // the task runs past the end of rectangle pi (into the next ones of a
    // run of small rectangles, or past the rectangle's end): walk the
    // rectangles it spans one by one, the same for every lane, each lane
    // keeping the one that holds its unit
    int32_t uu[UL];
#pragma unroll
    for (int k = 0; k < UL; ++k) {
      uu[k] = u0 + k * kThreads + (int32_t)threadIdx.x;
      soffs[k] = -1;
      doffs[k] = 0;
      srcs[k] = nullptr;
      dsts[k] = nullptr;
    }
    int32_t q = pi;
    int32_t rem = u0 + UL * kThreads;  // units of the task at or past rectangle q
    while (true) {
      const Piece& p = pieces[q];
      const int32_t nxu = wide ? p.nx / W : p.nx;
      const int32_t units = nxu * p.ny;
#pragma unroll
      for (int k = 0; k < UL; ++k) {
        if (uu[k] >= 0 && uu[k] < units) {
          int32_t y, x;
          divmod(uu[k], nxu, y, x);
          soffs[k] = p.src_off + (int64_t)y * p.src_ld + (int64_t)x * epu;
          doffs[k] = p.dst_off + (int64_t)y * p.dst_ld + (int64_t)x * epu;
          srcs[k] = reinterpret_cast<const S*>(bufs[p.src_buf]);
          dsts[k] = reinterpret_cast<S*>(bufs[p.dst_buf]);
        }
        uu[k] -= units;
      }
      rem -= units;
      if (rem <= 0 || !(p.flags & PIECE_GROUP_NEXT)) break;
      ++q;
    }
  }
  if (W > 1 && wide && allow_wide) {
    using U = Vec<S, TT::NS * W>;
    U bv[UL], av[UL];
#pragma unroll
    for (int k = 0; k < UL; ++k)
      if (soffs[k] >= 0) {
        bv[k] = load<TT::NT_WALK>(reinterpret_cast<const U*>(srcs[k] + soffs[k] * TT::NS));
        if constexpr (MODE == MODE_AXPBY) av[k] = load<COSTA_NT_ALOADS>(reinterpret_cast<U*>(dsts[k] + doffs[k] * TT::NS));
      }
#pragma unroll
    for (int k = 0; k < UL; ++k)
      if (soffs[k] >= 0)
        store(reinterpret_cast<U*>(dsts[k] + doffs[k] * TT::NS),
              combine<S, TT::NS * W, CPLX, MODE, CONJ>(bv[k], av[k], ar, ai, br, bi));
  } else {
    // one element at a time (epu of them: a PIECE_WIDE rectangle in a call
    // whose buffers are not 16-byte aligned)
    E bv[UL][W], av[UL][W];
#pragma unroll
    for (int k = 0; k < UL; ++k)
      if (soffs[k] >= 0) {
        const E* se = reinterpret_cast<const E*>(srcs[k]) + soffs[k];
        E* de = reinterpret_cast<E*>(dsts[k]) + doffs[k];
#pragma unroll
        for (int j = 0; j < W; ++j)
          if (j < epu) {
            bv[k][j] = load<TT::NT_WALK>(se + j);
            if constexpr (MODE == MODE_AXPBY) av[k][j] = load<COSTA_NT_ALOADS>(de + j);
          }
      }
#pragma unroll
    for (int k = 0; k < UL; ++k)
      if (soffs[k] >= 0) {
        E* de = reinterpret_cast<E*>(dsts[k]) + doffs[k];
#pragma unroll
        for (int j = 0; j < W; ++j)
          if (j < epu) store(de + j, combine<S, TT::NS, CPLX, MODE, CONJ>(bv[k][j], av[k][j], ar, ai, br, bi));
      }
  }
}

// The same row walk, with each lane finding its rectangle of a run on its
// own (the rectangle's fields and buffer pointers then live in vector
// registers).  Used for 16-byte elements: measured on MI355X, the complex128
// pack of the COSMA-like case runs 9% faster this way than with the
// walk above, while the 8-byte and smaller walks of short rows run 3-5%
// slower.  Task c of the rectangle covers units [c*UL*kThreads,
// (c+1)*UL*kThreads) of its flattened (y, x) index.
template <typename S, bool CPLX, int MODE, bool CONJ, int UL>
__device__ __forceinline__ void move_walk_lanes(const Piece* __restrict__ pieces, int32_t pi, int32_t c,
                                          Bufs bufs, int32_t allow_wide, S ar, S ai, S br,
                                          S bi) {
  using TT = TypeTraits<S, CPLX>;
  using E = Vec<S, TT::NS>;
  constexpr int W = TT::WIDE_NEL;
  const bool wide = (pieces[pi].flags & PIECE_WIDE) != 0;  // the same over a run
  const int32_t epu = wide ? W : 1;                         // elements per unit
  const S* __restrict__ srcs[UL];
  S* __restrict__ dsts[UL];
  int64_t soffs[UL], doffs[UL];
#pragma unroll
  for (int k = 0; k < UL; ++k) {
    int32_t u = c * (UL * kThreads) + k * kThreads + (int32_t)threadIdx.x;
    int64_t soff = -1, doff = 0;
    int32_t sbuf = 0, dbuf = 0;
    int32_t q = pi;
    while (true) {
      const Piece& p = pieces[q];
      const int32_t nxu = wide ? p.nx / W : p.nx;
      const int32_t units = nxu * p.ny;
      if (u >= 0 && u < units) {
        int32_t y, x;
        divmod(u, nxu, y, x);
        soff = p.src_off + (int64_t)y * p.src_ld + (int64_t)x * epu;
        doff = p.dst_off + (int64_t)y * p.dst_ld + (int64_t)x * epu;
        sbuf = p.src_buf;
        dbuf = p.dst_buf;
      }
      u -= units;
      if (!(p.flags & PIECE_GROUP_NEXT)) break;
      ++q;
    }
    soffs[k] = soff;
    doffs[k] = doff;
    srcs[k] = reinterpret_cast<const S*>(bufs[sbuf]);
    dsts[k] = reinterpret_cast<S*>(bufs[dbuf]);
  }
  if (W > 1 && wide && allow_wide) {
    using U = Vec<S, TT::NS * W>;
    U bv[UL], av[UL];
#pragma unroll
    for (int k = 0; k < UL; ++k)
      if (soffs[k] >= 0) {
        bv[k] = load<TT::NT_WALK>(reinterpret_cast<const U*>(srcs[k] + soffs[k] * TT::NS));
        if constexpr (MODE == MODE_AXPBY) av[k] = load<COSTA_NT_ALOADS>(reinterpret_cast<U*>(dsts[k] + doffs[k] * TT::NS));
      }
#pragma unroll
    for (int k = 0; k < UL; ++k)
      if (soffs[k] >= 0)
        store(reinterpret_cast<U*>(dsts[k] + doffs[k] * TT::NS),
              combine<S, TT::NS * W, CPLX, MODE, CONJ>(bv[k], av[k], ar, ai, br, bi));
  } else {
    // one element at a time (epu of them: a PIECE_WIDE rectangle in a call
    // whose buffers are not 16-byte aligned)
    E bv[UL][W], av[UL][W];
#pragma unroll
    for (int k = 0; k < UL; ++k)
      if (soffs[k] >= 0) {
        const E* se = reinterpret_cast<const E*>(srcs[k]) + soffs[k];
        E* de = reinterpret_cast<E*>(dsts[k]) + doffs[k];
#pragma unroll
        for (int j = 0; j < W; ++j)
          if (j < epu) {
            bv[k][j] = load<TT::NT_WALK>(se + j);
            if constexpr (MODE == MODE_AXPBY) av[k][j] = load<COSTA_NT_ALOADS>(de + j);
          }
      }
#pragma unroll
    for (int k = 0; k < UL; ++k)
      if (soffs[k] >= 0) {
        E* de = reinterpret_cast<E*>(dsts[k]) + doffs[k];
#pragma unroll
        for (int j = 0; j < W; ++j)
          if (j < epu) store(de + j, combine<S, TT::NS, CPLX, MODE, CONJ>(bv[k][j], av[k][j], ar, ai, br, bi));
      }
  }
}

// Stack walk (PIECE_STACK): the rectangles of a stack follow one another
// along x on one side, so the stack is walked as one band of hu units per y,
// in wave tasks of 64 units by kStackRows rows: wave v of task c takes wave
// task t = 4c + v, units [64 * (t % wb), +64) of x -- one per lane, the same
// for every row -- and rows [kStackRows * (t / wb), +kStackRows) of y.  The
// wave finds once which rectangle holds each lane's unit (a binary search for
// the last rectangle that starts at or before its first unit, then a scan
// over those that start before its last), then moves its rows with up to
// kStackRowsInFlight loads in flight per lane.  Every 64-lane access is
// contiguous on the stacked side, wherever the rectangles' edges fall in a
// 128-byte line.
#ifndef COSTA_STACK_ROWS_IN_FLIGHT
#define COSTA_STACK_ROWS_IN_FLIGHT 4
#endif
constexpr int kStackRowsInFlight = COSTA_STACK_ROWS_IN_FLIGHT;

template <typename S, bool CPLX, int MODE, bool CONJ>
__device__ __forceinline__ void move_stack(const Piece* __restrict__ pieces, int32_t pi, int32_t c,
                                           Bufs bufs, int32_t allow_wide, S ar, S ai, S br,
                                           S bi) {
  using TT = TypeTraits<S, CPLX>;
  using E = Vec<S, TT::NS>;
  constexpr int W = TT::WIDE_NEL;
  constexpr int YU = kStackRowsInFlight;
  static_assert(MODE != MODE_AXPBY, "stacks hold no rectangles of pairs that read A");
  const Piece& h = pieces[pi];
  const int32_t np = stack_size_of(h.flags);
  const bool on_dst = (h.flags & PIECE_STACK_DST) != 0;
  const bool wide = (h.flags & PIECE_WIDE) != 0;
  const int32_t epu = wide ? W : 1;  // elements per unit
  const Piece& last = pieces[pi + np - 1];
  const int64_t base = on_dst ? h.dst_off : h.src_off;
  const int32_t hu = (int32_t)(((on_dst ? last.dst_off : last.src_off) + last.nx - base) / epu);
  const int32_t wb = (hu + kStackWave - 1) / kStackWave;
  const int32_t nt = wb * ((h.ny + kStackRows - 1) / kStackRows);
  // this wave's task (wave-uniform)
  const int32_t t = c * (kThreads / kStackWave) + __builtin_amdgcn_readfirstlane((int32_t)threadIdx.x / kStackWave);
  if (t >= nt) return;  // past the stack's last wave task (no barrier follows)
  int32_t chunk, band;
  divmod(t, wb, chunk, band);
  const int32_t w0 = band * kStackWave;
  const int32_t xu = w0 + (int32_t)(threadIdx.x % kStackWave);
  const int64_t x = (int64_t)xu * epu;  // this lane's element offset along the stack
  const int64_t xw0 = (int64_t)w0 * epu;
  const int64_t xw1 = (int64_t)min(w0 + kStackWave, hu) * epu;
  // the last rectangle that starts at or before the wave's first unit
  int32_t lo = 0, hi = np - 1;
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    const Piece& m = pieces[pi + mid];
    if ((on_dst ? m.dst_off : m.src_off) - base <= xw0) lo = mid;
    else hi = mid - 1;
  }
  int64_t soff = 0, doff = 0, sld = 0, dld = 0;
  int32_t sbuf = 0, dbuf = 0;
  for (int32_t k = lo; k < np; ++k) {
    const Piece& p = pieces[pi + k];
    const int64_t s0 = (on_dst ? p.dst_off : p.src_off) - base;
    if (s0 >= xw1) break;
    if (x >= s0 && x < s0 + p.nx) {
      soff = p.src_off + (x - s0);
      doff = p.dst_off + (x - s0);
      sld = p.src_ld;
      dld = p.dst_ld;
      sbuf = p.src_buf;
      dbuf = p.dst_buf;
    }
  }
  if (xu >= hu) return;
  const int32_t y0 = chunk * kStackRows;
  const int32_t y1 = min(y0 + kStackRows, h.ny);
  const S* sb = reinterpret_cast<const S*>(bufs[sbuf]) + (soff + (int64_t)y0 * sld) * TT::NS;
  S* db = reinterpret_cast<S*>(bufs[dbuf]) + (doff + (int64_t)y0 * dld) * TT::NS;
  const int64_t ss = sld * TT::NS, ds = dld * TT::NS;  // row strides in scalars
  int32_t y = y0;
  if (W > 1 && wide && allow_wide) {
    using U = Vec<S, TT::NS * W>;
    for (; y + YU <= y1; y += YU) {
      U bv[YU];
#pragma unroll
      for (int k = 0; k < YU; ++k) bv[k] = load<TT::NT_WALK>(reinterpret_cast<const U*>(sb + k * ss));
#pragma unroll
      for (int k = 0; k < YU; ++k)
        store(reinterpret_cast<U*>(db + k * ds), combine<S, TT::NS * W, CPLX, MODE, CONJ>(bv[k], bv[k], ar, ai, br, bi));
      sb += YU * ss;
      db += YU * ds;
    }
    for (; y < y1; ++y) {
      const U bv = load<TT::NT_WALK>(reinterpret_cast<const U*>(sb));
      store(reinterpret_cast<U*>(db), combine<S, TT::NS * W, CPLX, MODE, CONJ>(bv, bv, ar, ai, br, bi));
      sb += ss;
      db += ds;
    }
  } else {
    // one element at a time (epu of them: a PIECE_WIDE stack in a call whose
    // buffers are not 16-byte aligned)
    const E* se = reinterpret_cast<const E*>(sb);
    E* de = reinterpret_cast<E*>(db);
    for (; y + YU <= y1; y += YU) {
      E bv[YU][W];
#pragma unroll
      for (int k = 0; k < YU; ++k)
#pragma unroll
        for (int j = 0; j < W; ++j)
          if (j < epu) bv[k][j] = load<TT::NT_WALK>(se + k * sld + j);
#pragma unroll
      for (int k = 0; k < YU; ++k)
#pragma unroll
        for (int j = 0; j < W; ++j)
          if (j < epu)
            store(de + k * dld + j, combine<S, TT::NS, CPLX, MODE, CONJ>(bv[k][j], bv[k][j], ar, ai, br, bi));
      se += YU * sld;
      de += YU * dld;
    }
    for (; y < y1; ++y) {
#pragma unroll
      for (int j = 0; j < W; ++j)
        if (j < epu) {
          const E bv = load<TT::NT_WALK>(se + j);
          store(de + j, combine<S, TT::NS, CPLX, MODE, CONJ>(bv, bv, ar, ai, br, bi));
        }
      se += sld;
      de += dld;
    }
  }
}

// One LDS tile of a rectangle whose source runs along y while the
// destination runs along x: tile c (tiles numbered along x first) of
// tile_x x tile_y elements, cut at the rectangle's edges to w x h.  Loads
// take the tile's elements in source order (y fastest: runs of h elements),
// stores in destination order (x fastest: runs of w elements); lanes walk
// the flattened tile, so every lane has work whatever its shape.  In LDS
// element (x, y) sits at x * (tile_y | 1) + y.  When A is read (beta != 0)
// its elements are loaded together with the source, before the barrier:
// loads issued between the stores could not be moved ahead of them (the
// compiler cannot tell that they touch other elements) and would each wait
// for a full memory round trip.
template <typename S, bool CPLX, int MODE, bool CONJ, int T>
__device__ __forceinline__ void move_tile(const Piece* __restrict__ pieces, int32_t pi, int32_t c,
                                          Bufs bufs, int32_t xcd_run,
                                          Vec<S, CPLX ? 2 : 1>* lds, S ar, S ai, S br, S bi) {
  using TT = TypeTraits<S, CPLX>;
  using E = Vec<S, TT::NS>;
  constexpr int NP = (tile_budget(TT::ES, T) + T - 1) / T;  // elements per lane
  const Piece& p = pieces[pi];
  const int32_t tid = threadIdx.x;
  const int32_t tx = tile_x_of(p.aux), ty = tile_y_of(p.aux);
  const int32_t stride = ty | 1;
  int32_t rows, ntx, cy, cx;
  divmod(p.nx + tx - 1, tx, ntx, rows);
  divmod(c, ntx, cy, cx);
  const int32_t x0 = cx * tx, y0 = cy * ty;
  const int32_t w = min(tx, p.nx - x0), h = min(ty, p.ny - y0);
  const int32_t n = w * h;
  const E* __restrict__ se = reinterpret_cast<const E*>(bufs[p.src_buf]) + p.src_off + (int64_t)x0 * p.src_ld + y0;
  E* __restrict__ de = reinterpret_cast<E*>(bufs[p.dst_buf]) + p.dst_off + (int64_t)y0 * p.dst_ld + x0;
  E v[NP];
  int32_t slot[NP];
  // (one loop per cache policy, kept apart by an empty asm: the compiler
  // merges two loads of one address into one without the non-temporal hint)
  auto load_source = [&](auto nt) {
    if constexpr (decltype(nt)::value) asm volatile("");
    TileWalk<T> in(tid, h, p.src_ld, stride, 1);
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      if (k * T >= n) break;
      slot[k] = in.lds;
      if (k * T + tid < n) v[k] = load<decltype(nt)::value>(se + in.off);
      in.next();
    }
  };
  // a tile as tall as its rectangle shares no source line with another one
  // when its columns start and end on lines, and few when they are long
  constexpr int32_t L = 128 / TT::ES;  // elements of a line
  const bool own_lines = h == p.ny && (h * TT::ES >= kShortTileColumn || (p.src_off | p.src_ld | h) % L == 0);
  if (own_lines) load_source(std::true_type{});
  else load_source(std::false_type{});
  E a[MODE == MODE_AXPBY ? NP : 1];
  auto load_a = [&](auto nt) {
    if constexpr (decltype(nt)::value) asm volatile("");
    TileWalk<T> ain(tid, w, p.dst_ld, 1, stride);
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      if (k * T >= n) break;
      if (k * T + tid < n) a[k] = load<decltype(nt)::value>(de + ain.off);
      ain.next();
    }
  };
  if constexpr (MODE == MODE_AXPBY) {
    if (xcd_run > 0 && w * TT::ES < kShortTileRow) load_a(std::false_type{});
    else load_a(std::true_type{});
  }
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    if (k * T >= n) break;
    if (k * T + tid < n) lds[slot[k]] = v[k];
  }
  __syncthreads();
  TileWalk<T> out(tid, w, p.dst_ld, 1, stride);
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    if (k * T >= n) break;
    if (k * T + tid < n)
      store(de + out.off,
            combine<S, TT::NS, CPLX, MODE, CONJ>(lds[out.lds], a[MODE == MODE_AXPBY ? k : 0], ar, ai, br, bi));
    out.next();
  }
}

// The row walk of one workgroup for a fixed arithmetic mode.
template <typename S, bool CPLX, int MODE, bool CONJ, int UL>
__device__ __forceinline__ void walk_task(const Piece* __restrict__ pieces, int32_t pi, int32_t c,
                                          Bufs bufs, Items ip,
                                          int32_t allow_wide) {
  S ar = S(0), ai = S(0), br = S(0), bi = S(0);
  if constexpr (MODE != MODE_COPY) {
    ar = (S)ip->alpha[0];
    ai = (S)ip->alpha[1];
    br = (S)ip->beta[0];
    bi = (S)ip->beta[1];
  }
  if constexpr (MODE != MODE_AXPBY) {
    // stacks outside the pack hold only rectangles of pairs that do not read A
    if (pieces[pi].flags & PIECE_STACK) {
      move_stack<S, CPLX, MODE, CONJ>(pieces, pi, c, bufs, allow_wide, ar, ai, br, bi);
      return;
    }
  }
  if constexpr (TypeTraits<S, CPLX>::ES >= 16)
    move_walk_lanes<S, CPLX, MODE, CONJ, UL>(pieces, pi, c, bufs, allow_wide, ar, ai, br, bi);
  else
    move_walk<S, CPLX, MODE, CONJ, UL>(pieces, pi, c * (UL * kThreads), bufs, allow_wide, ar, ai, br, bi);
}

// The LDS tile of one workgroup for a fixed arithmetic mode.
template <typename S, bool CPLX, int MODE, bool CONJ, int T>
__device__ __forceinline__ void tile_task(const Piece* __restrict__ pieces, int32_t pi, int32_t c,
                                          Bufs bufs, Items ip,
                                          int32_t xcd_run, Vec<S, CPLX ? 2 : 1>* lds) {
  S ar = S(0), ai = S(0), br = S(0), bi = S(0);
  if constexpr (MODE != MODE_COPY) {
    ar = (S)ip->alpha[0];
    ai = (S)ip->alpha[1];
    br = (S)ip->beta[0];
    bi = (S)ip->beta[1];
  }
  move_tile<S, CPLX, MODE, CONJ, T>(pieces, pi, c, bufs, xcd_run, lds, ar, ai, br, bi);
}

// MODE of a kernel that reads the mode and the conjugation of its rectangle's
// pair (batches that mix them; a workgroup's rectangles belong to one pair).
constexpr int MODE_ANY = 3;
#define COSTA_BY_MODE(TASK)                                  \
  do {                                                       \
    const bool conj = CPLX && ip->conj;                      \
    if (ip->mode == MODE_COPY) {                             \
      if (conj) TASK(MODE_COPY, CPLX);                       \
      else TASK(MODE_COPY, false);                           \
    } else if (ip->mode == MODE_SCALE) {                     \
      if (conj) TASK(MODE_SCALE, CPLX);                      \
      else TASK(MODE_SCALE, false);                          \
    } else {                                                 \
      if (conj) TASK(MODE_AXPBY, CPLX);                      \
      else TASK(MODE_AXPBY, false);                          \
    }                                                        \
  } while (0)

// Units per lane of a launch of row walks: two (the wide task table) in
// launches that copy -- the pack, and unpack/direct launches with alpha = 1,
// beta = 0 -- one otherwise.  Measured on MI355X: two units per lane +2 to
// +11% on copies; on an axpby walk of short misaligned rows -19%.
template <int KIND, int MODE>
constexpr int units_per_lane() {
  return KIND == KIND_PACK || MODE == MODE_COPY ? COSTA_COPY_UNITS : 1;
}

// One launch slice of row walks: workgroup b moves task task_off +
// xcd_order(b) of the launch's task table.
//   KIND: pack (bitwise copy into message buffers), unpack-transform, or
//         direct.
//   MODE, CONJ: the arithmetic of every pair of the call, or MODE_ANY.
// With two units per lane the table is the launch's wide task table, whose
// first task of a rectangle is in aux.
template <typename S, bool CPLX, int KIND, int MODE, bool CONJ>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4, 8)))
costa_mover(ArgTable, const Piece* __restrict__ pieces, const int32_t* __restrict__ tasks, int32_t task_off,
            const void* __restrict__ device_table, int32_t items_off, int32_t allow_wide, int32_t xcd_run) {
  using TT = TypeTraits<S, CPLX>;
  constexpr int UL = units_per_lane<KIND, MODE>();
  const char COSTA_CONST* table = call_table(device_table);
  const Bufs bufs = (Bufs)table;
  const int32_t b = task_off + xcd_order((int32_t)blockIdx.x, (int32_t)gridDim.x, xcd_run);
  const int32_t pi = tasks[b];
  const int32_t c = b - (UL == 1 ? pieces[pi].task0 : pieces[pi].aux);
  if constexpr (KIND == KIND_PACK) {
    if (pieces[pi].flags & PIECE_STACK) {
      move_stack<S, CPLX, MODE_COPY, false>(pieces, pi, c, bufs, allow_wide, S(0), S(0), S(0), S(0));
      return;
    }
    if constexpr (TT::ES >= 16)
      move_walk_lanes<S, CPLX, MODE_COPY, false, UL>(pieces, pi, c, bufs, allow_wide, S(0), S(0), S(0), S(0));
    else
      move_walk<S, CPLX, MODE_COPY, false, UL>(pieces, pi, c * (UL * kThreads), bufs, allow_wide, S(0), S(0), S(0),
                                               S(0));
  } else {
    const Items ip = (Items)(table + items_off) + pieces[pi].item;
    if constexpr (MODE != MODE_ANY) {
      walk_task<S, CPLX, MODE, CONJ, UL>(pieces, pi, c, bufs, ip, allow_wide);
    } else {
#define COSTA_TASK(M, CJ) walk_task<S, CPLX, M, CJ, UL>(pieces, pi, c, bufs, ip, allow_wide)
      COSTA_BY_MODE(COSTA_TASK);
#undef COSTA_TASK
    }
  }
}

// One launch slice of LDS tiles, T lanes per workgroup; the other parameters
// as above.
template <typename S, bool CPLX, int KIND, int MODE, bool CONJ, int T>
__global__ void __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(2, 8)))
costa_tiles(ArgTable, const Piece* __restrict__ pieces, const int32_t* __restrict__ tasks, int32_t task_off,
            const void* __restrict__ device_table, int32_t items_off, int32_t xcd_run) {
  using TT = TypeTraits<S, CPLX>;
  __shared__ Vec<S, TT::NS> lds[tile_lds_elems(TT::ES, T)];
  const char COSTA_CONST* table = call_table(device_table);
  const Bufs bufs = (Bufs)table;
  const int32_t b = task_off + xcd_order((int32_t)blockIdx.x, (int32_t)gridDim.x, xcd_run);
  const int32_t pi = tasks[b];
  const int32_t c = b - pieces[pi].task0;
  const Items ip = (Items)(table + items_off) + pieces[pi].item;
  if constexpr (MODE != MODE_ANY) {
    tile_task<S, CPLX, MODE, CONJ, T>(pieces, pi, c, bufs, ip, xcd_run, lds);
  } else {
#define COSTA_TASK(M, CJ) tile_task<S, CPLX, M, CJ, T>(pieces, pi, c, bufs, ip, xcd_run, lds)
    COSTA_BY_MODE(COSTA_TASK);
#undef COSTA_TASK
  }
}

// One slice of a call's table from the kernel's arguments to device memory,
// 16 bytes a lane.
constexpr int kStoreTableLanes = (int)(kArgTableBytes / 16);
using Quad = unsigned __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(kStoreTableLanes) costa_store_table(ArgTable, Quad* __restrict__ dst, int32_t n) {
  const Quad COSTA_CONST* src = (const Quad COSTA_CONST*)__builtin_amdgcn_kernarg_segment_ptr();
  const int32_t i = threadIdx.x;
  if (i < n) dst[i] = src[i];
}

// Volume of the grid overlay: every overlay block (k, l) adds its element
// count to V[s][t] (s: owner of its cover in L(B), t: owner of its cover in
// L(A)).  Histogram in LDS when P*P fits, flushed with 64-bit atomics.
__global__ void __launch_bounds__(kThreads) costa_volume(VolumeArgs a, int32_t use_lds) {
  extern __shared__ unsigned long long hist[];
  const int32_t PP = a.P * a.P;
  if (use_lds) {
    for (int32_t i = threadIdx.x; i < PP; i += kThreads) hist[i] = 0ull;
    __syncthreads();
  }
  const int64_t total = (int64_t)a.K * a.L;
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t idx = (int64_t)blockIdx.x * kThreads + threadIdx.x; idx < total; idx += stride) {
    const int32_t k = (int32_t)(idx / a.L), l = (int32_t)(idx % a.L);
    const Interval ri = a.rows[k], ci = a.cols[l];
    const int32_t t = a.ownerA[(int64_t)ri.a * a.nbcA + ci.a];
    const int32_t bi = a.transposed ? ci.b : ri.b, bj = a.transposed ? ri.b : ci.b;
    const int32_t s = a.ownerB[(int64_t)bi * a.nbcB + bj];
    const unsigned long long vol = (unsigned long long)(ri.len * ci.len);
    if (use_lds) atomicAdd(&hist[s * a.P + t], vol);
    else atomicAdd(&a.V[(int64_t)s * a.P + t], vol);
  }
  if (use_lds) {
    __syncthreads();
    for (int32_t i = threadIdx.x; i < PP; i += kThreads)
      if (hist[i]) atomicAdd(&a.V[i], hist[i]);
  }
}

struct Launch {
  hipStream_t stream;
  const Piece* pieces;
  const int32_t* tasks;  // the launch's task table
  int64_t ntasks;
  const int32_t* wide;   // its wide task table (launches of row walks)
  int64_t nwide;
  const ArgTable& args;
  const void* device_table;
  int32_t items_off;
  int32_t allow_wide;
  int32_t xcd_run;
};

// Separable volume in one launch.  Thread per block of the finer side: it
// walks the coarse blocks that its block meets (at most two unless the sides'
// block sizes are alike) and adds each overlap to an LDS histogram by
// (process in op(B), process in A).  Up to kVolumeOneGroup blocks one
// workgroup does both axes; otherwise the workgroups flush their histograms
// with device-scope atomics, and the last one to finish reads the sums and
// leaves them and its counter at zero for the next launch.  Then V[s][t] =
// rows * columns.  Bound by latency: the launch, V written to host memory, the
// host's wait.  Measured on MI355X, 10^5 x 10^5 over 10 x 10 ranks, blocks of
// 30 into 10^4: two launches among six uploads and seven allocations 140 us a
// call, this one 30 (the kernel 9.1; 13.1 with the classes read row by row,
// 16.7 with 64-bit divisions and several workgroups as well); blocks of 2,
// 50,000 an axis, 20 us in the kernel against 116.
constexpr int kVolumeThreads = 1024;
constexpr int kVolumeOneGroup = 16384;

__global__ void __launch_bounds__(kVolumeThreads) costa_volume_dealt(VolumeDealtArgs a) {
  __shared__ unsigned long long h[kVolumeHistMax];
  __shared__ int16_t cls[4 * kVolumeRanksMax];
  __shared__ int32_t last;
  const int32_t tid = threadIdx.x;
  const bool one = gridDim.x == 1;  // (then blockIdx.y is 0 alone)
  // all of the arguments' classes at once: read row by row below, each would
  // wait a memory round trip
  if (tid < 4 * a.P) cls[tid] = a.cls[tid];
  static_assert(4 * kVolumeRanksMax <= kVolumeThreads, "a class a lane");
  for (int32_t i = tid; i < a.nhist; i += kVolumeThreads) h[i] = 0ull;
  __syncthreads();
  for (int32_t d = one ? 0 : blockIdx.y; d <= (one ? 1 : (int32_t)blockIdx.y); ++d) {
    const VolumeAxis& x = a.axis[d];
    const int32_t first = blockIdx.x * kVolumeThreads + tid, step = gridDim.x * kVolumeThreads;
    unsigned long long* hx = h + x.hist0;
    auto add = [hx](int32_t entry, unsigned long long elems) { atomicAdd(&hx[entry], elems); };
    if (a.narrow) count_overlaps<uint32_t>(x, first, step, add);
    else count_overlaps<uint64_t>(x, first, step, add);
  }
  __syncthreads();
  if (!one) {
    for (int32_t i = tid; i < a.nhist; i += kVolumeThreads)
      if (h[i]) atomicAdd(&a.hist[i], h[i]);
    __threadfence();  // the sums are in device memory before this workgroup is counted
    __syncthreads();
    if (tid == 0) last = atomicAdd(&a.hist[a.nhist], 1ull) == (unsigned long long)gridDim.x * gridDim.y - 1;
    __syncthreads();
    if (!last) return;
    __threadfence();
    for (int32_t i = tid; i < a.nhist; i += kVolumeThreads) h[i] = atomicExch(&a.hist[i], 0ull);
    if (tid == 0) a.hist[a.nhist] = 0ull;
    __syncthreads();
  }
  // a wave per row of V
  const int32_t lane = tid % 64;
  const unsigned long long *hr = h + a.axis[0].hist0, *hc = h + a.axis[1].hist0;
  for (int32_t s = tid / 64; s < a.P; s += kVolumeThreads / 64) {
    const int32_t rb = cls[2 * (a.P + s)], cb = cls[2 * (a.P + s) + 1];
    for (int32_t t = lane; t < a.P; t += 64) {
      const int32_t ra = cls[2 * t], ca = cls[2 * t + 1];
      a.V[(int64_t)s * a.P + t] =
          (ra < 0 || rb < 0) ? 0ull : hr[rb * a.axis[0].nclass + ra] * hc[cb * a.axis[1].nclass + ca];
    }
  }
}

// Separable volume, step 1: histogram of overlay interval lengths by (class
// of the covering block in op(B), class of the covering block in A), for the
// rows (blockIdx.y == 0) and the columns (blockIdx.y == 1).
__global__ void __launch_bounds__(kThreads) costa_volume_hist(SeparableArgs a) {
  const bool rows = blockIdx.y == 0;
  const Interval* iv = rows ? a.rows : a.cols;
  const int32_t n = rows ? a.K : a.L;
  unsigned long long* h = rows ? a.hrow : a.hcol;
  const int32_t na = rows ? a.nra : a.nca;
  for (int32_t i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads) {
    const Interval v = iv[i];
    atomicAdd(&h[(int64_t)v.b * na + v.a], (unsigned long long)v.len);
  }
}

// Separable volume, step 2: V[s][t] = hrow[row class of s][row class of t] *
// hcol[col class of s][col class of t], 0 when s or t has no place in its
// grid (for op T the row overlay of op(B) runs over B's process columns and
// the column overlay over its rows; the host folds that into clsB).
__global__ void __launch_bounds__(kThreads) costa_volume_outer(SeparableArgs a) {
  const int32_t PP = a.P * a.P;
  for (int32_t k = blockIdx.x * kThreads + threadIdx.x; k < PP; k += gridDim.x * kThreads) {
    const int32_t s = k / a.P, t = k % a.P;
    const int32_t ra = a.clsA[2 * t], ca = a.clsA[2 * t + 1];
    const int32_t rb = a.clsB[2 * s], cb = a.clsB[2 * s + 1];
    a.V[k] = (ra < 0 || rb < 0) ? 0ull : a.hrow[(int64_t)rb * a.nra + ra] * a.hcol[(int64_t)cb * a.nca + ca];
  }
}

// One workgroup per task of the table the launch runs on, in slices that
// keep the grid below 2^32 work-items.
template <typename F>
hipError_t in_slices(int64_t ntasks, F&& launch) {
  if (ntasks > INT32_MAX) return hipErrorInvalidValue;
  constexpr int64_t kSlice = (int64_t)1 << 23;
  for (int64_t off = 0; off < ntasks; off += kSlice) {
    launch((unsigned)(ntasks - off < kSlice ? ntasks - off : kSlice), (int32_t)off);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <typename S, bool CPLX, int KIND, int MODE, bool CONJ>
hipError_t go_walks(const Launch& l) {
  constexpr bool WIDE = units_per_lane<KIND, MODE>() > 1;
  const int32_t* tasks = WIDE ? l.wide : l.tasks;
  return in_slices(WIDE ? l.nwide : l.ntasks, [&](unsigned n, int32_t off) {
    hipLaunchKernelGGL((costa_mover<S, CPLX, KIND, MODE, CONJ>), dim3(n), dim3(kThreads), 0, l.stream, l.args, l.pieces,
                       tasks, off, l.device_table, l.items_off, l.allow_wide, l.xcd_run);
  });
}

template <typename S, bool CPLX, int KIND, int MODE, bool CONJ, int T>
hipError_t go_tiles(const Launch& l) {
  return in_slices(l.ntasks, [&](unsigned n, int32_t off) {
    hipLaunchKernelGGL((costa_tiles<S, CPLX, KIND, MODE, CONJ, T>), dim3(n), dim3(T), 0, l.stream, l.args, l.pieces,
                       l.tasks, off, l.device_table, l.items_off, l.xcd_run);
  });
}

template <typename S, bool CPLX, int KIND, int MODE, bool CONJ>
hipError_t go(const Launch& l, int tile_lanes) {
  if (tile_lanes == 0) return go_walks<S, CPLX, KIND, MODE, CONJ>(l);
  if (tile_lanes == kSmallTileLanes) {  // (planned for the direct form alone)
    if constexpr (KIND == KIND_DIRECT) return go_tiles<S, CPLX, KIND, MODE, CONJ, kSmallTileLanes>(l);
    else return hipErrorInvalidValue;
  }
  return go_tiles<S, CPLX, KIND, MODE, CONJ, kThreads>(l);
}

template <typename S, bool CPLX, int KIND>
hipError_t go_mode(const Launch& l, const LaunchSpec& spec) {
  // one mode for the whole call: its own kernel (the per-pair kernel holds
  // the registers of every mode: float tiles 83 against 64, five waves per
  // SIMD against eight)
  const int conj = spec.conj, tl = spec.tile_lanes;
  if (spec.mode == MODE_COPY)
    return conj ? go<S, CPLX, KIND, MODE_COPY, CPLX>(l, tl) : go<S, CPLX, KIND, MODE_COPY, false>(l, tl);
  if (spec.mode == MODE_SCALE)
    return conj ? go<S, CPLX, KIND, MODE_SCALE, CPLX>(l, tl) : go<S, CPLX, KIND, MODE_SCALE, false>(l, tl);
  if (spec.mode == MODE_AXPBY)
    return conj ? go<S, CPLX, KIND, MODE_AXPBY, CPLX>(l, tl) : go<S, CPLX, KIND, MODE_AXPBY, false>(l, tl);
  return go<S, CPLX, KIND, MODE_ANY, false>(l, tl);
}

template <typename S, bool CPLX>
hipError_t launch_typed(MoverKind kind, const LaunchSpec& spec, const Launch& l) {
  if (kind == KIND_PACK) return go_walks<S, CPLX, KIND_PACK, MODE_COPY, false>(l);
  if (kind == KIND_UNPACK) return go_mode<S, CPLX, KIND_UNPACK>(l, spec);
  return go_mode<S, CPLX, KIND_DIRECT>(l, spec);
}

}  // namespace

hipError_t launch_mover(MoverKind kind, costa_dtype dtype, const LaunchSpec& spec, const Piece* pieces,
                        const int32_t* tasks, int64_t ntasks, const int32_t* wide, int64_t nwide,
                        const CallTable& table, int32_t allow_wide, int32_t xcd_run, hipStream_t stream) {
  if (ntasks <= 0) return hipSuccess;
  if (!spec.tile_lanes && nwide <= 0) return hipErrorInvalidValue;  // a launch of row walks has both tables
  static const ArgTable none{};
  Launch l{stream, pieces, tasks, ntasks, wide, nwide, table.args ? *table.args : none,
           table.args ? nullptr : table.device, table.items_off, allow_wide, xcd_run};
  switch (dtype) {
    case COSTA_R64: return launch_typed<double, false>(kind, spec, l);
    case COSTA_C128: return launch_typed<double, true>(kind, spec, l);
    case COSTA_R32: return launch_typed<float, false>(kind, spec, l);
    case COSTA_C64: return launch_typed<float, true>(kind, spec, l);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_store_table(const unsigned char* table, size_t bytes, void* dst, hipStream_t stream) {
  for (size_t at = 0; at < bytes; at += kArgTableBytes) {
    ArgTable args;
    const size_t n = bytes - at < kArgTableBytes ? bytes - at : kArgTableBytes;
    std::memcpy(args.bytes, table + at, n);
    hipLaunchKernelGGL(costa_store_table, dim3(1), dim3(kStoreTableLanes), 0, stream, args,
                       reinterpret_cast<Quad*>(static_cast<unsigned char*>(dst) + at), (int32_t)(n / 16));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_volume_dealt(const VolumeDealtArgs& a, hipStream_t stream) {
  const int32_t nmax = a.axis[0].nblocks > a.axis[1].nblocks ? a.axis[0].nblocks : a.axis[1].nblocks;
  // four blocks a thread, at most 64 workgroups an axis: every workgroup flushes a histogram
  unsigned gx = (unsigned)((nmax + 4 * kVolumeThreads - 1) / (4 * kVolumeThreads));
  gx = gx < 2 ? 2 : gx > 64 ? 64 : gx;
  const bool one = (int64_t)a.axis[0].nblocks + a.axis[1].nblocks <= kVolumeOneGroup;
  hipLaunchKernelGGL(costa_volume_dealt, one ? dim3(1, 1) : dim3(gx, 2), dim3(kVolumeThreads), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_volume_separable(const SeparableArgs& a, hipStream_t stream) {
  const int32_t nmax = a.K > a.L ? a.K : a.L;
  if (nmax > 0) {
    unsigned gx = (unsigned)((nmax + kThreads - 1) / kThreads);
    if (gx > 1024) gx = 1024;
    hipLaunchKernelGGL(costa_volume_hist, dim3(gx, 2), dim3(kThreads), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const int32_t PP = a.P * a.P;
  unsigned gx = (unsigned)((PP + kThreads - 1) / kThreads);
  if (gx > 1024) gx = 1024;
  if (gx == 0) return hipSuccess;
  hipLaunchKernelGGL(costa_volume_outer, dim3(gx), dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_volume(const VolumeArgs& a, hipStream_t stream) {
  const int64_t total = (int64_t)a.K * a.L;
  if (total == 0) return hipSuccess;
  int64_t blocks = (total + kThreads - 1) / kThreads;
  if (blocks > 2048) blocks = 2048;
  const size_t lds = (size_t)a.P * a.P * sizeof(unsigned long long);
  const int32_t use_lds = lds <= 64 * 1024 ? 1 : 0;
  hipLaunchKernelGGL(costa_volume, dim3((unsigned)blocks), dim3(kThreads), use_lds ? lds : 0, stream, a, use_lds);
  return hipGetLastError();
}

}  // namespace costa
