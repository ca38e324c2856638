// Index arithmetic of the kernels in a form that compiles for the host as
// well, where its tests run it.  Not part of the public interface.
#pragma once

#include <cmath>

#include "internal.hpp"

namespace costa {

#define COSTA_BOTH __host__ __device__ __forceinline__

// The task of workgroup b of n.  Workgroups are dispatched round-robin over
// the 8 XCDs (b % 8 is b's XCD).  run 0: task b.  run -1: XCD x takes the
// x-th of 8 contiguous ranges of tasks, workgroup b the (b/8)-th task of its
// XCD's range.  run k > 0: the XCDs take runs of k consecutive tasks in turn
// (tasks past the last whole round of runs: task b).
COSTA_BOTH int32_t xcd_order(int32_t b, int32_t n, int32_t run) {
  constexpr int32_t X = 8;
  if (run == 0) return b;
  const int32_t xcd = b % X, idx = b / X;
  if (run > 0) {
    const int32_t turn = idx / run;
    return (turn + 1) * X * run > n ? b : (turn * X + xcd) * run + idx - turn * run;
  }
  const int32_t q = n / X, r = n % X;
  const int32_t start = xcd < r ? xcd * (q + 1) : r * (q + 1) + (xcd - r) * q;
  return start + idx;
}

// 1 / x to within one ulp: the hardware's estimate; on the host, where tests run
// this code, the quotient moved by `reciprocal_ulps`.
#if !defined(__HIP_DEVICE_COMPILE__)
inline int reciprocal_ulps = 0;
#endif
COSTA_BOTH float reciprocal(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_rcpf(x);
#else
  const float r = 1.0f / x;
  return reciprocal_ulps == 0 ? r : std::nextafterf(r, reciprocal_ulps < 0 ? 0.0f : 4.0f);
#endif
}

constexpr int32_t kDivmodUnits = (1 << 22) + 1024, kDivmodUnits2 = 1 << 23;

// y = u / n and x = u - y*n for 0 <= u < kDivmodUnits and n >= 1, or
// u < kDivmodUnits2 and n >= 2:
// the estimate u * rcp(n) is off by at most 1.5 * 2^-23 of the quotient (rcp
// to 1 ulp, one rounding of the product), less than one, so one step each way
// makes it exact.  Selects, not loops: the corrections cost two instructions
// each and no branch.
COSTA_BOTH void divmod(int32_t u, int32_t n, int32_t& y, int32_t& x) {
  y = (int32_t)((float)u * reciprocal((float)n));
  x = u - y * n;
  const bool under = x < 0;
  y = under ? y - 1 : y;
  x = under ? x + n : x;
  const bool over = x >= n;
  y = over ? y + 1 : y;
  x = over ? x - n : x;
}

// A lane's way through the rows (`len` elements each) of a tile, T
// elements a step: the element's memory offset (row * ld + column) and its
// LDS slot (row * ls + column * lc).  One division places the lane; every
// step then adds the same two amounts, and one more where the step passes a
// row's end (a step passes at most one: T % len < len).
template <int T>
struct TileWalk {
  int32_t col, len, rem, lds, dlds, wlds;
  int64_t off, doff, woff;
  COSTA_BOTH TileWalk(int32_t tid, int32_t len_, int64_t ld, int32_t ls, int32_t lc) : len(len_) {
    int32_t q, row;
    divmod(T, len, q, rem);
    divmod(tid, len, row, col);
    off = (int64_t)row * ld + col;
    doff = (int64_t)q * ld + rem;
    woff = ld - len;
    lds = row * ls + col * lc;
    dlds = q * ls + rem * lc;
    wlds = ls - len * lc;
  }
  COSTA_BOTH void next() {
    col += rem;
    const bool wrap = col >= len;
    col -= wrap ? len : 0;
    off += doff + (wrap ? woff : 0);
    lds += dlds + (wrap ? wlds : 0);
  }
};

// The overlaps of blocks first, first + step, ... of an axis's finer side with
// the coarse blocks that each of them meets: add(histogram entry, elements).
// I holds every position up to one block past the window (see
// VolumeDealtArgs::narrow).
template <typename I, typename Add>
COSTA_BOTH void count_overlaps(const VolumeAxis& x, uint32_t first, uint32_t step, Add&& add) {
  const I off = (I)x.fine.off, blk = (I)x.fine.blk, coff = (I)x.coarse.off, cblk = (I)x.coarse.blk, n = (I)x.n;
  const I fnp = (I)x.fine.np, fsrc = (I)x.fine.src, cnp = (I)x.coarse.np, csrc = (I)x.coarse.src;
  const I k0 = off / blk;  // the window's first block in the dealt dimension
  for (uint32_t k = first; k < (uint32_t)x.nblocks; k += step) {  // (unsigned: k may pass 2^31 by a step)
    const I b = k0 + (I)k;
    const I start = b * blk, stop_f = (b + 1) * blk;
    I i = (off > start ? off : start) - off;  // in the window
    const I end = (off + n < stop_f ? off + n : stop_f) - off;
    const int32_t pf = (int32_t)((b + fsrc) % fnp);
    while (i < end) {
      const I cb = (coff + i) / cblk;
      const I stop_c = (cb + 1) * cblk - coff;
      const I stop = end < stop_c ? end : stop_c;
      const int32_t pc = (int32_t)((cb + csrc) % cnp);
      add(x.fine_is_b ? pf * x.nclass + pc : pc * x.nclass + pf, (unsigned long long)(stop - i));
      i = stop;
    }
  }
}

}  // namespace costa
