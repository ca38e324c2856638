// Index arithmetic of the kernels in a form that compiles for the host as
// well, where its tests run it.  Not part of the public interface.
#pragma once

#include "internal.hpp"

namespace costa {

#define COSTA_BOTH __host__ __device__ __forceinline__

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
