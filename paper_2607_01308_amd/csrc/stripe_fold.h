// The values of aligned runs of BLAKE3 chunks, folded by one wave: the 64 chunks
// of a stripe by the wave that hashed them (the chunk kernels, the fused render),
// the top of a tensor's tree and the chunks of a fragment's Id by one-wave
// workgroups.
#pragma once

#include "blake3_quad.h"
#include "internal.h"

namespace cm {

// The wave's LDS accesses before this come before those after it (a wave's LDS
// instructions execute in order; this keeps the compiler's order).
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Fold cnt (1 .. 64) chaining values held in LDS (word w of value p at lds[8 p + w],
// 16-byte aligned), `levels` levels up or into one (at lds[0 .. 7]), level by
// level: value j of a level is
// the BLAKE3 parent of values 2j and 2j+1 of the level below, an unpaired last
// value is carried up. ROOT marks the final compression when root is set. All
// lanes of the wave take part. A level of at most 16 values is made by quads
// (b3_compress_quad: value j by lanes 4j .. 4j + 3), which shortens the chain of
// dependent compressions about 2x; a wider level takes one lane per value
// (LEVELS: b3_compress_paired's, or -1 for b3_compress). 64 values cost about 3.3
// compressions, a fifth of hashing their chunks.
template <int LEVELS>
__device__ __forceinline__ void fold_cvs(uint32_t* lds, int cnt, bool root, int lane,
                                         int levels = 6) {
  const int Q = lane >> 2;
  const int q = lane & 3;
  u32x4* v = reinterpret_cast<u32x4*>(lds);
  auto pair_words = [&](int p, uint32_t (&m)[16]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const u32x4 x = v[4 * p + k];
#pragma unroll
      for (int w = 0; w < 4; ++w) m[4 * k + w] = x[w];
    }
  };
  wave_lds_order();
  for (; cnt > 1 && levels > 0; --levels) {
    const int nn = (cnt + 1) >> 1;
    const uint32_t flags = kB3Parent | (root && nn == 1 ? kB3Root : 0u);
    uint32_t m[16];
    if (nn <= 16) {
      uint32_t lo = 0, hi = 0;
      const bool pair = Q < nn && 2 * Q + 1 < cnt;   // uniform over the quad
      if (pair) {
        pair_words(Q, m);
      } else if (Q < nn) {
        lo = lds[(2 * Q) * 8 + q];
        hi = lds[(2 * Q) * 8 + 4 + q];
      }
      wave_lds_order();
      if (pair) {
        b3_init_quad(lo, hi, (q & 1) != 0, (q & 2) != 0);
        b3_compress_quad(lo, hi, m, 0, 64, flags, (q & 1) != 0, (q & 2) != 0);
      }
      if (Q < nn) {
        lds[Q * 8 + q] = lo;
        lds[Q * 8 + 4 + q] = hi;
      }
    } else {
      // nn = 17 .. 32 values, one lane each; an unpaired last value stays as it is
      const bool pair = lane < nn && 2 * lane + 1 < cnt;
      const bool copy = lane < nn && !pair;
      B3Cv cv;
      if (pair) {
        pair_words(lane, m);
      } else if (copy) {
        const u32x4 x0 = v[4 * lane], x1 = v[4 * lane + 1];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          cv.h[w] = x0[w];
          cv.h[4 + w] = x1[w];
        }
      }
      wave_lds_order();
      if (pair) {
        b3_init(cv);
        if constexpr (LEVELS >= 0) b3_compress_paired<LEVELS>(cv, m, 0, 64, flags);
        else b3_compress(cv, m, 0, 64, flags);
      }
      if (pair || copy) {
        v[2 * lane] = u32x4{cv.h[0], cv.h[1], cv.h[2], cv.h[3]};
        v[2 * lane + 1] = u32x4{cv.h[4], cv.h[5], cv.h[6], cv.h[7]};
      }
    }
    wave_lds_order();
    cnt = nn;
  }
}

// The level-v nodes (v = 3 .. 6, or below with one node) of a stripe of cnt chunks
// whose chaining values the wave has put into lds, to out: at most eight, 32
// bytes each. root: the stripe is the whole tensor (a single chunk has its ROOT
// already).
template <int LEVELS>
__device__ __forceinline__ void stripe_nodes(uint32_t* lds, int cnt, int v, bool root, int lane,
                                             uint8_t* out) {
  fold_cvs<LEVELS>(lds, cnt, root, lane, v);
  const int nodes = (cnt + (1 << v) - 1) >> v;
  if (lane < 8 * nodes) reinterpret_cast<uint32_t*>(out)[lane] = lds[lane];
}

// The lane's chaining value, its chunk the lane-th of the stripe, into lds.
__device__ __forceinline__ void put_cv(uint32_t* lds, const B3Cv& cv, int lane) {
  u32x4* v = reinterpret_cast<u32x4*>(lds);
  v[2 * lane] = u32x4{cv.h[0], cv.h[1], cv.h[2], cv.h[3]};
  v[2 * lane + 1] = u32x4{cv.h[4], cv.h[5], cv.h[6], cv.h[7]};
}

}  // namespace cm
