// mask[i] = 1 if another delivery has a bitwise-equal key (only those digests
// decide dedupe and ties), else 0. One workgroup of at least n threads.
//
// Re-deliveries by their bytes: a delivery that equals an earlier one of the
// same key and length byte for byte has that one's Id, so it needs no hash of its
// own, and no digest decides that it is absorbed. lead[i] is the first delivery
// of i's key and length; copy_kernel (hash.hip) compares i with it and sets
// differs[i]. A delivery is then a copy, or one whose digest the order reads if
// another of its key is no copy either, or one whose Id the render computes.
// (lead == nullptr: every delivery with an equal key is hashed before the order.)
// With a non-finite score in the set nothing is rendered, so nothing is left to the
// render: no delivery counts as a copy, and all with an equal key are hashed.
#pragma once

#include "internal.h"

namespace cm {

struct Copies {
  const double* keys;
  int32_t* lead;
  int32_t* differs;
  __device__ __forceinline__ bool is_copy(int i) const { return lead[i] != i && differs[i] == 0; }
  // whether delivery j makes the order read the digest of delivery i, no copy
  __device__ __forceinline__ bool ties(int i, int j) const {
    return j != i && keys[j] == keys[i] && !is_copy(j);
  }
  // whether the Id of i (the same on every lane of the wave) comes before the order
  __device__ __forceinline__ bool needed(int i, int32_t n, int lane) const {
    if (is_copy(i)) return false;
    for (int j0 = 0; j0 < n; j0 += 64)
      if (__builtin_amdgcn_ballot_w64(j0 + lane < n && ties(i, j0 + lane)) != 0) return true;
    return false;
  }
};

__device__ __forceinline__ void equal_key_mask_body(int32_t n, const double* __restrict__ keys,
                                                    uint8_t* __restrict__ mask,
                                                    const int64_t* __restrict__ table = nullptr,
                                                    int64_t stride = 0, int64_t token_bytes = 0,
                                                    int32_t L = 0, int32_t* lead = nullptr,
                                                    int32_t* differs = nullptr,
                                                    int32_t* end = nullptr) {
  __shared__ double s_key[1024];
  __shared__ int32_t s_end[1024];
  const int tid = threadIdx.x;
  int32_t stripes = 0;                     // to compare of this delivery
  double key = 0.0;
  if (tid < n) {
    key = keys[tid];
    s_key[tid] = key;
  }
  const bool renders = !__syncthreads_or(tid < n && !isfinite(key));
  if (tid < n) {
    bool shared = false;
    for (int j = 0; j < n; ++j) shared |= (j != tid && s_key[j] == key);
    mask[tid] = shared ? 1 : 0;
    if (lead) {
      const int64_t len = table[(int64_t)tid * stride];
      int l = tid;
      for (int j = 0; renders && shared && j < tid; ++j)
        if (s_key[j] == key && table[(int64_t)j * stride] == len) {
          l = j;
          break;
        }
      lead[tid] = l;
      differs[tid] = 0;
      if (l != tid) stripes = (int32_t)(2 * L * stripes_of(len * token_bytes));
    }
  }
  if (!lead) return;
  // their running total, unless there is nothing to compare
  const bool any = __syncthreads_or(stripes != 0);
  s_end[tid] = stripes;
  __syncthreads();
  for (int o = 1; any && o < (int)blockDim.x; o <<= 1) {
    const int32_t t = tid >= o ? s_end[tid - o] : 0;
    __syncthreads();
    s_end[tid] += t;
    __syncthreads();
  }
  if (tid < n) end[tid] = s_end[tid];
}

}  // namespace cm
