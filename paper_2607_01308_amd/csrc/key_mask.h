// mask[i] = 1 if another delivery has a bitwise-equal key (only those digests
// decide dedupe and ties), else 0. One workgroup of at least n threads.
//
// Re-deliveries by their bytes (Copies): a delivery that equals an earlier one of the
// same key and length byte for byte has that one's Id, so it needs no hash of its
// own, and no digest decides that it is absorbed. lead[i] is the first delivery
// of i's key and length; copy_kernel (hash.hip) compares i with it and marks
// lead[i] if they differ. A delivery is then a copy, or one whose digest the order
// reads if another of its key is no copy either (distinct counts them by key, so
// that every kernel after this one tells with a few loads, whatever n is: walking
// the deliveries for each took the order of 1024 distinct ones from 382 to 684 us),
// or one whose Id the render computes.
// (lead == nullptr: every delivery with an equal key is hashed before the order.)
// With a non-finite score in the set nothing is rendered, so nothing is left to the
// render: no delivery counts as a copy, and all with an equal key are hashed.
#pragma once

#include "internal.h"

namespace cm {

__device__ __forceinline__ void equal_key_mask_body(int32_t n, const double* __restrict__ keys,
                                                    uint8_t* __restrict__ mask,
                                                    const int64_t* __restrict__ table = nullptr,
                                                    int64_t stride = 0, int64_t token_bytes = 0,
                                                    int32_t L = 0, const Copies& copies = Copies{}) {
  __shared__ double s_key[1024];
  __shared__ int64_t s_len[1024];
  __shared__ int32_t s_distinct[1024];
  __shared__ int32_t s_end[1024];
  const int tid = threadIdx.x;
  const bool live = tid < n;
  double key = 0.0;
  if (live) {
    key = keys[tid];
    s_key[tid] = key;
    if (copies.lead) {
      s_len[tid] = table[(int64_t)tid * stride];
      s_distinct[tid] = 0;
    }
  }
  bool renders = true;
  if (copies.lead) renders = !__syncthreads_or(live && !isfinite(key));
  else __syncthreads();
  bool shared = false;
  if (live) {
    for (int j = 0; j < n; ++j) shared |= (j != tid && s_key[j] == key);
    mask[tid] = shared ? 1 : 0;
  }
  if (!copies.lead) return;
  int head = tid, lead = tid;              // first delivery of this key; and of this length
  int32_t stripes = 0;                     // to compare of this delivery
  if (live) {
    const int64_t len = s_len[tid];
    for (int j = 0; shared && j < tid; ++j)
      if (s_key[j] == key) {
        head = j;
        break;
      }
    for (int j = head; renders && j < tid; ++j)
      if (s_key[j] == key && s_len[j] == len) {
        lead = j;
        break;
      }
    if (lead == tid) atomicAdd(&s_distinct[head], 1);
    else stripes = (int32_t)(2 * L * stripes_of(len * token_bytes));
  }
  // their running total, unless there is nothing to compare
  s_end[tid] = stripes;
  const bool any = __syncthreads_or(stripes != 0);
  for (int o = 1; any && o < (int)blockDim.x; o <<= 1) {
    const int32_t t = tid >= o ? s_end[tid - o] : 0;
    __syncthreads();
    s_end[tid] += t;
    __syncthreads();
  }
  if (live) {
    copies.lead[tid] = lead;
    copies.head[tid] = head;
    copies.distinct[tid] = s_distinct[tid];
    copies.end[tid] = s_end[tid];
  }
}

}  // namespace cm
