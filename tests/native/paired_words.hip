// Compressions with message words that the compiler knows: zeros, and words equal
// to state words (compiled to assembly by test_paired_registers.py; never run).
#include "blake3.h"

template <int LEVELS>
__global__ void zero_words(uint32_t* out) {
  cm::B3Cv s;
  cm::b3_init(s);
  uint32_t m[16] = {0};
  cm::b3_compress_paired<LEVELS>(s, m, 0, 64, 11);
  for (int k = 0; k < 8; ++k) out[threadIdx.x * 8 + k] = s.h[k];
}

template <int LEVELS>
__global__ void state_words(uint32_t* out) {
  cm::B3Cv s;
  uint32_t m[16];
  for (int k = 0; k < 8; ++k) m[k] = m[8 + k] = s.h[k] = out[threadIdx.x * 8 + k];
  cm::b3_compress_paired<LEVELS>(s, m, 0, 64, 11);
  for (int k = 0; k < 8; ++k) out[threadIdx.x * 8 + k] = s.h[k];
}

template __global__ void zero_words<0>(uint32_t*);
template __global__ void zero_words<1>(uint32_t*);
template __global__ void state_words<0>(uint32_t*);
template __global__ void state_words<1>(uint32_t*);
