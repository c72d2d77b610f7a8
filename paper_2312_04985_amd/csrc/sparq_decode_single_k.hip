// Launches of the kernel for a key cache stored once.
#include "sparq_decode_single_k.h"

namespace sparq {

namespace {

// Lengths are served up to which the keys, the kernel's arrays and DH words more fit the LDS: what is refused stays refused.
template <int DH>
__host__ __device__ constexpr size_t limit_words_1k() { return lds_words_1k<DH>() + DH; }

}  // namespace

size_t decode_single_k_lds_bytes(int S_max, int d_h) {
  switch (d_h) {
    case 64: return 4 * ((size_t)S_max + limit_words_1k<64>());
    case 128: return 4 * ((size_t)S_max + limit_words_1k<128>());
    case 256: return 4 * ((size_t)S_max + limit_words_1k<256>());
    default: return 0;
  }
}

hipError_t launch_decode_single_k(const DecodeArgs& a, int dtype, hipStream_t s) {
  return decode_single_k_short(a) ? launch_decode_single_k_short(a, dtype, s) : launch_1k_any(a, dtype, s);
}

}  // namespace sparq
