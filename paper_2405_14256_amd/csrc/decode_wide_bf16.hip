// Instantiates the matrix-core decode kernel for caches with 8-bit codes and bf16 queries.
#include "decode_mfma_kernel.hpp"

namespace zc {
int launch_decode_wide_bf16(const DecArgs& a, hipStream_t st) { return launch_decode_mfma_dt<ZC_BF16, true>(a, st); }
}  // namespace zc
