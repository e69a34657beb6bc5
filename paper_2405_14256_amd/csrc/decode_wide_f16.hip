// Instantiates the matrix-core decode kernel for caches with 8-bit codes and f16 queries.
#include "decode_mfma_kernel.hpp"

namespace zc {
int launch_decode_wide_f16(const DecArgs& a, hipStream_t st) { return launch_decode_mfma_dt<ZC_F16, true>(a, st); }
}  // namespace zc
