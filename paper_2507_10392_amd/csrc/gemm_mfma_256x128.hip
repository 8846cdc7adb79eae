// Instantiation of the bf16 MFMA GEMM: 256 x 128 workgroup tile, 8 wavefronts.
#include "gemm_mfma_impl.h"
namespace zs {
hipError_t gemm_mfma_256x128(hipStream_t st, const Gemm& g) { return gemm_impl::gemm_mfma_tile<bf16, 256, 128, 8>(st, g); }
}  // namespace zs
