// The population-batched GEMM with results stored as they are or with a bias: weight gradients, products of the attention, logits.
#include "gemm_run.h"

namespace pbt {

hipError_t gemm_store_f32(const GemmOperands& o, float* C, int64_t ldc, int64_t sc, hipStream_t s) {
  return run_gemm(o, EpiStoreF32{C, ldc, sc}, s);
}
hipError_t gemm_store_bf16(const GemmOperands& o, bf16_t* C, int64_t ldc, int64_t sc, hipStream_t s) {
  return run_gemm(o, EpiStoreBF16{C, ldc, sc}, s);
}
hipError_t gemm_store_bf16_heads(const GemmOperands& o, bf16_t* C, int64_t ldc, int64_t sc, int64_t sc_in, hipStream_t s) {
  return run_gemm(o, EpiStoreBF16{C, ldc, sc, o.inner, sc_in}, s);
}
hipError_t gemm_bias_f32(const GemmOperands& o, const float* bias, int64_t sbias, float* C, int64_t ldc, int64_t sc, hipStream_t s) {
  return run_gemm(o, EpiBiasF32{bias, sbias, C, ldc, sc}, s);
}

}  // namespace pbt
