// The population-batched GEMM of a forward layer: bias, activation and, for the transformer, the dropout site behind it.
#include "gemm_run.h"

namespace pbt {

hipError_t gemm_bias_act(const GemmOperands& o, const float* bias, int64_t sbias, bf16_t* Z, bf16_t* Aout, int64_t ld,
                         int64_t so, int act, hipStream_t s, const DropSite& site) {
  if (site.record) {
    if (Z || o.N % 8 || ld % 8 || so % 8 || sbias % 4 || (reinterpret_cast<uintptr_t>(bias) & 15) || (reinterpret_cast<uintptr_t>(Aout) & 15)) return hipErrorInvalidValue;
    if (act != ACT_RELU) return hipErrorInvalidValue;   // (the transformer's feed-forward layer)
    return run_gemm(o, EpiBiasActDrop<ACT_RELU>{bias, sbias, Aout, ld, so, site.record, site.record_stride, site.args, site.site}, s);
  }
  switch (act) {
    case ACT_RELU: return run_gemm(o, EpiBiasAct<ACT_RELU>{bias, sbias, Z, Aout, ld, so}, s);
    case ACT_GELU: return run_gemm(o, EpiBiasAct<ACT_GELU>{bias, sbias, Z, Aout, ld, so}, s);
    case ACT_LEAKY_RELU: return run_gemm(o, EpiBiasAct<ACT_LEAKY_RELU>{bias, sbias, Z, Aout, ld, so}, s);
    case ACT_TANH: return run_gemm(o, EpiBiasAct<ACT_TANH>{bias, sbias, Z, Aout, ld, so}, s);
    default: return run_gemm(o, EpiBiasAct<ACT_NONE>{bias, sbias, Z, Aout, ld, so}, s);
  }
}

}  // namespace pbt
