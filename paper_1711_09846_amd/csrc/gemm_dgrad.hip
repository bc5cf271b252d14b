// The population-batched GEMM of an input gradient: times the activation's derivative and the keep factors of a dropout site.
#include "gemm_run.h"

namespace pbt {

template <int ACT>
static hipError_t dgrad(const GemmOperands& o, const bf16_t* Zprev, bf16_t* dZ, int64_t ld, int64_t so, hipStream_t s) {
  return run_gemm(o, EpiDgradAct<ACT, false>{Zprev, dZ, ld, so, nullptr, 0, nullptr, 0, -1}, s);
}
hipError_t gemm_dgrad_act(const GemmOperands& o, const bf16_t* Zprev, bf16_t* dZ, int64_t ld, int64_t so, int act,
                          hipStream_t s, const DropRecord& drop) {
  if (drop.mask) {
    if (o.N % 8 || ld % 8 || so % 8 || ((reinterpret_cast<uintptr_t>(Zprev) | reinterpret_cast<uintptr_t>(dZ)) & 15)) return hipErrorInvalidValue;
    if (act != ACT_RELU) return hipErrorInvalidValue;
    return run_gemm(o, EpiDgradAct<ACT_RELU, true>{Zprev, dZ, ld, so, drop.mask, drop.mask_stride, drop.H, drop.n_hyper, drop.col}, s);
  }
  switch (act) {
    case ACT_RELU: return dgrad<ACT_RELU>(o, Zprev, dZ, ld, so, s);
    case ACT_GELU: return dgrad<ACT_GELU>(o, Zprev, dZ, ld, so, s);
    case ACT_LEAKY_RELU: return dgrad<ACT_LEAKY_RELU>(o, Zprev, dZ, ld, so, s);
    case ACT_TANH: return dgrad<ACT_TANH>(o, Zprev, dZ, ld, so, s);
    default: return dgrad<ACT_NONE>(o, Zprev, dZ, ld, so, s);
  }
}

}  // namespace pbt
