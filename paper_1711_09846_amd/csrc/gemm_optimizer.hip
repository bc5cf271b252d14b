// The weight-gradient GEMM with the optimiser in its epilogue.
#include "gemm_run.h"

namespace pbt {

hipError_t gemm_wgrad_optimizer(const GemmOperands& o, const OptArgs& a, int64_t off, int64_t ldc, hipStream_t s) {
  const OptHyper hy{a.H, a.t, a.n_hyper, a.col_lr, a.col_beta1, a.col_wd, a.c0, a.c1, a.c2, a.c3, a.t_mul, a.t_add};
  const GemmArgs g = arguments(o);
  if (a.optimizer == OPT_SGD_MOMENTUM) return launch_gemm_bf16(g, o.a_m_contig, o.b_k_contig, EpiOptimizer<OPT_SGD_MOMENTUM>{a.W32, a.S0, a.S1, a.W16, a.stride, off, ldc, hy, {}}, s);
  if (a.optimizer == OPT_ADAM) return launch_gemm_bf16(g, o.a_m_contig, o.b_k_contig, EpiOptimizer<OPT_ADAM>{a.W32, a.S0, a.S1, a.W16, a.stride, off, ldc, hy, {}}, s);
  return launch_gemm_bf16(g, o.a_m_contig, o.b_k_contig, EpiOptimizer<OPT_RMSPROP>{a.W32, a.S0, a.S1, a.W16, a.stride, off, ldc, hy, {}}, s);
}

}  // namespace pbt
