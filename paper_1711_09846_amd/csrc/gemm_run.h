// From the callers' operands to a kernel launch.
#pragma once
#include "gemm_bf16.h"
#include "gemm_lds.h"
#include "internal.h"

namespace pbt {

inline GemmArgs arguments(const GemmOperands& o) {
  GemmArgs g;
  g.A = o.A; g.lda = o.lda; g.sa = o.sa;
  g.B = o.B; g.ldb = o.ldb; g.sb = o.sb;
  g.M = o.M; g.N = o.N; g.K = o.K; g.batch = o.batch;
  g.tiles_m = g.tiles_n = 0;
  g.inner = o.inner < 1 ? 1 : o.inner; g.sa_in = o.sa_in; g.sb_in = o.sb_in;
  g.colsum = o.colsum; g.colsum_stride = o.colsum_stride; g.colsum_k = o.colsum_k < 0 ? o.K : o.colsum_k;
  g.upper = o.symmetric;
  g.b_cols = o.b_cols > o.N ? o.b_cols : o.N;
  return g;
}
// (rows of 16 million elements are past what a buffer offset spans)
inline bool gemm_rows_fit_lds(const GemmOperands& o) { return o.lda < GL_MAX_PITCH && o.ldb < GL_MAX_PITCH; }
template <class E>
hipError_t run_gemm(const GemmOperands& o, const E& e, hipStream_t s) {
  if (!gemm_rows_fit_lds(o)) return launch_gemm_bf16(arguments(o), o.a_m_contig, o.b_k_contig, e, s);
  return launch_gemm_lds(arguments(o), o.a_m_contig, o.b_k_contig, e, s);
}

}  // namespace pbt
