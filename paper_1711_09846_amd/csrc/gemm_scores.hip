// The population-batched GEMM of the held-out scores: row statistics of logits, sums of an RBF kernel.
#include "gemm_run.h"

namespace pbt {

int gemm_head_piece(int M, int N, int K, int batch) { return gl_shape(gl_choose(M, N, K, batch, EpiHeadStats::HEAVY, false, K > N ? K : N)).bn == 64 ? 32 : 64; }
hipError_t gemm_head_stats(const GemmOperands& o, const float* bias, int64_t sbias, const int32_t* targets, float2* stats, float* target_logit,
                           int pieces, hipStream_t s) {
  if (o.a_m_contig || o.b_k_contig) return hipErrorInvalidValue;
  return run_gemm(o, EpiHeadStats{bias, sbias, targets, stats, target_logit, o.M, pieces}, s);
}
hipError_t gemm_rbf_sum(const GemmOperands& o, const float* na, int64_t sna, const float* nb, int64_t snb, float inv2d,
                        float* partial, int* tiles, hipStream_t s) {
  // tile count as the launch will choose it (the caller sizes `partial` with gemm_rbf_tiles, an upper bound)
  GemmOperands q = o;
  TileShape t{64, 64};   // of the kernel that takes longer rows, where a symmetric product is formed whole
  if (gemm_rows_fit_lds(o)) t = gl_shape(gl_choose(o.M, o.N, o.K, o.batch, EpiRbfSum::HEAVY, true, o.lda > o.ldb ? o.lda : o.ldb, o.symmetric));
  else q.symmetric = 0;
  *tiles = q.symmetric ? gl_upper_tiles(o.N, t) : ((o.M + t.bm - 1) / t.bm) * ((o.N + t.bn - 1) / t.bn);
  return run_gemm(q, EpiRbfSum{na, sna, nb, snb, inv2d, partial}, s);
}
int gemm_rbf_tiles(int M, int N, int) {
  return ((M + 63) / 64) * ((N + 63) / 64);  // the smallest tile gives the most partial sums
}

}  // namespace pbt
