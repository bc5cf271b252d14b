// What the two population-batched GEMM kernels share: arguments, the order of tiles, 16-byte bf16 runs.
#pragma once
#include <type_traits>

#include "common.h"
#include "dropout.h"
#include "gemm_choose.h"
#include "optim_math.h"
#include "per_device.h"

namespace pbt {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;

// n / d for 0 <= n < 2^31 and a d >= 1 that is known at the launch: with l = ceil(log2 d) and mul = floor(2^(31 + l) / d) + 1, which is below 2^32,
// n * mul exceeds n * 2^(31 + l) / d by at most n * 2^l / d < 2^(31 + l) / d.  (A division by a kernel argument is 25 dependent scalar instructions; a tile
// needs four before its first load.)
struct Divisor {
  uint32_t mul = 0x80000001u, shift = 31;
  Divisor() = default;
  explicit Divisor(int d) {
    int l = 0;
    while ((int64_t)1 << l < d) ++l;
    shift = (uint32_t)(31 + l);
    mul = (uint32_t)((((uint64_t)1 << shift) / (uint32_t)d) + 1);
  }
  __device__ __forceinline__ int divide(int n) const { return (int)(((uint64_t)(uint32_t)n * mul) >> shift); }
};

struct GemmArgs {
  const bf16_t* A;
  int64_t lda, sa;
  const bf16_t* B;
  int64_t ldb, sb;
  int M, N, K, batch;
  int tiles_m, tiles_n;
  // two-level batch index (attention: outer = sequence, inner = head): the operand of batch element b
  // starts at (b / inner) * s? + (b % inner) * s?_in
  int inner;
  int64_t sa_in, sb_in;
  // optional by-product: colsum[b * colsum_stride + n] = sum_k B[k][n] (float), written by the first tile
  // row of every batch element from the B slabs it stages anyway (the bias gradient of a weight-gradient
  // contraction, whose B operand is dZ); null = not wanted
  float* colsum = nullptr;
  int64_t colsum_stride = 0;
  int colsum_k = 0;   // the column sums run over k < colsum_k (the launcher sets K when the caller gives no limit)
  int upper = 0;      // RBF sums only: C is symmetric, only the tiles that reach the diagonal or lie right of it are computed
  int tiles = 0;      // tiles per batch element (set by the launcher)
  // (set by the launcher) by tiles, by the tiles of a group of tile rows, by the rows of the last group, by inner
  Divisor by_tiles, by_group, by_last, by_inner;
  int b_cols = 0;     // columns of an N-contiguous B that may be read (N, or more where the rows are padded with zeros)
};

// Workgroups are handed to the 8 XCDs round-robin by linear id.  Remap the id
// so that each XCD works on a contiguous run of tiles (neighbouring tiles
// share an A or B slab, which then stays in that XCD's L2).
__device__ __forceinline__ int xcd_remap(int id, int total) {
  constexpr int XCDS = 8;
  const int per = total / XCDS;
  if (id >= per * XCDS) return id;  // ragged tail keeps its place
  return (id % XCDS) * per + id / XCDS;
}

// Tile order inside one batch element: tiles are numbered down groups of GROUP_M tile rows, so that the
// workgroups resident on an XCD at one time (consecutive numbers) form a block of tiles that shares
// few A and B slabs and keeps them in that XCD's L2.
constexpr int GROUP_M = 8;

// A kernel's permission to use more than 64 KB of LDS belongs to the device that is current when it is given.
template <auto Kernel>
hipError_t allow_lds(int bytes) {
  static std::atomic<uint64_t> allowed{0};   // devices that have it
  int device = 0;
  const hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return e;
  return once_per_device(allowed, device, [&] { return hipFuncSetAttribute(reinterpret_cast<const void*>(Kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes); });
}

__device__ __forceinline__ uint4 pack_bf16x8(const float* v) {
  return make_uint4(f2bf_pair(v[0], v[1]), f2bf_pair(v[2], v[3]), f2bf_pair(v[4], v[5]), f2bf_pair(v[6], v[7]));
}
__device__ __forceinline__ void unpack_bf16x8(uint4 p, float* v) {
  const uint32_t w[4] = {p.x, p.y, p.z, p.w};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    v[2 * q] = __uint_as_float(w[q] << 16);
    v[2 * q + 1] = __uint_as_float(w[q] & 0xffff0000u);
  }
}
__device__ __forceinline__ bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

__device__ __forceinline__ void store_bf16_run(bf16_t* dst, const float* v, int count) {
  if (count == 8 && aligned16(dst)) {
    *reinterpret_cast<uint4*>(dst) = pack_bf16x8(v);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (e < count) dst[e] = f2bf(v[e]);
  }
}


}  // namespace pbt
