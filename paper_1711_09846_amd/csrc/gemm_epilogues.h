// What the GEMM does with its accumulators: functors that receive runs of 8 consecutive columns of one row.
//
// begin(member) moves a functor's pointers to the member's arrays; `o` is the run's offset in them, m * pitch() + n.  FULL: the run has all
// eight columns, and vectors() said that 16-byte accesses are aligned; otherwise `count` columns exist and the accesses are chosen per run.
// cols: what load_cols read for the lane's eight columns (the same for every run the lane handles).  data: what load_run read for
// this run, requested before the accumulators are staged (read inside put, after the stores of the run before, every run paid a
// memory latency of its own).
#pragma once
#include "gemm_common.h"

namespace pbt {

struct NoData {};
// the functors without columns, data or a closing step inherit these
struct EpiPlain {
  static constexpr bool HAS_FINISH = false;
  static constexpr bool COLSUM = false;   // weight gradients: the bias gradient can ride along
  static constexpr bool HAS_COLS = false;
  static constexpr bool HAS_DATA = false;
  static constexpr bool PREFETCH = false; // reads what it updates (the optimiser, in the kernel that stages through registers)
  static constexpr bool HEAVY = false;    // a long epilogue (gl_choose)
  static constexpr bool ROWWISE = false;  // put exchanges between the lanes of a row: every lane calls it, count 0 where nothing of the run exists
  typedef NoData Data;
  struct Fetched {};
  __device__ __forceinline__ void load_cols(int, int, float*) const {}
  __device__ __forceinline__ Data load_run(int, int, int64_t, int) const { return {}; }
};
// the biases of eight columns, zero past N
__device__ __forceinline__ void load_bias8(const float* bias, int n, int N, float* b) {
  if (n + 8 <= N && aligned16(bias + n)) {
    const float4 lo = *reinterpret_cast<const float4*>(bias + n), hi = *reinterpret_cast<const float4*>(bias + n + 4);
    b[0] = lo.x; b[1] = lo.y; b[2] = lo.z; b[3] = lo.w; b[4] = hi.x; b[5] = hi.y; b[6] = hi.z; b[7] = hi.w;
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) b[e] = n + e < N ? bias[n + e] : 0.f;
  }
}
template <bool FULL>
__device__ __forceinline__ void store_f32_run(float* dst, const float* v, int count) {
  if (FULL || (count == 8 && aligned16(dst))) {
    *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4*>(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (e < count) dst[e] = v[e];
  }
}
template <bool FULL>
__device__ __forceinline__ void store_run(bf16_t* dst, const float* v, int count) {
  if (FULL) *reinterpret_cast<uint4*>(dst) = pack_bf16x8(v);
  else store_bf16_run(dst, v, count);
}
struct EpiStoreF32 : EpiPlain {
  static constexpr bool COLSUM = true;
  static constexpr int LAYOUTS = 15;
  float* C;
  int64_t ldc, sc;
  __host__ __device__ EpiStoreF32(float* c, int64_t l, int64_t s) : C(c), ldc(l), sc(s) {}
  __device__ __forceinline__ void begin(int member) { C += (int64_t)member * sc; }
  __device__ __forceinline__ int64_t pitch() const { return ldc; }
  __device__ __forceinline__ bool vectors() const { return aligned16(C) && ldc % 4 == 0; }
  template <bool FULL>
  __device__ __forceinline__ void put(int, int, int64_t o, const float* v, int count, const float*, const Data&) const {
    store_f32_run<FULL>(C + o, v, count);
  }
};

struct EpiStoreBF16 : EpiPlain {
  static constexpr int LAYOUTS = 15;
  bf16_t* C;
  int64_t ldc, sc;
  int inner;       // two-level batch index as in GemmArgs
  int64_t sc_in;
  __host__ __device__ EpiStoreBF16(bf16_t* c, int64_t l, int64_t s, int in = 1, int64_t s_in = 0) : C(c), ldc(l), sc(s), inner(in), sc_in(s_in) {}
  __device__ __forceinline__ void begin(int member) {
    if (inner == 1) C += (int64_t)member * sc;
    else C += (int64_t)(member / inner) * sc + (int64_t)(member % inner) * sc_in;
  }
  __device__ __forceinline__ int64_t pitch() const { return ldc; }
  __device__ __forceinline__ bool vectors() const { return aligned16(C) && ldc % 8 == 0; }
  template <bool FULL>
  __device__ __forceinline__ void put(int, int, int64_t o, const float* v, int count, const float*, const Data&) const {
    store_run<FULL>(C + o, v, count);
  }
};

// Output layer over a large vocabulary: logits = acc + b[n], kept in float.  (Streaming stores for the logits made
// this launch 4 % faster and the two that follow it slower by more: plain stores.)
struct EpiBiasF32 : EpiPlain {
  static constexpr bool HAS_COLS = true;
  static constexpr int LAYOUTS = 1;
  const float* bias;
  int64_t sbias;
  float* C;
  int64_t ldc, sc;
  __host__ __device__ EpiBiasF32(const float* b, int64_t sb, float* c, int64_t l, int64_t s) : bias(b), sbias(sb), C(c), ldc(l), sc(s) {}
  __device__ __forceinline__ void begin(int member) { bias += (int64_t)member * sbias; C += (int64_t)member * sc; }
  __device__ __forceinline__ int64_t pitch() const { return ldc; }
  __device__ __forceinline__ bool vectors() const { return aligned16(C) && ldc % 4 == 0; }
  __device__ __forceinline__ void load_cols(int n, int N, float* b) const { load_bias8(bias, n, N, b); }
  template <bool FULL>
  __device__ __forceinline__ void put(int, int, int64_t o, const float* v, int count, const float* b, const Data&) const {
    float z[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) z[e] = v[e] + b[e];
    store_f32_run<FULL>(C + o, z, count);
  }
};

// The same output layer where only the cross-entropy is wanted (held-out loss): the float logits stay in registers.  Of every row
// and piece of 8 RUNS columns (64, or 32 with the narrow tile) the largest logit m and the sum of exp(logit - m) go to
// stats[row][piece], the target's logit to target_logit[row]; a later pass puts a row's pieces together.  16 members x 4096 rows x 8192
// logits: writing and re-reading 2.1 GB of logits cost 1161 + 388 us per chunk.
// RUNS neighbouring lanes hold a row's piece; they exchange through the data-parallel modifiers of the vector instructions.
template <int CTRL>
__device__ __forceinline__ float lane_swap(float x) {
  return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), CTRL, 0xf, 0xf, true));
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141;   // quad_perm [1,0,3,2], [2,3,0,1]; lane i <- 7 - i of its eight
struct EpiHeadStats : EpiPlain {
  static constexpr bool HAS_COLS = true, HAS_DATA = true, ROWWISE = true, HEAVY = true;
  static constexpr int LAYOUTS = 1;
  struct Data { int y = 0; };
  const float* bias;
  int64_t sbias;
  const int32_t* targets;   // [batch][M]
  float2* stats;            // [batch][M][pieces]
  float* target_logit;      // [batch][M]
  int M, pieces;
  __host__ __device__ EpiHeadStats(const float* b, int64_t sb, const int32_t* t, float2* s, float* tl, int m, int p)
      : bias(b), sbias(sb), targets(t), stats(s), target_logit(tl), M(m), pieces(p) {}
  __device__ __forceinline__ void begin(int member) {
    bias += (int64_t)member * sbias;
    targets += (int64_t)member * M;
    stats += (int64_t)member * M * pieces;
    target_logit += (int64_t)member * M;
  }
  __device__ __forceinline__ int64_t pitch() const { return pieces; }
  __device__ __forceinline__ bool vectors() const { return true; }
  __device__ __forceinline__ void load_cols(int n, int N, float* b) const { load_bias8(bias, n, N, b); }
  __device__ __forceinline__ Data load_run(int m, int, int64_t, int) const { return {targets[m]}; }
  template <bool FULL, int RUNS>
  __device__ __forceinline__ void put_row(int m, int n, const float* v, int count, const float* b, const Data& data) const {
    float l[8], mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      l[e] = v[e] + b[e];
      if (FULL || e < count) mx = fmaxf(mx, l[e]);
    }
    mx = fmaxf(mx, lane_swap<DPP_XOR1>(mx));
    mx = fmaxf(mx, lane_swap<DPP_XOR2>(mx));
    if (RUNS == 8) mx = fmaxf(mx, lane_swap<DPP_HALF_MIRROR>(mx));
    const float base = mx == -INFINITY ? 0.f : mx;   // (a piece of nothing but -inf has the sum 0)
    float se = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) se += FULL || e < count ? expf(l[e] - base) : 0.f;
    se += lane_swap<DPP_XOR1>(se);
    se += lane_swap<DPP_XOR2>(se);
    if (RUNS == 8) se += lane_swap<DPP_HALF_MIRROR>(se);
    if (FULL || count > 0) {
      const int y = data.y - n;
      if ((unsigned)y < (unsigned)(FULL ? 8 : count)) {
        float t = l[0];
#pragma unroll
        for (int e = 1; e < 8; ++e) t = y == e ? l[e] : t;
        target_logit[m] = t;
      }
      if (n % (8 * RUNS) == 0) stats[(int64_t)m * pieces + n / (8 * RUNS)] = make_float2(mx, se);
    }
  }
};

// Forward layer: z = acc + b[n]; stores z (for the backward pass, may be null) and act(z), both bf16.
template <int ACT>
struct EpiBiasAct : EpiPlain {
  static constexpr bool HAS_COLS = true, HEAVY = ACT == ACT_GELU || ACT == ACT_TANH;
  static constexpr int LAYOUTS = 1;
  const float* bias;  // + member * sbias + n
  int64_t sbias;
  bf16_t* Z;
  bf16_t* Aout;
  int64_t ld, so;
  __host__ __device__ EpiBiasAct(const float* b, int64_t sb, bf16_t* z, bf16_t* a, int64_t l, int64_t s) : bias(b), sbias(sb), Z(z), Aout(a), ld(l), so(s) {}
  __device__ __forceinline__ void begin(int member) {
    bias += (int64_t)member * sbias;
    if (Z) Z += (int64_t)member * so;
    Aout += (int64_t)member * so;
  }
  __device__ __forceinline__ int64_t pitch() const { return ld; }
  __device__ __forceinline__ bool vectors() const { return aligned16(Z) && aligned16(Aout) && ld % 8 == 0; }
  __device__ __forceinline__ void load_cols(int n, int N, float* b) const { load_bias8(bias, n, N, b); }
  template <bool FULL>
  __device__ __forceinline__ void put(int, int, int64_t o, const float* v, int count, const float* b, const Data&) const {
    float z[8], a[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) z[e] = FULL || e < count ? v[e] + b[e] : 0.f;
    act_fwd8(z, a, ACT);
    if (Z) store_run<FULL>(Z + o, z, count);
    store_run<FULL>(Aout + o, a, count);
  }
};

// Forward layer followed by a dropout site: the stored activation is act(acc + b[n]), rounded, times the keep factor
// of its element (Philox block (m ld + n) / 4 of the site, as the stand-alone dropout kernel draws it), rounded
// again; the keep bits go to the site's record (bit e % 8 of byte e / 8 of the member's [rows][ld] array).  N and ld
// are multiples of 8 and the arrays 16-byte aligned, so every run has eight columns.
template <int ACT>
struct EpiBiasActDrop : EpiPlain {
  static constexpr bool HAS_COLS = true, HEAVY = true;
  static constexpr int LAYOUTS = 1;
  const float* bias;
  int64_t sbias;
  bf16_t* Aout;
  int64_t ld, so;
  uint8_t* rec;
  int64_t rec_stride;   // bytes of record per member
  DropArgs drop;
  int site;
  int member_ = 0;
  DropRate rate = {0u, 1.f};
  __host__ __device__ EpiBiasActDrop(const float* b, int64_t sb, bf16_t* a, int64_t l, int64_t s, uint8_t* r, int64_t rs, const DropArgs& d, int si)
      : bias(b), sbias(sb), Aout(a), ld(l), so(s), rec(r), rec_stride(rs), drop(d), site(si) {}
  __device__ __forceinline__ void begin(int member) {
    bias += (int64_t)member * sbias;
    Aout += (int64_t)member * so;
    rec += (int64_t)member * rec_stride;
    rate = drop_rate(drop.H, drop.n_hyper, drop.col, member, drop.active);
    member_ = member;
  }
  __device__ __forceinline__ int64_t pitch() const { return ld; }
  __device__ __forceinline__ bool vectors() const { return true; }
  __device__ __forceinline__ void load_cols(int n, int N, float* b) const { load_bias8(bias, n, N, b); }
  template <bool FULL>
  __device__ __forceinline__ void put(int, int, int64_t o, const float* v, int, const float* b, const Data&) const {
    float z[8], a[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) z[e] = v[e] + b[e];
    act_fwd8(z, a, ACT);
    const uint32_t b0 = drop_bits4(drop, rate, member_, site, (uint32_t)(o >> 2)), b1 = drop_bits4(drop, rate, member_, site, (uint32_t)(o >> 2) + 1u);
    const uint32_t bits = b0 | (b1 << 4);
    *reinterpret_cast<uint4*>(Aout + o) = keep_times_scale(a, bits, rate.scale);
    rec[o >> 3] = (uint8_t)bits;
  }
};

// Input gradient: dz_prev = acc * act'(z_prev), bf16.  DROP: the result is then multiplied by the keep factor of the site that followed
// the activation in the forward pass: the value is rounded to bf16, multiplied by 0 or by the member's scale (the float nearest 1 / (1 - p), p from
// column col of H) in double, and rounded once more.  The record holds one bit per element of the member's [rows][ld]
// array (bit e % 8 of byte e / 8), as the forward pass of that site left it; N and ld are multiples of 8 then.
template <int ACT, bool DROP>
struct EpiDgradAct : EpiPlain {
  static constexpr bool HAS_DATA = true, HEAVY = true;
  static constexpr int LAYOUTS = DROP ? 2 : 3;
  struct Data { uint4 z = {0u, 0u, 0u, 0u}; uint32_t bits = 0u; };
  const bf16_t* Zprev;
  bf16_t* dZ;
  int64_t ld, so;
  const uint8_t* mask;
  int64_t mask_stride;       // bytes of record per member
  const float* H;
  int n_hyper, col;
  float scale = 1.f;
  __host__ __device__ EpiDgradAct(const bf16_t* z, bf16_t* d, int64_t l, int64_t s, const uint8_t* m, int64_t ms, const float* h, int nh, int c)
      : Zprev(z), dZ(d), ld(l), so(s), mask(m), mask_stride(ms), H(h), n_hyper(nh), col(c) {}
  __device__ __forceinline__ void begin(int member) {
    Zprev += (int64_t)member * so; dZ += (int64_t)member * so;
    if constexpr (DROP) {
      mask += (int64_t)member * mask_stride;
      const float p = col >= 0 ? H[(int64_t)member * n_hyper + col] : 0.f;
      scale = p > 0.f ? (float)(1.0 / (1.0 - (double)p)) : 1.f;
    }
  }
  __device__ __forceinline__ int64_t pitch() const { return ld; }
  __device__ __forceinline__ bool vectors() const { return aligned16(Zprev) && aligned16(dZ) && ld % 8 == 0; }
  __device__ __forceinline__ Data load_run(int, int, int64_t o, int count) const {
    Data r;
    if constexpr (DROP) r.bits = mask[o >> 3];
    if (count == 8 && aligned16(Zprev + o)) { r.z = *reinterpret_cast<const uint4*>(Zprev + o); return r; }
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (e < count) w[e >> 1] |= (uint32_t)Zprev[o + e] << (16 * (e & 1));
    r.z = make_uint4(w[0], w[1], w[2], w[3]);
    return r;
  }
  template <bool FULL>
  __device__ __forceinline__ void put(int, int, int64_t o, const float* v, int count, const float*, const Data& run) const {
    float z[8], d[8];
    unpack_bf16x8(run.z, z);
    act_bwd_scale8(v, z, d, ACT);
    if constexpr (DROP) *reinterpret_cast<uint4*>(dZ + o) = keep_times_scale(d, run.bits, scale);
    else store_run<FULL>(dZ + o, d, count);
  }
};

// Sum over the tile of exp(-(|a_m|^2 + |b_n|^2 - 2 a_m.b_n) / (2 d)): the RBF kernel of the MMD
// score evaluated on the Gram tile while it is still in the accumulators.  Every thread adds its
// elements in a fixed order, the wavefront and then the wavefronts are combined in a fixed
// order, and the tile's sum goes to partial[member][tile]; a later pass adds the tiles.
// Of a symmetric product (a = b) only the tiles at and right of the diagonal are computed: an element right of the diagonal counts
// twice, one left of it (inside a tile on the diagonal) not at all.  32 members of 2048 x 784: 397 us as all tiles, 205 as
// those that reach the diagonal.
struct EpiRbfSum : EpiPlain {
  static constexpr bool HAS_FINISH = true, HAS_COLS = true, HAS_DATA = true, HEAVY = true;
  static constexpr int LAYOUTS = 2;
  struct Data { float na = 0.f; };
  const float* na;  // squared norms of the A rows, + member * sna
  int64_t sna;
  const float* nb;
  int64_t snb;
  float inv2d;
  float* partial;
  float sum = 0.f;
  int region = 0;         // 0: every element once, 1: tile on the diagonal of a symmetric product, 2: right of it
  __host__ __device__ EpiRbfSum(const float* a, int64_t sa, const float* b, int64_t sb, float i2d, float* p) : na(a), sna(sa), nb(b), snb(sb), inv2d(i2d), partial(p) {}
  __device__ __forceinline__ void begin(int member) { na += (int64_t)member * sna; nb += (int64_t)member * snb; }
  __device__ __forceinline__ int64_t pitch() const { return 0; }
  __device__ __forceinline__ bool vectors() const { return region != 1; }
  __device__ __forceinline__ void load_cols(int n, int N, float* b) const { load_bias8(nb, n, N, b); }
  __device__ __forceinline__ Data load_run(int m, int, int64_t, int) const { return {na[m]}; }
  template <bool FULL>
  __device__ __forceinline__ void put(int m, int n, int64_t, const float* v, int count, const float* b, const Data& row) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float k = expf(-(row.na + b[e] - 2.f * v[e]) * inv2d);
      if (FULL) {   // (not on the diagonal)
        sum = fmaf(region == 0 ? 1.f : 2.f, k, sum);
      } else {
        const float weight = region == 0 ? 1.f : region == 2 || n + e > m ? 2.f : n + e == m ? 1.f : 0.f;
        if (e < count && weight != 0.f) sum = fmaf(weight, k, sum);
      }
    }
  }
  // wsum: LDS of the workgroup that nothing else uses
  __device__ __forceinline__ void finish(int member, int tile, int tiles, float* wsum) {
    const float w = wave_sum(sum);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = w;
    __syncthreads();
    if (threadIdx.x == 0) {
      float t = wsum[0];
      for (unsigned k = 1; k < blockDim.x / 64; ++k) t += wsum[k];
      partial[(int64_t)member * tiles + tile] = t;
    }
  }
};

}  // namespace pbt
