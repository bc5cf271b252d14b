// Fully fused fp32 population step for networks small enough to live in LDS: one workgroup per
// member gathers its mini-batch, runs forward, softmax cross-entropy, backward and the optimiser
// update, for n_steps consecutive steps, touching HBM only for the data rows.  Members are
// independent between exploit points (Algorithm 1 of the PBT paper), so no grid-wide
// synchronisation is needed and one launch covers a whole ready interval.
//
// Row pitches in LDS are (width + 1) floats so that both "lanes along the batch" and "lanes
// along the features" access patterns are free of bank conflicts.
#include <algorithm>

#include "common.h"
#include "internal.h"
#include "optim_math.h"
#include "philox.h"

namespace pbt {

size_t fused_small_plan(FusedSmallArgs& a, bool for_eval) {
  int off = 0;
  a.lds_w = off; off += (int)a.stride;
  a.lds_s0 = a.lds_s1 = 0;
  if (!for_eval) {
    a.lds_s0 = off; off += (int)a.stride;
    if (a.optimizer == 1) { a.lds_s1 = off; off += (int)a.stride; }
  }
  int maxd = 0;
  for (int l = 0; l < a.n_layers; ++l) {
    a.lds_a[l] = off; off += a.B * (a.dims[l] + 1);
    a.lds_z[l] = off; off += a.B * (a.dims[l + 1] + 1);
    if (a.dims[l + 1] > maxd) maxd = a.dims[l + 1];
    if (a.dims[l] > maxd) maxd = a.dims[l];
  }
  a.lds_dz[0] = a.lds_dz[1] = 0;
  if (!for_eval) {
    a.lds_dz[0] = off; off += a.B * (maxd + 1);
    a.lds_dz[1] = off; off += a.B * (maxd + 1);
  }
  a.lds_rowloss = off; off += a.B;
  a.lds_y = off; off += a.B;
  a.lds_total = off;
  return (size_t)off * sizeof(float);
}

constexpr int FS_THREADS = 256;

// Forward through all layers for the B rows whose inputs sit in lds_a[0]; leaves logits in
// lds_z[L-1] and per-row losses in lds_rowloss.
// (The sums of the plain form are chains of two LDS reads and a multiply-add, in order.  Unrolled eight times the reads of several terms are on their way; as
// loops of two terms they took 157 or 172 us per step of 8 members 40-50-17 with 128 rows, as the code around them shifted their alignment; 85 now.)
__device__ __forceinline__ void fs_forward(const FusedSmallArgs& a, float* lds, int nrows) {
  const int tid = threadIdx.x;
  const float* W = lds + a.lds_w;
  for (int l = 0; l < a.n_layers; ++l) {
    const int K = a.dims[l], N = a.dims[l + 1];
    const float* in = lds + a.lds_a[l];
    float* z = lds + a.lds_z[l];
    const float* Wl = W + a.w_off[l];
    const float* bl = W + a.b_off[l];
    for (int idx = tid; idx < nrows * N; idx += FS_THREADS) {
      const int b = idx / N, n = idx - b * N;
      float acc = 0.f;
#pragma unroll 8
      for (int k = 0; k < K; ++k) acc = fmaf(in[b * (K + 1) + k], Wl[k * N + n], acc);
      acc += bl[n];
      z[b * (N + 1) + n] = acc;
      if (l < a.n_layers - 1) lds[a.lds_a[l + 1] + b * (N + 1) + n] = act_fwd(acc, a.act);
    }
    __syncthreads();
  }
}

// Softmax cross-entropy per row; when dz != null also (softmax - onehot) * gscale into dz (pitch C+1).
__device__ __forceinline__ void fs_loss(const FusedSmallArgs& a, float* lds, int nrows, float* dz, float gscale) {
  const int C = a.dims[a.n_layers];
  const float* logits = lds + a.lds_z[a.n_layers - 1];
  const int* y = reinterpret_cast<const int*>(lds + a.lds_y);
  for (int b = threadIdx.x; b < nrows; b += FS_THREADS) {
    const float* lg = logits + b * (C + 1);
    // log-sum-exp with the largest term split off: lse = mx + log1p(sum of the others), which
    // keeps full relative accuracy when one class dominates (small losses)
    float mx = lg[0];
    int cm = 0;
    for (int c = 1; c < C; ++c)
      if (lg[c] > mx) { mx = lg[c]; cm = c; }
    float rest = 0.f;
    for (int c = 0; c < C; ++c)
      if (c != cm) rest += expf(lg[c] - mx);
    const float l1p = log1pf(rest);
    const int yb = y[b];
    lds[a.lds_rowloss + b] = l1p + (mx - lg[yb]);
    if (dz) {
      const float inv = 1.f / (1.f + rest);
      // softmax_y - 1 = -(sum of the other classes' terms) / S: no cancellation when softmax_y -> 1
      float others = (yb == cm) ? 0.f : 1.f;
      for (int c = 0; c < C; ++c)
        if (c != yb && c != cm) others += expf(lg[c] - mx);
      for (int c = 0; c < C; ++c)
        dz[b * (C + 1) + c] = (c == yb ? -others * inv : expf(lg[c] - mx) * inv) * gscale;
    }
  }
  __syncthreads();
}

__device__ __forceinline__ float fs_sum_rowloss(const float* lds_rowloss, int nrows) {
  // first wavefront: lane adds rows lane, lane+64, ... then butterfly; valid in wave 0 only
  float acc = 0.f;
  for (int r = threadIdx.x & 63; r < nrows; r += 64) acc += lds_rowloss[r];
  return wave_sum(acc);
}

__global__ __launch_bounds__(FS_THREADS) void fused_small_step_kernel(FusedSmallArgs a) {
  extern __shared__ float lds[];
  const int i = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int64_t base = (int64_t)i * a.stride;
  const int n = (int)a.stride;
  float* W = lds + a.lds_w;
  float* S0 = lds + a.lds_s0;
  float* S1 = lds + a.lds_s1;
  for (int j = tid; j < n; j += FS_THREADS) {
    W[j] = a.W32[base + j];
    S0[j] = a.S0[base + j];
    if (a.optimizer == 1) S1[j] = a.S1[base + j];
  }
  const float* h = a.H + (int64_t)i * a.n_hyper;
  const float lr = h[a.col_lr];
  const float b1 = (a.optimizer == 1 && a.col_beta1 >= 0) ? h[a.col_beta1] : a.c0;
  const float wd = (a.optimizer == 1 && a.col_wd >= 0) ? h[a.col_wd] : a.c3;
  int t = a.t[i];
  const uint32_t k0 = (uint32_t)a.seed, k1 = (uint32_t)(a.seed >> 32);
  const int L = a.n_layers, B = a.B, d0 = a.dims[0];
  int* ylds = reinterpret_cast<int*>(lds + a.lds_y);
  float last_loss = 0.f;
  __syncthreads();

  for (int s = 0; s < a.n_steps; ++s) {
    const uint32_t step = a.step0 + (uint32_t)s;
    ++t;
    // mini-batch rows (Philox domain 1), one wavefront per row
    for (int r = wave; r < B; r += FS_THREADS / 64) {
      const uint32_t x = philox4x32_10(step, (uint32_t)i, DOMAIN_BATCH, (uint32_t)r, k0, k1).x;
      const int64_t src = (int64_t)philox_bounded(x, (uint32_t)a.n_rows);
      for (int c = lane; c < d0; c += 64) lds[a.lds_a[0] + r * (d0 + 1) + c] = a.x[src * d0 + c];
      if (lane == 0) ylds[r] = a.y[src];
    }
    __syncthreads();
    fs_forward(a, lds, B);
    float* dz = lds + a.lds_dz[0];
    float* dprev = lds + a.lds_dz[1];
    fs_loss(a, lds, B, dz, 1.f / (float)B);
    if (wave == 0) last_loss = fs_sum_rowloss(lds + a.lds_rowloss, B) / (float)B;

    float inv_bc1 = 1.f, inv_bc2 = 1.f;
    if (a.optimizer == 1) {
      inv_bc1 = 1.f / (1.f - powf(b1, (float)t));
      inv_bc2 = 1.f / (1.f - powf(a.c1, (float)t));
    }
    for (int l = L - 1; l >= 0; --l) {
      const int K = a.dims[l], N = a.dims[l + 1];
      const float* in = lds + a.lds_a[l];
      float* Wl = W + a.w_off[l];
      // input gradient first: it needs W_l from before the update
      if (l > 0) {
        const float* zp = lds + a.lds_z[l - 1];
        for (int idx = tid; idx < B * K; idx += FS_THREADS) {
          const int k = idx / B, b = idx - k * B;  // lanes along the batch
          float acc = 0.f;
#pragma unroll 8
          for (int nn = 0; nn < N; ++nn) acc = fmaf(dz[b * (N + 1) + nn], Wl[k * N + nn], acc);
          dprev[b * (K + 1) + k] = acc * act_bwd(zp[b * (K + 1) + k], a.act);
        }
      }
      __syncthreads();
      // weight and bias gradient, optimiser update in place (idx < K*N: weights; then N biases)
      for (int idx = tid; idx < K * N + N; idx += FS_THREADS) {
        float g = 0.f;
        int p;
        if (idx < K * N) {
          const int k = idx / N, nn = idx - k * N;
#pragma unroll 8
          for (int b = 0; b < B; ++b) g = fmaf(in[b * (K + 1) + k], dz[b * (N + 1) + nn], g);
          p = a.w_off[l] + idx;
        } else {
          const int nn = idx - K * N;
#pragma unroll 8
          for (int b = 0; b < B; ++b) g += dz[b * (N + 1) + nn];
          p = a.b_off[l] + nn;
        }
        if (s == a.n_steps - 1) a.G[base + p] = g;
        float w = W[p];
        if (a.optimizer == 0) {
          const float v = a.c0 * S0[p] + g;
          S0[p] = v;
          w = w - lr * v;
        } else if (a.optimizer == 1) {
          const float m = b1 * S0[p] + (1.f - b1) * g;
          const float v = a.c1 * S1[p] + (1.f - a.c1) * g * g;
          S0[p] = m;
          S1[p] = v;
          w = w - lr * ((m * inv_bc1) / (sqrtf(v * inv_bc2) + a.c2) + wd * w);
        } else {
          const float v = a.c0 * S0[p] + (1.f - a.c0) * g * g;
          S0[p] = v;
          w = w - lr * g / sqrtf(v + a.c1);
        }
        W[p] = w;
      }
      __syncthreads();
      float* tmp = dz; dz = dprev; dprev = tmp;
    }
  }
  for (int j = tid; j < n; j += FS_THREADS) {
    a.W32[base + j] = W[j];
    a.S0[base + j] = S0[j];
    if (a.optimizer == 1) a.S1[base + j] = S1[j];
  }
  if (tid == 0) {
    a.t[i] = t;
    a.loss[i] = last_loss;
  }
}

// ---- tiled form ------------------------------------------------------------------------------------------------
// The same step with every contraction on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands and accumulation).
// What bounds the plain form above is LDS reads (two per multiply-add) and wavefronts that wait for each other's and the
// data rows' latencies: 63 us per step of a 32-64-4 network with 64 rows.  Here an operand is read once per 16
// multiply-adds, every array is padded to whole 16 x 16 blocks (so no loop has a remainder), wavefronts of their own
// fetch the rows of step s + 1 while the others compute step s (four and twelve of them, fewer in large populations: ft_size()), and phases that do not depend on each other share a
// barrier interval: 2 L barriers per step of an L-layer network.  5.3 us per step (50 steps in one launch: 3.13 -> 0.27 ms);
// what is left is instruction issue and LDS latency of the chain fragment -> MFMA -> activation -> fragment of each
// interval.  The optimiser and the number of layers are template parameters: as branches inside the element loops they cost
// a third of the time, and with the rows' loads in the computing wavefronts every loop waited for them.
// LDS pitch of a padded array: 16-wide blocks plus 4 floats.  Pitch / 4 is odd, so the 16 rows x 4 columns of a fragment
// whose lanes walk down rows fall on 64 different banks; one whose lanes walk along a row reads runs of 16.
__host__ __device__ inline int fs_pad(int w) { return (w + 15) & ~15; }
__host__ __device__ inline int fs_pitch(int w) { return fs_pad(w) + 4; }

constexpr int FT_EVAL_ROWS = 64;    // held-out rows per workgroup: four wavefronts of 16 rows each

size_t fused_tiled_plan(FusedSmallArgs& a, bool for_eval) {
  int off = 0;
  for (int l = 0; l < a.n_layers; ++l) {
    a.lt_w[l] = off; off += fs_pad(a.dims[l]) * fs_pitch(a.dims[l + 1]);
    a.lt_b[l] = off; off += fs_pad(a.dims[l + 1]);
  }
  if (for_eval) {
    int maxp = 0;
    for (int l = 0; l <= a.n_layers; ++l) maxp = fs_pitch(a.dims[l]) > maxp ? fs_pitch(a.dims[l]) : maxp;
    a.lt_pitch = maxp;
    a.lt_a[0] = off; off += FT_EVAL_ROWS * maxp;
    a.lt_a[1] = off; off += FT_EVAL_ROWS * maxp;
    a.lt_total = off;
    return (size_t)off * sizeof(float);
  }
  a.lt_s0 = off; off += (int)a.stride;
  a.lt_s1 = off; if (a.optimizer == 1) off += (int)a.stride;
  const int rows = fs_pad(a.B);
  a.lt_x[0] = off; off += rows * fs_pitch(a.dims[0]);
  a.lt_x[1] = off; off += rows * fs_pitch(a.dims[0]);
  for (int l = 0; l < a.n_layers; ++l) {
    a.lt_a[l + 1] = off; if (l + 1 < a.n_layers) off += rows * fs_pitch(a.dims[l + 1]);
    a.lt_d[l] = off; off += rows * fs_pitch(a.dims[l + 1]);   // z (GELU), logits, then the gradient with respect to z
  }
  a.lt_y = off; off += 2 * rows;
  a.lt_rowloss = off; off += rows;
  a.lt_sc = off; off += 4;
  a.lt_total = off;
  if (rows * a.dims[0] > 65535) return SIZE_MAX;   // (ft_div's range)
  a.lt_inv_d0 = (uint32_t)(((1ull << 32) + a.dims[0] - 1) / a.dims[0]);
  return (size_t)off * sizeof(float);
}

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// One 16 x 16 block of A B over k < KP (a multiple of 16: the padding is zero in at least one operand).  pa / pb point at
// the lane's row or column (lane % 16) of the operand at k = 0; sa / sb are the steps along k (AC / BC: 1, and 16-byte aligned).  Result: column
// lane % 16, rows 4 (lane / 16) + e.
// The j-th MFMA of 16 k takes k = 4 (lane / 16) + j from every lane: a lane's four k are neighbours, one 16-byte read where k is contiguous, and where it is not
// the four groups of lanes are four rows apart, which with pitches of 4 mod 16 floats are different banks (with k = lane / 16 + 4 j neighbouring rows: four
// runs of 16 banks on top of each other).  
// colsum: the sum of the lane's column of B.
template <bool AC, bool BC, bool COLSUM>
__device__ __forceinline__ f32x4_t ft_block(int fg, const float* pa, int sa, const float* pb, int sb, int KP, float& colsum) {
  const int kg = 4 * fg;
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f}, x[2], y[2];
  float sum = 0.f;
  pa += kg * (AC ? 1 : sa);
  pb += kg * (BC ? 1 : sb);
  auto fetch = [&](int q) {
    if constexpr (AC) x[q] = *reinterpret_cast<const f32x4_t*>(pa);
    else
#pragma unroll
      for (int j = 0; j < 4; ++j) x[q][j] = pa[j * sa];
    if constexpr (BC) y[q] = *reinterpret_cast<const f32x4_t*>(pb);
    else
#pragma unroll
      for (int j = 0; j < 4; ++j) y[q][j] = pb[j * sb];
    pa += 16 * (AC ? 1 : sa);
    pb += 16 * (BC ? 1 : sb);
  };
  auto multiply = [&](int q) {
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[q][j], y[q][j], acc, 0, 0, 0);
    if (COLSUM) sum += (y[q][0] + y[q][1]) + (y[q][2] + y[q][3]);
  };
  // the operands of the next 16 k are on their way while one 16 is multiplied
  fetch(0);
  for (int left = KP >> 4;;) {
    if (left > 1) fetch(1);
    __builtin_amdgcn_sched_barrier(0);
    multiply(0);
    if (--left == 0) break;
    if (left > 1) fetch(0);
    __builtin_amdgcn_sched_barrier(0);
    multiply(1);
    if (--left == 0) break;
  }
  if (COLSUM) {   // the four groups' parts
    const uint32_t u = __float_as_uint(sum);
    const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const uint32_t v = __float_as_uint(__uint_as_float(h[0]) + __uint_as_float(h[1]));
    const auto g = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    colsum = __uint_as_float(g[0]) + __uint_as_float(g[1]);
  }
  return acc;
}
template <bool AC, bool BC>
__device__ __forceinline__ f32x4_t ft_block(int fg, const float* pa, int sa, const float* pb, int sb, int KP) {
  float unused;
  return ft_block<AC, BC, false>(fg, pa, sa, pb, sb, KP, unused);
}
// LDS written before is visible behind it; loads from memory stay in flight (a __syncthreads would wait for them)
__device__ __forceinline__ void ft_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// the value of the lane whose number differs in bit 0 (bit 1): within four lanes, without LDS
__device__ __forceinline__ float ft_xor(float v, int bit) {
  const int x = __float_as_int(v);
  return __int_as_float(bit == 1 ? __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false) : __builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false));
}
__device__ __forceinline__ int ft_xor(int v, int bit) { return __float_as_int(ft_xor(__int_as_float(v), bit)); }
// the value of the first of each four lanes
__device__ __forceinline__ int ft_first(int v) { return __builtin_amdgcn_update_dpp(v, v, 0x00, 0xF, 0xF, false); }
__device__ __forceinline__ float ft_first(float v) { return __int_as_float(ft_first(__float_as_int(v))); }

// Softmax cross-entropy of 16 rows whose logits sit in LDS (written by this wavefront): four lanes per row, classes in
// turn.  Same split as fs_loss: the largest term apart, softmax_y - 1 as minus the sum of the others.  grad: the
// gradient replaces the logits (rows from nrows on get zeros).
// Class 0 starts as the largest and only a larger logit takes its place, as in fs_loss: a NaN there stays and is the row's maximum, a
// NaN elsewhere never becomes it and turns the sum of the others into NaN, so a row with a NaN logit has a NaN loss and NaN
// gradients whatever the class.  The four lanes have to agree on the maximum for that; the first one, which holds class 0, decides.
__device__ __forceinline__ void ft_loss16(float* lg_rows, int pitch, int C, const int* y, int nrows, float* rowloss, bool grad, float gscale) {
  const int lane = threadIdx.x & 63, r = lane >> 2, q = lane & 3;
  float* lg = lg_rows + r * pitch;
  const bool live = r < nrows;
  const int yb = live ? y[r] : 0;
  float v[8], mx = -INFINITY;
  int cm = 1 << 20;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (4 * j >= C) break;
    const int c = q + 4 * j;
    v[j] = c < C ? lg[c] : -INFINITY;
    if (c == 0 || v[j] > mx) { mx = v[j]; cm = c; }
  }
#pragma unroll
  for (int o = 1; o < 3; ++o) {
    const float m2 = ft_xor(mx, o);
    const int c2 = ft_xor(cm, o);
    if (m2 > mx || (m2 == mx && c2 < cm)) { mx = m2; cm = c2; }
  }
  mx = ft_first(mx);
  cm = ft_first(cm);
  float rest = 0.f, others = 0.f, ly = 0.f;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (4 * j >= C) break;
    const int c = q + 4 * j;
    ly += c == yb ? v[j] : 0.f;
    v[j] = c == cm ? 1.f : c < C ? expf(v[j] - mx) : 0.f;
    rest += c == cm ? 0.f : v[j];
    others += c == yb ? 0.f : v[j];
  }
#pragma unroll
  for (int o = 1; o < 3; ++o) {
    rest += ft_xor(rest, o);
    others += ft_xor(others, o);
    ly += ft_xor(ly, o);
  }
  if (rowloss && q == 0) rowloss[r] = live ? log1pf(rest) + (mx - ly) : 0.f;
  if (grad) {
    const float inv = 1.f / (1.f + rest), top = 1.f + (mx - mx);   // (NaN for an infinite maximum, as exp(mx - mx) is)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (4 * j >= C) break;
      const int c = q + 4 * j;
      if (c < C) lg[c] = live ? (c == yb ? -others * inv : (c == cm ? top : v[j]) * inv) * gscale : 0.f;
    }
  }
}

// e / d for 0 <= e < 65536, inv = ceil(2^32 / d) (d > 1; 2^32 / 1 does not fit and is taken as 0)
__device__ __forceinline__ int ft_div(int e, uint32_t inv) { return inv ? (int)__umulhi((uint32_t)e, inv) : e; }

// Block numbers wave, wave + WAVES, ... of a grid with `rows` block rows, as (row, column)
template <int WAVES>
struct FtWalk {
  int row, col, rows;
  __device__ __forceinline__ void start(int first, int n) {
    rows = n; row = first; col = 0;
    settle();
  }
  __device__ __forceinline__ void settle() { while (row >= rows) { row -= rows; ++col; } }
  __device__ __forceinline__ void next() { row += WAVES; settle(); }
};

__device__ __forceinline__ void ft_act4(float* v, int kind) {
  switch (kind) {
    case ACT_RELU:
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
      break;
    case ACT_LEAKY_RELU:
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.2f * v[e];
      break;
    case ACT_GELU:
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = act_fwd(v[e], ACT_GELU);
      break;
    case ACT_TANH:
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = tanhf(v[e]);
      break;
    default: break;
  }
}
// act'(z), from z for GELU, else from the activation (v holds the one or the other)
__device__ __forceinline__ void ft_act4_bwd(float* v, int kind) {
  switch (kind) {
    case ACT_RELU:
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? 1.f : 0.f;
      break;
    case ACT_LEAKY_RELU:
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? 1.f : 0.2f;
      break;
    case ACT_GELU:
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = act_bwd(v[e], ACT_GELU);
      break;
    case ACT_TANH:
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = 1.f - v[e] * v[e];
      break;
    default:
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = 1.f;
  }
}

// Rows and labels of the steps' mini-batches (Philox domain 1) into LDS, by the LOADERS wavefronts: each takes its share of the rows, 64 at a time (a lane draws
// the number of one row), in pieces of 512 elements.  A piece is requested one barrier interval or more before it is put into LDS: fetched and stored in
// one go, its latency held everybody at the first barrier of a step (900 of 14900 cycles).
struct FtLoader {
  const FusedSmallArgs& a;
  int member, rbeg, rend, px, lane;
  float* lds;
  int* ytab;
  int yhalf;             // labels per half of the double buffer
  int step = 0, r0, e0 = 0, src = 0, yv = 0;
  float v[8];
  int at[8];
  __device__ __forceinline__ FtLoader(const FusedSmallArgs& args, int m, int loader, int loaders, float* l, int* y, int half, int pitch)
      : a(args), member(m), px(pitch), lane(threadIdx.x & 63), lds(l), ytab(y), yhalf(half) {
    const int share = (a.B + loaders - 1) / loaders;
    rbeg = loader * share;
    rend = min(a.B, rbeg + share);
    r0 = rbeg;
  }
  __device__ __forceinline__ int rows() const { return min(64, rend - r0); }
  __device__ __forceinline__ int pieces() const {   // per step
    const int n = rend - rbeg;
    return n <= 0 ? 0 : n / 64 * ((64 * a.dims[0] + 511) / 512) + (n % 64 * a.dims[0] + 511) / 512;
  }
  __device__ __forceinline__ void request() {
    if (step >= a.n_steps) return;
    if (e0 == 0 && lane < rows()) {
      src = (int)philox_bounded(philox4x32_10(a.step0 + (uint32_t)step, (uint32_t)member, DOMAIN_BATCH, (uint32_t)(r0 + lane), (uint32_t)a.seed, (uint32_t)(a.seed >> 32)).x, (uint32_t)a.n_rows);
      yv = a.y[src];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int e = min(e0 + 64 * j + lane, rows() * a.dims[0] - 1), r = ft_div(e, a.lt_inv_d0), c = e - r * a.dims[0];   // (past the end: the last element again)
      at[j] = (r0 + r) * px + c;
      v[j] = a.x[(int64_t)__shfl(src, r) * a.dims[0] + c];
    }
  }
  __device__ __forceinline__ void store() {   // and move on to the next piece
    float* X = lds + a.lt_x[step & 1];
    if (e0 == 0 && lane < rows()) ytab[(step & 1) * yhalf + r0 + lane] = yv;
#pragma unroll
    for (int j = 0; j < 8; ++j) X[at[j]] = v[j];
    e0 += 512;
    if (e0 < rows() * a.dims[0]) return;
    e0 = 0;
    r0 += 64;
    if (r0 < rend) return;
    r0 = rbeg;
    ++step;
  }
};

// WAVES wavefronts compute and LOADERS fetch.  A block of a contraction is formed by one wavefront in the same order whatever their
// number, so results do not depend on it.
// NL: number of layers when it is known (its loops are unrolled and what they read of the argument block stays in scalar
// registers), 0: any.  OPT: optimiser.
template <int NL, int OPT, int WAVES, int LOADERS>
__global__ __launch_bounds__((WAVES + LOADERS) * 64) void fused_tiled_step_kernel(FusedSmallArgs a) {
  constexpr int FT_THREADS = (WAVES + LOADERS) * 64;
  extern __shared__ float lds[];
  const int i = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = lane & 15, fg = lane >> 4;   // fragment row / column, group of four rows (or of four k)
  const int64_t base = (int64_t)i * a.stride;
  const int L = NL ? NL : a.n_layers, B = a.B, d0 = a.dims[0], RB = fs_pad(B) / 16, px = fs_pitch(d0);
  int* const ytab = reinterpret_cast<int*>(lds + a.lt_y);
  for (int j = tid; j < a.lt_total; j += FT_THREADS) lds[j] = 0.f;   // every padding element stays zero (or finite where no result uses it)
  __syncthreads();
  for (int l = 0; l < L; ++l) {
    const int N = a.dims[l + 1], KN = a.dims[l] * N, p = fs_pitch(N);
    for (int e = tid; e < KN; e += FT_THREADS) {
      const int k = e / N;
      lds[a.lt_w[l] + k * p + (e - k * N)] = a.W32[base + a.w_off[l] + e];
    }
    for (int e = tid; e < N; e += FT_THREADS) lds[a.lt_b[l] + e] = a.W32[base + a.b_off[l] + e];
  }
  for (int e = tid; e < (int)a.stride; e += FT_THREADS) {
    lds[a.lt_s0 + e] = a.S0[base + e];
    if (OPT == OPT_ADAM) lds[a.lt_s1 + e] = a.S1[base + e];
  }
  const float* h = a.H + (int64_t)i * a.n_hyper;
  const float lr = h[a.col_lr];
  const float b1 = (OPT == OPT_ADAM && a.col_beta1 >= 0) ? h[a.col_beta1] : a.c0;
  const float wd = (OPT == OPT_ADAM && a.col_wd >= 0) ? h[a.col_wd] : a.c3;
  const int t0 = a.t[i];
  const float gscale = 1.f / (float)B;
  float last_loss = 0.f;

  if (wave >= WAVES) {
    // the fetching wavefronts: step s + 1's rows, labels and bias corrections go into the half of the double buffers that
    // step s does not read; they meet the others at every barrier
    FtLoader ld(a, i, wave - WAVES, LOADERS, lds, ytab, RB * 16, px);
    const int pieces = ld.pieces(), share = (pieces + 2 * L - 1) / (2 * L);
    auto corrections = [&](int s) {   // 1 / (1 - beta^t)
      if (OPT == OPT_ADAM && tid - WAVES * 64 < 2 && s < a.n_steps) lds[a.lt_sc + 2 * (s & 1) + lane] = 1.f / (1.f - powf(lane == 0 ? b1 : a.c1, (float)(t0 + s + 1)));
    };
    corrections(0);
    if (pieces > 0) ld.request();
    for (int q = 0; q < pieces; ++q) {
      ld.store();
      ld.request();
    }
    __syncthreads();
    for (int s = 0; s < a.n_steps; ++s) {
      corrections(s + 1);
      int left = s + 1 < a.n_steps ? pieces : 0;
      for (int k = 0; k < 2 * L; ++k) {
        for (int q = 0; q < share && left > 0; ++q, --left) {
          ld.store();
          ld.request();
        }
        ft_barrier();
      }
    }
  } else {
    // A run of up to 4 parameters, w + e * wp in LDS and p + e * pp in the member's vector: theta and the optimiser's state are read before the
    // gradient is formed.  (Parameters past the n-th are read, inside the workgroup's LDS, and not written.)
    struct Run { float w[4], s0[4], s1[4]; };
    auto read_run = [&](Run& r, const float* w, int wp, int p, int pp) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        r.w[e] = w[e * wp];
        r.s0[e] = lds[a.lt_s0 + p + e * pp];
        if (OPT == OPT_ADAM) r.s1[e] = lds[a.lt_s1 + p + e * pp];
      }
    };
    // (the fused multiply-adds are written out: the sizes of workgroups must round alike)
    auto update = [&](float& w, float& s0, float& s1, float g, float bc1, float bc2) {
      if (OPT == OPT_SGD_MOMENTUM) {
        s0 = fmaf(a.c0, s0, g);
        w = fmaf(-lr, s0, w);
      } else if (OPT == OPT_ADAM) {
        s0 = fmaf(b1, s0, (1.f - b1) * g);
        s1 = fmaf(a.c1, s1, (1.f - a.c1) * g * g);
        w = fmaf(-lr, fmaf(wd, w, (s0 * bc1) / (sqrtf(s1 * bc2) + a.c2)), w);
      } else {
        s0 = fmaf(a.c0, s0, (1.f - a.c0) * g * g);
        w = w - lr * g / sqrtf(s0 + a.c1);
      }
    };
    auto write_run = [&](Run& r, float* w, int wp, int p, int pp, const f32x4_t g, int n, const float* sc, bool last) {
      const float bc1 = OPT == OPT_ADAM ? sc[0] : 1.f, bc2 = OPT == OPT_ADAM ? sc[1] : 1.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) update(r.w[e], r.s0[e], r.s1[e], g[e], bc1, bc2);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < n) {
          w[e * wp] = r.w[e];
          lds[a.lt_s0 + p + e * pp] = r.s0[e];
          if (OPT == OPT_ADAM) lds[a.lt_s1 + p + e * pp] = r.s1[e];
        }
      if (last)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (e < n) a.G[base + p + e * pp] = g[e];
    };
    // gradient and update of a 16 x 16 block of W_l; the blocks of the first block row also form the bias gradient of their
    // columns (column sums of dz, from the operands that are there anyway)
    auto weight_unit = [&](int l, int kb, int nb, const float* in, int pin, const float* sc, bool last) {
      const int K = a.dims[l], N = a.dims[l + 1], pn = fs_pitch(N), n = nb * 16 + fr, k = kb * 16 + 4 * fg;
      const bool inside = k < K && n < N, bias = kb == 0 && fg == 0 && n < N;
      float* const w = lds + a.lt_w[l] + k * pn + n;
      const int p = a.w_off[l] + k * N + n;
      Run r;
      float bw = 0.f, bs0 = 0.f, bs1 = 0.f, bsum = 0.f;
      // (ahead of the product, whose time hides their latency; where several members share a compute unit the registers are worth more)
      constexpr bool AHEAD = WAVES > 8;
      if (AHEAD && inside) read_run(r, w, pn, p, N);
      if (AHEAD && bias) {
        bw = lds[a.lt_b[l] + n];
        bs0 = lds[a.lt_s0 + a.b_off[l] + n];
        if (OPT == OPT_ADAM) bs1 = lds[a.lt_s1 + a.b_off[l] + n];
      }
      const float* const pa = in + kb * 16 + fr;
      const float* const pb = lds + a.lt_d[l] + n;
      const f32x4_t acc = kb == 0 ? ft_block<false, false, true>(fg, pa, pin, pb, pn, RB * 16, bsum) : ft_block<false, false>(fg, pa, pin, pb, pn, RB * 16);
      if (!AHEAD && inside) read_run(r, w, pn, p, N);
      if (inside) write_run(r, w, pn, p, N, acc, K - k, sc, last);
      if (bias) {
        if (!AHEAD) {
          bw = lds[a.lt_b[l] + n];
          bs0 = lds[a.lt_s0 + a.b_off[l] + n];
          if (OPT == OPT_ADAM) bs1 = lds[a.lt_s1 + a.b_off[l] + n];
        }
        update(bw, bs0, bs1, bsum, OPT == OPT_ADAM ? sc[0] : 1.f, OPT == OPT_ADAM ? sc[1] : 1.f);
        lds[a.lt_b[l] + n] = bw;
        lds[a.lt_s0 + a.b_off[l] + n] = bs0;
        if (OPT == OPT_ADAM) lds[a.lt_s1 + a.b_off[l] + n] = bs1;
        if (last) a.G[base + a.b_off[l] + n] = bsum;
      }
    };
    __syncthreads();
    for (int s = 0; s < a.n_steps; ++s) {
      const int cur = s & 1;
      const bool last = s == a.n_steps - 1;
      const float* X = lds + a.lt_x[cur];
      const float* sc = lds + a.lt_sc + 2 * cur;
      FtWalk<WAVES> w;
#pragma unroll
      for (int l = 0; l < L; ++l) {
        const int KP = fs_pad(a.dims[l]), N = a.dims[l + 1], pk = fs_pitch(a.dims[l]), pn = fs_pitch(N), NB = fs_pad(N) / 16;
        const float* in = l == 0 ? X : lds + a.lt_a[l];
        if (l < L - 1) {
          for (w.start(wave, RB); w.col < NB; w.next()) {
            const int n = w.col * 16 + fr, o = (w.row * 16 + 4 * fg) * pn + n;
            const float bias = lds[a.lt_b[l] + n];
            const f32x4_t acc = ft_block<true, false>(fg, in + (w.row * 16 + fr) * pk, 1, lds + a.lt_w[l] + n, pn, KP);
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = acc[e] + bias;
            if (a.act == ACT_GELU) {
#pragma unroll
              for (int e = 0; e < 4; ++e) lds[a.lt_d[l] + o + e * pn] = v[e];
            }
            ft_act4(v, a.act);
#pragma unroll
            for (int e = 0; e < 4; ++e) lds[a.lt_a[l + 1] + o + e * pn] = v[e];
          }
        } else {
          for (int rb = wave; rb < RB; rb += WAVES) {
            for (int nb = 0; nb < NB; ++nb) {
              const int n = nb * 16 + fr, o = (rb * 16 + 4 * fg) * pn + n;
              const float bias = lds[a.lt_b[l] + n];
              const f32x4_t acc = ft_block<true, false>(fg, in + (rb * 16 + fr) * pk, 1, lds + a.lt_w[l] + n, pn, KP);
#pragma unroll
              for (int e = 0; e < 4; ++e) lds[a.lt_d[l] + o + e * pn] = acc[e] + bias;
            }
            // (written and read by the same wavefront: in order, no barrier)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            ft_loss16(lds + a.lt_d[l] + rb * 16 * pn, pn, N, ytab + (cur * RB + rb) * 16, B - rb * 16, last ? lds + a.lt_rowloss + rb * 16 : nullptr,
                      true, gscale);
          }
        }
        ft_barrier();
      }
      if (last && wave == 0) last_loss = fs_sum_rowloss(lds + a.lt_rowloss, B) / (float)B;
      // backward: the input gradient of layer l shares an interval with the weight gradient of layer l + 1
#pragma unroll
      for (int l = L - 1; l >= 0; --l) {
        int left = wave;   // number of this wavefront's next unit in what follows
        if (l > 0) {
          const int K = a.dims[l], N = a.dims[l + 1], pn = fs_pitch(N), pk = fs_pitch(K), KB = fs_pad(K) / 16;
          for (w.start(wave, RB); w.col < KB; w.next()) {   // dz_{l-1} = (dz_l W_l^T) * act'
            const int o = (w.row * 16 + 4 * fg) * pk + w.col * 16 + fr;
            float* d = lds + a.lt_d[l - 1] + o;
            const float* from = a.act == ACT_GELU ? d : lds + a.lt_a[l] + o;
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = from[e * pk];
            const f32x4_t acc = ft_block<true, true>(fg, lds + a.lt_d[l] + (w.row * 16 + fr) * pn, 1, lds + a.lt_w[l] + (w.col * 16 + fr) * pn, 1, fs_pad(N));
            ft_act4_bwd(v, a.act);
#pragma unroll
            for (int e = 0; e < 4; ++e) d[e * pk] = acc[e] * v[e];
            left += WAVES;
          }
          left -= RB * KB;
        }
        if (l + 1 < L) {
          const int NB = fs_pad(a.dims[l + 2]) / 16, KB = fs_pad(a.dims[l + 1]) / 16;
          for (w.start(left, NB); w.col < KB; w.next()) { weight_unit(l + 1, w.col, w.row, lds + a.lt_a[l + 1], fs_pitch(a.dims[l + 1]), sc, last); left += WAVES; }
          left -= NB * KB;
        }
        if (l == 0) {
          const int NB = fs_pad(a.dims[1]) / 16, KB = fs_pad(d0) / 16;
          for (w.start(left, NB); w.col < KB; w.next()) weight_unit(0, w.col, w.row, X, px, sc, last);
        }
        ft_barrier();
      }
    }
  }
  __syncthreads();
  for (int l = 0; l < L; ++l) {
    const int N = a.dims[l + 1], KN = a.dims[l] * N, p = fs_pitch(N);
    for (int e = tid; e < KN; e += FT_THREADS) {
      const int k = e / N;
      a.W32[base + a.w_off[l] + e] = lds[a.lt_w[l] + k * p + (e - k * N)];
    }
    for (int e = tid; e < N; e += FT_THREADS) a.W32[base + a.b_off[l] + e] = lds[a.lt_b[l] + e];
  }
  for (int e = tid; e < (int)a.stride; e += FT_THREADS) {
    a.S0[base + e] = lds[a.lt_s0 + e];
    if (OPT == OPT_ADAM) a.S1[base + e] = lds[a.lt_s1 + e];
  }
  if (tid == 0) {
    a.t[i] = t0 + a.n_steps;
    a.loss[i] = last_loss;
  }
}

// The sizes of the step's workgroup.  Twelve and four wavefronts are fastest for a member by itself (32-64-4, 64 rows: 5.5 us per step, 5.9 with eight and
// four), but a compute unit holds one of them; populations of more members than that take eight and four, of which it holds one or two (registers), four and
// two, or three and one, of which it holds two and four.
constexpr int FT_N_SIZES = 4;
constexpr struct { int waves, loaders; } FT_SIZES[FT_N_SIZES] = {{12, 4}, {8, 4}, {4, 2}, {3, 1}};
template <int OPT, int SIZE>
static void (*ft_step_kernel(int n_layers))(FusedSmallArgs) {
  constexpr int W = FT_SIZES[SIZE].waves, LD = FT_SIZES[SIZE].loaders;
  return n_layers == 2 ? fused_tiled_step_kernel<2, OPT, W, LD> : n_layers == 3 ? fused_tiled_step_kernel<3, OPT, W, LD> : fused_tiled_step_kernel<0, OPT, W, LD>;
}
template <int OPT>
static void (*ft_step_kernel(int n_layers, int size))(FusedSmallArgs) {
  return size == 0 ? ft_step_kernel<OPT, 0>(n_layers) : size == 1 ? ft_step_kernel<OPT, 1>(n_layers) : size == 2 ? ft_step_kernel<OPT, 2>(n_layers) : ft_step_kernel<OPT, 3>(n_layers);
}
static void (*ft_step_kernel(int optimizer, int n_layers, int size))(FusedSmallArgs) {
  return optimizer == OPT_SGD_MOMENTUM ? ft_step_kernel<OPT_SGD_MOMENTUM>(n_layers, size)
         : optimizer == OPT_ADAM ? ft_step_kernel<OPT_ADAM>(n_layers, size) : ft_step_kernel<OPT_RMSPROP>(n_layers, size);
}

// (1024 rows x 8 members: 506 -> 18 us with the sum over workgroups, against one workgroup per member that walks all rows.)
// eval: every workgroup takes 64 held-out rows of one member (blockIdx.x), a wavefront 16 of them through all layers on
// its own; the workgroup's sum of row losses goes to part[member][blockIdx.x].
__global__ __launch_bounds__(256) void fused_tiled_eval_kernel(FusedSmallArgs a, float* __restrict__ part) {
  extern __shared__ float lds[];
  __shared__ int ylds[FT_EVAL_ROWS];
  __shared__ float rowloss[FT_EVAL_ROWS];
  const int i = blockIdx.y, r0 = blockIdx.x * FT_EVAL_ROWS, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = lane & 15, fg = lane >> 4, L = a.n_layers, d0 = a.dims[0];
  const int64_t base = (int64_t)i * a.stride;
  const int nrows = min(FT_EVAL_ROWS, a.n_rows - r0);
  for (int l = 0; l < L; ++l) {
    const int K = a.dims[l], N = a.dims[l + 1], p = fs_pitch(N), NP = fs_pad(N), total = fs_pad(K) * NP;
    for (int e = tid; e < total; e += 256) {   // (with the padding)
      const int k = e / NP, n = e - k * NP;
      lds[a.lt_w[l] + k * p + n] = k < K && n < N ? a.W32[base + a.w_off[l] + k * N + n] : 0.f;
    }
    for (int n = tid; n < NP; n += 256) lds[a.lt_b[l] + n] = n < N ? a.W32[base + a.b_off[l] + n] : 0.f;
  }
  const int p = a.lt_pitch, D = fs_pad(d0);
  for (int e = tid; e < FT_EVAL_ROWS * D; e += 256) {
    const int r = e / D, c = e - r * D;
    lds[a.lt_a[0] + r * p + c] = r < nrows && c < d0 ? a.x[(int64_t)(r0 + r) * d0 + c] : 0.f;
  }
  if (tid < FT_EVAL_ROWS) ylds[tid] = tid < nrows ? a.y[r0 + tid] : 0;
  __syncthreads();
  for (int l = 0; l < L; ++l) {
    const int KP = fs_pad(a.dims[l]), N = a.dims[l + 1], pn = fs_pitch(N), NB = fs_pad(N) / 16;
    const float* in = lds + a.lt_a[l & 1] + wave * 16 * p;
    float* out = lds + a.lt_a[(l + 1) & 1] + wave * 16 * p;
    for (int nb = 0; nb < NB; ++nb) {
      const int n = nb * 16 + fr;
      const f32x4_t acc = ft_block<true, false>(fg, in + fr * p, 1, lds + a.lt_w[l] + n, pn, KP);
      const float bias = lds[a.lt_b[l] + n];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float z = acc[e] + bias;
        out[(4 * fg + e) * p + n] = l < L - 1 ? act_fwd(z, a.act) : z;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  ft_loss16(lds + a.lt_a[L & 1] + wave * 16 * p, p, a.dims[L], ylds + wave * 16, nrows - wave * 16, rowloss + wave * 16, false, 0.f);
  __syncthreads();
  if (wave == 0) {
    const float t = wave_sum(rowloss[lane]);
    if (lane == 0) part[(int64_t)i * gridDim.x + blockIdx.x] = t;
  }
}

static hipError_t set_lds(const void* kernel, size_t bytes) {
  if (bytes > FUSED_SMALL_MAX_LDS) return hipErrorInvalidValue;
  return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

constexpr int FS_CUS = 256;
// How often the compute units are filled when each holds up to `resident` workgroups of a kernel that needs `lds` bytes.
static int fs_rounds(int P, size_t lds, int resident) {
  const int each = std::max(1, std::min(resident, (int)(FUSED_SMALL_MAX_LDS / lds)));
  return (P + FS_CUS * each - 1) / (FS_CUS * each);
}

// Networks for which the plain form is faster although the tiled one fits.  The tiled form pads batches and widths to 16, which costs
// nothing while there is a compute unit for every member; with more members the padded arrays of a mini-batch of a few rows can take a
// second round where the plain ones take one (1024 members 24-24-24-24-3, Adam, one row: 17 us against 39 per step), and four or more layers of a
// handful of units are a serial chain that 16 x 16 blocks only lengthen (8 members 8-8-8-8-8-2, one row, one step per call: 14 us against 17).
// From the configuration alone: how an interval is divided into calls does not change a result.
static bool fs_plain_is_faster(const FusedSmallArgs& a, size_t tiled, size_t plain) {
  int widest = 0;
  for (int l = 0; l <= a.n_layers; ++l) widest = std::max(widest, a.dims[l]);
  const bool fewer_rounds = fs_rounds(a.P, plain, 8) < fs_rounds(a.P, tiled, 4);
  if (a.B <= 8 && widest <= 32 && fewer_rounds) return true;
  return a.n_layers > 3 && widest <= 8 && a.B <= (fewer_rounds ? 32 : 4);
}

// The size that fills the compute units the fewest times, the larger of two that are equal.  20 steps a call, us per step of eight and four wavefronts
// only, with the smaller sizes, and in the plain form: 1024 members 4-8-2, Adam, 16 rows: 17.6, 5.1, 10.0; 512 members 8-8-8-2, momentum, 16 rows: 9.8, 5.2,
// 9.8; 1024 members 32-64-4, Adam, 16 rows: 22.9, 15.8, 48.1.  The smallest only where no phase of a step has more than eight 16 x 16
// blocks: with more its three wavefronts become the bound (768 members 32-64-4, 32 rows: 11.4 us in two rounds of the largest, 15.6 in one
// of the smallest), and with a mini-batch of more than 2048 values the one that fetches (768 members 64-10, 64 rows: 8.2 and 9.8).
static int ft_size(const FusedSmallArgs& a, size_t tiled) {
  const int RB = fs_pad(a.B) / 16;
  auto blocks = [&](int l) { return fs_pad(a.dims[l]) / 16; };
  int most = 0;
  for (int l = 0; l < a.n_layers; ++l) {
    most = std::max(most, l + 1 < a.n_layers ? RB * blocks(l + 1) : RB);
    most = std::max(most, (l > 0 ? RB * blocks(l) : blocks(0) * blocks(1)) + (l + 1 < a.n_layers ? blocks(l + 1) * blocks(l + 2) : 0));
  }
  // (more than eight wavefronts have nothing to do where no phase has more than eight blocks, and cost a launch of one step up to 9 %)
  const int largest = most > 8 ? 0 : 1;
  if (a.P <= FS_CUS) return largest;
  // workgroups of a size that a compute unit's registers hold
  auto held = [&](int size) {
    int n = 1;
    const auto kernel = ft_step_kernel(a.optimizer, a.n_layers, size);
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, reinterpret_cast<const void*>(kernel), (FT_SIZES[size].waves + FT_SIZES[size].loaders) * 64, 0) != hipSuccess) {
      (void)hipGetLastError();
      n = 1;
    }
    return n;
  };
  const int rounds[FT_N_SIZES] = {fs_rounds(a.P, tiled, 1), fs_rounds(a.P, tiled, held(1)), fs_rounds(a.P, tiled, 2), fs_rounds(a.P, tiled, 4)};
  int size = largest;
  if (rounds[1] < rounds[size]) size = 1;
  // (Four wavefronts have a block each where no phase has more than four, and a smaller workgroup starts and meets at barriers sooner; past 1024 values its
  // two fetching wavefronts become the bound.  512 members, us per call with eight and four wavefronts and with four and two: 4-2, Adam, 4 rows, one
  // step 9.4 and 9.1; 4-8-2, momentum, 16 rows, one step 9.7 and 8.9, 20 steps 77.7 and 70.8; 32-4, momentum, 32 rows, 20 steps 62.6 and 58.8; 64-4, Adam,
  // 32 rows, one step 10.9 and 11.5.  With a compute unit per member the two are within 2 % of each other either way for one step.)
  if (size == 1 && rounds[2] == rounds[1] && most <= 4 && a.B * a.dims[0] <= 1024) size = 2;
  if (rounds[2] < rounds[size]) size = 2;
  if (rounds[3] < rounds[size] && most <= 8 && a.B * a.dims[0] <= 2048) size = 3;
  return size;
}

// The tiled form whenever its padded arrays fit a compute unit and fs_plain_is_faster() knows nothing better; the plain form (no padding,
// no double buffers) is left for those and for networks that fill the LDS nearly to the last byte.
hipError_t fused_small_step(FusedSmallArgs a, hipStream_t s) {
  const size_t tiled = fused_tiled_plan(a, false), bytes = fused_small_plan(a, false);
  if (tiled <= FUSED_SMALL_MAX_LDS && !fs_plain_is_faster(a, tiled, bytes)) {
    const int size = ft_size(a, tiled);
    const auto kernel = ft_step_kernel(a.optimizer, a.n_layers, size);
    hipError_t e = set_lds(reinterpret_cast<const void*>(kernel), tiled);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(a.P), dim3((FT_SIZES[size].waves + FT_SIZES[size].loaders) * 64), tiled, s, a);
    return hipGetLastError();
  }
  hipError_t e = set_lds(reinterpret_cast<const void*>(fused_small_step_kernel), bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fused_small_step_kernel, dim3(a.P), dim3(FS_THREADS), bytes, s, a);
  return hipGetLastError();
}

// eval: score[i] = -(mean cross-entropy over the held-out rows), chunks of B rows through LDS.
__global__ __launch_bounds__(FS_THREADS) void fused_small_eval_kernel(FusedSmallArgs a) {
  extern __shared__ float lds[];
  const int i = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int64_t base = (int64_t)i * a.stride;
  float* W = lds + a.lds_w;
  for (int j = tid; j < (int)a.stride; j += FS_THREADS) W[j] = a.W32[base + j];
  int* ylds = reinterpret_cast<int*>(lds + a.lds_y);
  const int d0 = a.dims[0];
  float total = 0.f;  // meaningful in wave 0
  __syncthreads();
  for (int r0 = 0; r0 < a.n_rows; r0 += a.B) {
    const int nrows = a.n_rows - r0 < a.B ? a.n_rows - r0 : a.B;
    for (int r = wave; r < nrows; r += FS_THREADS / 64) {
      const int64_t src = r0 + r;
      for (int c = lane; c < d0; c += 64) lds[a.lds_a[0] + r * (d0 + 1) + c] = a.x[src * d0 + c];
      if (lane == 0) ylds[r] = a.y[src];
    }
    __syncthreads();
    fs_forward(a, lds, nrows);
    fs_loss(a, lds, nrows, nullptr, 0.f);
    if (wave == 0) total += fs_sum_rowloss(lds + a.lds_rowloss, nrows);
    __syncthreads();
  }
  if (tid == 0) a.score[i] = -total / (float)a.n_rows;
}

int fused_small_eval_parts(int n_rows) { return (n_rows + FT_EVAL_ROWS - 1) / FT_EVAL_ROWS; }
// part: P x fused_small_eval_parts(n_rows) floats of working memory
hipError_t fused_small_eval(FusedSmallArgs a, float* part, hipStream_t s) {
  const size_t tiled = fused_tiled_plan(a, true);
  if (tiled <= FUSED_SMALL_MAX_LDS - 1024) {   // (1 KB for the kernel's static arrays)
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fused_tiled_eval_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)tiled);
    if (e != hipSuccess) return e;
    const int parts = fused_small_eval_parts(a.n_rows);
    hipLaunchKernelGGL(fused_tiled_eval_kernel, dim3(parts, a.P), dim3(256), tiled, s, a, part);
    e = hipGetLastError();
    return e != hipSuccess ? e : row_reduce(part, parts, a.P, parts, -1.f / (float)a.n_rows, a.score, 1, s);
  }
  const size_t bytes = fused_small_plan(a, true);
  hipError_t e = set_lds(reinterpret_cast<const void*>(fused_small_eval_kernel), bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(fused_small_eval_kernel, dim3(a.P), dim3(FS_THREADS), bytes, s, a);
  return hipGetLastError();
}

}  // namespace pbt
