// The population-batched GEMM that stages its operands through registers: for weight gradients dW = X^T dY with the optimiser in
// the epilogue (its loads of theta and the optimiser state are what the launch waits for, and half of the first strip's go out ahead of the
// K loop), and, with every other functor, for rows too long for the direct-to-LDS kernel's buffer offsets (gemm_lds.h, which everything else takes).
//
// Tiling (wave64): a workgroup of WM x WN wavefronts owns a BM x BN tile of C; each wavefront owns a (BM/WM) x (BN/WN) sub-tile made of 32x32
// accumulator blocks fed by v_mfma_f32_32x32x16_bf16.  The K loop moves BK wide slabs of A and B from HBM into registers (16-byte loads), then
// into LDS in a "K-contiguous" layout, so that every MFMA operand is one 16-byte LDS read.  Operands whose memory layout is contiguous along M or
// N instead of K (X and dY in the weight gradient) are transposed in registers on their way into LDS.  The loads of slab k+1 (k+2 with two
// LDS buffers) are in flight while slab k is multiplied.
#pragma once
#include "gemm_epilogues.h"

namespace pbt {

// LDS row pitch in elements for a slab width BK: +8 keeps 16-byte alignment and skews the banks
constexpr int gemm_pitch(int bk) { return bk + 8; }
// Within an LDS row the 16-byte slots (8 k values each) are permuted by the row's group of sixteen:
// slot' = slot ^ ((row / 16) & mask).  The transposing writers (lanes 8 rows apart, same slot) would
// otherwise all hit two bank groups, because 8 row pitches are a multiple of half the bank period; the
// XOR spreads them over all banks.  Readers take 16 consecutive rows of one slot per LDS cycle, and
// the odd slot pitch already spreads those, so the permutation has to be constant over such a group:
// keyed by row / 8 it costs every fragment read 4 to 8 extra cycles (measured), keyed by row / 16 none.
template <int BK>
__device__ __forceinline__ int lds_offset(int row, int k) {
  constexpr int MASK = (BK / 8 < 8 ? BK / 8 : 8) - 1;
  return row * gemm_pitch(BK) + ((((k >> 3) ^ ((row >> 4) & MASK)) << 3) | (k & 7));
}

// ---- global -> register staging -------------------------------------------------------------
// Operand tile of ROWS x BK (ROWS along M or N).  KCONTIG: memory is [row][k].
// Otherwise memory is [k][row] and a thread fetches a KB x 8 block (KB k-rows of
// 8 consecutive rows each) that it transposes before the LDS write.

template <int ROWS, int GEMM_BK, bool KCONTIG, int THREADS>
struct TileLoader {
  static constexpr int GEMM_PITCH = gemm_pitch(GEMM_BK);
  static constexpr int CHUNKS = ROWS * GEMM_BK / 8;            // 16-byte pieces per tile
  static constexpr int PER_THREAD = CHUNKS / THREADS;     // pieces per thread
  static constexpr int KB = PER_THREAD;                        // k-rows per thread in the transposed case
  static_assert(CHUNKS % THREADS == 0, "tile must divide evenly over the workgroup");
  uint4 r[PER_THREAD];

  // base points at this member's operand; row0 / k0 select the tile; nrows / K bound it.
  __device__ __forceinline__ void load(const bf16_t* __restrict__ base, int64_t ld, int row0, int k0, int nrows, int K) {
    const int t = threadIdx.x;
    if constexpr (KCONTIG) {
#pragma unroll
      for (int j = 0; j < PER_THREAD; ++j) {
        const int c = t + THREADS * j;
        const int row = row0 + c / (GEMM_BK / 8);
        const int k = k0 + (c % (GEMM_BK / 8)) * 8;
        r[j] = fetch8(base, (int64_t)row * ld + k, row < nrows, K - k);
      }
    } else {
      const int rb = t % (ROWS / 8);
      const int kb = t / (ROWS / 8);
      const int row = row0 + rb * 8;
#pragma unroll
      for (int j = 0; j < KB; ++j) {
        const int k = k0 + kb * KB + j;
        r[j] = fetch8(base, (int64_t)k * ld + row, k < K, nrows - row);
      }
    }
  }

  // The same tile when its K range lies wholly inside the operand: straight 16-byte loads, no guards.
  // Rows past the operand's last row (a ragged last tile in M or N) read the last row (K-contiguous
  // operand) or the last whole group of eight rows (the other layout; the launcher checks that the row
  // count is a multiple of 8 then): always in bounds, and the epilogue drops those rows' results.
  __device__ __forceinline__ void load_interior(const bf16_t* __restrict__ base, int64_t ld, int row0, int k0, int nrows) {
    const int t = threadIdx.x;
    if constexpr (KCONTIG) {
#pragma unroll
      for (int j = 0; j < PER_THREAD; ++j) {
        const int c = t + THREADS * j;
        const int row = min(row0 + c / (GEMM_BK / 8), nrows - 1);
        r[j] = *reinterpret_cast<const uint4*>(base + (int64_t)row * ld + k0 + (c % (GEMM_BK / 8)) * 8);
      }
    } else {
      const int rb = t % (ROWS / 8);
      const int kb = t / (ROWS / 8);
      const int row = min(row0 + rb * 8, nrows - 8);
#pragma unroll
      for (int j = 0; j < KB; ++j)
        r[j] = *reinterpret_cast<const uint4*>(base + (int64_t)(k0 + kb * KB + j) * ld + row);
    }
  }

  // 8 consecutive elements starting at base[off]; `valid` false or `left` <= 0 gives zeros,
  // 0 < left < 8 loads only the first `left` elements.
  static __device__ __forceinline__ uint4 fetch8(const bf16_t* __restrict__ base, int64_t off, bool valid, int left) {
    uint4 v = make_uint4(0, 0, 0, 0);
    if (valid && left >= 8) {
      v = *reinterpret_cast<const uint4*>(base + off);
    } else if (valid && left > 0) {
      bf16_t e[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) e[i] = i < left ? base[off + i] : (bf16_t)0;
      v.x = e[0] | ((uint32_t)e[1] << 16);
      v.y = e[2] | ((uint32_t)e[3] << 16);
      v.z = e[4] | ((uint32_t)e[5] << 16);
      v.w = e[6] | ((uint32_t)e[7] << 16);
    }
    return v;
  }

  __device__ __forceinline__ void store(bf16_t* __restrict__ lds) const {
    const int t = threadIdx.x;
    if constexpr (KCONTIG) {
#pragma unroll
      for (int j = 0; j < PER_THREAD; ++j) {
        const int c = t + THREADS * j;
        const int row = c / (GEMM_BK / 8);
        const int k = (c % (GEMM_BK / 8)) * 8;
        *reinterpret_cast<uint4*>(lds + lds_offset<GEMM_BK>(row, k)) = r[j];
      }
    } else {
      const int rb = t % (ROWS / 8);
      const int kb = t / (ROWS / 8);
      // r[j] holds rows rb*8 .. rb*8+7 at k = kb*KB + j.  Emit, per row, KB consecutive k values.
      const uint32_t* w = reinterpret_cast<const uint32_t*>(r);  // w[j*4 + q]: rows 2q (low half), 2q+1 (high half)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint32_t lo[KB / 2 > 0 ? KB / 2 : 1], hi[KB / 2 > 0 ? KB / 2 : 1];
#pragma unroll
        for (int j = 0; j < KB; j += 2) {
          const uint32_t a = w[j * 4 + q], b = w[(j + 1) * 4 + q];
          lo[j / 2] = (a & 0xffffu) | (b << 16);          // row 2q:   k = j, j+1
          hi[j / 2] = (a >> 16) | (b & 0xffff0000u);      // row 2q+1: k = j, j+1
        }
        bf16_t* p0 = lds + lds_offset<GEMM_BK>(rb * 8 + 2 * q, kb * KB);      // both rows are in the same group of sixteen
        bf16_t* p1 = p0 + GEMM_PITCH;
        if constexpr (KB == 2) {
          *reinterpret_cast<uint32_t*>(p0) = lo[0];
          *reinterpret_cast<uint32_t*>(p1) = hi[0];
        } else if constexpr (KB == 4) {
          *reinterpret_cast<uint2*>(p0) = make_uint2(lo[0], lo[1]);
          *reinterpret_cast<uint2*>(p1) = make_uint2(hi[0], hi[1]);
        } else {
          static_assert(KB == 8, "unsupported tile shape");
          *reinterpret_cast<uint4*>(p0) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
          *reinterpret_cast<uint4*>(p1) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
        }
      }
    }
  }
};

template <int BM, int BN, int GEMM_BK, int WM, int WN, bool A_MCONTIG, bool B_KCONTIG, bool DOUBLE_BUF, class Epilogue>
__global__ __launch_bounds__(WM * WN * 64) void gemm_bf16_kernel(GemmArgs g, Epilogue epi) {
  constexpr int THREADS = WM * WN * 64;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  constexpr int GEMM_PITCH = gemm_pitch(GEMM_BK);
  constexpr int SLAB = (BM + BN) * GEMM_PITCH;  // elements of one A + B slab pair
  // LDS (sized by the launcher): one or two slab pairs during the K loop, then (reused) a 32-row strip of C
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];

  const int total = g.tiles * g.batch;
  int id = xcd_remap(blockIdx.x, total);
  const int per_member = g.tiles;
  const int member = id / per_member;
  id -= member * per_member;
  const int tile = id;
  const int group = id / (GROUP_M * g.tiles_n);
  const int first_m = group * GROUP_M;
  const int rows_in_group = g.tiles_m - first_m < GROUP_M ? g.tiles_m - first_m : GROUP_M;
  id -= group * GROUP_M * g.tiles_n;
  const int tm = first_m + id % rows_in_group;
  const int tn = id / rows_in_group;
  const int m0 = tm * BM, n0 = tn * BN;

  const bf16_t* __restrict__ A = g.A + (int64_t)(member / g.inner) * g.sa + (int64_t)(member % g.inner) * g.sa_in;
  const bf16_t* __restrict__ B = g.B + (int64_t)(member / g.inner) * g.sb + (int64_t)(member % g.inner) * g.sb_in;

  TileLoader<BM, GEMM_BK, !A_MCONTIG, THREADS> la;
  TileLoader<BN, GEMM_BK, B_KCONTIG, THREADS> lb;

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int frag_row = lane & 31, frag_k = (lane >> 5) * 8;

  f32x16_t acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // A functor that reads what it updates (the optimiser) takes runs of 4 columns, consecutive lanes side
  // by side (whole 256-byte row segments per access, which streaming loads need: nothing keeps the other
  // half of a line).  The runs of the first 32-row strip are requested right after the K loop, each later
  // strip's while the one before it is applied.
  constexpr int WCOLS = BN / WN, RUNS4 = WCOLS / 4, NQ4 = 32 * RUNS4 / 64;
  epi.begin(member);

  // (half of the first strip goes out ahead of the K loop so that memory is never left idle while the
  // workgroups of a compute unit are all busy with their operands; all of it would cost an occupancy step)
  typename Epilogue::Fetched pre[NQ4];
  constexpr int EARLY_RUNS = NQ4 / 2;
  auto fetch_first_strip = [&](int q0, int q1) {
    if constexpr (Epilogue::PREFETCH) {
#pragma unroll
      for (int q = 0; q < NQ4; ++q) {
        if (q < q0 || q >= q1) continue;
        const int run = q * 64 + lane;
        const int m = m0 + wm * (BM / WM) + run / RUNS4, n = n0 + wn * WCOLS + (run % RUNS4) * 4;
        if (m < g.M && n < g.N) pre[q] = epi.fetch(m, n, g.N - n < 4 ? g.N - n : 4);
      }
    }
  };
  fetch_first_strip(0, EARLY_RUNS);

  // (only the weight-gradient functors carry this code: elsewhere its registers would cost an occupancy step)
  const bool want_colsum = Epilogue::COLSUM && g.colsum != nullptr && tm == 0;
  float csum = 0.f;

  // One K loop per kind of launch: straight 16-byte loads when K is a multiple of the slab depth (ragged
  // last tiles in M or N read clamped rows), the guarded loads otherwise; keeping the two apart keeps the
  // guards' branches out of the common loop.  (A third loop for a K with a
  // remainder, guarded in its last slab only: 2 % on a ragged transformer, but 1.5 to 6 % slower wherever it is not taken.)
  auto k_loop = [&](auto interior_tag) {
    constexpr bool INTERIOR = decltype(interior_tag)::value;
    auto fetch_slab = [&](int k) {
      if constexpr (INTERIOR) {
        la.load_interior(A, g.lda, m0, k, g.M);
        lb.load_interior(B, g.ldb, n0, k, B_KCONTIG ? g.N : g.b_cols);
      } else {
        la.load(A, g.lda, m0, k, g.M, g.K);
        lb.load(B, g.ldb, n0, k, g.N, g.K);
      }
    };
    // the MFMAs of one slab
    auto multiply_slab = [&](const bf16_t* As, const bf16_t* Bs) {
#pragma unroll
      for (int kk = 0; kk < GEMM_BK; kk += 16) {
        bf16x8_t af[TM], bfr[TN];
#pragma unroll
        for (int i = 0; i < TM; ++i)
          af[i] = *reinterpret_cast<const bf16x8_t*>(As + lds_offset<GEMM_BK>(wm * (BM / WM) + i * 32 + frag_row, kk + frag_k));
#pragma unroll
        for (int j = 0; j < TN; ++j)
          bfr[j] = *reinterpret_cast<const bf16x8_t*>(Bs + lds_offset<GEMM_BK>(wn * (BN / WN) + j * 32 + frag_row, kk + frag_k));
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[j], af[i], acc[i][j], 0, 0, 0);
      }
    };
    // column sums of the B slab in LDS (rows of Bs are columns n; the slot permutation only reorders k)
    auto colsum_slab = [&](const bf16_t* Bs, int k0) {
      if constexpr (Epilogue::COLSUM) if (want_colsum && (int)threadIdx.x < BN && k0 < g.colsum_k) {
        const bool whole = k0 + GEMM_BK <= g.colsum_k;   // (uniform: only the slab that straddles the limit masks)
#pragma unroll
        for (int ks = 0; ks < GEMM_BK; ks += 8) {
          const uint4 v = *reinterpret_cast<const uint4*>(Bs + lds_offset<GEMM_BK>((int)threadIdx.x, ks));
          const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const float lo = __uint_as_float(w[q] << 16), hi = __uint_as_float(w[q] & 0xffff0000u);
            csum += whole || k0 + ks + 2 * q < g.colsum_k ? lo : 0.f;
            csum += whole || k0 + ks + 2 * q + 1 < g.colsum_k ? hi : 0.f;
          }
        }
      }
    };
    if constexpr (DOUBLE_BUF) {
      // slab s+1 goes from registers into the other LDS buffer and slab s+2 leaves for the registers
      // before slab s is multiplied: one barrier per slab, and a load has a whole slab's MFMAs to land
      fetch_slab(0);
      la.store(smem);
      lb.store(smem + BM * GEMM_PITCH);
      if (GEMM_BK < g.K) fetch_slab(GEMM_BK);
      __syncthreads();
      int buf = 0;
      for (int k0 = 0; k0 < g.K; k0 += GEMM_BK, buf ^= 1) {
        if (k0 + GEMM_BK < g.K) {
          la.store(smem + (buf ^ 1) * SLAB);
          lb.store(smem + (buf ^ 1) * SLAB + BM * GEMM_PITCH);
          if (k0 + 2 * GEMM_BK < g.K) fetch_slab(k0 + 2 * GEMM_BK);
        }
        multiply_slab(smem + buf * SLAB, smem + buf * SLAB + BM * GEMM_PITCH);
        colsum_slab(smem + buf * SLAB + BM * GEMM_PITCH, k0);
        __syncthreads();
      }
    } else {
      fetch_slab(0);
      for (int k0 = 0; k0 < g.K; k0 += GEMM_BK) {
        __syncthreads();  // previous slab fully consumed
        la.store(smem);
        lb.store(smem + BM * GEMM_PITCH);
        __syncthreads();
        if (k0 + GEMM_BK < g.K) fetch_slab(k0 + GEMM_BK);
        multiply_slab(smem, smem + BM * GEMM_PITCH);
        colsum_slab(smem + BM * GEMM_PITCH, k0);
      }
    }
  };
  // (uniform over the launch: a ragged K needs the zero fill of the guarded loads; ragged M or N only
  // needs in-bounds addresses, unless the operand is stored eight rows per 16 bytes and does not end on one)
  const bool a_rows_ok = A_MCONTIG ? (g.M % 8 == 0 && g.M >= 8) : true;
  const bool b_rows_ok = B_KCONTIG ? true : (g.b_cols % 8 == 0 && g.b_cols >= 8);
  if (g.K % GEMM_BK == 0 && a_rows_ok && b_rows_ok) k_loop(std::true_type{});
  else k_loop(std::false_type{});

  if constexpr (Epilogue::COLSUM) if (want_colsum && (int)threadIdx.x < BN && n0 + (int)threadIdx.x < g.N)
    g.colsum[(int64_t)member * g.colsum_stride + n0 + threadIdx.x] = csum;

  // Epilogue.  The MFMAs above take the B fragment as their first operand, so an accumulator block
  // holds the transposed product: lane -> row m (lane % 32) of C, register e -> column
  // 8*(e/4) + 4*(lane/32) + e%4, i.e. a lane holds runs of four consecutive columns.  To reach memory
  // with 16-byte accesses of whole 128-byte rows, every wavefront passes its accumulators, one row of
  // 32x32 blocks at a time, through a private LDS region (16-byte writes, no conflicts at a pitch of
  // 4 mod 64 floats) and reads them back as runs of 8 consecutive columns for the functor.  LDS
  // operations of one wavefront execute in order, so no workgroup barrier is needed between strips.
  constexpr int CPITCH = WCOLS + 4, RUNS = WCOLS / 8;
  static_assert(WM * WN * 32 * CPITCH * 4 <= SLAB * 2, "C strips must fit the slab LDS");
  float* const Cw = reinterpret_cast<float*>(smem) + wave * 32 * CPITCH;
  fetch_first_strip(EARLY_RUNS, NQ4);
  float colv[8];   // (a lane handles the same eight columns in every run)
  if constexpr (!Epilogue::PREFETCH) if constexpr (Epilogue::HAS_COLS) {
    static_assert(64 % RUNS == 0, "a lane's runs must share their columns");
    epi.load_cols(n0 + wn * WCOLS + (lane % RUNS) * 8, g.N, colv);
  }
  __syncthreads();  // every wavefront is done with the slabs
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    // a functor that reads what it updates asks for all of a strip's runs first, so that their
    // latencies overlap each other and the staging below
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<float4*>(Cw + (lane & 31) * CPITCH + j * 32 + 8 * q + 4 * (lane >> 5)) =
            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if constexpr (Epilogue::PREFETCH) {
#pragma unroll
      for (int q = 0; q < NQ4; ++q) {
        const int run = q * 64 + lane;
        const int row = run / RUNS4, col = (run % RUNS4) * 4;
        const int m = m0 + wm * (BM / WM) + i * 32 + row, n = n0 + wn * WCOLS + col;
        const float4 x = *reinterpret_cast<const float4*>(Cw + row * CPITCH + col);
        if (m < g.M && n < g.N) {
          const float v[4] = {x.x, x.y, x.z, x.w};
          epi.apply4_fetched(pre[q], m, n, v, g.N - n < 4 ? g.N - n : 4);
        }
        // the registers of this run are free again: the same run of the next strip goes into them
        if (i + 1 < TM && m + 32 < g.M && n < g.N) pre[q] = epi.fetch(m + 32, n, g.N - n < 4 ? g.N - n : 4);
      }
    } else {
#pragma unroll
      for (int q = 0; q < 32 * RUNS / 64; ++q) {
        const int run = q * 64 + lane;
        const int row = run / RUNS, col = (run % RUNS) * 8;
        const int m = m0 + wm * (BM / WM) + i * 32 + row, n = n0 + wn * WCOLS + col;
        const float4 lo = *reinterpret_cast<const float4*>(Cw + row * CPITCH + col);
        const float4 hi = *reinterpret_cast<const float4*>(Cw + row * CPITCH + col + 4);
        const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        const bool inside = m < g.M && n < g.N;
        const int count = inside ? min(g.N - n, 8) : 0;
        const int64_t o = (int64_t)m * epi.pitch() + n;
        typename Epilogue::Data data{};
        if constexpr (Epilogue::HAS_DATA) if (inside) data = epi.load_run(m, n, o, count);
        if constexpr (Epilogue::ROWWISE) epi.template put_row<false, RUNS>(m, n, v, count, colv, data);
        else if (inside) epi.template put<false>(m, n, o, v, count, colv, data);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  if constexpr (!Epilogue::PREFETCH) if constexpr (Epilogue::HAS_FINISH) {
    __syncthreads();   // (every wavefront is done with its strip)
    epi.finish(member, tile, g.tiles, reinterpret_cast<float*>(smem));
  }
}

// Weight gradient with the optimiser applied in place: v = dW[m][n .. n+3] never goes to memory;
// the run of theta, its optimiser state and the bf16 shadow is read, updated and written back
// (16-byte streaming accesses).  Saves writing and re-reading the gradient (8 of 34 bytes per
// parameter and step).  The layer's input-gradient GEMM must already have read the bf16 shadow.
template <int OPT>
struct EpiOptimizer {
  static constexpr bool PREFETCH = true;
  static constexpr bool COLSUM = true;
  static constexpr int LAYOUTS = 4;
  struct Fetched { float w[4], s0[4], s1[4]; };  // one run of theta and its state, read ahead of use
  float* W32; float* S0; float* S1; bf16_t* W16;
  int64_t stride, off, ldc;   // member stride, offset of the matrix in the member's vector, row pitch
  OptHyper hy;
  OptScalars sc;
  __device__ __forceinline__ void begin(int member) { sc = opt_scalars<OPT>(hy, member); off += (int64_t)member * stride; }
  __device__ __forceinline__ Fetched fetch(int m, int n, int count) const {
    Fetched f;
    const int64_t o = off + (int64_t)m * ldc + n;
    if (count == 4 && (o & 3) == 0) {
      const float4 a = stream_load(W32 + o), b = stream_load(S0 + o);
      f.w[0] = a.x; f.w[1] = a.y; f.w[2] = a.z; f.w[3] = a.w;
      f.s0[0] = b.x; f.s0[1] = b.y; f.s0[2] = b.z; f.s0[3] = b.w;
      if (OPT == OPT_ADAM) {
        const float4 c = stream_load(S1 + o);
        f.s1[0] = c.x; f.s1[1] = c.y; f.s1[2] = c.z; f.s1[3] = c.w;
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        f.w[e] = e < count ? W32[o + e] : 0.f;
        f.s0[e] = e < count ? S0[o + e] : 0.f;
        f.s1[e] = (OPT == OPT_ADAM && e < count) ? S1[o + e] : 0.f;
      }
    }
    return f;
  }
  __device__ __forceinline__ void apply4_fetched(Fetched& f, int m, int n, const float* v, int count) const {
    const int64_t o = off + (int64_t)m * ldc + n;
#pragma unroll
    for (int e = 0; e < 4; ++e) opt_update<OPT>(f.w[e], e < count ? v[e] : 0.f, f.s0[e], f.s1[e], sc, hy);
    if (count == 4 && (o & 3) == 0) {
      stream_store(make_float4(f.w[0], f.w[1], f.w[2], f.w[3]), W32 + o);
      stream_store(make_float4(f.s0[0], f.s0[1], f.s0[2], f.s0[3]), S0 + o);
      if (OPT == OPT_ADAM) stream_store(make_float4(f.s1[0], f.s1[1], f.s1[2], f.s1[3]), S1 + o);
      if (W16) *reinterpret_cast<uint2*>(W16 + o) = make_uint2(f2bf_pair(f.w[0], f.w[1]), f2bf_pair(f.w[2], f.w[3]));
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (e < count) {
          W32[o + e] = f.w[e];
          S0[o + e] = f.s0[e];
          if (OPT == OPT_ADAM) S1[o + e] = f.s1[e];
          if (W16) W16[o + e] = f2bf(f.w[e]);
        }
    }
  }
};

// Tile shapes of the weight gradients with the optimiser in the epilogue: 128x128 (four wavefronts, three workgroups per compute unit) unless that leaves
// the 256 compute units with fewer than four workgroups each to hide the optimiser's latency with; then 128x64; 64x64 for at most 64 rows or
// where 128x64 tiles are fewer than two per compute unit; 256x256 (eight wavefronts, LDS slabs double-buffered) for contractions of at least 1024
// over large matrices.  Per step with the rule, and with 64x64, 128x64, 128x128 and 256x256 tiles throughout (us, Adam):
//   64 members 256-1024-1024-10, 128 rows     548    542   548   548   636
//   the same, 1024 rows                      1244   1236  1217  1185  1242
//   8 members 1024-2048-2048-10, 2048 rows    993   1048  1037   984   994
//   21 members 200-712-360-7, 75 rows         132    131   132   127   205
//   16 members 128-512-512-10, 64 rows         77     73    83    93   159
//   64 members 64-64-64-4, 64 rows             48     48    54    64    82
//   32 GANs 128-512-512-784, 64 rows          448    417   454   442   571
//   128 agents 512-256-256-19, 672 rows       436    418   435   421   444
// (64x64 tiles would take more of the short contractions than the rule gives them, 128x128 the long ones it gives to 256x256.)
enum GemmTile { TILE_128x64 = 0, TILE_128x128, TILE_256x256, TILE_64x64 };
inline GemmTile choose_tile(int M, int N, int K, int batch) {
  constexpr int CUS = 256;
  if (K >= 1024 && M > 128 && N > 128 && tile_count(M, N, batch, 256, 256) >= CUS * 3 / 4) return TILE_256x256;
  if (M <= 64 || tile_count(M, N, batch, 128, 64) < 2 * CUS) return TILE_64x64;
  if (tile_count(M, N, batch, 128, 128) < 4 * CUS || N <= 64) return TILE_128x64;
  return TILE_128x128;
}

template <int BM, int BN, int BK, int WM, int WN, bool DOUBLE_BUF, bool A_M, bool B_K, class Epilogue>
hipError_t launch_gemm_kernel(const GemmArgs& g, const Epilogue& epi, hipStream_t stream) {
  constexpr int SLAB_BYTES = (BM + BN) * gemm_pitch(BK) * 2;
  constexpr int LDS_BYTES = SLAB_BYTES * (DOUBLE_BUF ? 2 : 1);
  constexpr auto kernel = gemm_bf16_kernel<BM, BN, BK, WM, WN, A_M, B_K, DOUBLE_BUF, Epilogue>;
  if constexpr (LDS_BYTES > 64 * 1024) {
    const hipError_t e = allow_lds<kernel>(LDS_BYTES);
    if (e != hipSuccess) return e;
  }
  const int64_t total = (int64_t)g.tiles * g.batch;
  hipLaunchKernelGGL(kernel, dim3((unsigned)total), dim3(WM * WN * 64), LDS_BYTES, stream, g, epi);
  return hipGetLastError();
}

template <int BM, int BN, int BK, int WM, int WN, bool DOUBLE_BUF, class Epilogue>
hipError_t launch_gemm_tile(const GemmArgs& g0, bool a_m_contig, bool b_k_contig, const Epilogue& epi, hipStream_t stream) {
  GemmArgs g = g0;
  if (g.upper || (g.colsum && (!Epilogue::COLSUM || b_k_contig))) return hipErrorInvalidValue;
  g.tiles_m = (g.M + BM - 1) / BM;
  g.tiles_n = (g.N + BN - 1) / BN;
  g.tiles = g.tiles_m * g.tiles_n;
  const int64_t total = (int64_t)g.tiles * g.batch;
  if (total <= 0 || total > 0x7fffffff) return hipErrorInvalidValue;
  // operand layouts as bits of Epilogue::LAYOUTS: 1 both row-major, 2 B K-contiguous, 4 A M-contiguous, 8 both (only those a caller uses
  // with the functor are compiled)
  const int layout = (a_m_contig ? 2 : 0) + (b_k_contig ? 1 : 0);
  if constexpr (Epilogue::LAYOUTS & 1) if (layout == 0) return launch_gemm_kernel<BM, BN, BK, WM, WN, DOUBLE_BUF, false, false>(g, epi, stream);
  if constexpr (Epilogue::LAYOUTS & 2) if (layout == 1) return launch_gemm_kernel<BM, BN, BK, WM, WN, DOUBLE_BUF, false, true>(g, epi, stream);
  if constexpr (Epilogue::LAYOUTS & 4) if (layout == 2) return launch_gemm_kernel<BM, BN, BK, WM, WN, DOUBLE_BUF, true, false>(g, epi, stream);
  if constexpr (Epilogue::LAYOUTS & 8) if (layout == 3) return launch_gemm_kernel<BM, BN, BK, WM, WN, DOUBLE_BUF, true, true>(g, epi, stream);
  return hipErrorInvalidValue;
}

// Host-side launcher.  Caller guarantees 16-byte alignment of pitches / strides / bases.  (Functors other than the optimiser come here for rows of 2^24
// elements or more only: one tile shape serves them.)
template <class Epilogue>
hipError_t launch_gemm_bf16(const GemmArgs& g, bool a_m_contig, bool b_k_contig, const Epilogue& epi, hipStream_t stream) {
  if constexpr (!Epilogue::PREFETCH) return launch_gemm_tile<64, 64, 64, 2, 2, false, Epilogue>(g, a_m_contig, b_k_contig, epi, stream);
  else switch (choose_tile(g.M, g.N, g.K, g.batch)) {
    case TILE_256x256: return launch_gemm_tile<256, 256, 64, 2, 4, true, Epilogue>(g, a_m_contig, b_k_contig, epi, stream);
    case TILE_64x64: return launch_gemm_tile<64, 64, 64, 2, 2, false, Epilogue>(g, a_m_contig, b_k_contig, epi, stream);
    case TILE_128x64: return launch_gemm_tile<128, 64, 64, 2, 2, false, Epilogue>(g, a_m_contig, b_k_contig, epi, stream);
    default: return launch_gemm_tile<128, 128, 64, 2, 2, false, Epilogue>(g, a_m_contig, b_k_contig, epi, stream);
  }
}

}  // namespace pbt
