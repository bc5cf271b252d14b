// The population-batched GEMM with operands that go from memory straight into LDS, for every operand layout.
//
// Slabs of 64 k (128-byte rows: whole cache lines) are moved by buffer loads with an LDS destination: a wavefront
// instruction fills 1 KB of LDS, lane l its bytes 16 l .. 16 l + 15, and nothing passes through registers.  What lies outside the
// operand (a ragged last tile, a K that is no multiple of the slab) is given an offset past the buffer's end, which the
// hardware's range check turns into zeros, so one K loop serves every size.  A K-contiguous operand lies in LDS as [row][64 k] and is
// read with 16-byte reads; an M- or N-contiguous one lies as [k][rows] and is read with gfx950's transposing reads
// (ds_read_b64_tr_b16: sixteen lanes fetch 4 k x 16 rows and each receives one row's four k).  In both the 16-byte chunks of an LDS row are
// permuted (by the choice of what each lane fetches) so that the lanes of a read cycle touch different banks.
//
// The A and the B slabs have rings of their own, NA and NB deep.  One barrier per slab: before it a wavefront waits for its own part of the
// next slab (loads return in order, so a count of younger loads says that) and for its last LDS reads; behind it the slab's slots are
// refilled, the loads spread between the MFMAs (issued in one burst they held the wavefront: 3520-4050 instead of 3160-3330 cycles per slab of 64).  LDS
// reads of the next MFMA group are issued before the MFMAs of the current one.
//
// What bounds it: 4096 x 4096 x 4096, four members, 256x256 tiles: 440 us = 1.25 PFLOP/s at the 1.9 GHz the clock falls to (register-staged kernel:
// 500 us; its loads alone take 285 us, its MFMAs alone 330).  Short contractions add the epilogue, which a persistent workgroup does not overlap with its
// products: 16 members' 4096 x 2048 x 512, plain epilogue: 150 us alone (197 register-staged), 180 (216) inside a transformer's pass.
//
// The loads are issued as assembly (they have no register result): the compiler, which cannot tell the slots apart, would wait for all
// of them before any LDS read.
#pragma once
#include "gemm_epilogues.h"

namespace pbt {

typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));

constexpr uint32_t GL_OUTSIDE = 0x80000000u;   // a byte offset past the end of every buffer

typedef __attribute__((address_space(3))) bf16_t lds_bf16_t;

// 64 lanes x 16 bytes from buffer[voff + soff] to LDS bytes lds .. lds + 1023.  (The waits: one state between the write of m0 and its use, five if
// a scalar operand came from a vector instruction.)
__device__ __forceinline__ void load_to_lds(uint32_t lds, uint32_t voff, i32x4_t rsrc, uint32_t soff) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}

// One operand: ROWS along M or N.  KC: memory is [row][k]; otherwise [k][row].
template <int ROWS, int BK, bool KC, int WAVES>
struct GlSide {
  static constexpr int SLOT = ROWS * BK * 2;             // bytes of one slab
  static constexpr int LOADS = SLOT / 1024 / WAVES;         // wavefront instructions per wavefront and slab
  static constexpr int KROWS = 1024 / (ROWS * 2);           // k rows per instruction (row-contiguous operand)
  static_assert(LOADS >= 1 && SLOT % (1024 * WAVES) == 0 && WAVES % 2 == 0, "a slab must divide evenly over the wavefronts");
  uint64_t addr;        // where the buffer begins: the tile's first row (K-contiguous), or the slab's first k
  int64_t left;         // bytes from there to the operand's end
  uint32_t voff[LOADS];
  int kofs;             // k of this lane's first load inside the slab
  int64_t slab_bytes;   // from a slab's first k to the next one's (row-contiguous operand)

  static __device__ __forceinline__ int chunk_swap(int krow) { return ROWS >= 128 ? (krow & 3) << 2 : ((krow >> 1) & 1) << 2; }

  // base: the batch element's operand; nrows and K bound it
  __device__ __forceinline__ void set_tile(const bf16_t* base, int64_t ld, int row0, int nrows, int K, int wave, int lane) {
    addr = reinterpret_cast<uint64_t>(base + (KC ? (int64_t)row0 * ld : 0));
    // (the range check works on whole dwords: an odd last element's lies in the same one)
    left = (2 * (KC ? (int64_t)(nrows - 1 - row0) * ld + K : (int64_t)(K - 1) * ld + nrows) + 3) & ~(int64_t)3;
    slab_bytes = (int64_t)BK * ld * 2;
    if constexpr (KC) {
      // BK = 64: 8 rows of 8 chunks per instruction, chunk c of row r lies at c ^ ((r >> 1) & 7); BK = 32: 16 rows of 4, at c ^ ((r >> 2) & 3)
      const int chunk = BK == 64 ? (lane & 7) ^ (((wave & 1) << 2) | (lane >> 4)) : (lane & 3) ^ (lane >> 4);
      kofs = chunk * 8;
#pragma unroll
      for (int j = 0; j < LOADS; ++j) {
        const int row = (wave + WAVES * j) * (512 / BK) + lane / (BK / 8);
        voff[j] = row0 + row < nrows ? (uint32_t)(row * (int)ld + chunk * 8) * 2u : GL_OUTSIDE;
      }
    } else {
      kofs = wave * KROWS + lane / (ROWS / 8);
#pragma unroll
      for (int j = 0; j < LOADS; ++j) {
        const int k = kofs + WAVES * KROWS * j;
        const int row = row0 + ((lane % (ROWS / 8)) ^ chunk_swap(k)) * 8;
        voff[j] = row < nrows ? (uint32_t)(k * (int)ld + row) * 2u : GL_OUTSIDE;
      }
    }
  }
  // load j of the slab at k0 (the last one moves on to the next slab)
  __device__ __forceinline__ void issue(uint32_t slot, int k0, int K, int wave, int j) {
    uint32_t v = voff[j];
    if (k0 + BK > K && k0 + kofs + (KC ? 0 : WAVES * KROWS * j) >= K) v = GL_OUTSIDE;
    const i32x4_t rsrc = {(int)(uint32_t)addr, (int)(uint32_t)(addr >> 32), (int)(left < 0x7fffffff ? left : 0x7fffffff), 0x00020000};
    load_to_lds(slot + (uint32_t)(wave + WAVES * j) * 1024u, v, rsrc, KC ? (uint32_t)k0 * 2u : 0u);
    if (!KC && j + 1 == LOADS) {
      addr += (uint64_t)slab_bytes;
      left -= slab_bytes;
    }
  }
};

// K-contiguous operand whose K is no multiple of 8: the chunk that straddles K came with what lies behind the row's end; its lane clears that
template <class Side>
__device__ __forceinline__ void clear_past_k(const Side& side, lds_bf16_t* smem, uint32_t slot, int loads, int waves, int k0, int K, int wave, int lane) {
  const int left = K - (k0 + side.kofs);   // elements of the lane's chunk that exist
  if (left <= 0 || left >= 8) return;
  for (int j = 0; j < loads; ++j) {
    lds_bf16_t* p = (lds_bf16_t*)((__attribute__((address_space(3))) char*)smem + slot + (wave + waves * j) * 1024 + lane * 16);
    for (int e = left; e < 8; ++e) p[e] = 0;
  }
}

// Fragments of a side: T blocks of 32 rows starting at row `first` of the slab.
template <int ROWS, int BK, bool KC, int T>
struct GlFrag {
  static constexpr int ADDRS = KC ? BK / 16 : T;   // KC: one per 16-wide step (a block of 32 rows is a constant apart); otherwise one per block
  uint32_t addr[ADDRS];
  __device__ __forceinline__ void init(int first, int lane) {
    const int half = lane >> 5;
    if constexpr (KC) {
      const int r = lane & 31, f = BK == 64 ? (r >> 1) & 7 : (r >> 2) & 3;
#pragma unroll
      for (int st = 0; st < BK / 16; ++st) addr[st] = (uint32_t)((first + r) * (BK * 2) + (((2 * st + half) ^ f) << 4));
    } else {
      const int j = lane & 15, g = (lane >> 4) & 1;
      const int swap = ROWS >= 128 ? (j >> 2) << 2 : (j >> 3) << 2;
#pragma unroll
      for (int i = 0; i < T; ++i) {
        const int chunk = ((first + 32 * i) >> 3) + 2 * g + ((j & 3) >> 1);
        addr[i] = (uint32_t)((8 * half + (j >> 2)) * (ROWS * 2) + ((chunk ^ swap) << 4) + ((j & 1) << 3));
      }
    }
  }
  __device__ __forceinline__ void read(bf16x8_t* f, const lds_bf16_t* smem, uint32_t slot, int st) const {
#pragma unroll
    for (int i = 0; i < T; ++i) {
      if constexpr (KC) {
        const auto* p = (const __attribute__((address_space(3))) char*)smem + slot + addr[st] + i * (32 * BK * 2);
        f[i] = *(const __attribute__((address_space(3))) bf16x8_t*)p;
      } else {
        auto* p = (__attribute__((address_space(3))) char*)smem + slot + addr[i] + st * (16 * ROWS * 2);
        const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)p);
        const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)(p + 4 * ROWS * 2));
        f[i] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      }
    }
  }
};

// A tile shape: WM x WN wavefronts, rings of NA and NB slabs.  PERSISTENT: one workgroup per compute unit walks over several tiles, the next tile's
// first slabs on their way while the epilogue of the last one runs.
template <int BM_, int BN_, int BK_, int WM_, int WN_, int NA_, int NB_, bool PERSISTENT_>
struct GlTile {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_, NA = NA_, NB = NB_;
  static constexpr bool PERSISTENT = PERSISTENT_;
  static constexpr int WAVES = WM * WN, THREADS = WAVES * 64;
  static constexpr int LDS_BYTES = (BM * NA + BN * NB) * BK * 2;
  static constexpr int STRIP_BYTES = WAVES * 32 * (BN / WN) * 4;   // the epilogue's strips
  // what a launch over K needs
  static int lds_bytes(int K) {
    const int slabs = (K + BK - 1) / BK;
    if (PERSISTENT || NA != NB || slabs >= NA) return LDS_BYTES;
    const int bytes = slabs * (BM + BN) * BK * 2;
    return bytes > STRIP_BYTES ? bytes : STRIP_BYTES;
  }
  static constexpr int PER_CU = PERSISTENT ? 1 : (160 * 1024) / LDS_BYTES;   // workgroups per compute unit that LDS admits
  static constexpr int WAVES_PER_SIMD = PER_CU * WAVES / 4 < 1 ? 1 : PER_CU * WAVES / 4 > 4 ? 4 : PER_CU * WAVES / 4;
  static_assert(NA == NB || NA == NB + 1, "the wait counts below are written for these");
};

template <int N>
__device__ __forceinline__ void gl_wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

template <class T, bool A_KC, bool B_KC, class Epilogue>
__global__ __launch_bounds__(T::THREADS, T::WAVES_PER_SIMD) void gemm_lds_kernel(GemmArgs g, Epilogue epi0) {
  constexpr int BM = T::BM, BN = T::BN, BK = T::BK, STEPS = BK / 16, WM = T::WM, WN = T::WN, NA = T::NA, NB = T::NB;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32, WAVES = T::WAVES;
  typedef GlSide<BM, BK, A_KC, WAVES> SideA;
  typedef GlSide<BN, BK, B_KC, WAVES> SideB;
  static_assert(!std::is_same_v<Epilogue, EpiRbfSum> || BM == BN, "the tiles of a symmetric product");
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  lds_bf16_t* const lds = (lds_bf16_t*)smem;
  const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
  // Rings of equal depth lie slab by slab (a launch with fewer slabs than slots needs only theirs), otherwise B's behind A's.
  constexpr uint32_t A_STEP = SideA::SLOT + (NA == NB ? SideB::SLOT : 0), A_END = NA * A_STEP;
  constexpr uint32_t B_BASE = NA == NB ? SideA::SLOT : A_END, B_STEP = SideB::SLOT + (NA == NB ? SideA::SLOT : 0), B_END = B_BASE + NB * B_STEP;

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int K = g.K, n_slabs = (K + BK - 1) / BK;

  // tiles of this workgroup: t, t + stride, ... < t_end.  Workgroups go to the 8 XCDs round-robin; each XCD gets a contiguous run.
  const int total = g.tiles * g.batch;
  int t, t_end, stride;
  if (!T::PERSISTENT || (int)gridDim.x == total) {
    t = xcd_remap(blockIdx.x, total);
    t_end = t + 1;
    stride = 1;
  } else {
    const int xcd = blockIdx.x & 7;
    t = (int)((int64_t)total * xcd / 8) + (blockIdx.x >> 3);
    t_end = (int)((int64_t)total * (xcd + 1) / 8);
    stride = gridDim.x >> 3;
  }
  if (t >= t_end) return;

  auto locate = [&](int id, int& member, int& tile, int& m0, int& n0) {
    member = g.by_tiles.divide(id);
    id -= member * g.tiles;
    tile = id;
    if (std::is_same_v<Epilogue, EpiRbfSum> && g.upper) {
      // (only tiles on the diagonal or right of it)
      int tm = 0;
      for (; id >= g.tiles_n - tm; ++tm) id -= g.tiles_n - tm;
      m0 = tm * BM;
      n0 = (tm + id) * BN;
      return;
    }
    const int group = g.by_group.divide(id), first_m = group * GROUP_M;
    id -= first_m * g.tiles_n;
    const bool last = g.tiles_m - first_m < GROUP_M;
    const int col = last ? g.by_last.divide(id) : id / GROUP_M;
    m0 = (first_m + id - col * (last ? g.tiles_m - first_m : GROUP_M)) * BM;
    n0 = col * BN;
  };

  // where the next slab of either operand comes from and goes to
  SideA la;
  SideB lb;
  int ta = t, ka = 0, tb = t, kb = 0;
  uint32_t slot_a = 0, slot_b = B_BASE;
  // (a batch element's operand begins at outer * s + rest * s_in)
  auto outer = [&](int member, int& rest) {
    const int q = g.by_inner.divide(member);
    rest = member - q * g.inner;
    return q;
  };
  auto set_a = [&]() {
    int member, tile, m0, n0;
    locate(ta, member, tile, m0, n0);
    int rest;
    const int q = outer(member, rest);
    la.set_tile(g.A + (int64_t)q * g.sa + (int64_t)rest * g.sa_in, g.lda, m0, g.M, K, wave, lane);
  };
  auto set_b = [&]() {
    int member, tile, m0, n0;
    locate(tb, member, tile, m0, n0);
    int rest;
    const int q = outer(member, rest);
    lb.set_tile(g.B + (int64_t)q * g.sb + (int64_t)rest * g.sb_in, g.ldb, n0, B_KC ? g.N : g.b_cols, K, wave, lane);
  };
  auto after_a = [](uint32_t slot) { return slot + A_STEP == A_END ? 0u : slot + A_STEP; };
  auto after_b = [](uint32_t slot) { return slot + B_STEP == B_END ? B_BASE : slot + B_STEP; };
  // load j of the next slab (the last one moves on); nothing when the work is done
  auto issue_a = [&](int j) {
    if (ta >= t_end) return;
    la.issue(lds0 + slot_a, ka, K, wave, j);
    if (j + 1 < SideA::LOADS) return;
    slot_a = after_a(slot_a);
    ka += BK;
    if (ka >= K) {
      ka = 0;
      ta += stride;
      if (T::PERSISTENT && ta < t_end) set_a();
    }
  };
  auto issue_b = [&](int j) {
    if (tb >= t_end) return;
    lb.issue(lds0 + slot_b, kb, K, wave, j);
    if (j + 1 < SideB::LOADS) return;
    slot_b = after_b(slot_b);
    kb += BK;
    if (kb >= K) {
      kb = 0;
      tb += stride;
      if (T::PERSISTENT && tb < t_end) set_b();
    }
  };
  auto issue_slab_a = [&]() {
#pragma unroll
    for (int j = 0; j < SideA::LOADS; ++j) issue_a(j);
  };
  auto issue_slab_b = [&]() {
#pragma unroll
    for (int j = 0; j < SideB::LOADS; ++j) issue_b(j);
  };

  GlFrag<BM, BK, A_KC, TM> fra;
  GlFrag<BN, BK, B_KC, TN> frb;
  fra.init(wm * (BM / WM), lane);
  frb.init(wn * (BN / WN), lane);
  uint32_t ra = 0, rb = B_BASE;   // slots that are being read
  bf16x8_t fa[2][TM], fb[2][TN];
  auto read_step = [&](int st) {
    fra.read(fa[st & 1], lds, ra, st);
    frb.read(fb[st & 1], lds, rb, st);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto next_slots = [&]() {
    ra = after_a(ra);
    rb = after_b(rb);
  };
  f32x16_t acc[TM][TN];
  // Column sums of B (the bias gradient beside a weight gradient) from the fragments of the first tile row: the WM wavefronts that hold the same columns
  // share its blocks.  csum[j]: the lane's column of block j, its half of the k.
  constexpr bool COLSUM = Epilogue::COLSUM && !B_KC;
  constexpr int CS_BLOCKS = (TN + WM - 1) / WM;
  constexpr bool CS_SPLIT = COLSUM && TN == 1 && WM == 2;   // one block: its two wavefronts take every other step (six
  // members' 192 x 192 from 720 rows 11.0 -> 9.0 us)
  static_assert(!CS_SPLIT || !T::PERSISTENT, "their sums meet when the workgroup is done");
  float csum[CS_BLOCKS];
  bool want_colsum = false;
  int cs_k = 0;   // k of the slab being multiplied
  auto colsum_step = [&](int st) {
    if constexpr (COLSUM) if (want_colsum) {
      // (a slab that reaches past colsum_k, which is rare, masks the fragment; doing that to every slab took as long as the loads: 14.4 us for six
      // members' 192 x 192 from 720 rows, 11.0 so)
      const bool whole = g.colsum_k >= K || cs_k + BK <= g.colsum_k;
#pragma unroll
      for (int b = 0; b < CS_BLOCKS; ++b)
#pragma unroll
        for (int w = 0; w < WM; ++w)
          if (w == wm && (CS_SPLIT ? st % 2 == w : b * WM + w < TN)) {
            u32x4_t v = __builtin_bit_cast(u32x4_t, fb[st & 1][!CS_SPLIT && b * WM + w < TN ? b * WM + w : 0]);
            if (__builtin_expect(!whole, 0)) {
              const int left = g.colsum_k - (cs_k + st * 16 + 8 * (lane >> 5));
#pragma unroll
              for (int q = 0; q < 4; ++q) v[q] &= 2 * q + 1 < left ? 0xffffffffu : 2 * q < left ? 0xffffu : 0u;
            }
            float f[8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              f[2 * q] = __uint_as_float(v[q] << 16);
              f[2 * q + 1] = __uint_as_float(v[q] & 0xffff0000u);
            }
            csum[b] += ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
          }
    }
  };

  // the MFMAs of a step, with n loads spread between them (a burst of them would hold the wavefront at its issue)
  auto mfma_step = [&](int st, int n, auto&& load) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int at = i * TN + j;
#pragma unroll
        for (int q = 0; q < n; ++q)
          if (q * TM * TN / n == at) {
            load(q);
            __builtin_amdgcn_sched_barrier(0);
          }
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[st & 1][j], fa[st & 1][i], acc[i][j], 0, 0, 0);
      }
    __builtin_amdgcn_s_setprio(0);
    colsum_step(st);
    __builtin_amdgcn_sched_barrier(0);
  };
  auto no_load = [](int) {};

  // slabs still to come after the one that is being waited for
  int to_come = ((t_end - t + stride - 1) / stride) * n_slabs - 1;
  // (tail: K ends inside a chunk of a K-contiguous operand, and the slab waited for, in slots a and b, is a tile's last)
  const bool ragged_k = (A_KC || B_KC) && (K & 7);
  auto clear_tail = [&](uint32_t a, uint32_t b) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const int k0 = (n_slabs - 1) * BK;
    if constexpr (A_KC) clear_past_k(la, lds, a, SideA::LOADS, WAVES, k0, K, wave, lane);
    if constexpr (B_KC) clear_past_k(lb, lds, b, SideB::LOADS, WAVES, k0, K, wave, lane);
  };
  auto wait_slab = [&]() {
    if constexpr (NA == NB + 1) {
      if (to_come >= 1) gl_wait_barrier<SideA::LOADS>();
      else gl_wait_barrier<0>();
    } else {
      constexpr int PER = SideA::LOADS + SideB::LOADS;
      const int younger = to_come < NA - 2 ? to_come : NA - 2;
      if (younger >= 6) gl_wait_barrier<PER * 6>();
      else if (younger == 5) gl_wait_barrier<PER * 5>();
      else if (younger == 4) gl_wait_barrier<PER * 4>();
      else if (younger == 3) gl_wait_barrier<PER * 3>();
      else if (younger == 2) gl_wait_barrier<PER * 2>();
      else if (younger == 1) gl_wait_barrier<PER>();
      else gl_wait_barrier<0>();
    }
    --to_come;
  };
  static_assert(NA <= 8, "the ladder above");

  set_a();
  set_b();
#pragma unroll
  for (int s = 0; s < NA; ++s) {
    issue_slab_a();
    if (s < NB) issue_slab_b();
  }
  if (ragged_k && n_slabs == 1) clear_tail(ra, rb);
  // (all but the first slab may still be on their way; the ring is full, or holds the whole work)
  if constexpr (NA == NB + 1) {
    if (to_come >= 2) gl_wait_barrier<NA * SideA::LOADS + NB * SideB::LOADS - SideA::LOADS - SideB::LOADS>();
    else gl_wait_barrier<0>();
    --to_come;
  } else {
    if (to_come >= NA - 1) {
      gl_wait_barrier<(NA - 1) * (SideA::LOADS + SideB::LOADS)>();
      --to_come;
    } else {
      wait_slab();
    }
  }
  read_step(0);
  bool a_due = false;   // a slab of A waits to be requested

  for (;;) {
    int member, tile, m0, n0;
    locate(t, member, tile, m0, n0);
    if constexpr (COLSUM) {
      want_colsum = g.colsum != nullptr && m0 == 0;
      cs_k = 0;
#pragma unroll
      for (int b = 0; b < CS_BLOCKS; ++b) csum[b] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
    // B's part of the slab that goes into the slots freed by the last barrier was requested beside the step behind that barrier; A's goes beside
    // step 0, and step 1 if another step follows it
    auto first_steps = [&]() {
      constexpr int H = STEPS > 2 ? (SideA::LOADS + 1) / 2 : SideA::LOADS;
      read_step(1);
      mfma_step(0, H, [&](int q) { if (a_due) issue_a(q); });
      if constexpr (STEPS > 2) {
        read_step(2);
        mfma_step(1, SideA::LOADS - H, [&](int q) { if (a_due) issue_a(H + q); });
        read_step(3);
        mfma_step(2, 0, no_load);
      }
      a_due = true;
    };
    for (int s = 1; s < n_slabs; ++s) {
      first_steps();
      if (ragged_k && s + 1 == n_slabs) clear_tail(after_a(ra), after_b(rb));
      wait_slab();
      next_slots();
      read_step(0);
      mfma_step(STEPS - 1, SideB::LOADS, issue_b);
      cs_k += BK;
    }
    first_steps();
    mfma_step(STEPS - 1, 0, no_load);
    if constexpr (COLSUM && !CS_SPLIT) if (want_colsum) {
#pragma unroll
      for (int b = 0; b < CS_BLOCKS; ++b) {
        const float sum = csum[b] + __shfl_xor(csum[b], 32, 64);
        const int j = b * WM + wm, n = n0 + wn * (BN / WN) + j * 32 + lane;
        if (j < TN && lane < 32 && n < g.N) g.colsum[(int64_t)member * g.colsum_stride + n] = sum;
      }
    }
    Epilogue epi = epi0;
    epi.begin(member);
    if constexpr (std::is_same_v<Epilogue, EpiRbfSum>) epi.region = !g.upper ? 0 : n0 < m0 + BM ? 1 : 2;
    constexpr int WCOLS = BN / WN, RUNS = WCOLS / 8, CBYTES = 32 * WCOLS * 4;
    static_assert(WCOLS == 64 || WCOLS == 32, "the strip's chunk permutation");
    // (a copy of the lane the compiler knows nothing about: it would compute the epilogue's addresses ahead of the first tile and keep them in
    // registers the K loop needs)
    int elane = lane;
    asm volatile("" : "+v"(elane));
    float colv[8];
    if constexpr (Epilogue::HAS_COLS) epi.load_cols(n0 + wn * WCOLS + (elane % RUNS) * 8, g.N, colv);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // every wavefront has read the last slab: its slots are free for the strips

    // Epilogue.  The MFMAs take the B fragment first, so a lane holds runs of four consecutive columns of row lane % 32.  Each wavefront
    // passes its accumulators, one row of 32x32 blocks at a time, through LDS of its own and reads them back as runs of eight columns.
    uint32_t strip;
    if constexpr (T::PERSISTENT) {
      static_assert(!T::PERSISTENT || (SideA::SLOT % CBYTES == 0 && WAVES * CBYTES <= SideA::SLOT + SideB::SLOT), "the strips lie in the last slab's slots");
      strip = wave * CBYTES < SideA::SLOT ? ra + wave * CBYTES : rb + (wave * CBYTES - SideA::SLOT);
    } else {
      static_assert(WAVES * CBYTES <= T::LDS_BYTES, "C strips must fit the LDS");
      strip = wave * CBYTES;
    }
    char* const Cw = reinterpret_cast<char*>(smem) + strip;
    // 16-byte chunk c of row r lies at chunk c ^ f(r): no bank conflicts on either side
    auto chunk_at = [&](int row, int chunk) { return Cw + row * (WCOLS * 4) + ((chunk ^ (WCOLS == 64 ? row & 15 : (row >> 1) & 7)) << 4); };
    constexpr int NRUN = 32 * RUNS / 64, RSTEP = 64 / RUNS;   // runs of eight columns per lane and strip, rows between two of them
    typedef typename Epilogue::Data Data;
    const int mlane = m0 + wm * (BM / WM) + elane / RUNS, ncol = n0 + wn * WCOLS + (elane % RUNS) * 8;
    const int64_t o0 = (int64_t)mlane * epi.pitch() + ncol;
    auto strips = [&](auto full_tag) {
      constexpr bool FULL = decltype(full_tag)::value;
      const int count = FULL ? 8 : min(max(g.N - ncol, 0), 8);
      int64_t o = o0;   // offset of the lane's first run of the strip
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        asm volatile("" : "+v"(o));   // (or the offsets of every strip are computed ahead and kept)
        auto offset = [&](int q) { return o + (int64_t)(q * RSTEP) * epi.pitch(); };
        auto load_run = [&](int q) {
          Data r{};
          const int m = mlane + i * 32 + q * RSTEP;
          if constexpr (Epilogue::HAS_DATA) if (FULL || (m < g.M && count > 0)) r = epi.load_run(m, ncol, offset(q), count);
          return r;
        };
        // what a functor reads per run is requested ahead: all of a strip's, or (on the general path, whose code is kept small) two runs'
        constexpr int AHEAD = FULL ? NRUN : 2;
        Data data[AHEAD];
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) data[q] = load_run(q);
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *reinterpret_cast<float4*>(chunk_at(elane & 31, j * 8 + 2 * q + (elane >> 5))) =
                make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        // (the next tile's first slabs have landed before the last strip's stores: what is still out at the top of the next tile is those stores alone)
        if constexpr (T::PERSISTENT) if (i == TM - 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        auto run = [&](int q, const Data& d) {
          const int row = q * RSTEP + elane / RUNS, m = mlane + i * 32 + q * RSTEP;
          const float4 lo = *reinterpret_cast<const float4*>(chunk_at(row, (elane % RUNS) * 2));
          const float4 hi = *reinterpret_cast<const float4*>(chunk_at(row, (elane % RUNS) * 2 + 1));
          const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
          if constexpr (Epilogue::ROWWISE) epi.template put_row<FULL, RUNS>(m, ncol, v, FULL || m < g.M ? count : 0, colv, d);
          else if (FULL || (m < g.M && count > 0)) epi.template put<FULL>(m, ncol, offset(q), v, count, colv, d);
        };
        if constexpr (FULL) {
#pragma unroll
          for (int q = 0; q < NRUN; ++q) {
            run(q, data[q]);
            if constexpr (T::PERSISTENT) __builtin_amdgcn_sched_barrier(0);
          }
        } else {
#pragma unroll 1
          for (int q = 0; q < NRUN; ++q) {
            Data next{};
            if (q + 2 < NRUN) next = load_run(q + 2);
            run(q, data[0]);
            data[0] = data[1];
            data[1] = next;
          }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        o += (int64_t)32 * epi.pitch();
      }
    };
    // (uniform over the workgroup: the tile lies inside C and 16-byte accesses are aligned)
    if (m0 + BM <= g.M && n0 + BN <= g.N && epi.vectors()) strips(std::true_type{});
    else strips(std::false_type{});
    if constexpr (Epilogue::HAS_FINISH) {
      __syncthreads();   // (every wavefront is done with its strip)
      epi.finish(member, tile, g.tiles, reinterpret_cast<float*>(smem) + (T::PERSISTENT ? ra / 4 : 0));
    }
    if constexpr (CS_SPLIT) if (want_colsum) {
      const float sum = csum[0] + __shfl_xor(csum[0], 32, 64);
      const int n = n0 + wn * (BN / WN) + lane;
      if (wm == 1 && lane < 32) *reinterpret_cast<float*>(Cw + lane * 4) = sum;   // (the wavefront is done with its strip)
      __syncthreads();
      if (wm == 0 && lane < 32 && n < g.N) g.colsum[(int64_t)member * g.colsum_stride + n] = sum + *reinterpret_cast<const float*>(Cw + WN * CBYTES + lane * 4);
    }
    if constexpr (!T::PERSISTENT) return;
    t += stride;
    if (t >= t_end) return;
    if (ragged_k && n_slabs == 1) clear_tail(after_a(ra), after_b(rb));
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the strips are read, and every wavefront's part of the next tile's first slab has landed
    --to_come;
    issue_slab_b();
    next_slots();
    read_step(0);
  }
}

// Tile shapes.  256x256: eight wavefronts, one persistent workgroup per compute unit with 160 KB of LDS; its epilogue has the compute unit to itself.  128x128
// and 64x64: four wavefronts, three workgroups per compute unit (128x64: two), one's epilogue beside the others' products.
// (128x256 tiles with four wavefronts, two workgroups per compute unit: 5 to 20 % slower than 256x256 with plain epilogues, no faster than 128x128
// with heavy ones.)
typedef GlTile<256, 256, 64, 2, 4, 3, 2, true> GlTile256;
typedef GlTile<128, 128, 32, 2, 2, 3, 3, false> GlTile128;
typedef GlTile<128, 64, 64, 2, 2, 3, 3, false> GlTile128x64;
typedef GlTile<64, 64, 64, 2, 2, 3, 3, false> GlTile64;

template <class T, bool A_KC, bool B_KC, class Epilogue>
hipError_t launch_gl_kernel(GemmArgs g, const Epilogue& epi, hipStream_t stream) {
  constexpr auto kernel = gemm_lds_kernel<T, A_KC, B_KC, Epilogue>;
  if constexpr (T::LDS_BYTES > 64 * 1024) {
    const hipError_t e = allow_lds<kernel>(T::LDS_BYTES);
    if (e != hipSuccess) return e;
  }
  const int64_t total = (int64_t)g.tiles * g.batch;
  g.by_tiles = Divisor(g.tiles);
  g.by_group = Divisor(GROUP_M * g.tiles_n);
  g.by_last = Divisor(g.tiles_m % GROUP_M ? g.tiles_m % GROUP_M : 1);
  g.by_inner = Divisor(g.inner);
  hipLaunchKernelGGL(kernel, dim3((unsigned)(T::PERSISTENT && total > 256 ? 256 : total)), dim3(T::THREADS), T::lds_bytes(g.K), stream, g, epi);
  return hipGetLastError();
}

template <class T, class Epilogue>
hipError_t launch_gl_tile(const GemmArgs& g0, bool a_m_contig, bool b_k_contig, const Epilogue& epi, hipStream_t stream) {
  GemmArgs g = g0;
  g.tiles_m = (g.M + T::BM - 1) / T::BM;
  g.tiles_n = (g.N + T::BN - 1) / T::BN;
  if (g.upper && (!std::is_same_v<Epilogue, EpiRbfSum> || g.M != g.N)) return hipErrorInvalidValue;
  g.tiles = g.upper ? gl_upper_tiles(g.N, {T::BM, T::BN}) : g.tiles_m * g.tiles_n;
  const int64_t total = (int64_t)g.tiles * g.batch;
  if (total <= 0 || total > 0x7fffffff) return hipErrorInvalidValue;
  // operand layouts as bits of Epilogue::LAYOUTS: 1 both row-major, 2 B K-contiguous, 4 A M-contiguous, 8 both (only those a caller uses
  // with the functor are compiled)
  const int layout = (a_m_contig ? 2 : 0) + (b_k_contig ? 1 : 0);
  if constexpr (Epilogue::LAYOUTS & 1) if (layout == 0) return launch_gl_kernel<T, true, false>(g, epi, stream);
  if constexpr (Epilogue::LAYOUTS & 2) if (layout == 1) return launch_gl_kernel<T, true, true>(g, epi, stream);
  if constexpr (Epilogue::LAYOUTS & 4) if (layout == 2) return launch_gl_kernel<T, false, false>(g, epi, stream);
  if constexpr (Epilogue::LAYOUTS & 8) if (layout == 3) return launch_gl_kernel<T, false, true>(g, epi, stream);
  return hipErrorInvalidValue;
}

// Caller guarantees 16-byte alignment of pitches, strides and bases (checked at the ABI).
template <class Epilogue>
hipError_t launch_gemm_lds(const GemmArgs& g, bool a_m_contig, bool b_k_contig, const Epilogue& epi, hipStream_t stream) {
  if (g.lda >= GL_MAX_PITCH || g.ldb >= GL_MAX_PITCH) return hipErrorInvalidValue;
  if (g.colsum && (!Epilogue::COLSUM || b_k_contig)) return hipErrorInvalidValue;
  switch (gl_choose(g.M, g.N, g.K, g.batch, Epilogue::HEAVY, std::is_same_v<Epilogue, EpiRbfSum>, g.lda > g.ldb ? g.lda : g.ldb, g.upper)) {
    case GL_256: return launch_gl_tile<GlTile256>(g, a_m_contig, b_k_contig, epi, stream);
    case GL_128: return launch_gl_tile<GlTile128>(g, a_m_contig, b_k_contig, epi, stream);
    case GL_128x64:
      if constexpr (!std::is_same_v<Epilogue, EpiRbfSum>) return launch_gl_tile<GlTile128x64>(g, a_m_contig, b_k_contig, epi, stream);
      return hipErrorInvalidValue;
    default: return launch_gl_tile<GlTile64>(g, a_m_contig, b_k_contig, epi, stream);
  }
}

}  // namespace pbt
