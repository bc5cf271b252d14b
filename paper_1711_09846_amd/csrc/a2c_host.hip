// The actor-critic workload (Section 4.1.1 of the PBT paper: A3C-style agents trained with RMSProp,
// learning rate and entropy cost adapted per member, evaluated by the last 10 episodic returns).
// Device kernels for the trajectory bookkeeping and the loss, and the host-side kernel sequence.
#include <cstring>
#include <type_traits>

#include "common.h"
#include "dense_host.h"
#include "philox.h"

namespace pbt {

constexpr int HIST_SLOTS = 10, HIST_PITCH = 12;  // ring of returns, slot 10 = count (int bits), slot 11 unused

// Per member: copies actions and rewards of the B drawn trajectories (the same Philox draws as the
// observation gather) and pushes the unroll's return (mean over trajectories of the summed
// rewards, accumulated in double in a fixed order) into the member's history ring.
__global__ __launch_bounds__(64) void a2c_fetch_aux_kernel(const int32_t* __restrict__ pool_act,
                                                           const float* __restrict__ pool_rew, int n_traj, int B, int T,
                                                           uint32_t step, uint32_t k0, uint32_t k1,
                                                           int32_t* __restrict__ act, float* __restrict__ rew,
                                                           float* __restrict__ hist) {
  const int i = blockIdx.x;
  __shared__ double tsum[64];
  double mean = 0.0;
  for (int r0 = 0; r0 < B; r0 += 64) {
    const int r = r0 + threadIdx.x;
    double sacc = 0.0;
    if (r < B) {
      const uint32_t x = philox4x32_10(step, (uint32_t)i, DOMAIN_BATCH, (uint32_t)r, k0, k1).x;
      const int64_t src = (int64_t)philox_bounded(x, (uint32_t)n_traj) * T;
      const int64_t dst = ((int64_t)i * B + r) * T;
      for (int t = 0; t < T; ++t) {
        act[dst + t] = pool_act[src + t];
        const float rv = pool_rew[src + t];
        rew[dst + t] = rv;
        sacc += (double)rv;
      }
    }
    tsum[threadIdx.x] = sacc;
    __syncthreads();
    if (threadIdx.x == 0)
      for (int k = 0; k < 64 && r0 + k < B; ++k) mean += tsum[k];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    float* hrow = hist + (int64_t)i * HIST_PITCH;
    const int n = __float_as_int(hrow[HIST_SLOTS]);
    hrow[n % HIST_SLOTS] = (float)(mean / (double)B);
    hrow[HIST_SLOTS] = __int_as_float(n + 1);
  }
}

// Loss and its gradient with respect to the head outputs, one workgroup per member.
// Phase 1: the rewards of the member's trajectories are brought into LDS by all threads, then one
//   thread per trajectory walks it backwards in place for the bootstrapped returns
//   R_T = V(s_T), R_t = r_t + gamma R_{t+1}.
// Phase 2 (one thread per transition) evaluates, with A_t = R_t - V_t and R_t constants,
//   loss_t = -A_t log pi(a_t) + value_cost (R_t - V_t)^2 - entropy_cost H_t
//   dlogit_c = ( -A_t (1[c = a_t] - pi_c) + entropy_cost pi_c (log pi_c + H_t) ) / n
//   dV_t = 2 value_cost (V_t - R_t) / n,   n = B T;  the bootstrap rows get zeros.
// out: head outputs float [P][B][T+1][32] (n_act logits, then the value).  The exponentials of a row
// are evaluated once and kept in registers.  The per-thread losses are combined in a fixed order
// (lane butterfly, then the wavefronts in order).
__global__ __launch_bounds__(1024) void a2c_loss_kernel(const float* __restrict__ out, const int32_t* __restrict__ act,
                                                        const float* __restrict__ rew, const float* __restrict__ H,
                                                        int n_hyper, int col_ent, int B, int T, int n_act, float gamma,
                                                        float value_cost, bf16_t* __restrict__ dout, float* __restrict__ loss) {
  extern __shared__ float Rl[];  // [B][T]
  __shared__ float wsum[16];
  const int i = blockIdx.x;
  const int threads = blockDim.x;
  const float ent_cost = H[i * n_hyper + col_ent];
  const float inv_n = 1.f / (float)(B * T);
  for (int e = threadIdx.x; e < B * T; e += threads) Rl[e] = rew[(int64_t)i * B * T + e];
  __syncthreads();
  for (int r = threadIdx.x; r < B; r += threads) {
    float R = out[(((int64_t)i * B + r) * (T + 1) + T) * 32 + n_act];
    for (int t = T - 1; t >= 0; --t) {
      R = Rl[r * T + t] + gamma * R;
      Rl[r * T + t] = R;
    }
  }
  __syncthreads();
  float lacc = 0.f;
  for (int idx = threadIdx.x; idx < B * (T + 1); idx += threads) {
    const int r = idx / (T + 1), t = idx - r * (T + 1);
    const float4* __restrict__ lg4 = reinterpret_cast<const float4*>(out + ((int64_t)i * B * (T + 1) + idx) * 32);
    uint4* __restrict__ d4 = reinterpret_cast<uint4*>(dout + ((int64_t)i * B * (T + 1) + idx) * 32);
    if (t == T) {
#pragma unroll
      for (int q = 0; q < 4; ++q) d4[q] = make_uint4(0, 0, 0, 0);
      continue;
    }
    float lg[32];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float4 x = lg4[q];
      lg[4 * q] = x.x; lg[4 * q + 1] = x.y; lg[4 * q + 2] = x.z; lg[4 * q + 3] = x.w;
    }
    const int a = act[((int64_t)i * B + r) * T + t];
    const float R = Rl[r * T + t];
    float v = 0.f, la = 0.f, mx = -INFINITY;
#pragma unroll
    for (int c = 0; c < 32; ++c) {
      if (c < n_act) mx = fmaxf(mx, lg[c]);
      if (c == n_act) v = lg[c];
      if (c == a) la = lg[c];
    }
    const float adv = R - v;
    float ex[32], se = 0.f;
#pragma unroll
    for (int c = 0; c < 32; ++c) {
      ex[c] = c < n_act ? expf(lg[c] - mx) : 0.f;
      se += ex[c];
    }
    const float lse = mx + logf(se), inv_se = 1.f / se;
    float ent = 0.f;
#pragma unroll
    for (int c = 0; c < 32; ++c)
      if (c < n_act) ent -= ex[c] * inv_se * (lg[c] - lse);
    lacc += -adv * (la - lse) + value_cost * adv * adv - ent_cost * ent;
    float dv[32];
#pragma unroll
    for (int c = 0; c < 32; ++c) {
      const float pi = ex[c] * inv_se, lp = lg[c] - lse;
      dv[c] = c < n_act ? (-adv * ((c == a ? 1.f : 0.f) - pi) + ent_cost * pi * (lp + ent)) * inv_n
              : c == n_act ? 2.f * value_cost * (v - R) * inv_n : 0.f;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
      d4[q] = make_uint4(f2bf_pair(dv[8 * q], dv[8 * q + 1]), f2bf_pair(dv[8 * q + 2], dv[8 * q + 3]),
                         f2bf_pair(dv[8 * q + 4], dv[8 * q + 5]), f2bf_pair(dv[8 * q + 6], dv[8 * q + 7]));
  }
  lacc = wave_sum(lacc);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = lacc;
  __syncthreads();
  if (threadIdx.x == 0) {
    float total = 0.f;
    for (int w = 0; w < threads / 64; ++w) total += wsum[w];
    loss[i] = total * inv_n;
  }
}

// score = mean of the last min(count, 10) returns (double accumulation), -inf when there are none
__global__ void a2c_score_kernel(const float* __restrict__ hist, int P, float* __restrict__ score) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P) return;
  const float* hrow = hist + (int64_t)i * HIST_PITCH;
  const int n = __float_as_int(hrow[HIST_SLOTS]);
  const int m = n < HIST_SLOTS ? n : HIST_SLOTS;
  if (m == 0) { score[i] = -INFINITY; return; }
  // oldest first, as a list that keeps the most recent entries would hold them
  double acc = 0.0;
  for (int k = 0; k < m; ++k) acc += (double)hrow[(n - m + k) % HIST_SLOTS];
  score[i] = (float)(acc / (double)m);
}

// scratch of the one-kernel unroll (below), in elements per member
static int64_t a2c_packed_elems(const pbt_config* c);
static int64_t a2c_draw_count(const pbt_config* c);

pbt_status a2c_check_and_plan(const pbt_config* c, Plan* pl, Carver* w) {
  A2CPlan& a = pl->a2c;
  const int L = c->n_layers;
  if (L < 2) return fail(nullptr, PBT_EUNSUPPORTED, "the actor-critic network needs at least one torso layer before its head");
  if (c->unroll < 1) return fail(nullptr, PBT_EINVAL, "unroll must be positive");
  // the step passes one optimiser-state array and no beta1 / decay columns to the update kernels
  if (c->optimizer != PBT_OPT_RMSPROP && c->optimizer != PBT_OPT_SGD_MOMENTUM)
    return fail(nullptr, PBT_EUNSUPPORTED, "the actor-critic workload is built for RMSProp and SGD with momentum");
  if ((int64_t)c->batch * c->unroll * 4 > 48 * 1024) return fail(nullptr, PBT_EUNSUPPORTED, "batch x unroll above 12288 transitions per member");
  if (c->dims[L] < 2 || c->dims[L] > 32) return fail(nullptr, PBT_EUNSUPPORTED, "head width (actions + value) must be 2..32");
  for (int l = 0; l < L; ++l)
    if (c->dims[l] % 8) return fail(nullptr, PBT_EUNSUPPORTED, "torso widths must be multiples of 8");
  if (!(c->gamma >= 0.f && c->gamma <= 1.f)) return fail(nullptr, PBT_EINVAL, "gamma outside [0, 1]");
  const int64_t P = c->P, R = (int64_t)c->batch * (c->unroll + 1);
  a.rows = (int)R;
  a.o_a[0] = w->take((size_t)P * R * c->dims[0] * 2);
  a.o_act = w->take((size_t)P * c->batch * c->unroll * 4);
  a.o_rew = w->take((size_t)P * c->batch * c->unroll * 4);
  // what only the update uses, and over it what only the unroll ahead of the update uses
  const Carver shared = *w;
  for (int l = 0; l < L - 1; ++l) {
    a.o_a[l + 1] = w->take((size_t)P * R * c->dims[l + 1] * 2);
    a.o_z[l] = w->take((size_t)P * R * c->dims[l + 1] * 2);
    a.o_dz[l] = w->take((size_t)P * R * c->dims[l + 1] * 2);
  }
  a.o_out = w->take((size_t)P * R * 32 * 4);
  a.o_dout = w->take((size_t)P * R * 32 * 2);
  a.o_lat = a.o_gout = a.o_packed = a.o_draws = 0;
  a.one_kernel = a.packed_in_grad = false;
  if (c->on_policy) {
    if (c->latent_dim < 1 || c->latent_dim > 64) return fail(nullptr, PBT_EINVAL, "latent_dim outside 1..64");
    // (LDS of the generator's kernels: the latents of a member's trajectories, plus an action each in the transition
    // kernel or a 64-component slab of the observation matrix, 65 doubles per latent component, in the observation kernel)
    if ((int64_t)c->batch * (c->latent_dim * 8 + 4) + (int64_t)c->latent_dim * 65 * 8 > 64 * 1024)
      return fail(nullptr, PBT_EUNSUPPORTED, "batch x latent_dim too large for the trajectory generator's LDS");
    if ((int64_t)R * c->dims[0] >= (1LL << 31)) return fail(nullptr, PBT_EUNSUPPORTED, "more than 2^31 observation elements per member");
    // The one-kernel unroll: draws made ahead, weights as matrix fragments.  Many parameters and few rows make the fragments larger than
    // the update's buffers; where that would push a step past the array of pbt_step_static, they lie over the gradients if they fit there, and if
    // the step is past it even so, the kernels of one round each do the unroll, in memory that the update has anyway: whatever fits the
    // array in one of these forms is run in it.  (22 members 320-128-256-3, 2 trajectories of 2 steps: 10.3 MB with fragments of their own.)
    const size_t packed = (size_t)(P * a2c_packed_elems(c)) * 2;
    auto carve = [&](bool one_kernel, bool in_grad) {
      Carver u = shared;
      a.one_kernel = one_kernel;
      a.packed_in_grad = in_grad;
      if (one_kernel) {
        a.o_draws = u.take((size_t)(P * a2c_draw_count(c)) * 8);
        a.o_packed = in_grad ? pl->o_grad : u.take(packed);
      } else {
        a.o_lat = u.take((size_t)P * c->batch * c->latent_dim * 8);
        for (int l = 1; l < L; ++l) a.o_ga[l] = u.take((size_t)P * c->batch * c->dims[l] * 2);
        a.o_gout = u.take((size_t)P * c->batch * 32 * 4);
      }
      return u.off > w->off ? u.off : w->off;
    };
    const bool covered = packed > 0, fits_grad = packed <= (size_t)P * pl->lay.stride * 4;
    size_t end = carve(covered, false);
    if (covered && end > PBT_STATIC_SCRATCH_BYTES) {
      if (fits_grad) end = carve(true, true);
      if (end > PBT_STATIC_SCRATCH_BYTES) end = carve(false, false);
      if (end > PBT_STATIC_SCRATCH_BYTES) end = carve(true, false);
    }
    w->off = end;
  }
  pl->step_scratch_bytes = w->off;
  return PBT_OK;
}

// Forward, loss, backward and update on the unroll that sits in the step's input buffers (observations in
// the first activation buffer, actions and rewards in theirs).
static pbt_status a2c_update(pbt_handle* h, hipStream_t s) {
  const pbt_config& c = h->cfg;
  const Plan& p = h->plan;
  const A2CPlan& a = p.a2c;
  const int P = c.P, B = c.batch, T = c.unroll, L = c.n_layers, R = a.rows;
  const int Kh = c.dims[L - 1], C = c.dims[L];
  const int64_t S = p.lay.stride;
  const Net net{L, c.dims, 0, c.act, PBT_ACT_NONE};
  bf16_t* A[PBT_MAX_DIMS]; bf16_t* Z[PBT_MAX_DIMS]; bf16_t* dZ[PBT_MAX_DIMS];
  for (int l = 0; l < L; ++l) { A[l] = h->sc<bf16_t>(a.o_a[l]); Z[l] = l < L - 1 ? h->sc<bf16_t>(a.o_z[l]) : nullptr; dZ[l] = l < L - 1 ? h->sc<bf16_t>(a.o_dz[l]) : nullptr; }
  const float* W32 = h->st<float>(p.o_w32);
  const bf16_t* W16 = h->st<bf16_t>(p.o_w16);
  float* G = h->sc<float>(p.o_grad);
  float* out = h->sc<float>(a.o_out);
  bf16_t* dout = h->sc<bf16_t>(a.o_dout);
  int32_t* act = h->sc<int32_t>(a.o_act);
  float* rew = h->sc<float>(a.o_rew);
  pbt_status st;
  if ((st = forward(h, net, L - 1, R, A, Z, nullptr, 0, s)) != PBT_OK) return st;
  PBT_LAUNCH(h, PBT_K_HEAD, s, head_fwd_loss(A[L - 1], (int64_t)R * Kh, W16 + p.lay.w_off[L - 1], S, W32 + p.lay.b_off[L - 1], S, nullptr,
                                             0, P, R, Kh, C, 0.f, -2, nullptr, out, 0, s));
  hipLaunchKernelGGL(a2c_loss_kernel, dim3(P), dim3(B * (T + 1) > 512 ? 1024 : B * (T + 1) > 256 ? 512 : 256), (size_t)B * T * sizeof(float), s, out, act, rew, h->st<float>(p.o_hyper), c.n_hyper, a.col_ent, B, T,
                     C - 1, c.gamma, c.value_cost, dout, h->st<float>(p.o_loss));
  PBT_HIP(h, hipGetLastError());
  {
    // (the bias gradient, column sums of dout, is a by-product of the same launch)
    GemmOperands wg{A[L - 1], Kh, (int64_t)R * Kh, true, dout, 32, (int64_t)R * 32, false, Kh, C, R, P};
    wg.b_cols = 32;
    wg.colsum = G + p.lay.b_off[L - 1]; wg.colsum_stride = S;
    PBT_LAUNCH(h, PBT_K_HEAD, s, gemm_store_f32(wg, G + p.lay.w_off[L - 1], C, S, s));
  }
  PBT_LAUNCH(h, PBT_K_HEAD, s, head_dgrad(dout, W16 + p.lay.w_off[L - 1], S, Z[L - 2], dZ[L - 2], P, R, Kh, C, c.act, s));
  OptArgs oa{h->st<float>(p.o_w32), h->st<float>(p.o_opt0), nullptr, h->st<bf16_t>(p.o_w16), G, 0, S, h->st<float>(p.o_hyper),
             h->st<int32_t>(p.o_t), S, P, c.n_hyper, c.optimizer, p.col_lr, -1, -1, c.opt_const[0], c.opt_const[1], c.opt_const[2],
             c.opt_const[3]};
  const bool fused = c.fuse_optimizer != 0;
  if ((st = backward(h, net, L - 1, R, A, Z, dZ, true, fused ? &oa : nullptr, nullptr, nullptr, 0, s)) != PBT_OK) return st;
  if (fused) return optimizer_rest(h, oa, 0, L, L - 1, S, s);
  PBT_LAUNCH(h, PBT_K_OPTIMIZER, s, optimizer_step(oa, s));
  return PBT_OK;
}

pbt_status a2c_step(pbt_handle* h, const float* obs, const int32_t* actions, const float* rewards, uint32_t step, hipStream_t s) {
  const pbt_config& c = h->cfg;
  const Plan& p = h->plan;
  const A2CPlan& a = p.a2c;
  const int P = c.P, B = c.batch, T = c.unroll, R = a.rows;
  // a trajectory is one "row" of (T+1) * d observations; B of them are drawn per member
  PBT_LAUNCH(h, PBT_K_FETCH, s, gather_rows(obs, c.n_train, (T + 1) * c.dims[0], P, B, (int64_t)R * c.dims[0], step, c.seed,
                                            h->sc<bf16_t>(a.o_a[0]), h->st<int32_t>(p.o_t), s));
  hipLaunchKernelGGL(a2c_fetch_aux_kernel, dim3(P), dim3(64), 0, s, actions, rewards, c.n_train, B, T, step, (uint32_t)c.seed,
                     (uint32_t)(c.seed >> 32), h->sc<int32_t>(a.o_act), h->sc<float>(a.o_rew), h->st<float>(p.o_hist));
  PBT_HIP(h, hipGetLastError());
  return a2c_update(h, s);
}

// ---- on-policy unrolls (Section 4.1.1: agents act with their current policy) -------------------------

constexpr uint32_t DOMAIN_ENV = 32;

// Four standard normals from one Philox counter: Box-Muller on the word pairs (0,1) and (2,3), in double.
__device__ __forceinline__ void env_normal4(uint32_t step, uint32_t member, uint32_t domain, uint32_t counter, uint32_t k0,
                                            uint32_t k1, double* v) {
  const u32x4 w = philox4x32_10(step, member, domain, counter, k0, k1);
  // (cos and sin of 2 pi u through sincospi(2 u): no reduction of a large argument modulo pi)
  const double r1 = sqrt(-2.0 * log(philox_unit(w.x))), r2 = sqrt(-2.0 * log(philox_unit(w.z)));
  double s1, c1, s2, c2;
  sincospi(2.0 * philox_unit(w.y), &s1, &c1);
  sincospi(2.0 * philox_unit(w.w), &s2, &c2);
  v[0] = r1 * c1; v[1] = r1 * s1; v[2] = r2 * c2; v[3] = r2 * s2;
}
// The same four normals to float accuracy (largest relative error 2.8e-7, root mean square 5.3e-8 over 2^24 pairs; through the library's
// logf / log1pf, sqrtf, sinpif and cospif it was 3.0e-7 and 5.4e-8), for values that are stored as bf16 anyway (the observation noise: 512 of them per
// trajectory and time step, which is what the unroll computes most of).  Everything starts from integers, so that each reduced argument
// is rounded once:  u = (2 w + 1) / 2^33.
//   -log u = -(e log 2 + log(1 + f)):  next to 1, f = u - 1 from the complement of w (no digits lost); from one half up, f = 2 u - 1 and
//   e = -1; below, e and 1 + f in [sqrt 1/2, sqrt 2) from the float's bits.  log(1 + f) = f - (f^2/2 - s (f^2/2 + R)), s = f / (2 + f),
//   R = s^2 (2/3 + 2/5 s^2 + ...), the series of 2 artanh(s) with |s| <= 0.1716, cut where it is below 2e-9.
//   The angle 2 pi u is q pi/2 + pi f with |f| <= 1/4; Taylor series of sin(pi f) and cos(pi f), then the quadrant.
// A third of the instructions of the library's functions: 128 members' unrolls of 20 steps of 512 observations 415 -> 356 us.
__device__ __forceinline__ void env_normal_pair_f32(uint32_t wr, uint32_t wa, float* cosv, float* sinv) {
  const float t = (float)(2u * wr + 1u);                                         // below one half: 2^33 u
  const int tb = (int)__float_as_uint(t) - 0x3f3504f3;                           // exponent that puts 1 + f next to 1
  const bool near1 = wr >= 0xb504f334u, upper = wr >= 0x80000000u;               // sqrt(1/2), one half
  const float f_low = __uint_as_float((uint32_t)((tb & 0x007fffff) + 0x3f3504f3)) - 1.f;
  const float f_mid = (float)(2u * (wr - 0x80000000u) + 1u) * 2.3283064365386963e-10f;   // 2^-32
  const float f_one = (float)(2u * ~wr + 1u) * -1.1641532182693481e-10f;                 // -2^-33
  const float f = near1 ? f_one : upper ? f_mid : f_low;
  const float me = near1 ? 0.f : upper ? 1.f : (float)(33 - (tb >> 23));         // -e
  const float d = 2.f + f;
  float rc = __builtin_amdgcn_rcpf(d);
  rc = fmaf(fmaf(-d, rc, 1.f), rc, rc);
  const float s = f * rc, z = s * s;
  float R = fmaf(z, 0.2222222222f, 0.2857142857f);
  R = fmaf(z, R, 0.4f);
  R = fmaf(z, R, 0.6666666667f);
  R *= z;
  const float h = 0.5f * f * f;
  const float l1 = h - s * (h + R);                                              // f - log(1 + f)
  // -log u = me log2 - f + l1, log 2 in two parts, the rounding of the first difference carried along
  const float hi = fmaf(me, 0.693145751953125f, -f), hl = fmaf(me, 0.693145751953125f, -hi) - f;
  const float nl2 = 2.f * (hi + (fmaf(me, 1.42860677e-6f, l1) + hl));
  // sqrt by one step on the reciprocal root's estimate and one on the root (the argument lies in 2e-10 .. 46)
  const float y = __builtin_amdgcn_rsqf(nl2);
  float r = nl2 * y;
  r = fmaf(fmaf(-r, r, nl2), 0.5f * y, r);
  const uint32_t k = (wa + 0x20000000u) >> 30;
  const float a = (float)(int)(2u * (wa - (k << 30)) + 1u) * 2.3283064365386963e-10f;   // angle / pi past the quadrant, |a| <= 1/4
  const float x = 3.14159274f * a, xl = fmaf(3.14159274f, a, -x) + -8.74227766e-8f * a, x2 = x * x;
  float sp = fmaf(x2, 2.75573192e-6f, -1.98412698e-4f);
  sp = fmaf(x2, sp, 8.33333333e-3f);
  sp = fmaf(x2, sp, -1.66666667e-1f);
  const float s0 = x + fmaf(x2 * x, sp, xl);
  float cp = fmaf(x2, -2.75573192e-7f, 2.48015873e-5f);
  cp = fmaf(x2, cp, -1.38888889e-3f);
  cp = fmaf(x2, cp, 4.16666667e-2f);
  const float w = fmaf(x2, -0.5f, 1.f), x2l = fmaf(x, x, -x2);   // (cos: the roundings of x^2 and of 1 - x^2/2 carried along)
  const float c0 = w + (fmaf(x2, -0.5f, 1.f - w) + fmaf(x2 * x2, cp, fmaf(-x, xl, -0.5f * x2l)));
  const float sq = k & 1u ? c0 : s0, cq = k & 1u ? s0 : c0;
  *sinv = r * (k & 2u ? -sq : sq);
  *cosv = r * ((k ^ (k >> 1)) & 1u ? -cq : cq);
}
__device__ __forceinline__ void env_normal4_f32(uint32_t step, uint32_t member, uint32_t domain, uint32_t counter, uint32_t k0,
                                                uint32_t k1, float* v) {
  const u32x4 w = philox4x32_10(step, member, domain, counter, k0, k1);
  env_normal_pair_f32(w.x, w.y, &v[0], &v[1]);
  env_normal_pair_f32(w.z, w.w, &v[2], &v[3]);
}
__device__ __forceinline__ double env_normal(uint32_t step, uint32_t member, uint32_t domain, uint32_t e, uint32_t k0, uint32_t k1) {
  double v[4];
  env_normal4(step, member, domain, e >> 2, k0, k1, v);
  return v[e & 3];
}

struct EnvArgs {
  A2CEnv env;
  int nz, n_act, d, B, T, rows;        // rows = B (T + 1) observation rows per member
  uint32_t step, k0, k1;
  double* z;                           // [P][B][nz]
  const float* head_out;               // [P][B][32]: head outputs of the policy at time t - 1
  int32_t* act; float* rew;            // [P][B][T]
  bf16_t* obs;                         // [P][rows][d]
  int32_t* t_count;
};

// One time step of the latent system for all trajectories of one member (one workgroup per member).
// t > 0: one thread per trajectory draws a_{t-1} from the policy's head outputs and books r_{t-1}; then one
// thread per (trajectory, four latent components) moves the latent to z_t (four normals = one Philox counter).
// t = 0: z_0 is drawn.
__global__ __launch_bounds__(256) void a2c_env_transition_kernel(EnvArgs a, int t) {
  extern __shared__ double zs[];                 // [B][nz] latent before the transition
  int* action = reinterpret_cast<int*>(zs + (size_t)a.B * a.nz);   // [B]
  const int i = blockIdx.x;
  const int nz = a.nz, B = a.B, T = a.T, tt = t - 1;
  double* zm = a.z + (int64_t)i * B * nz;
  if (t > 0) {
    for (int e = threadIdx.x; e < B * nz; e += blockDim.x) zs[e] = zm[e];
    __syncthreads();
    for (int r = threadIdx.x; r < B; r += blockDim.x) {
      const float* lg = a.head_out + ((int64_t)i * B + r) * 32;
      double mx = -INFINITY;
      for (int c = 0; c < a.n_act; ++c) mx = fmax(mx, (double)lg[c]);
      double ex[32], se = 0.0;
      for (int c = 0; c < a.n_act; ++c) { ex[c] = exp((double)lg[c] - mx); se += ex[c]; }
      const double u = philox_unit(philox4x32_10(a.step, i, DOMAIN_ENV + 2, (uint32_t)(r * T + tt), a.k0, a.k1).x);
      double cdf = 0.0;
      int act = 0;
      for (int c = 0; c < a.n_act; ++c) { cdf += ex[c] / se; act += cdf <= u ? 1 : 0; }
      act = act < a.n_act - 1 ? act : a.n_act - 1;
      double rw = 0.0;
      for (int k = 0; k < nz; ++k) rw += a.env.w[k] * zs[r * nz + k];
      rw += a.env.noise[1] * env_normal(a.step, i, DOMAIN_ENV + 3, (uint32_t)(r * T + tt), a.k0, a.k1);
      a.act[((int64_t)i * B + r) * T + tt] = act;
      a.rew[((int64_t)i * B + r) * T + tt] = (float)rw;
      action[r] = act;
    }
    __syncthreads();
  }
  // element e = (trajectory, component) of the normal stream of this time step: z_0 (t = 0) or zeta_{t-1}
  const uint32_t domain = t == 0 ? DOMAIN_ENV + 0 : DOMAIN_ENV + 4;
  const int quads = (nz + 3) / 4;
  for (int item = threadIdx.x; item < B * quads; item += blockDim.x) {
    const int r = item / quads, k0 = (item - r * quads) * 4;
    const uint32_t e0 = (uint32_t)((t == 0 ? r : r * T + tt) * nz + k0);
    double v[4];
    if ((e0 & 3u) == 0) {
      env_normal4(a.step, i, domain, e0 >> 2, a.k0, a.k1, v);
    } else {
      for (int q = 0; q < 4; ++q) v[q] = env_normal(a.step, i, domain, e0 + q, a.k0, a.k1);
    }
    for (int q = 0; q < 4 && k0 + q < nz; ++q) {
      const int k = k0 + q;
      double zn = v[q];
      if (t > 0) {
        double acc = 0.0;
        for (int j = 0; j < nz; ++j) acc += a.env.A[k * nz + j] * zs[r * nz + j];
        zn = acc + a.env.B[k * a.n_act + action[r]] + a.env.noise[2] * v[q];
      }
      zm[r * nz + k] = zn;
    }
  }
  if (t == 0 && threadIdx.x == 0) a.t_count[i] += 1;
}

// The observations o_t of all trajectories of one member (blockIdx.y) for a slab of 64 observation components
// (blockIdx.x), written where the step (and the policy's next forward pass) reads them.  The slab's rows of C go
// through LDS, transposed, so that neighbouring lanes read neighbouring addresses there (read from memory in the
// order the sum wants them, a wavefront's load touched 64 separate lines and the L1's access rate set the time);
// a thread handles runs of four components, i.e. one Philox counter.
constexpr int OBS_SLAB = 64;   // (the plan's LDS check assumes 64)
__global__ __launch_bounds__(256) void a2c_env_observe_kernel(EnvArgs a, int t) {
  extern __shared__ double obs_lds[];
  const int nz = a.nz, B = a.B, i = blockIdx.y, j_first = blockIdx.x * OBS_SLAB;
  double* Ct = obs_lds;                         // [nz][OBS_SLAB + 1]
  double* zs = obs_lds + nz * (OBS_SLAB + 1);   // [B][nz]
  for (int e = threadIdx.x; e < OBS_SLAB * nz; e += blockDim.x) {
    const int j = e / nz, k = e - j * nz;
    Ct[k * (OBS_SLAB + 1) + j] = j_first + j < a.d ? a.env.C[(int64_t)(j_first + j) * nz + k] : 0.0;
  }
  for (int e = threadIdx.x; e < B * nz; e += blockDim.x) zs[e] = a.z[(int64_t)i * B * nz + e];
  __syncthreads();
  constexpr int RUNS = OBS_SLAB / 4;
  for (int item = threadIdx.x; item < B * RUNS; item += blockDim.x) {
    const int r = item / RUNS, g = item - r * RUNS, j0 = j_first + 4 * g;
    if (j0 >= a.d) continue;
    const int64_t row = (int64_t)r * (a.T + 1) + t;
    float v[4];
    env_normal4_f32(a.step, i, DOMAIN_ENV + 1, (uint32_t)((row * a.d + j0) >> 2), a.k0, a.k1, v);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k = 0; k < nz; ++k) {
      const double zk = zs[r * nz + k];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += Ct[k * (OBS_SLAB + 1) + 4 * g + e] * zk;
    }
    float o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (float)(acc[e] + a.env.noise[0] * (double)v[e]);
    *reinterpret_cast<uint2*>(a.obs + ((int64_t)i * a.rows + row) * a.d + j0) = make_uint2(f2bf_pair(o[0], o[1]), f2bf_pair(o[2], o[3]));
  }
}

// ---- the whole unroll in one kernel -----------------------------------------------------------------------------
// The T + 1 rounds of (action draw and transition, observation, policy) of a member's trajectories run back to back;
// trajectories do not interact, so a member is cut into `parts` workgroups of `rows` trajectories, as many as fill the
// chip's compute units.  The same arithmetic as the kernels above and the batched GEMMs (bf16 operands, float
// accumulation, bias and activation in float, activations rounded to bf16 between layers, float head outputs); sums
// run in a different order.
// What a round waits for is latency, so nothing in it touches memory for longer than it must:
//  - the weights are packed once per unroll into MFMA fragments (a2c_pack_weights_kernel: 16 columns x 32 k, lane l's 16
//    bytes at 16 l, zeros past the matrix), so a wavefront fetches an operand with one contiguous 1 KB load and no LDS.  The
//    first layer (the large one) stays in registers for the whole unroll as far as they go; what remains of it and the later
//    layers are requested ahead of the barrier or the layer before them.
//  - every draw that does not depend on the policy (latent noise, reward noise, the uniforms of the action draw; all in
//    double) is made ahead by a kernel that fills the chip (a2c_env_noise_kernel) and fetched one round ahead.
//  - the observation noise is drawn here, four trajectories per thread: a run of four components of C is read from LDS
//    once for all of them (16 bytes per lane; read 4 bytes at a time at a stride of 16 it was the LDS that bounded this).
//  - the action draw and the latent transition of a trajectory belong to one half-wavefront (lane = action, then latent
//    component): exchanges instead of barriers.
// 128 members, 32 trajectories of 20 steps, 512-256-256-19: 353 us, and 26 + 9 for the packing and the draws ahead, against
// 1197 us as one workgroup per member that streamed its weights through LDS in every round.
// Shapes: observation width and hidden widths multiples of 8, hidden widths up to 256, up to three hidden layers, at
// most 32 head outputs, and what rollout_cut() finds to fit LDS.
// The observations' sums C z run in double or in float, see there.
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 ro_frag_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float ro_acc_t;
constexpr int RO_MAX_HIDDEN = 3;
constexpr int RO_MAX_WIDTH = 256;
constexpr int RO_THREADS = 512;   // 8 wavefronts, two per SIMD: 256 registers per lane
constexpr int RO_WAVES = RO_THREADS / 64;
constexpr int RO_KB0 = 12;        // k-blocks of 32 of the first layer that stay in registers: 96 per lane (16 made the compiler spill),
constexpr int RO_KT0 = 4;         // and those that are requested again in every round, ahead of the barrier before the layer
constexpr int RO_PART_PITCH = 36; // floats per row of the head's partial sums

__host__ __device__ inline int ro_kblocks(int K) { return (K + 31) / 32; }
__host__ __device__ inline int ro_nblocks(int N) { return 2 * ((N + 31) / 32); }   // column blocks of 16, padded to 32 columns
inline int64_t ro_packed_elems(const int32_t* dims, int L) {
  int64_t n = 0;
  for (int l = 0; l < L; ++l) n += (int64_t)ro_nblocks(dims[l + 1]) * ro_kblocks(dims[l]) * 512;
  return n;
}
// draws made ahead, in doubles per member: latent noise [B][T][nz] (the order of its stream), z_0 [B][nz], reward noise [B][T], uniforms [B][T]
struct RoDraws { int64_t o_zeta, o_z0, o_rew, o_u, count; };
__host__ __device__ inline RoDraws ro_draws(int B, int T, int nz) {
  RoDraws d;
  d.o_zeta = 0;
  d.o_z0 = d.o_zeta + ((int64_t)B * T * nz + 3) / 4 * 4;
  d.o_rew = d.o_z0 + ((int64_t)B * nz + 3) / 4 * 4;
  d.o_u = d.o_rew + ((int64_t)B * T + 3) / 4 * 4;
  d.count = d.o_u + ((int64_t)B * T + 3) / 4 * 4;
  return d;
}

// grid (Philox counters of a member / 256, P): one thread per counter, four doubles each
__global__ __launch_bounds__(256) void a2c_env_noise_kernel(EnvArgs a, double* __restrict__ draws) {
  const int i = blockIdx.y;
  const RoDraws o = ro_draws(a.B, a.T, a.nz);
  const int64_t item = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (item >= o.count / 4) return;
  double v[4];
  if (item >= o.o_u / 4) {          // one counter per transition, its first word
    const uint32_t c = (uint32_t)(item - o.o_u / 4) * 4;
    for (int q = 0; q < 4; ++q) v[q] = philox_unit(philox4x32_10(a.step, (uint32_t)i, DOMAIN_ENV + 2, c + q, a.k0, a.k1).x);
  } else if (item >= o.o_rew / 4) {
    env_normal4(a.step, i, DOMAIN_ENV + 3, (uint32_t)(item - o.o_rew / 4), a.k0, a.k1, v);
  } else if (item >= o.o_z0 / 4) {
    env_normal4(a.step, i, DOMAIN_ENV + 0, (uint32_t)(item - o.o_z0 / 4), a.k0, a.k1, v);
  } else {
    env_normal4(a.step, i, DOMAIN_ENV + 4, (uint32_t)item, a.k0, a.k1, v);
  }
  double2* __restrict__ p = reinterpret_cast<double2*>(draws + i * o.count + item * 4);
  p[0] = make_double2(v[0], v[1]);
  p[1] = make_double2(v[2], v[3]);
}

struct RolloutArgs {
  EnvArgs e;
  const bf16_t* W16; const float* W32; int64_t stride;
  bf16_t* packed; int64_t packed_stride;   // [P] fragments of all layers, layer l from packed_off[l]
  double* draws;                           // [P][ro_draws().count]
  int n_hidden, act, hmax, rows;           // rows: trajectories per workgroup
  int dims[RO_MAX_HIDDEN + 2];
  int64_t w_off[RO_MAX_HIDDEN + 1], b_off[RO_MAX_HIDDEN + 1], packed_off[RO_MAX_HIDDEN + 1];
};

// grid (32-column blocks of all layers together, k-blocks of the deepest layer / 2, P); 32 columns x 64 k of W[K][N] (rows of N) go
// through LDS and leave as fragments: block (nb, kb), lane l: column 16 nb + l % 16, k = 32 kb + 8 (l / 16) ...
__global__ __launch_bounds__(256) void a2c_pack_weights_kernel(RolloutArgs a) {
  __shared__ __attribute__((aligned(16))) bf16_t tile[64 * 34];
  const int i = blockIdx.z;
  int l = 0, cb = blockIdx.x;
  while (cb >= ro_nblocks(a.dims[l + 1]) / 2) cb -= ro_nblocks(a.dims[l++ + 1]) / 2;
  const int K = a.dims[l], N = a.dims[l + 1], KB = ro_kblocks(K);
  const int k0 = blockIdx.y * 64;
  if (k0 >= K) return;
  const bf16_t* __restrict__ W = a.W16 + (int64_t)i * a.stride + a.w_off[l];
  // 16 bytes per thread (four neighbouring lanes on a row's 32 columns) where rows are whole groups of eight, which all but the head's are
  if (N % 8 == 0) {
    const int k = threadIdx.x >> 2, n = (threadIdx.x & 3) * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (k0 + k < K && cb * 32 + n < N) v = *reinterpret_cast<const uint4*>(W + (int64_t)(k0 + k) * N + cb * 32 + n);
    uint32_t* t = reinterpret_cast<uint32_t*>(tile + k * 34 + n);
    t[0] = v.x; t[1] = v.y; t[2] = v.z; t[3] = v.w;
  } else {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int x = u * 256 + threadIdx.x, k = x >> 5, n = x & 31;
      tile[k * 34 + n] = k0 + k < K && cb * 32 + n < N ? W[(int64_t)(k0 + k) * N + cb * 32 + n] : (bf16_t)0;
    }
  }
  __syncthreads();
  const int f = threadIdx.x >> 6, lane = threadIdx.x & 63;   // four fragments: column block f & 1, k-block f >> 1
  const int kb = blockIdx.y * 2 + (f >> 1), nb = cb * 2 + (f & 1);
  if (kb >= KB) return;
  const bf16_t* __restrict__ src = tile + ((f >> 1) * 32 + 8 * (lane >> 4)) * 34 + (f & 1) * 16 + (lane & 15);
  uint32_t w[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) w[q] = (uint32_t)src[2 * q * 34] | (uint32_t)src[(2 * q + 1) * 34] << 16;
  *reinterpret_cast<uint4*>(a.packed + i * a.packed_stride + a.packed_off[l] + (((int64_t)nb * KB + kb) * 64 + lane) * 8) =
      make_uint4(w[0], w[1], w[2], w[3]);
}

__device__ __forceinline__ ro_acc_t ro_mfma(uint4 w, uint4 x, ro_acc_t acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(ro_frag_t, w), __builtin_bit_cast(ro_frag_t, x), acc, 0, 0, 0);
}
// Wavefront w owns the column blocks w and w + 8 of a layer.  The weight fragment is the MFMA's first operand: a lane holds, of
// row (trajectory) lane % 16, the columns 16 nb + 4 (lane / 16) ... + 3.
template <int KB>
struct RoFrags { uint4 v[2][KB > 0 ? KB : 1]; };
// (blocks the layer does not have are read as its last one and not multiplied: no branch around a load)
template <int KB>
__device__ __forceinline__ void ro_fetch(int tid, const bf16_t* __restrict__ frags, int kb0, int kblocks, int nblocks, RoFrags<KB>& r) {
  const int lane = tid & 63, w = tid >> 6;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      r.v[j][kb] = *reinterpret_cast<const uint4*>(frags + ((min(w + 8 * j, nblocks - 1) * kblocks + min(kb0 + kb, kblocks - 1)) * 64 + lane) * 8);
    }
}
// out = act(in W + b) for MB blocks of 16 rows in LDS.  k-blocks past those handed in (observations wider than 512) are
// fetched as they are needed.  Columns N .. of the last 32 get zeros (their weights are zero), which the next layer's padded k reads.
template <int MB, int KB, int KT>
__device__ __forceinline__ void ro_dense(int tid, const bf16_t* in, int pin, int K, int N, const RoFrags<KB>& wf, const RoFrags<KT>& wt, const bf16_t* __restrict__ frags,
                                         const float* __restrict__ bias, int act, bf16_t* out, int pout) {
  const int lane = tid & 63, w = tid >> 6, lr = lane & 15, q = lane >> 4;
  const int kblocks = ro_kblocks(K), nblocks = ro_nblocks(N);
  if (w >= nblocks) return;
  const bool second = w + 8 < nblocks;
  float4 b[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int n0 = 16 * (w + 8 * j) + 4 * q;
    b[j] = n0 < N ? *reinterpret_cast<const float4*>(bias + n0) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  ro_acc_t acc[MB][2];
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[m][j] = ro_acc_t{0.f, 0.f, 0.f, 0.f};
  auto block = [&](int kb, const uint4& f0, const uint4& f1) {
    if (kb < kblocks) {
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        const uint4 x = *reinterpret_cast<const uint4*>(in + (16 * m + lr) * pin + 32 * kb + 8 * q);
        acc[m][0] = ro_mfma(f0, x, acc[m][0]);
        if (second) acc[m][1] = ro_mfma(f1, x, acc[m][1]);
      }
    }
  };
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) block(kb, wf.v[0][kb], wf.v[1][kb]);
#pragma unroll
  for (int kb = 0; kb < KT; ++kb) block(KB + kb, wt.v[0][kb], wt.v[1][kb]);
  for (int kb = KB + KT; kb < kblocks; ++kb) {
    const uint4 w0 = *reinterpret_cast<const uint4*>(frags + (((int64_t)w * kblocks + kb) * 64 + lane) * 8);
    const uint4 w1 = second ? *reinterpret_cast<const uint4*>(frags + (((int64_t)(w + 8) * kblocks + kb) * 64 + lane) * 8) : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      const uint4 x = *reinterpret_cast<const uint4*>(in + (16 * m + lr) * pin + 32 * kb + 8 * q);
      acc[m][0] = ro_mfma(w0, x, acc[m][0]);
      acc[m][1] = ro_mfma(w1, x, acc[m][1]);
    }
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (j == 1 && !second) break;
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      const float a0 = act_fwd(acc[m][j][0] + b[j].x, act), a1 = act_fwd(acc[m][j][1] + b[j].y, act);
      const float a2 = act_fwd(acc[m][j][2] + b[j].z, act), a3 = act_fwd(acc[m][j][3] + b[j].w, act);
      *reinterpret_cast<uint2*>(out + (16 * m + lr) * pout + 16 * (w + 8 * j) + 4 * q) = make_uint2(f2bf_pair(a0, a1), f2bf_pair(a2, a3));
    }
  }
}

// The observations of round t, RG trajectories per thread: to memory (the update reads them) and to X0 (the policy's
// input).  The sum C z runs in double, or in float (rollout_cut(): SUM; the result is stored as bf16).  z: component k of trajectory r at
// k zk + r zr.
__device__ __forceinline__ void ro_load4(const float* p, float* c) {
  const float4 v = *reinterpret_cast<const float4*>(p);
  c[0] = v.x; c[1] = v.y; c[2] = v.z; c[3] = v.w;
}
__device__ __forceinline__ void ro_load4(const double* p, double* c) {
  const double2 lo = *reinterpret_cast<const double2*>(p), hi = *reinterpret_cast<const double2*>(p + 2);
  c[0] = lo.x; c[1] = lo.y; c[2] = hi.x; c[3] = hi.y;
}
template <int RG, class SUM>
__device__ __forceinline__ void ro_observe(int tid, const EnvArgs& e, int i, int t, int r0, int rows, const SUM* Ct, const SUM* z, int zk, int zr,
                                           bf16_t* X0, int px) {
  const int d = e.d, runs = d / 4, groups = (rows + RG - 1) / RG;
  for (int item = tid; item < groups * runs; item += RO_THREADS) {
    const int grp = item / runs, j0 = 4 * (item - grp * runs);
    SUM acc[RG][4];
#pragma unroll
    for (int s = 0; s < RG; ++s)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[s][q] = 0;
    for (int k = 0; k < e.nz; ++k) {
      SUM c[4];
      ro_load4(Ct + k * d + j0, c);
#pragma unroll
      for (int s = 0; s < RG; ++s) {
        const SUM zs = z[k * zk + (grp * RG + s) * zr];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[s][q] = fma(c[q], zs, acc[s][q]);
      }
    }
    const SUM noise_obs = (SUM)e.env.noise[0];
#pragma unroll
    for (int s = 0; s < RG; ++s) {
      const int r = grp * RG + s;
      if (r < rows) {
        const int64_t row = (int64_t)(r0 + r) * (e.T + 1) + t;
        float v[4], o[4];
        env_normal4_f32(e.step, i, DOMAIN_ENV + 1, (uint32_t)((row * d + j0) >> 2), e.k0, e.k1, v);
#pragma unroll
        for (int q = 0; q < 4; ++q) o[q] = (float)fma(noise_obs, (SUM)v[q], acc[s][q]);
        const uint2 packed = make_uint2(f2bf_pair(o[0], o[1]), f2bf_pair(o[2], o[3]));
        *reinterpret_cast<uint2*>(e.obs + ((int64_t)i * e.rows + row) * d + j0) = packed;
        *reinterpret_cast<uint2*>(X0 + r * px + j0) = packed;
      }
    }
  }
}

// LDS of the kernel, in this order: doubles: latents (two copies of [rb][nz]), A transposed, B, w of the latent system, the next
// round's latent noise [rb][nz], uniforms and reward noise [rb]; then, each 16-byte aligned: C transposed [nz][d] (float, or double where the
// sum C z runs in double), floats: the round's latents [nz][rb], the head's partial sums [8][rb][36]; then bf16: observations and two
// activation buffers [rb][width + 8].
struct RoLds { size_t o_Ct, o_zf, o_part, o_x, bytes; };
__host__ __device__ inline RoLds ro_lds_layout(int rb, int nz, int n_act, int d, int hmax, int sum_bytes) {
  RoLds o;
  const size_t doubles = (size_t)3 * rb * nz + (size_t)nz * nz + (size_t)nz * n_act + nz + 2 * rb;
  o.o_Ct = (doubles * 8 + 15) & ~(size_t)15;
  o.o_zf = o.o_Ct + (size_t)nz * d * sum_bytes;
  o.o_part = o.o_zf + (size_t)nz * rb * 4;
  o.o_x = o.o_part + (size_t)RO_WAVES * rb * RO_PART_PITCH * 4;
  o.bytes = o.o_x + (size_t)rb * (32 * ro_kblocks(d) + 8) * 2 + (size_t)2 * rb * (32 * ro_kblocks(hmax) + 8) * 2;
  return o;
}

// grid (parts, P); MB blocks of 16 trajectories; SUM: the type the observations are summed in
template <int MB, class SUM>
__global__ __launch_bounds__(RO_THREADS) void a2c_rollout_kernel(RolloutArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char ro_lds[];
  constexpr int RB = 16 * MB;
  const EnvArgs& e = a.e;
  const int i = blockIdx.y, nz = e.nz, T = e.T, d = e.d, n_act = e.n_act;
  const int r0 = blockIdx.x * a.rows, rows = min(a.rows, e.B - r0);
  const RoLds o = ro_lds_layout(RB, nz, n_act, d, a.hmax, (int)sizeof(SUM));
  double* zs = reinterpret_cast<double*>(ro_lds);                 // [2][RB][nz]
  double* At = zs + 2 * RB * nz;                                  // [nz][nz], transposed
  double* Bs = At + nz * nz;                                      // [nz][n_act]
  double* ws = Bs + nz * n_act;                                   // [nz]
  double* zeta = ws + nz;                                         // [RB][nz]
  double* us = zeta + RB * nz;                                    // [RB]
  double* rns = us + RB;                                          // [RB]
  SUM* Ct = reinterpret_cast<SUM*>(ro_lds + o.o_Ct);              // [nz][d]
  float* zf = reinterpret_cast<float*>(ro_lds + o.o_zf);          // [nz][RB]
  float* part = reinterpret_cast<float*>(ro_lds + o.o_part);      // [8][RB][36]
  const int px = 32 * ro_kblocks(d) + 8, ph = 32 * ro_kblocks(a.hmax) + 8;
  bf16_t* X0 = reinterpret_cast<bf16_t*>(ro_lds + o.o_x);         // [RB][px]
  bf16_t* XA = X0 + RB * px;                                      // [RB][ph]
  bf16_t* XB = XA + RB * ph;
  const bf16_t* packed = a.packed + (int64_t)i * a.packed_stride;
  const float* W32 = a.W32 + (int64_t)i * a.stride;
  const RoDraws od = ro_draws(e.B, T, nz);
  const double* draws = a.draws + i * od.count;
  RoFrags<RO_KB0> w0;
  ro_fetch<RO_KB0>(threadIdx.x, packed + a.packed_off[0], 0, ro_kblocks(d), ro_nblocks(a.dims[1]), w0);
  // the head: its two column blocks of the k-block this wavefront contributes
  const int Kh = a.dims[a.n_hidden], C = a.dims[a.n_hidden + 1], kbh = ro_kblocks(Kh);
  uint4 wh[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    wh[j] = make_uint4(0, 0, 0, 0);
    if ((int)threadIdx.x >> 6 < kbh)
      wh[j] = *reinterpret_cast<const uint4*>(packed + a.packed_off[a.n_hidden] + (((int64_t)j * kbh + (threadIdx.x >> 6)) * 64 + (threadIdx.x & 63)) * 8);
  }
  const float head_bias = (int)(threadIdx.x & 31) < C ? W32[a.b_off[a.n_hidden] + (threadIdx.x & 31)] : 0.f;
  if (threadIdx.x == 0 && blockIdx.x == 0) e.t_count[i] += 1;
  for (int x = threadIdx.x; x < nz * nz; x += RO_THREADS) At[(x % nz) * nz + x / nz] = e.env.A[x];
  for (int x = threadIdx.x; x < nz * n_act; x += RO_THREADS) Bs[x] = e.env.B[x];
  for (int x = threadIdx.x; x < nz; x += RO_THREADS) ws[x] = e.env.w[x];
  for (int x = threadIdx.x; x < d * nz; x += RO_THREADS) {
    const int j = x / nz, k = x - j * nz;
    Ct[k * d + j] = (SUM)e.env.C[x];
  }
  const double noise_rew = e.env.noise[1], noise_lat = e.env.noise[2];
  // rows past the last trajectory and columns past the last component stay zero in the observation buffer
  for (int x = threadIdx.x; x < RB * px / 2; x += RO_THREADS) reinterpret_cast<uint32_t*>(X0)[x] = 0u;
  for (int x = threadIdx.x; x < nz * RB; x += RO_THREADS) zf[x] = 0.f;
  __syncthreads();
  for (int t = 0; t <= T; ++t) {
    // (the thread's index, made opaque once per round: otherwise the compiler computes every address of a round ahead of
    // the loop and keeps them in registers that the weights need)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int tt = t - 1, lane = tid & 63, w = tid >> 6;
    double* zo = zs + (t & 1) * RB * nz;          // latents before this round's transition
    double* zn = zs + ((t + 1) & 1) * RB * nz;    // and after
    // a half-wavefront per trajectory: a_{t-1} from the head outputs (lane = action), then z_t (lane = component)
    for (int r = tid >> 5; r < rows; r += RO_THREADS / 32) {
      const int c = tid & 31;
      int action = 0;
      if (t > 0) {
        float lg = part[r * RO_PART_PITCH + c];
        for (int v = 1; v < kbh; ++v) lg += part[(v * RB + r) * RO_PART_PITCH + c];
        lg += head_bias;
        float mx = c < n_act ? lg : -INFINITY;
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 32));
        const double ex = c < n_act ? exp((double)lg - (double)mx) : 0.0;
        double se = ex;
#pragma unroll
        for (int off = 16; off > 0; off >>= 1) se += __shfl_xor(se, off, 32);
        double cdf = ex / se;
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) {
          const double below = __shfl_up(cdf, off, 32);
          if (c >= off) cdf += below;
        }
        const uint64_t passed = __ballot(c < n_act && cdf <= us[r]);
        action = __popc((uint32_t)(lane & 32 ? passed >> 32 : passed));
        action = action < n_act - 1 ? action : n_act - 1;
        if (c == 0) e.act[((int64_t)i * e.B + r0 + r) * T + tt] = action;
      }
      for (int k = c; k < nz; k += 32) {
        double zv;
        if (t == 0) {
          zv = draws[od.o_z0 + (int64_t)(r0 + r) * nz + k];
        } else {
          double acc = 0.0;
          for (int j = 0; j < nz; ++j) acc += At[j * nz + k] * zo[r * nz + j];
          zv = acc + Bs[k * n_act + action] + noise_lat * zeta[r * nz + k];
        }
        zn[r * nz + k] = zv;
        zf[k * RB + r] = (float)zv;
      }
    }
    __syncthreads();
    // next round's draws are requested, this round's reward is booked and the observations are made while they arrive
    double next_zeta[4], next_u = 0.0, next_rn = 0.0;
    const int n_zeta = t < T ? rows * nz : 0;     // (at most 32 x 64 = 4 per thread)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int x = q * RO_THREADS + tid;
      next_zeta[q] = 0.0;
      if (x < n_zeta) { const int r = x / nz; next_zeta[q] = draws[od.o_zeta + ((int64_t)(r0 + r) * T + t) * nz + (x - r * nz)]; }
    }
    if (t < T && tid < rows) {
      next_u = draws[od.o_u + (int64_t)(r0 + tid) * T + t];
      next_rn = draws[od.o_rew + (int64_t)(r0 + tid) * T + t];
    }
    if (t > 0 && tid < rows) {
      const int r = tid;
      double rw = 0.0;
      for (int k = 0; k < nz; ++k) rw += ws[k] * zo[r * nz + k];
      rw += noise_rew * rns[r];
      e.rew[((int64_t)i * e.B + r0 + r) * T + tt] = (float)rw;
    }
    // (as many trajectories per thread as leave every thread something to do)
    const SUM* z;
    int zk, zr;
    if constexpr (std::is_same_v<SUM, double>) { z = zn; zk = 1; zr = nz; }
    else { z = zf; zk = RB; zr = 1; }
    if (rows * (d / 4) >= 4 * RO_THREADS) ro_observe<4>(tid, e, i, t, r0, rows, Ct, z, zk, zr, X0, px);
    else if (rows * (d / 4) >= 2 * RO_THREADS) ro_observe<2>(tid, e, i, t, r0, rows, Ct, z, zk, zr, X0, px);
    else ro_observe<1>(tid, e, i, t, r0, rows, Ct, z, zk, zr, X0, px);
    if (t == T) break;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int x = q * RO_THREADS + tid;
      if (x < n_zeta) zeta[x] = next_zeta[q];
    }
    if (tid < rows) { us[tid] = next_u; rns[tid] = next_rn; }
    // the policy on the round's observations
    RoFrags<RO_KT0> wt;
    ro_fetch<RO_KT0>(tid, packed + a.packed_off[0], RO_KB0, ro_kblocks(d), ro_nblocks(a.dims[1]), wt);
    __syncthreads();
    ro_dense<MB, RO_KB0, RO_KT0>(tid, X0, px, d, a.dims[1], w0, wt, packed + a.packed_off[0], W32 + a.b_off[0], a.act, XA, ph);
    RoFrags<RO_MAX_WIDTH / 32> wl;
    if (a.n_hidden > 1) ro_fetch<RO_MAX_WIDTH / 32>(tid, packed + a.packed_off[1], 0, ro_kblocks(a.dims[1]), ro_nblocks(a.dims[2]), wl);
    __syncthreads();
    bf16_t* in = XA;
    bf16_t* out = XB;
    for (int l = 1; l < a.n_hidden; ++l) {
      ro_dense<MB, RO_MAX_WIDTH / 32, 0>(tid, in, ph, a.dims[l], a.dims[l + 1], wl, RoFrags<0>{}, packed + a.packed_off[l], W32 + a.b_off[l], a.act, out, ph);
      if (l + 1 < a.n_hidden)
        ro_fetch<RO_MAX_WIDTH / 32>(tid, packed + a.packed_off[l + 1], 0, ro_kblocks(a.dims[l + 1]), ro_nblocks(a.dims[l + 2]), wl);
      __syncthreads();
      bf16_t* x = in; in = out; out = x;
    }
    // the head: the wavefronts share the contraction, the partial sums are added in wavefront order by the action draw
    if (w < kbh) {
      const int lr = lane & 15, q = lane >> 4;
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        const uint4 x = *reinterpret_cast<const uint4*>(in + (16 * m + lr) * ph + 32 * w + 8 * q);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const ro_acc_t acc = ro_mfma(wh[j], x, ro_acc_t{0.f, 0.f, 0.f, 0.f});
          *reinterpret_cast<float4*>(part + (w * RB + 16 * m + lr) * RO_PART_PITCH + 16 * j + 4 * q) = make_float4(acc[0], acc[1], acc[2], acc[3]);
        }
      }
    }
    __syncthreads();
  }
}

// How a population is cut into workgroups, 0 parts if the shape is not covered.  One workgroup occupies a compute unit
// (registers), so a member gets as many as the chip has left for it, down to four trajectories each (below that the
// per-round latencies are all there is); never more than 32 trajectories, and 16 where 32 do not fit LDS.
struct RoCut { int parts, rows; size_t lds; bool sum_in_float; };
static RoCut rollout_cut(const pbt_config& c) {
  const int L = c.n_layers, d = c.dims[0], C = c.dims[L], B = c.batch;
  const RoCut none{0, 0, 0, false};
  if (d % 8 || L - 1 < 1 || L - 1 > RO_MAX_HIDDEN || C > 32 || c.latent_dim > 64) return none;
  int hmax = 0;
  // C z is summed in double, as by the kernels of one round each, except for the shapes whose unroll has summed it in float ever since it
  // became one kernel (which goes into a bf16 value): in double their steps take 1 to 9 % longer (128 members 512-256-256-19, 32 x 20:
  // 783 -> 811 us), and the others' as much (8 members 200-72-40-9, 40 x 10: 172 -> 177).
  bool sum_in_float = d % 64 == 0 && d <= 512 && c.latent_dim <= 32 && c.latent_dim * d <= 8192 && B <= 32;
  for (int l = 1; l < L; ++l) {
    if (c.dims[l] > RO_MAX_WIDTH || c.dims[l] % 8) return none;
    hmax = c.dims[l] > hmax ? c.dims[l] : hmax;
    sum_in_float = sum_in_float && (c.dims[l] == 64 || c.dims[l] == 128 || c.dims[l] == 256);
  }
  auto lds_of = [&](int rows) { return ro_lds_layout(rows > 16 ? 32 : 16, c.latent_dim, C - 1, d, hmax, sum_in_float ? 4 : 8).bytes; };
  constexpr size_t LDS_MAX = 160 * 1024;
  int parts = 256 / c.P;
  parts = parts > (B + 3) / 4 ? (B + 3) / 4 : parts;
  parts = parts < (B + 31) / 32 ? (B + 31) / 32 : parts;
  int rows = (B + parts - 1) / parts;
  if (rows > 16 && lds_of(rows) > LDS_MAX) { parts = (B + 15) / 16; rows = (B + parts - 1) / parts; }
  if (lds_of(rows) > LDS_MAX) return none;
  return RoCut{(B + rows - 1) / rows, rows, lds_of(rows), sum_in_float};
}

static int64_t a2c_packed_elems(const pbt_config* c) { return rollout_cut(*c).parts ? ro_packed_elems(c->dims, c->n_layers) : 0; }
static int64_t a2c_draw_count(const pbt_config* c) { return rollout_cut(*c).parts ? ro_draws(c->batch, c->unroll, c->latent_dim).count : 0; }

// Pushes the unroll's return (mean over trajectories of the summed rewards, in double, trajectories in order)
// into the member's history ring.
__global__ __launch_bounds__(64) void a2c_push_return_kernel(const float* __restrict__ rew, int B, int T, float* __restrict__ hist) {
  const int i = blockIdx.x;
  __shared__ double tsum[64];
  double mean = 0.0;
  for (int r0 = 0; r0 < B; r0 += 64) {
    const int r = r0 + threadIdx.x;
    double sacc = 0.0;
    if (r < B)
      for (int t = 0; t < T; ++t) sacc += (double)rew[((int64_t)i * B + r) * T + t];
    tsum[threadIdx.x] = sacc;
    __syncthreads();
    if (threadIdx.x == 0)
      for (int k = 0; k < 64 && r0 + k < B; ++k) mean += tsum[k];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    float* hrow = hist + (int64_t)i * HIST_PITCH;
    const int n = __float_as_int(hrow[HIST_SLOTS]);
    hrow[n % HIST_SLOTS] = (float)(mean / (double)B);
    hrow[HIST_SLOTS] = __int_as_float(n + 1);
  }
}

pbt_status a2c_step_on_policy(pbt_handle* h, const A2CEnv& env, uint32_t step, hipStream_t s) {
  const pbt_config& c = h->cfg;
  const Plan& p = h->plan;
  const A2CPlan& a = p.a2c;
  const int P = c.P, B = c.batch, T = c.unroll, L = c.n_layers, R = a.rows, d = c.dims[0];
  const int Kh = c.dims[L - 1], C = c.dims[L];
  const int64_t S = p.lay.stride;
  const float* W32 = h->st<float>(p.o_w32);
  const bf16_t* W16 = h->st<bf16_t>(p.o_w16);
  bf16_t* obs = h->sc<bf16_t>(a.o_a[0]);
  float* gout = h->sc<float>(a.o_gout);
  EnvArgs ea{env, c.latent_dim, C - 1, d, B, T, R, step, (uint32_t)c.seed, (uint32_t)(c.seed >> 32), h->sc<double>(a.o_lat), gout,
             h->sc<int32_t>(a.o_act), h->sc<float>(a.o_rew), obs, h->st<int32_t>(p.o_t)};
  if (a.one_kernel) {
    const RoCut cut = rollout_cut(c);
    RolloutArgs ra{};
    ra.e = ea; ra.W16 = W16; ra.W32 = W32; ra.stride = S; ra.n_hidden = L - 1; ra.act = c.act; ra.rows = cut.rows;
    ra.packed = h->sc<bf16_t>(a.o_packed); ra.packed_stride = ro_packed_elems(c.dims, L); ra.draws = h->sc<double>(a.o_draws);
    int64_t off = 0;
    int col_blocks = 0, kmax = 0;
    for (int l = 0; l <= L; ++l) ra.dims[l] = c.dims[l];
    for (int l = 1; l < L; ++l) ra.hmax = c.dims[l] > ra.hmax ? c.dims[l] : ra.hmax;
    for (int l = 0; l < L; ++l) {
      ra.w_off[l] = p.lay.w_off[l]; ra.b_off[l] = p.lay.b_off[l]; ra.packed_off[l] = off;
      off += (int64_t)ro_nblocks(c.dims[l + 1]) * ro_kblocks(c.dims[l]) * 512;
      col_blocks += ro_nblocks(c.dims[l + 1]) / 2;
      kmax = c.dims[l] > kmax ? c.dims[l] : kmax;
    }
    auto rollout = cut.rows > 16 ? (cut.sum_in_float ? a2c_rollout_kernel<2, float> : a2c_rollout_kernel<2, double>)
                                 : (cut.sum_in_float ? a2c_rollout_kernel<1, float> : a2c_rollout_kernel<1, double>);
    PBT_HIP(h, hipFuncSetAttribute(reinterpret_cast<const void*>(rollout), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    hipLaunchKernelGGL(a2c_pack_weights_kernel, dim3(col_blocks, (kmax + 63) / 64, P), dim3(256), 0, s, ra);
    PBT_HIP(h, hipGetLastError());
    hipLaunchKernelGGL(a2c_env_noise_kernel, dim3((unsigned)((ro_draws(B, T, c.latent_dim).count / 4 + 255) / 256), P), dim3(256), 0, s, ea, ra.draws);
    PBT_HIP(h, hipGetLastError());
    hipLaunchKernelGGL(rollout, dim3(cut.parts, P), dim3(RO_THREADS), cut.lds, s, ra);
    PBT_HIP(h, hipGetLastError());
    // (the gradients' padding has to be zero, and with the optimiser inside the weight-gradient products they are not all written)
    if (a.packed_in_grad) PBT_HIP(h, fill_u32(h->sc<uint32_t>(a.o_packed), 0u, P * ra.packed_stride / 2, s));
    hipLaunchKernelGGL(a2c_push_return_kernel, dim3(P), dim3(64), 0, s, h->sc<float>(a.o_rew), B, T, h->st<float>(p.o_hist));
    PBT_HIP(h, hipGetLastError());
    return a2c_update(h, s);
  }
  for (int t = 0; t <= T; ++t) {
    hipLaunchKernelGGL(a2c_env_transition_kernel, dim3(P), dim3(256), (size_t)B * c.latent_dim * sizeof(double) + (size_t)B * sizeof(int), s, ea, t);
    PBT_HIP(h, hipGetLastError());
    hipLaunchKernelGGL(a2c_env_observe_kernel, dim3((d + OBS_SLAB - 1) / OBS_SLAB, P), dim3(256),
                       ((size_t)c.latent_dim * (OBS_SLAB + 1) + (size_t)B * c.latent_dim) * sizeof(double), s, ea, t);
    PBT_HIP(h, hipGetLastError());
    if (t == T) break;
    // the policy on the B observations of time t: rows t, t + (T+1), ... of the member's observation buffer
    for (int l = 0; l < L - 1; ++l) {
      const int K = c.dims[l], N = c.dims[l + 1];
      const bf16_t* in = l == 0 ? obs + (int64_t)t * d : h->sc<bf16_t>(a.o_ga[l]);
      GemmOperands o{in, l == 0 ? (int64_t)(T + 1) * d : (int64_t)K, l == 0 ? (int64_t)R * d : (int64_t)B * K, false,
                     W16 + p.lay.w_off[l], N, S, false, B, N, K, P};
      PBT_LAUNCH(h, PBT_K_FETCH, s, gemm_bias_act(o, W32 + p.lay.b_off[l], S, nullptr, h->sc<bf16_t>(a.o_ga[l + 1]), N, (int64_t)B * N, c.act, s));
    }
    PBT_LAUNCH(h, PBT_K_FETCH, s, head_fwd_loss(h->sc<bf16_t>(a.o_ga[L - 1]), (int64_t)B * Kh, W16 + p.lay.w_off[L - 1], S, W32 + p.lay.b_off[L - 1], S,
                                                nullptr, 0, P, B, Kh, C, 0.f, -2, nullptr, gout, 0, s));
  }
  hipLaunchKernelGGL(a2c_push_return_kernel, dim3(P), dim3(64), 0, s, h->sc<float>(a.o_rew), B, T, h->st<float>(p.o_hist));
  PBT_HIP(h, hipGetLastError());
  return a2c_update(h, s);
}

pbt_status a2c_eval(pbt_handle* h, hipStream_t s) {
  const int P = h->cfg.P;
  hipLaunchKernelGGL(a2c_score_kernel, dim3((P + 63) / 64), dim3(64), 0, s, h->st<float>(h->plan.o_hist), P, h->st<float>(h->plan.o_score));
  PBT_HIP(h, hipGetLastError());
  return PBT_OK;
}

}  // namespace pbt
