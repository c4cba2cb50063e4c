// A whole layer step of a small layer in one launch (paper Table 2 steps 8-13).
//
// Rows of a layer are independent: a row's residuals, its gradient and its update need that row's weights and all activations.  A
// workgroup takes 16 rows from the residual through the update, so nothing waits for another launch: what bounds such a step is the
// chain of loads, barriers and launches, not bytes or operations.  The gradient dY stays in LDS, G in the accumulators.  The losses
// are added up by the workgroup that is done last.  A sum is two, of the even and of the odd groups of 32 terms, as in the small tiles of
// the products: the same bits as in three launches.
// 256x256 float32 at 64 tokens, steps of a running chain: 17.0 us in three launches (19 of host time) -> 12.8 (12); 1024x256 at 64: 16.7 ->
// 14.2.  A layer's first step has its forward in a launch of its own before it.
#include <type_traits>

#include "faar_internal.h"
#include "faar_step.h"

namespace faar {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kSmallThreads = 512, kSmallWaves = kSmallThreads / 64, kSmallRows = 16;

struct SmallStep {
  StepUpdate p;
  const bf16_t *X, *Xt;
  const float* C;          // null: the layer carries its constant as p.H
  double* mse_partials;    // one per workgroup
  float two_alpha;
  int O, K, T, Tp;
  bool check; ForwardTag expect;
};

__device__ __forceinline__ bf16x8 frag(const bf16_t* p, bool in) {
  const uint4 v = in ? *reinterpret_cast<const uint4*>(p) : make_uint4(0u, 0u, 0u, 0u);
  return __builtin_bit_cast(bf16x8, v);
}

// three sums at once over a wavefront (kSpan 64) or its first lanes
template <int kSpan>
__device__ __forceinline__ void sum3(double& a, double& b, double& c) {
#pragma unroll
  for (int o = kSpan / 2; o > 0; o >>= 1) {
    const double x = __shfl_xor(a, o), y = __shfl_xor(b, o), z = __shfl_xor(c, o);
    a += x;
    b += y;
    c += z;
  }
}

template <typename WT>
__global__ void __launch_bounds__(kSmallThreads) k_small_step(SmallStep a) {
  extern __shared__ __attribute__((aligned(16))) bf16_t dy[];     // [16][Tp + 8]
  const StepUpdate& p = a.p;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = lane & 15, rq = lane >> 4;
  const int o0 = blockIdx.x * kSmallRows, o = o0 + col, pitch = a.Tp + 8;
  const bool row = o < a.O;
  const float xs = p.x_scale ? *p.x_scale : 1.0f, sg = *p.s_global;
  bool valid = true;       // a forward made by this step's own first kernel, or a prepared one under this tag
  if (a.check)
    for (int i = 0; i < kTagWords; ++i) valid &= p.guard_slot[i] == a.expect.w[i];   // all loads at once

  // What the second half reads -- 32 columns of X^T a wavefront and the state of their weights -- is on its way from the start
  const bool emit = p.beta_next > 0.0f;
  float v[8], m[8], u[8], h[8], w[8];
  uint32_t codes = 0, sb = 0;
  bf16x8 xa[8], xb[8];
  auto fetch_state = [&](int k0) {
    const int k = k0 + 8 * rq;                                   // this lane's columns k .. k + 7 of row o
    if (!(row && k < a.K)) return;
    const int64_t e = (int64_t)o * a.K + k;
    sb = p.scales[e >> 4];
    codes = p.icodes[e >> 3];
    load8(p.V + e, v);
    load8(p.M + e, m);
    load8(p.U + e, u);
    if (p.H) load8(p.H + e, h);
    if (emit) W8<WT>::load(static_cast<const WT*>(p.W) + e, w);
  };
  auto fetch_x = [&](int k0, int t0) {                           // 256 tokens of this lane's rows of the two products
    const int ka = k0 + 8 * (col >> 2) + (col & 3);
    const bf16_t* x0 = a.Xt + (int64_t)(ka < a.K ? ka : a.K - 1) * a.Tp + t0 + 8 * rq;
    const bf16_t* x1 = a.Xt + (int64_t)(ka + 4 < a.K ? ka + 4 : a.K - 1) * a.Tp + t0 + 8 * rq;
#pragma unroll
    for (int s = 0; s < 8; ++s)
      if (t0 + 32 * s < a.Tp) {                                  // Tp is a multiple of 64
        xa[s] = frag(x0 + 32 * s, true);
        xb[s] = frag(x1 + 32 * s, true);
      }
  };
  if (32 * wave < a.K) {
    fetch_state(32 * wave);
    fetch_x(32 * wave, 0);
  }

  // R = x_scale X (W_q - W)^T [- C] of 16 tokens at a time, dY of it to LDS: accumulator lane -> row o, tokens 4 (lane / 16) + 0..3
  double mse = 0.0;
  const bf16_t* drow = p.delta + (int64_t)(row ? o : a.O - 1) * a.K;
  for (int t0 = 16 * wave; t0 < a.Tp; t0 += 16 * kSmallWaves) {
    const int tx = t0 + col < a.T ? t0 + col : a.T - 1, tg = t0 + 4 * rq;
    float4 c = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (a.C && row && tg < a.T) c = *reinterpret_cast<const float4*>(a.C + ((int64_t)(tg >> 2) * a.O + o) * 4);
    f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f}, odd = acc;
    const bf16_t* xrow = a.X + (int64_t)tx * a.K;
    for (int k0 = 8 * rq; k0 - 8 * rq < a.K; k0 += 256) {
      bf16x8 fx[8], fd[8];
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const int k = k0 + 32 * s;
        fx[s] = frag(xrow + k, k < a.K);
        fd[s] = frag(drow + k, k < a.K);
      }
#pragma unroll
      for (int s = 0; s < 8; s += 2) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fx[s], fd[s], acc, 0, 0, 0);
        odd = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fx[s + 1], fd[s + 1], odd, 0, 0, 0);
      }
    }
    acc += odd;
    const float cc[4] = {c.x, c.y, c.z, c.w};
    uint32_t b[4];
    float sum = 0.0f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float r = row && tg + v < a.T ? xs * acc[v] - cc[v] : 0.0f;
      sum += r * r;
      b[v] = f32_to_bf16(a.two_alpha * r);
    }
    mse += sum;
    *reinterpret_cast<uint2*>(dy + col * pitch + tg) = make_uint2(b[0] | (b[1] << 16), b[2] | (b[3] << 16));
  }
  __syncthreads();          // dY is complete, and nobody reads W_q - W any more

  // G of 32 columns at a time, and the update where it is: two products whose rows are dealt so that a lane holds 8 consecutive columns
  double rsum = 0.0, cross = 0.0;
  const bf16_t* yr = dy + col * pitch + 8 * rq;
  for (int k0 = 32 * wave; k0 < a.K; k0 += 32 * kSmallWaves) {
    const int k = k0 + 8 * rq;
    const bool in = row && k < a.K && valid;
    const int64_t e = (int64_t)o * a.K + k;
    if (k0 > 32 * wave) {
      fetch_state(k0);
      fetch_x(k0, 0);
    }
    f32x4 g0 = {0.0f, 0.0f, 0.0f, 0.0f}, g1 = g0, odd0 = g0, odd1 = g0;
    for (int t0 = 0;;) {
#pragma unroll
      for (int s = 0; s < 8; s += 2)
        if (t0 + 32 * s < a.Tp) {                                  // Tp is a multiple of 64
          const bf16x8 y = *reinterpret_cast<const bf16x8*>(yr + t0 + 32 * s), z = *reinterpret_cast<const bf16x8*>(yr + t0 + 32 * s + 32);
          g0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[s], y, g0, 0, 0, 0);
          g1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xb[s], y, g1, 0, 0, 0);
          odd0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[s + 1], z, odd0, 0, 0, 0);
          odd1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xb[s + 1], z, odd1, 0, 0, 0);
        }
      t0 += 256;
      if (t0 >= a.Tp) break;
      fetch_x(k0, t0);
    }
    g0 += odd0;
    g1 += odd1;
    if (in) {
      float g[8] = {g0[0], g0[1], g0[2], g0[3], g1[0], g1[1], g1[2], g1[3]};
      if (p.H) {
#pragma unroll
        for (int j = 0; j < 8; ++j) g[j] -= p.two_alpha_h * h[j];
      }
      const float s = effective_scale(sb, sg);
      adam8(g, codes, s, xs, p.beta, p.lam_over_n, p.o, v, m, u);
      store8(p.V + e, v);
      store8(p.M + e, m);
      store8(p.U + e, u);
      if (emit) {
        float x = 0.0f;
        rsum += soft_forward8(w, codes, s, v, p.beta_next, p.delta + e, nullptr, p.H != nullptr, h, x);
        cross += x;
      }
    }
  }

  // The sums of the workgroup meet in its first wavefront, which goes on alone: those of the next forward to their slots, this step's
  // to where the workgroup that arrives last finds it (see finish_gram of the products that end in the update)
  __shared__ double part[3][kSmallWaves];
  sum3<64>(mse, rsum, cross);
  if (lane == 0) {
    part[0][wave] = mse;
    part[1][wave] = rsum;
    part[2][wave] = cross;
  }
  __syncthreads();
  if (wave > 0) return;
  double total = part[0][lane % kSmallWaves], r = part[1][lane % kSmallWaves], c = part[2][lane % kSmallWaves];
  sum3<kSmallWaves>(total, r, c);
  const int item = blockIdx.x, items = gridDim.x;
  bool last = false;
  if (lane == 0) {
    __hip_atomic_store(a.mse_partials + item, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // the sum is where the others see it before the count says so
    last = __hip_atomic_fetch_add(p.guard_slot + kArrivals, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == items - 1u;
  }
  last = __shfl(static_cast<int>(last), 0) != 0;
  if (emit && valid)
    for (int k = item + items * lane; k < p.n_next; k += items * 64) {
      p.round_next[k] = lane == 0 && k == item ? r : 0.0;
      if (p.H) p.cross_next[k] = lane == 0 && k == item ? c : 0.0;
    }
  if (!valid && (item == 0 || last) && lane == 0) {              // the first one also where the counter is not a count
    const float nan = __uint_as_float(0x7FC00000u);
    *p.fin.loss_mse = *p.fin.loss_round = *p.fin.loss_total = nan;
  }
  if (!last) return;
  if (valid) {
    double sm = 0.0, sr = 0.0, sc = 0.0;
    for (int i = lane; i < items; i += 64) sm += __hip_atomic_load(a.mse_partials + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll 4
    for (int64_t i = lane; i < p.fin.n_round; i += 64) sr += p.fin.round_partials[i];
    if (p.fin.cross_partials)
#pragma unroll 4
      for (int64_t i = lane; i < p.fin.n_cross; i += 64) sc += p.fin.cross_partials[i];
    sum3<64>(sm, sr, sc);
    if (lane == 0) write_losses(p.fin, sm, sr, sc);
  }
  if (lane < kTagWords) p.guard_slot[lane] = emit && valid ? p.next_tag.w[lane] : 0u;
  if (lane == 0) p.guard_slot[kArrivals] = 0u;
}

}  // namespace

// Every workgroup reads all activations twice, at the 20 GB/s or so that one compute unit gets from beyond its die's L2: up to 2^15 of
// them that costs less than two launches, as long as a wavefront has one group of 32 columns to update (time in one launch over that
// in three, 256 / 1024 / 4096 outputs, K inputs by T tokens: 256x64 0.77 / 0.83 / 0.84, 128x256 0.87 / 0.90 / 1.00, 256x128 0.95 / 1.00 /
// 0.97; 128x384 1.04 / 1.04 / 1.07, 192x192 0.97 / 1.03 / 1.04, 256x192 1.10 / 1.13 / 1.04).  With two groups up to 320 inputs and 64 tokens
// (320x64 0.93 / 0.97 / 0.92; 384x64 0.99 / 1.01 / 0.93, 320x96 1.10 / 1.12 / 1.02, 512x32 1.12 / 1.05 / -, 1024x16 - / 1.29 / -).
// From 1024 tokens on the plan may split the sums over them, which this kernel does not.
// And no more workgroups than there are slots for the next step's sums, one for 2048 weights: with fewer than 128 inputs up to 16 outputs.
bool small_step(int64_t O, int64_t K, int64_t T) {
  return O <= 4096 && K <= 320 && padded_tokens(T) < 1024 && (K <= 256 ? T * K <= kSmallMax : T <= 64) && (O + kSmallRows - 1) / kSmallRows <= step_bwd_blocks(O * K);
}

hipError_t launch_small_step(const bf16_t* X, const bf16_t* Xt, const float* C, int64_t O, int64_t K, int64_t T, float two_alpha,
                             double* partials, const ForwardGuard& guard, StepBwdArgs a, hipStream_t st) {
  if (!small_step(O, K, T)) return hipErrorInvalidValue;
  const unsigned grid = static_cast<unsigned>((O + kSmallRows - 1) / kSmallRows);
  a.mse_partials = partials;
  a.n_mse = grid;
  const int Tp = static_cast<int>(padded_tokens(T));
  const SmallStep s{step_update(a), X, Xt, C, partials, two_alpha, static_cast<int>(O), static_cast<int>(K), static_cast<int>(T), Tp,
                    guard.slot != nullptr, guard.expect};
  const size_t lds = kSmallRows * (Tp + 8) * sizeof(bf16_t);     // at most 33 KB
  if (a.w_bf16) hipLaunchKernelGGL(k_small_step<bf16_t>, dim3(grid), dim3(kSmallThreads), lds, st, s);
  else hipLaunchKernelGGL(k_small_step<float>, dim3(grid), dim3(kSmallThreads), lds, st, s);
  return hipGetLastError();
}

}  // namespace faar
