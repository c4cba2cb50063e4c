// Device code of the pass that updates V (paper Eq. 2-5; Table 2 steps 11-13), shared by the kernels that make it on its own
// (faar_elementwise.hip) and the products that end in it (faar_gemm.hip).
#pragma once
#include "faar_internal.h"

namespace faar {

__device__ __forceinline__ double wave_sum(double a) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
  return a;
}

// lower node and interval width of magnitude code k in 0..6
__device__ __forceinline__ float node_lo(uint32_t k) {
  return k < 2u ? 0.5f * static_cast<float>(k) : __uint_as_float(((126u + (k >> 1)) << 23) | ((k & 1u) << 22));
}
__device__ __forceinline__ float node_width(uint32_t k) { return k < 4u ? 0.5f : (k < 6u ? 1.0f : 2.0f); }
// sigmoid through the hardware exp2 / reciprocal units (about 1 ulp each; not decision arithmetic)
__device__ __forceinline__ float h_beta_fast(float v, float beta) {
  return __builtin_amdgcn_rcpf(1.0f + __expf(-beta * (v - 0.5f)));
}
// signed scale  sign(w) * s  of a coded weight (0 for a zero weight)
__device__ __forceinline__ float signed_scale(uint32_t nib, float s) {
  return (nib & 7u) == 7u ? 0.0f : ((nib & 8u) ? -s : s);
}

// soft-quantised weight of one coded element
__device__ __forceinline__ float soft_weight(uint32_t nib, float s, float v, float beta) {
  const uint32_t k = nib & 7u;
  return signed_scale(nib, s) * (node_lo(k) + h_beta_fast(v, beta) * node_width(k));
}

__device__ __forceinline__ void store_bf16x8(bf16_t* p, const float (&x)[8]) {
  *reinterpret_cast<uint4*>(p) = make_uint4(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]),
                                            pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7]));
}

// delta = bf16(W_q - W) (and bf16(W_q) where Wq_full is given) for eight weights, plus their Round-Loss terms sum(1 - (2v - 1)^2)
// and, when the layer carries the constant H = C^T X_q (use_h; hh its eight values), the cross term sum(delta * H) of the loss, taken
// on the ROUNDED delta -- the operand the residual GEMM actually multiplies
__device__ __forceinline__ float soft_forward8(const float (&w)[8], uint32_t codes, float s, const float (&v)[8], float beta,
                                               bf16_t* __restrict__ delta, bf16_t* __restrict__ Wq_full, bool use_h,
                                               const float (&hh)[8], float& cross) {
  float out[8], full[8];
  float rsum = 0.0f;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float wq = soft_weight((codes >> (4 * j)) & 15u, s, v[j], beta);
    out[j] = wq - w[j];
    full[j] = wq;
    const float t = 2.0f * v[j] - 1.0f;
    rsum += 1.0f - t * t;
  }
  const uint4 packed = make_uint4(pack_bf16x2(out[0], out[1]), pack_bf16x2(out[2], out[3]),
                                  pack_bf16x2(out[4], out[5]), pack_bf16x2(out[6], out[7]));
  *reinterpret_cast<uint4*>(delta) = packed;
  if (use_h) {   // hh stays in registers: indexed by constants only
    const uint32_t r[4] = {packed.x, packed.y, packed.z, packed.w};
#pragma unroll
    for (int j = 0; j < 4; ++j)
      cross += __uint_as_float(r[j] << 16) * hh[2 * j] + __uint_as_float(r[j] & 0xFFFF0000u) * hh[2 * j + 1];
  }
  if (Wq_full) store_bf16x8(Wq_full, full);
  return rsum;
}

// dL/dV from the product's gradient g (units of 1 / xs), Adam and clip for eight weights, in place on v, m, u
__device__ __forceinline__ void adam8(const float (&g)[8], uint32_t codes, float s, float xs, float beta, float lam_over_n,
                                      const AdamScalars& o, float (&v)[8], float (&m)[8], float (&u)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const uint32_t nib = (codes >> (4 * j)) & 15u;
    const float h = h_beta_fast(v[j], beta);
    const float d = (xs * g[j]) * (signed_scale(nib, s) * node_width(nib & 7u) * beta * (h * (1.0f - h))) +
                    lam_over_n * (4.0f - 8.0f * v[j]);
    m[j] = o.beta1 * m[j] + (1.0f - o.beta1) * d;
    u[j] = o.beta2 * u[j] + (1.0f - o.beta2) * (d * d);
    const float step = o.lr * (m[j] * o.inv_bc1) * __builtin_amdgcn_rcpf(__builtin_amdgcn_sqrtf(u[j] * o.inv_bc2) + o.eps);
    v[j] = fminf(fmaxf(v[j] - step, 0.0f), 1.0f);  // V clipped to [0, 1] after every update
  }
}

// ---- loss finalisation: fixed-order sums of the per-block partials by one workgroup -------------
struct LossSums {
  const double* mse_partials;
  int64_t n_mse;
  float mse_scale;
  // with the constant part of the residual carried separately (R = A - C, A = x_scale * acc):
  // ||R||^2 = sum A^2 - 2 x_scale <delta, H> + ||C||^2; cross_partials sum to <delta, H>.  Null: mse_partials are ||R||^2.
  const double* cross_partials;
  int64_t n_cross;
  const double* c_norm2;
  const float* x_scale;
  const double* round_partials;
  int64_t n_round;
  double inv_n;
  float lambda_round;
  float *loss_mse, *loss_round, *loss_total;
};

// the step's losses from the sums of its partials
__device__ __forceinline__ void write_losses(const LossSums& f, double a, double b, double c) {
  if (f.cross_partials) a += *f.c_norm2 - 2.0 * static_cast<double>(f.x_scale ? *f.x_scale : 1.0f) * c;
  const double mse = a * static_cast<double>(f.mse_scale);
  const double rl = b * f.inv_n;
  if (f.loss_mse) *f.loss_mse = static_cast<float>(mse);
  if (f.loss_round) *f.loss_round = static_cast<float>(rl);
  if (f.loss_total) *f.loss_total = static_cast<float>(mse + static_cast<double>(f.lambda_round) * rl);
}

// kSameLaunch: mse_partials were stored past the writers' L2 in this launch, and are read past this one's
template <int kThreads, bool kSameLaunch = false>
__device__ __forceinline__ void finalize_block(const LossSums& f, bool valid = true) {
  if (!valid) {  // the step ran on a forward pass that is not the one its caller described: no result
    if (threadIdx.x == 0) {
      const float nan = __uint_as_float(0x7FC00000u);
      if (f.loss_mse) *f.loss_mse = nan;
      if (f.loss_round) *f.loss_round = nan;
      if (f.loss_total) *f.loss_total = nan;
    }
    return;
  }
  double a = 0.0, b = 0.0, c = 0.0;
  // per-thread partial sums in a fixed order; loads of one batch are independent
#pragma unroll 4
  for (int64_t i = threadIdx.x; i < f.n_mse; i += kThreads) {
    if (kSameLaunch) a += __hip_atomic_load(f.mse_partials + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else a += f.mse_partials[i];
  }
#pragma unroll 4
  for (int64_t i = threadIdx.x; i < f.n_round; i += kThreads) b += f.round_partials[i];
  if (f.cross_partials) {
#pragma unroll 4
    for (int64_t i = threadIdx.x; i < f.n_cross; i += kThreads) c += f.cross_partials[i];
  }
  __shared__ double sa[kThreads / 64], sb[kThreads / 64], sc[kThreads / 64];
  a = wave_sum(a);
  b = wave_sum(b);
  c = wave_sum(c);
  if ((threadIdx.x & 63) == 0) {
    sa[threadIdx.x >> 6] = a;
    sb[threadIdx.x >> 6] = b;
    sc[threadIdx.x >> 6] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    a = 0.0;
    b = 0.0;
    c = 0.0;
    for (int i = 0; i < kThreads / 64; ++i) {
      a += sa[i];
      b += sb[i];
      c += sc[i];
    }
    write_losses(f, a, b, c);
  }
}

// Everything the pass over V takes besides the gradient
struct StepUpdate {
  const float* s_global; const uint8_t* scales; const uint32_t* icodes;
  float *V, *M, *U;
  const float* x_scale;
  const float* H; float two_alpha_h;
  float beta, lam_over_n; AdamScalars o;
  LossSums fin;
  const void* W; float beta_next; bf16_t *delta, *wq_full;   // the next step's forward (beta_next 0: none)
  double *round_next, *cross_next; int n_next;               // its partial sums: n_next slots
  uint32_t* guard_slot; ForwardTag next_tag;
};
StepUpdate step_update(const StepBwdArgs& a);                // faar_elementwise.hip

}  // namespace faar
