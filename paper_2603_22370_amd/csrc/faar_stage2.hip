// Stage-2 objective on given model outputs (paper Sec. 3.5 "Stage 2", Eq. 6; Table 2 steps 18-22):
// temperature softmax of two logit tensors, KL(P_fp || P_q) and its gradient with respect to the quantised
// model's logits, the Frobenius MSE of the last hidden states and its gradient, and the sum of the layers'
// Round Losses.  HBM-bound row kernels: one workgroup per token row, a single pass for the loss (online
// max / sum / weighted-sum), a second pass over the same row (served from cache) only when the gradient is wanted.
#include <cmath>

#include "faar_device.h"
#include "faar_internal.h"

namespace faar {
namespace {

constexpr int kRowThreads = 1024;

// Running statistics of one row's logits a (z_fp) and b (z_q), k = log2(e) / tau:
//   ma = max a, sa = sum 2^(k (a - ma)), w = ws sum 2^(k (a - ma)) (a - b);  mb = max b, sb = sum 2^(k (b - mb))
// with ws = min(1, 1 / tau): entries of z_q at the type's lowest value make terms of that size, and their sum over tau has to stay
// finite where it is
// The vector unit bounds these kernels as much as memory does (four exponentials of four issue slots an entry), so what
// surrounds the exponentials counts: the maxima are those of the logits as they are (the subtraction comes first, so logits of any
// size and masks of the type's lowest value keep their meaning), one product makes the exponent, and nothing is compared with -inf.
// 2048 rows of 128256 bf16 logits, losses and gradient: 467 -> 396 us (3.4 -> 4.0 TB/s).
struct RowStats { float ma, sa, w, mb, sb; };

__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }
// a maximum to subtract: one that is still -inf would make 2^(-inf - -inf) of a masked entry NaN
__device__ __forceinline__ float finite_ref(float m) { return m == -INFINITY ? 0.0f : m; }

__device__ __forceinline__ RowStats merge(const RowStats& x, const RowStats& y, float k) {
  RowStats r;
  // a side that has seen no element has max -inf and sums 0: its factor is 2^-inf = 0, or 1 when both are empty
  r.ma = fmaxf(x.ma, y.ma);
  const float fx = x.ma == r.ma ? 1.0f : exp2_hw((x.ma - r.ma) * k), fy = y.ma == r.ma ? 1.0f : exp2_hw((y.ma - r.ma) * k);
  r.sa = x.sa * fx + y.sa * fy;
  r.w = (fx != 0.0f ? x.w * fx : 0.0f) + (fy != 0.0f ? y.w * fy : 0.0f);   // w of entries masked in z_fp alone may be infinite
  r.mb = fmaxf(x.mb, y.mb);
  const float gx = x.mb == r.mb ? 1.0f : exp2_hw((x.mb - r.mb) * k), gy = y.mb == r.mb ? 1.0f : exp2_hw((y.mb - r.mb) * k);
  r.sb = x.sb * gx + y.sb * gy;
  return r;
}

__device__ __forceinline__ RowStats shuffle_xor(const RowStats& x, int o) {
  RowStats r;
  r.ma = __shfl_xor(x.ma, o); r.sa = __shfl_xor(x.sa, o); r.w = __shfl_xor(x.w, o);
  r.mb = __shfl_xor(x.mb, o); r.sb = __shfl_xor(x.sb, o);
  return r;
}

// Eight vocabulary entries added to the running sums.  A logit of -inf (a masked entry) has probability 0: it adds nothing to
// either sum, and by the convention 0 log 0 = 0 nothing to the KL term either -- also where only z_fp is -inf.  Where P_fp > 0
// and z_q = -inf the term, and the row's KL, is +inf.  A row whose logits are all -inf has no softmax; its results are NaN.
__device__ __forceinline__ void accumulate8(RowStats& st, const float (&a)[8], const float (&b)[8], float k, float ws) {
  float ca = a[0], cb = b[0];
#pragma unroll
  for (int j = 1; j < 8; ++j) {
    ca = fmaxf(ca, a[j]);
    cb = fmaxf(cb, b[j]);
  }
  if (ca > st.ma) {  // rescale the running sums to the new maximum
    const float f = exp2_hw((st.ma - ca) * k);
    st.sa *= f;
    st.w = f != 0.0f ? st.w * f : 0.0f;
    st.ma = ca;
  }
  if (cb > st.mb) {
    st.sb *= exp2_hw((st.mb - cb) * k);
    st.mb = cb;
  }
  const float ra = finite_ref(st.ma), rb = finite_ref(st.mb);
  float w = 0.0f;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float e = exp2_hw((a[j] - ra) * k);
    st.sa += e;
    st.sb += exp2_hw((b[j] - rb) * k);
    w = __builtin_fmaf(e, a[j] - b[j], w);
  }
  w *= ws;
  if (!(fabsf(w) <= 3.402823466e+38f)) {   // 0 * inf: a masked entry among them, left out (or a NaN, which stays); or too large unscaled
    w = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float e = exp2_hw((a[j] - ra) * k);   // again: eight registers less over the common path
      if (e != 0.0f) w += e * (a[j] * ws - b[j] * ws);
    }
  }
  st.w += w;
}

// KL(P_fp || P_q) of a row: sum_j P_fp (log P_fp - log P_q) = w / (ws tau sa) - (ma - mb) / tau - log(sa / sb); combined in double, with
// the two log-sum-exp terms taken as one difference so that nearly equal distributions do not cancel at size log(vocab)
__device__ __forceinline__ double row_kl(const RowStats& t, float inv_tau, float ws) {
  return (static_cast<double>(t.w) / (static_cast<double>(ws) * static_cast<double>(t.sa)) -
          (static_cast<double>(t.ma) - static_cast<double>(t.mb))) * static_cast<double>(inv_tau) -
         log(static_cast<double>(t.sa) / static_cast<double>(t.sb));
}

// grad_coef (P_q - P_fp) of eight entries from their logits
struct GradCoef {
  float ra, rb, ca, cb;
  __device__ __forceinline__ GradCoef(const RowStats& t, float grad_coef)
      : ra(finite_ref(t.ma)), rb(finite_ref(t.mb)), ca(grad_coef / t.sa), cb(grad_coef / t.sb) {}
  __device__ __forceinline__ void operator()(const float (&a)[8], const float (&b)[8], float k, float (&o)[8]) const {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      o[j] = exp2_hw((b[j] - rb) * k) * cb - exp2_hw((a[j] - ra) * k) * ca;   // not fused: equal logits give exactly 0
  }
};

template <typename ZT>
__global__ void __launch_bounds__(kRowThreads)
k_stage2_kl(const ZT* __restrict__ Zf, const ZT* __restrict__ Zq, int64_t v8, float inv_tau, float ws, float k, float grad_coef,
            ZT* __restrict__ dZq, double* __restrict__ kl_rows) {
  const int64_t row = blockIdx.x;
  const ZT* zf = Zf + row * v8 * 8;
  const ZT* zq = Zq + row * v8 * 8;
  const float ninf = -INFINITY;
  RowStats st{ninf, 0.0f, 0.0f, ninf, 0.0f};
  // the next chunk is on its way while this one is added up (1408 rows of 72488 float32 logits: 406 -> 399 us)
  float na[8], nb[8];
  if (threadIdx.x < v8) {
    W8<ZT>::load(zf + threadIdx.x * 8, na);
    W8<ZT>::load(zq + threadIdx.x * 8, nb);
  }
  for (int64_t c = threadIdx.x; c < v8; c += kRowThreads) {
    float a[8], b[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      a[j] = na[j];
      b[j] = nb[j];
    }
    if (c + kRowThreads < v8) {
      W8<ZT>::load(zf + (c + kRowThreads) * 8, na);
      W8<ZT>::load(zq + (c + kRowThreads) * 8, nb);
    }
    accumulate8(st, a, b, k, ws);
  }
  // fixed-order reduction: butterfly inside each wavefront, then the wavefronts in index order
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) st = merge(st, shuffle_xor(st, o), k);
  __shared__ RowStats per_wave[kRowThreads / 64];
  __shared__ RowStats row_stats;
  if ((threadIdx.x & 63) == 0) per_wave[threadIdx.x >> 6] = st;
  __syncthreads();
  if (threadIdx.x == 0) {
    RowStats t = per_wave[0];
    for (int i = 1; i < kRowThreads / 64; ++i) t = merge(t, per_wave[i], k);
    row_stats = t;
    kl_rows[row] = row_kl(t, inv_tau, ws);
  }
  if (!dZq) return;
  __syncthreads();
  const GradCoef grad(row_stats, grad_coef);
  ZT* g = dZq + row * v8 * 8;
  for (int64_t c = threadIdx.x; c < v8; c += kRowThreads) {
    float a[8], b[8], o[8];
    W8<ZT>::load(zf + c * 8, a);
    W8<ZT>::load(zq + c * 8, b);
    grad(a, b, k, o);
    W8<ZT>::store(g + c * 8, o);
  }
}

// bf16 rows of up to NC * 1024 chunks (8 logits each): the row of Z_fp stays in registers (packed bf16, NC x 4
// VGPRs per lane) and the first kLdsChunks chunks per lane of Z_q's row stay in LDS between the loss pass and
// the gradient pass, so that only the rest of Z_q is read a second time.
constexpr int kLdsChunks = 9;  // 9 x 1024 lanes x 16 B = 144 KB of the 160 KB LDS

__device__ __forceinline__ void unpack8(const uint4& q, float (&x)[8]) {
  const uint32_t r[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    x[2 * i] = __uint_as_float(r[i] << 16);
    x[2 * i + 1] = __uint_as_float(r[i] & 0xFFFF0000u);
  }
}

template <int NC>
__global__ void __launch_bounds__(kRowThreads)
k_stage2_kl_resident(const bf16_t* __restrict__ Zf, const bf16_t* __restrict__ Zq, int64_t v8, float inv_tau, float ws, float k,
                     float grad_coef, bf16_t* __restrict__ dZq, double* __restrict__ kl_rows) {
  static_assert(NC >= kLdsChunks, "the LDS part is a prefix of the per-lane chunks");
  __shared__ uint4 q_lds[kLdsChunks][kRowThreads];
  const int64_t row = blockIdx.x;
  const uint4* zf = reinterpret_cast<const uint4*>(Zf + row * v8 * 8);
  const uint4* zq = reinterpret_cast<const uint4*>(Zq + row * v8 * 8);
  const unsigned n8 = static_cast<unsigned>(v8);   // at most NC * 1024
  const float ninf = -INFINITY;
  RowStats st{ninf, 0.0f, 0.0f, ninf, 0.0f};
  constexpr int kHeld = NC < 18 ? NC : 18;         // a 19th chunk's four registers are not there: it is read again
  uint4 rf[kHeld];
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const unsigned c = threadIdx.x + q * kRowThreads;
    if (q < kHeld) rf[q % kHeld] = make_uint4(0u, 0u, 0u, 0u);
    if (c < n8) {
      const uint4 ra = zf[c], rq = zq[c];
      if (q < kHeld) rf[q % kHeld] = ra;
      if (q < kLdsChunks) q_lds[q][threadIdx.x] = rq;
      float a[8], b[8];
      unpack8(ra, a);
      unpack8(rq, b);
      accumulate8(st, a, b, k, ws);
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) st = merge(st, shuffle_xor(st, o), k);
  __shared__ RowStats per_wave[kRowThreads / 64];
  __shared__ RowStats row_stats;
  if ((threadIdx.x & 63) == 0) per_wave[threadIdx.x >> 6] = st;
  __syncthreads();
  if (threadIdx.x == 0) {
    RowStats t = per_wave[0];
    for (int i = 1; i < kRowThreads / 64; ++i) t = merge(t, per_wave[i], k);
    row_stats = t;
  }
  // the row's KL, whose logarithm takes more registers than are left beside the row, when the row is no longer needed
  auto finish = [&] {
    if (threadIdx.x == 0) kl_rows[row] = row_kl(row_stats, inv_tau, ws);
  };
  if (!dZq) return finish();
  __syncthreads();
  const GradCoef grad(row_stats, grad_coef);
  uint4* g = reinterpret_cast<uint4*>(dZq + row * v8 * 8);
#pragma unroll
  for (int q = 0; q < NC; ++q) {
    const unsigned c = threadIdx.x + q * kRowThreads;
    if (c < n8) {
      const uint4 ra = q < kHeld ? rf[q % kHeld] : zf[c];
      const uint4 rq = q < kLdsChunks ? q_lds[q][threadIdx.x] : zq[c];   // each lane reads back its own LDS slots
      float a[8], b[8];
      unpack8(ra, a);
      unpack8(rq, b);
      float o[8];
      grad(a, b, k, o);
      g[c] = make_uint4(pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]), pack_bf16x2(o[4], o[5]), pack_bf16x2(o[6], o[7]));
    }
  }
  finish();
}

template <typename HT>
__global__ void __launch_bounds__(kEltThreads)
k_stage2_mse(const HT* __restrict__ Hf, const HT* __restrict__ Hq, int64_t n8, float two_scale, HT* __restrict__ dHq,
             double* __restrict__ partials) {
  float s = 0.0f;
  for (int64_t i = blockIdx.x * (int64_t)kEltThreads + threadIdx.x; i < n8; i += (int64_t)gridDim.x * kEltThreads) {
    float f[8], q[8], o[8];
    W8<HT>::load(Hf + i * 8, f);
    W8<HT>::load(Hq + i * 8, q);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float d = q[j] - f[j];
      s += d * d;
      o[j] = two_scale * d;
    }
    if (dHq) W8<HT>::store(dHq + i * 8, o);
  }
  double a = static_cast<double>(s);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
  __shared__ double sw[kEltThreads / 64];
  if ((threadIdx.x & 63) == 0) sw[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int i = 0; i < kEltThreads / 64; ++i) t += sw[i];
    partials[blockIdx.x] = t;
  }
}

// losses[0] = kl_scale * sum kl_rows, [1] = mse_scale * sum partials, [2] = sum round_losses,
// [3] = lambda_kl [0] + [1] + lambda_round [2]; sums in a fixed order, in double
__global__ void __launch_bounds__(kEltThreads)
k_stage2_finalize(const double* __restrict__ kl_rows, int64_t n_rows, float kl_scale, const double* __restrict__ mse_partials,
                  int64_t n_mse, float mse_scale, const float* __restrict__ round_losses, int64_t n_layers, float lambda_kl,
                  float lambda_round, float* __restrict__ losses) {
  double a = 0.0, b = 0.0, c = 0.0;
  for (int64_t i = threadIdx.x; i < n_rows; i += kEltThreads) a += kl_rows[i];
  for (int64_t i = threadIdx.x; i < n_mse; i += kEltThreads) b += mse_partials[i];
  for (int64_t i = threadIdx.x; i < n_layers; i += kEltThreads) c += static_cast<double>(round_losses[i]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o);
    b += __shfl_xor(b, o);
    c += __shfl_xor(c, o);
  }
  __shared__ double sa[kEltThreads / 64], sb[kEltThreads / 64], sc[kEltThreads / 64];
  if ((threadIdx.x & 63) == 0) {
    sa[threadIdx.x >> 6] = a;
    sb[threadIdx.x >> 6] = b;
    sc[threadIdx.x >> 6] = c;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    a = b = c = 0.0;
    for (int i = 0; i < kEltThreads / 64; ++i) {
      a += sa[i];
      b += sb[i];
      c += sc[i];
    }
    const double kl = a * static_cast<double>(kl_scale), mse = b * static_cast<double>(mse_scale);
    losses[0] = static_cast<float>(kl);
    losses[1] = static_cast<float>(mse);
    losses[2] = static_cast<float>(c);
    losses[3] = static_cast<float>(static_cast<double>(lambda_kl) * kl + mse + static_cast<double>(lambda_round) * c);
  }
}

}  // namespace

int64_t stage2_mse_blocks(int64_t n) {
  const int64_t b = (n / 8 + kEltThreads - 1) / kEltThreads;
  return b < kStepBwdMaxBlocks ? (b > 0 ? b : 1) : kStepBwdMaxBlocks;
}

hipError_t launch_stage2(const Stage2Args& a, hipStream_t st) {
  const float inv_tau = 1.0f / a.tau;
  const float ws = std::fmin(1.0f, inv_tau);
  const float grad_coef = a.lambda_kl * a.kl_scale * inv_tau;
  const float k = static_cast<float>(1.4426950408889634 / static_cast<double>(a.tau));   // logits -> exponents of two
  const int64_t v8 = a.vocab / 8;
  if (a.z_bf16 && v8 <= 16 * kRowThreads)
    hipLaunchKernelGGL(k_stage2_kl_resident<16>, dim3(static_cast<unsigned>(a.T)), dim3(kRowThreads), 0, st,
                       static_cast<const bf16_t*>(a.Z_fp), static_cast<const bf16_t*>(a.Z_q), v8, inv_tau, ws, k, grad_coef,
                       static_cast<bf16_t*>(a.dZ_q), a.kl_rows);
  else if (a.z_bf16 && v8 <= 19 * kRowThreads)
    hipLaunchKernelGGL(k_stage2_kl_resident<19>, dim3(static_cast<unsigned>(a.T)), dim3(kRowThreads), 0, st,
                       static_cast<const bf16_t*>(a.Z_fp), static_cast<const bf16_t*>(a.Z_q), v8, inv_tau, ws, k, grad_coef,
                       static_cast<bf16_t*>(a.dZ_q), a.kl_rows);
  else if (a.z_bf16)
    hipLaunchKernelGGL(k_stage2_kl<bf16_t>, dim3(static_cast<unsigned>(a.T)), dim3(kRowThreads), 0, st,
                       static_cast<const bf16_t*>(a.Z_fp), static_cast<const bf16_t*>(a.Z_q), a.vocab / 8, inv_tau, ws, k, grad_coef,
                       static_cast<bf16_t*>(a.dZ_q), a.kl_rows);
  else
    hipLaunchKernelGGL(k_stage2_kl<float>, dim3(static_cast<unsigned>(a.T)), dim3(kRowThreads), 0, st,
                       static_cast<const float*>(a.Z_fp), static_cast<const float*>(a.Z_q), a.vocab / 8, inv_tau, ws, k, grad_coef,
                       static_cast<float*>(a.dZ_q), a.kl_rows);
  if (hipError_t e = hipGetLastError()) return e;
  const int64_t nh = a.T * a.D;
  const int64_t blocks = stage2_mse_blocks(nh);
  const float two_scale = 2.0f * a.mse_scale;
  if (a.h_bf16)
    hipLaunchKernelGGL(k_stage2_mse<bf16_t>, dim3(static_cast<unsigned>(blocks)), dim3(kEltThreads), 0, st,
                       static_cast<const bf16_t*>(a.H_fp), static_cast<const bf16_t*>(a.H_q), nh / 8, two_scale,
                       static_cast<bf16_t*>(a.dH_q), a.mse_partials);
  else
    hipLaunchKernelGGL(k_stage2_mse<float>, dim3(static_cast<unsigned>(blocks)), dim3(kEltThreads), 0, st,
                       static_cast<const float*>(a.H_fp), static_cast<const float*>(a.H_q), nh / 8, two_scale,
                       static_cast<float*>(a.dH_q), a.mse_partials);
  if (hipError_t e = hipGetLastError()) return e;
  hipLaunchKernelGGL(k_stage2_finalize, dim3(1), dim3(kEltThreads), 0, st, a.kl_rows, a.T, a.kl_scale, a.mse_partials, blocks,
                     a.mse_scale, a.round_losses, a.round_losses ? a.n_layers : 0, a.lambda_kl, a.lambda_round, a.losses);
  return hipGetLastError();
}

}  // namespace faar
