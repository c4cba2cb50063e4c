// bf16 MFMA GEMMs of the FAAR layer step for gfx950 (paper Table 2 steps 8-10 and the chain rule
// of Eq. 5): the residual GEMM  X_q (W_q - W)^T - C  with its loss / dY epilogue, the weight
// gradient  dY^T X_q  and the optional input gradient  dY W_q.
//
// Every product is computed as an "NT" GEMM  acc[m][n] = sum_k A[m][k] B[n][k]  with both operands
// row-major and the contraction index contiguous; operands that the mathematics wants transposed
// (X_q^T, dY^T) are produced in that layout by the kernel that writes them, so one tuned
// main loop serves all of them.  The exceptions are the weight gradient of LLM-sized layers, whose
// contraction index is the token -- the row index of everything the layers produce: k_gemm_dma64 has a
// token-major form (acc[m][n] = sum_t A[t][m] B[t][n], LDS transposing reads) that takes dY and X_q as
// they are -- and the input gradient, which takes W_q that way (where a transposed copy is not faster).
//
// One main loop, k_gemm_dma64: slices of 64 of the contraction copied global -> LDS by global_load_lds_dwordx4 (no VGPR
// staging) into a ring of stages, 128-byte LDS rows, v_mfma_f32_16x16x32_bf16, one workgroup barrier per slice.  Described at
// the kernel.  Four tile shapes (plan_gemm): 256x256 and 256x128 with 8 wavefronts for products that fill the chip with them,
// 128x128 and 128x64 with a deep ring and the contraction shared out inside the workgroup for those that do not; the token-major
// form has 192-wide ones besides.  A contraction that is not a multiple of 64 ends
// in a slice whose missing chunks are copied from zeros.  Workgroups are dealt to the 8 XCDs in contiguous chunks of a grouped
// tile order so that each XCD's L2 sees a compact sub-grid.
#include <algorithm>
#include <type_traits>

#include "faar_copies.h"
#include "faar_internal.h"
#include "faar_step.h"

namespace faar {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---- epilogues -----------------------------------------------------------------------------

// fixed-order sum of one float per lane over the workgroup's wavefronts (4 or 8), as a double, to partials[item]
// (the sum itself comes back in thread 0)
__device__ __forceinline__ double workgroup_sum(double a) {
  __shared__ double s[8];
  a = wave_sum(a);
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = a;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0) {
    const int nw = blockDim.x >> 6;
    for (int i = 0; i < nw; ++i) t += s[i];
  }
  return t;
}
__device__ __forceinline__ void finish_sum(double sum, double* partials, int item) {
  const double t = workgroup_sum(sum);
  if (threadIdx.x == 0) partials[item] = t;
}

// kWithC:  R = x_scale * acc - C;  sum R^2;  dYt[n][m] = bf16(two_alpha R) (zero-padded to ldt); optional dY[m][n].
// !kWithC: the V-dependent part alone, for steps that carry the constant part of the gradient separately
//          (G = dY^T X_q = (2 alpha x_scale acc)^T X_q - 2 alpha C^T X_q):  A = x_scale * acc;  sum A^2;
//          dYt[n][m] = bf16(two_alpha A).  Nothing is read in the epilogue.
template <bool kWithC>
struct EpiResidualT {
  static constexpr bool kRowStaged = false;
  static constexpr bool kTransposedOut = true;  // the fast kernel stages dYt through LDS for full-line stores
  static constexpr int kMode = 0;               // 0: the whole main loop (1, 2: measurement variants, see EpiProbe)
  static constexpr bool kPaddedContraction = false;
  // The GEMM that follows (dW = dY^T X_q) reads X_q^T, which the pass that updates V has meanwhile pushed out of the
  // last-level cache; with either operand coming from HBM that GEMM runs ~25 % slower.  The BK = 64 main loop of this
  // kernel therefore reads `warm` (X_q^T, warm_chunks KB) on the side, 1 KB per wavefront and slice, and keeps nothing.
  static constexpr bool kWarm = true;
  const float* C;
  const float* x_scale;  // device scalar multiplying the A operand (activations stored in units of it); null = 1
  float xs;
  __device__ __forceinline__ void begin() { xs = x_scale ? *x_scale : 1.0f; }
  ForwardGuard guard;
  __device__ __forceinline__ void once() { consume_forward_tag(guard); }
  float two_alpha;
  bf16_t* dYt;
  int64_t ldt;
  bf16_t* dY;
  double* partials;
  float sum;
  const void* warm;      // null: nothing to read on the side
  int64_t warm_chunks;   // its size in KB (whole 1 KB chunks)
  // C of rows m..m+3 (m a multiple of 4) of column n: one 16-byte load from the row-group-interleaved layout
  // [ceil(M/4)][N][4] (zero outside the matrix); kept separate from value4 so that a whole slab's loads can be
  // issued before the first dependent store
  __device__ __forceinline__ float4 load4(int64_t m, int64_t n, const GemmDims& d) const {
    if (kWithC && n < d.N && m < d.M) return *reinterpret_cast<const float4*>(C + ((m >> 2) * d.N + n) * 4);
    return make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  }
  // four consecutive rows m..m+3 of column n -> four bf16 dY values (zero outside the matrix)
  __device__ __forceinline__ uint2 value4(const float (&acc)[4], const float4& c4, int64_t m, int64_t n, const GemmDims& d) {
    uint32_t b[4] = {0u, 0u, 0u, 0u};
    const float c[4] = {c4.x, c4.y, c4.z, c4.w};
    if (n < d.N) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (m + q < d.M) {
          const float r = kWithC ? xs * acc[q] - c[q] : xs * acc[q];
          sum += r * r;
          b[q] = f32_to_bf16(two_alpha * r);
          if (kWithC && dY) dY[(m + q) * d.N + n] = static_cast<bf16_t>(b[q]);
        }
      }
    }
    return make_uint2(b[0] | (b[1] << 16), b[2] | (b[3] << 16));
  }
  __device__ __forceinline__ void store_chunk(const uint4& v, int64_t m, int64_t n, const GemmDims& d) {
    if (n < d.N && m < ldt) *reinterpret_cast<uint4*>(dYt + n * ldt + m) = v;  // m, ldt multiples of 8
  }
  __device__ __forceinline__ void rows4(const float (&acc)[4], int64_t m, int64_t n, int, const GemmDims& d) {
    if (n >= d.N || m >= ldt) return;
    *reinterpret_cast<uint2*>(dYt + n * ldt + m) = value4(acc, load4(m, n, d), m, n, d);
  }
  // fixed-order sum over the workgroup's wavefronts (4 or 8)
  __device__ __forceinline__ void finish(int item) { finish_sum(sum, partials, item); }
};
typedef EpiResidualT<true> EpiResidual;
typedef EpiResidualT<false> EpiPerturbation;

// The V-dependent part of the residual with dY stored TOKEN-major, for the token-major dW GEMM that follows:
// A = x_scale * acc;  sum A^2 per work item;  dY[m][n] = bf16(two_alpha * A)  ([M, N] row-major, N a multiple of 8).
struct EpiPerturbationRows {
  static constexpr bool kTransposedOut = false;
  static constexpr bool kRowStaged = true;
  static constexpr bool kWarm = false;
  static constexpr int kMode = 0;
  static constexpr bool kPaddedContraction = false;
  const float* x_scale;
  float xs;
  ForwardGuard guard;
  float two_alpha;
  bf16_t* dY;
  double* partials;
  float sum;
  double total;   // of several tiles (run4)
  __device__ __forceinline__ void once() { consume_forward_tag(guard); }
  __device__ __forceinline__ void begin() { xs = x_scale ? *x_scale : 1.0f; }
  __device__ __forceinline__ void rows4(const float (&acc)[4], int64_t m, int64_t n, int, const GemmDims& d) {
    if (n >= d.N) return;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (m + q < d.M) {
        const float r = xs * acc[q];
        sum += r * r;
        dY[(m + q) * d.N + n] = static_cast<bf16_t>(f32_to_bf16(two_alpha * r));
      }
  }
  __device__ __forceinline__ void run8(const float (&acc)[8], int64_t m, int64_t n, int, const GemmDims& d) {
    if (m >= d.M || n >= d.N) return;
    uint32_t w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float r0 = xs * acc[2 * j], r1 = xs * acc[2 * j + 1];
      sum += r0 * r0;
      sum += r1 * r1;
      w[j] = f32_to_bf16(two_alpha * r0) | (f32_to_bf16(two_alpha * r1) << 16);
    }
    *reinterpret_cast<uint4*>(dY + m * d.N + n) = make_uint4(w[0], w[1], w[2], w[3]);
  }
  // columns n .. n + 3 of row m of the tile at m0, n0
  __device__ __forceinline__ void run4(const float (&acc)[4], int64_t m0, int64_t n0, int m, int n, const GemmDims& d) {
    if (m0 + m >= d.M || n0 + n >= d.N) return;
    uint32_t b[4];
    float s4 = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float r = xs * acc[j];
      s4 += r * r;
      b[j] = f32_to_bf16(two_alpha * r);
    }
    total += s4;
    *reinterpret_cast<uint2*>(reinterpret_cast<char*>(dY + m0 * d.N + n0) + (static_cast<uint32_t>(m) * static_cast<uint32_t>(d.N) + n) * 2u) =
        make_uint2(b[0] | (b[1] << 16), b[2] | (b[3] << 16));
  }
  __device__ __forceinline__ void finish(int item) { finish_sum(total + sum, partials, item); }
};

// The loss of a step whose dY comes from upstream, and nothing else: per work item the sum of (x_scale * acc - C)^2, or without C
// of (x_scale * acc)^2
template <bool kWithC>
struct EpiSumSq {
  static constexpr bool kRowStaged = false;
  static constexpr bool kWarm = false;
  static constexpr bool kTransposedOut = false;
  static constexpr int kMode = 0;
  static constexpr bool kPaddedContraction = false;
  const float* C;        // as in EpiResidualT
  const float* x_scale;
  float xs;
  ForwardGuard guard;
  double* partials;
  float sum;
  __device__ __forceinline__ void once() { consume_forward_tag(guard); }
  __device__ __forceinline__ void begin() { xs = x_scale ? *x_scale : 1.0f; }
  __device__ __forceinline__ void rows4(const float (&acc)[4], int64_t m, int64_t n, int, const GemmDims& d) {
    if (n >= d.N || m >= d.M) return;   // m is a multiple of 4
    float4 c4 = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (kWithC) c4 = *reinterpret_cast<const float4*>(C + ((m >> 2) * d.N + n) * 4);
    const float c[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (m + q < d.M) {
        const float r = xs * acc[q] - c[q];
        sum += r * r;
      }
  }
  __device__ __forceinline__ void finish(int item) { finish_sum(sum, partials, item); }
};

// out[split][m][n] = acc
struct EpiF32 {
  static constexpr bool kWarm = false;
  static constexpr bool kRowStaged = true;   // the main loop hands it runs of 8 columns of a row (run8)
  static constexpr bool kTransposedOut = false;
  static constexpr int kMode = 0;
  static constexpr bool kPaddedContraction = true;   // its contractions are padded token counts, multiples of 64
  float* out;
  __device__ __forceinline__ void once() {}
  __device__ __forceinline__ void begin() {}
  __device__ __forceinline__ void rows4(const float (&acc)[4], int64_t m, int64_t n, int split, const GemmDims& d) {
    if (n >= d.N) return;
    float* o = out + (int64_t)split * d.M * d.N;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (m + q < d.M) o[(m + q) * d.N + n] = acc[q];
  }
  // columns n..n+7 of row m (n and N multiples of 8)
  __device__ __forceinline__ void run8(const float (&r)[8], int64_t m, int64_t n, int split, const GemmDims& d) {
    if (m >= d.M || n >= d.N) return;
    float4* o = reinterpret_cast<float4*>(out + (int64_t)split * d.M * d.N + m * d.N + n);
    o[0] = make_float4(r[0], r[1], r[2], r[3]);
    o[1] = make_float4(r[4], r[5], r[6], r[7]);
  }
  __device__ __forceinline__ void finish(int) {}
};

struct GramOperands {
  const bf16_t* delta;     // the A operand, [M, N] row-major: not the buffer that the next step's forward goes to
  const float* diag_lo;    // [N]
  double* partials;        // one per work item
  bool check; ForwardTag expect;
};
// The weight gradient, used where it is made: dL/dV, Adam, clip and the next step's forward of the tile's weights straight from the
// accumulators (a product that is not split).  Bound by HBM: V, m, u, W, H, codes in and V, m, u, the next W_q - W out; the gradient
// itself, 8 of 42.5 bytes a weight, is neither written nor read, and a launch is saved.  The loads of the next 8 weights a lane takes
// are on their way while it works on its 8.  The losses of the step, whose partial sums are complete, are added up by workgroup 0.
// Whole steps, us: 6144x2048 at 8192 tokens, alone 422.8 -> 396.5; 8192x2048 at 4096 346.5 -> 312; 2048x8192 at 4096 in a chain
// 472 -> 446; 1024x2048 at 512 38.1 -> 34.5; seven linears on three streams 6.92 -> 6.78 ms.
// kGram: the same for delta * gram (EpiGram), on the buffer of W_q - W that the next step's does not go to.  6144x2048 145 -> 132 on
// 192x256 tiles, 4096x4096 236 -> 212, 8192x2048 187 -> 164; 2048x6144 level alone, three jobs side by side 217 -> 203.
template <typename WT, bool kGram = false>
struct EpiStep {
  static constexpr bool kWarm = false;
  static constexpr bool kRowStaged = false;
  static constexpr bool kTransposedOut = false;
  static constexpr int kMode = 0;
  static constexpr bool kPaddedContraction = !kGram;
  static constexpr bool kLateFetch = kGram;  // the first fetch after the first strips have left their registers
  static constexpr bool kChunked = true;     // the main loop hands it runs of 8 columns with what fetch() brought for them
  StepUpdate p;
  GramOperands gr;           // kGram only
  float sg, xs;
  double rsum, cross;   // 96 to 128 weights a lane: their runs of 8 meet in double
  bool valid;
  double mse;
  struct Chunk { float4 v0, v1, m0, m1, u0, u1, h0, h1; uint4 w, a; uint32_t codes, scale; };
  static constexpr bool kFetchW = sizeof(WT) == 2 && !kGram;   // ahead of their use; there are no registers for the others
  __device__ __forceinline__ void once() {
    if (!kGram && blockIdx.x == 0) finish_losses();
  }
  __device__ __forceinline__ void begin() {
    sg = *p.s_global;
    xs = p.x_scale ? *p.x_scale : 1.0f;
    if constexpr (kGram) {
      valid = true;                            // a forward made by this step's own first kernel, or a prepared one under this tag
      if (gr.check)
        for (int i = 0; i < kTagWords; ++i) valid &= p.guard_slot[i] == gr.expect.w[i];   // all loads at once
    } else {
      valid = p.guard_slot[kTagWords] != 0u;   // written by an earlier kernel of this step
    }
  }
  __device__ __forceinline__ void finish_losses() {
    const bool ok = p.guard_slot[kTagWords] != 0u;
    finalize_block<512>(p.fin, ok);
    if (p.beta_next > 0.0f && ok && threadIdx.x == 0) {   // nobody in this launch reads the tag words
      for (int i = 0; i < kTagWords; ++i) p.guard_slot[i] = p.next_tag.w[i];
    }
  }
  __device__ __forceinline__ bool skip() const { return !valid; }
  // Addresses: one 32-bit offset within the tile for all arrays, on bases that are uniform.  e0: first element of the tile (a multiple
  // of 16); o: offset of the run's first one (a multiple of 8).  (A pointer each would take the registers of a run.)
  template <typename P> static __device__ __forceinline__ const P* at(const P* base, int64_t e0, uint32_t bytes) {
    return reinterpret_cast<const P*>(reinterpret_cast<const char*>(base + e0) + bytes);
  }
  __device__ __forceinline__ void fetch(Chunk& c, int64_t e0, uint32_t o) const {
    c.scale = p.scales[(e0 >> 4) + (o >> 4)];
    c.codes = p.icodes[(e0 >> 3) + (o >> 3)];
    const float4* v = reinterpret_cast<const float4*>(at(p.V, e0, 4 * o));
    const float4* mm = reinterpret_cast<const float4*>(at(p.M, e0, 4 * o));
    const float4* uu = reinterpret_cast<const float4*>(at(p.U, e0, 4 * o));
    c.v0 = v[0]; c.v1 = v[1]; c.m0 = mm[0]; c.m1 = mm[1]; c.u0 = uu[0]; c.u1 = uu[1];
    if (p.H) {
      const float4* h = reinterpret_cast<const float4*>(at(p.H, e0, 4 * o));
      c.h0 = h[0]; c.h1 = h[1];
    }
    if (kGram) c.a = *reinterpret_cast<const uint4*>(at(gr.delta, e0, 2 * o));
    if (kFetchW && p.beta_next > 0.0f) c.w = *reinterpret_cast<const uint4*>(at(static_cast<const WT*>(p.W), e0, 2 * o));
  }
  __device__ __forceinline__ void run8(const float (&r)[8], const Chunk& c, int64_t e0, uint32_t o, int64_t n) {
    float g[8], hh[8] = {c.h0.x, c.h0.y, c.h0.z, c.h0.w, c.h1.x, c.h1.y, c.h1.z, c.h1.w};
    float v[8] = {c.v0.x, c.v0.y, c.v0.z, c.v0.w, c.v1.x, c.v1.y, c.v1.z, c.v1.w};
    float mm[8] = {c.m0.x, c.m0.y, c.m0.z, c.m0.w, c.m1.x, c.m1.y, c.m1.z, c.m1.w};
    float uu[8] = {c.u0.x, c.u0.y, c.u0.z, c.u0.w, c.u1.x, c.u1.y, c.u1.z, c.u1.w};
    if constexpr (kGram) {
      const float4 l0 = *reinterpret_cast<const float4*>(gr.diag_lo + n), l1 = *reinterpret_cast<const float4*>(gr.diag_lo + n + 4);
      const float lo[8] = {l0.x, l0.y, l0.z, l0.w, l1.x, l1.y, l1.z, l1.w};
      const uint32_t dw[4] = {c.a.x, c.a.y, c.a.z, c.a.w};
      const float k_out = p.two_alpha_h * xs, k_sum = xs * xs;
      float sum = 0.0f;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float a = __uint_as_float((j & 1) ? (dw[j >> 1] & 0xFFFF0000u) : (dw[j >> 1] << 16));
        const float t = r[j] + a * lo[j];
        sum += k_sum * (t * a);
        g[j] = k_out * t - p.two_alpha_h * hh[j];
      }
      mse += sum;
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) g[j] = p.H ? r[j] - p.two_alpha_h * hh[j] : r[j];
    }
    const float s = effective_scale(c.scale, sg);
    adam8(g, c.codes, s, xs, p.beta, p.lam_over_n, p.o, v, mm, uu);
    store8(const_cast<float*>(at(p.V, e0, 4 * o)), v);
    store8(const_cast<float*>(at(p.M, e0, 4 * o)), mm);
    store8(const_cast<float*>(at(p.U, e0, 4 * o)), uu);
    if (p.beta_next > 0.0f) {
      float w[8];
      if constexpr (kFetchW) {
        const uint32_t q[4] = {c.w.x, c.w.y, c.w.z, c.w.w};
#pragma unroll
        for (int j = 0; j < 8; ++j) w[j] = __uint_as_float((j & 1) ? (q[j >> 1] & 0xFFFF0000u) : (q[j >> 1] << 16));
      } else {
        W8<WT>::load(at(static_cast<const WT*>(p.W), e0, sizeof(WT) * o), w);
      }
      float x = 0.0f;
      rsum += soft_forward8(w, c.codes, s, v, p.beta_next, const_cast<bf16_t*>(at(p.delta, e0, 2 * o)),
                            p.wq_full ? const_cast<bf16_t*>(at(p.wq_full, e0, 2 * o)) : nullptr, p.H != nullptr, hh, x);
      cross += x;
    }
  }
  // the partial sums of the next step's forward, one per work item, and zeros in the slots that no work item has
  __device__ __forceinline__ void finish(int item, int items) {
    if (p.beta_next > 0.0f && valid) next_sums(item, items);
    if constexpr (kGram) finish_gram(item, items);
  }
  // The loss needs this launch's own sums: the workgroup that arrives last adds them up.  What it reads of the others are the partial
  // sums alone, stored past the L2 of the writer's die and read past the reader's (no write-back of a whole L2, which is what a
  // release at device scope costs); the tag, which every workgroup has read by then, is cleared or replaced by it as well.
  __device__ __forceinline__ void finish_gram(int item, int items) {
    __shared__ uint32_t last;
    if (!valid && item == 0) finalize_block<512>(p.fin, false);      // also where the counter is not a count
    __syncthreads();
    const double t = workgroup_sum(mse);
    if (threadIdx.x == 0) {
      uint32_t* counter = p.guard_slot + kArrivals;
      __hip_atomic_store(gr.partials + item, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");               // the sum is where the others see it before the count says so
      last = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == static_cast<uint32_t>(items) - 1u;
    }
    __syncthreads();
    if (!last) return;
    if (valid) finalize_block<512, true>(p.fin);
    if (threadIdx.x == 0) {
      for (int i = 0; i < kTagWords; ++i) p.guard_slot[i] = p.beta_next > 0.0f && valid ? p.next_tag.w[i] : 0u;
      p.guard_slot[kArrivals] = 0u;
    }
  }
  __device__ __forceinline__ void next_sums(int item, int items) {
    finish_sum(rsum, p.round_next, item);
    __syncthreads();
    if (p.H) {
      finish_sum(cross, p.cross_next, item);
      __syncthreads();
    }
    for (int k = item + items * (1 + static_cast<int>(threadIdx.x)); k < p.n_next; k += items * static_cast<int>(blockDim.x)) {
      p.round_next[k] = 0.0;
      if (p.H) p.cross_next[k] = 0.0;
    }
  }
};

// As EpiF32, for an A operand that is the sum of kTerms bf16 matrices side by side ([M, kTerms * Kd]): every work item walks its
// slices once per term, the last term first, so that the small ones are added up before the sums are large.
// 2048 x 2048 outputs, 8192 tokens, 4 splits: three products of 59 us, 13 of them writing partials, and three passes over the
// partials of 14 -> 160 and one of 13; the error against 64 bits is that of the separate products or less (2.7e-7 of the norm).
struct EpiF32Terms : EpiF32 {
  static constexpr int kTerms = 3;
};
template <class E, class = void> struct TermsOf { static constexpr int value = 1; };
template <class E> struct TermsOf<E, std::void_t<decltype(E::kTerms)>> { static constexpr int value = E::kTerms; };

// C_out(m, n) = (first ? Y[m][n] : C_out(m, n)) - x_scale * acc, with C_out in the row-group-interleaved layout
// [ceil(M/4)][N][4]: element (m, n) at ((m / 4) * N + n) * 4 + m % 4, so that the four consecutive rows a lane
// holds of one column are one 16-byte access and the 16 or 32 lanes of a row group touch contiguous memory.
// Rows M..4*ceil(M/4)-1 are written as zero.
// A bf16 Y whose rows are whole 16-byte chunks passes through LDS (stage_y): a lane's four rows of one column are four loads of two
// bytes otherwise, in segments of 32 bytes (8192 x 2048 outputs, contraction 2048: 104 -> 69 us).
template <bool kYbf16>
struct EpiSub {
  static constexpr bool kStagedInput = kYbf16;
  static constexpr bool kRowStaged = false;
  static constexpr bool kWarm = false;
  static constexpr bool kTransposedOut = false;
  static constexpr int kMode = 0;
  static constexpr bool kPaddedContraction = false;
  const void* Y;
  bool first;
  float* C_out;
  const float* x_scale;  // as in EpiResidual
  float xs;
  __device__ __forceinline__ void once() {}
  __device__ __forceinline__ void begin() { xs = x_scale ? *x_scale : 1.0f; }
  __device__ __forceinline__ void rows4(const float (&acc)[4], int64_t m, int64_t n, int, const GemmDims& d) {
    if (n >= d.N || m >= d.M) return;  // m is a multiple of 4
    float y[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (!first) {
      const float4 c = *reinterpret_cast<const float4*>(C_out + ((m >> 2) * d.N + n) * 4);
      y[0] = c.x; y[1] = c.y; y[2] = c.z; y[3] = c.w;
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (m + q < d.M) {
          const int64_t idx = (m + q) * d.N + n;
          y[q] = kYbf16 ? bf16_to_f32(static_cast<const bf16_t*>(Y)[idx]) : static_cast<const float*>(Y)[idx];
        }
    }
    store4(acc, y, m, n, d);
  }
  __device__ __forceinline__ void store4(const float (&acc)[4], const float (&y)[4], int64_t m, int64_t n, const GemmDims& d) {
    if (n >= d.N || m >= d.M) return;
    float o[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = (m + q < d.M) ? y[q] - xs * acc[q] : 0.0f;
    *reinterpret_cast<float4*>(C_out + ((m >> 2) * d.N + n) * 4) = make_float4(o[0], o[1], o[2], o[3]);
  }
  __device__ __forceinline__ bool staged_input(const GemmDims& d) const { return first && d.N % 8 == 0; }
  // columns n..n+7 of row m of Y (n and N multiples of 8), zero outside
  __device__ __forceinline__ uint4 input8(int64_t m, int64_t n, const GemmDims& d) const {
    if (m >= d.M || n >= d.N) return make_uint4(0u, 0u, 0u, 0u);
    return *reinterpret_cast<const uint4*>(static_cast<const bf16_t*>(Y) + m * d.N + n);
  }
  __device__ __forceinline__ void finish(int) {}
};

// out[m][n] = bf16(scale * acc)
struct EpiBf16 {
  static constexpr bool kRowStaged = true;    // the main loop hands it runs of 8 columns of a row (run8)
  static constexpr bool kWarm = false;
  static constexpr bool kTransposedOut = false;
  static constexpr int kMode = 0;
  static constexpr bool kPaddedContraction = false;
  bf16_t* out;
  const float* scale;   // device scalar multiplying the product (activations stored in units of it); null = 1
  float sc;
  __device__ __forceinline__ void once() {}
  __device__ __forceinline__ void begin() { sc = scale ? *scale : 1.0f; }
  __device__ __forceinline__ void rows4(const float (&acc)[4], int64_t m, int64_t n, int, const GemmDims& d) {
    if (n >= d.N) return;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (m + q < d.M) out[(m + q) * d.N + n] = static_cast<bf16_t>(f32_to_bf16(sc * acc[q]));
  }
  // columns n..n+7 of row m (n a multiple of 8): one 16-byte store when the row pitch allows it
  __device__ __forceinline__ void run8(const float (&r)[8], int64_t m, int64_t n, int, const GemmDims& d) {
    if (m >= d.M || n >= d.N) return;
    bf16_t* o = out + m * d.N + n;
    if (n + 8 <= d.N && (d.N & 7) == 0) {
      uint32_t w[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j] = f32_to_bf16(sc * r[2 * j]) | (f32_to_bf16(sc * r[2 * j + 1]) << 16);
      *reinterpret_cast<uint4*>(o) = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
      for (int j = 0; j < 8 && n + j < d.N; ++j) o[j] = static_cast<bf16_t>(f32_to_bf16(sc * r[j]));
    }
  }
  // columns n .. n + 3 of row m of the tile at m0, n0; N a multiple of 4
  __device__ __forceinline__ void run4(const float (&r)[4], int64_t m0, int64_t n0, int m, int n, const GemmDims& d) {
    if (m0 + m >= d.M || n0 + n >= d.N) return;
    *reinterpret_cast<uint2*>(reinterpret_cast<char*>(out + m0 * d.N + n0) + (static_cast<uint32_t>(m) * static_cast<uint32_t>(d.N) + n) * 2u) =
        make_uint2(f32_to_bf16(sc * r[0]) | (f32_to_bf16(sc * r[1]) << 16), f32_to_bf16(sc * r[2]) | (f32_to_bf16(sc * r[3]) << 16));
  }
  __device__ __forceinline__ void finish(int) {}
};

// Gram-matrix form of the step: A = W_q - W (M x N = O x K outputs, the contraction runs over K as well), B = bf16(Xq^T Xq).
// t = acc + (split 0: A[m][n] * diag_lo[n]) restores what the rounding took from B's diagonal;
// out[split][m][n] = two_alpha * x_scale * t  (what the dW GEMM of the token form leaves for the pass that updates V);
// per work item the partial sum of x_scale^2 * t * A[m][n], which over all items is ||x_scale Xq (W_q - W)^T||^2.
struct EpiGram {
  static constexpr bool kWarm = false;
  static constexpr bool kRowStaged = true;
  static constexpr bool kTransposedOut = false;
  static constexpr int kMode = 0;
  static constexpr bool kPaddedContraction = false;
  const bf16_t* delta;     // the A operand, [M, N] row-major
  const float* diag_lo;    // [N]
  const float* x_scale;
  float xs;
  ForwardGuard guard;
  float two_alpha;
  float* out;
  double* partials;
  float sum;
  __device__ __forceinline__ void once() { consume_forward_tag(guard); }
  __device__ __forceinline__ void begin() { xs = x_scale ? *x_scale : 1.0f; }
  __device__ __forceinline__ void rows4(const float (&acc)[4], int64_t m, int64_t n, int split, const GemmDims& d) {
    if (n >= d.N) return;
    float* o = out + (int64_t)split * d.M * d.N;
    const float lo = split == 0 ? diag_lo[n] : 0.0f;
    const float k_out = two_alpha * xs, k_sum = xs * xs;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (m + q < d.M) {
        const float a = bf16_to_f32(delta[(m + q) * d.N + n]);
        const float t = acc[q] + a * lo;
        o[(m + q) * d.N + n] = k_out * t;
        sum += k_sum * (t * a);
      }
  }
  // columns n..n+7 of row m (n and N multiples of 8): one 16-byte load of delta, two of diag_lo, two 16-byte stores
  __device__ __forceinline__ void run8(const float (&r)[8], int64_t m, int64_t n, int split, const GemmDims& d) {
    if (m >= d.M || n >= d.N) return;
    const uint4 dv = *reinterpret_cast<const uint4*>(delta + m * d.N + n);
    const uint32_t dw[4] = {dv.x, dv.y, dv.z, dv.w};
    float lo[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    if (split == 0) {
      const float4 l0 = *reinterpret_cast<const float4*>(diag_lo + n), l1 = *reinterpret_cast<const float4*>(diag_lo + n + 4);
      lo[0] = l0.x; lo[1] = l0.y; lo[2] = l0.z; lo[3] = l0.w; lo[4] = l1.x; lo[5] = l1.y; lo[6] = l1.z; lo[7] = l1.w;
    }
    const float k_out = two_alpha * xs, k_sum = xs * xs;
    float o[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float a = __uint_as_float((j & 1) ? (dw[j >> 1] & 0xFFFF0000u) : (dw[j >> 1] << 16));
      const float t = r[j] + a * lo[j];
      o[j] = k_out * t;
      sum += k_sum * (t * a);
    }
    float4* op = reinterpret_cast<float4*>(out + (int64_t)split * d.M * d.N + m * d.N + n);
    op[0] = make_float4(o[0], o[1], o[2], o[3]);
    op[1] = make_float4(o[4], o[5], o[6], o[7]);
  }
  __device__ __forceinline__ void finish(int item) { finish_sum(sum, partials, item); }
};

// Measurement epilogue (faar_gemm_probe): no output; every work item reports how many shader-clock cycles and how
// many ticks of the constant 100 MHz counter it took, so that the clock the compute units ran at can be read off.
// kMode selects what the main loop of k_gemm_dma64 keeps: 0 everything, 1 only the matrix instructions and their
// LDS reads (the stages are filled once and never refilled), 2 only the global->LDS copies.
template <int MODE>
struct EpiProbe {
  static constexpr bool kTransposedOut = false;
  static constexpr bool kWarm = false;
  static constexpr bool kRowStaged = false;
  static constexpr int kMode = MODE;
  static constexpr bool kPaddedContraction = false;
  unsigned long long* clocks;   // [items][2]
  float* sink;
  long long t0, w0;
  float sum;
  __device__ __forceinline__ void once() { t0 = clock64(); w0 = wall_clock64(); sum = 0.0f; }
  __device__ __forceinline__ void begin() {}
  __device__ __forceinline__ void rows4(const float (&acc)[4], int64_t, int64_t, int, const GemmDims&) {
    sum += (acc[0] + acc[1]) + (acc[2] + acc[3]);
  }
  __device__ __forceinline__ void finish(int item) {
    if (sum == 1.2345e-30f) *sink = sum;   // keeps the accumulators alive; never true for real operands
    if (threadIdx.x == 0) {
      clocks[2 * item] = static_cast<unsigned long long>(clock64() - t0);
      clocks[2 * item + 1] = static_cast<unsigned long long>(wall_clock64() - w0);
    }
  }
};

// ---- main loop: direct-to-LDS ring, swizzled LDS, interleaved schedule ------------------------------

// 16 bytes per lane from global memory straight into LDS at lds_addr + 16 * lane (lds_addr wave-uniform).
// Written as inline assembly so that the compiler's wait-count bookkeeping for ordinary LDS reads stays
// exact; completion is tracked by hand through vmcnt (wait_vmcnt) and the workgroup barrier.
__device__ __forceinline__ void dma16(const void* gptr, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(gptr) : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_addr_of(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const char*)p));
}
#define FAAR_WAIT_VMCNT(N) __builtin_amdgcn_s_waitcnt(0x0F70 | ((N)&0xF) | (((N) >> 4) << 14))

// Work item -> (tile, split).  Workgroup ids are dealt round-robin to the 8 XCDs by the hardware; XCD x
// takes the x-th contiguous chunk of the item list, and the list walks the tile grid in column-major
// groups of 8 tile rows, so the 32 workgroups resident on an XCD cover a compact 8 x 4 block of tiles.
__device__ __forceinline__ bool item_coords(int pid, int tiles_m, int tiles_n, int n_split, int& tm, int& tn, int& split,
                                            int& item) {
  const int nt = tiles_m * tiles_n, items = nt * n_split;
  const int chunk = (items + 7) / 8;
  item = (pid % 8) * chunk + pid / 8;
  if (pid / 8 >= chunk || item >= items) return false;
  split = item / nt;
  const int lin = item - split * nt;
  constexpr int GM = 8;
  const int per_group = GM * tiles_n;
  const int g = lin / per_group;
  const int first_m = g * GM;
  const int gsz = (tiles_m - first_m) < GM ? (tiles_m - first_m) : GM;
  const int r = lin - g * per_group;
  tm = first_m + r % gsz;
  tn = r / gsz;
  return true;
}

// The chip runs this loop power-limited on large products, and two things lower the energy per flop: global->LDS copies whose
// eight lanes per row make one 128-byte request (BK = 64) instead of two 64-byte ones, and the 16x16x32 MFMA,
// which reads and writes a quarter of the accumulator values per instruction of the 32x32x16 form for half
// its flops.  With BK = 64 only two stages fit next to a 256x256 tile (2 x 64 KB; three for 256x128), so a stage
// is refilled as soon as the workgroup has read it: ONE barrier per slice, placed before the slice's last MFMA phase, at
// which point every wavefront holds the last fragments of the slice in registers and the copies of the next
// slice (issued NS - 1 slices earlier, right after a barrier) have landed.
// Small tiles are bound by latencies: the time goes with the slices one workgroup walks, not with the bytes or the flops.  They
// use the LDS that their size leaves for a ring of four or six stages, and a second group of four wavefronts (WGK = 2): each
// group takes one of a slice's two MFMA phases on the whole tile, so that every SIMD has two wavefronts to switch between
// without a byte more read from LDS; the groups' sums meet once, at the end.  Measured per slice with about half of the compute
// units busy, against four wavefronts: 128x128 0.53-0.62 -> 0.31 us, 128x64 0.37 -> 0.21 us.  Against the former
// kernels for these shapes (BK = 32 slices in a 4-stage ring; register-staged where the contraction was not a multiple of 32):
// residual GEMM of a 512x2048 layer at 4096 tokens 25.2 -> 16.3 us, of 1000x1488 at 3001 tokens 30.4 -> 21 us.

constexpr int DBK64 = 64;

// How the operands are stored.  kNT: both with the contraction index contiguous.  kTN: both with the contraction index as the
// ROW index (A [Kd, lda], B [Kd, ldb]; acc[m][n] = sum_t A[t][m] B[t][n]) -- activations and their gradients as the layers
// produce them, token-major.  kNN: B alone that way (the input gradient dY W_q on W_q as the forward product reads it).  Of an
// operand with the contraction index as the row index a stage holds 64 rows (tokens) of BM or BN columns, and a wavefront gathers
// the 8 tokens x 1 column an MFMA lane needs with two of the LDS transposing reads of this architecture (ds_read_b64_tr_b16)
// instead of one 16-byte read.
enum { kNT = 0, kTN = 1, kNN = 2 };
template <int BM_, int BN_, int WGM_, int WGN_, int NS_, int kOperands_ = kNT, int WGK_ = 1>
struct Dma64Cfg {
  static constexpr int BM = BM_, BN = BN_, WGM = WGM_, WGN = WGN_, NS = NS_;  // NS ring stages
  static constexpr bool kTokenA = kOperands_ == kTN, kTokenB = kOperands_ != kNT;
  static constexpr int WGK = WGK_;                 // groups of wavefronts that share out a slice's MFMA phases
  static constexpr int NW = WGM * WGN * WGK, THREADS = 64 * NW;
  static constexpr int WM = BM / WGM, WN = BN / WGN;
  static constexpr int TM = WM / 16, TN = WN / 16;
  static constexpr int CPR = DBK64 / 8;            // 16-byte chunks per LDS row (8)
  static constexpr int RPI = 64 / CPR;             // rows written by one wave-wide DMA instruction (8)
  static constexpr int RB = 2;                     // rows per 256-byte bank cycle
  static constexpr int STAGE = (BM + BN) * DBK64;  // elements per stage
  static constexpr int P = (BM + BN) / RPI / NW;   // DMA instructions per wavefront per stage
  static constexpr int KK = DBK64 / 32 / WGK;      // MFMA phases per stage and wavefront (2, or 1 of the two)
  static constexpr int NF = TM + TN, NM = TM * TN;
  static constexpr int FSTEP = NM / NF >= 2 ? 2 : 1;  // one fragment prefetch every FSTEP MFMAs
  static constexpr int DSTEP = NM / P;                // one DMA issue every DSTEP MFMAs of the last phase
  static_assert(NF * FSTEP <= NM && P * DSTEP <= NM && DSTEP >= 1, "phase schedule");
  static_assert((WGK == 1 || (WGK == 2 && TM % 2 == 0)) && !(kTokenA && WGK != 1), "contraction groups");
  static_assert((BM + BN) % (RPI * NW) == 0 && TN % 2 == 0 && NS >= 2 && STAGE * NS * 2 <= 160 * 1024, "tile shape");
};

// Eight consecutive tokens of one column for every lane, from a token-major stage: two transposing reads of 4 tokens each.
// Within a group of 16 lanes, lane r supplies the address of 4 consecutive columns of one token; lane i receives column
// i % 4 of the tokens that lanes i / 4 + {0, 4, 8, 12} pointed at.  With lane r pointing at token r / 4, columns 4 (r % 4) ..,
// lane i therefore receives column i of tokens 0..3: an MFMA operand row per lane.  `p`: this lane's address for the first
// read; the second reads 4 tokens (4 * pitch elements) further on.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
template <int PITCH>
__device__ __forceinline__ bf16x8 read_tokens8(const bf16_t* p) {
  typedef __attribute__((address_space(3))) s16x4* lds_ptr;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 4 * PITCH));
  const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}
// XOR key of a token row's pairs of 16-byte chunks (32 bytes = the 16 columns one transposing read takes from a token) in a
// token-major stage of COLS columns per token.  One read touches 16 token rows -- 4 consecutive tokens in each of 4 groups 8
// apart -- and they must fall into the 8 different 32-byte bank groups, two rows each (the two cycles 512 bytes take anyway).
// 256 and 128 columns: a row is 512 or 256 bytes, every row starts at bank 0, so the key has 3 bits (token bits 0, 1, 3) and
// permutes a row's pairs within aligned groups of 8.  192 and 64 columns: a row is 384 or 128 bytes, odd rows start half-way
// round the banks, so token bit 0 is taken care of and the key has 2 bits (token bits 1, 3), permuting pairs within aligned groups of
// 4 -- which 12 pairs divide into.
template <int COLS>
__device__ __forceinline__ int token_key(int t) {
  static_assert(COLS == 256 || COLS == 128 || COLS == 192 || COLS == 64, "token-major operand width");
  return COLS % 128 == 0 ? (t & 3) | (((t >> 3) & 1) << 2) : ((t >> 1) & 1) | (((t >> 3) & 1) << 1);
}

// Hands a wavefront's TMW x TN accumulator tiles (rows wm .., columns wn .. of the output tile at m0, n0) to the epilogue
template <class E, class = void> struct StagedInput { static constexpr bool value = false; };
template <class E> struct StagedInput<E, std::void_t<decltype(E::kStagedInput)>> { static constexpr bool value = E::kStagedInput; };

template <class E, class = void> struct Chunked { static constexpr bool value = false; };
template <class E> struct Chunked<E, std::void_t<decltype(E::kChunked)>> { static constexpr bool value = E::kChunked; };

template <class C, int TMW, class Epi>
__device__ __forceinline__ void epilogue(Epi& epi, f32x4 (&acc)[TMW][C::TN], bf16_t* lds, int64_t m0, int64_t n0, int wm, int wn,
                                         int split, const GemmDims& d, int tid, int lane, int wave, int wc) {
  constexpr int TN = C::TN;
  const int col = lane & 15, rq = lane >> 4;
  if constexpr (StagedInput<Epi>::value) {
    if (epi.staged_input(d)) {
      // every wavefront brings 16 x WN of the bf16 input at a time through its own piece of LDS, a whole row group ahead
      constexpr int PITCH = C::WN + 4, RUNS = C::WN / 32;   // 4 * PITCH = 32 bytes mod 256: the four row groups miss each other
      static_assert(C::NW * 16 * PITCH <= C::NS * C::STAGE && C::WN % 32 == 0, "staging fits in the ring");
      bf16_t* stg = lds + wave * 16 * PITCH;
      uint4 next[RUNS];
      auto fetch = [&](int i) {
#pragma unroll
        for (int t = 0; t < RUNS; ++t) {
          const int idx = lane + 64 * t;
          next[t] = epi.input8(m0 + wm + i * 16 + idx / (C::WN / 8), n0 + wn + (idx % (C::WN / 8)) * 8, d);
        }
      };
      fetch(0);
      __syncthreads();                               // nobody reads the ring any more
#pragma unroll
      for (int i = 0; i < TMW; ++i) {
#pragma unroll
        for (int t = 0; t < RUNS; ++t) {
          const int idx = lane + 64 * t;
          uint2* p = reinterpret_cast<uint2*>(stg + (idx / (C::WN / 8)) * PITCH + (idx % (C::WN / 8)) * 8);
          p[0] = make_uint2(next[t].x, next[t].y);
          p[1] = make_uint2(next[t].z, next[t].w);
        }
        if (i + 1 < TMW) fetch(i + 1);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          float y[4];
#pragma unroll
          for (int v = 0; v < 4; ++v) y[v] = bf16_to_f32(stg[(4 * rq + v) * PITCH + j * 16 + col]);
          const float r[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
          epi.store4(r, y, m0 + wm + i * 16 + 4 * rq, n0 + wn + j * 16 + col, d);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
      return;
    }
  }
  if constexpr (Epi::kTransposedOut) {
    // Output is wanted transposed ([n][m], m contiguous) while a lane holds 4 consecutive m of one n: stage a 32-column slab
    // (two 16-column tiles) per wavefront column through LDS and write whole rows with 16 B per lane
    constexpr int LDT = C::BM + 4;          // pitch of 2 words beyond a multiple of 32: conflict-free 8-byte writes
    constexpr int ROWS = C::WGN * 32;
    constexpr int CPRW = C::BM / 8;
    static_assert(ROWS * LDT <= C::NS * C::STAGE, "staging buffer fits in the ring");
    bf16_t* stg = lds;
#pragma unroll
    for (int jj = 0; jj < TN / 2; ++jj) {
      __syncthreads();
      float4 cv[TMW][2];
#pragma unroll
      for (int i = 0; i < TMW; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          cv[i][h] = epi.load4(m0 + wm + i * 16 + 4 * rq, n0 + wn + (2 * jj + h) * 16 + col, d);
#pragma unroll
      for (int i = 0; i < TMW; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int ml = wm + i * 16 + 4 * rq;
          const float r[4] = {acc[i][2 * jj + h][0], acc[i][2 * jj + h][1], acc[i][2 * jj + h][2], acc[i][2 * jj + h][3]};
          *reinterpret_cast<uint2*>(stg + (wc * 32 + h * 16 + col) * LDT + ml) =
              epi.value4(r, cv[i][h], m0 + ml, n0 + wn + (2 * jj + h) * 16 + col, d);
        }
      __syncthreads();
      for (int idx = tid; idx < ROWS * CPRW; idx += C::THREADS) {
        const int row = idx / CPRW, ch = idx % CPRW;
        const uint2* src = reinterpret_cast<const uint2*>(stg + row * LDT + ch * 8);   // 8-byte aligned
        const uint2 lo = src[0], hi = src[1];
        epi.store_chunk(make_uint4(lo.x, lo.y, hi.x, hi.y), m0 + ch * 8, n0 + (row / 32) * C::WN + jj * 32 + (row % 32), d);
      }
    }
  } else if constexpr (Chunked<Epi>::value) {
    // strips of 16 rows of the wavefront's accumulator tiles, two or, where the ring has room, four at a time, through its own piece of
    // LDS, as above, and out again in runs of 8 columns of a row; the epilogue's own operands of a run are fetched while the run before
    // it is worked on (which takes the registers of the accumulators that have left).  Four strips of 64 columns fill the ring without
    // padding: their 16-column groups are XOR-permuted by the row group instead.
    constexpr bool kFour = Epi::kLateFetch && C::WN == 64 && TMW % 4 == 0 && C::NW * 64 * 64 * 4 <= C::NS * C::STAGE * 2;
    constexpr int STRIPS = kFour ? 4 : 2, PITCH = kFour ? 64 : C::WN + 4, CPR = C::WN / 8, RUNS = 16 * STRIPS * CPR / 64;
    constexpr int STAGES = TMW / STRIPS;
    static_assert(TMW % STRIPS == 0 && RUNS % 2 == 0 && C::NW * 16 * STRIPS * PITCH * 4 <= C::NS * C::STAGE * 2, "staging fits in the ring");
    if (epi.skip()) return;
    float* stg = reinterpret_cast<float*>(lds) + wave * 16 * STRIPS * PITCH;
    typename Epi::Chunk ck[2];
    const int64_t e0 = m0 * d.N + n0;
    const int mrows = static_cast<int>(d.M - m0 < C::BM ? d.M - m0 : C::BM), ncols = static_cast<int>(d.N - n0 < C::BN ? d.N - n0 : C::BN);
    auto place = [&](int g, int& m, int& n) {
      int idx = lane + 64 * g;
      asm volatile("" : "+v"(idx));                  // nothing of the addresses is kept from run to run
      m = wm + idx / CPR;
      n = wn + (idx % CPR) * 8;
      return m < mrows && n < ncols;
    };
    auto fetch = [&](typename Epi::Chunk& c, int g) {
      int m, n;
      if (place(g, m, n)) epi.fetch(c, e0, static_cast<uint32_t>(m) * static_cast<uint32_t>(d.N) + n);
    };
    auto work = [&](const typename Epi::Chunk& c, int st, int t) {
      const int idx = lane + 64 * t, row = idx / CPR, cg = idx % CPR;
      const float* src = stg + row * PITCH + (kFour ? (cg * 8) ^ (((row >> 2) & 3) * 16) : cg * 8);
      const float4 a = *reinterpret_cast<const float4*>(src);
      const float4 b = *reinterpret_cast<const float4*>(src + 4);
      const float r[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
      int m, n;
      if (place(st * RUNS + t, m, n)) epi.run8(r, c, e0, static_cast<uint32_t>(m) * static_cast<uint32_t>(d.N) + n, n0 + n);
    };
    if (!Epi::kLateFetch) fetch(ck[0], 0);
    __syncthreads();                                 // nobody reads the ring any more
#pragma unroll
    for (int st = 0; st < STAGES; ++st) {
#pragma unroll
      for (int h = 0; h < STRIPS; ++h)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            stg[(16 * h + 4 * rq + v) * PITCH + (kFour ? (j * 16) ^ (rq * 16) : j * 16) + col] = acc[STRIPS * st + h][j][v];
      if (Epi::kLateFetch && st == 0) fetch(ck[0], 0);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 1
      for (int t = 0; t < RUNS; t += 2) {
        const int g = st * RUNS + t;
        fetch(ck[1], g + 1);
        work(ck[0], st, t);
        if (g + 2 < STAGES * RUNS) fetch(ck[0], g + 2);
        work(ck[1], st, t + 1);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  } else if constexpr (Epi::kRowStaged) {
    // every wavefront stages one 16 x WN row of its accumulator tiles at a time through its own piece of LDS and hands the
    // epilogue runs of 8 consecutive columns of a row: 16-byte operand loads and stores, a quarter of the instructions
    constexpr int PITCH = C::WN + 4;                 // floats; 4 * PITCH = 16 mod 32: the two row groups of a half-wave miss each other
    constexpr int RUNS = 16 * (C::WN / 8) / 64;      // runs per lane and staged row
    static_assert(C::NW * 16 * PITCH * 4 <= C::NS * C::STAGE * 2 && (16 * (C::WN / 8)) % 64 == 0, "staging fits in the ring");
    float* stg = reinterpret_cast<float*>(lds) + wave * 16 * PITCH;
    __syncthreads();                                 // nobody reads the ring any more
#pragma unroll
    for (int i = 0; i < TMW; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) stg[(4 * rq + v) * PITCH + j * 16 + col] = acc[i][j][v];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int t = 0; t < RUNS; ++t) {
        const int idx = lane + 64 * t, row = idx / (C::WN / 8), cg = idx % (C::WN / 8);
        const float4 a = *reinterpret_cast<const float4*>(stg + row * PITCH + cg * 8);
        const float4 b = *reinterpret_cast<const float4*>(stg + row * PITCH + cg * 8 + 4);
        const float r[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        epi.run8(r, m0 + wm + i * 16 + row, n0 + wn + cg * 8, split, d);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  } else {
#pragma unroll
    for (int i = 0; i < TMW; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const float r[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
        epi.rows4(r, m0 + wm + i * 16 + 4 * rq, n0 + wn + j * 16 + col, split, d);
      }
  }
}

// what the chunks beyond the end of a contraction are copied from
__device__ const uint4 kZeroChunk = {0u, 0u, 0u, 0u};

// kTail: the contraction (a multiple of 8) ends inside its last slice
template <class C, bool kTail, class Epi>
__global__ void __launch_bounds__(C::THREADS)
k_gemm_dma64(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, GemmDims d, int tiles_m, int tiles_n, int n_split,
             int ksteps_per_split, Epi epi) {
  __shared__ __attribute__((aligned(1024))) bf16_t lds[C::NS * C::STAGE];
  // where the side reads of an epilogue with kWarm land: 1 KB per wavefront, never read
  __shared__ __attribute__((aligned(1024))) uint32_t warm_sink[Epi::kWarm ? C::NW * 256 : 4];
  epi.once();
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / (C::WGM * C::WGN), wxy = wave % (C::WGM * C::WGN);   // contraction group, position in the tile
  const int wm = (wxy / C::WGN) * C::WM, wn = (wxy % C::WGN) * C::WN;
  int tm, tn, split, item;
  if (!item_coords(blockIdx.x, tiles_m, tiles_n, n_split, tm, tn, split, item)) return;
  const int64_t m0 = (int64_t)tm * C::BM, n0 = (int64_t)tn * C::BN;
  const int ksteps = static_cast<int>((d.Kd + DBK64 - 1) / DBK64);
  const int kbeg = split * ksteps_per_split;
  const int kend = kbeg + ksteps_per_split < ksteps ? kbeg + ksteps_per_split : ksteps;
  constexpr int kTerms = TermsOf<Epi>::value;
  const int nk = kTerms * (kend - kbeg);
  constexpr int P = C::P, KK = C::KK, NF = C::NF, NM = C::NM, TM = C::TM, TN = C::TN;
  // vector-memory instructions a wavefront issues per slice: the copies, and one side read with kWarm.  Loads complete
  // in order, so the wait counts below are in units of this
  constexpr int PW = P + (Epi::kWarm ? 1 : 0);
  static_assert(PW * (C::NS - 1) < 64, "vmcnt is a 6-bit counter");

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.0f;

  if (nk > 0) {
    // DMA instruction q of this wavefront fills rows [(wave*P + q)*RPI, +RPI) of the stacked [A rows; B rows]
    // stage: lane -> row = base + lane / CPR, LDS slot = lane % CPR, global chunk = slot ^ ((row / RB) % CPR).
    // Rows beyond M (or N) are clamped to the last valid row: their products are never stored.
    const bf16_t* gsrc[P];
    int64_t gstep[P];   // elements from one slice to the next
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const int u = wave * P + q;                 // copy u fills 64 consecutive 16-byte slots of the stage
      const bool is_a = u < C::BM / 8;
      if (is_a ? C::kTokenA : C::kTokenB) {
        // an operand of COLS columns owns 64 tokens x COLS / 8 slots (a whole number of copies), slot -> token =
        // slot / (COLS / 8), LDS chunk = slot % (COLS / 8), global chunk = that ^ 2 key(token).  Columns beyond M (or N) are
        // clamped to the last whole chunk: their products are never stored.
        int t, chunk;
        if constexpr (C::kTokenA && C::BM == 256 && C::BN == 256) {   // two whole token rows per copy
          t = 2 * (is_a ? u : u - C::BM / 8) + lane / 32;
          chunk = (lane % 32) ^ (2 * token_key<256>(t));
        } else {
          const int slot = (is_a ? u : u - C::BM / 8) * 64 + lane;
          t = is_a ? slot / (C::BM / 8) : slot / (C::BN / 8);
          chunk = is_a ? (slot % (C::BM / 8)) ^ (2 * token_key<C::BM>(t)) : (slot % (C::BN / 8)) ^ (2 * token_key<C::BN>(t));
        }
        const int64_t first = is_a ? m0 : n0, width = is_a ? d.M : d.N, ld = is_a ? d.lda : d.ldb;
        const int64_t col = first + chunk * 8 <= width - 8 ? first + chunk * 8 : width - 8;
        gsrc[q] = (is_a ? A : B) + t * ld + col;
        gstep[q] = DBK64 * ld;
      } else {
        const int trow = u * C::RPI + lane / C::CPR;
        const int chunk = (lane % C::CPR) ^ ((trow / C::RB) % C::CPR);
        if (is_a) {
          const int64_t m = m0 + trow < d.M ? m0 + trow : d.M - 1;
          gsrc[q] = A + m * d.lda + chunk * 8;
        } else {
          const int64_t n = n0 + (trow - C::BM) < d.N ? n0 + (trow - C::BM) : d.N - 1;
          gsrc[q] = B + n * d.ldb + chunk * 8;
        }
        gstep[q] = DBK64;
      }
    }
    // side read (kWarm) that goes with slice `rel` of this work item: the 1 KB chunk of the epilogue's buffer whose number
    // counts (workgroup, slice, wavefront) triples from the END of the launch (workgroups are dispatched in the order of
    // their ids), so that the buffer is read late, close to the kernel that wants it; triples beyond the buffer re-read one
    // valid address (the instruction count per slice stays uniform)
    const uint32_t warm_dst = __builtin_amdgcn_readfirstlane(lds_addr_of(warm_sink + (Epi::kWarm ? wave * 256 : 0)));
    const int64_t warm_last = ((int64_t)gridDim.x - blockIdx.x) * nk - 1;   // triple number of slice 0, before the wavefront
    static_assert(!Epi::kWarm || (P - 1) * C::DSTEP + 1 < NM, "room for the side read after the slice's last copy");
#define FAAR_SIDE_READ(REL)                                                                                              \
  if constexpr (Epi::kWarm) {                                                                                            \
    const int64_t chunk_ = (warm_last - (REL)) * C::NW + wave;                                                           \
    const bool in_ = epi.warm != nullptr && (REL) < nk && chunk_ < epi.warm_chunks;                                      \
    dma16(in_ ? static_cast<const char*>(epi.warm) + chunk_ * 1024 + lane * 16 : reinterpret_cast<const char*>(A), warm_dst); \
  }
    // source of copy q of slice t
    static_assert(!(kTail && C::kTokenA), "the dW GEMM's contraction is a multiple of the slice");
    const int tail = static_cast<int>(d.Kd - (int64_t)(ksteps - 1) * DBK64);
    auto source = [&](int q, int64_t t) -> const bf16_t* {
      const bf16_t* g = gsrc[q] + t * gstep[q];
      if constexpr (kTail) {
        if (t == ksteps - 1) {
          const int u = wave * P + q;
          const int k = u < C::BM / 8 || !C::kTokenB
                            ? ((lane % C::CPR) ^ (((u * C::RPI + lane / C::CPR) / C::RB) % C::CPR)) * 8   // first of the chunk
                            : ((u - C::BM / 8) * 64 + lane) / (C::BN / 8);                                // token row
          if (k >= tail) g = reinterpret_cast<const bf16_t*>(&kZeroChunk);
        }
      }
      return g;
    };
    // with kTerms: slice `rel` of the work item is slice rel % per of its tokens, in the operand's last term first; the offsets (of A
    // and B) from the first slice's sources, the same for every copy
    static_assert(kTerms == 1 || (!C::kTokenA && !C::kTokenB && !kTail), "terms lie side by side in the rows of A");
    auto term_offsets = [&](int rel, int64_t& of_a, int64_t& of_b) {
      const int per = kend - kbeg, pass = (rel >= per) + (rel >= 2 * per);
      of_b = (int64_t)(kbeg + rel - pass * per) * DBK64;
      of_a = of_b + (kTerms - 1 - pass) * d.Kd;
    };
    // A product of fewer slices than the ring has stages copies no more than it has: every copy is then waited for before the first
    // slice, and the counted waits of the loop hold of themselves (with the half slice below: 8192 x 32 forward at 8192 tokens 46.3 ->
    // 41.7 us, 3072 x 96 at 2048 12.5 -> 12.1, 12288 x 160 at 4096 48.8 -> 46.9)
    const bool short_loop = nk < C::NS;
#pragma unroll
    for (int s = 0; s < C::NS; ++s) {
      if (short_loop && s >= nk) break;
      const int t = kbeg + s;
      int64_t of_a = 0, of_b = 0;
      if constexpr (kTerms > 1) term_offsets(t - kbeg, of_a, of_b);
#pragma unroll
      for (int q = 0; q < P; ++q)
        dma16(kTerms > 1 ? gsrc[q] + (wave * P + q < C::BM / 8 ? of_a : of_b) : source(q, t),
              __builtin_amdgcn_readfirstlane(lds_addr_of(lds + s * C::STAGE + (wave * P + q) * C::RPI * DBK64)));
      FAAR_SIDE_READ(s)
    }

    // fragment addresses: row = w? + i*16 + lane % 16, chunk = 4*kk + lane / 16, slot = chunk ^ ((row / RB) % CPR);
    // the 16 lanes that share a chunk index then cover 16 distinct 16-byte bank groups
    const int fr = lane & 15, kc = lane >> 4;
    const int sw = (fr / C::RB) % C::CPR;
    int a_off[KK], b_off[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const int slot = ((4 * (kg * KK + kk) + kc) ^ sw) * 8;
      a_off[kk] = (wm + fr) * DBK64 + slot;
      b_off[kk] = C::BM * DBK64 + (wn + fr) * DBK64 + slot;
    }
    // token-major stage: element offset of this lane's first transposing read for fragment i (A) / j (B) of phase 0.  The
    // lane points at token 8 (lane / 16) + (lane % 16) / 4 of the phase's 32 and at columns w? + 16 i + 4 (lane % 4); that
    // token's XOR key is the same in every phase and for both reads of a fragment (no key uses token bits 2, 4 or 5)
    int a_tr[TM] = {}, b_tr[TN] = {};
    const int tok = 8 * kc + (fr >> 2), phase0 = 32 * kg * KK;
    if constexpr (C::kTokenA) {
#pragma unroll
      for (int i = 0; i < TM; ++i) a_tr[i] = (phase0 + tok) * C::BM + (((wm / 16 + i) ^ token_key<C::BM>(tok)) * 16) + (fr & 3) * 4;
    }
    if constexpr (C::kTokenB) {
#pragma unroll
      for (int j = 0; j < TN; ++j)
        b_tr[j] = C::BM * DBK64 + (phase0 + tok) * C::BN + (((wn / 16 + j) ^ token_key<C::BN>(tok)) * 16) + (fr & 3) * 4;
    }
    // fragment i of the A rows (j of the B rows) for phase kk, from the stage at `src`
    auto frag_a = [&](const bf16_t* src, int kk, int i) -> bf16x8 {
      if constexpr (C::kTokenA) return read_tokens8<C::BM>(src + a_tr[i] + 32 * kk * C::BM);
      else return *reinterpret_cast<const bf16x8*>(src + a_off[kk] + i * 16 * DBK64);
    };
    auto frag_b = [&](const bf16_t* src, int kk, int j) -> bf16x8 {
      if constexpr (C::kTokenB) return read_tokens8<C::BN>(src + b_tr[j] + 32 * kk * C::BN);
      else return *reinterpret_cast<const bf16x8*>(src + b_off[kk] + j * 16 * DBK64);
    };
    bf16x8 fa[2][TM], fb[2][TN];

    if (short_loop) FAAR_WAIT_VMCNT(0);
    else FAAR_WAIT_VMCNT(PW * (C::NS - 1));  // slice 0 has landed (mine); barrier: everybody's
    __builtin_amdgcn_s_barrier();
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      fa[0][i] = frag_a(lds, 0, i);
      fa[1][i] = fa[0][i];
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      fb[0][j] = frag_b(lds, 0, j);
      fb[1][j] = fb[0][j];
    }

    // one slice; kOdd: which of the two fragment sets holds its first phase (with two phases a slice, always the first set)
    auto slice = [&](int it, auto kOdd) {
      bf16_t* st = lds + (it % C::NS) * C::STAGE;
      const bf16_t* sn = lds + ((it + 1) % C::NS) * C::STAGE;
      const bool more = it + C::NS < nk;
      const int64_t gslice = kbeg + it + C::NS;
      int64_t of_a = 0, of_b = 0;
      if constexpr (kTerms > 1) term_offsets(more ? it + C::NS : 0, of_a, of_b);
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        constexpr int kFirst = decltype(kOdd)::value;
        const int cur = (kFirst + kk) & 1;
        if (kk == KK - 1) {
          // this wavefront's copies of slice it+1 have landed and its reads of slice it are complete;
          // after the barrier that holds for the workgroup: stage `st` may be refilled, `sn` may be read
          constexpr int kInFlight = PW * (C::NS - 2);  // copies of later slices may stay in flight
          __builtin_amdgcn_s_waitcnt(0x0070 | (kInFlight & 0xF) | ((kInFlight >> 4) << 14));  // vmcnt(kInFlight) lgkmcnt(0)
          __builtin_amdgcn_s_barrier();
        }
        const bf16_t* src = (kk + 1 < KK) ? st : sn;
        const int nkk = (kk + 1 < KK) ? kk + 1 : 0;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          // boustrophedon over the tile grid: consecutive MFMAs share one operand
          const int mi = m / TN, mj = (mi & 1) ? TN - 1 - m % TN : m % TN;
          if constexpr (Epi::kMode != 2)
            acc[mi][mj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[cur][mi], fb[cur][mj], acc[mi][mj], 0, 0, 0);
          if constexpr (Epi::kMode != 2 && C::kTokenA && C::FSTEP == 2) {
            // token-major: a fragment is two transposing reads; one of them per MFMA instead of both every other MFMA
            // (in a slice's last phase, where the copies are issued too, spread over all of the phase's MFMAs: every
            // SKIP-th one goes without; in the others the reads have to be complete at the next barrier, so they go first)
            constexpr int SKIP = NM / (NM - 2 * NF);
            static_assert(NM % (NM - 2 * NF) == 0, "read schedule");
            const bool spread = kk == KK - 1;
            const int r = spread ? m - m / SKIP : m;
            if (r < 2 * NF && !(spread && m % SKIP == SKIP - 1)) {
              const int f = r / 2, h = r % 2;
              typedef __attribute__((address_space(3))) s16x4* lds_ptr;
              if (f == 0 || f > TN) {
                const int i = f == 0 ? 0 : f - TN;
                const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(src + a_tr[i] + 32 * nkk * C::BM + h * 4 * C::BM));
                s16x8 t = __builtin_bit_cast(s16x8, fa[cur ^ 1][i]);
                if (h == 0) t.lo = v; else t.hi = v;
                fa[cur ^ 1][i] = __builtin_bit_cast(bf16x8, t);
              } else {
                const int j = f - 1;
                const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(src + b_tr[j] + 32 * nkk * C::BN + h * 4 * C::BN));
                s16x8 t = __builtin_bit_cast(s16x8, fb[cur ^ 1][j]);
                if (h == 0) t.lo = v; else t.hi = v;
                fb[cur ^ 1][j] = __builtin_bit_cast(bf16x8, t);
              }
            }
          } else if constexpr (C::kTokenB && !C::kTokenA && C::WGK == 1 && 2 * (TM + 2 * TN) <= NM) {
            // B alone token-major, where there are MFMAs to spare: the same, one read each -- two for a fragment of B, one for a
            // fragment of A (dX on 256x256 tiles 1-4 % faster, T = 8192, 2048 x 6144: 176.5 -> 173.9 us; 256x128 tiles, with 12
            // reads to 16 MFMAs, lost as much and stay as they were)
            constexpr int R = TM + 2 * TN;
            const int r = kk == KK - 1 ? (m * R + NM - 1) / NM : m;
            if (r < R && (kk < KK - 1 || r * NM / R == m)) {
              if (r == 0 || r > 2 * TN) {
                const int i = r == 0 ? 0 : r - 2 * TN;
                fa[cur ^ 1][i] = frag_a(src, nkk, i);
              } else {
                const int j = (r - 1) / 2, h = (r - 1) % 2;
                typedef __attribute__((address_space(3))) s16x4* lds_ptr;
                const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(src + b_tr[j] + 32 * nkk * C::BN + h * 4 * C::BN));
                s16x8 t = __builtin_bit_cast(s16x8, fb[cur ^ 1][j]);
                if (h == 0) t.lo = v; else t.hi = v;
                fb[cur ^ 1][j] = __builtin_bit_cast(bf16x8, t);
              }
            }
          } else
          if (Epi::kMode != 2 && m % C::FSTEP == 0 && m / C::FSTEP < NF) {  // next phase's fragments: A0, B0..B(TN-1), A1..A(TM-1)
            const int f = m / C::FSTEP;
            if (f == 0) fa[cur ^ 1][0] = frag_a(src, nkk, 0);
            else if (f <= TN) fb[cur ^ 1][f - 1] = frag_b(src, nkk, f - 1);
            else fa[cur ^ 1][f - TN] = frag_a(src, nkk, f - TN);
          }
          if (Epi::kMode != 1 && kk == KK - 1 && m % C::DSTEP == 0 && m / C::DSTEP < P) {
            // slice it+NS into the stage just released; past the end every lane re-reads one valid address
            const int q = m / C::DSTEP;
            const bf16_t* g;
            if constexpr (kTerms > 1) g = gsrc[q] + (wave * P + q < C::BM / 8 ? of_a : of_b);
            else g = more ? source(q, gslice) : A;
            dma16(g, __builtin_amdgcn_readfirstlane(lds_addr_of(st + (wave * P + q) * C::RPI * DBK64)));
          }
          if (Epi::kMode != 1 && kk == KK - 1 && m == (P - 1) * C::DSTEP + 1) {   // right after the slice's last copy
            FAAR_SIDE_READ(it + C::NS)
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    };
    if constexpr (KK == 2) {
      // where the contraction ends in the first half of its last slice, the second half is zeros: one phase of matrix instructions on
      // the fragments at hand
      const bool half = kTail && kend == ksteps && tail <= DBK64 / 2;
      for (int it = 0; it < nk - half; ++it) slice(it, std::integral_constant<int, 0>{});
      if constexpr (kTail) {
        if (half) {
#pragma unroll
          for (int m = 0; m < NM; ++m)
            acc[m / TN][m % TN] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[0][m / TN], fb[0][m % TN], acc[m / TN][m % TN], 0, 0, 0);
        }
      }
    } else {
      for (int it = 0; it < nk; it += 2) {
        slice(it, std::integral_constant<int, 0>{});
        if (it + 1 < nk) slice(it + 1, std::integral_constant<int, 1>{});
      }
    }
    FAAR_WAIT_VMCNT(0);  // no copy may still be in flight into this workgroup's LDS when it retires
#undef FAAR_SIDE_READ
  }

  // accumulator layout of the 16x16 tile: lane -> column lane % 16, rows 4 * (lane / 16) + 0..3
  epi.begin();
  if constexpr (C::WGK == 2) {
    // the two groups exchange halves of their accumulators through LDS: each ends up with the sums of half the tile's rows
    constexpr int HT = TM / 2;
    f32x4* ex = reinterpret_cast<f32x4*>(lds) + (size_t)wave * HT * TN * 64 + lane;
    const f32x4* ex_in = reinterpret_cast<const f32x4*>(lds) + (size_t)(wave ^ (C::WGM * C::WGN)) * HT * TN * 64 + lane;
    static_assert(C::NW * HT * TN * 64 * 16 <= C::NS * C::STAGE * 2, "exchange fits in the ring");
    __syncthreads();
    f32x4 half[HT][TN];
#pragma unroll
    for (int i = 0; i < HT; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        half[i][j] = kg == 0 ? acc[i][j] : acc[HT + i][j];
        ex[(i * TN + j) * 64] = kg == 0 ? acc[HT + i][j] : acc[i][j];
      }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < HT; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) half[i][j] += ex_in[(i * TN + j) * 64];
    epilogue<C, HT>(epi, half, lds, m0, n0, wm + kg * (C::WM / 2), wn, split, d, tid, lane, wave, wxy % C::WGN);
  } else {
    epilogue<C, TM>(epi, acc, lds, m0, n0, wm, wn, split, d, tid, lane, wave, wxy % C::WGN);
  }
  if constexpr (Chunked<Epi>::value) epi.finish(item, tiles_m * tiles_n * n_split);
  else epi.finish(item);
}

// ---- several tiles a workgroup ----------------------------------------------------------------------------------------
// The same main loop for NT products of two and more rounds of the compute units: 256 resident workgroups walk their tiles, and the
// copies past the end of a tile are those of the next one's first slices, so that neither a tile's stores nor the latency of its first
// copies stand by themselves.  The ring therefore stays in use during the epilogue, which goes without LDS: the copies place the rows of
// B so that a lane's TN accumulator tiles are TN consecutive columns, and 16 lanes store a whole line.  The copies' addresses are buffer
// descriptors with one 32-bit offset a lane and copy (RoundsCopy), half the registers of pointers.
// A wavefront's stores count in the same in-order counter as its copies: those of the first two slices are older than the stores, and
// the wait in the first slice's last phase covers both.
// 16384x6144x2048, bf16 out: 321 -> 292 us between other kernels, 350 -> 332 with nothing but itself running (bound by power).  Whole
// steps: 6144x2048 at 8192 tokens 407 -> 399, 8192x2048 at 4096 (two rounds) 304.5 -> 299.5; a block 1.4 %.
typedef uint32_t u32x4r __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void dma16_buffer(u32x4r rsrc, uint32_t voff, uint32_t soff, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
}
__device__ __forceinline__ u32x4r buffer_of(const void* p, int64_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  u32x4r r;
  r.x = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a));
  r.y = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(a >> 32) & 0xFFFFu);
  r.z = __builtin_amdgcn_readfirstlane(bytes > 0xFFFFFFFFll ? 0xFFFFFFFFu : static_cast<uint32_t>(bytes));
  r.w = 0x00020000u;
  return r;
}

template <class C, class Epi>
__global__ void __launch_bounds__(C::THREADS)
k_gemm_dma64_rounds(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, GemmDims d, int tiles_m, int tiles_n, Epi epi) {
  __shared__ __attribute__((aligned(1024))) bf16_t lds[C::NS * C::STAGE];
  static_assert(!C::kTokenA && !C::kTokenB && C::WGK == 1 && C::KK == 2 && C::NS == 2 && C::TN == 4, "NT, two phases, two stages");
  static_assert(C::BM == C::BN, "one bound for the rows of either operand's tile");
  constexpr int P = C::P, NF = C::NF, NM = C::NM, TM = C::TM, TN = C::TN;
  static_assert((C::BM / 8) % P == 0, "a wavefront copies rows of one operand");
  epi.once();
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave / C::WGN) * C::WM, wn = (wave % C::WGN) * C::WN;
  int pid = blockIdx.x, tm, tn, split, item;
  if (!item_coords(pid, tiles_m, tiles_n, 1, tm, tn, split, item)) return;
  const int nk = static_cast<int>(d.Kd / DBK64);
  epi.begin();

  // A wavefront's copies are u = wave P .. wave P + P - 1, all of one operand; their offsets are made anew for every tile
  typedef RoundsCopy<C::BM, C::WN, TN> Copies;
  static_assert(P % 2 == 0, "the parity of a copy is that of its number in the wavefront");
  const bool of_a = wave * P < C::BM / 8;
  const uint32_t ld2 = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>((of_a ? d.lda : d.ldb) * 2));
  u32x4r rs;
  uint32_t voff[P];
  auto set_tile = [&](int tm_, int tn_) {
    const int64_t left = of_a ? d.M - (int64_t)tm_ * C::BM : d.N - (int64_t)tn_ * C::BN;
    rs = of_a ? buffer_of(A + (int64_t)tm_ * C::BM * d.lda, left * ld2) : buffer_of(B + (int64_t)tn_ * C::BN * d.ldb, left * ld2);
    const uint32_t rows = __builtin_amdgcn_readfirstlane(left < C::BM ? static_cast<uint32_t>(left) : C::BM);
#pragma unroll
    for (int q = 0; q < P; ++q) voff[q] = Copies::offset(wave * P + q, lane, rows, ld2);
  };
  auto copy = [&](int q, int slice, int stage) {
    const int u = wave * P + q;
    dma16_buffer(rs, voff[q], __builtin_amdgcn_readfirstlane(slice * (DBK64 * 2)),
                 __builtin_amdgcn_readfirstlane(lds_addr_of(lds + stage * C::STAGE + u * C::RPI * DBK64)));
  };
  set_tile(tm, tn);
#pragma unroll
  for (int s = 0; s < C::NS; ++s)
#pragma unroll
    for (int q = 0; q < P; ++q) copy(q, s, s);

  f32x4 acc[TM][TN];
  const int fr = lane & 15, kc = lane >> 4, sw = (fr / C::RB) % C::CPR;
  int a_off[2], b_off[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    const int slot = ((4 * kk + kc) ^ sw) * 8;
    a_off[kk] = (wm + fr) * DBK64 + slot;
    b_off[kk] = C::BM * DBK64 + (wn + fr) * DBK64 + slot;
  }
  auto frag_a = [&](const bf16_t* src, int kk, int i) -> bf16x8 { return *reinterpret_cast<const bf16x8*>(src + a_off[kk] + i * 16 * DBK64); };
  auto frag_b = [&](const bf16_t* src, int kk, int j) -> bf16x8 { return *reinterpret_cast<const bf16x8*>(src + b_off[kk] + j * 16 * DBK64); };
  bf16x8 fa[2][TM], fb[2][TN];
  FAAR_WAIT_VMCNT(P * (C::NS - 1));
  __builtin_amdgcn_s_barrier();
  int stage = 0;
  for (;;) {
    const int64_t m0 = (int64_t)tm * C::BM, n0 = (int64_t)tn * C::BN;
    pid += gridDim.x;
    const bool more = item_coords(pid, tiles_m, tiles_n, 1, tm, tn, split, item);
    const bf16_t* st0 = lds + stage * C::STAGE;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      fa[0][i] = frag_a(st0, 0, i);
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[0][j] = frag_b(st0, 0, j);
    int rel = C::NS;                 // the slice that this iteration's copies bring, of the tile they stand at
    for (int it = 0; it < nk; ++it) {
      bf16_t* st = lds + stage * C::STAGE;
      const bf16_t* sn = lds + (stage ^ 1) * C::STAGE;
      if (rel == nk) {               // from here on the next tile's (without one, this tile's again: never read)
        rel = 0;
        if (more) set_tile(tm, tn);
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        if (kk == 1) {               // as in k_gemm_dma64: the next slice has landed, this one's last fragments are in registers
          __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
          __builtin_amdgcn_s_barrier();
        }
        const bf16_t* src = kk == 0 ? st : sn;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
          const int mi = m / TN, mj = (mi & 1) ? TN - 1 - m % TN : m % TN;
          acc[mi][mj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[kk][mi], fb[kk][mj], acc[mi][mj], 0, 0, 0);
          if (m % C::FSTEP == 0 && m / C::FSTEP < NF) {
            const int f = m / C::FSTEP;
            if (f == 0) fa[kk ^ 1][0] = frag_a(src, kk ^ 1, 0);
            else if (f <= TN) fb[kk ^ 1][f - 1] = frag_b(src, kk ^ 1, f - 1);
            else fa[kk ^ 1][f - TN] = frag_a(src, kk ^ 1, f - TN);
          }
          if (kk == 1 && m % C::DSTEP == 0 && m / C::DSTEP < P) copy(m / C::DSTEP, rel, stage);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      ++rel;
      stage ^= 1;
    }
    // lane -> columns wn + 4 (lane % 16) + 0..3, rows wm + 16 i + 4 (lane / 16) + 0..3
    int mrow = wm + 4 * kc, ncol = wn + fr * TN;
    asm volatile("" : "+v"(mrow), "+v"(ncol));   // no address is kept across the main loop
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float r[4] = {acc[i][0][v], acc[i][1][v], acc[i][2][v], acc[i][3][v]};
        epi.run4(r, m0, n0, mrow + i * 16 + v, ncol, d);
      }
    if (!more) break;
  }
  FAAR_WAIT_VMCNT(0);   // no copy may still be in flight into this workgroup's LDS when it retires
  epi.finish(blockIdx.x);
}

typedef Dma64Cfg<256, 256, 2, 4, 2> CfgL64;  // 2 x 64 KB
typedef Dma64Cfg<256, 128, 4, 2, 3> CfgM64;  // 3 x 48 KB: copies stay in flight for two slices
typedef Dma64Cfg<128, 128, 2, 2, 4, kNT, 2> CfgS64;  // 4 x 32 KB, two contraction groups
typedef Dma64Cfg<128, 64, 2, 2, 6, kNT, 2> CfgN64;   // 6 x 24 KB, two contraction groups
typedef Dma64Cfg<256, 256, 2, 4, 2, kNN> CfgL64N;   // the same four on a token-major B
typedef Dma64Cfg<256, 128, 4, 2, 3, kNN> CfgM64N;
typedef Dma64Cfg<128, 128, 2, 2, 4, kNN, 2> CfgS64N;
typedef Dma64Cfg<128, 64, 2, 2, 6, kNN, 2> CfgN64N;
typedef Dma64Cfg<256, 256, 2, 4, 2, kTN> CfgT64;  // CfgL64 on token-major operands
// ... and with 192 rows (columns) per tile: 6144 x 2048 is 24 x 8 = 192 tiles of 256 x 256 -- a quarter of the 256 compute units
// idle -- but 32 x 8 = 256 tiles of 192 x 256
typedef Dma64Cfg<192, 256, 2, 4, 2, kTN> CfgT64A;
typedef Dma64Cfg<256, 192, 4, 2, 2, kTN> CfgT64B;
typedef Dma64Cfg<192, 256, 2, 4, 2> CfgL64A;   // the same on NT operands, for the Gram-form product that ends in the pass over V
typedef Dma64Cfg<256, 192, 4, 2, 2> CfgL64B;

inline int ceil_div(int64_t a, int64_t b) { return static_cast<int>((a + b - 1) / b); }

enum { KIND_L64 = 0, KIND_M64 = 1, KIND_S64 = 2, KIND_N64 = 3, KINDS = 4 };   // + FAAR_GEMM_L64: FAAR_GEMM_*
constexpr int kTileRows[KINDS] = {256, 256, 128, 128}, kTileCols[KINDS] = {256, 128, 128, 64};

struct Plan {
  int kind, tiles_m, tiles_n, n_split;
  int64_t items() const { return (int64_t)tiles_m * tiles_n * n_split; }
};

// Tile shape and contraction split, chosen by a small cost model (all times in microseconds, calibrated on
// MI355X with every compute unit busy).  A compute unit works through one 64-wide slice of a tile in slice_us;
// (0.66 and 0.42 are the small tiles' values with the chip full of them; alone they take half that, but then the rounds decide);
// an item's epilogue costs a fixed part plus its global traffic (reads count fully, writes half: they do not
// stall the wave) at one compute unit's share of the memory bandwidth.  Items are dealt in rounds of 256.
// Large tiles cut LDS and L2 traffic per flop but quantise badly on small outputs; splitting the contraction
// (allowed only where partial sums may be written separately) buys back occupancy at the price of one more
// float32 partial per split, which the consumer has to read.
// (Tiles with one side of 192 would fill units that these leave idle: alone, the Gram-form product of a 2048x6144 layer takes 165
// instead of 175 us on them, single-stream steps of layers 768 to 2304 wide 3-5 % less.  They move more bytes a flop, which costs
// where other streams use those units: seven linears on three streams 1.3-4.1 % more, three Gram-form jobs of 2304x2304 12 %, of
// 2048x6144 7 %.  So only the token-major dW GEMM of a step that is said to be alone takes them, gemm_tn_tiles, and the Gram-form
// product that ends in the pass over V, as long as that saves what they cost there, gram_update_tiles.)
struct EpiCost { float read_bytes, write_bytes; };  // per output element

constexpr double kSliceUs[KINDS] = {1.666, 1.104, 0.66, 0.42};
Plan plan_gemm(const GemmDims& d, bool may_split, EpiCost epi, int kinds = KINDS, const double* slice_us = kSliceUs) {
  const double cu_bytes_per_us = 17600.0;   // ~4.5 TB/s over 256 compute units
  const int64_t ksteps = (d.Kd + DBK64 - 1) / DBK64;
  Plan best{-1, 0, 0, 0};
  double best_cost = 0.0;
  for (int kind = 0; kind < kinds; ++kind) {
    for (int sp = 1; sp <= (may_split ? 8 : 1); ++sp) {
      if (sp > 1 && d.Kd / sp < 512) break;
      const int64_t per = (ksteps + sp - 1) / sp;
      if ((sp - 1) * per >= ksteps) continue;  // the last split would be empty
      const Plan p{kind, ceil_div(d.M, kTileRows[kind]), ceil_div(d.N, kTileCols[kind]), sp};
      const double rounds = static_cast<double>((p.items() + 255) / 256);
      const double epilogue = 3.0 + kTileRows[kind] * kTileCols[kind] * (epi.read_bytes + 0.5 * epi.write_bytes) / cu_bytes_per_us;
      double cost = rounds * (static_cast<double>(per) * slice_us[kind] + epilogue);
      // every extra split is one more float32 partial written here and read back by the consumer
      cost += (sp - 1) * static_cast<double>(d.M) * static_cast<double>(d.N) * 8.0 / 5.0e6;
      if (best.kind < 0 || cost < best_cost) {
        best = p;
        best_cost = cost;
      }
    }
  }
  return best;
}

constexpr EpiCost kEpiGram{2.0f, 4.0f}, kEpiResidual{4.0f, 2.0f}, kEpiF32{0.0f, 4.0f}, kEpiSub{4.0f, 4.0f}, kEpiBf16{0.0f, 2.0f}, kEpiNone{0.0f, 0.0f}, kEpiLoss{4.0f, 0.0f};

// kB: the B operand is [Kd, ldb] (kNN)
template <bool kB = false, class Epi>
hipError_t run(const bf16_t* A, const bf16_t* B, GemmDims d, Plan p, Epi epi, hipStream_t st) {
  if constexpr (Chunked<Epi>::value) {
    if (p.items() > epi.p.n_next) return hipErrorInvalidValue;
  }
  const bool tail = d.Kd % DBK64 != 0;
  const int ksteps = static_cast<int>((d.Kd + DBK64 - 1) / DBK64);
  const int per_split = (ksteps + p.n_split - 1) / p.n_split;
  const dim3 grid(static_cast<unsigned>((p.items() + 7) / 8 * 8));
#define FAAR_LAUNCH(CFG)                                                                                                      \
  do {                                                                                                                        \
    if (!tail)                                                                                                                \
      hipLaunchKernelGGL((k_gemm_dma64<CFG, false, Epi>), grid, dim3(CFG::THREADS), 0, st, A, B, d, p.tiles_m, p.tiles_n,     \
                         p.n_split, per_split, epi);                                                                          \
    else if constexpr (!Epi::kPaddedContraction)                                                                              \
      hipLaunchKernelGGL((k_gemm_dma64<CFG, true, Epi>), grid, dim3(CFG::THREADS), 0, st, A, B, d, p.tiles_m, p.tiles_n,      \
                         p.n_split, per_split, epi);                                                                          \
    else return hipErrorInvalidValue;                                                                                         \
  } while (0)
  if constexpr (kB) {
    if (p.kind == KIND_L64) FAAR_LAUNCH(CfgL64N);
    else if (p.kind == KIND_M64) FAAR_LAUNCH(CfgM64N);
    else if (p.kind == KIND_S64) FAAR_LAUNCH(CfgS64N);
    else FAAR_LAUNCH(CfgN64N);
  } else {
    if (p.kind == KIND_L64) FAAR_LAUNCH(CfgL64);
    else if (p.kind == KIND_M64) FAAR_LAUNCH(CfgM64);
    else if (p.kind == KIND_S64) FAAR_LAUNCH(CfgS64);
    else FAAR_LAUNCH(CfgN64);
  }
#undef FAAR_LAUNCH
  return hipGetLastError();
}

// Whether a product walks several tiles a workgroup: 256x256 tiles, two rounds of them, whole slices, more of them than the ring holds,
// offsets within a tile's rows below 2^32.  Long contractions have fewer ends of tiles to hide, and their rows, a multiple of 4 KB apart,
// meet in the same channels when all workgroups walk in step (16384x2048, contraction 6144: 309 us, 320 this way)
constexpr int kRoundsGrid = 256;
bool walks_rounds(const GemmDims& d, const Plan& p) {
  return p.kind == KIND_L64 && p.items() >= 2 * kRoundsGrid && d.Kd <= 4096 && p.n_split == 1 && d.Kd % DBK64 == 0 && d.Kd > 2 * DBK64 && d.N % 4 == 0 &&
         std::max(std::max(d.lda, d.ldb), d.N) <= (1 << 22);
}

template <class Epi>
hipError_t run_rounds(const bf16_t* A, const bf16_t* B, const GemmDims& d, const Plan& p, Epi epi, hipStream_t st) {
  hipLaunchKernelGGL((k_gemm_dma64_rounds<CfgL64, Epi>), dim3(kRoundsGrid), dim3(CfgL64::THREADS), 0, st, A, B, d, p.tiles_m, p.tiles_n, epi);
  return hipGetLastError();
}

}  // namespace

int64_t gemm_residual_partials(int64_t M, int64_t N, int64_t Kd) {  // the most any of the epilogues writes
  const GemmDims d{M, N, Kd, Kd, Kd};
  int64_t most = 0;
  for (const EpiCost& e : {kEpiResidual, kEpiBf16, kEpiNone, kEpiLoss}) most = std::max(most, plan_gemm(d, false, e).items());
  return most;
}

hipError_t launch_gemm_residual_rows(const bf16_t* A, const bf16_t* B, GemmDims d, const float* x_scale, float two_alpha,
                                     bf16_t* dY, double* mse_partials, int64_t* n_partials, const ForwardGuard& guard,
                                     hipStream_t st) {
  if (d.N % 8 != 0) return hipErrorInvalidValue;
  EpiPerturbationRows e{x_scale, 1.0f, guard, two_alpha, dY, mse_partials, 0.0f, 0.0};
  const Plan p = plan_gemm(d, false, kEpiBf16);
  if (walks_rounds(d, p)) {
    *n_partials = kRoundsGrid;
    return run_rounds(A, B, d, p, e, st);
  }
  *n_partials = p.items();
  return run(A, B, d, p, e, st);
}

hipError_t launch_gemm_residual(const bf16_t* A, const bf16_t* B, GemmDims d, const float* C, const float* x_scale,
                                float two_alpha, bf16_t* dYt, int64_t ldt, bf16_t* dY,
                                double* mse_partials, int64_t* n_partials, const ForwardGuard& guard, const void* warm,
                                int64_t warm_bytes, hipStream_t st) {
  const int64_t warm_chunks = warm ? warm_bytes / 1024 : 0;
  if (!dYt && !dY) {
    const Plan p = plan_gemm(d, false, C ? kEpiLoss : kEpiNone);
    *n_partials = p.items();
    if (C) return run(A, B, d, p, EpiSumSq<true>{C, x_scale, 1.0f, guard, mse_partials, 0.0f}, st);
    return run(A, B, d, p, EpiSumSq<false>{nullptr, x_scale, 1.0f, guard, mse_partials, 0.0f}, st);
  }
  if (C) {
    EpiResidual e{C, x_scale, 1.0f, guard, two_alpha, dYt, ldt, dY, mse_partials, 0.0f, warm, warm_chunks};
    const Plan p = plan_gemm(d, false, kEpiResidual);
    *n_partials = p.items();
    return run(A, B, d, p, e, st);
  }
  if (dY) return hipErrorInvalidValue;   // the un-transposed dY exists only with the constant
  EpiPerturbation e{nullptr, x_scale, 1.0f, guard, two_alpha, dYt, ldt, nullptr, mse_partials, 0.0f, warm, warm_chunks};
  const Plan p = plan_gemm(d, false, kEpiBf16);
  *n_partials = p.items();
  return run(A, B, d, p, e, st);
}

int choose_split(int64_t M, int64_t N, int64_t Kd) { return plan_gemm(GemmDims{M, N, Kd, Kd, Kd}, true, kEpiF32).n_split; }

GemmPlanInfo gemm_plan_info(int epilogue, int64_t M, int64_t N, int64_t Kd) {
  const GemmDims d{M, N, Kd, Kd, Kd};
  const Plan p = epilogue == kGemmEpiResidual ? plan_gemm(d, false, kEpiResidual)
               : epilogue == kGemmEpiF32    ? plan_gemm(d, true, kEpiF32)
               : epilogue == kGemmEpiSub    ? plan_gemm(d, false, kEpiSub)
               : epilogue == kGemmEpiNone   ? plan_gemm(d, false, kEpiNone)
               : epilogue == kGemmEpiLoss   ? plan_gemm(d, false, kEpiLoss)
               : epilogue == kGemmEpiGram   ? plan_gemm(d, true, kEpiGram)
                                            : plan_gemm(d, false, kEpiBf16);
  return GemmPlanInfo{p.kind, kTileRows[p.kind], kTileCols[p.kind], p.n_split};
}

hipError_t launch_gemm_f32(const bf16_t* A, const bf16_t* B, GemmDims d, float* out, int n_split,
                           hipStream_t st) {
  EpiF32 e{out};
  Plan p = plan_gemm(d, true, kEpiF32);
  if (p.n_split != n_split) return hipErrorInvalidValue;  // the caller sized its workspace with choose_split
  return run(A, B, d, p, e, st);
}

hipError_t launch_gemm_f32_terms(const bf16_t* A, const bf16_t* B, GemmDims d, float* out, int n_split, hipStream_t st) {
  const Plan p = plan_gemm(GemmDims{d.M, d.N, d.Kd, d.Kd, d.Kd}, true, kEpiF32);
  if (p.n_split != n_split || d.Kd % DBK64 != 0 || d.lda < 3 * d.Kd || d.lda % 8 != 0) return hipErrorInvalidValue;
  return run(A, B, d, p, EpiF32Terms{{out}}, st);
}

template <class C, class Epi>
static hipError_t run_tn(const bf16_t* A, const bf16_t* B, const GemmDims& d, int n_split, Epi epi, hipStream_t st) {
  const int tiles_m = ceil_div(d.M, C::BM), tiles_n = ceil_div(d.N, C::BN);
  const int ksteps = static_cast<int>(d.Kd / DBK64);
  const int per_split = (ksteps + n_split - 1) / n_split;
  const int64_t items = (int64_t)tiles_m * tiles_n * n_split;
  if constexpr (Chunked<Epi>::value) {
    if (items > epi.p.n_next) return hipErrorInvalidValue;
  }
  const dim3 grid(static_cast<unsigned>((items + 7) / 8 * 8));
  hipLaunchKernelGGL((k_gemm_dma64<C, false, Epi>), grid, dim3(C::THREADS), 0, st, A, B, d, tiles_m, tiles_n, n_split, per_split, epi);
  return hipGetLastError();
}

// 1 256 x 256, 2 192 x 256, 3 256 x 192: whichever needs the fewest rounds of the 256 compute units, weighted by the tile's area; the
// 192-wide ones, which are up to a third more, not where they are more than `most`
static int fewest_rounds(int64_t M, int64_t N, int n_split, int64_t most = INT64_MAX) {
  const int64_t cus = 256;
  auto rounds_area = [&](int64_t bm, int64_t bn) {
    const int64_t items = (int64_t)ceil_div(M, bm) * ceil_div(N, bn) * n_split;
    return items > most && bm * bn < 256 * 256 ? INT64_MAX : (items + cus - 1) / cus * bm * bn;
  };
  const int64_t c1 = rounds_area(256, 256), c2 = rounds_area(192, 256), c3 = rounds_area(256, 192);
  if (c2 < c1 && c2 <= c3) return 2;
  if (c3 < c1) return 3;
  return 1;
}

// The dW product updates V in its epilogue, token-major (tn) or on transposed operands, where it is not split -- and not by a few
// workgroups, whose 8192 weights each then take longer than a kernel over all of them (512x512 at 512 tokens, 32 work items: 21.5 us a
// step, 23.2 this way; 400x1024 at 300, 64: 23.1 / 23.7; 1280x1280 at 320, 200: 32.6 / 29.8; 1024x1024 at 64, 128: 24.8 / 23.2).
constexpr int64_t kUpdateMinItems = 96;
// The Gram form's loss waits for the last of its workgroups, about 4 us, which smaller layers do not get back (768x768 17.1 -> 20.5
// us, 1000x1488 27.7 -> 30.7, 1024x2048 32.7 -> 33.0; 2048x2048 49.1 -> 48.2); nor do larger ones that leave units idle (below).
constexpr int64_t kGramUpdateMin = (int64_t)1 << 22;
constexpr int64_t kUpdateMaxColumns = 1 << 21;   // 256 rows of them, 4 bytes each, are 32-bit offsets
// What the plan splits stays split, although a single sum with the update behind it can be faster (6144x2048 at 16384 tokens, 4 splits of
// 192 tiles and a pass over V that reads four gradients 433 us; one sum that ends in it 403): rounding errors grow with the root of a
// sum's length, and the gradient there was 7.9e-7 of its norm from 64 bits that way, 4.4e-7 as four partial sums.
// A work item leaves one partial sum of the next step's losses, for which there are step_bwd_blocks(O K) slots.
// In several rounds of the compute units the last one's update runs on those that it has work for, and the pass of its own on all of
// them: worth it from 13/16 of the rounds' places on, of three 256x256 rounds from 7/8 on (time over that with a pass of its own; at
// 0.69-0.79: 4208x7760 at 1920 tokens 1.08, 5440x6576 at 3136 1.05, 4672x7104 at 4475 1.05; two rounds at 0.81-0.86: 4096x6784 at 704 0.96,
// 5120x5184 at 1680 0.98, 5440x5040 at 2368 1.00; three: (0.84) 7040x5680 at 5056 1.03, (0.87) 5760x7344 at 704 1.02, (0.91) 6528x6848 at
// 1408 0.95; with 256x128 tiles and no dX from 3/4 on, 4096x4672 at 970, 0.77, 0.93).  One round: with dX, which finds less in the
// caches (with_dx), on transposed operands not of fewer than 192 large tiles over many tokens (2432x4048 at 3062 1.05, 7360x1344 at
// 1561 1.04; 1728x5952 at 1234 0.89; 4224x3264 at 1565, 221 tiles, 0.95).
bool gemm_dw_updates(int64_t O, int64_t K, int64_t T, bool with_dx) {
  const int64_t Tp = padded_tokens(T);
  const Plan p = plan_gemm(GemmDims{O, K, Tp, Tp, Tp}, true, kEpiF32);
  if (p.n_split != 1 || p.items() < kUpdateMinItems || p.items() > step_bwd_blocks(O * K) || K > kUpdateMaxColumns) return false;
  const int64_t rounds = (p.items() + 255) / 256;
  const int least = p.kind == KIND_M64 && !with_dx ? 12 : p.kind == KIND_L64 && rounds > 2 ? 14 : 13;
  if (rounds > 1 && p.items() * 16 < rounds * 256 * least) return false;
  return !(with_dx && p.kind == KIND_L64 && p.items() < 192 && T >= 1408 && !gemm_tn_usable(O, K, T));
}
bool gemm_dx_before_dw(int64_t O, int64_t K, int64_t T) {
  const int64_t Tp = padded_tokens(T);
  const Plan p = plan_gemm(GemmDims{O, K, Tp, Tp, Tp}, true, kEpiF32);
  return (p.kind == KIND_L64 || p.kind == KIND_M64) && !(K > 2 * O && T * O >= (int64_t)1 << 23);
}

template <typename WT>
static hipError_t run_dw_update(const bf16_t* A, const bf16_t* B, GemmDims d, bool tn, bool fill_device, const StepBwdArgs& a, hipStream_t st) {
  const EpiStep<WT> e{step_update(a), GramOperands{}, 0.0f, 1.0f, 0.0, 0.0, true, 0.0};
  if (!tn) return run(A, B, d, plan_gemm(d, true, kEpiF32), e, st);
  const int tiles = gemm_tn_tiles(d.M, d.N, d.Kd, fill_device);
  if (tiles == 2) return run_tn<CfgT64A>(A, B, d, 1, e, st);
  if (tiles == 3) return run_tn<CfgT64B>(A, B, d, 1, e, st);
  if (tiles == 1) return run_tn<CfgT64>(A, B, d, 1, e, st);
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_dw_update(const bf16_t* A, const bf16_t* B, GemmDims d, bool tn, bool fill_device, const StepBwdArgs& a,
                                 hipStream_t st) {
  if (plan_gemm(GemmDims{d.M, d.N, padded_tokens(d.Kd), 0, 0}, true, kEpiF32).n_split != 1 || d.N > kUpdateMaxColumns || d.lda % 8 != 0 ||
      d.ldb % 8 != 0)
    return hipErrorInvalidValue;
  return a.w_bf16 ? run_dw_update<bf16_t>(A, B, d, tn, fill_device, a, st) : run_dw_update<float>(A, B, d, tn, fill_device, a, st);
}

// 256 x 256 tiles become 192-wide ones where these need fewer rounds of the compute units, weighted by the tile's area, as in
// gemm_tn_tiles -- up to contractions over which they lose more beside other streams than the update saves (time over that of two
// launches, one job / two / three side by side: 192x256 tiles 2880x4352 0.92 / 1.00 / 0.99, 2688x4608 0.91 / 1.00 / 0.99, 2048x5120
// 0.98 / 1.02 / 1.03, 2304x5376 0.89 / 0.97 / 1.02, 7168x4736 0.94 / 1.04 / 1.01; 256x192 5888x2112 0.93 / 1.00 / 0.98, 4608x2688
// 0.94 / 0.96 / 0.99, 4096x3072 0.93 / 1.03 / 1.03, 2048x6144 0.92 / 1.05 / 1.05)
static int gram_update_tiles(int64_t O, int64_t K, Plan* p) {
  *p = plan_gemm(GemmDims{O, K, K, K, K}, true, kEpiGram);
  const int fewest = p->kind != KIND_L64 ? 1 : fewest_rounds(O, K, 1);
  const int tiles = fewest == 2 && K > 4608 ? 1 : fewest == 3 && K > 2688 ? 1 : fewest;
  if (tiles == 2) p->tiles_m = ceil_div(O, 192);
  if (tiles == 3) p->tiles_n = ceil_div(K, 192);
  return tiles;
}

bool gemm_gram_updates(int64_t O, int64_t K) {
  Plan p;
  const int tiles = gram_update_tiles(O, K, &p);
  if (p.n_split != 1 || O * K < kGramUpdateMin || K > kUpdateMaxColumns || 2 * p.items() > step_bwd_blocks(O * K)) return false;
  // The update on the units that the tiles occupy against one on all of them (time over that of two launches; share of the rounds' places
  // in brackets).  One round on 192-wide tiles, which the product alone would be faster on: 0.83-0.95.  On 256x128, by their weights:
  // 8192x544 1.04, 5376x880 1.04, 4992x1024 0.99, 5120x1280 0.94.  Otherwise from 0.9 on: (0.78) 7168x1792 1.06, (0.88) 14336x896 1.08,
  // (0.90) 5136x2688 0.98, (0.94) 7680x1920 0.96, (1) 8192x2048 0.88; in several rounds (0.73) 5696x2976 1.09, (0.82) 6720x3712 1.05,
  // (0.87) 5760x3648 1.00, (0.91) 4368x6464 1.00, (0.94) 7168x4736 0.95; on 128x128 (1) 2048x2048 0.96, (0.94) 1408x5632 0.90 -- but not
  // where the product is most of it: 8128x5712 in three rounds 1.02, 8192x8192 in four 1.02 to 1.13
  const int64_t rounds = (p.items() + 255) / 256;
  if (rounds == 1 && tiles != 1) return true;
  // where these would fill one round and the contraction is too long for them, on 256x256 tiles: level alone, and faster beside other
  // streams, which use the units that are left (as above: 2048x6144 1.00 / 0.95 / 0.94, 1536x8192 0.96 / 0.94 / 0.93, 2304x5376 1.01 /
  // 0.94 / 0.95; not of shorter ones, 4096x3072 1.05 / 0.93 / 0.94)
  if (rounds == 1 && p.kind == KIND_L64 && K >= 5120 && p.items() >= 176 && fewest_rounds(O, K, 1) != 1) return true;
  if (rounds == 1 && p.kind == KIND_M64) return O * K >= (int64_t)5 << 20;
  return p.items() * 10 >= rounds * 256 * 9 && rounds <= (p.kind == KIND_L64 && tiles == 1 ? 2 : 3);
}

template <typename WT>
static hipError_t run_gram_update(const bf16_t* delta, const bf16_t* gram, const GemmDims& d, const GramOperands& g, StepBwdArgs a,
                                  hipStream_t st) {
  Plan p;
  const int tiles = gram_update_tiles(d.M, d.N, &p), tm = p.tiles_m, tn = p.tiles_n;
  a.n_mse = p.items();
  const EpiStep<WT, true> e{step_update(a), g, 0.0f, 1.0f, 0.0, 0.0, true, 0.0};
  if (tiles == 1) return run(delta, gram, d, p, e, st);
  const int ksteps = static_cast<int>((d.Kd + DBK64 - 1) / DBK64);
  const dim3 grid(static_cast<unsigned>((a.n_mse + 7) / 8 * 8));
#define FAAR_LAUNCH(CFG, TAIL) \
  hipLaunchKernelGGL((k_gemm_dma64<CFG, TAIL, EpiStep<WT, true>>), grid, dim3(CFG::THREADS), 0, st, delta, gram, d, tm, tn, 1, ksteps, e)
  if (d.Kd % DBK64 == 0) { if (tiles == 2) FAAR_LAUNCH(CfgL64A, false); else FAAR_LAUNCH(CfgL64B, false); }
  else                   { if (tiles == 2) FAAR_LAUNCH(CfgL64A, true);  else FAAR_LAUNCH(CfgL64B, true); }
#undef FAAR_LAUNCH
  return hipGetLastError();
}

hipError_t launch_gemm_gram_update(const bf16_t* delta, const bf16_t* gram, int64_t O, int64_t K, const float* diag_lo, double* partials,
                                   const ForwardGuard& guard, StepBwdArgs a, hipStream_t st) {
  if (!gemm_gram_updates(O, K)) return hipErrorInvalidValue;
  const GemmDims d{O, K, K, K, K};
  a.mse_partials = partials;
  const GramOperands g{delta, diag_lo, partials, guard.slot != nullptr, guard.expect};
  return a.w_bf16 ? run_gram_update<bf16_t>(delta, gram, d, g, a, st) : run_gram_update<float>(delta, gram, d, g, a, st);
}

int choose_split_gram(int64_t O, int64_t K) { return plan_gemm(GemmDims{O, K, K, K, K}, true, kEpiGram).n_split; }
int64_t gemm_gram_partials(int64_t O, int64_t K) { return plan_gemm(GemmDims{O, K, K, K, K}, true, kEpiGram).items(); }

hipError_t launch_gemm_gram(const bf16_t* delta, const bf16_t* gram, int64_t O, int64_t K, const float* diag_lo,
                            const float* x_scale, float two_alpha, float* out, int n_split, double* partials,
                            int64_t* n_partials, const ForwardGuard& guard, hipStream_t st) {
  const GemmDims d{O, K, K, K, K};
  const Plan p = plan_gemm(d, true, kEpiGram);
  if (p.n_split != n_split) return hipErrorInvalidValue;  // the caller sized its workspace with choose_split_gram
  *n_partials = p.items();
  EpiGram e{delta, diag_lo, x_scale, 1.0f, guard, two_alpha, out, partials, 0.0f};
  return run(delta, gram, d, p, e, st);
}

// Tile shape of the token-major product: 0 not usable, 1 256 x 256, 2 192 x 256, 3 256 x 192.  The contraction split is the
// one planned for 256 x 256 tiles.  fill_device: the kernel has the device to itself, so a 192-wide shape is taken when its
// work items need fewer rounds of the 256 compute units, weighted by the tile's area (6144 x 2048, one split: 192 items of
// 65536 -> one round at 65536; 256 items of 49152 -> one round at 49152).  Otherwise other kernels run on whatever units this
// one leaves idle, and the tile with the most work per byte moved wins: 256 x 256.
int gemm_tn_tiles(int64_t M, int64_t N, int64_t T, bool fill_device) {
  if (T <= 0 || T % DBK64 != 0 || M % 8 != 0 || N % 8 != 0) return 0;
  const Plan p = plan_gemm(GemmDims{M, N, T, T, T}, true, kEpiF32);
  if (p.kind != KIND_L64) return 0;
  if (!fill_device) return 1;
  const int64_t slots = step_bwd_blocks(M * N);   // of a product that updates V, one a work item
  return fewest_rounds(M, N, p.n_split, p.n_split == 1 && p.items() <= slots ? slots : INT64_MAX);
}
bool gemm_tn_usable(int64_t M, int64_t N, int64_t T) { return gemm_tn_tiles(M, N, T, false) != 0; }

hipError_t launch_gemm_f32_tn(const bf16_t* A, const bf16_t* B, GemmDims d, float* out, int n_split, bool fill_device,
                              hipStream_t st) {
  const int tiles = gemm_tn_tiles(d.M, d.N, d.Kd, fill_device);
  if (tiles == 0 || d.lda % 8 != 0 || d.ldb % 8 != 0) return hipErrorInvalidValue;
  const Plan p = plan_gemm(GemmDims{d.M, d.N, d.Kd, d.Kd, d.Kd}, true, kEpiF32);
  if (p.n_split != n_split) return hipErrorInvalidValue;
  if (tiles == 2) return run_tn<CfgT64A>(A, B, d, n_split, EpiF32{out}, st);
  if (tiles == 3) return run_tn<CfgT64B>(A, B, d, n_split, EpiF32{out}, st);
  return run_tn<CfgT64>(A, B, d, n_split, EpiF32{out}, st);
}

// What the probe runs a product on: the two large tiles, which have its variants.  Whether it takes a product at all is a matter of
// its own, not of the tiles that the library's products have come to take since: it refuses those that 128x128 tiles at 0.72 us a
// slice would finish first.
static Plan plan_probe(const GemmDims& d, bool may_split) {
  static constexpr double slice_us[KIND_S64 + 1] = {kSliceUs[KIND_L64], kSliceUs[KIND_M64], 0.72};
  return plan_gemm(d, may_split, kEpiF32, KIND_S64 + 1, slice_us);
}

template <class Epi>
static hipError_t run_probe(const bf16_t* A, const bf16_t* B, const GemmDims& d, const Plan& p, Epi epi, hipStream_t st) {
  const dim3 grid(static_cast<unsigned>((p.items() + 7) / 8 * 8));
  const int ksteps = static_cast<int>(d.Kd / DBK64);
  if (p.kind == KIND_L64)
    hipLaunchKernelGGL((k_gemm_dma64<CfgL64, false, Epi>), grid, dim3(CfgL64::THREADS), 0, st, A, B, d, p.tiles_m, p.tiles_n, 1, ksteps, epi);
  else
    hipLaunchKernelGGL((k_gemm_dma64<CfgM64, false, Epi>), grid, dim3(CfgM64::THREADS), 0, st, A, B, d, p.tiles_m, p.tiles_n, 1, ksteps, epi);
  return hipGetLastError();
}

hipError_t launch_gemm_probe(int mode, const bf16_t* A, const bf16_t* B, GemmDims d, unsigned long long* clocks,
                             int64_t capacity, float* sink, int* kind, int64_t* items, hipStream_t st) {
  const Plan p = plan_probe(d, false);
  *kind = p.kind;
  *items = p.items();
  if (p.kind != KIND_L64 && p.kind != KIND_M64) return hipErrorNotSupported;
  if (p.items() > capacity) return hipErrorInvalidValue;
  if (mode & 4) {   // the same loops on token-major operands: the buffers are read as A [Kd, M], B [Kd, N]
    if (d.M % 8 != 0 || d.N % 8 != 0 || plan_probe(d, true).kind != KIND_L64) return hipErrorNotSupported;
    const GemmDims t{d.M, d.N, d.Kd, d.M, d.N};
    if (mode & 8) {   // ... on 192-wide tiles (whole loop only), whichever of the two shapes divides the product better
      if ((mode & 3) != 0) return hipErrorNotSupported;
      const bool a192 = ceil_div(d.M, 192) * (int64_t)ceil_div(d.N, 256) <= ceil_div(d.M, 256) * (int64_t)ceil_div(d.N, 192);
      *items = a192 ? ceil_div(d.M, 192) * (int64_t)ceil_div(d.N, 256) : ceil_div(d.M, 256) * (int64_t)ceil_div(d.N, 192);
      if (*items > capacity) return hipErrorInvalidValue;
      const EpiProbe<0> e{clocks, sink, 0, 0, 0.0f};
      return a192 ? run_tn<CfgT64A>(A, B, t, 1, e, st) : run_tn<CfgT64B>(A, B, t, 1, e, st);
    }
    if ((mode & 3) == 0) return run_tn<CfgT64>(A, B, t, 1, EpiProbe<0>{clocks, sink, 0, 0, 0.0f}, st);
    if ((mode & 3) == 1) return run_tn<CfgT64>(A, B, t, 1, EpiProbe<1>{clocks, sink, 0, 0, 0.0f}, st);
    return run_tn<CfgT64>(A, B, t, 1, EpiProbe<2>{clocks, sink, 0, 0, 0.0f}, st);
  }
  if (mode & 8) return hipErrorNotSupported;
  if (mode == 0) return run_probe(A, B, d, p, EpiProbe<0>{clocks, sink, 0, 0, 0.0f}, st);
  if (mode == 1) return run_probe(A, B, d, p, EpiProbe<1>{clocks, sink, 0, 0, 0.0f}, st);
  return run_probe(A, B, d, p, EpiProbe<2>{clocks, sink, 0, 0, 0.0f}, st);
}

hipError_t launch_gemm_sub(const bf16_t* A, const bf16_t* B, GemmDims d, const void* Y, bool y_bf16,
                           bool first, float* C_out, const float* x_scale, hipStream_t st) {
  const Plan p = plan_gemm(d, false, kEpiSub);
  if (y_bf16) {
    EpiSub<true> e{Y, first, C_out, x_scale, 1.0f};
    return run(A, B, d, p, e, st);
  }
  EpiSub<false> e{Y, first, C_out, x_scale, 1.0f};
  return run(A, B, d, p, e, st);
}

hipError_t launch_gemm_bf16_nn(const bf16_t* A, const bf16_t* B, GemmDims d, bf16_t* out, hipStream_t st) {
  if (d.N % 8 != 0 || d.Kd % 8 != 0 || d.lda % 8 != 0 || d.ldb % 8 != 0) return hipErrorInvalidValue;
  EpiBf16 e{out, nullptr, 1.0f};
  return run<true>(A, B, d, plan_gemm(d, false, kEpiBf16), e, st);
}

bool gemm_bf16_walks(const GemmDims& d) { return walks_rounds(d, plan_gemm(d, false, kEpiBf16)); }

hipError_t launch_gemm_bf16(const bf16_t* A, const bf16_t* B, GemmDims d, bf16_t* out, const float* scale, hipStream_t st) {
  EpiBf16 e{out, scale, 1.0f};
  const Plan p = plan_gemm(d, false, kEpiBf16);
  return walks_rounds(d, p) ? run_rounds(A, B, d, p, e, st) : run(A, B, d, p, e, st);
}

}  // namespace faar
