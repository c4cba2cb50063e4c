// The attention core between the q / k / v and the output projections of a block, for a Stage-2-style joint step (paper
// Sec. 3.5 "Stage 2"; Table 2 steps 15-17 and 23: the quantised model runs forward and one loss is back-propagated into
// every layer's rounding variables).  The operations are those of the Llama3 / Qwen3 blocks the paper evaluates: rotary
// position embedding ("rotate-half" form) and causal softmax attention with grouped key / value heads, forward and
// backward.  Activations and gradients are bf16 between kernels, arithmetic is float32, products run on the matrix
// cores (v_mfma_f32_32x32x16_bf16) with the probabilities and their gradients rounded to bf16 as operands.
//
// Layouts.  q, o, dO, dq: [T, n_q * dh]; k, v, dk, dv: [T, n_kv * dh]; T = n_seq * S tokens, sequence b = rows b*S ..
// (b+1)*S-1, S a multiple of 32; query head j reads key / value head j / (n_q / n_kv).
//
// A workgroup of four wavefronts owns 128 query positions (forward, dq) or 128 key positions (dk, dv) of one head and
// sequence, 32 per wavefront, and walks the causal range in blocks of 64 tokens whose tiles it shares through LDS (Tile
// below).  Products run as v_mfma_f32_32x32x16_bf16:
//   * a product whose contraction runs over dh takes rows of a tile as they lie there (16-byte LDS reads);
//   * a product whose contraction runs over tokens (P V, dS K, P^T dO, dS^T Q) takes COLUMNS of the same tile through the LDS
//     transposing reads of this architecture (ds_read_b64_tr_b16): no transposed copy exists anywhere;
//   * the probabilities enter those products in the accumulator layout they were computed in: of a 32x32 accumulator tile a
//     lane holds, for its column, rows 8 j + 4 (lane / 32) + 0..3 (j = 0..3) -- registers 8 t .. 8 t + 7 are the 8 contraction
//     values it must supply for 16-token step t, with the contraction index permuted, which the transposing reads follow.
// What bounds these kernels: the vector unit as much as the matrix cores (an exponential costs four issue slots, the rest of
// the softmax as many again: about one VALU cycle per matrix cycle), so the aim is to keep both busy: two independent
// workgroups per compute unit (256 registers a lane, 64 KB of LDS each; with heads of 64 three or four), one barrier per 64 tokens, the softmax reductions
// inside a lane but for one exchange between the two halves of the wavefront.
//
// Measured, forward and backward in us (calls back to back, the former kernels' transposes included), against 16x16x32 products on
// transposed copies with 32-token blocks, whose dk / dv kernel held one workgroup per compute unit: 2 sequences of 4096 tokens,
// 16 / 8 heads of 128: 341 and 1424 -> 146 and 476; of 64: 194 and 642 -> 84 and 269; 32 sequences of 512, heads of 128: 120 and
// 551 -> 68 and 228.  By kernel, forward / dq / dk + dv: 2 x 4096, heads of 128: 168 / 217 / 319.
#include <algorithm>

#include "faar_internal.h"

namespace faar {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
constexpr int kTok = 64;       // tokens per LDS tile

union Frag {
  bf16x8 v;
  uint4 q;
  uint32_t w[4];
};

__device__ __forceinline__ bf16x8 load_frag16(const bf16_t* p) {   // 8 consecutive bf16
  Frag f;
  f.q = *reinterpret_cast<const uint4*>(p);
  return f.v;
}
// accumulator registers 8 t .. 8 t + 7 of a tile -> the second operand of a 16-token step
template <int T>
__device__ __forceinline__ bf16x8 pack8(const f32x16& a) {
  Frag f;
#pragma unroll
  for (int i = 0; i < 4; ++i) f.w[i] = pack_bf16x2(a[8 * T + 2 * i], a[8 * T + 2 * i + 1]);
  return f.v;
}
__device__ __forceinline__ f32x16 mfma(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.0f;
  return z;
}
// the values of lane i and lane i ^ 32, in either order (v_permlane32_swap: a vector instruction, no LDS round trip)
__device__ __forceinline__ void both_halves(float x, float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
__device__ __forceinline__ float half_max(float x) {
  float a, b;
  both_halves(x, a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float half_sum(float x) {
  float a, b;
  both_halves(x, a, b);
  return a + b;
}
__device__ __forceinline__ void store4_bf16(bf16_t* p, float a, float b, float c, float d) {
  *reinterpret_cast<uint2*>(p) = make_uint2(pack_bf16x2(a, b), pack_bf16x2(c, d));
}

struct AttnDims {
  int S, n_q, n_kv;
  int64_t T;          // tokens
  float scale;        // of the scores (1 / sqrt(dh) for the models here)
};

// 2^x by the hardware instruction alone: the arguments here are at most a few units above zero and results far below one
// may flush to zero
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// 16 bytes (4 in the second form) per lane from global memory straight into LDS at lds_addr + 16 * lane (4 * lane), lds_addr
// wave-uniform.  Inline assembly: the compiler does not see the LDS write, so completion is tracked by hand (wait_vmcnt, then
// the workgroup barrier); its own wait counts for ordinary loads stay sufficient, since memory operations return in order.
__device__ __forceinline__ void dma16(const void* base, uint32_t lane_offset, uint32_t lds_addr) {   // base wave-uniform
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(lane_offset), "s"(base)
               : "memory", "m0");
}
__device__ __forceinline__ void dma4(const void* gptr, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_addr), "v"(gptr) : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_addr_of(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const char*)p));
}
#define FAAR_WAIT_VMCNT(N) __builtin_amdgcn_s_waitcnt(0x0F70 | ((N)&0xF) | (((N) >> 4) << 14))

// A [64 tokens][dh] tile of a token-major tensor in LDS, rows un-padded.  The 16-byte chunks of a row are stored XOR-permuted
// by a key of the row so that both kinds of read spread over the 64 banks: the 16 rows of a 16-byte row read fall on 16
// distinct chunk positions, and the 16 32-byte segments of a transposing read (8 tokens x 2 groups of 16 columns) on the 8 bank
// groups twice each.  dh = 128: a row is one turn of the banks, key = row bits 0..2 on chunk bits 1..3 (which 32-byte pair)
// and row bit 3 on chunk bit 0; dh = 64: two rows to a turn, key = row bits 1, 2 on chunk bits 1, 2 and row bit 3 on bit 0.
template <int DH>
struct Tile {
  static constexpr int CPR = DH / 8;                  // 16-byte chunks per row
  static constexpr int COPIES = kTok * CPR / 256;     // copies per thread
  static constexpr int ELEMS = kTok * DH;

  static __device__ __forceinline__ int key(int row) {
    return (DH == 128 ? 2 * (row & 7) : 2 * ((row >> 1) & 3)) | ((row >> 3) & 1);
  }
  // rows row0 .. row0+63, columns col0 .. col0+dh-1, global -> LDS without passing through registers: chunk i = tid + 256 j of
  // the tile lands at byte 16 i.  A pass of the workgroup covers 2048 / dh rows, a divisor of 32, and starts at a row whose key
  // is 0, so one lane offset (of_lane) serves every pass.  `valid` rows are there (32, or 64 and more): the passes beyond them
  // repeat the first one, and callers mask what comes of those rows.
  static __device__ __forceinline__ uint32_t of_lane(int64_t ld, int tid) {
    const int row = tid / CPR;
    return static_cast<uint32_t>(row * ld * 2) + ((tid % CPR) ^ key(row)) * 16;
  }
  static __device__ __forceinline__ void copy(const bf16_t* __restrict__ src, int64_t row0, int valid, int64_t ld, int64_t col0,
                                              uint32_t lane_offset, uint32_t tile, int wave) {
#pragma unroll
    for (int j = 0; j < COPIES; ++j) {
      const int row = j * (256 / CPR);
      dma16(src + (row0 + (row < valid ? row : 0)) * ld + col0, lane_offset,
            __builtin_amdgcn_readfirstlane(tile + 4096u * j + 1024u * wave));
    }
  }
  // LDS byte addresses of a lane's reads: everything but the compile-time parts, which are added, or XORed into the chunk bits
  // (a row is a power of two long: the bits above it never change).  rows: row lane % 32, the 8 values at 8 (lane / 32).  cols:
  // within 16 lanes, lane r supplies the address of 4 columns of one token and receives one column of 4 tokens; the tokens come
  // in the order a lane holds them in an accumulator tile: 4 (lane / 32) + 0..3, then 8 further on (chunk bit 0 flips, key).
  static __device__ __forceinline__ uint32_t rows_at(int lane) {
    return (lane & 31) * (DH * 2) + ((lane >> 5) ^ key(lane & 31)) * 16;
  }
  static __device__ __forceinline__ uint32_t cols_at(int lane) {
    const int r = lane & 15, row = 4 * (lane >> 5) + (r >> 2);   // token of a 16-token step
    return row * (DH * 2) + ((2 * ((lane >> 4) & 1) + ((r & 3) >> 1)) ^ key(row)) * 16 + (r & 1) * 8;
  }
  // rows 32 half .. +31 x 16 of dh (step ks) of the tile whose LDS address is already in `at` (an aligned tile: a plain sum, but
  // the compiler does not know; formed per step and made opaque, it leaves the constant parts to the instruction's offset field)
  static __device__ __forceinline__ bf16x8 rows(uint32_t at, int half, int ks) {
    typedef __attribute__((address_space(3))) const bf16x8* ptr;
    uint32_t x = at ^ (32u * ks);
    asm("" : "+v"(x));
    return *reinterpret_cast<ptr>(x + half * (32 * DH * 2));
  }
  // dh rows 32 dt .. +31 x 16 tokens (step st of the 32 tokens `half`)
  static __device__ __forceinline__ bf16x8 cols(uint32_t at, int half, int st, int dt) {
    typedef __attribute__((address_space(3))) s16x4* ptr;
    uint32_t x = at ^ (64u * dt), y = at ^ (64u * dt + 16u);
    asm("" : "+v"(x), "+v"(y));
    const uint32_t off = (half * 32 + st * 16) * (DH * 2);
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<ptr>(x + off));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<ptr>(y + off + 8 * (DH * 2)));
    const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
  }
};

// Workgroup -> (group of 128 positions by rank, head and sequence).  Workgroups take the heavy groups first, so that the light
// ones fill the tail; those of the second round of 256 -- the second resident workgroup of every compute unit -- run from
// light to heavy, so that a unit's two residents add up to about the same work everywhere.  The head / sequence index varies
// fastest and by key / value head first, so that (where their number is a multiple of 8) an XCD sees the same few of them.
// Without the turn of the second round the forward takes 146 -> 150 us (2 x 4096 tokens, 16 / 8 heads of 128) and 172 -> 179
// (1 x 8192, 8 / 1 heads).  Heads of 64 leave room for three or four residents, and the same rule serves them: 83 -> 86 (2 x 4096)
// and 157 -> 165 (1 x 8192, 16 / 8 heads) without it, while turning every other round of four is within 2 % either way.
__device__ __forceinline__ void work_item(int id, int pairs, int ranks, int& rank, int& pair) {
  rank = id / pairs;
  pair = id - rank * pairs;
  const int r0 = (256 + pairs - 1) / pairs, r1 = min(ranks, 512 / pairs) - 1;
  if (rank >= r0 && rank <= r1) rank = r0 + r1 - rank;
}

// o = softmax(q k^T scale, causal) v and lse = log sum exp of the scaled scores per query ([n_q][T]).
// The running maximum of a query's scores is only raised when a block exceeds it by more than 2^kLazy (the probabilities are
// then at most 2^kLazy instead of 1, harmless in float32 and bf16): the accumulators are rescaled in a branch that is
// rarely taken after the first blocks, and otherwise only matrix instructions touch them.
constexpr float kLazy = 8.0f;

template <int DH>
struct FwdState {
  bf16x8 qf[DH / 16];
  f32x16 oacc[DH / 32];   // rows = dh, column = query lane % 32
  float mc, l;            // reference maximum (score units of log 2), and this half-wave's share of the denominator
};

// kMode 0: 64 keys before the wavefront's queries; 1: the queries' own 32 positions (first half of the block) only; 2: 32
// earlier keys and the own positions
template <int DH, int kMode>
__device__ __forceinline__ void fwd_block(FwdState<DH>& st, uint32_t k_lds, uint32_t v_lds, uint32_t ra, uint32_t ca, float c, int lane) {
  constexpr int KS = DH / 16, DT = DH / 32, NT = kMode == 1 ? 1 : 2;
  typedef Tile<DH> Tl;
  f32x16 s[NT];            // rows = keys, column = query
#pragma unroll
  for (int kt = 0; kt < NT; ++kt) s[kt] = zero16();
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int kt = 0; kt < NT; ++kt) s[kt] = mfma(Tl::rows(k_lds + ra, kt, ks), st.qf[ks], s[kt]);
  if (kMode != 0) {
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if (8 * (v / 4) + 4 * (lane >> 5) + v % 4 > (lane & 31)) s[NT - 1][v] = -INFINITY;   // a key after the query
  }
  float mx = s[0][0];
#pragma unroll
  for (int kt = 0; kt < NT; ++kt)
#pragma unroll
    for (int v = 0; v < 16; ++v) mx = fmaxf(mx, s[kt][v]);
  mx = half_max(mx) * c;   // finite: a query's own position is never masked, and key 0 comes first
  if (__any(mx > st.mc + kLazy)) {
    const float nm = fmaxf(st.mc, mx);
    const float alpha = fast_exp2(st.mc - nm);
    st.mc = nm;
    st.l *= alpha;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) st.oacc[dt] *= alpha;
  }
  float ps = 0.0f;
#pragma unroll
  for (int kt = 0; kt < NT; ++kt)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float p = fast_exp2(fmaf(s[kt][v], c, -st.mc));
      s[kt][v] = p;
      ps += p;
    }
  st.l += ps;              // this half-wave's keys only; the two halves add up at the end
#pragma unroll
  for (int kt = 0; kt < NT; ++kt) {
    const bf16x8 p0 = pack8<0>(s[kt]), p1 = pack8<1>(s[kt]);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) st.oacc[dt] = mfma(Tl::cols(v_lds + ca, kt, 0, dt), p0, st.oacc[dt]);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) st.oacc[dt] = mfma(Tl::cols(v_lds + ca, kt, 1, dt), p1, st.oacc[dt]);
  }
}

template <int DH>
__global__ void __launch_bounds__(256, 2)
k_attn_fwd(const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V, AttnDims d,
           bf16_t* __restrict__ O, float* __restrict__ lse) {
  constexpr int KS = DH / 16, DT = DH / 32;
  typedef Tile<DH> Tl;
  __shared__ __attribute__((aligned(1024))) bf16_t lds[2][2][Tl::ELEMS];   // [stage][k, v]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = lane & 31, hi = lane >> 5;
  const int blocks = d.S / 32, groups = (blocks + 3) / 4, rep = d.n_q / d.n_kv;
  const int pairs = static_cast<int>(gridDim.x) / groups, kv_pairs = pairs / rep;
  int rank, pair;
  work_item(blockIdx.x, pairs, groups, rank, pair);
  const int grp = groups - 1 - rank;               // the last positions see the most keys
  const int kvh = (pair % kv_pairs) % d.n_kv, head = kvh * rep + pair / kv_pairs;
  const int64_t b = (pair % kv_pairs) / d.n_kv;
  const int64_t t0 = b * d.S, ldq = (int64_t)d.n_q * DH, ldk = (int64_t)d.n_kv * DH;
  const int qb = grp * 4 + wave;                   // this wavefront's block of 32 positions
  const bool active = qb < blocks;                 // the last group of a sequence may be short
  const int last = min(grp * 4 + 3, blocks - 1) / 2;   // last 64-key block any wavefront of the group needs
  const int p0 = qb * 32;
  const float c = d.scale * kLog2e;     // scores in units of log 2

  FwdState<DH> st;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    st.qf[ks] = active ? load_frag16(Q + (t0 + p0 + n) * ldq + head * DH + ks * 16 + 8 * hi) : bf16x8{};
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) st.oacc[dt] = zero16();
  st.mc = -INFINITY;
  st.l = 0.0f;
  // Two LDS stages: a block's tiles are requested one block ahead, by copies that bypass the registers
  const int64_t kvcol = (int64_t)kvh * DH;
#define FAAR_FWD_COPY(KB)                                                                                             \
  do {                                                                                                                \
    const uint32_t at_ = lds0 + ((KB) & 1) * (2 * Tl::ELEMS * 2);                                                     \
    Tl::copy(K, t0 + (KB) * kTok, d.S - (KB) * kTok, ldk, kvcol, from, at_, wave);                                    \
    Tl::copy(V, t0 + (KB) * kTok, d.S - (KB) * kTok, ldk, kvcol, from, at_ + Tl::ELEMS * 2, wave);                    \
  } while (0)
  const uint32_t lds0 = lds_addr_of(lds), ra = Tl::rows_at(lane), ca = Tl::cols_at(lane), from = Tl::of_lane(ldk, tid);
  FAAR_FWD_COPY(0);
  for (int kb = 0; kb <= last; ++kb) {
    FAAR_WAIT_VMCNT(0);                            // block kb has landed (mine); the barrier: everybody's, and nobody reads
    __syncthreads();                               // the other stage any more
    if (kb < last) FAAR_FWD_COPY(kb + 1);
    const uint32_t k_lds = lds0 + (kb & 1) * (2 * Tl::ELEMS * 2), v_lds = k_lds + Tl::ELEMS * 2;
    if (active) {
      if (kb < qb / 2) fwd_block<DH, 0>(st, k_lds, v_lds, ra, ca, c, lane);
      else if (kb == qb / 2) {
        if (qb & 1) fwd_block<DH, 2>(st, k_lds, v_lds, ra, ca, c, lane);
        else fwd_block<DH, 1>(st, k_lds, v_lds, ra, ca, c, lane);
      }
    }
  }
#undef FAAR_FWD_COPY
  if (!active) return;
  const float lt = half_sum(st.l);
  const float inv = 1.0f / lt;
  const int64_t t = t0 + p0 + n;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      store4_bf16(O + t * ldq + head * DH + dt * 32 + 8 * j + 4 * hi, st.oacc[dt][4 * j] * inv, st.oacc[dt][4 * j + 1] * inv,
                  st.oacc[dt][4 * j + 2] * inv, st.oacc[dt][4 * j + 3] * inv);
  if (hi == 0) lse[(int64_t)head * d.T + t] = st.mc * kLn2 + logf(lt);
}

// dq = scale * dS k with dS = P * (dP - delta), P = exp(scores - lse), dP = dO v^T.  Workgroups and wavefronts as in the
// forward kernel.  delta[head][t] = sum_d dO[t][head, d] * O[t][head, d] (= sum_k P dP of that query: the softmax Jacobian's
// second term) is formed here, where dO is in registers anyway, and left for the dk / dv kernel.
template <int DH, int kMode>
__device__ __forceinline__ void dq_block(f32x16 (&acc)[DH / 32], const bf16x8 (&qf)[DH / 16], const bf16x8 (&dof)[DH / 16],
                                         float lse2, float dl, uint32_t k_lds, uint32_t v_lds, uint32_t ra, uint32_t ca, float c,
                                         int lane) {
  constexpr int KS = DH / 16, DT = DH / 32, NT = kMode == 1 ? 1 : 2;
  typedef Tile<DH> Tl;
#pragma unroll
  for (int kt = 0; kt < NT; ++kt) {
    f32x16 s = zero16(), dp = zero16();    // rows = keys, column = query
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      s = mfma(Tl::rows(k_lds + ra, kt, ks), qf[ks], s);
      dp = mfma(Tl::rows(v_lds + ra, kt, ks), dof[ks], dp);
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      float p = fast_exp2(fmaf(s[v], c, -lse2));
      if (kMode != 0 && kt == NT - 1 && 8 * (v / 4) + 4 * (lane >> 5) + v % 4 > (lane & 31)) p = 0.0f;   // a key after the query
      dp[v] = p * (dp[v] - dl);
    }
    const bf16x8 d0 = pack8<0>(dp), d1 = pack8<1>(dp);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[dt] = mfma(Tl::cols(k_lds + ca, kt, 0, dt), d0, acc[dt]);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) acc[dt] = mfma(Tl::cols(k_lds + ca, kt, 1, dt), d1, acc[dt]);
  }
}

template <int DH>
__global__ void __launch_bounds__(256, 2)
k_attn_bwd_dq(const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
              const bf16_t* __restrict__ dO, const bf16_t* __restrict__ O, const float* __restrict__ lse,
              float* __restrict__ delta, AttnDims d, bf16_t* __restrict__ dQ) {
  constexpr int KS = DH / 16, DT = DH / 32;
  typedef Tile<DH> Tl;
  __shared__ __attribute__((aligned(1024))) bf16_t lds[2][2][Tl::ELEMS];   // [stage][k, v]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = lane & 31, hi = lane >> 5;
  const int blocks = d.S / 32, groups = (blocks + 3) / 4, rep = d.n_q / d.n_kv;
  const int pairs = static_cast<int>(gridDim.x) / groups, kv_pairs = pairs / rep;
  int rank, pair;
  work_item(blockIdx.x, pairs, groups, rank, pair);
  const int grp = groups - 1 - rank;
  const int kvh = (pair % kv_pairs) % d.n_kv, head = kvh * rep + pair / kv_pairs;
  const int64_t b = (pair % kv_pairs) / d.n_kv;
  const int64_t t0 = b * d.S, ldq = (int64_t)d.n_q * DH, ldk = (int64_t)d.n_kv * DH;
  const int qb = grp * 4 + wave;
  const bool active = qb < blocks;
  const int last = min(grp * 4 + 3, blocks - 1) / 2;
  const int64_t t = t0 + qb * 32 + n;
  const float c = d.scale * kLog2e;

  bf16x8 qf[KS], dof[KS];
  float lse2 = 0.0f, dl = 0.0f;
  f32x16 acc[DT];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int64_t at = t * ldq + head * DH + ks * 16 + 8 * hi;
    qf[ks] = active ? load_frag16(Q + at) : bf16x8{};
    dof[ks] = active ? load_frag16(dO + at) : bf16x8{};
    const bf16x8 of = active ? load_frag16(O + at) : bf16x8{};
#pragma unroll
    for (int j = 0; j < 8; ++j) dl += static_cast<float>(dof[ks][j]) * static_cast<float>(of[j]);
  }
  dl = half_sum(dl);
  if (active) {
    lse2 = lse[(int64_t)head * d.T + t] * kLog2e;
    if (hi == 0) delta[(int64_t)head * d.T + t] = dl;
  }
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) acc[dt] = zero16();
  const int64_t kvcol = (int64_t)kvh * DH;
#define FAAR_DQ_COPY(KB)                                                                                             \
  do {                                                                                                                \
    const uint32_t at_ = lds0 + ((KB) & 1) * (2 * Tl::ELEMS * 2);                                                     \
    Tl::copy(K, t0 + (KB) * kTok, d.S - (KB) * kTok, ldk, kvcol, from, at_, wave);                                    \
    Tl::copy(V, t0 + (KB) * kTok, d.S - (KB) * kTok, ldk, kvcol, from, at_ + Tl::ELEMS * 2, wave);                    \
  } while (0)
  const uint32_t lds0 = lds_addr_of(lds), ra = Tl::rows_at(lane), ca = Tl::cols_at(lane), from = Tl::of_lane(ldk, tid);
  FAAR_DQ_COPY(0);
  for (int kb = 0; kb <= last; ++kb) {
    FAAR_WAIT_VMCNT(0);
    __syncthreads();
    if (kb < last) FAAR_DQ_COPY(kb + 1);
    const uint32_t k_lds = lds0 + (kb & 1) * (2 * Tl::ELEMS * 2), v_lds = k_lds + Tl::ELEMS * 2;
    if (active) {
      if (kb < qb / 2) dq_block<DH, 0>(acc, qf, dof, lse2, dl, k_lds, v_lds, ra, ca, c, lane);
      else if (kb == qb / 2) {
        if (qb & 1) dq_block<DH, 2>(acc, qf, dof, lse2, dl, k_lds, v_lds, ra, ca, c, lane);
        else dq_block<DH, 1>(acc, qf, dof, lse2, dl, k_lds, v_lds, ra, ca, c, lane);
      }
    }
  }
#undef FAAR_DQ_COPY
  if (!active) return;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      store4_bf16(dQ + t * ldq + head * DH + dt * 32 + 8 * j + 4 * hi, acc[dt][4 * j] * d.scale, acc[dt][4 * j + 1] * d.scale,
                  acc[dt][4 * j + 2] * d.scale, acc[dt][4 * j + 3] * d.scale);
}

// dv = P^T dO and dk = scale * dS^T q, summed over the query heads that share the key / value head.  A workgroup owns
// 128 / QW key positions of a key / value head and sequence (32 per wavefront; with QW = 2 the other two wavefronts take the
// second 32 queries of every block for the same keys, and the two sums meet through LDS at the end) and walks the blocks of
// 64 queries at or after them, for each query head of the group in turn; the block's lse and delta go through LDS beside its
// tiles.
template <int DH>
__device__ __forceinline__ void dkv_tile(f32x16 (&dk)[DH / 32], f32x16 (&dv)[DH / 32], const bf16x8 (&kf)[DH / 16],
                                         const bf16x8 (&vf)[DH / 16], const float* lse_lds, const float* delta_lds,
                                         uint32_t q_rows, uint32_t q_cols, float c, bool diagonal, int lane) {
  constexpr int KS = DH / 16, DT = DH / 32;
  constexpr uint32_t kDo = Tile<DH>::ELEMS * 2;     // the dO tile follows the q tile
  typedef Tile<DH> Tl;
  // 128 accumulators and 64 operand registers are resident, so the operands read from LDS pass through a ring of kRing, each
  // requested kRing - 1 matrix instructions ahead, and scheduling barriers keep the compiler from requesting more
  constexpr int kRing = 3;
  bf16x8 f[kRing];
  f32x16 s = zero16(), dp = zero16();      // rows = queries, column = key
  auto fetch_rows = [&](int i) { f[i % kRing] = Tl::rows(q_rows + (i & 1) * kDo, 0, i / 2); };
#pragma unroll
  for (int i = 0; i < kRing - 1; ++i) fetch_rows(i);
#pragma unroll
  for (int i = 0; i < 2 * KS; ++i) {
    if (i + kRing - 1 < 2 * KS) fetch_rows(i + kRing - 1);
    if (i % 2 == 0) s = mfma(f[i % kRing], kf[i / 2], s);
    else dp = mfma(f[i % kRing], vf[i / 2], dp);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (diagonal) {
#pragma unroll
    for (int v = 0; v < 16; ++v)
      if ((lane & 31) > 8 * (v / 4) + 4 * (lane >> 5) + v % 4) s[v] = -INFINITY;   // the key comes after the query
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = 8 * j + 4 * (lane >> 5);
    const float4 l4 = *reinterpret_cast<const float4*>(lse_lds + row);
    const float4 d4 = *reinterpret_cast<const float4*>(delta_lds + row);
    const float lr[4] = {l4.x, l4.y, l4.z, l4.w}, dr[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float p = fast_exp2(fmaf(s[4 * j + r], c, -lr[r] * kLog2e));
      s[4 * j + r] = p;
      dp[4 * j + r] = p * (dp[4 * j + r] - dr[r]);
    }
    if (j == 1) __builtin_amdgcn_sched_barrier(0);
  }
  const bf16x8 pf[2] = {pack8<0>(s), pack8<1>(s)}, df[2] = {pack8<0>(dp), pack8<1>(dp)};
  __builtin_amdgcn_sched_barrier(0);
  // i = 4 dt + 2 (0: dv, 1: dk) + step would make an accumulator's two instructions neighbours; dv and dk alternate instead
  auto fetch_cols = [&](int i) { f[i % kRing] = Tl::cols(q_cols + (i & 1 ? 0u : kDo), 0, (i / 2) & 1, i / 4); };
#pragma unroll
  for (int i = 0; i < kRing - 1; ++i) fetch_cols(i);
#pragma unroll
  for (int i = 0; i < 4 * DT; ++i) {
    if (i + kRing - 1 < 4 * DT) fetch_cols(i + kRing - 1);
    if (i % 2 == 0) dv[i / 4] = mfma(f[i % kRing], pf[(i / 2) & 1], dv[i / 4]);
    else dk[i / 4] = mfma(f[i % kRing], df[(i / 2) & 1], dk[i / 4]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <int DH, int QW>
__global__ void __launch_bounds__(256, 2)
k_attn_bwd_dkv(const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
               const bf16_t* __restrict__ dO, const float* __restrict__ lse, const float* __restrict__ delta, AttnDims d,
               bf16_t* __restrict__ dK, bf16_t* __restrict__ dV) {
  constexpr int KS = DH / 16, DT = DH / 32, KW = 4 / QW;   // KW: blocks of 32 keys
  typedef Tile<DH> Tl;
  __shared__ __attribute__((aligned(1024))) bf16_t lds[2][2][Tl::ELEMS];   // [stage][q, dO]
  __shared__ __attribute__((aligned(16))) float stats[2][2][kTok];         // [stage][lse, delta]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = lane & 31, hi = lane >> 5;
  const int kw = wave % KW, qw = wave / KW;
  const int blocks = d.S / 32, groups = (blocks + KW - 1) / KW;
  const int pairs = static_cast<int>(gridDim.x) / groups;
  int grp, pair;
  work_item(blockIdx.x, pairs, groups, grp, pair);   // the first positions are seen by the most queries
  const int kvh = pair % d.n_kv;
  const int64_t b = pair / d.n_kv;
  const int rep = d.n_q / d.n_kv;
  const int64_t t0 = b * d.S, ldq = (int64_t)d.n_q * DH, ldk = (int64_t)d.n_kv * DH;
  const int kb = grp * KW + kw;                 // this wavefront's block of 32 positions
  const bool active = kb < blocks;
  const int64_t t = t0 + kb * 32 + n;
  const float c = d.scale * kLog2e;

  bf16x8 kf[KS], vf[KS];     // second operands: column = key
  f32x16 dk[DT], dv[DT];     // rows = dh, column = key
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int64_t at = t * ldk + kvh * DH + ks * 16 + 8 * hi;
    kf[ks] = active ? load_frag16(K + at) : bf16x8{};
    vf[ks] = active ? load_frag16(V + at) : bf16x8{};
  }
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    dk[dt] = zero16();
    dv[dt] = zero16();
  }
  // steps: query head of the group (outer) x 64-query block first .. last (inner); groups of 128 and of 64 positions start on such a block
  const int first = grp * KW / 2, n_blk = (blocks + 1) / 2, steps = rep * (n_blk - first);
#define FAAR_DKV_COPY(STAGE, HEAD, BLK)                                                                  \
  do {                                                                                                  \
    const int q0_ = (BLK) * kTok;                                                                       \
    const uint32_t at_ = lds0 + (STAGE) * (2 * Tl::ELEMS * 2);                                          \
    Tl::copy(Q, t0 + q0_, d.S - q0_, ldq, (int64_t)(HEAD) * DH, from, at_, wave);                       \
    Tl::copy(dO, t0 + q0_, d.S - q0_, ldq, (int64_t)(HEAD) * DH, from, at_ + Tl::ELEMS * 2, wave);      \
    if (wave < 2)                                                                                       \
      dma4((wave == 0 ? lse : delta) + (int64_t)(HEAD) * d.T + t0 + min(q0_ + lane, d.S - 1),           \
           __builtin_amdgcn_readfirstlane(lds_addr_of(stats[STAGE][wave])));                            \
  } while (0)
  const uint32_t lds0 = lds_addr_of(lds), from = Tl::of_lane(ldq, tid);
  const uint32_t ra = Tl::rows_at(lane), ca = Tl::cols_at(lane);
  int head = kvh * rep, blk = first;
  FAAR_DKV_COPY(0, head, blk);
  for (int it = 0; it < steps; ++it) {
    FAAR_WAIT_VMCNT(0);
    __syncthreads();
    const int qb0 = 2 * blk;
    if (++blk == n_blk) {
      blk = first;
      ++head;
    }
    if (it + 1 < steps) FAAR_DKV_COPY((it + 1) & 1, head, blk);
    const uint32_t q_lds = lds0 + (it & 1) * (2 * Tl::ELEMS * 2);
    const float *lse_lds = stats[it & 1][0], *delta_lds = stats[it & 1][1];
#pragma unroll 1
    for (int qt = qw; qt < 2; qt += QW) {
      const int qb = qb0 + qt;               // block of 32 queries
      if (!active || qb < kb || qb >= blocks) continue;
      const uint32_t tile = q_lds + qt * (32 * DH * 2);
      dkv_tile<DH>(dk, dv, kf, vf, lse_lds + qt * 32, delta_lds + qt * 32, tile + ra, tile + ca, c, qb == kb, lane);
    }
  }
#undef FAAR_DKV_COPY
  if constexpr (QW == 2) {
    // the two wavefronts of a block of keys: one hands over its dv and finishes dk, the other the reverse
    f32x16* give = reinterpret_cast<f32x16*>(lds) + (size_t)wave * DT * 64 + lane;
    const f32x16* take = reinterpret_cast<const f32x16*>(lds) + (size_t)(wave ^ KW) * DT * 64 + lane;
    static_assert(4 * DT * 64 * sizeof(f32x16) <= sizeof(lds), "exchange fits in the stages");
    __syncthreads();
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) give[dt * 64] = qw == 0 ? dv[dt] : dk[dt];
    __syncthreads();
    if (!active) return;
    const float k = qw == 0 ? d.scale : 1.0f;
    bf16_t* out = qw == 0 ? dK : dV;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const f32x16 r = (qw == 0 ? dk[dt] : dv[dt]) + take[dt * 64];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        store4_bf16(out + t * ldk + kvh * DH + dt * 32 + 8 * j + 4 * hi, r[4 * j] * k, r[4 * j + 1] * k, r[4 * j + 2] * k, r[4 * j + 3] * k);
    }
    return;
  }
  if (!active) return;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t at = t * ldk + kvh * DH + dt * 32 + 8 * j + 4 * hi;
      store4_bf16(dK + at, dk[dt][4 * j] * d.scale, dk[dt][4 * j + 1] * d.scale, dk[dt][4 * j + 2] * d.scale, dk[dt][4 * j + 3] * d.scale);
      store4_bf16(dV + at, dv[dt][4 * j], dv[dt][4 * j + 1], dv[dt][4 * j + 2], dv[dt][4 * j + 3]);
    }
}

// rotate-half rotary embedding of every head: pair (i, i + dh/2) by the angle whose cosine / sine are in the tables' row
// t % S; sign = -1 rotates back (the backward pass)
__global__ void __launch_bounds__(kEltThreads)
k_rope(const bf16_t* X, int64_t n_chunks, int H, int dh, const float* __restrict__ cos_t,
       const float* __restrict__ sin_t, int S, float sign, bf16_t* Y) {   // Y may be X: a thread reads what it overwrites first
  const int64_t i = blockIdx.x * (int64_t)kEltThreads + threadIdx.x;   // one 8-element chunk of a head's first half
  if (i >= n_chunks) return;
  const int cph = dh / 16;                       // chunks per half head
  const int ch = static_cast<int>(i % cph);
  const int64_t th = i / cph;                    // = t * H + head
  const int64_t t = th / H;
  const int64_t base = th * dh + ch * 8;
  const int64_t tab = (t % S) * (dh / 2) + ch * 8;
  float a[8], b[8], c[8], s[8], ya[8], yb[8];
  W8<bf16_t>::load(X + base, a);
  W8<bf16_t>::load(X + base + dh / 2, b);
  load8(cos_t + tab, c);
  load8(sin_t + tab, s);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float sj = sign * s[j];
    ya[j] = a[j] * c[j] - b[j] * sj;
    yb[j] = b[j] * c[j] + a[j] * sj;
  }
  W8<bf16_t>::store(Y + base, ya);
  W8<bf16_t>::store(Y + base + dh / 2, yb);
}

}  // namespace

hipError_t launch_rope(const bf16_t* X, int64_t T, int64_t H, int64_t dh, const float* cos_t, const float* sin_t, int64_t S,
                       bool inverse, bf16_t* Y, hipStream_t st) {
  const int64_t n_chunks = T * H * (dh / 16);
  hipLaunchKernelGGL(k_rope, dim3(static_cast<unsigned>((n_chunks + kEltThreads - 1) / kEltThreads)), dim3(kEltThreads), 0, st, X,
                     n_chunks, static_cast<int>(H), static_cast<int>(dh), cos_t, sin_t, static_cast<int>(S), inverse ? -1.0f : 1.0f, Y);
  return hipGetLastError();
}

hipError_t launch_attention_fwd(const bf16_t* Q, const bf16_t* K, const bf16_t* V, int64_t n_seq, int64_t S, int64_t n_q,
                                int64_t n_kv, int64_t dh, float scale, bf16_t* O, float* lse, hipStream_t st) {
  const AttnDims d{static_cast<int>(S), static_cast<int>(n_q), static_cast<int>(n_kv), n_seq * S, scale};
  const dim3 grid(static_cast<unsigned>(n_seq * n_q * ((S + 127) / 128)));    // 128 query positions of a head and sequence each
  if (dh == 128)
    hipLaunchKernelGGL(k_attn_fwd<128>, grid, dim3(256), 0, st, Q, K, V, d, O, lse);
  else
    hipLaunchKernelGGL(k_attn_fwd<64>, grid, dim3(256), 0, st, Q, K, V, d, O, lse);
  return hipGetLastError();
}

hipError_t launch_attention_bwd(const bf16_t* dO, const bf16_t* Q, const bf16_t* K, const bf16_t* V, const bf16_t* O,
                                const float* lse, float* delta, int64_t n_seq, int64_t S, int64_t n_q, int64_t n_kv, int64_t dh,
                                float scale, bf16_t* dQ, bf16_t* dK, bf16_t* dV, hipStream_t st) {
  const AttnDims d{static_cast<int>(S), static_cast<int>(n_q), static_cast<int>(n_kv), n_seq * S, scale};
  const int64_t groups = (S + 127) / 128;
  const dim3 gq(static_cast<unsigned>(n_seq * n_q * groups));
  // The work of a group of keys falls linearly with its position and two workgroups share a compute unit: with fewer than 1024
  // groups of 128 keys the first ones end the launch alone on their units (2 x 4096 tokens, 8 heads: 512 groups), and 64 keys
  // a workgroup halve the longest and leave twice as many to fill in behind them.  With more, the larger group's fewer
  // copies count.  dq + dk + dv in us on 128 / 64 keys, heads of 128: 64 groups (1 x 8192, one key / value head) 2430 / 1468,
  // 512 groups (2 x 4096) 508 / 462, 1024 (8 x 2048) 1003 / 1027; heads of 64, of which three share a unit: 64 groups 1624 / 978,
  // 512 (2 x 4096) 306 / 261, 1024 (4 x 4096) 478 / 491, 2048 (16 x 2048) 517 / 554.
  const bool halves = n_seq * n_kv * groups < 1024;
  const dim3 gk(static_cast<unsigned>(n_seq * n_kv * (halves ? (S + 63) / 64 : groups)));
#define FAAR_BWD(DH)                                                                                                          \
  do {                                                                                                                        \
    hipLaunchKernelGGL(k_attn_bwd_dq<DH>, gq, dim3(256), 0, st, Q, K, V, dO, O, lse, delta, d, dQ);                           \
    if (halves)                                                                                                               \
      hipLaunchKernelGGL((k_attn_bwd_dkv<DH, 2>), gk, dim3(256), 0, st, Q, K, V, dO, lse, delta, d, dK, dV);                  \
    else                                                                                                                      \
      hipLaunchKernelGGL((k_attn_bwd_dkv<DH, 1>), gk, dim3(256), 0, st, Q, K, V, dO, lse, delta, d, dK, dV);                  \
  } while (0)
  if (dh == 128) FAAR_BWD(128);
  else FAAR_BWD(64);
#undef FAAR_BWD
  return hipGetLastError();
}

}  // namespace faar
