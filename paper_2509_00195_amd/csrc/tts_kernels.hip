// HIP kernels (gfx950) for prefix-shared beam decode attention.
//
// attn_kernel: one workgroup (8 waves, two per SIMD) per compute unit walks a
// chain of work units (tts_work.h), each the query rows of whole beams for
// one KV head against a list of KV blocks (up to 128, in two windows of 64).
//  * Narrow units (up to 64 rows): every wave keeps the softmax state of two
//    row tiles (16 rows each) in registers and streams its own share of the
//    block pairs straight from HBM into registers; no LDS staging and no
//    barriers until the waves combine their states. Up to 32 rows all eight
//    waves split the pairs; more rows make two groups of waves, each with
//    the pairs of its rows.
//  * Wide units (a segment shared by many beams, up to 256 rows): each block
//    pair is loaded once, an eighth per wave, staged in LDS two pairs at a
//    time and read from there. Up to 128 rows, each half of the waves takes
//    one pair of every step for all rows; above, every wave takes every pair
//    for its own two row tiles.
// Two waves per SIMD, because a wave's step is a chain (scores, softmax,
// value product) that leaves the matrix cores and the vector units idle in
// turn: with four waves of up to three tiles a wide unit of 11 row tiles took
// 0.61 us per block, against 0.30 (7B 64-beam tree); fp8 units of 7 tiles
// 0.47 against 0.40 (long chain). At 256 registers per wave nothing may spill:
// scratch stores alone took 8 to 25 us per launch. Against four waves: long
// chain (fp8) 342 -> 285 us per call, paged 64-beam call 103 -> 92.5, 7B
// 64-beam tree 23.65 -> 22.5, straggler batch 87.5 -> 85.1, verification of
// four tokens 46.9 -> 42.5; balanced tree unchanged. Where tails stream the
// middle of a launch runs at the memory's rate (balanced tree: half of its
// 45 us at about 6 TB/s, 4.7 over the whole launch, the rest its start, its
// uneven end and the combines); wide units are bound by LDS reads and vector
// issue, small batches by the units' round trips and the second launch.
//
// Products on MFMA, two 16-token blocks ("a pair") at a time, per row tile:
//   S^T = K Q^T   : 2 x 4 v_mfma_f32_16x16x32_bf16 (M = 16 tokens, N = 16
//                   rows, K = 128 head dims)
//   O^T += V^T P^T: 8 x v_mfma_f32_16x16x32_bf16 (M = 16 dims, N = 16 rows,
//                   K = the pair's 32 tokens)
// The two S tiles of a pair take their 16 token rows in an interleaved
// order (tile t, row m -> token 8*(m/4) + 4*t + m%4), so after the first
// product every lane holds the scores of 8 consecutive tokens of one row,
// all in one block of the pair: exactly the B operand of the second
// product. Values are stored dim-major inside a block, so the matching A
// operand is one contiguous 16-byte read.
//
// Softmax without a running maximum: probabilities are exp2(s - m_ref) with
// a fixed reference m_ref = 0 (log2 units), so the hot loop has no
// cross-lane reductions, no accumulator rescaling and no data-dependent
// branches. Each lane tracks the largest score it has seen; if a row's
// maximum leaves [-kRefWindow, kRefWindow] (where exp2 could overflow the
// fp32 accumulators or underflow every weight), its pairs are computed again
// with m_ref = that row's exact maximum: per wave in narrow units (no
// barrier inside their loop), by the whole workgroup in wide units (whose
// loop holds barriers, so the decision is taken over all eight waves).
// Either way each row ends with a consistent (m_ref, l, o) triple; a state
// that saw no token (l = 0) carries m = -inf, so it never sets the maximum
// of a combine or a merge.
//
// Every unit writes one partial softmax state per row; merge_kernel
// combines each (beam, query head)'s states in a fixed order
// (deterministic, no float atomics).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <type_traits>

#include "tts_work.h"

namespace tts {

#ifdef TTS_PROFILE_UNITS
// Per-unit timestamps for tuning builds only (indexed by record): start,
// end of wave 0's block loop, end, the XCC / HW_ID registers, all waves
// done, next unit issued, combine area written. (bf16 and fp8 kernels only:
// with the marks in the fp32 kernels too, the compiler's AGPR-copy rewrite
// pass crashes on the VGPR-form build.)
constexpr int kProfSlots = 1 << 15;
__device__ uint64_t g_prof[kProfSlots][8];
#define TTS_PROF_MARK(k, i) \
  do { if (KV != kKvF32 && threadIdx.x == 0 && (i) < kProfSlots) g_prof[(i)][k] = wall_clock64(); } while (0)
#else
#define TTS_PROF_MARK(k, i) do {} while (0)
#endif

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kTok = 16;  // tokens per KV block
constexpr int kThreads = 64 * kUnitWaves;
constexpr int kWaves = kThreads / 64;
constexpr int kTiles = kMaxRows / 16;
constexpr int kWideTiles = kMaxWideRows / 16 / kWaves;  // row tiles per wave in a wide unit
constexpr int kStepPairs = 2;                           // block pairs a wide unit stages between two barriers
constexpr float kNegInf = -__builtin_inff();
constexpr float kInf = __builtin_inff();
constexpr float kRefWindow = 64.0f;  // |row max| (log2 units) handled with m_ref = 0

enum KvKind : int { kKvF32 = 0, kKvBf16 = 1, kKvFp8 = 2 };

template <int KV>
struct KvBytes {
  static constexpr int value = KV == kKvF32 ? 4 : (KV == kKvBf16 ? 2 : 1);
};

template <int D, int KV>
struct Geo {
  static constexpr int eb = KvBytes<KV>::value;
  static constexpr int row_bytes = D * eb;           // one token of K
  static constexpr int blk_bytes = kTok * row_bytes;  // one (block, head) of K or V
  static constexpr int vrow_bytes = kTok * eb;        // one dim of V (16 tokens)
  // End-of-unit combine: per (wave, tile) 16 rows of D floats padded by 4
  // (bank spread), then m and l.
  static constexpr int comb_row = D + 4;
  static constexpr int comb_floats = kTok * comb_row + 2 * kTok;
};

__device__ __forceinline__ uint32_t f32_bits(float x) { return __builtin_bit_cast(uint32_t, x); }

// Two OCP E4M3 codes (byte pair kHi of w) -> two bf16 in one dword, in one
// conversion instruction with unit scale. Every E4M3 value fits bf16
// exactly, so the conversion is exact.
template <bool kHi>
__device__ __forceinline__ uint32_t fp8x2_to_bf16x2(uint32_t w) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, kHi));
}

__device__ __forceinline__ uint4 fp8x8_to_bf16x8(uint2 w) {
  return uint4{fp8x2_to_bf16x2<false>(w.x), fp8x2_to_bf16x2<true>(w.x), fp8x2_to_bf16x2<false>(w.y),
               fp8x2_to_bf16x2<true>(w.y)};
}

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));  // RNE
}

__device__ __forceinline__ float xlane_max16(float x) {
  x = fmaxf(x, __shfl_xor(x, 16));
  return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ float xlane_sum16(float x) {
  x += __shfl_xor(x, 16);
  return x + __shfl_xor(x, 32);
}

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// A row's partial state: m, l, the output row and its factor z, with
// (stored element) x z = o / l. For bf16 and fp8 caches the elements are o
// scaled by a power of two, 2^-e, in fp16 (z = 2^e / l); for fp32 caches
// they are o / l in fp32 (z = 1). Elements in lane order: lane (ln, lq)
// holds dimensions 16 t + 4 lq + j of row ln in o[t][j]; the four lanes of
// a row call together.
//
// partial_exp: the exponent e with every |o| / 2^e below 1, reduced across
// the row's lanes (every lane of the wave must call it). This and
// store_partial serve wide units, which fp32 caches do not have.
template <int D>
__device__ __forceinline__ int partial_exp(const f32x4 (&o)[D / 16]) {
  float amax = 0.f;
#pragma unroll
  for (int t = 0; t < D / 16; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) amax = fmaxf(amax, __builtin_fabsf(o[t][j]));
  amax = fmaxf(amax, __shfl_xor(amax, 16));
  amax = fmaxf(amax, __shfl_xor(amax, 32));
  // amax = f 2^e with f in [0.5, 1): every element over 2^e is in [-1, 1].
  return (amax > 0.f && amax <= 3.0e38f) ? __builtin_amdgcn_frexp_expf(amax) : 0;
}

// store_partial: the row's stores, with inv = 1 / l (0 for l = 0) and e
// from above. (Scaling by 2^-e alone, not by 1 / l as well, takes one
// instruction per element instead of two.)
template <int D>
__device__ __forceinline__ void store_partial(void* part_o, float* part_ml, int64_t prow, const f32x4 (&o)[D / 16],
                                              float m, float l, float inv, int e, int lq) {
  uint32_t w[D / 8];
#pragma unroll
  for (int t = 0; t < D / 16; ++t)
#pragma unroll
    for (int j = 0; j < 4; j += 2) {
      const f16x2 h = {static_cast<_Float16>(__builtin_ldexpf(o[t][j], -e)),
                       static_cast<_Float16>(__builtin_ldexpf(o[t][j + 1], -e))};
      w[2 * t + j / 2] = __builtin_bit_cast(uint32_t, h);
    }
  uint4* dst = reinterpret_cast<uint4*>(static_cast<uint16_t*>(part_o) + prow * D + (D / 4) * lq);
#pragma unroll
  for (int c = 0; c < D / 32; ++c) dst[c] = uint4{w[4 * c], w[4 * c + 1], w[4 * c + 2], w[4 * c + 3]};
  // A state without tokens (l = 0) takes no part in the merge's maximum; a
  // NaN m (a bad row) is kept.
  const float m_out = (l > 0.f || m != m) ? m : kNegInf;
  if (lq == 0)
    *reinterpret_cast<f32x4*>(part_ml + prow * kPartMl) = f32x4{m_out, l, __builtin_ldexpf(inv, e), 0.f};
}

// Largest value over the sixteen lanes of a DPP row (rotations within it).
__device__ __forceinline__ float row16_max(float x) {
  auto ror = [](float v, auto n) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),
                                                                 0x120 | decltype(n)::value, 0xf, 0xf, false));
  };
  x = fmaxf(x, ror(x, std::integral_constant<int, 8>{}));
  x = fmaxf(x, ror(x, std::integral_constant<int, 4>{}));
  x = fmaxf(x, ror(x, std::integral_constant<int, 2>{}));
  return fmaxf(x, ror(x, std::integral_constant<int, 1>{}));
}

// The same state from sixteen lanes of a wave's DPP row, lane c holding
// stored elements (D / 16) c .. (all sixteen call together; `active` says
// whether the row exists).
template <int D, int KV>
__device__ __forceinline__ void store_partial_row(void* part_o, float* part_ml, int64_t prow, const f32x4 (&o)[D / 64],
                                                  float m, float l, float inv, int c, bool active) {
  constexpr int kEl = D / 16;
  float z = 1.f;
  if constexpr (KV != kKvF32) {
    float amax = 0.f;
#pragma unroll
    for (int e = 0; e < kEl / 4; ++e)
#pragma unroll
      for (int j = 0; j < 4; ++j) amax = fmaxf(amax, __builtin_fabsf(o[e][j]));
    amax = row16_max(amax);
    const int e2 = (amax > 0.f && amax <= 3.0e38f) ? __builtin_amdgcn_frexp_expf(amax) : 0;
    uint32_t w[kEl / 2];
#pragma unroll
    for (int e = 0; e < kEl / 4; ++e)
#pragma unroll
      for (int j = 0; j < 4; j += 2) {
        const f16x2 h = {static_cast<_Float16>(__builtin_ldexpf(o[e][j], -e2)),
                         static_cast<_Float16>(__builtin_ldexpf(o[e][j + 1], -e2))};
        w[2 * e + j / 2] = __builtin_bit_cast(uint32_t, h);
      }
    if (active) {
      uint16_t* dst = static_cast<uint16_t*>(part_o) + prow * D + kEl * c;
      if constexpr (kEl == 8)
        *reinterpret_cast<uint4*>(dst) = uint4{w[0], w[1], w[2], w[3]};
      else
        *reinterpret_cast<uint2*>(dst) = uint2{w[0], w[1]};
    }
    z = __builtin_ldexpf(inv, e2);
  } else if (active) {
    f32x4* dst = reinterpret_cast<f32x4*>(static_cast<float*>(part_o) + prow * D + kEl * c);
#pragma unroll
    for (int e = 0; e < kEl / 4; ++e) dst[e] = o[e] * inv;
  }
  const float m_out = (l > 0.f || m != m) ? m : kNegInf;
  if (active && c == 0) *reinterpret_cast<f32x4*>(part_ml + prow * kPartMl) = f32x4{m_out, l, z, 0.f};
}

__device__ __forceinline__ int rl(int x, int i) { return __builtin_amdgcn_readlane(x, i); }
__device__ __forceinline__ float rlf(float x, int i) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), i));
}

// Token row of S tile t, MFMA row m inside a pair (see the header).
__device__ __forceinline__ int pair_token(int t, int m) { return ((m >> 2) << 3) + (t << 2) + (m & 3); }

// Operands of one block pair in compute form: bf16 bits (bf16 and fp8
// caches) or fp32. Lane (ln, lq):
//   k[t][j]: K of token pair_token(t, ln), dims 32j + 8lq .. + 8 (bf16)
//            or 16j + 4lq .. + 4 (fp32);
//   v[dt]  : V of dim 16dt + ln, tokens 8lq .. 8lq + 7 of the pair.
template <int D, int KV>
struct KOps {
  static constexpr bool f32 = KV == kKvF32;
  static constexpr int kk = f32 ? D / 16 : D / 32;
  typedef typename std::conditional<f32, f32x4, uint4>::type T;
  T k[2][kk];
};
template <int D, int KV>
struct VOps {
  static constexpr bool f32 = KV == kKvF32;
  typedef typename std::conditional<f32, f32x4, uint4>::type T;
  T v[D / 16][f32 ? 2 : 1];
};
template <int D, int KV>
struct Ops : KOps<D, KV>, VOps<D, KV> {
  typedef typename KOps<D, KV>::T T;
};

// fp8 caches load raw codes (half the registers) and convert per pair.
template <int D>
struct Fp8Frags {
  static constexpr int kk = D / 32;
  typedef uint2 T;
  uint2 k[2][kk];
  uint2 v[D / 16][1];
};

template <int D, int KV>
using Frags = typename std::conditional<KV == kKvFp8, Fp8Frags<D>, Ops<D, KV>>::type;

template <int D, int KV>
__device__ __forceinline__ void load_k(Frags<D, KV>& f, const unsigned char* kb0, const unsigned char* kb1, int ln,
                                       int lq) {
  using G = Geo<D, KV>;
  using F = Frags<D, KV>;
  typedef typename F::T T;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int tok = pair_token(t, ln);
    const unsigned char* kr = (tok < 16 ? kb0 : kb1) + (tok & 15) * G::row_bytes;
#pragma unroll
    for (int j = 0; j < F::kk; ++j)
      f.k[t][j] = *reinterpret_cast<const T*>(kr + (KV == kKvFp8 ? 32 * j + 8 * lq : (4 * j + lq) * 16));
  }
}

template <int D, int KV>
__device__ __forceinline__ void load_v(Frags<D, KV>& f, const unsigned char* vb0, const unsigned char* vb1, int ln,
                                       int lq) {
  using G = Geo<D, KV>;
  typedef typename Frags<D, KV>::T T;
  const unsigned char* vb = (lq >= 2 ? vb1 : vb0) + (lq & 1) * 8 * G::eb + ln * G::vrow_bytes;
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) {
    const unsigned char* vr = vb + 16 * dt * G::vrow_bytes;
    f.v[dt][0] = *reinterpret_cast<const T*>(vr);
    if constexpr (KV == kKvF32) f.v[dt][1] = *reinterpret_cast<const T*>(vr + 16);
  }
}

// Loaded fragments in compute form.
template <int D, int KV>
__device__ __forceinline__ KOps<D, KV> k_ops(const Frags<D, KV>& f) {
  if constexpr (KV == kKvFp8) {
    KOps<D, KV> o;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int j = 0; j < D / 32; ++j) o.k[t][j] = fp8x8_to_bf16x8(f.k[t][j]);
    return o;
  } else {
    return f;
  }
}
template <int D, int KV>
__device__ __forceinline__ VOps<D, KV> v_ops(const Frags<D, KV>& f) {
  if constexpr (KV == kKvFp8) {
    VOps<D, KV> o;
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) o.v[dt][0] = fp8x8_to_bf16x8(f.v[dt][0]);
    return o;
  } else {
    return f;
  }
}

// Zero the V^T operands of tokens past `valid` in this lane's block, so
// unused slots of a partial block never reach the value product.
template <int D, int KV>
__device__ __forceinline__ void mask_v(VOps<D, KV>& o, int lq, int valid0, int valid1) {
  const int valid = lq >= 2 ? valid1 : valid0;
  const int slot0 = 8 * (lq & 1);
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) {
    if constexpr (KV == kKvF32) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (slot0 + 4 * h + e >= valid) o.v[dt][h][e] = 0.f;
    } else {
      uint32_t* a = reinterpret_cast<uint32_t*>(&o.v[dt][0]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t keep =
            (slot0 + 2 * e < valid ? 0x0000FFFFu : 0u) | (slot0 + 2 * e + 1 < valid ? 0xFFFF0000u : 0u);
        a[e] &= keep;
      }
    }
  }
}

// A row's state from those that ns of up to kN waves published in LDS
// (slot(k): state k of the tile, rows of D + 4 floats, then m and l), summed
// in order: this thread's elements (D / 16) c .. in stored order, the
// maximum and the sum. ns = 0: an empty state.
template <int D, int KV, int kN, typename Slot>
__device__ __forceinline__ void combine_row(Slot slot, int ns, int row, int c, f32x4 (&o)[D / 64], float& mx,
                                            float& l) {
  using G = Geo<D, KV>;
  constexpr int kEl = D / 16, kHalf = kN < 4 ? kN : 4;
  // Stored elements (D / 16) c .. are dimensions 16 t + 4 q + j.
  const int q4 = c >> 2, tt = (c & 3) * (kEl / 4);
  // (Past the last state the reads repeat the first place; what they bring
  // is not used.)
  float mw[kN], lw[kN];
  f32x4 ov[kHalf][kEl / 4];
  auto read_states = [&](int k0) {
#pragma unroll
    for (int k = 0; k < kHalf; ++k) {
      const float* x = slot(k0 + k < ns ? k0 + k : 0);
#pragma unroll
      for (int e = 0; e < kEl / 4; ++e)
        ov[k][e] = *reinterpret_cast<const f32x4*>(x + row * G::comb_row + 16 * (tt + e) + 4 * q4);
    }
  };
#pragma unroll
  for (int k = 0; k < kN; ++k) {
    const float* x = slot(k < ns ? k : 0) + kTok * G::comb_row + row;
    mw[k] = x[0];
    lw[k] = x[kTok];
  }
  read_states(0);
  mx = kNegInf;
#pragma unroll
  for (int k = 0; k < kN; ++k) {
    if (k >= ns) {
      mw[k] = kNegInf;
      lw[k] = 0.f;
    }
    mx = fmaxf(mx, mw[k]);
  }
  l = 0.f;
#pragma unroll
  for (int k = 0; k < kN; ++k) {
    mw[k] = mw[k] == kNegInf ? 0.f : __builtin_amdgcn_exp2f(mw[k] - mx);  // now the weight
    l += lw[k] * mw[k];
  }
#pragma unroll
  for (int e = 0; e < kEl / 4; ++e) o[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < kN; ++k) {
    if (k >= ns) break;  // uniform
    if (k == kHalf) read_states(kHalf);
#pragma unroll
    for (int e = 0; e < kEl / 4; ++e) o[e] += ov[k % kHalf][e] * mw[k];
  }
}

// Query rows of the unit in LDS (B operand of S^T = K Q^T): row r is D
// elements (bf16, or fp32 for fp32 caches), its 16-byte columns XOR-swizzled
// by the row so that the 16 lanes of a column read distinct banks.
template <int D, int KV>
struct QLds {
  static constexpr int eb = KV == kKvF32 ? 4 : 2;
  static constexpr int row_bytes = D * eb;
  static constexpr int ncol = row_bytes / 16;
  static constexpr int swz_mask = (ncol < 16 ? ncol : 16) - 1;
  static constexpr int bytes = kMaxRows * row_bytes;
  static __device__ __forceinline__ int offset(int row, int col) {
    return row * row_bytes + ((col ^ (row & swz_mask)) << 4);
  }
};

// Softmax state of one row tile (lane ln = row, lq = token / dim group).
template <int D>
struct RowState {
  f32x4 o[D / 16];
  float m;     // reference (log2 units), uniform over the 4 lanes of a row
  float l;     // per-lane partial sum
  float seen;  // largest exponent argument (scaled score - m) this lane has seen (-inf: none)
};

// Uniform description of one pair: blocks' valid tokens, row ranges and
// (fp8) scales.
struct PairInfo {
  int v0, v1;      // valid tokens (0: no block)
  int a0, e0;      // rows [a0, e0) of block 0
  int a1, e1;      // rows [a1, e1) of block 1
  float ks0, ks1;  // logit scale (softmax scale * log2 e * k_scale)
  float vs0, vs1;  // value scale (fp8) or 1
};

// Query operands of one row tile (lane: row 16r + ln, dims as K's).
template <int D, int KV>
struct QFrag {
  typename Ops<D, KV>::T q[Ops<D, KV>::kk];
};

template <int D, int KV>
__device__ __forceinline__ QFrag<D, KV> q_from_lds(const unsigned char* qlds, int r, int ln, int lq) {
  using O = Ops<D, KV>;
  using Q = QLds<D, KV>;
  QFrag<D, KV> qf;
#pragma unroll
  for (int j = 0; j < O::kk; ++j)
    qf.q[j] = *reinterpret_cast<const typename O::T*>(qlds + Q::offset(16 * r + ln, 4 * j + lq));
  return qf;
}

// One pair against one row tile, in three parts: the scores of its tokens
// (S^T = K Q^T), their probabilities, and the value product (O^T += V^T P^T).
struct Scores {
  f32x4 acc[2];
};

template <int D, int KV>
__device__ __forceinline__ Scores tile_scores(const KOps<D, KV>& f, const QFrag<D, KV>& qfr) {
  using O = KOps<D, KV>;
  const auto& qf = qfr.q;
  Scores s = {{{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}}};
  auto& acc = s.acc;
  if constexpr (O::f32) {
#pragma unroll
    for (int j = 0; j < O::kk; ++j)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.k[t][j].x, qf[j].x, acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.k[t][j].y, qf[j].y, acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.k[t][j].z, qf[j].z, acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.k[t][j].w, qf[j].w, acc[t], 0, 0, 0);
      }
  } else {
#pragma unroll
    for (int j = 0; j < O::kk; ++j)
#pragma unroll
      for (int t = 0; t < 2; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f.k[t][j]),
                                                         __builtin_bit_cast(bf16x8, qf[j]), acc[t], 0, 0, 0);
  }
  return s;
}

// The probabilities as the value product's operand: bf16 (fp8 caches: times
// the V scale), or fp32 for fp32 caches.
template <int KV>
struct Probs {
  float p[8];
};
template <>
struct Probs<kKvBf16> {
  bf16x8 p;
};
template <>
struct Probs<kKvFp8> {
  bf16x8 p;
};

// kWide: the pair applies to every row of the tile (rows past the unit's
// end hold zero queries and are never written) and only a missing second
// block (pi.v1 == 0) is masked, by a reference of +inf for its half of the
// lanes: no branch, so the compiler interleaves consecutive tiles.
template <int D, int KV, bool kWide = false>
__device__ __forceinline__ Probs<KV> tile_probs(const Scores& s, RowState<D>& st, const PairInfo& pi, int r, int ln,
                                                int lq) {
  // Lane (ln, lq) holds row 16r + ln, tokens 8lq + 4t + i of the pair: all in
  // block lq >> 1, at slots 8(lq & 1) + 4t + i.
  const bool hi = lq >= 2;
  const float sc = hi ? pi.ks1 : pi.ks0;
  // Exponent arguments x = score * scale - m (the fp8 K scale is part of
  // `sc`), masked to -inf past the valid tokens and outside the rows the
  // blocks apply to. `seen` tracks the largest x: it is taken over the fma
  // results, which are canonical, so the maximum needs no NaN quieting.
  float x[8];
  const float mref = (kWide && hi && pi.v1 == 0) ? kInf : st.m;
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) x[4 * t + i] = __builtin_fmaf(s.acc[t][i], sc, -mref);
  const int row = 16 * r + ln;
  const int valid = hi ? pi.v1 : pi.v0;
  const int ra = hi ? pi.a1 : pi.a0, re = hi ? pi.e1 : pi.e0;
  const bool full = pi.v0 == kTok && pi.v1 == kTok && pi.a0 <= 16 * r && pi.e0 >= 16 * r + 16 &&
                    pi.a1 <= 16 * r && pi.e1 >= 16 * r + 16;
  if (!kWide && !full) {
    const int lim = (row >= ra && row < re) ? valid : 0;
    const int slot0 = 8 * (lq & 1);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (slot0 + i >= lim) x[i] = kNegInf;
  }
  st.seen = fmaxf(fmaxf(fmaxf(fmaxf(st.seen, x[0]), fmaxf(x[1], x[2])), fmaxf(x[3], x[4])),
                  fmaxf(fmaxf(x[5], x[6]), x[7]));
  float p[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) p[i] = __builtin_amdgcn_exp2f(x[i]);
  st.l += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
  Probs<KV> out;
  if constexpr (KV == kKvF32) {
#pragma unroll
    for (int i = 0; i < 8; ++i) out.p[i] = p[i];
  } else {
    const float vs = hi ? pi.vs1 : pi.vs0;
    float pv[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) pv[i] = (KV == kKvFp8) ? p[i] * vs : p[i];
    const uint4 pb = {pack_bf16x2(pv[0], pv[1]), pack_bf16x2(pv[2], pv[3]), pack_bf16x2(pv[4], pv[5]),
                      pack_bf16x2(pv[6], pv[7])};
    out.p = __builtin_bit_cast(bf16x8, pb);
  }
  return out;
}

template <int D, int KV>
__device__ __forceinline__ void tile_values(const VOps<D, KV>& f, const Probs<KV>& pr, RowState<D>& st) {
  const auto& p = pr.p;
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt) {
    if constexpr (KV == kKvF32) {
      const f32x4 a0 = f.v[dt][0], a1 = f.v[dt][1];
      f32x4 o = st.o[dt];
      o = __builtin_amdgcn_mfma_f32_16x16x4f32(a0.x, p[0], o, 0, 0, 0);
      o = __builtin_amdgcn_mfma_f32_16x16x4f32(a0.y, p[1], o, 0, 0, 0);
      o = __builtin_amdgcn_mfma_f32_16x16x4f32(a0.z, p[2], o, 0, 0, 0);
      o = __builtin_amdgcn_mfma_f32_16x16x4f32(a0.w, p[3], o, 0, 0, 0);
      o = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.x, p[4], o, 0, 0, 0);
      o = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.y, p[5], o, 0, 0, 0);
      o = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.z, p[6], o, 0, 0, 0);
      o = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.w, p[7], o, 0, 0, 0);
      st.o[dt] = o;
    } else {
      st.o[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f.v[dt][0]), p, st.o[dt], 0, 0, 0);
    }
  }
}

// ---- wide units: block pairs shared by the eight waves through LDS -------
// A pair's operands are kChunks 16-byte fragments per lane (K: tile t, slice
// j; then V: dim tile dt). Each wave loads an eighth of them (the
// fragments of all 64 lanes, from the addresses load_pair reads) into
// registers ahead of use, stores them to an LDS stage -- chunk c holds
// fragment c of every lane, lane i at byte 16 i -- and after a barrier every
// wave reads all chunks. (Plain loads stream faster than global-to-LDS
// copies here.)
template <int D, int KV>
struct Stage {  // bf16 operands (fp8 caches stage their codes converted)
  static constexpr int kKChunks = 2 * (D / 32);
  static constexpr int kChunks = kKChunks + D / 16;
  static constexpr int kPerWave = kChunks / kWaves;
  static constexpr int bytes = kChunks * 1024;
  static_assert(kChunks % kWaves == 0, "whole chunks per wave");
};

template <int D, int KV>
__device__ __forceinline__ const unsigned char* frag_src(int c, const unsigned char* kb0, const unsigned char* kb1,
                                                         const unsigned char* vb0, const unsigned char* vb1, int ln,
                                                         int lq) {
  using G = Geo<D, KV>;
  using S = Stage<D, KV>;
  if (c < S::kKChunks) {
    const int t = c / (D / 32), j = c % (D / 32);
    const int tok = pair_token(t, ln);
    return (tok < 16 ? kb0 : kb1) + (tok & 15) * G::row_bytes + (KV == kKvFp8 ? 32 * j + 8 * lq : (4 * j + lq) * 16);
  }
  const int dt = c - S::kKChunks;
  return (lq >= 2 ? vb1 : vb0) + (lq & 1) * 8 * G::eb + ln * G::vrow_bytes + 16 * dt * G::vrow_bytes;
}

// (A vector value rather than an array, so that it stays in registers.)
// fp8 caches hold the raw codes (8 bytes per fragment) until the slice is
// stored, converted, to the stage.
template <int D, int KV>
struct Slice {
  static constexpr int kWords = KV == kKvFp8 ? 2 : 4;  // dwords per fragment
  typedef unsigned int V __attribute__((ext_vector_type(kWords * Stage<D, KV>::kPerWave)));
  V v;
};

// This wave's slice of pair (id0, id1).
template <int D, int KV>
__device__ __forceinline__ void load_slice(Slice<D, KV>& q, int id0, int id1, const unsigned char* kbase,
                                             const unsigned char* vbase, size_t blk_stride, int wave, int ln, int lq) {
  using S = Stage<D, KV>;
  const unsigned char* kb0 = kbase + id0 * blk_stride;
  const unsigned char* kb1 = kbase + id1 * blk_stride;
  const unsigned char* vb0 = vbase + id0 * blk_stride;
  const unsigned char* vb1 = vbase + id1 * blk_stride;
#pragma unroll
  for (int i = 0; i < S::kPerWave; ++i) {
    const unsigned char* src = frag_src<D, KV>(wave + kWaves * i, kb0, kb1, vb0, vb1, ln, lq);
    if constexpr (KV == kKvFp8) {
      const uint2 t = *reinterpret_cast<const uint2*>(src);
      q.v[2 * i] = t.x;
      q.v[2 * i + 1] = t.y;
    } else {
      const uint4 t = *reinterpret_cast<const uint4*>(src);
      q.v[4 * i] = t.x;
      q.v[4 * i + 1] = t.y;
      q.v[4 * i + 2] = t.z;
      q.v[4 * i + 3] = t.w;
    }
  }
}

template <int D, int KV>
__device__ __forceinline__ void store_slice(const Slice<D, KV>& q, unsigned char* stage, int wave, int lane) {
#pragma unroll
  for (int i = 0; i < Stage<D, KV>::kPerWave; ++i) {
    uint4 w;
    if constexpr (KV == kKvFp8)
      w = fp8x8_to_bf16x8(uint2{q.v[2 * i], q.v[2 * i + 1]});
    else
      w = uint4{q.v[4 * i], q.v[4 * i + 1], q.v[4 * i + 2], q.v[4 * i + 3]};
    *reinterpret_cast<uint4*>(stage + (wave + kWaves * i) * 1024 + lane * 16) = w;
  }
}

template <int D, int KV>
__device__ __forceinline__ void read_stage(Ops<D, KV>& o, const unsigned char* stage, int lane) {
  using S = Stage<D, KV>;
#pragma unroll
  for (int c = 0; c < S::kKChunks; ++c)
    o.k[c / (D / 32)][c % (D / 32)] = *reinterpret_cast<const uint4*>(stage + c * 1024 + lane * 16);
#pragma unroll
  for (int dt = 0; dt < D / 16; ++dt)
    o.v[dt][0] = *reinterpret_cast<const uint4*>(stage + (S::kKChunks + dt) * 1024 + lane * 16);
}

// Per-lane view of up to 64 block entries of a unit: lane i holds entry i.
struct Window {
  int id;      // physical block id (clamped into the pool)
  uint32_t w;  // rows [a, e) and valid tokens (0: skip), packed by win_word
  float ks, vs;
};

__device__ __forceinline__ uint32_t win_word(int a, int e, int valid) {
  return static_cast<uint32_t>(a) | (static_cast<uint32_t>(e - 1) << 6) | (static_cast<uint32_t>(valid) << 12);
}
__device__ __forceinline__ int win_a(uint32_t w) { return w & 63; }
__device__ __forceinline__ int win_e(uint32_t w) { return ((w >> 6) & 63) + 1; }
__device__ __forceinline__ int win_valid(uint32_t w) { return w >> 12; }

__device__ __forceinline__ int ent_r0(uint32_t inf) { return inf & 63; }
__device__ __forceinline__ int ent_r1(uint32_t inf) { return ((inf >> 6) & 63) + 1; }
__device__ __forceinline__ int ent_valid(uint32_t inf) { return ((inf >> 12) & 15) + 1; }

// Loads of pair pp of a window (n entries) into f.
template <int D, int KV>
__device__ __forceinline__ void issue_k(Frags<D, KV>& f, const Window& win, int n, int pp, const unsigned char* kbase,
                                        size_t blk_stride, int ln, int lq) {
  const int id0 = rl(win.id, 2 * pp);
  const int id1 = 2 * pp + 1 < n ? rl(win.id, 2 * pp + 1) : id0;
  load_k<D, KV>(f, kbase + id0 * blk_stride, kbase + id1 * blk_stride, ln, lq);
}
template <int D, int KV>
__device__ __forceinline__ void issue_v(Frags<D, KV>& f, const Window& win, int n, int pp, const unsigned char* vbase,
                                        size_t blk_stride, int ln, int lq) {
  const int id0 = rl(win.id, 2 * pp);
  const int id1 = 2 * pp + 1 < n ? rl(win.id, 2 * pp + 1) : id0;
  load_v<D, KV>(f, vbase + id0 * blk_stride, vbase + id1 * blk_stride, ln, lq);
}
template <int D, int KV>
__device__ __forceinline__ void issue_pair(Frags<D, KV>& f, const Window& win, int n, int pp,
                                           const unsigned char* kbase, const unsigned char* vbase, size_t blk_stride,
                                           int ln, int lq) {
  issue_k<D, KV>(f, win, n, pp, kbase, blk_stride, ln, lq);
  issue_v<D, KV>(f, win, n, pp, vbase, blk_stride, ln, lq);
}

// How the waves of a workgroup share a narrow unit: a wave holds the states
// of kNt row tiles (NarrowTiles), so units of more tiles split the waves
// into groups by tile, and the waves of a group take its block pairs in
// turn. A pair with rows of two groups is read by both (from L2 the second
// time).
template <int KV>
struct NarrowTiles {
  static constexpr int value = KV == kKvF32 ? 1 : 2;  // row tiles per wave
};

struct Split {
  int ng;    // groups
  int n;     // waves of this wave's group
  int grp;   // the group: row tiles grp * kNt .. + kNt
  int sub;   // this wave's place in it: pairs sub, sub + n, ...
  int n0;    // two groups: waves of the first
};

// First wave of group g, and its waves (ng = 1: all; two groups: n0 and the
// rest; four: two each).
__device__ __forceinline__ int group_first(const Split& w, int g) { return w.ng == 2 ? (g ? w.n0 : 0) : g * 2; }
__device__ __forceinline__ int group_waves(const Split& w, int g) {
  return w.ng == 1 ? kWaves : (w.ng == 2 ? (g ? kWaves - w.n0 : w.n0) : 2);
}

// n0: the record's share of the first group when there are two (its pairs
// over all of the unit's).
template <int KV>
__device__ __forceinline__ Split split_waves(int nrows, int n0, int wave) {
  constexpr int kNt = NarrowTiles<KV>::value;
  Split w;
  w.ng = nrows <= 16 * kNt ? 1 : (nrows <= 32 * kNt ? 2 : 4);
  w.n0 = n0;
  w.grp = w.ng == 1 ? 0 : (w.ng == 2 ? (wave >= n0 ? 1 : 0) : wave >> 1);
  w.n = group_waves(w, w.grp);
  w.sub = wave - group_first(w, w.grp);
  return w;
}

// The pairs of a window (n entries) that hold rows of group grp: bit 2 i
// set for pair i. drop_pairs takes the first k of them away.
template <int KV>
__device__ __forceinline__ uint64_t group_pairs(const Window& win, int n, int grp, int lane) {
  constexpr int kRows = 16 * NarrowTiles<KV>::value;
  const int r0 = grp * kRows;
  const bool in = lane < n && win_a(win.w) < r0 + kRows && win_e(win.w) > r0;
  const uint64_t e = __builtin_amdgcn_ballot_w64(in);
  return (e | (e >> 1)) & 0x5555555555555555ull;
}
__device__ __forceinline__ uint64_t drop_pairs(uint64_t m, int k) {
  for (int i = 0; i < k; ++i) m &= m - 1;
  return m;
}
__device__ __forceinline__ int first_pair(uint64_t m) { return static_cast<int>(__builtin_ctzll(m)) >> 1; }

// Runs every pair of a window (n entries) through this wave's row tiles
// (rows outside a block's range are masked): the pairs set in `pairs` (its
// share starts at the first, then every ws.n-th). The first has been issued
// into fa by the caller. One pair of load registers, refilled with the next
// pair when it has been used (the eight waves of a workgroup keep up to
// 128 KB in flight, and the other wave of the SIMD computes meanwhile).
template <int D, int KV>
__device__ __forceinline__ void run_window(const Window& win, int n, int nrows, const Split& ws,
                                           const unsigned char* kbase, const unsigned char* vbase, size_t blk_stride,
                                           float sc, const unsigned char* qlds,
                                           RowState<D> (&st)[NarrowTiles<KV>::value], Frags<D, KV>& fa,
                                           uint64_t pairs, int ln, int lq) {
  constexpr int kNt = NarrowTiles<KV>::value;
  if (pairs == 0) return;
  auto info = [&](int pp) {
    PairInfo pi;
    const int i0 = 2 * pp, i1 = 2 * pp + 1;
    const bool has1 = i1 < n;
    const uint32_t w0 = rl(win.w, i0), w1 = rl(win.w, i1 & 63);
    pi.v0 = win_valid(w0);
    pi.v1 = has1 ? win_valid(w1) : 0;
    pi.a0 = win_a(w0);
    pi.e0 = win_e(w0);
    pi.a1 = has1 ? win_a(w1) : 0;
    pi.e1 = has1 ? win_e(w1) : 0;
    pi.ks0 = sc;
    pi.ks1 = sc;
    pi.vs0 = 1.f;
    pi.vs1 = 1.f;
    if constexpr (KV == kKvFp8) {
      pi.ks0 = sc * rlf(win.ks, i0);
      pi.vs0 = rlf(win.vs, i0);
      pi.ks1 = has1 ? sc * rlf(win.ks, i1) : pi.ks0;
      pi.vs1 = has1 ? rlf(win.vs, i1) : pi.vs0;
    }
    return pi;
  };
  for (;;) {
    const PairInfo pi = info(first_pair(pairs));
    pairs = drop_pairs(pairs, ws.n);
    // Row tiles the pair's valid blocks apply to.
    int lo = kMaxRows, hi = 0;
    if (pi.v0 > 0) {
      lo = pi.a0;
      hi = pi.e0;
    }
    if (pi.v1 > 0) {
      lo = lo < pi.a1 ? lo : pi.a1;
      hi = hi > pi.e1 ? hi : pi.e1;
    }
    bool act[kNt];
#pragma unroll
    for (int i = 0; i < kNt; ++i) {
      const int r = ws.grp * kNt + i;
      act[i] = 16 * r < nrows && 16 * r < hi && 16 * r + 16 > lo;
    }
    if constexpr (KV == kKvFp8) {
      // All tiles' scores, then all value products, so that only one of the
      // converted operands is held at a time.
      Scores s[kNt];
      {
        const KOps<D, KV> k = k_ops<D, KV>(fa);
#pragma unroll
        for (int i = 0; i < kNt; ++i)
          if (act[i]) s[i] = tile_scores<D, KV>(k, q_from_lds<D, KV>(qlds, ws.grp * kNt + i, ln, lq));
      }
      if (pairs != 0) issue_k<D, KV>(fa, win, n, first_pair(pairs), kbase, blk_stride, ln, lq);
      Probs<KV> pr[kNt];
#pragma unroll
      for (int i = 0; i < kNt; ++i)
        if (act[i]) pr[i] = tile_probs<D, KV>(s[i], st[i], pi, ws.grp * kNt + i, ln, lq);
      VOps<D, KV> v = v_ops<D, KV>(fa);
      if (pi.v0 < kTok || pi.v1 < kTok) mask_v<D, KV>(v, lq, pi.v0, pi.v1);
#pragma unroll
      for (int i = 0; i < kNt; ++i)
        if (act[i]) tile_values<D, KV>(v, pr[i], st[i]);
      if (pairs == 0) break;
      issue_v<D, KV>(fa, win, n, first_pair(pairs), vbase, blk_stride, ln, lq);
    } else {
      if (pi.v0 < kTok || pi.v1 < kTok) mask_v<D, KV>(fa, lq, pi.v0, pi.v1);
#pragma unroll
      for (int i = 0; i < kNt; ++i)
        if (act[i]) {
          const int r = ws.grp * kNt + i;
          const Scores s = tile_scores<D, KV>(fa, q_from_lds<D, KV>(qlds, r, ln, lq));
          tile_values<D, KV>(fa, tile_probs<D, KV>(s, st[i], pi, r, ln, lq), st[i]);
        }
      if (pairs == 0) break;
      issue_pair<D, KV>(fa, win, n, first_pair(pairs), kbase, vbase, blk_stride, ln, lq);
    }
  }
}

// A unit's record as held by a wave: the header in scalar registers (read
// through the scalar cache; the records are not written while the kernel
// runs) and, per lane, beam `lane` and entry `lane`.
struct UnitRegs {
  int kvh, nrows, nstatic, nent, prow0, next, mode, nstatic2;
  int beam_l;
  int ent_id;
  uint32_t ent_inf;
};

// The record's second window (lane i: entry 64 + i), read only by units
// that have one, when they start.
__device__ __forceinline__ void load_window2(const UnitRec* recs, int idx, int lane, int* id, uint32_t* inf) {
  *id = recs[idx].ent_id2[lane];
  *inf = recs[idx].ent_info2[lane];
}

__device__ __forceinline__ int rfl(int x) { return __builtin_amdgcn_readfirstlane(x); }

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef const i32x8 __attribute__((address_space(4))) * ConstI32x8;

__device__ __forceinline__ UnitRegs load_unit(const UnitRec* recs, int idx, int lane) {
  const UnitRec* r = recs + idx;
  UnitRegs u;
  const i32x8 h = *(ConstI32x8)(reinterpret_cast<uintptr_t>(&r->kvh));
  u.kvh = h[0];
  u.nrows = h[1];
  u.nstatic = h[2];
  u.nent = h[3];
  u.prow0 = h[4];
  u.next = h[5];
  u.mode = h[6];
  u.nstatic2 = h[7];
  u.beam_l = r->beams[lane];
  u.ent_id = r->ent_id[lane];
  u.ent_inf = r->ent_info[lane];
  return u;
}

// Live and build-time lengths of the beams whose entries depend on them
// (the partial last block, the extension marker), loaded by those lanes.
// Current length of beam vb: for verification, virtual beam b * q_len + i
// is beam b's first seq_lens[b] - (q_len - 1 - i) tokens.
template <typename P>
__device__ __forceinline__ int beam_len(const P& p, int vb) {
  if (p.q_len <= 1) return p.seq_lens[vb];
  return p.seq_lens[vb / p.q_len] - (p.q_len - 1 - vb % p.q_len);
}

__device__ __forceinline__ void issue_live(const AttnParams& p, const UnitRegs& u, int lane, int* len, int* build) {
  const bool live = lane < u.nent && (u.ent_inf & (kEntLive | kEntExt)) != 0;
  const int slot = (u.ent_inf & kEntExt) ? u.ent_id : static_cast<int>(ent_r0(u.ent_inf)) / p.g;
  const int lb = __shfl(u.beam_l, slot & 15);  // all lanes take part in the shuffle
  *len = 0;
  *build = 0;
  if (live) {
    *len = beam_len(p, lb);
    *build = p.build_len[lb];
  }
}

// The unit's query rows, fetched into registers (thread t holds 16-byte
// chunks t, t + 512, ... of the rows) while the previous unit finishes, then
// stored to LDS in the swizzled layout. Rows past nrows repeat row 0 (their
// scores are always masked).
// (A vector value rather than an array, so that it stays in registers.)
template <int D, int KV>
struct QRegs {
  static constexpr int kPer = QLds<D, KV>::bytes / (kThreads * 16);
  typedef unsigned int V __attribute__((ext_vector_type(4 * kPer)));
  V v;
};

template <int D, int KV>
__device__ __forceinline__ void load_q(const AttnParams& p, const UnitRegs& u, QRegs<D, KV>& qr, int tid) {
  using Q = QLds<D, KV>;
#pragma unroll
  for (int i = 0; i < QRegs<D, KV>::kPer; ++i) {
    const int c = tid + kThreads * i;
    int row = c / Q::ncol;
    const int col = c % Q::ncol;
    row = row < u.nrows ? row : 0;
    const int b = __shfl(u.beam_l, row / p.g);
    const int qh = u.kvh * p.g + row % p.g;
    const uint4 t = *reinterpret_cast<const uint4*>(static_cast<const unsigned char*>(p.q) +
                                                    (static_cast<int64_t>(b) * p.hq + qh) * Q::row_bytes + col * 16);
    qr.v[4 * i] = t.x;
    qr.v[4 * i + 1] = t.y;
    qr.v[4 * i + 2] = t.z;
    qr.v[4 * i + 3] = t.w;
  }
}

template <int D, int KV>
__device__ __forceinline__ void store_q(const QRegs<D, KV>& qr, unsigned char* qbuf, int tid) {
  using Q = QLds<D, KV>;
#pragma unroll
  for (int i = 0; i < QRegs<D, KV>::kPer; ++i) {
    const int c = tid + kThreads * i;
    *reinterpret_cast<uint4*>(qbuf + Q::offset(c / Q::ncol, c % Q::ncol)) =
        uint4{qr.v[4 * i], qr.v[4 * i + 1], qr.v[4 * i + 2], qr.v[4 * i + 3]};
  }
}

// kWin2: some unit of the plan has a second entry window. kPaged: the paged
// path, whose units come from the workgroup id and not from records.
template <int D, int KV, bool kWin2, bool kPaged>
__global__ __launch_bounds__(kThreads, 1) void attn_kernel(AttnParams p) {
  using G = Geo<D, KV>;
  using Q = QLds<D, KV>;
  // LDS: the current unit's query rows, and the end-of-unit combine area
  // where every wave publishes its row tiles' states.
  // Wide units (bf16 and fp8) use the area after the query rows for their
  // pair stages instead.
  constexpr int kNt = NarrowTiles<KV>::value;
  constexpr int kGroups = kTiles / kNt;  // wave groups of the largest narrow unit
  constexpr int kCombBytes = kWaves * kNt * G::comb_floats * 4;
  constexpr int kStageBytes = KV != kKvF32 ? 2 * kStepPairs * Stage<D, KV>::bytes : 0;
  constexpr int kFoldBytes = KV != kKvF32 ? kWaves * (64 * (D + 8)) : 0;  // wide units' halves: a tile per wave
  constexpr int kAreaBytes = kCombBytes > kStageBytes ? (kCombBytes > kFoldBytes ? kCombBytes : kFoldBytes)
                                                      : (kStageBytes > kFoldBytes ? kStageBytes : kFoldBytes);
  // Narrow units with a second window park its entries (per lane: block id
  // and info word; every wave writes the same values) until the first one
  // is done, instead of holding two more registers through the pair loop.
  constexpr int kWin2Bytes = kWin2 ? 8 * kMaxEntries : 0;
  // Wide units: each wave's "redo" vote (one word per wave).
  constexpr int kVoteBytes = 4 * kWaves;
  __shared__ __attribute__((aligned(16))) unsigned char lds[Q::bytes + kAreaBytes + kWin2Bytes + kVoteBytes];
  unsigned char* qbuf = lds;
  float* comb = reinterpret_cast<float*>(lds + Q::bytes);
  uint2* win2_lds = reinterpret_cast<uint2*>(lds + Q::bytes + kAreaBytes);
  int* votes = reinterpret_cast<int*>(lds + Q::bytes + kAreaBytes + kWin2Bytes);

  const int wave = rfl(static_cast<int>(threadIdx.x) >> 6);
  // The thread's coordinates, opaque to the optimiser once per unit: lane
  // address arithmetic hoisted out of the unit loop as constants of the
  // whole kernel would be spilled to scratch memory (244 bytes per thread,
  // written by every workgroup of every launch).
  int tid, lane, ln, lq;
  auto coords = [&]() {
    tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    lane = tid & 63;
    ln = lane & 15;
    lq = lane >> 4;
  };
  coords();
  const size_t blk_stride = static_cast<size_t>(p.hkv) * G::blk_bytes;
  constexpr bool paged = kPaged;
  const float sc = p.scale_log2;
  auto comb_slot = [&](int w, int i) { return comb + (w * kNt + i) * G::comb_floats; };  // (wave, its tile)

  // The parameters of the first steps in one read.
  asm volatile("" ::"s"(p.q), "s"(p.k_cache), "s"(p.v_cache), "s"(p.recs), "s"(p.seq_lens), "s"(p.build_len),
               "s"(p.hq), "s"(p.hkv), "s"(p.g), "s"(p.q_len));
  // ---- first unit -----------------------------------------------------------
  int rec_idx;
  UnitRegs u;
  int paged_b = 0, paged_split = 0;
  if (!paged) {
    rec_idx = blockIdx.x;
    u = load_unit(p.recs, rec_idx, lane);
  } else {
    // Paged path: unit = (beam, KV head, split) from the workgroup id, one
    // beam's g rows against up to 32 of its blocks.
    rec_idx = 0;
    paged_split = blockIdx.x % p.paged_nsplit;
    const int bh = blockIdx.x / p.paged_nsplit;
    paged_b = bh / p.hkv;
    u.kvh = bh % p.hkv;
    u.nrows = p.g;
    u.nstatic = 0;
    u.nent = 0;
    u.prow0 = 0;
    u.next = -1;
    u.mode = kModeNarrow | (kWaves / 2) << 8;
    u.beam_l = paged_b;
    u.ent_id = 0;
    u.ent_inf = 0;
    u.nstatic2 = 0;
  }
  QRegs<D, KV> qr;
  Frags<D, KV> fa;
  bool fa_ready = false;  // the unit's first pair and lengths are in flight
  // fp32 at D = 128: a pair is 128 registers, too many to hold while the
  // previous unit combines.
  constexpr bool kEarlyPair = KV != kKvF32 || D < 128;
  int ext_len = 0, ext_build = 0;  // live / extension lanes: live and build-time length
  UnitRegs nu;
  // Hand-over to unit n: a narrow unit's query rows, first pair and lengths
  // go out before this unit's combine. Every path assigns the carried
  // registers, so their previous contents are dead while a unit runs.
  auto handover = [&](const UnitRegs& n) {
    if ((n.mode & 0xff) == kModeNarrow) {
      load_q<D, KV>(p, n, qr, tid);
      if (!kEarlyPair) {
        fa_ready = false;
        return;
      }
      const int nn = rfl(n.nstatic), nkvh = rfl(n.kvh);
      Window nw;
      nw.id = n.ent_id;
      const Split nws = split_waves<KV>(n.nrows, n.mode >> 8, wave);
      nw.w = win_word(ent_r0(n.ent_inf), ent_r1(n.ent_inf), 0);
      const uint64_t npairs = drop_pairs(group_pairs<KV>(nw, nn, nws.grp, lane), nws.sub);
      if (npairs != 0)
        issue_pair<D, KV>(fa, nw, nn, first_pair(npairs),
                          static_cast<const unsigned char*>(p.k_cache) + nkvh * G::blk_bytes,
                          static_cast<const unsigned char*>(p.v_cache) + nkvh * G::blk_bytes, blk_stride, ln, lq);
      else
        fa = Frags<D, KV>{};
      issue_live(p, n, lane, &ext_len, &ext_build);
    } else {
      qr = QRegs<D, KV>{};
      fa = Frags<D, KV>{};
      ext_len = 0;
      ext_build = 0;
    }
    fa_ready = true;
  };
  // The record's loads all go out before any is waited for (left to itself
  // the compiler moves most of them behind the wait for the header and the
  // test of it), then the first unit's query rows, first pair and lengths
  // together (in the unit's own code the pair waited for the query rows). An
  // idle workgroup's record holds no rows and names beam 0, so its loads are
  // in bounds.
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (kPaged)
    load_q<D, KV>(p, u, qr, tid);
  else
    handover(u);
  if (rfl(u.nrows) <= 0) return;

  for (;;) {
    coords();
    TTS_PROF_MARK(0, rec_idx);
    const int kvh = rfl(u.kvh), nrows = rfl(u.nrows), nent = rfl(u.nent), prow0 = rfl(u.prow0),
              unext = rfl(u.next);
    const int nt = (nrows + 15) >> 4;
    const unsigned char* kbase = static_cast<const unsigned char*>(p.k_cache) + kvh * G::blk_bytes;
    const unsigned char* vbase = static_cast<const unsigned char*>(p.v_cache) + kvh * G::blk_bytes;

    if constexpr (KV != kKvF32 && !kPaged) {
      if ((u.mode & 0xff) == kModeWide) {
        // ---- wide unit: every block pair is copied to an LDS stage once and
        // read from there. Up to eight row tiles: four waves hold all of them
        // (wave w tiles w % 4 and w % 4 + 4) and each half of the workgroup
        // takes one pair of every step; the halves' states are added at the
        // end. (LDS reads bound this loop: 128 bytes a clock, 16 KB per wave
        // and pair. With two tiles per wave a pair is read four times
        // instead of eight.) More tiles: wave w holds tiles w and w + 8 and
        // computes every pair.
        using SG = Stage<D, KV>;
        const int nst = rfl(u.nstatic);
        const bool halves = nt <= kWaves;
        const int half = halves ? wave >> 2 : 0;
        const int tile0 = halves ? wave & 3 : wave, tstep = halves ? 4 : kWaves;
        nu.nrows = 0;
        if (unext >= 0) nu = load_unit(p.recs, unext, lane);
        QFrag<D, KV> qw[kWideTiles];
#pragma unroll
        for (int i = 0; i < kWideTiles; ++i) {
          const int row = 16 * (tile0 + tstep * i) + ln;
          const bool ok = row < nrows;
          const int b = __shfl(u.beam_l, ok ? row / p.g : 0);
          const int qh = kvh * p.g + (ok ? row % p.g : 0);
          const uint16_t* qrow = static_cast<const uint16_t*>(p.q) + (static_cast<int64_t>(b) * p.hq + qh) * D;
#pragma unroll
          for (int j = 0; j < Ops<D, KV>::kk; ++j)
            qw[i].q[j] = ok ? *reinterpret_cast<const uint4*>(qrow + 32 * j + 8 * lq) : uint4{0u, 0u, 0u, 0u};
        }
        unsigned char* stages = lds + Q::bytes;
        const int np = (nst + 1) >> 1;
        const int nsteps = (np + kStepPairs - 1) / kStepPairs;
        // Row tiles of this wave: a wave with none still stages its share.
        const int wtiles = nt > tile0 + tstep ? 2 : (nt > tile0 ? 1 : 0);
        // A wide unit has up to kMaxUnitEntries blocks, numbered across its
        // two windows: entry i < 64 in lane i of ent_id, entry 64 + i in lane
        // i of ent_id2. Entries (e0, e1) and block ids of pair pp; a pair
        // never straddles the two windows.
        int ent_id2 = 0;
        uint32_t ent_inf2 = 0;
        if (kWin2 && nst > kMaxEntries) load_window2(p.recs, rec_idx, lane, &ent_id2, &ent_inf2);
        int e0, e1, id0, id1;
        auto pair_ids = [&](int pp) {
          pp = pp < np ? pp : np - 1;  // past the end: a repeat of the last pair (a cache hit, never used)
          e0 = 2 * pp;
          e1 = 2 * pp + 1 < nst ? 2 * pp + 1 : e0;
          const int ids = (!kWin2 || e0 < kMaxEntries) ? u.ent_id : ent_id2;
          id0 = rl(ids, e0 & (kMaxEntries - 1));
          id1 = rl(ids, e1 & (kMaxEntries - 1));
        };
        // fp8: lane i holds the K and V scales of entries i and 64 + i, read
        // once per unit.
        float ksl = 1.f, vsl = 1.f, ksl2 = 1.f, vsl2 = 1.f;
        if constexpr (KV == kKvFp8) {
          if (lane < nst) {
            ksl = p.k_scale[u.ent_id];
            vsl = p.v_scale[u.ent_id];
          }
          if (kWin2 && lane + kMaxEntries < nst) {
            ksl2 = p.k_scale[ent_id2];
            vsl2 = p.v_scale[ent_id2];
          }
        }
        RowState<D> st[kWideTiles];
        float m_exact[kWideTiles];
#pragma unroll
        for (int i = 0; i < kWideTiles; ++i) m_exact[i] = 0.f;
        for (int attempt = 0;; ++attempt) {
#pragma unroll
          for (int i = 0; i < kWideTiles; ++i) {
#pragma unroll
            for (int d = 0; d < D / 16; ++d) st[i].o[d] = f32x4{0.f, 0.f, 0.f, 0.f};
            st[i].m = m_exact[i];
            st[i].l = 0.f;
            st[i].seen = kNegInf;
          }
          // This wave's slices of the step's pairs: refilled with the next
          // step's as soon as they are staged, so the loads are in flight for
          // a whole step.
          Slice<D, KV> cur[kStepPairs];
          auto load_step = [&](int sidx) {
#pragma unroll
            for (int h = 0; h < kStepPairs; ++h) {
              pair_ids(kStepPairs * sidx + h);
              load_slice<D, KV>(cur[h], id0, id1, kbase, vbase, blk_stride, wave, ln, lq);
            }
          };
          load_step(0);
          __syncthreads();  // every wave is done with the stage area (previous unit or attempt)
          // kTpw: this wave's row tiles.
          auto run = [&](auto tpw_c) {
            constexpr int kTpw = decltype(tpw_c)::value;
            for (int sidx = 0; sidx < nsteps; ++sidx) {
              unsigned char* stage = stages + (sidx & 1) * kStepPairs * SG::bytes;
#pragma unroll
              for (int h = 0; h < kStepPairs; ++h) store_slice<D, KV>(cur[h], stage + h * SG::bytes, wave, lane);
              load_step(sidx + 1);
              __syncthreads();  // the step's pairs are in the stage
              if constexpr (kTpw > 0) {
                const int h0 = halves ? half : 0, h1 = halves ? half + 1 : kStepPairs;
#pragma unroll 1
                for (int h = h0; h < h1; ++h) {
                  const int pp = kStepPairs * sidx + h;
                  if (pp >= np) break;  // the last step's missing pair
                  pair_ids(pp);
                  PairInfo pi;
                  pi.v0 = kTok;
                  pi.v1 = 2 * pp + 1 < nst ? kTok : 0;
                  pi.a0 = pi.a1 = 0;
                  pi.e0 = pi.e1 = nrows;
                  pi.ks0 = pi.ks1 = sc;
                  pi.vs0 = pi.vs1 = 1.f;
                  if constexpr (KV == kKvFp8) {
                    const float ks = e0 < kMaxEntries ? ksl : ksl2, vs = e0 < kMaxEntries ? vsl : vsl2;
                    const int i0 = e0 & (kMaxEntries - 1), i1 = e1 & (kMaxEntries - 1);
                    pi.ks0 = sc * rlf(ks, i0);
                    pi.ks1 = sc * rlf(ks, i1);
                    pi.vs0 = rlf(vs, i0);
                    pi.vs1 = rlf(vs, i1);
                  }
                  Ops<D, KV> o;
                  read_stage<D, KV>(o, stage + h * SG::bytes, lane);
                  if (pi.v1 == 0) mask_v<D, KV>(o, lq, pi.v0, pi.v1);
                  // The scores of all tiles first (K's registers are free early);
                  // from there to the last value product this wave goes ahead
                  // of the SIMD's other one, so that the two drift apart and
                  // one's products run beside the other's LDS reads: long
                  // chain (fp8) 263.2 -> 261.1 us per call, verification of
                  // four tokens 39.7 -> 39.5, others unchanged. (The priority
                  // alone, or opposite pair orders for the two: no change.)
                  Scores sco[kTpw];
#pragma unroll
                  for (int i = 0; i < kTpw; ++i) sco[i] = tile_scores<D, KV>(o, qw[i]);
                  __builtin_amdgcn_s_setprio(1);
#pragma unroll
                  for (int i = 0; i < kTpw; ++i)
                    tile_values<D, KV>(o, tile_probs<D, KV, true>(sco[i], st[i], pi, 0, ln, lq), st[i]);
                  __builtin_amdgcn_s_setprio(0);
                }
              }
            }
          };
          // One copy of the loop per tile count: branch-free tile steps, and
          // no accumulator copies at joins. (Waves of one workgroup run
          // different copies; every copy meets the same barriers.)
          if (wtiles == 2)
            run(std::integral_constant<int, 2>{});
          else if (wtiles == 1)
            run(std::integral_constant<int, 1>{});
          else
            run(std::integral_constant<int, 0>{});
          if (attempt == 0) TTS_PROF_MARK(1, rec_idx);
          if (attempt > 0) {
            if (halves) __syncthreads();  // every wave is done with the stages (the vote's barrier, after the first)
            break;
          }
          bool redo = false;
#pragma unroll
          for (int i = 0; i < kWideTiles; ++i) {
            const float mx = xlane_max16(st[i].seen);
            redo |= mx > kRefWindow || (mx < -kRefWindow && mx != kNegInf);
            m_exact[i] = mx == kNegInf ? 0.f : mx;
          }
          // The loop holds barriers, so every wave repeats it or none does:
          // each wave votes, and all eight read every vote. (The votes are
          // written again only after the next unit's first barrier.)
          const bool wave_redo = __builtin_amdgcn_ballot_w64(redo) != 0;
          if (lane == 0) votes[wave] = wave_redo ? 1 : 0;
          __syncthreads();
          int any = 0;
#pragma unroll
          for (int w = 0; w < kWaves; ++w) any |= votes[w];
          if (any == 0) break;
        }
        // Halves: each wave hands one of its tiles to the wave that shares its
        // rows and adds that wave's other tile: half 0 ends with tile w % 4,
        // half 1 with w % 4 + 4. (The area is the stages': after either
        // attempt a barrier lies between their last read and these stores.)
        // Lane order, one 16-byte column per 16 dims.
        if (halves) {
          auto fold_at = [&](int w) { return comb + w * (16 * (D + 8)); };
          auto give = [&](RowState<D>& x) {
            float* c = fold_at(wave);
#pragma unroll
            for (int dt = 0; dt < D / 16; ++dt) *reinterpret_cast<f32x4*>(c + 256 * dt + 4 * lane) = x.o[dt];
            *reinterpret_cast<f32x2*>(c + 16 * D + 2 * lane) = f32x2{x.m, x.l};
          };
          auto take = [&](RowState<D>& x) {
            const float* c = fold_at(wave ^ 4);
            f32x4 t[D / 16];
#pragma unroll
            for (int dt = 0; dt < D / 16; ++dt) t[dt] = *reinterpret_cast<const f32x4*>(c + 256 * dt + 4 * lane);
            const f32x2 ml = *reinterpret_cast<const f32x2*>(c + 16 * D + 2 * lane);
            // A half that saw no token of the row must not set the reference.
            const float l1 = xlane_sum16(x.l), l2 = xlane_sum16(ml.y);
            const float m1 = l1 > 0.f ? x.m : kNegInf, m2 = l2 > 0.f ? ml.x : kNegInf;
            const float mx = fmaxf(m1, m2);
            const float f1 = m1 == kNegInf ? 0.f : __builtin_amdgcn_exp2f(m1 - mx);
            const float f2 = m2 == kNegInf ? 0.f : __builtin_amdgcn_exp2f(m2 - mx);
            x.m = mx;
            x.l = x.l * f1 + ml.y * f2;
#pragma unroll
            for (int dt = 0; dt < D / 16; ++dt) x.o[dt] = x.o[dt] * f1 + t[dt] * f2;
          };
          if (half == 0 && wtiles == 2) give(st[1]);
          if (half == 1 && wtiles >= 1) give(st[0]);
          __syncthreads();
          if (half == 0 && wtiles >= 1) take(st[0]);
          if (half == 1 && wtiles == 2) take(st[1]);
        }
        // Each wave writes the partial states of its own rows. The sums and
        // scales of all its tiles first, in straight-line code, so that the
        // tiles' cross-lane reductions overlap (a tile past the unit's rows
        // holds l = 0 and zeros, and is not written).
        float lw_[kWideTiles], inv_[kWideTiles];
        int e_[kWideTiles];
#pragma unroll
        for (int i = 0; i < kWideTiles; ++i) lw_[i] = xlane_sum16(st[i].l);
#pragma unroll
        for (int i = 0; i < kWideTiles; ++i) inv_[i] = lw_[i] > 0.f ? 1.f / lw_[i] : 0.f;
#pragma unroll
        for (int i = 0; i < kWideTiles; ++i) e_[i] = partial_exp<D>(st[i].o);
#pragma unroll
        for (int i = 0; i < kWideTiles; ++i) {
          if (i >= wtiles || (halves && i != half)) continue;  // wave-uniform
          const int row = 16 * (tile0 + tstep * i) + ln;
          const int64_t prow = static_cast<int64_t>(kvh) * p.rows_per_head + prow0 + row;
          if (row < nrows) store_partial<D>(p.part_o, p.part_ml, prow, st[i].o, st[i].m, lw_[i], inv_[i], e_[i], lq);
        }
        TTS_PROF_MARK(2, rec_idx);
        const int nu_rows_w = rfl(nu.nrows);
        if (nu_rows_w <= 0) break;
        handover(nu);
        rec_idx = unext;
        u = nu;
        continue;
      }
    }

    // ---- the unit's block window ------------------------------------------
    Window win;
    uint64_t bad_rows = 0;  // rows that met a bad block id or an over-long beam: NaN
    int nstatic = rfl(u.nstatic);
    if (!paged) {
      win.id = u.ent_id;
      win.w = win_word(ent_r0(u.ent_inf), ent_r1(u.ent_inf), lane < nstatic ? ent_valid(u.ent_inf) : 0);
      if (!fa_ready) issue_live(p, u, lane, &ext_len, &ext_build);
    } else {
      const int L = p.seq_lens[paged_b];
      // Split j covers blocks [j * per, (j + 1) * per) of the beam (per <= 32).
      const int per = (p.paged_max_len + kTok * p.paged_nsplit - 1) / (kTok * p.paged_nsplit);
      const int j = paged_split * per + lane;
      int nb = (L + kTok - 1) / kTok;
      bool bad = false;
      if (L < 0 || L > p.paged_max_len || nb > p.max_blocks) {
        bad = true;
        nb = 0;
      }
      nstatic = nb - paged_split * per;
      nstatic = nstatic < 0 ? 0 : (nstatic < per ? nstatic : per);
      int id = 0, v = 0;
      if (lane < nstatic) {
        id = p.block_tables[static_cast<int64_t>(paged_b) * p.max_blocks + j];
        v = L - j * kTok;
        v = v < kTok ? v : kTok;
        if (id < 0 || id >= p.num_blocks) {
          bad = true;
          id = 0;
          v = 0;
        }
      }
      win.id = id;
      win.w = win_word(0, nrows, v);
      if (__builtin_amdgcn_ballot_w64(bad) != 0) bad_rows = ~0ull;
    }
    win.ks = 1.f;
    win.vs = 1.f;
    if constexpr (KV == kKvFp8) {
      if (win_valid(win.w) > 0) {
        win.ks = p.k_scale[win.id];
        win.vs = p.v_scale[win.id];
      }
    }
    // The second window (static entries only, validated at build time) is
    // set up when the first one is done.
    const int nstatic2 = (!kWin2 || paged) ? 0 : rfl(u.nstatic2);
    if (kWin2 && nstatic2 > 0) {
      int id2;
      uint32_t inf2;
      load_window2(p.recs, rec_idx, lane, &id2, &inf2);
      win2_lds[lane] = uint2{static_cast<uint32_t>(id2), inf2};
    }
    const Split ws = split_waves<KV>(nrows, u.mode >> 8, wave);
    const uint64_t pairs_static = drop_pairs(group_pairs<KV>(win, nstatic, ws.grp, lane), ws.sub);
    if (!fa_ready && pairs_static != 0)
      issue_pair<D, KV>(fa, win, nstatic, first_pair(pairs_static), kbase, vbase, blk_stride, ln, lq);
    // The next unit's record: it has this unit's pair loop to arrive.
    nu.nrows = 0;
    if (unext >= 0) nu = load_unit(p.recs, unext, lane);

    store_q<D, KV>(qr, qbuf, tid);
    __syncthreads();  // query rows in LDS

    // ---- the unit's blocks with m_ref = 0; again with every row's exact
    // maximum in the rare case that a row's maximum left the safe window ----
    RowState<D> st[kNt];
    float m_exact[kNt];
#pragma unroll
    for (int r = 0; r < kNt; ++r) m_exact[r] = 0.f;
    if (!paged && lane < nstatic && (u.ent_inf & kEntLive)) {
      // The beam's partial last block: it fills up as tokens are appended.
      const int v = win_valid(win.w) + (ext_len - ext_build);
      win.w = win_word(win_a(win.w), win_e(win.w), v < 0 ? 0 : (v > kTok ? kTok : v));
    }
    // ---- blocks its beams gained after the metadata was built ---------------
    // Numbered over the unit's beams and packed into windows of 64, whatever
    // beam they belong to, and in the first window where they fit: read beam
    // by beam, every beam cost a round trip to the table and one to its
    // blocks (append and call on the 7B 64-beam tree, 100 tokens on: 34.3 us
    // against 32.0; what is left of growth is its bytes and the balance of a
    // plan made without it).
    int grow = 0, first_new = 0;  // lane e (extension entry): blocks gained, the first one
    if (!paged && lane >= nstatic && lane < nent && (u.ent_inf & kEntExt) != 0) {
      first_new = (ext_build + kTok - 1) / kTok;
      // (Shorter than at build time: the merge reports NaN.)
      if (ext_len >= ext_build) grow = (ext_len + kTok - 1) / kTok - first_new;
    }
    auto rows_mask = [](uint32_t w) {
      const int a = win_a(w), e = win_e(w);
      return (e >= 64 ? ~0ull : ((1ull << e) - 1)) & ~((1ull << a) - 1);
    };
    // A beam longer than its table row: NaN rows.
    for (uint64_t over = __builtin_amdgcn_ballot_w64(grow > 0 && first_new + grow > p.max_blocks); over != 0;
         over &= over - 1) {
      bad_rows |= rows_mask(rl(win.w, static_cast<int>(__builtin_ctzll(over))));
    }
    if (first_new + grow > p.max_blocks) grow = 0;
    const uint64_t grown = __builtin_amdgcn_ballot_w64(grow > 0);
    int ngrown = 0;
    for (uint64_t left = grown; left != 0; left &= left - 1) ngrown += rl(grow, static_cast<int>(__builtin_ctzll(left)));
    // Entries t0, t0 + 1, ... of them into lanes l0 .. of id and w.
    auto new_entries = [&](int t0, int l0, int* id, uint32_t* w) {
      int beam = -1, j = 0, len = 0;
      uint32_t inf = 0;
      int at = l0 - t0;
      for (uint64_t left = grown; left != 0; left &= left - 1) {
        const int e = static_cast<int>(__builtin_ctzll(left));
        const int n = rl(grow, e);
        if (lane >= l0 && lane >= at && lane < at + n) {
          beam = rl(u.beam_l, rl(u.ent_id, e) & 15);
          j = rl(first_new, e) + lane - at;
          len = rl(ext_len, e);
          inf = rl(static_cast<int>(u.ent_inf), e);
        }
        at += n;
      }
      bool bad = false;
      if (beam >= 0) {
        if (p.q_len > 1) beam /= p.q_len;
        int x = p.block_tables[static_cast<int64_t>(beam) * p.max_blocks + j];
        int v = len - j * kTok;
        v = v < kTok ? v : kTok;
        bad = x < 0 || x >= p.num_blocks;
        if (bad) {
          x = 0;
          v = 0;
        }
        *id = x;
        *w = win_word(ent_r0(inf), ent_r1(inf), v);
      }
      for (uint64_t m = __builtin_amdgcn_ballot_w64(bad); m != 0; m &= m - 1)
        bad_rows |= rows_mask(rl(*w, static_cast<int>(__builtin_ctzll(m))));
    };
    // In the first window they start at an even place, so that the pairs of
    // its own entries stay as they are (an odd last one is paired with a
    // repeat of itself that holds no token).
    const int new0 = (nstatic + 1) & ~1;
    int nfirst = nstatic, next_new = 0;
    if (ngrown > 0 && new0 + ngrown <= kMaxEntries) {
      if (nstatic & 1) {
        const int last_id = rl(win.id, nstatic - 1);
        const uint32_t last_w = rl(win.w, nstatic - 1);
        if (lane == nstatic) {
          win.id = last_id;
          win.w = win_word(win_a(last_w), win_e(last_w), 0);
        }
      }
      new_entries(0, new0, &win.id, &win.w);
      if constexpr (KV == kKvFp8) {
        if (lane >= new0 && lane < new0 + ngrown && win_valid(win.w) > 0) {
          win.ks = p.k_scale[win.id];
          win.vs = p.v_scale[win.id];
        }
      }
      nfirst = new0 + ngrown;
      next_new = ngrown;
    }
    const uint64_t pairs0 = drop_pairs(group_pairs<KV>(win, nfirst, ws.grp, lane), ws.sub);
    if (pairs_static == 0 && pairs0 != 0)
      issue_pair<D, KV>(fa, win, nfirst, first_pair(pairs0), kbase, vbase, blk_stride, ln, lq);
    // Waves of each group that are given a pair: those of its first window,
    // or all (when the unit has more windows).
    bool wave_has = pairs0 != 0;
    int nsrc[kGroups];
#pragma unroll
    for (int gq = 0; gq < kGroups; ++gq) {
      const int c = __builtin_popcountll(group_pairs<KV>(win, nfirst, gq, lane)), n = group_waves(ws, gq);
      nsrc[gq] = c < n ? c : n;
    }
    for (int attempt = 0;; ++attempt) {
#pragma unroll
      for (int r = 0; r < kNt; ++r) {
#pragma unroll
        for (int i = 0; i < D / 16; ++i) st[r].o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        st[r].m = m_exact[r];
        st[r].l = 0.f;
        st[r].seen = kNegInf;
      }
      if (attempt > 0 && pairs0 != 0)
        issue_pair<D, KV>(fa, win, nfirst, first_pair(pairs0), kbase, vbase, blk_stride, ln, lq);
      // Windows of blocks: the unit's own entries first (one or two
      // windows), then what its beams gained and the first had no room for,
      // 64 at a time. One
      // call site keeps the register allocation of the pair loop in one
      // piece.
      Window cw = win;
      int cn = nfirst;
      uint64_t cpairs = pairs0;
      bool second = nstatic2 > 0;
      int done_new = next_new;
      for (;;) {
        run_window<D, KV>(cw, cn, nrows, ws, kbase, vbase, blk_stride, sc, qbuf, st, fa, cpairs, ln, lq);
        if (attempt == 0) TTS_PROF_MARK(1, rec_idx);
        // The next window: the unit's second one, else the next of gained
        // blocks; one issue site below for both.
        int id = 0;
        uint32_t w = win_word(0, 1, 0);
        if (second) {
          second = false;
          cn = nstatic2;
          const uint2 w2 = win2_lds[lane];
          id = static_cast<int>(w2.x);
          w = win_word(ent_r0(w2.y), ent_r1(w2.y), lane < cn ? ent_valid(w2.y) : 0);
        } else {
          if (done_new >= ngrown) break;
          cn = (ngrown - done_new) < kMaxEntries ? (ngrown - done_new) : kMaxEntries;
          new_entries(done_new, 0, &id, &w);
          done_new += cn;
        }
        wave_has = true;
#pragma unroll
        for (int gq = 0; gq < kGroups; ++gq) nsrc[gq] = group_waves(ws, gq);
        cw.id = id;
        cw.w = w;
        cw.ks = 1.f;
        cw.vs = 1.f;
        if constexpr (KV == kKvFp8) {
          if (win_valid(w) > 0) {
            cw.ks = p.k_scale[id];
            cw.vs = p.v_scale[id];
          }
        }
        cpairs = drop_pairs(group_pairs<KV>(cw, cn, ws.grp, lane), ws.sub);
        if (cpairs != 0) issue_pair<D, KV>(fa, cw, cn, first_pair(cpairs), kbase, vbase, blk_stride, ln, lq);
      }
      if (attempt > 0) break;
      bool redo = false;
#pragma unroll
      for (int r = 0; r < kNt; ++r) {
        const float mx = xlane_max16(st[r].seen);
        redo |= mx > kRefWindow || (mx < -kRefWindow && mx != kNegInf);
        m_exact[r] = mx == kNegInf ? 0.f : mx;
      }
      if (__builtin_amdgcn_ballot_w64(redo) == 0) break;
    }

    // ---- hand over: the next unit's query copies and first pair go out
    // before this unit's combine ---------------------------------------------
    __syncthreads();  // every wave is done with qbuf
    TTS_PROF_MARK(4, rec_idx);
    const int nu_rows = rfl(nu.nrows);
    if (nu_rows > 0) handover(nu);

    TTS_PROF_MARK(5, rec_idx);
    // ---- combine the states of each group's waves --------------------------
    // The waves publish their states in LDS, then sixteen threads per row
    // sum them, in wave order. A wave that was given no pair publishes
    // nothing and is not read.
#pragma unroll
    for (int i = 0; i < kNt; ++i) st[i].l = xlane_sum16(st[i].l);
    // A wave that saw no token of a row (l = 0: every score masked) keeps
    // its initial reference; it must not set the maximum, or a row whose
    // scores all lie far below it would lose every weight to underflow.
#pragma unroll
    for (int i = 0; i < kNt; ++i)
      if (!(st[i].l > 0.f)) st[i].m = kNegInf;
#pragma unroll
    for (int i = 0; i < kNt; ++i) {
      if (wave_has && 16 * (ws.grp * kNt + i) < nrows) {
        float* c = comb_slot(wave, i);
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt)
          *reinterpret_cast<f32x4*>(c + ln * G::comb_row + 16 * dt + 4 * lq) = st[i].o[dt];
        if (lq == 0) {
          c[kTok * G::comb_row + ln] = st[i].m;
          c[kTok * G::comb_row + kTok + ln] = st[i].l;
        }
      }
    }
    __syncthreads();
    TTS_PROF_MARK(6, rec_idx);
    // Thread (tile, row, c), sixteen to a row, even tiles by the first four
    // waves and odd ones by the others: stored elements (D / 16) c .. of the
    // row, which are dimensions 16 t + 4 q + j (partial states' lane order).
    {
#pragma unroll
      for (int r = 0; r < kTiles; ++r) {
        if ((r & 1) != (wave >> 2) || 16 * r >= nrows) continue;  // wave-uniform
        constexpr int kEl = D / 16;
        const int c16 = ln, rrow = (tid >> 4) & 15, row = 16 * r + rrow;
        const int q4 = c16 >> 2, tt = (c16 & 3) * (kEl / 4);
        const int w0 = group_first(ws, r / kNt), ns = nsrc[r / kNt], ti = r % kNt;
        float mx, l;
        f32x4 o[kEl / 4];
        combine_row<D, KV, kWaves>([&](int k) { return comb_slot(w0 + k, ti); }, ns, rrow, c16, o, mx, l);
        const bool bad = ((bad_rows >> row) & 1ull) != 0;
        const float inv = l > 0.f ? 1.f / l : 0.f;
        if (paged && p.paged_nsplit == 1) {
          // Whole sequence in this unit: the normalised result.
          if (row < nrows) {
            float* orow = p.out + (static_cast<int64_t>(paged_b) * p.hq + kvh * p.g + row) * D;
            const float qnan = __builtin_nanf("");
#pragma unroll
            for (int e = 0; e < kEl / 4; ++e) {
              f32x4 v = o[e] * inv;
              if (bad) v = f32x4{qnan, qnan, qnan, qnan};
              *reinterpret_cast<f32x4*>(orow + 16 * (tt + e) + 4 * q4) = v;
            }
          }
        } else {
          int64_t prow;
          if (paged)
            prow = (static_cast<int64_t>(paged_b) * p.paged_nsplit + paged_split) * p.hq + kvh * p.g + row;
          else
            prow = static_cast<int64_t>(kvh) * p.rows_per_head + prow0 + row;
          store_partial_row<D, KV>(p.part_o, p.part_ml, prow, o, bad ? __builtin_nanf("") : mx, l, inv, c16,
                                   row < nrows);
        }
      }
    }
#ifdef TTS_PROFILE_UNITS
    TTS_PROF_MARK(2, rec_idx);
    if (KV != kKvF32 && threadIdx.x == 0 && rec_idx < kProfSlots)
      g_prof[rec_idx][3] = (static_cast<uint64_t>(__builtin_amdgcn_s_getreg((3 << 11) | 20)) << 32) |
                           static_cast<uint32_t>(__builtin_amdgcn_s_getreg((31 << 11) | 4));
#endif
    if (nu_rows <= 0) break;
    rec_idx = unext;
    u = nu;
  }
}

// ---- the paged path, up to 16 query heads per KV head ------------------------
// One workgroup of four waves per (split of up to 32 blocks, KV head, beam):
// one row tile, query rows held in registers, each wave streaming its share
// of the pairs. Three workgroups share a compute unit (at most 168 registers
// and 36 KB of LDS each), so that one's round trips to the length, the table
// and its first blocks run beside another's streaming. The units are ordered
// by (split, KV head) with the beams next to each other and dealt to the
// XCDs in eight contiguous runs: beams of one prefix read its blocks through
// one L2 at about the same time. Paged call on the 7B 64-beam tree: 87 ->
// 51 us (eight waves, one workgroup per compute unit, splits next to each
// other), 10 TB/s of logical KV.
constexpr int kPagedWaves = 4;
constexpr int kPagedRows = 16;
constexpr int kXcds = 8;

template <int D, int KV>
__global__ __launch_bounds__(64 * kPagedWaves, KV == kKvF32 && D == 128 ? 2 : 3) void paged_kernel(AttnParams p) {
  using G = Geo<D, KV>;
  __shared__ __attribute__((aligned(16))) float comb[kPagedWaves * G::comb_floats];
  const unsigned total = static_cast<unsigned>(p.num_seqs) * p.hkv * p.paged_nsplit;
  const unsigned at = blockIdx.x % kXcds * ((total + kXcds - 1) / kXcds) + blockIdx.x / kXcds;
  if (at >= total) return;
  const int unit = static_cast<int>(at);
  const int b = unit % p.num_seqs, kvh = unit / p.num_seqs % p.hkv, split = unit / p.num_seqs / p.hkv;
  const int wave = rfl(static_cast<int>(threadIdx.x) >> 6);
  const int lane = threadIdx.x & 63, ln = lane & 15, lq = lane >> 4;
  const size_t blk_stride = static_cast<size_t>(p.hkv) * G::blk_bytes;
  const unsigned char* kbase = static_cast<const unsigned char*>(p.k_cache) + kvh * G::blk_bytes;
  const unsigned char* vbase = static_cast<const unsigned char*>(p.v_cache) + kvh * G::blk_bytes;
  // Split j covers blocks [j * per, (j + 1) * per) of the beam (per <= 32).
  const int per = (p.paged_max_len + kTok * p.paged_nsplit - 1) / (kTok * p.paged_nsplit);
  const int j = split * per + lane;
  // Length and query rows together; the table only up to the length.
  const int L = p.seq_lens[b];
  QFrag<D, KV> q;
  {
    constexpr int kRowBytes = D * (KV == kKvF32 ? 4 : 2);
    const unsigned char* row = static_cast<const unsigned char*>(p.q) +
                               (static_cast<int64_t>(b) * p.hq + kvh * p.g + (ln < p.g ? ln : 0)) * kRowBytes;
#pragma unroll
    for (int i = 0; i < KOps<D, KV>::kk; ++i)
      q.q[i] = *reinterpret_cast<const typename KOps<D, KV>::T*>(row + (4 * i + lq) * 16);
  }
  int nb = (L + kTok - 1) / kTok;
  bool bad = false;
  if (L < 0 || L > p.paged_max_len || nb > p.max_blocks) {
    bad = true;
    nb = 0;
  }
  int n = nb - split * per;
  n = n < 0 ? 0 : (n < per ? n : per);
  int id = 0, v = 0;
  if (lane < n) {
    id = p.block_tables[static_cast<int64_t>(b) * p.max_blocks + j];
    v = L - j * kTok;
    v = v < kTok ? v : kTok;
  }
  if (lane >= n || id < 0 || id >= p.num_blocks) {
    bad |= lane < n;
    id = 0;
    v = 0;
  }
  bad = __builtin_amdgcn_ballot_w64(bad) != 0;
  if (p.num_blocks <= 0) n = 0;  // no block to read at all
  Window win;
  win.id = id;
  win.w = win_word(0, p.g, v);
  win.ks = 1.f;
  win.vs = 1.f;
  if constexpr (KV == kKvFp8) {
    if (v > 0) {
      win.ks = p.k_scale[id];
      win.vs = p.v_scale[id];
    }
  }
  const int np = (n + 1) >> 1;
  RowState<D> st;
  float m_exact = 0.f;
  for (int attempt = 0;; ++attempt) {
#pragma unroll
    for (int i = 0; i < D / 16; ++i) st.o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    st.m = m_exact;
    st.l = 0.f;
    st.seen = kNegInf;
    Frags<D, KV> f;
    for (int pp = wave; pp < np; pp += kPagedWaves) {
      issue_pair<D, KV>(f, win, n, pp, kbase, vbase, blk_stride, ln, lq);
      const int i0 = 2 * pp, i1 = 2 * pp + 1;
      const bool has1 = i1 < n;
      PairInfo pi;
      pi.v0 = win_valid(rl(win.w, i0));
      pi.v1 = has1 ? win_valid(rl(win.w, i1)) : 0;
      pi.a0 = pi.a1 = 0;
      pi.e0 = pi.e1 = kPagedRows;  // rows past g repeat row 0 and are not written
      pi.ks0 = pi.ks1 = p.scale_log2;
      pi.vs0 = pi.vs1 = 1.f;
      if constexpr (KV == kKvFp8) {
        pi.ks0 = p.scale_log2 * rlf(win.ks, i0);
        pi.vs0 = rlf(win.vs, i0);
        pi.ks1 = has1 ? p.scale_log2 * rlf(win.ks, i1) : pi.ks0;
        pi.vs1 = has1 ? rlf(win.vs, i1) : pi.vs0;
      }
      if (pi.v0 <= 0 && pi.v1 <= 0) continue;
      const Scores s = tile_scores<D, KV>(k_ops<D, KV>(f), q);
      const Probs<KV> pr = tile_probs<D, KV>(s, st, pi, 0, ln, lq);
      VOps<D, KV> vo = v_ops<D, KV>(f);
      if (pi.v0 < kTok || pi.v1 < kTok) mask_v<D, KV>(vo, lq, pi.v0, pi.v1);
      tile_values<D, KV>(vo, pr, st);
    }
    if (attempt > 0) break;
    const float mx = xlane_max16(st.seen);
    const bool redo = mx > kRefWindow || (mx < -kRefWindow && mx != kNegInf);
    m_exact = mx == kNegInf ? 0.f : mx;
    if (__builtin_amdgcn_ballot_w64(redo) == 0) break;
  }
  // The waves' states through LDS, sixteen threads to a row (as in
  // attn_kernel).
  auto slot = [&](int w) { return comb + w * G::comb_floats; };
  st.l = xlane_sum16(st.l);
  if (!(st.l > 0.f)) st.m = kNegInf;
  if (wave < np) {
    float* c = slot(wave);
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt)
      *reinterpret_cast<f32x4*>(c + ln * G::comb_row + 16 * dt + 4 * lq) = st.o[dt];
    if (lq == 0) {
      c[kTok * G::comb_row + ln] = st.m;
      c[kTok * G::comb_row + kTok + ln] = st.l;
    }
  }
  __syncthreads();
  constexpr int kEl = D / 16;
  const int row = static_cast<int>(threadIdx.x) >> 4;
  float mx, l;
  f32x4 o[kEl / 4];
  combine_row<D, KV, kPagedWaves>(slot, np < kPagedWaves ? np : kPagedWaves, row, ln, o, mx, l);
  const float inv = l > 0.f ? 1.f / l : 0.f;
  const float qnan = __builtin_nanf("");
  if (p.paged_nsplit == 1) {
    // Whole sequence in this unit: the normalised result.
    if (row < p.g) {
      float* orow = p.out + (static_cast<int64_t>(b) * p.hq + kvh * p.g + row) * D;
#pragma unroll
      for (int e = 0; e < kEl / 4; ++e) {
        f32x4 x = o[e] * inv;
        if (bad) x = f32x4{qnan, qnan, qnan, qnan};
        *reinterpret_cast<f32x4*>(orow + 16 * ((ln & 3) * (kEl / 4) + e) + 4 * (ln >> 2)) = x;
      }
    }
  } else {
    const int64_t prow = (static_cast<int64_t>(b) * p.paged_nsplit + split) * p.hq + kvh * p.g + row;
    store_partial_row<D, KV>(p.part_o, p.part_ml, prow, o, bad ? qnan : mx, l, inv, ln, row < p.g);
  }
}

// Exact merge of the partial softmax states of each (beam, query head), in
// the order of the beam's slot list. With M = max_k m_k over the states
// that saw tokens (l_k > 0), w_k = l_k 2^(m_k - M), and e_k the stored
// elements with factor z_k (e_k z_k = o_k / l_k):
//   out = sum_k w_k z_k e_k / sum_k w_k.
// A slot-table row of zeros for the paged path, which has no table (the
// merges read their table entries without a branch).
__device__ const int kZeroTabRow[kSlotTabReadAhead] = {};

// One wave per row, D / 64 elements per lane, bound by
// its chain of memory round trips: the table row, then the states. Lane j
// holds slot j's table entry (the row's first 64 in one load, with its
// count and the beam's lengths), reads slot j's (m, l, z) and computes its
// weight, once per slot and not once per lane; the elements of up to
// kMergeRound slots are loaded in the same round trip and weighed with the
// lanes' weights as scalars: two round trips for up to 32 slots, one more
// for each 32 further. Against 16 slots per round trip with every weight
// computed by every lane, and a kernel of sixteen lanes per row above 4,096
// rows: 7B 64-beam tree 24.2 -> 23.65 us per call (1,792 rows of 13 slots),
// balanced tree 51.1 -> 49.7, straggler batch 88.7 -> 87.5 (7,168 rows),
// paged 64-beam call 106.1 -> 102.9.
constexpr int kMergeThreads = 256;
constexpr int kMergeRound = 32;  // slots whose elements are loaded together

__device__ __forceinline__ float wave_max(float x) {
  x = row16_max(x);
  return fmaxf(fmaxf(rlf(x, 0), rlf(x, 16)), fmaxf(rlf(x, 32), rlf(x, 48)));
}

// Sum over the wave, in a fixed order.
__device__ __forceinline__ float wave_sum(float x) {
  auto ror = [](float v, auto n) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),
                                                                 0x120 | decltype(n)::value, 0xf, 0xf, false));
  };
  x += ror(x, std::integral_constant<int, 8>{});
  x += ror(x, std::integral_constant<int, 4>{});
  x += ror(x, std::integral_constant<int, 2>{});
  x += ror(x, std::integral_constant<int, 1>{});
  return (rlf(x, 0) + rlf(x, 16)) + (rlf(x, 32) + rlf(x, 48));
}

// One lane's stored elements of a row: D / 64 of them, fp16 or fp32.
template <int D, bool F16>
struct RowElems {
  static constexpr int kEl = D / 64;
  typedef typename std::conditional<F16, _Float16, float>::type E;
  typedef E V __attribute__((ext_vector_type(kEl)));
  V v;
};
template <bool F16>
struct RowElems<64, F16> {
  static constexpr int kEl = 1;
  typedef typename std::conditional<F16, _Float16, float>::type E;
  E v[1];
};

template <int D, bool F16>
__global__ __launch_bounds__(kMergeThreads) void merge_kernel(MergeParams p) {
  using R = RowElems<D, F16>;
  constexpr int kEl = R::kEl;
  const int lane = threadIdx.x & 63;
  const int r = rfl(static_cast<int>(blockIdx.x) * (kMergeThreads / 64) + static_cast<int>(threadIdx.x >> 6));
  if (r >= p.num_seqs * p.hq) return;
  const int b = r / p.hq;
  const int h = r % p.hq;
  // The row's inputs in one round trip: its table row (the paged path reads
  // a row of zeros), its live length and its build-time length (the paged
  // path, which has none, reads the live one again). The entries are read
  // past the count (the table's read-ahead zeros keep that in bounds).
  const int* tab = p.slot_tab ? p.slot_tab + static_cast<int64_t>(b) * p.slot_stride : kZeroTabRow;
  int ent = tab[1 + lane];
  const int n = p.slot_tab ? rfl(tab[0]) : p.paged_nsplit;
  const int head_base = p.slot_tab ? (h / p.g) * p.rows_per_head + h % p.g : 0;
  const int L = beam_len(p, b);
  const int blen = (p.build_len ? p.build_len : p.seq_lens)[b];
  bool nan = p.build_len && L < blen;
  float mx = kNegInf, den = 0.f;
  float acc[kEl];
#pragma unroll
  for (int e = 0; e < kEl; ++e) acc[e] = 0.f;
  for (int k0 = 0; k0 < n; k0 += 64) {
    const int left = n - k0 < 64 ? n - k0 : 64;  // slots of this round
    if (k0 > 0) ent = p.slot_tab && lane < left ? tab[1 + k0 + lane] : 0;
    // Lane j: slot k0 + j (past the end: a repeat of slot k0, with no weight).
    const int j = lane < left ? lane : 0;
    const int first = rfl(ent);
    const int row_j = p.slot_tab ? head_base + (lane < left ? ent : first)
                                 : (b * p.paged_nsplit + k0 + j) * p.hq + h;
    f32x4 ml = *reinterpret_cast<const f32x4*>(p.part_ml + static_cast<int64_t>(row_j) * kPartMl);
    R o[kMergeRound];
    auto load = [&](int c0, int c1) {  // slots c0 .. c1 of the round (c1 - c0 <= kMergeRound)
#pragma unroll
      for (int k = 0; k < kMergeRound; ++k) {
        if (k % 8 == 0 && c0 + k >= c1) break;  // uniform
        const int64_t row = rl(row_j, c0 + k);
        o[k] = *reinterpret_cast<const R*>(static_cast<const typename R::E*>(p.part_o) + row * D + kEl * lane);
      }
    };
    load(0, left);
    if (lane >= left) ml = f32x4{kNegInf, 0.f, 0.f, 0.f};
    if (ml.y == 0.f && ml.x == ml.x) ml.x = kNegInf;  // a state without tokens
    nan |= __builtin_amdgcn_ballot_w64(ml.x != ml.x) != 0;
    const float mn = fmaxf(mx, wave_max(ml.x));
    if (mn == kNegInf) continue;
    const float a = (mx == kNegInf) ? 0.f : __builtin_amdgcn_exp2f(mx - mn);
    const float w = (ml.x == kNegInf) ? 0.f : ml.y * __builtin_amdgcn_exp2f(ml.x - mn);
    const float wz = w * ml.z;
    den = den * a + wave_sum(w);
#pragma unroll
    for (int e = 0; e < kEl; ++e) acc[e] *= a;
    auto add = [&](int c0, int c1) {
#pragma unroll
      for (int k = 0; k < kMergeRound; ++k) {
        if (k % 8 == 0 && c0 + k >= c1) break;
        if (c0 + k < c1) {  // uniform (past the end: a repeat, whose weight of 0 could meet an infinity)
          const float wk = rlf(wz, c0 + k);
#pragma unroll
          for (int e = 0; e < kEl; ++e) acc[e] = __builtin_fmaf(static_cast<float>(o[k].v[e]), wk, acc[e]);
        }
      }
    };
    add(0, left);
    if (left > kMergeRound) {
      load(kMergeRound, left);
      add(kMergeRound, left);
    }
    mx = mn;
  }
  const float inv = (den > 0.f && L > 0) ? 1.f / den : 0.f;
  // Stored position pos holds dimension 16 t + 4 q + i for pos = (D / 4) q + 4 t + i.
  const int pos = kEl * lane;
  const int dim = 16 * ((pos % (D / 4)) / 4) + 4 * (pos / (D / 4)) + pos % 4;
  float* dst = p.out + static_cast<int64_t>(r) * D + dim;
  const float q = __builtin_nanf("");
  if constexpr (kEl == 2) {
    *reinterpret_cast<f32x2*>(dst) = nan ? f32x2{q, q} : f32x2{acc[0] * inv, acc[1] * inv};
  } else {
    *dst = nan ? q : acc[0] * inv;
  }
}

// A launch holds fewer than 2^32 threads; calls of more are made in runs of
// whole beams.
constexpr int64_t kMaxLaunchThreads = 0xFFFFFFFFll;

// The paged path. (More than 16 query heads per KV head: several row tiles.)
template <int D, int KV>
static hipError_t launch_paged_t(AttnParams p, hipStream_t stream) {
  const bool small = p.g <= kPagedRows;
  const int threads = small ? 64 * kPagedWaves : kThreads;
  const int64_t per = static_cast<int64_t>(p.hkv) * p.paged_nsplit;  // workgroups of a beam
  const int64_t fit = kMaxLaunchThreads / threads / kXcds * kXcds / per, most = fit > 1 ? fit : 1;
  const int64_t q_beam = static_cast<int64_t>(p.hq) * D * (KV == kKvF32 ? 4 : 2);
  for (int64_t left = p.num_seqs; left > 0; left -= most) {
    const int64_t n = left < most ? left : most;
    p.num_seqs = static_cast<int32_t>(n);
    const unsigned grid = static_cast<unsigned>(n * per);
    if (small)
      hipLaunchKernelGGL((paged_kernel<D, KV>), dim3((grid + kXcds - 1) / kXcds * kXcds), dim3(threads), 0, stream, p);
    else
      hipLaunchKernelGGL((attn_kernel<D, KV, false, true>), dim3(grid), dim3(threads), 0, stream, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    p.q = static_cast<const char*>(p.q) + n * q_beam;
    p.block_tables += n * p.max_blocks;
    p.seq_lens += n;
    p.out += n * p.hq * D;
    if (p.paged_nsplit > 1) {
      const int64_t rows = n * p.paged_nsplit * p.hq;
      p.part_o = static_cast<char*>(p.part_o) + rows * D * (KV == kKvF32 ? 4 : 2);
      p.part_ml += rows * kPartMl;
    }
  }
  return hipSuccess;
}

template <int D, int KV>
static hipError_t launch_attn_t(const AttnParams& p, int grid, hipStream_t stream) {
  if (p.recs == nullptr) return launch_paged_t<D, KV>(p, stream);
  if (p.two_windows)
    hipLaunchKernelGGL((attn_kernel<D, KV, true, false>), dim3(grid), dim3(kThreads), 0, stream, p);
  else
    hipLaunchKernelGGL((attn_kernel<D, KV, false, false>), dim3(grid), dim3(kThreads), 0, stream, p);
  return hipGetLastError();
}

template <int D, bool F16>
static hipError_t launch_merge_t(MergeParams p, hipStream_t stream) {
  constexpr int kPer = kMergeThreads / 64;  // rows per workgroup
  // (Whole beams, and whole beams' virtual ones.)
  const int64_t fit = kMaxLaunchThreads / kMergeThreads * kPer / p.hq / p.q_len * p.q_len;
  const int64_t most = fit > p.q_len ? fit : p.q_len;
  for (int64_t left = p.num_seqs; left > 0; left -= most) {
    const int64_t n = left < most ? left : most;
    p.num_seqs = static_cast<int32_t>(n);
    const unsigned grid = static_cast<unsigned>((n * p.hq + kPer - 1) / kPer);
    hipLaunchKernelGGL((merge_kernel<D, F16>), dim3(grid), dim3(kMergeThreads), 0, stream, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    p.seq_lens += n / p.q_len;
    p.out += n * p.hq * D;
    if (p.slot_tab) {
      p.slot_tab += n * p.slot_stride;
      p.build_len += n;
    } else {
      const int64_t rows = n * p.paged_nsplit * p.hq;
      p.part_o = static_cast<const char*>(p.part_o) + rows * D * (F16 ? 2 : 4);
      p.part_ml += rows * kPartMl;
    }
  }
  return hipSuccess;
}

hipError_t launch_merge(const MergeParams& p, int head_dim, int kv_kind, hipStream_t stream) {
  const bool f16 = kv_kind != kKvF32;
  if (head_dim == 128) return f16 ? launch_merge_t<128, true>(p, stream) : launch_merge_t<128, false>(p, stream);
  return f16 ? launch_merge_t<64, true>(p, stream) : launch_merge_t<64, false>(p, stream);
}

hipError_t launch_attn(const AttnParams& p, int grid, int head_dim, int kv_kind, hipStream_t stream) {
  if (grid <= 0) return hipSuccess;
  if (head_dim == 128) {
    if (kv_kind == kKvBf16) return launch_attn_t<128, kKvBf16>(p, grid, stream);
    if (kv_kind == kKvFp8) return launch_attn_t<128, kKvFp8>(p, grid, stream);
    return launch_attn_t<128, kKvF32>(p, grid, stream);
  }
  if (kv_kind == kKvBf16) return launch_attn_t<64, kKvBf16>(p, grid, stream);
  if (kv_kind == kKvFp8) return launch_attn_t<64, kKvFp8>(p, grid, stream);
  return launch_attn_t<64, kKvF32>(p, grid, stream);
}

// ---- scratch of the allocation-free entry point ----------------------------
// Partial softmax states of one prefix-attention call for callers that cannot
// allocate device memory. The array is part of the code object: every GPU
// the library runs on holds its own copy, at its own address, until the
// process ends. In host code the name `scratch` is only a stand-in; the
// device address comes from hipGetSymbolAddress, looked up once per device
// with that device current.
__device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kScratchMaxDevices = 64;

hipError_t scratch_buffer(void** ptr, size_t* bytes) {
  static std::mutex mu;
  static void* dev_ptr[kScratchMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kScratchMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!dev_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    dev_ptr[dev] = p;
  }
  *ptr = dev_ptr[dev];
  *bytes = kScratchBytes;
  return hipSuccess;
}

}  // namespace tts

#ifdef TTS_PROFILE_UNITS
extern "C" int tts_prof_read(uint64_t* host, int n) {
  if (n > tts::kProfSlots) n = tts::kProfSlots;
  return static_cast<int>(hipMemcpyFromSymbol(host, HIP_SYMBOL(tts::g_prof), sizeof(uint64_t) * 8 * n, 0,
                                              hipMemcpyDeviceToHost));
}
extern "C" int tts_prof_clear() {
  static uint64_t zeros[tts::kProfSlots][8];
  return static_cast<int>(hipMemcpyToSymbol(HIP_SYMBOL(tts::g_prof), zeros, sizeof(zeros), 0, hipMemcpyHostToDevice));
}
#endif
