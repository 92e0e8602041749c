// KV-cache maintenance around the decode step: appending each beam's new
// token to its block (with the fp8 block-scale policy) and copying blocks
// for copy-on-write beam duplication.
//
// A decode step of the search writes one token per beam into the paged
// cache before attention reads it (the current token is part of seq_len),
// and a duplicated beam shares its parent's full blocks while its partially
// filled last block is copied (DuplicateThenTruncate, Sec. 3.1 and Alg. 1;
// the duplicates' speculative tokens are truncated, Sec. 4.1).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace tts {
namespace {

constexpr int kKvThreads = 256;
constexpr int kSlots = 16;  // tokens per block

// Round-to-nearest-even OCP E4M3FN encoding of an fp32 value (already
// divided by its block scale), saturating at +-448 (code 0x7E); NaN gives
// 0x7F. Built from the format: subnormals are multiples of 2^-9 below 2^-6,
// normals keep 3 mantissa bits of the fp32 significand.
__device__ __forceinline__ uint32_t e4m3_encode(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  const uint32_t sign = (u >> 24) & 0x80u;
  const float a = __builtin_fabsf(x);
  if (a != a) return 0x7Fu;
  if (a >= 448.f) return sign | 0x7Eu;
  if (a < 0.015625f) {  // 2^-6: subnormal codes q * 2^-9, q in [0, 8]
    const uint32_t q = static_cast<uint32_t>(__builtin_rintf(a * 512.f));  // exact scaling, RNE
    return sign | q;
  }
  const uint32_t ua = __builtin_bit_cast(uint32_t, a);
  int e = static_cast<int>(ua >> 23) - 127;  // -6 .. 8
  uint32_t keep = (ua >> 20) & 7u;
  const uint32_t rest = ua & 0xFFFFFu;
  if (rest > 0x80000u || (rest == 0x80000u && (keep & 1u))) ++keep;
  if (keep == 8u) {
    keep = 0;
    ++e;
  }
  return sign | (static_cast<uint32_t>(e + 7) << 3) | keep;
}

__device__ __forceinline__ float e4m3_decode(uint32_t code) {
  return __builtin_amdgcn_cvt_f32_fp8(static_cast<int>(code), 0);  // exact
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  return __builtin_bit_cast(float, static_cast<uint32_t>(b) << 16);
}

__device__ __forceinline__ float block_max(float v, float* red) {
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  const int w = threadIdx.x >> 6;
  __syncthreads();  // red is free (a previous reduction is done with it)
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  float m = red[0];
  for (int i = 1; i < kKvThreads / 64; ++i) m = fmaxf(m, red[i]);
  return m;
}

struct AppendParams {
  const void* k_new;  // [S][Hkv][D]: bf16 (bf16 and fp8 caches) or fp32
  const void* v_new;
  const int32_t* block_tables;
  const int32_t* seq_lens;
  void* k_cache;  // [NB][Hkv][16][D]
  void* v_cache;  // [NB][Hkv][D][16]
  float* k_scale;
  float* v_scale;
  int32_t max_blocks;
  int32_t num_blocks;
  int32_t hkv;
  int32_t head_dim;
};

// Elements of a token that a thread holds in registers (tokens of more are
// read again from memory).
constexpr int kHeld = 4;

// Sixteen codes of a 16-byte word, each of the first n through the table
// (and code `at`, if it is one of them, replaced by `code`).
__device__ __forceinline__ uint4 map_codes(uint4 x, const uint8_t* lut, int n, int at, uint32_t code) {
  uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t r = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int j = 4 * i + k;
      const uint32_t c = (w[i] >> (8 * k)) & 0xFFu;
      r |= (j == at ? code : (j < n ? lut[c] : c)) << (8 * k);
    }
    w[i] = r;
  }
  return uint4{w[0], w[1], w[2], w[3]};
}

// One tensor (K or V) of one beam's new token into an fp8 block: element
// i = h * D + d of the token to slot `slot` of head h, dim d. The block's
// scale is set from the token when the token opens the block (slot 0); when
// a later token exceeds the range of the current scale the scale grows to
// fit it and the block's earlier codes are re-encoded under the new scale.
//
// Bound by its chain of round trips (length, table, scale, earlier codes;
// the token and its maximum travel beside them) and by the re-encoding: the
// 256 codes' new values are computed once, one per thread, into a table in
// LDS, and the earlier codes go through it sixteen at a time. 512 beams, 512
// values per token, sixteen tokens: 12.5 -> 6.7 us per call (a conversion, a
// product and a division per code, a byte at a time, and the token read
// after the table).
template <bool kV>
__device__ void append_fp8(const float (&held)[kHeld], float amax, const uint16_t* src, int n, int slot,
                           float* scale_p, uint8_t* blk, int D, uint8_t* lut) {
  // (A cache that starts at no multiple of 16 bytes is re-encoded by bytes.)
  const bool wide = (reinterpret_cast<uintptr_t>(blk) & 15) == 0;
  const float s_old = *scale_p;
  float s = s_old;
  bool requant = false;
  if (slot == 0) {
    s = amax > 0.f ? amax / 448.f : 1.f;
  } else if (amax > 448.f * s_old) {
    s = amax / 448.f;
    requant = true;
  }
  if (requant) {
    lut[threadIdx.x] = static_cast<uint8_t>(e4m3_encode(e4m3_decode(threadIdx.x) * s_old / s));
    __syncthreads();
    if constexpr (!kV) {
      // Rows of D codes: the earlier slots of a head are contiguous.
      const int per = slot * D / 16, total = n / D * per;
      for (int c = threadIdx.x; c < total; c += kKvThreads) {
        uint8_t* x = blk + (c / per) * kSlots * D + c % per * 16;
        if (wide)
          *reinterpret_cast<uint4*>(x) = map_codes(*reinterpret_cast<const uint4*>(x), lut, 16, -1, 0);
        else
          for (int j = 0; j < 16; ++j) x[j] = lut[x[j]];
      }
    }
  }
  for (int k = 0, i = threadIdx.x; i < n; ++k, i += kKvThreads) {
    float v = k < kHeld ? 0.f : bf16_to_f32(src[i]);
#pragma unroll
    for (int j = 0; j < kHeld; ++j) v = k == j ? held[j] : v;
    const uint32_t code = e4m3_encode(v / s);
    if constexpr (kV) {
      // Row i holds the sixteen slots of one dimension.
      uint8_t* x = blk + static_cast<int64_t>(i) * kSlots;
      if (requant && wide) {
        *reinterpret_cast<uint4*>(x) = map_codes(*reinterpret_cast<const uint4*>(x), lut, slot, slot, code);
      } else {
        for (int j = 0; requant && j < slot; ++j) x[j] = lut[x[j]];
        x[slot] = static_cast<uint8_t>(code);
      }
    } else {
      blk[(static_cast<int64_t>(i / D) * kSlots + slot) * D + i % D] = static_cast<uint8_t>(code);
    }
  }
  __syncthreads();  // every thread has read s_old
  if (threadIdx.x == 0) *scale_p = s;
}

// Two workgroups per beam, one for K and one for V (their dependent steps
// run side by side): the beam's current token (position seq_len - 1) into
// slot (seq_len - 1) % 16 of its block. Beams with seq_len 0, a block index
// past the table row or a block id outside the pool write nothing.
template <int KV>  // 0 fp32, 1 bf16, 2 fp8
__global__ __launch_bounds__(kKvThreads) void append_kernel(AppendParams p) {
  __shared__ float red[kKvThreads / 64];
  __shared__ uint8_t lut[kKvThreads];
  typedef typename std::conditional<KV == 0, float, uint16_t>::type E;
  const int b = static_cast<int>(blockIdx.x >> 1);
  const bool is_v = (blockIdx.x & 1) != 0;
  const int D = p.head_dim, n = p.hkv * D;
  // The token is read beside the length and the table entry, not after them.
  const E* src = static_cast<const E*>(is_v ? p.v_new : p.k_new) + static_cast<int64_t>(b) * n;
  E tok[kHeld];
#pragma unroll
  for (int k = 0; k < kHeld; ++k) {
    const int i = threadIdx.x + kKvThreads * k;
    tok[k] = i < n ? src[i] : E{};
  }
  const int L = p.seq_lens[b];
  if (L <= 0) return;
  const int t = L - 1;
  const int lb = t / kSlots, slot = t % kSlots;
  if (lb >= p.max_blocks) return;
  const int blk = p.block_tables[static_cast<int64_t>(b) * p.max_blocks + lb];
  float held[kHeld], a = 0.f;
  if constexpr (KV == 2) {
#pragma unroll
    for (int k = 0; k < kHeld; ++k) {
      held[k] = bf16_to_f32(tok[k]);
      a = fmaxf(a, __builtin_fabsf(held[k]));
    }
    for (int i = threadIdx.x + kKvThreads * kHeld; i < n; i += kKvThreads)
      a = fmaxf(a, __builtin_fabsf(bf16_to_f32(src[i])));
    a = block_max(a, red);
  }
  if (blk < 0 || blk >= p.num_blocks) return;
  const int64_t base = static_cast<int64_t>(blk) * p.hkv;  // (block, head 0)
  if constexpr (KV == 2) {
    uint8_t* cache = static_cast<uint8_t*>(is_v ? p.v_cache : p.k_cache) + base * kSlots * D;
    if (is_v)
      append_fp8<true>(held, a, src, n, slot, p.v_scale + blk, cache, D, lut);
    else
      append_fp8<false>(held, a, src, n, slot, p.k_scale + blk, cache, D, lut);
  } else {
    E* dst = static_cast<E*>(is_v ? p.v_cache : p.k_cache) + base * kSlots * D;
    for (int k = 0, i = threadIdx.x; i < n; ++k, i += kKvThreads) {
      E v = k < kHeld ? E{} : src[i];
#pragma unroll
      for (int j = 0; j < kHeld; ++j) v = k == j ? tok[j] : v;
      dst[is_v ? static_cast<int64_t>(i) * kSlots + slot
               : (static_cast<int64_t>(i / D) * kSlots + slot) * D + i % D] = v;
    }
  }
}

struct CopyParams {
  const int32_t* pairs;  // [n][2]: source, destination block
  void* k_cache;
  void* v_cache;
  float* k_scale;
  float* v_scale;
  int64_t blk_bytes;  // bytes of one block of K (all KV heads), = V's
  int32_t num_blocks;
};

// K and V of every KV head (and the fp8 scales) of each pair's source block
// into its destination block. A workgroup copies one piece of kCopyBytes of
// one tensor, its two 16-byte loads per thread in flight together: bound by
// the memory and by the round trip to the pair and back (235 pairs of 32 KB:
// 8.1 -> 5.7 us; one workgroup per pair took four dependent rounds per
// tensor). Pairs naming a block outside the pool, or a block onto itself,
// copy nothing.
constexpr int kCopyBytes = kKvThreads * 32;
constexpr int kMaxGridY = 65535;

__global__ __launch_bounds__(kKvThreads) void copy_kernel(CopyParams p) {
  const int pair = static_cast<int>(blockIdx.y);
  const int src = p.pairs[2 * pair], dst = p.pairs[2 * pair + 1];
  if (src < 0 || src >= p.num_blocks || dst < 0 || dst >= p.num_blocks || src == dst) return;
  const bool is_v = (blockIdx.x & 1) != 0;
  unsigned char* cache = static_cast<unsigned char*>(is_v ? p.v_cache : p.k_cache);
  const int64_t n16 = p.blk_bytes / 16;
  const int64_t i0 = static_cast<int64_t>(blockIdx.x >> 1) * (kCopyBytes / 16) + threadIdx.x, i1 = i0 + kKvThreads;
  const uint4* s = reinterpret_cast<const uint4*>(cache + src * p.blk_bytes);
  uint4* d = reinterpret_cast<uint4*>(cache + dst * p.blk_bytes);
  uint4 x0, x1;
  if (i0 < n16) x0 = s[i0];
  if (i1 < n16) x1 = s[i1];
  if (i0 < n16) d[i0] = x0;
  if (i1 < n16) d[i1] = x1;
  if (blockIdx.x == 0 && threadIdx.x == 0 && p.k_scale) {
    p.k_scale[dst] = p.k_scale[src];
    p.v_scale[dst] = p.v_scale[src];
  }
}

}  // namespace

// (A launch holds fewer than 2^32 threads: calls of more beams are made in
// runs.)
constexpr int kMaxAppendBeams = 0xFFFFFFFFu / kKvThreads / 2;

template <int KV>
static hipError_t launch_append_t(AppendParams p, int num_seqs, hipStream_t stream) {
  const int64_t token = static_cast<int64_t>(p.hkv) * p.head_dim * (KV == 0 ? 4 : 2);
  for (int left = num_seqs; left > 0; left -= kMaxAppendBeams) {
    const int n = left < kMaxAppendBeams ? left : kMaxAppendBeams;
    hipLaunchKernelGGL(append_kernel<KV>, dim3(2 * n), dim3(kKvThreads), 0, stream, p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    p.k_new = static_cast<const char*>(p.k_new) + n * token;
    p.v_new = static_cast<const char*>(p.v_new) + n * token;
    p.block_tables += static_cast<int64_t>(n) * p.max_blocks;
    p.seq_lens += n;
  }
  return hipSuccess;
}

hipError_t launch_append(const void* k_new, const void* v_new, const int32_t* block_tables, const int32_t* seq_lens,
                         void* k_cache, void* v_cache, float* k_scale, float* v_scale, int num_seqs, int max_blocks,
                         int num_blocks, int hkv, int head_dim, int kv_kind, hipStream_t stream) {
  const AppendParams p{k_new, v_new, block_tables, seq_lens, k_cache, v_cache, k_scale, v_scale,
                       max_blocks, num_blocks, hkv, head_dim};
  if (kv_kind == 0) return launch_append_t<0>(p, num_seqs, stream);
  if (kv_kind == 1) return launch_append_t<1>(p, num_seqs, stream);
  return launch_append_t<2>(p, num_seqs, stream);
}

hipError_t launch_copy_blocks(const int32_t* pairs, int num_pairs, void* k_cache, void* v_cache, float* k_scale,
                              float* v_scale, int64_t blk_bytes, int num_blocks, hipStream_t stream) {
  if (num_pairs <= 0) return hipSuccess;
  CopyParams p{pairs, k_cache, v_cache, k_scale, v_scale, blk_bytes, num_blocks};
  const int pieces = static_cast<int>((blk_bytes + kCopyBytes - 1) / kCopyBytes);
  // Pairs along the grid's second dimension, at most 65,535 to a launch.
  for (int done = 0; done < num_pairs; done += kMaxGridY) {
    const int n = num_pairs - done < kMaxGridY ? num_pairs - done : kMaxGridY;
    p.pairs = pairs + 2 * static_cast<int64_t>(done);
    hipLaunchKernelGGL(copy_kernel, dim3(2 * pieces, n), dim3(kKvThreads), 0, stream, p);
  }
  return hipGetLastError();
}

}  // namespace tts
