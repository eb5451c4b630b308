// What the kernels of scheme U's compressor share: scale and reciprocal of a range, quantizing (U2),
// packing of codes (U3).
#pragma once

#include "common.hpp"

namespace accept {
namespace {

constexpr float kTinyRange = 0x1p-100f;     // smaller ranges count as an all-zero tensor
constexpr float kRoundMagic = 12582912.0f;  // 1.5 * 2^23: adding it rounds to integer, half to even

// s = c / L and r = L / c as correctly rounded float32 quotients (L is a small integer, exact in
// float32; __fdiv_rn is the IEEE round-to-nearest-even division).
__device__ __forceinline__ void scale_from_range(float c, int k, float& s, float& r) {
  const float L = float((1 << (k - 1)) - 1);
  if (c >= kTinyRange) {
    s = __fdiv_rn(c, L);
    r = __fdiv_rn(L, c);
  } else {
    s = 0.0f;
    r = 0.0f;
  }
}

// =========================================================================== quantize (U2)
// One element, round half to even: v = x * r (one float32 multiply), round, clamp, offset to a
// k-bit code.  The _raw form leaves other bits above the low k.
template <int K>
__device__ __forceinline__ uint32_t quantize_rne_raw(float f, float r) {
  constexpr int HALF = 1 << (K - 1);
  const float v = __fmul_rn(f, r);
  // Round half to even through the magic-number add.  |v| <= L(1 + 2^-23), so the rounded
  // value lies in [-L, L] and the clamp of the definition never binds; taking k bits only keeps
  // codes of non-finite inputs inside them.  The sum's low mantissa bits are q + HALF (k < 8) or
  // q mod 256 (k = 8).
  return f32_as_u32(__fadd_rn(v, kRoundMagic + float(K == 8 ? 0 : HALF)));
}
template <int K>
__device__ __forceinline__ uint32_t quantize_rne(float f, float r) {
  return quantize_rne_raw<K>(f, r) & ((1u << K) - 1u);
}

// One element, stochastic: floor(v) + (u < v - floor(v)), clamped; the signed value.  z is the
// element's random state.  TILES: an element of a whole tile (see mad_low).
template <bool TILES>
__device__ __forceinline__ int quantize_stochastic(float f, float r, int half, uint64_t z) {
  const float v = __fmul_rn(f, r);
  const float fl = floorf(v);
  const float pr = __fsub_rn(v, fl);
  const int q = int(fl) + (rand_u32<TILES>(z) < pr * 0x1p32f ? 1 : 0);
  return min(max(q, -half), half - 1);
}

// Four consecutive elements -> one 4k-bit piece in the top bits of a dword (zeros below), first
// element most significant.  z0: random state of the first (stochastic rounding only).
// The codes enter from the top, last element first: one funnel shift per element takes the low k
// bits of the sum (whatever stands above them) and moves the earlier ones down.
template <int K, bool STOCH>
__device__ __forceinline__ uint32_t quantize4(const float* f, const float* r, uint64_t z0) {
  constexpr int HALF = 1 << (K - 1);
  uint32_t piece = 0;
#pragma unroll
  for (int e = 3; e >= 0; --e) {
    uint32_t code;
    if constexpr (STOCH)
      code = uint32_t(quantize_stochastic<true>(f[e], r[e], HALF, z0 + uint64_t(e) * kRandStep));
    else
      code = quantize_rne_raw<K>(f[e], r[e]);
    piece = __builtin_amdgcn_alignbit(code, piece, K);
  }
  if constexpr (STOCH && K < 8) {  // two's complement -> offset binary: flip the top bit of each field
    constexpr uint64_t TOP = uint64_t(HALF) * (1ull + (1ull << K) + (1ull << (2 * K)) + (1ull << (3 * K)));
    piece ^= uint32_t(TOP << (32 - 4 * K));
  }
  return piece;
}

// U3: a group of 32 consecutive codes, eight 4k-bit pieces (in the top bits of a dword each), is k dwords of the
// big-endian bit stream, each byte-swapped into memory order.  A thread packs one part of it at a time: the
// largest of whole dwords that one store instruction takes (k = 8 and 6: half a group, 4 and 3 dwords), so that the
// 64 lanes' parts lie together in memory, or the whole group (k = 5 and 7 have no such parts).
template <int K>
struct CodeParts {
  static constexpr int PARTS = K == 6 || K == 8 ? 2 : 1;
  static constexpr int PIECES = 8 / PARTS, DWORDS = K / PARTS;
};
template <int K>
__device__ __forceinline__ void pack_part(const uint32_t* pieces, uint32_t (&out)[CodeParts<K>::DWORDS]) {
  constexpr int W = 4 * K, NP = CodeParts<K>::PIECES;
  uint32_t P[NP];
#pragma unroll
  for (int i = 0; i < NP; i += 4) {
    const uint4 v = *reinterpret_cast<const uint4*>(&pieces[i]);
    P[i] = v.x; P[i + 1] = v.y; P[i + 2] = v.z; P[i + 3] = v.w;
  }
#pragma unroll
  for (int o = 0; o < CodeParts<K>::DWORDS; ++o) {
    uint32_t w = 0;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int at = W * i - 32 * o;  // first bit of the piece, counted from the dword's first bit
      if (at >= 0 && at < 32) w |= P[i] >> at;
      if (at < 0 && at > -W) w |= P[i] << -at;
    }
    out[o] = __builtin_bswap32(w);
  }
}
// Stores a part at byte `at` of the buffer; where the lanes' parts lie together, through the cache.
// Plain / streaming / written through (us): held pass, 103 MB float32, k = 4 27.7 / 25.7 / 25.5 and with
// the decoder behind it 46.4 / 46.2 / 44.6; 64 x 256 x 3136 bfloat16 with a range per channel, k = 6 33.6 / 30.3 / 30.4 and
// 55.3 / 60.5 / 52.7; stochastic, 205 MB, k = 4 84.9 plain, 81.0.  (With parts that do not lie together, k = 8 as
// whole groups: 30.6 plain, 32.2 written through.)
template <int K>
__device__ __forceinline__ void store_part(__amdgpu_buffer_rsrc_t payload, uint32_t at, const uint32_t (&v)[CodeParts<K>::DWORDS]) {
  constexpr int ND = CodeParts<K>::DWORDS;
  if constexpr (ND <= 4) {
    store_through<ND>(payload, at, v);
  } else {
    typedef uint32_t v3u_t __attribute__((ext_vector_type(3)));
    __builtin_amdgcn_raw_buffer_store_b128(v4u_t{v[0], v[1], v[2], v[3]}, payload, at, 0, 0);
    if constexpr (ND == 5) __builtin_amdgcn_raw_buffer_store_b32(v[4], payload, at + 16, 0, 0);
    if constexpr (ND == 7) __builtin_amdgcn_raw_buffer_store_b96(v3u_t{v[4], v[5], v[6]}, payload, at + 16, 0, 0);
  }
}

// k-bit code of a signed value.
__device__ __forceinline__ uint32_t code_of_q(int q, int k) {
  return k == 8 ? (uint32_t(q) & 0xFFu) : uint32_t(q + (1 << (k - 1)));
}

// Slow path for one group of 8 elements -> k bytes (tails and odd channel geometries):
// scalar loads, per-byte stores guarded by the payload size.  Elements at or beyond N
// contribute zero bits.
template <typename T, int K, bool STOCH, typename RFn>
__device__ __forceinline__ void quantize_group8(const T* __restrict__ x, uint8_t* __restrict__ payload, int64_t grp,
                                                int64_t N, int64_t payload_bytes, uint64_t seed, RFn r_of) {
  uint64_t acc = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int64_t i = grp * 8 + e;
    uint64_t code = 0;
    if (i < N) {
      const float f = load_one(x + i), r = r_of(i);
      code = STOCH ? code_of_q(quantize_stochastic<false>(f, r, 1 << (K - 1), rand_state(seed, uint64_t(i))), K)
                   : quantize_rne<K>(f, r);
    }
    acc = (acc << K) | code;
  }
#pragma unroll
  for (int b = 0; b < K; ++b) {
    const int64_t byte = grp * K + b;
    if (byte < payload_bytes) payload[byte] = uint8_t(acc >> (8 * (K - 1 - b)));
  }
}

}  // namespace
}  // namespace accept
