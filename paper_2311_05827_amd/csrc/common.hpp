// Internal declarations shared by the HIP translation units of libaccept (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "accept.h"
#include "accept_profile.h"

namespace accept {

constexpr int kBlock = 256;       // threads per workgroup: 4 wavefronts of 64
constexpr int kWave = 64;
constexpr int kTileElems = 8192;  // elements one workgroup quantizes and packs per iteration

struct bf16_t {
  uint16_t bits;
};

template <typename T>
struct Elem;
template <>
struct Elem<float> {
  static constexpr int VEC = 4;  // elements per 16-byte vector
};
template <>
struct Elem<bf16_t> {
  static constexpr int VEC = 8;
};

// ---- event bracketing for the *_timed entry points -------------------------------------
struct StageTimer {
  hipEvent_t ev[ACCEPT_MAX_STAGES + 1];
  int n = 0;
  bool failed = false;
  void mark(hipStream_t s) {
    if (n > ACCEPT_MAX_STAGES) return;
    if (hipEventCreate(&ev[n]) != hipSuccess) { failed = true; return; }
    if (hipEventRecord(ev[n], s) != hipSuccess) failed = true;
    ++n;
  }
};
inline void mark(StageTimer* t, hipStream_t s) {
  if (t) t->mark(s);
}

// Every workspace starts with a control block that the library keeps between calls.  The caller zero-fills the
// workspace once; no kernel of either scheme writes anything else there.  It holds
// - the multi-bit encoder's work counters, which are zero when a call starts and are put back to zero before it ends,
//   and its count of finished workgroups, in the first half (see WorkQueue and last_workgroup in mbq.hip);
// - mailboxes, which nothing empties (see ChipMail): the second half, and between the counters.
constexpr size_t kCtrlBytes = 16384;
constexpr size_t kMailOffset = 8192;

// ---- scheme U (uniform) -----------------------------------------------------------------
enum UMode { U_TENSOR = 0, U_SEGMENTED = 1, U_GENERIC = 2 };

struct UPlan {
  int mode;
  int vec;             // elements per 16-byte vector of the input type
  int64_t N, m, C, seg_len;
  int range_grid;      // U_TENSOR: workgroups of the range kernel = number of partial maxima
  int64_t cps;         // U_SEGMENTED: chunks per segment
  int64_t chunk_vecs;  // U_SEGMENTED: 16-byte vectors per chunk
  int64_t items;       // U_SEGMENTED: n*C*cps partial maxima
  int col_tx;          // U_GENERIC: column threads per workgroup of the column pass (a power of two)
  int64_t col_grid_x;  // U_GENERIC: workgroups across the columns
  int col_grid_y;      // U_GENERIC: row blocks = maxima kept per column
  bool fast;           // vector path usable (every 16-byte vector lies inside one range group, or per_element, or straddling)
  bool local_ranges;   // U_SEGMENTED: the quantize pass finishes the per-channel ranges itself, tile by tile
  bool per_element;    // U_GENERIC: one element per segment and rows of whole vectors (channels-last)
  bool straddling;     // U_GENERIC: segments longer than a vector but not whole vectors
  bool held;           // U_TENSOR: the range pass keeps the end of the tensor on the chip and quantizes it itself
  int64_t held_units;  // held: whole units (see kUnitElems) of the tensor
  int held_lds;        // held: units per workgroup that stay in local memory (the others in registers)
  int64_t held_first;  // held: units [held_first, held_units) are kept, the others are read again
  uint32_t whole_per;  // U_TENSOR: groups of 32 elements per workgroup of the pass that keeps the tensor in registers; 0: not taken
  uint32_t chan_per;   // per channel: groups of 32 elements per workgroup of the pass that keeps the tensor on the chip; 0: not taken
  size_t off_rtab;     // byte offset of the per-channel reciprocal table in the workspace
  size_t bytes;        // workspace bytes
};

UPlan make_uplan(const accept_desc& d);
// Compute units of the current device (0 if there is none), and whether the held pass of a plan that
// has one runs on a device of that many: its 256 workgroups wait for each other, one per compute unit.
int compute_units();
constexpr int kHeldGrid = 256;
inline bool held_runs(const UPlan& p, int units) { return p.held && units >= kHeldGrid; }
inline bool whole_runs(const UPlan& p, int units) { return p.whole_per != 0 && units >= kHeldGrid; }
inline bool channels_run(const UPlan& p, int units) { return p.chan_per != 0 && units >= kHeldGrid; }

// What the workgroups of calls with one workspace leave each other, in its control block.  Every exchange of a
// call has a number of its own, and a value bears the number of its exchange, so nothing has to be emptied.
// How many exchanges there have been, every workgroup knows from a word of its own: it reads the word when it
// starts, and adds this call's exchanges before it ends (also to the words of the workgroups that this call does
// not have), so all of them agree.  It adds to the word, and does not store a sum: so the words agree again, and are
// ahead of every value left behind, even when calls that overlapped on one workspace, which they must not, have ended.
// (Counting the workgroups off on one counter, and the last one emptying everything, cost small tensors
// 1.5 us.)
struct ChipMail {
  uint64_t first[kHeldGrid], last[kHeldGrid];  // tag and the workgroup's maximum: of its first (or only), its last
                                               // channel; or tag and half of its sum (see mbq_first_kernel)
  uint64_t more[kHeldGrid];
  uint32_t calls[kHeldGrid];
};
static_assert(kMailOffset + sizeof(ChipMail) <= kCtrlBytes, "the control block holds them");
// Three more boxes for a workgroup lie between the multi-bit encoder's counters, in the first half of the block: the
// counters take the first 8 of 32 words of 64 bits, eight workgroups' boxes of a kind (0 .. 2) the next 8 each.
constexpr int kBetweenStride = 32;
static_assert(kHeldGrid / 8 * kBetweenStride * sizeof(uint64_t) <= kMailOffset, "in front of the mailboxes");

// held_polls: how often a workgroup of the held pass looks for the others' maxima before it gives up
// (kHeldPolls; fewer only where a test wants the case that it gives up).  64 looks take about 50 us.  Alone
// on the chip, 205 MB, 16 are too few (72.8 us a call) and 32 enough (56.8; 64: 55.8, the spread of the
// workgroups' ends being that of the memory); next to a kernel that fills the chip, more only keep
// compute units longer: 100 MB beside copies on another stream 92 us a call at 32, 94 at 64, 108 at 128,
// 130 at 512.
constexpr int kHeldPolls = 64;
hipError_t launch_uniform_compress(const accept_desc& d, const UPlan& p, const void* x, void* header,
                                   void* payload, void* ws, hipStream_t s, StageTimer* tm,
                                   int held_polls = kHeldPolls);
hipError_t launch_uniform_decompress(const accept_desc& d, const void* header, const void* payload,
                                     void* xhat, hipStream_t s, StageTimer* tm);

// ---- scheme M (multi-bit) ---------------------------------------------------------------
struct MPlan {
  int vec;                // columns per work item: those of a 16-byte vector, or 1 (the rule is at vec_for)
  int64_t G;              // ceil(n/8) row groups
  bool ragged;            // vectors, but rows are not whole ones: at any alignment, then m % vec single columns
  bool wide;              // a row group holds at least one full wave-item
  bool stream;            // wide, and complete row groups exist: row groups go through the pipelined stream
  bool mixed;             // the stream's last row group is a partial one
  uint32_t wpg;           // wave-items (64 items) per row group
  uint32_t n_wave_items;  // of the stream
  uint8_t queue_shift;    // a group of workgroups takes 1 << queue_shift of them out of a sweep
  int grid;               // workgroups of the encode kernel = number of partial-sum records
  bool direct;            // levels are found by comparisons, not through tables
  bool finish;            // the encode kernel also does the finalize kernel's work
  size_t bytes;
};

MPlan make_mplan(const accept_desc& d);

hipError_t launch_mbq_compress(const accept_desc& d, const MPlan& p, const void* x, const float* alpha_prev,
                               void* header, void* payload, void* ws, hipStream_t s, StageTimer* tm);
hipError_t launch_mbq_decompress(const accept_desc& d, const void* header, const void* payload, void* xhat,
                                 hipStream_t s, StageTimer* tm);
hipError_t launch_mbq_init(const accept_desc& d, const MPlan& p, const void* x, float* alpha_out, void* payload,
                           void* ws, hipStream_t s, int polls = kHeldPolls);

// ---- device helpers ---------------------------------------------------------------------
#if defined(__HIPCC__)

__device__ __forceinline__ float u32_as_f32(uint32_t u) { return __uint_as_float(u); }
__device__ __forceinline__ uint32_t f32_as_u32(float f) { return __float_as_uint(f); }

// Box of workgroup t between the counters.
__device__ __forceinline__ uint64_t* between_box(ChipMail* mail, int kind, uint32_t t) {
  uint64_t* const ctrl = reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(mail) - kMailOffset);
  return ctrl + t / 8 * kBetweenStride + 8 * (1 + kind) + t % 8;
}
// Counts the call's exchanges, `before` of which there were before; by the workgroup's first threads, after it has
// posted its values.
// The number wraps after 2^32 exchanges.  A box may not have been written for as long (a call with many workgroups,
// then none for half a day), and would then bear the number of the exchange at hand.  So a call that goes past a
// multiple of 2^30 gives every box that none of its own exchanges has written the number of the one before.
constexpr int kRenumberShift = 30;
__device__ __forceinline__ void count_exchanges(ChipMail* mail, uint32_t before, uint32_t exchanges) {
  const uint32_t t = blockIdx.x + gridDim.x * threadIdx.x;  // this workgroup's word, and those of absent ones
  if (t >= uint32_t(kHeldGrid)) return;
  __hip_atomic_fetch_add(&mail->calls[t], exchanges, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (((before ^ (before + exchanges)) >> kRenumberShift) == 0) return;
  uint64_t* const boxes[6] = {mail->first + t,           mail->last + t,            mail->more + t,
                              between_box(mail, 0, t), between_box(mail, 1, t), between_box(mail, 2, t)};
  for (uint64_t* box : boxes) {
    const uint64_t v = __hip_atomic_load(box, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (before + exchanges - uint32_t(v >> 32) >= exchanges)
      __hip_atomic_store(box, uint64_t(before) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

typedef float v4f_t __attribute__((ext_vector_type(4)));
typedef uint32_t v4u_t __attribute__((ext_vector_type(4)));

// Cache policy.  Tensors here are far larger than the caches and each byte is used once per
// kernel.  Streaming (non-temporal) stores let output lines drain to HBM while the kernel that
// wrote them still runs, instead of sitting dirty in L2 / the memory-side cache and stealing
// bandwidth from the next kernel; streaming loads keep single-use input from evicting them.
__device__ __forceinline__ uint4 load16(const void* p) { return *reinterpret_cast<const uint4*>(p); }
__device__ __forceinline__ uint4 load16_stream(const void* p) {
  const v4u_t v = __builtin_nontemporal_load(reinterpret_cast<const v4u_t*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store16_stream(void* p, uint4 v) {
  const v4u_t u = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(u, reinterpret_cast<v4u_t*>(p));
}

// The same for rows that start at any element.  (Vector memory takes any alignment; the 64 lanes'
// contiguous kilobyte then touches nine cache lines instead of eight.)  The store is a plain one: the
// two lines at its ends are each written by two wavefronts, and only a cache that keeps them puts the
// parts together.  Multi-bit decoder, float32, k = 4, single columns / streaming / plain (us):
// 101148 x 535 42 / 65 / 40, 64 x 802817 39 / 50 / 36, 93586 x 477 35 / 55 / 34, 15 x 390403 7.8 / 6.6 / 6.6;
// bfloat16 36 / 38 / 25, 34 / 26 / 22, 31 / 31 / 31, 7.6 / 6.4 / 6.1.
typedef uint32_t v4u_any_t __attribute__((ext_vector_type(4), aligned(2)));
__device__ __forceinline__ uint4 load16_stream_any(const void* p) {
  const v4u_any_t v = __builtin_nontemporal_load(reinterpret_cast<const v4u_any_t*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store16_any(void* p, uint4 v) {
  const v4u_any_t u = {v.x, v.y, v.z, v.w};
  *reinterpret_cast<v4u_any_t*>(p) = u;
}

// NDW consecutive dwords of payload (plain stores: streaming stores of the payload gained nothing),
// aligned to 16 bytes when NDW % 4 == 0, to 8 when NDW % 2 == 0, else 4.
template <int NDW>
__device__ __forceinline__ void store_dwords(uint32_t* p, const uint32_t (&v)[NDW]) {
  struct alignas((NDW % 4 == 0) ? 16 : (NDW % 2 == 0) ? 8 : 4) Block { uint32_t w[NDW]; };
  Block b;
#pragma unroll
  for (int i = 0; i < NDW; ++i) b.w[i] = v[i];
  *reinterpret_cast<Block*>(p) = b;
}

// The same with streaming stores (the MBQ encoder's planes: fewer dirty lines are left for the
// end of the kernel, which the finalize kernel's start waits for).
template <int NDW>
__device__ __forceinline__ void store_dwords_stream(uint32_t* p, const uint32_t (&v)[NDW]) {
  if constexpr (NDW % 4 == 0) {
#pragma unroll
    for (int i = 0; i < NDW; i += 4) {
      const v4u_t u = {v[i], v[i + 1], v[i + 2], v[i + 3]};
      __builtin_nontemporal_store(u, reinterpret_cast<v4u_t*>(p + i));
    }
  } else if constexpr (NDW % 2 == 0) {
    typedef uint32_t v2u_t __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int i = 0; i < NDW; i += 2) {
      const v2u_t u = {v[i], v[i + 1]};
      __builtin_nontemporal_store(u, reinterpret_cast<v2u_t*>(p + i));
    }
  } else {
#pragma unroll
    for (int i = 0; i < NDW; ++i) __builtin_nontemporal_store(v[i], p + i);
  }
}

// Payload stores that write through the second-level cache: the lines stay in it for whoever reads the payload next,
// and none is left dirty for the end of the kernel, which the next one's start waits for.  For wavefronts whose
// lanes' dwords lie together (lines written in parts cost a trip to memory each).  The instruction takes a buffer
// (`bytes` from p on, p the same in all lanes) and a byte offset.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t payload_buffer(void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, int(bytes), 0x00020000);
}
template <int ND>
__device__ __forceinline__ void store_through(__amdgpu_buffer_rsrc_t payload, uint32_t at, const uint32_t (&v)[ND]) {
  static_assert(ND >= 1 && ND <= 4, "one instruction");
  constexpr int kWriteThrough = 16;  // the instruction's sc1 bit
  typedef uint32_t v2u_t __attribute__((ext_vector_type(2)));
  typedef uint32_t v3u_t __attribute__((ext_vector_type(3)));
  if constexpr (ND == 1) __builtin_amdgcn_raw_buffer_store_b32(v[0], payload, at, 0, kWriteThrough);
  if constexpr (ND == 2) __builtin_amdgcn_raw_buffer_store_b64(v2u_t{v[0], v[1]}, payload, at, 0, kWriteThrough);
  if constexpr (ND == 3) __builtin_amdgcn_raw_buffer_store_b96(v3u_t{v[0], v[1], v[2]}, payload, at, 0, kWriteThrough);
  if constexpr (ND == 4) __builtin_amdgcn_raw_buffer_store_b128(v4u_t{v[0], v[1], v[2], v[3]}, payload, at, 0, kWriteThrough);
}

__device__ __forceinline__ void widen(const uint4 v, float (&f)[4]) {
  f[0] = u32_as_f32(v.x); f[1] = u32_as_f32(v.y); f[2] = u32_as_f32(v.z); f[3] = u32_as_f32(v.w);
}
__device__ __forceinline__ void widen(const uint4 v, float (&f)[8]) {  // eight bfloat16, element 0 in the low half
  f[0] = u32_as_f32(v.x << 16); f[1] = u32_as_f32(v.x & 0xFFFF0000u);
  f[2] = u32_as_f32(v.y << 16); f[3] = u32_as_f32(v.y & 0xFFFF0000u);
  f[4] = u32_as_f32(v.z << 16); f[5] = u32_as_f32(v.z & 0xFFFF0000u);
  f[6] = u32_as_f32(v.w << 16); f[7] = u32_as_f32(v.w & 0xFFFF0000u);
}
// 16-byte vector load widened to float32; the _stream form is for data read once.
__device__ __forceinline__ void load_vec(const float* p, float (&f)[4]) { widen(load16(p), f); }
__device__ __forceinline__ void load_vec(const bf16_t* p, float (&f)[8]) { widen(load16(p), f); }
__device__ __forceinline__ void load_vec_stream(const float* p, float (&f)[4]) { widen(load16_stream(p), f); }
__device__ __forceinline__ void load_vec_stream(const bf16_t* p, float (&f)[8]) { widen(load16_stream(p), f); }
__device__ __forceinline__ float load_one(const float* p) { return *p; }
__device__ __forceinline__ float load_one(const bf16_t* p) { return u32_as_f32(uint32_t(p->bits) << 16); }

// float32 -> bfloat16 bits, round to nearest even (finite values).
__device__ __forceinline__ uint32_t bf16_rne(float f) {
  const uint32_t b = f32_as_u32(f);
  return (b + 0x7FFFu + ((b >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ uint4 narrow(const float (&f)[4]) {
  return make_uint4(f32_as_u32(f[0]), f32_as_u32(f[1]), f32_as_u32(f[2]), f32_as_u32(f[3]));
}
// Two float32 -> two bfloat16 in a dword (first in the low half), round to nearest even: one
// instruction, bit for bit bf16_rne on every finite float32, denormals included (all 2^32 patterns
// were compared), where the integer form takes nine.  The decoders of bfloat16 tensors are bound by
// their instructions: 51.4 M values, scheme M at
// k = 4 23.0 -> 20.9 us, scheme U at k = 6 with a range per channel 26.4 -> 25.0 us.
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ uint4 narrow(const float (&f)[8]) {
  return make_uint4(bf16_pair(f[0], f[1]), bf16_pair(f[2], f[3]), bf16_pair(f[4], f[5]), bf16_pair(f[6], f[7]));
}
// 16-byte vector store of decompressed values (streaming).
__device__ __forceinline__ void store_vec(float* p, const float (&f)[4]) { store16_stream(p, narrow(f)); }
__device__ __forceinline__ void store_vec(bf16_t* p, const float (&f)[8]) { store16_stream(p, narrow(f)); }
__device__ __forceinline__ void store_one(float* p, float f) { *p = f; }
__device__ __forceinline__ void store_one(bf16_t* p, float f) { p->bits = uint16_t(bf16_rne(f)); }

// Four consecutive elements (16 bytes of float32, 8 bytes of bfloat16; p aligned to that).
template <typename T>
__device__ __forceinline__ void load_quad(const T* p, float (&f)[4]) {
  if constexpr (sizeof(T) == 4) {
    widen(load16_stream(p), f);
  } else {
    const uint2 v = *reinterpret_cast<const uint2*>(p);
    f[0] = u32_as_f32(v.x << 16); f[1] = u32_as_f32(v.x & 0xFFFF0000u);
    f[2] = u32_as_f32(v.y << 16); f[3] = u32_as_f32(v.y & 0xFFFF0000u);
  }
}
template <typename T>
__device__ __forceinline__ void store_quad(T* p, const float (&f)[4]) {
  if constexpr (sizeof(T) == 4) {
    store_vec(p, f);
  } else {
    uint2 v;
    v.x = bf16_pair(f[0], f[1]);
    v.y = bf16_pair(f[2], f[3]);
    *reinterpret_cast<uint2*>(p) = v;
  }
}

// Lane exchange inside a row of 16 lanes with a DPP control word (all lanes stay valid).
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u32(uint32_t v) {
  return uint32_t(__builtin_amdgcn_update_dpp(int(v), int(v), CTRL, 0xF, 0xF, false));
}
constexpr int kDppQuadSwap1 = 0xB1;      // quad_perm [1,0,3,2]
constexpr int kDppQuadSwap2 = 0x4E;      // quad_perm [2,3,0,1]
constexpr int kDppRowHalfMirror = 0x141;
constexpr int kDppRowMirror = 0x140;

// Maximum over the 64 lanes of a wavefront; every lane receives the result.  Operands are
// non-negative floats, compared through their bit patterns' float view.
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, u32_as_f32(dpp_u32<kDppQuadSwap1>(f32_as_u32(v))));
  v = fmaxf(v, u32_as_f32(dpp_u32<kDppQuadSwap2>(f32_as_u32(v))));
  v = fmaxf(v, u32_as_f32(dpp_u32<kDppRowHalfMirror>(f32_as_u32(v))));
  v = fmaxf(v, u32_as_f32(dpp_u32<kDppRowMirror>(f32_as_u32(v))));
  v = fmaxf(v, __shfl_xor(v, 16, kWave));
  v = fmaxf(v, __shfl_xor(v, 32, kWave));
  return v;
}

// Lane exchange of a float64 inside a row of 16 lanes (two 32-bit DPP moves).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t b = uint64_t(__double_as_longlong(v));
  const uint32_t lo = dpp_u32<CTRL>(uint32_t(b)), hi = dpp_u32<CTRL>(uint32_t(b >> 32));
  return __longlong_as_double((long long)((uint64_t(hi) << 32) | lo));
}
__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const uint64_t b = uint64_t(__double_as_longlong(v));
  const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(b)), lane));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(b >> 32)), lane));
  return __longlong_as_double((long long)((uint64_t(hi) << 32) | lo));
}

// Sum over the 64 lanes in a fixed order (so the result does not depend on timing); every lane
// receives the same value.  Four butterfly steps inside each row of 16 lanes (partners add in
// either order: the same float64 either way), then the four row sums as (r0 + r1) + (r2 + r3).
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_f64<kDppQuadSwap1>(v);
  v += dpp_f64<kDppQuadSwap2>(v);
  v += dpp_f64<kDppRowHalfMirror>(v);
  v += dpp_f64<kDppRowMirror>(v);
  const double r0 = readlane_f64(v, 0), r1 = readlane_f64(v, 16), r2 = readlane_f64(v, 32), r3 = readlane_f64(v, 48);
  return (r0 + r1) + (r2 + r3);
}

// The same for counts (exact in any order; the sum of 16 lanes has to fit 32 bits).
__device__ __forceinline__ uint64_t wave_sum(uint32_t v) {
  v += dpp_u32<kDppQuadSwap1>(v);
  v += dpp_u32<kDppQuadSwap2>(v);
  v += dpp_u32<kDppRowHalfMirror>(v);
  v += dpp_u32<kDppRowMirror>(v);
  const uint64_t r0 = uint32_t(__builtin_amdgcn_readlane(int(v), 0)), r1 = uint32_t(__builtin_amdgcn_readlane(int(v), 16));
  const uint64_t r2 = uint32_t(__builtin_amdgcn_readlane(int(v), 32)), r3 = uint32_t(__builtin_amdgcn_readlane(int(v), 48));
  return (r0 + r1) + (r2 + r3);
}

// Counter-based uniform numbers: element idx gets u = (top 24 bits of h) * 2^-24, h = splitmix64's
// output function at the state z = seed + (idx+1) * kRandStep.  States of neighbouring elements
// differ by a constant, so a kernel forms one state per thread and adds from there.
constexpr uint64_t kRandStep = 0x9E3779B97F4A7C15ull;
__device__ __forceinline__ uint64_t rand_state(uint64_t seed, uint64_t idx) { return seed + (idx + 1ull) * kRandStep; }

// The low word of a * b + c in one instruction, v_mad_u64_u32, whose addend is a register pair: what its high word holds does
// not matter.  (The compiler makes a multiplication and an addition of it, as the high word would be 0 to it.  Stochastic
// rounding, whole call, two instructions / one, us: 64 x 802816 k = 4 float32 72.3 / 71.6, k = 8 bfloat16 61.9 / 60.4, 64 x 262144 29.7 /
// 29.1, 128 x 160 4.61 / 4.56; element by element, in the code for odd channel geometries, which 64-bit divisions hold up, the compiler's two are
// better: 192367 x 251 channels-last bfloat16, k = 2 157.6 / 163.4, 131427 x 19 x 7 k = 4 53.9 / 55.3.)
__device__ __forceinline__ uint32_t mad_low(uint32_t a, uint32_t b, uint32_t c) {
  typedef uint32_t v2u_t __attribute__((ext_vector_type(2)));
  uint32_t any;
  asm("" : "=v"(any) : "v"(c));
  uint64_t sum, carry;
  asm("v_mad_u64_u32 %0, %1, %2, %3, %4" : "=v"(sum), "=s"(carry) : "v"(a), "s"(b), "v"(__builtin_bit_cast(uint64_t, v2u_t{c, any})));
  return uint32_t(sum);
}

// u * 2^32 as a float32 (exact: 24 significant bits).  Written on 32-bit halves: the output
// function's last step z ^ (z >> 31) leaves the top 31 bits as they are, so only the high word of
// the second product is formed, and a 64-bit source would be converted to float by a sequence of
// seven instructions where one does.
template <bool MAD>
__device__ __forceinline__ float rand_u32(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z ^= z >> 27;
  constexpr uint64_t C2 = 0x94D049BB133111EBull;
  const uint32_t lo = uint32_t(z), hi = uint32_t(z >> 32);
  uint32_t h;
  if constexpr (MAD) h = mad_low(hi, uint32_t(C2), mad_low(lo, uint32_t(C2 >> 32), __umulhi(lo, uint32_t(C2))));
  else h = __umulhi(lo, uint32_t(C2)) + lo * uint32_t(C2 >> 32) + hi * uint32_t(C2);
  h &= 0xFFFFFF00u;
  return float(h);
}

#endif  // __HIPCC__

}  // namespace accept
