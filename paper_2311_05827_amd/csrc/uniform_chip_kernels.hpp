// The kernels of uniform_chip.hpp.
#pragma once

#include <type_traits>

#include "uniform_chip.hpp"

namespace accept {

namespace {

// One value of every workgroup of a list (all of a call's, or those that share a channel), exchanged through
// mailboxes: the largest of all.  The wait is bounded: nothing says that all workgroups run at the same time (another
// kernel may hold some compute units).  Where a workgroup has looked `polls` times in vain, it finds the values that
// are missing itself, one workgroup's part after the other, and posts them: those that wait share
// the work of those that have not started, which later post the same values.  So every workgroup ends whatever else
// runs, and the result does not depend on it.
// The list has at most 256 members, 0 .. n-1; box(i) is the mailbox of member i.
struct Exchange {
  float top[kHeldBlock / kWave];  // of the values seen so far, by wavefront
  float part[kHeldBlock / kWave];
  uint64_t missing[kHeldGrid / kWave];
};
__device__ __forceinline__ void post(uint64_t* box, uint32_t tag, float v) {
  __hip_atomic_store(box, (uint64_t(tag) << 32) | f32_as_u32(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t look(const uint64_t* box) {
  return __hip_atomic_load(box, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Four wavefronts look for member `i` each lane (0 .. 255), at most `polls` times; on return (in front of a barrier) ex
// holds what is missing and the wavefronts' maxima of what is there.  Returns what this wavefront misses.
// Looking in vain holds up the others' posts, which go to the same lines: where many look, the first look comes when
// most posts are there (sleep units of 64 cycles).  Whole call, at once / after 8 / 16 / 24 units, us, tensors in registers,
// float32, k = 8: 1.05 M 5.8 / 5.5 / 5.15 / 5.3, 2.1 M 6.4 / 5.7 / 5.3 / 5.5, 8.3 M 10.6 / 10.1 / 9.9 / 9.9; stochastic, 0.5 M 6.0 / 5.6 /
// 5.1 / 5.3; held pass, after 0 / 12 / 24 / 36: 103 MB 23.9 / 23.4 / 23.3 / 23.3, 205 MB 55.7 / 55.5 / 55.3 / 55.35; two channels of 51 MB
// 23.7 / 23.6 (8) / 23.3 (16) / 23.2 (24), while channels of few workgroups lose by any (8 x 32 x 12288 bfloat16 5.7 / 5.9 (24)).
constexpr int kManyLook = 32;  // workgroups
template <typename Box>
__device__ __forceinline__ uint64_t look_for_mail(int i, int n, uint32_t tag, int polls, Exchange& ex, Box box) {
  const bool member = i < n;
  uint64_t missing = __ballot(member);
  uint64_t v = 0;
  for (int p = 0; p < polls; ++p) {
    if (member) v = look(box(i));
    missing = __ballot(member && uint32_t(v >> 32) != tag);
    if (missing == 0) break;
    __builtin_amdgcn_s_sleep(4);
  }
  const float t = wave_max(u32_as_f32(member && uint32_t(v >> 32) == tag ? uint32_t(v) : 0u));
  if ((i & (kWave - 1)) == 0) {
    ex.top[i / kWave] = t;
    ex.missing[i / kWave] = missing;
  }
  return missing;
}
// After look_for_mail and a barrier: how many members are missing, and one of them, another for neighbouring
// workgroups (both in scalar registers).
__device__ __forceinline__ int missing_count(const Exchange& ex) {
  int count = 0;
#pragma unroll
  for (int w = 0; w < kHeldGrid / kWave; ++w) count += __popcll((unsigned long long)ex.missing[w]);
  return __builtin_amdgcn_readfirstlane(count);
}
__device__ __forceinline__ int missing_one(const Exchange& ex, int count) {
  int skip = int(blockIdx.x) % count, found = 0;
#pragma unroll
  for (int w = 0; w < kHeldGrid / kWave; ++w) {
    uint64_t m = ex.missing[w];
    m = (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(m >> 32))))) << 32) |
        uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(m))));
    const int here = __popcll((unsigned long long)m);
    if (skip >= 0 && skip < here) {
      for (; skip > 0; --skip) m &= m - 1;
      found = w * kWave + __ffsll((unsigned long long)m) - 1;
    }
    skip -= here;
  }
  return found;
}
__device__ __forceinline__ float largest_mail(const Exchange& ex) {
  float c = ex.top[0];
#pragma unroll
  for (int w = 1; w < kHeldGrid / kWave; ++w) c = fmaxf(c, ex.top[w]);
  return c;
}
// Finds and posts what is missing until nothing is; part(i): a thread's share of member i's largest value; put(i, v), by
// some threads from 0 on, posts it.  Every turn takes at least one member off the list, whatever becomes of its mailbox.
template <typename Box, typename Part, typename Put>
__device__ __forceinline__ void post_missing(uint32_t tag, Exchange& ex, Box box, Part part, Put put) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  for (int count = missing_count(ex); count != 0; count = missing_count(ex)) {
    const int w = missing_one(ex, count);
    const float v = wave_max(part(w));
    if (lane == 0) ex.part[wave] = v;
    __syncthreads();
    if (wave < kHeldGrid / kWave) {
      float t = ex.part[0];
      for (int i = 1; i < kHeldBlock / kWave; ++i) t = fmaxf(t, ex.part[i]);
      put(w, t);
      const uint64_t missing = ex.missing[wave];
      const bool wanted = (missing >> lane) & 1u;
      const uint64_t found = wanted ? look(box(tid)) : 0;
      const bool there = wanted && uint32_t(found >> 32) == tag;
      const float seen = wave_max(tid == w ? t : there ? u32_as_f32(uint32_t(found)) : 0.0f);
      const uint64_t left = missing & ~__ballot(there || tid == w);
      if (lane == 0) {
        ex.top[wave] = fmaxf(ex.top[wave], seen);
        ex.missing[wave] = left;
      }
    }
    __syncthreads();
  }
}

// The codes of unit `unit`: pieces of the thread's vectors through local memory (one barrier; the caller alternates
// between two buffers), then the parts it packs.
template <typename T, int K, typename VecOf>
__device__ __forceinline__ void quantize_unit(uint32_t* buf, float r, uint32_t* __restrict__ payload32, int64_t unit,
                                              VecOf vec_of) {
  constexpr int VEC = Elem<T>::VEC;
  constexpr int LOADS = kUnitElems / (kHeldBlock * VEC), QPV = VEC / 4;
  const int tid = threadIdx.x;
  float rv[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) rv[e] = r;
#pragma unroll
  for (int u = 0; u < LOADS; ++u) {
    float f[VEC];
    widen(vec_of(u), f);
#pragma unroll
    for (int h = 0; h < QPV; ++h) buf[(u * kHeldBlock + tid) * QPV + h] = quantize4<K, false>(&f[4 * h], rv, 0);
  }
  __syncthreads();
  const __amdgpu_buffer_rsrc_t codes = payload_buffer(payload32 + unit * (kHeldBlock * K), kHeldBlock * K * 4);
#pragma unroll
  for (int i = 0; i < CodeParts<K>::PARTS; ++i) {
    const int part = i * kHeldBlock + tid;
    uint32_t out[CodeParts<K>::DWORDS];
    pack_part<K>(&buf[part * CodeParts<K>::PIECES], out);
    store_part<K>(codes, uint32_t(part * CodeParts<K>::DWORDS * 4), out);
  }
}
// Workgroup b's elements behind the last whole unit, 64 of them: 8 threads take 8 each.
template <typename T, int K>
__device__ __forceinline__ void quantize_behind(const T* __restrict__ x, uint32_t* __restrict__ payload32, float r, int64_t N,
                                                int64_t units, int64_t payload_bytes, int b) {
  const int64_t g = (units * kUnitElems + int64_t(b) * kWave) / 8 + threadIdx.x;
  if (threadIdx.x < kWave / 8 && g * 8 < N)
    quantize_group8<T, K, false>(x, reinterpret_cast<uint8_t*>(payload32), g, N, payload_bytes, 0, [&](int64_t) { return r; });
}

// U1, and U2 + U3 for the end of the tensor, in one kernel (one range for the tensor, rounding to
// nearest).  The range has to be known before the first element can be quantized, so the plain way
// reads the tensor twice, and the memory-side cache does not help: it delivers 7.4 TB/s, memory
// itself 7.2.  The registers and local memories of the chip hold 168 MiB, though.  Here one workgroup per compute unit
// reads units (16384 elements) b, b + 256, ..., keeps the last of them (float32: 7 units in registers
// and 2 in local memory, 151 MB over the chip; bfloat16: 14 and 4, the same), hands its maximum to the
// other workgroups through a mailbox, waits for theirs, quantizes what it kept and reads the units
// before held_first once more.  The up to 16383 elements behind the last whole unit are shared out, 64 to a
// workgroup, for the range and for the codes.
//
// A workgroup that does not see all the others' maxima in time (see Exchange) no longer uses what it kept, so that
// its registers serve for the others' parts, and reads its own units again, the way it reads those that it did not keep.
// (With code of its own for that, seven slots were spilled; a second kernel for such workgroups' units took 2 us of every
// call above 134 MB: 205 MB, k = 8 / 4 55.7 / 52.8 -> 54.1 / 51.2 us, 154 MB 37.0 -> 35.5.)
//
// Beside other work: a workgroup needs a whole compute unit (160 KiB of local memory, all registers), so
// next to a kernel whose workgroups keep filling the chip it starts late, and the early ones give up.
// Time of a call on one stream while another is busy, k = 8, two reads / this (us; calls one behind the other, all measured in
// turn): float32 103, 154, 205 MB, bfloat16 103, 205 MB beside small elementwise kernels 41 / 26, 59 / 39, 78 / 55, 45 / 31,
// 87 / 61; beside matrix products 219 / 123, 228 / 134, - / 150, 233 / 127, 250 / 156; beside copies of 512 MB without a pause
// 73 / 97, 103 / 136, 133 / 192, 78 / 120, 148 / 221, which is lost.  The second kernel for late workgroups, which float32 had
// above 134 MB, was better beside copies and worse beside matrix products: 154 MB 106 and 239, 205 MB 130 and 270.
//
// 51.4 M float32 values (205 MB), k = 8: 54.1 us a call (two reads 69.5): 31 us to the mailboxes, 2 to 3 for the
// exchange.  103 MB: 32 -> 26 us against the held pass with a second kernel and plain stores, bfloat16 103 MB 36 -> 30.
// Stochastic rounding keeps the two reads: it is bound by its instructions, which the second read
// hides behind.
template <typename T, int K, int SLOTS>
__global__ __launch_bounds__(kHeldBlock, 2) void quantize_held_kernel(const T* __restrict__ x,
                                                                      uint32_t* __restrict__ payload32,
                                                                      float* __restrict__ header,
                                                                      ChipMail* __restrict__ mail, int64_t N,
                                                                      int64_t units, int64_t held_first, int lds_units,
                                                                      int64_t payload_bytes, int polls) {
  constexpr int VEC = Elem<T>::VEC;
  constexpr int LOADS = kUnitElems / (kHeldBlock * VEC);  // vectors per thread and unit
  constexpr int RING = 32 / (4 * LOADS) * 2;  // units in flight while nothing is kept yet: 128 KiB per workgroup
  constexpr int WAVES = kHeldBlock / kWave;
  constexpr int LDS_UNITS = kHeldLdsUnits<T>;
  static_assert(RING >= 2 && RING < SLOTS, "registers");
  static_assert(LDS_UNITS % RING == 0 && LDS_UNITS < SLOTS, "units kept in local memory pass through the ring in whole turns");
  // local memory, all 160 KiB of it: what is kept, and two buffers of pieces (the second of which the
  // exchange uses before)
  struct Local {
    uint4 kept[LDS_UNITS][LOADS][kHeldBlock];
    uint32_t pieces[2][kUnitElems / 4];
  };
  static_assert(sizeof(Local) <= 160 * 1024, "local memory of a compute unit");
  __shared__ __attribute__((aligned(16))) Local local;
  Exchange& ex = *reinterpret_cast<Exchange*>(local.pieces[1]);
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1), wave = tid / kWave;

  // units of this workgroup: ordinals 0 .. count-1, unit = ordinal * 256 + b; those before `first`
  // (held_first is a multiple of 256) are only looked at
  const int count = int((units - blockIdx.x + kHeldGrid - 1) / kHeldGrid);  // at least 1 (host)
  const int first = int(held_first / kHeldGrid);
  uint4 kept[SLOTS][LOADS];
  auto ask = [&](int slot_ordinal, uint4 (&raw)[LOADS]) {
    const T* xu = x + (int64_t(slot_ordinal) * kHeldGrid + blockIdx.x) * kUnitElems;
#pragma unroll
    for (int u = 0; u < LOADS; ++u) raw[u] = load16_stream(xu + (u * kHeldBlock + tid) * VEC);
  };
  // Elements behind the last whole unit: workgroup b has the 64 from units * 16384 + 64 b on, its
  // wavefronts all the same ones; where there are none, the tensor's last element stands in for them.
  static_assert(kUnitElems == kHeldGrid * kWave, "one element per workgroup and lane covers what is behind the last unit");
  const int64_t behind = units * kUnitElems + int64_t(blockIdx.x) * kWave + lane;
  const float tail = load_one(x + (behind < N ? behind : N - 1));
  float c = 0.0f;
  auto look = [&](const uint4 (&raw)[LOADS]) {
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      float f[VEC];
      widen(raw[u], f);
#pragma unroll
      for (int e = 0; e < VEC; ++e) c = fmaxf(c, fabsf(f[e]));
    }
  };
  // Slots 0 .. RING-1 are a ring while the units before `first` go by: a unit looked at makes room
  // for the one RING ordinals later (it exists: the held part is longer than the ring), and when
  // the loop ends slot j holds ordinal first + j, like the other slots.  The loop runs whole turns;
  // what is left over by a division goes through the slots behind the ring beforehand.  (Loads and
  // looks of the loop are unconditional, so that the compiler knows how many loads are in flight
  // and waits for no more than it needs.)
  const int extra = first % RING;
#pragma unroll
  for (int j = 0; j < RING - 1; ++j)
    if (j < extra) ask(j, kept[RING + j]);
#pragma unroll
  for (int j = 0; j < RING; ++j) ask(extra + j < count ? extra + j : count - 1, kept[j]);
  const uint32_t calls = mail->calls[blockIdx.x];
  c = fabsf(tail);
#pragma unroll
  for (int j = 0; j < RING - 1; ++j)
    if (j < extra) look(kept[RING + j]);
  for (int o = extra; o < first; o += RING) {
#pragma unroll
    for (int j = 0; j < RING; ++j) {
      look(kept[j]);
      __builtin_amdgcn_sched_barrier(0);  // the next unit's loads are issued here, before the other slots are waited for
      ask(o + RING + j, kept[j]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (lds_units != 0) {  // 0 or LDS_UNITS: ordinals first .. first + LDS_UNITS - 1 go on to local memory
#pragma unroll
    for (int q = 0; q < LDS_UNITS; ++q) {
      look(kept[q % RING]);
#pragma unroll
      for (int u = 0; u < LOADS; ++u) local.kept[q][u][tid] = kept[q % RING][u];
      __builtin_amdgcn_sched_barrier(0);
      ask(first + q + RING, kept[q % RING]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  const int base = first + lds_units;  // slot j: ordinal base + j
#pragma unroll
  for (int j = RING; j < SLOTS; ++j)
    if (base + j < count) ask(base + j, kept[j]);
#pragma unroll
  for (int j = 0; j < RING; ++j) look(kept[j]);  // (a clamped copy of the last unit does no harm)
#pragma unroll
  for (int j = RING; j < SLOTS; ++j)
    if (base + j < count) look(kept[j]);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // nothing is in flight from here on, whichever slots are in use

  const uint32_t tag = uint32_t(__builtin_amdgcn_readfirstlane(int(calls))) + 1u;
  c = wave_max(c);
  if (lane == 0) ex.top[wave] = c;
  __syncthreads();
  if (tid == 0) {
    c = ex.top[0];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) c = fmaxf(c, ex.top[w]);
    post(mail->first + blockIdx.x, tag, c);
    count_exchanges(mail, tag - 1u, 1u);
  }
  __syncthreads();
  auto box = [&](int w) { return mail->first + w; };
  if (wave < kHeldGrid / kWave) {
    __builtin_amdgcn_s_sleep(24);
    look_for_mail(tid, kHeldGrid, tag, polls, ex, box);
  }
  __syncthreads();

  float r = 0.0f;
  int buf_i = 0;
  auto quantize = [&](int ordinal, auto vec_of) {
    quantize_unit<T, K>(local.pieces[buf_i], r, payload32, int64_t(ordinal) * kHeldGrid + blockIdx.x, vec_of);
    buf_i ^= 1;
  };
  const bool late = missing_count(ex) != 0;
  int from = first, held_from = base, in_lds = lds_units;  // ordinals before `from` are to be read again
  if (late) {
    post_missing(tag, ex, box, [&](int w) {
      float v = 0.0f;
      for (int64_t unit = w; unit < units; unit += kHeldGrid) {
        const T* xu = x + unit * kUnitElems;
#pragma nounroll
        for (int half = 0; half < LOADS; half += 4) {  // four loads at a time: registers
          uint4 raw[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) raw[u] = load16_stream(xu + ((half + u) * kHeldBlock + tid) * VEC);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            float f[VEC];
            widen(raw[u], f);
#pragma unroll
            for (int e = 0; e < VEC; ++e) v = fmaxf(v, fabsf(f[e]));
          }
        }
      }
      const int64_t b = units * kUnitElems + int64_t(w) * kWave + lane;
      return fmaxf(v, fabsf(load_one(x + (b < N ? b : N - 1))));
    }, [&](int w, float v) { if (tid == 0) post(box(w), tag, v); });
    from = held_from = count;
    in_lds = 0;
    // (an empty asm: what was kept need not live through the above)
#pragma unroll
    for (int j = 0; j < SLOTS; ++j)
#pragma unroll
      for (int u = 0; u < LOADS; ++u)
        asm volatile("" : "=v"(kept[j][u].x), "=v"(kept[j][u].y), "=v"(kept[j][u].z), "=v"(kept[j][u].w));
  }
  {
    float s;
    scale_from_range(largest_mail(ex), K, s, r);
    if (blockIdx.x == 0 && tid == 0) header[0] = s;
  }
  // A slot that has been quantized takes a unit that was only looked at, the last of them first;
  // those loads are under way while the other kept units are quantized.  (Conditions are the same
  // in all threads.)
#pragma unroll
  for (int j = 0; j < SLOTS; ++j) {
    if (held_from + j < count) quantize(held_from + j, [&](int u) { return kept[j][u]; });
    if (j < from) ask(from - 1 - j, kept[j]);
  }
  if (in_lds != 0) {
    for (int q = 0; q < LDS_UNITS; ++q) quantize(first + q, [&](int u) { return local.kept[q][u][tid]; });
  }
  for (int o = from - 1; o >= 0; o -= SLOTS) {
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
      if (o - j >= 0) {
        quantize(o - j, [&](int u) { return kept[j][u]; });
        if (o - j - SLOTS >= 0) ask(o - j - SLOTS, kept[j]);
      }
    }
  }
  quantize_behind<T, K>(x, payload32, r, N, units, payload_bytes, blockIdx.x);
}

// U1, U1b, U2 and U3 of a tensor with one range per channel, in one kernel and with one read: the
// tensor stays on the chip between the two steps.  The tensor's groups of 32 elements (k whole dwords
// of payload each; segments are whole groups) are numbered channel after channel, row after row inside a
// channel, and workgroup b has the groups b*per .. (b+1)*per - 1 of that order: most of its channels are
// its own altogether, and at most two, its first and its last, it shares with neighbours.  For these it
// leaves its maximum in a mailbox and looks for those of the others, as far as they have a part of the channel (see
// Exchange).
//
// A mailbox is one 64-bit word, value and the exchange's number together, as in quantize_held_kernel (see ChipMail).
//
// What bounds it: the read of the tensor (16 of 33 us at 103 MB of bfloat16, with the looking hidden behind
// it), then the instructions that quantize and pack, two wavefronts on a SIMD, and the payload's stores
// (38 MB there).  The places of a thread's vectors are stepped, not divided out, and only the loads and
// stores need them: which channel a unit belongs to is known from scalars (per element, as at first, the
// kernel took 42 us).  Streaming stores of the payload make a call alone 3 us faster and a decoder that
// reads it next 8 us slower.
//
// Beside other work on another stream, two or three kernels / this one (us): matrix products 224 / 121 (4 x 4 x 1605632
// float32), small kernels 40.5 / 21.9, 35.5 / 21.5 (64 x 128 x 3136); 512 MB copies without a pause 85 / 74 to 89, 71 / 72 to 80,
// and 45 to 92 / 61 to 68 (1 x 2 x 12845056).  There workgroups start late, and how others make up for them counts: as
// long as each that had waited in vain read the whole channel itself, 370 to 410 and 230 to 650; and where all look in
// vain, 25.7 M values in two channels took 2756 us, now 43 (24 if they see each other).
//
// Place of a group of 32 elements: group inside its segment, batch row, and the group's number in the tensor.
struct GroupPos {
  uint32_t pos, row, at;
};
struct ChanHeldGeom {
  uint32_t seg_groups, rows;  // groups of a segment, batch rows
  uint32_t m_groups;          // groups of a row of the tensor
  uint32_t total, per;        // groups of the tensor, and of a workgroup
  GroupPos load_step;         // groups between two loads of a thread
  GroupPos part_step;         // groups between two parts of a thread
  uint32_t next_row, next_channel;  // what a step past a segment's, and past a channel's, end adds to `at`
  uint32_t shared;            // whether any channel lies in two workgroups
};
__device__ __forceinline__ GroupPos group_pos(const ChanHeldGeom& g, uint32_t q) {
  GroupPos p;
  const uint32_t seg = q / g.seg_groups;
  p.pos = q - seg * g.seg_groups;
  const uint32_t ch = seg / g.rows;
  p.row = seg - ch * g.rows;
  p.at = p.row * g.m_groups + ch * g.seg_groups + p.pos;
  return p;
}
__device__ __forceinline__ void group_advance(const ChanHeldGeom& g, GroupPos& p, const GroupPos& st) {
  p.pos += st.pos;
  p.row += st.row;
  p.at += st.at;
  if (p.pos >= g.seg_groups) { p.pos -= g.seg_groups; p.row += 1; p.at += g.next_row; }
  if (p.row >= g.rows) { p.row -= g.rows; p.at += g.next_channel; }
}


template <typename T, int K, int SLOTS, int LDS_UNITS>
__global__ __launch_bounds__(kHeldBlock, 2) void quantize_channels_kernel(const T* __restrict__ x,
                                                                          uint32_t* __restrict__ payload32,
                                                                          float* __restrict__ header,
                                                                          ChipMail* __restrict__ mail, ChanHeldGeom g,
                                                                          int polls) {
  constexpr int VEC = Elem<T>::VEC;
  constexpr int GV = 32 / VEC;                            // vectors of a group
  constexpr int LOADS = kUnitElems / (kHeldBlock * VEC);  // vectors per thread and unit
  static_assert(LOADS * (kHeldBlock / GV) == kHeldBlock && kUnitElems == 32 * kHeldBlock, "a unit is a group per thread");
  static_assert(LDS_UNITS <= SLOTS, "units kept in local memory pass through the first slots");
  constexpr int QPV = VEC / 4;
  // What finds others' missing parts needs registers, of which the largest forms have none left: vectors that are kept
  // make room then.
  constexpr int ASIDE = SLOTS * LOADS < 44 ? 0 : sizeof(T) == 4 ? 7 : 3;
  constexpr int ASK = ASIDE > 0 ? 2 : 4;  // loads in flight there
  static_assert(ASIDE <= LOADS, "they are of one slot");
  struct Local {
    uint4 kept[LDS_UNITS > 0 ? LDS_UNITS : 1][LDS_UNITS > 0 ? LOADS : 1][LDS_UNITS > 0 ? kHeldBlock : 1];
    uint32_t pieces[2][kUnitElems / 4];
    uint32_t top[kChanMaxLocal];  // largest magnitude of the workgroup's channels, as bits
    float r[kChanMaxLocal];
    Exchange ex[2];  // of the first channel and of the last
    int late;        // something was not seen in time
    uint4 aside[ASIDE > 0 ? ASIDE : 1][ASIDE > 0 ? kHeldBlock : 1];
  };
  static_assert(sizeof(Local) <= 160 * 1024, "local memory of a compute unit");
  __shared__ __attribute__((aligned(16))) Local local;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);

  const uint32_t q0 = blockIdx.x * g.per;  // below total (host)
  const uint32_t count = g.total - q0 < g.per ? g.total - q0 : g.per;
  const uint32_t units = (count + kHeldBlock - 1) / kHeldBlock;
  const uint32_t mine = uint32_t(tid) / GV;  // the thread's first vector is in this group of the workgroup's
  uint4 kept[SLOTS][LOADS];
  // The loads of the units in ordinal order, one after the other; behind the workgroup's last group its
  // first vector stands in.  (The place passes through an empty asm at every unit, or the compiler forms
  // the addresses of all of them first.)
  auto fresh = [](GroupPos& p) { asm volatile("" : "+v"(p.pos), "+v"(p.row), "+v"(p.at)); };
  GroupPos from = group_pos(g, q0 + mine);
  const uint32_t first_at = group_pos(g, q0).at;
  auto ask = [&](uint32_t ordinal, uint4 (&raw)[LOADS]) {
    fresh(from);
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      const uint32_t at = ordinal * kHeldBlock + uint32_t(u * (kHeldBlock / GV)) + mine < count ? from.at : first_at;
      raw[u] = load16_stream(reinterpret_cast<const char*>(x) + (at * uint32_t(GV) + uint32_t(tid) % GV) * 16u);
      group_advance(g, from, g.load_step);
    }
  };
#pragma unroll
  for (int j = 0; j < SLOTS; ++j) ask(j, kept[j]);
  const uint32_t tag = g.shared != 0 ? mail->calls[blockIdx.x] + 1u : 0u;
  const uint32_t per_channel = g.rows * g.seg_groups;
  const uint32_t ch_lo = q0 / per_channel;
  const uint32_t ch_hi = (q0 + count - 1) / per_channel;
  const uint32_t nloc = ch_hi - ch_lo + 1;
  if (tid < kChanMaxLocal) local.top[tid] = 0u;
  if (tid == 0) local.late = 0;
  __syncthreads();
  // The workgroup's channels, the first one's index 0; channel i ends before group end_of(i).  Units inside
  // one channel, which are most, know it from scalars; the others split at the ends inside them.
  const uint32_t first_end = (ch_lo + 1) * per_channel - q0;
  float c = 0.0f;             // of the channel at hand
  uint32_t chan = 0, end = first_end < count ? first_end : count;
  auto hand_over = [&] {
    const float t = wave_max(c);
    if (lane == 0) atomicMax(&local.top[chan], f32_as_u32(t));
    c = 0.0f;
  };
  auto look = [&](uint32_t ordinal, const uint4 (&raw)[LOADS]) {
    const uint32_t g0 = ordinal * kHeldBlock;
    auto largest = [&](int u) {
      float f[VEC];
      widen(raw[u], f);
      float v = 0.0f;
#pragma unroll
      for (int e = 0; e < VEC; ++e) v = fmaxf(v, fabsf(f[e]));
      return v;
    };
    if (g0 + kHeldBlock <= end) {
#pragma unroll
      for (int u = 0; u < LOADS; ++u) c = fmaxf(c, largest(u));
    } else {
      uint32_t begin = g0;
      while (begin < g0 + kHeldBlock && begin < count) {  // the same in all lanes
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
          const uint32_t grp = g0 + uint32_t(u * (kHeldBlock / GV)) + mine;
          c = fmaxf(c, grp >= begin && grp < end ? largest(u) : 0.0f);
        }
        if (end > g0 + kHeldBlock || end == count) break;
        hand_over();
        begin = end;
        ++chan;
        end = end + per_channel < count ? end + per_channel : count;
      }
    }
  };
  if constexpr (LDS_UNITS > 0) {
#pragma unroll
    for (int j = 0; j < LDS_UNITS; ++j) {
      look(j, kept[j]);
#pragma unroll
      for (int u = 0; u < LOADS; ++u) local.kept[j][u][tid] = kept[j][u];
      __builtin_amdgcn_sched_barrier(0);
      ask(SLOTS + j, kept[j]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int j = 0; j < SLOTS; ++j) look(LDS_UNITS + j, kept[(j + LDS_UNITS) % SLOTS]);
  hand_over();
  __syncthreads();

  const bool starts_inside = q0 % per_channel != 0;           // the first channel began before
  const bool ends_inside = (q0 + count) % per_channel != 0;   // the last one goes on behind
  if (g.shared != 0) {
    uint32_t thread = threadIdx.x;
    asm volatile("" : "+v"(thread));
    const bool one = ch_lo == ch_hi;
    // what the workgroup shares: e = 0 its first channel, 1 its last one
    auto watched = [&](int e) { return e == 0 ? starts_inside || (one && ends_inside) : !one && ends_inside; };
    // the workgroups that have a part of channel ch, the list's members; it is the first channel of all but the first
    auto first_of = [&](uint32_t ch) { return ch * per_channel / g.per; };
    auto members = [&](uint32_t ch) { return int((ch * per_channel + per_channel - 1) / g.per - first_of(ch) + 1); };
    auto boxes = [&](uint32_t ch) {
      const uint32_t from = first_of(ch);
      const bool its_first = from * g.per == ch * per_channel;
      return [=](int i) { return (i > 0 || its_first ? mail->first : mail->last) + from + i; };
    };
    if (thread == 0 && watched(0)) post(mail->first + blockIdx.x, tag, u32_as_f32(local.top[0]));
    if (thread == 0 && watched(1)) post(mail->last + blockIdx.x, tag, u32_as_f32(local.top[nloc - 1]));
    __syncthreads();
    // four wavefronts look for the first channel's other workgroups, four for the last one's
    const int half = wave / (kHeldGrid / kWave);
    if (watched(half)) {
      const uint32_t ch = half == 0 ? ch_lo : ch_hi;
      const int i = int(thread % uint32_t(kHeldGrid));
      if (members(ch) >= kManyLook) __builtin_amdgcn_s_sleep(24);
      const uint64_t missing = look_for_mail(i, members(ch), tag, polls, local.ex[half], boxes(ch));
      if (i % kWave == 0) {
        atomicMax(&local.top[ch - ch_lo], f32_as_u32(local.ex[half].top[i / kWave]));
        if (missing != 0) local.late = 1;
      }
    }
    __syncthreads();
    const bool late = __builtin_amdgcn_readfirstlane(local.late) != 0;
    if (ASIDE > 0 && late) {
#pragma unroll
      for (int u = 0; u < ASIDE; ++u) local.aside[u][thread] = kept[SLOTS - 1][u];
    }
#pragma nounroll
    for (int e = 0; e < 2 && late; ++e) {
      if (!watched(e)) continue;  // the same in all threads
      const uint32_t ch = e == 0 ? ch_lo : ch_hi;
      const uint32_t from = first_of(ch);
      post_missing(tag, local.ex[e], boxes(ch), [&](int i) {  // the channel's groups that workgroup from + i has
        const uint32_t begin = max(ch * per_channel, (from + uint32_t(i)) * g.per);
        const uint32_t behind = min((ch + 1) * per_channel, (from + uint32_t(i) + 1) * g.per);
        const uint32_t at0 = group_pos(g, begin).at;
        GroupPos p = group_pos(g, begin + thread / uint32_t(GV));
        float v = 0.0f;
#pragma nounroll
        for (uint32_t q = begin; q < behind; q += ASK * (kHeldBlock / GV)) {
          uint4 raw[ASK];
#pragma unroll
          for (int u = 0; u < ASK; ++u) {
            const uint32_t at = q + uint32_t(u * (kHeldBlock / GV)) + thread / uint32_t(GV) < behind ? p.at : at0;
            raw[u] = load16_stream(reinterpret_cast<const char*>(x) + (at * uint32_t(GV) + thread % uint32_t(GV)) * 16u);
            group_advance(g, p, g.load_step);
          }
#pragma unroll
          for (int u = 0; u < ASK; ++u) {
            float f[VEC];
            widen(raw[u], f);
#pragma unroll
            for (int k = 0; k < VEC; ++k) v = fmaxf(v, fabsf(f[k]));
          }
        }
        return v;
      }, [&](int i, float v) { if (thread == 0) post(boxes(ch)(i), tag, v); });
      if (thread == 0) local.top[ch - ch_lo] = f32_as_u32(largest_mail(local.ex[e]));
    }
    if (ASIDE > 0 && late) {
#pragma unroll
      for (int u = 0; u < ASIDE; ++u) kept[SLOTS - 1][u] = local.aside[u][thread];
    }
    if (late) __syncthreads();
    count_exchanges(mail, tag - 1u, 1u);
  }
  if (tid < int(nloc)) {
    float s, r;
    scale_from_range(u32_as_f32(local.top[tid]), K, s, r);
    local.r[tid] = r;
    if (tid > 0 || !starts_inside) header[ch_lo + tid] = s;
  }
  __syncthreads();

  constexpr int PARTS = CodeParts<K>::PARTS;
  GroupPos to = group_pos(g, q0 + uint32_t(tid) / PARTS);  // the group a part of whose codes the thread writes next
  const __amdgpu_buffer_rsrc_t codes = payload_buffer(payload32, g.total * uint32_t(K * 4));
  int buf_i = 0;
  chan = 0;
  end = first_end < count ? first_end : count;
  float r_chan = local.r[0];
  auto quantize_unit = [&](uint32_t ordinal, auto vec_of) {
    uint32_t* buf = local.pieces[buf_i];
    buf_i ^= 1;
    const uint32_t g0 = ordinal * kHeldBlock;
    auto vector = [&](int u, float r) {
      uint4 raw = vec_of(u);
      // (an empty asm: the values widened for the maximum would stay in registers from then to here)
      asm volatile("" : "+v"(raw.x), "+v"(raw.y), "+v"(raw.z), "+v"(raw.w));
      float f[VEC];
      widen(raw, f);
      const float rv[4] = {r, r, r, r};
#pragma unroll
      for (int h = 0; h < QPV; ++h) buf[(u * kHeldBlock + tid) * QPV + h] = quantize4<K, false>(&f[4 * h], rv, 0);
    };
    float r[LOADS];
#pragma unroll
    for (int u = 0; u < LOADS; ++u) r[u] = r_chan;
    while (end < g0 + kHeldBlock && end < count) {  // the same in all lanes
      r_chan = local.r[++chan];
#pragma unroll
      for (int u = 0; u < LOADS; ++u) r[u] = g0 + uint32_t(u * (kHeldBlock / GV)) + mine >= end ? r_chan : r[u];
      end = end + per_channel < count ? end + per_channel : count;
    }
#pragma unroll
    for (int u = 0; u < LOADS; ++u) vector(u, r[u]);
    __syncthreads();  // double buffered: one barrier per unit
#pragma unroll
    for (int i = 0; i < PARTS; ++i) {
      const uint32_t part = uint32_t(i * kHeldBlock + tid);
      uint32_t out[CodeParts<K>::DWORDS];
      pack_part<K>(&buf[part * CodeParts<K>::PIECES], out);
      fresh(to);
      if (g0 + part / PARTS < count)
        store_part<K>(codes, (to.at * uint32_t(K) + part % PARTS * CodeParts<K>::DWORDS) * 4u, out);
      group_advance(g, to, g.part_step);
    }
  };
  if constexpr (LDS_UNITS > 0) {
    for (int q = 0; q < LDS_UNITS; ++q)
      quantize_unit(q, [&](int u) { return local.kept[q][u][tid]; });
  }
#pragma unroll
  for (int j = 0; j < SLOTS; ++j)
    if (uint32_t(LDS_UNITS + j) < units) quantize_unit(LDS_UNITS + j, [&](int u) { return kept[(j + LDS_UNITS) % SLOTS][u]; });
}

// U1, U1b, U2 and U3 of a tensor with one range, in one kernel and with one read: small tensors, where a kernel more
// is a launch more, and larger ones, whose second read it saves.  Workgroup b has the groups of 32 elements b*per ..
// (b+1)*per - 1, all of them in registers; the last one also has the up to 31 elements behind the last group.  The
// workgroups' maxima are exchanged as in the held pass; one that has to find others' itself keeps
// what it has.
// Latency bounds it: the loads, a mailbox's way to memory and back (2 us), the stores.  Figures are at whole_groups.
template <typename T, int K, int SLOTS, bool STOCH>
__global__ __launch_bounds__(kHeldBlock, 2) void quantize_whole_kernel(const T* __restrict__ x,
                                                                       uint32_t* __restrict__ payload32,
                                                                       float* __restrict__ header,
                                                                       ChipMail* __restrict__ mail, int64_t N,
                                                                       uint32_t per, int64_t payload_bytes, uint64_t seed,
                                                                       int polls) {
  constexpr int VEC = Elem<T>::VEC;
  constexpr int GV = 32 / VEC;                            // vectors of a group
  constexpr int LOADS = kUnitElems / (kHeldBlock * VEC);  // vectors per thread and unit
  constexpr int QPV = VEC / 4, WAVES = kHeldBlock / kWave;
  __shared__ __attribute__((aligned(16))) uint32_t pieces[2][kUnitElems / 4];
  __shared__ Exchange ex;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const uint32_t total = uint32_t(N / 32);
  auto groups_of = [&](uint32_t w) { return total - w * per < per ? total - w * per : per; };
  const uint32_t q0 = blockIdx.x * per, count = groups_of(blockIdx.x);
  const uint32_t units = (count + kHeldBlock - 1) / kHeldBlock;
  const uint32_t mine = uint32_t(tid) / GV;  // the thread's first vector is in this group of the workgroup's
  const T* const xw = x + size_t(q0) * 32;
  // elements behind the last group, of the last workgroup
  const T* const xt = x + size_t(total) * 32;
  const int tail = blockIdx.x + 1 == gridDim.x ? int(N - int64_t(total) * 32) : 0;
  uint4 kept[SLOTS][LOADS];
#pragma unroll
  for (int j = 0; j < SLOTS; ++j)
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      const uint32_t grp = uint32_t(j * kHeldBlock + u * (kHeldBlock / GV)) + mine;
      // (behind the last group the first vector stands in)
      const uint32_t v = grp < count ? uint32_t((j * LOADS + u) * kHeldBlock + tid) : 0u;
      kept[j][u] = load16_stream(xw + size_t(v) * VEC);
    }
  // (asked for behind the tensor's loads, which do not wait for it: in front of them it took 0.2 to 0.5 us)
  const uint32_t tag = mail->calls[blockIdx.x] + 1u;
  float c = tid < tail ? fabsf(load_one(xt + tid)) : 0.0f;
#pragma unroll
  for (int j = 0; j < SLOTS; ++j)
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      float f[VEC];
      widen(kept[j][u], f);
#pragma unroll
      for (int e = 0; e < VEC; ++e) c = fmaxf(c, fabsf(f[e]));
    }
  c = wave_max(c);
  if (lane == 0) ex.top[wave] = c;
  __syncthreads();
  if (gridDim.x > 1) {
    // Many workgroups that look at the same boxes wait for each other there: every value is posted six times then, and
    // each workgroup looks at one set of boxes.  One set / six (us, k = 4): 1.05 M float32 5.12 / 4.89, 2.1 M 6.80 / 5.68, 8.3 M
    // 10.9 / 10.2, 4.2 M bfloat16 6.3 / 5.5; 65536 (4 workgroups) 3.95 / 4.1, so only from 32 workgroups on.
    constexpr int SETS = 6;
    const bool many = gridDim.x >= uint32_t(kManyLook);
    auto box_of = [&](int set, int w) { return set < 3 ? mail->first + set * kHeldGrid + w : between_box(mail, set - 3, w); };
    static_assert(offsetof(ChipMail, more) == 2 * sizeof(mail->first) && offsetof(ChipMail, last) == sizeof(mail->first), "sets 0 to 2 in a row");
    auto put = [&](int w, float v) { if (tid < (many ? SETS : 1)) post(box_of(tid, w), tag, v); };
    if (tid < SETS) {
      c = ex.top[0];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) c = fmaxf(c, ex.top[w]);
      put(int(blockIdx.x), c);
    }
    __syncthreads();
    const int mine_set = many ? int(blockIdx.x % uint32_t(SETS)) : 0;
    auto box = [&](int w) { return box_of(mine_set, w); };
    if (wave < kHeldGrid / kWave) {
      if (many) __builtin_amdgcn_s_sleep(16);
      look_for_mail(tid, int(gridDim.x), tag, polls, ex, box);
    }
    __syncthreads();
    if (missing_count(ex) != 0)
      post_missing(tag, ex, box, [&](int w) {
        float v = w + 1 == int(gridDim.x) && tid < int(N - int64_t(total) * 32) ? fabsf(load_one(xt + tid)) : 0.0f;
        const T* const xo = x + size_t(w) * per * 32;
        for (uint32_t i = tid; i < groups_of(w) * GV; i += kHeldBlock) {
          float f[VEC];
          load_vec(xo + size_t(i) * VEC, f);
#pragma unroll
          for (int e = 0; e < VEC; ++e) v = fmaxf(v, fabsf(f[e]));
        }
        return v;
      }, put);
    c = largest_mail(ex);
    count_exchanges(mail, tag - 1u, 1u);
  } else {
    c = ex.top[0];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) c = fmaxf(c, ex.top[w]);
  }
  float s, r;
  scale_from_range(c, K, s, r);
  if (blockIdx.x == 0 && tid == 0) header[0] = s;
  const float rv[4] = {r, r, r, r};

  // random state of the thread's first element; its other vectors' are whole steps of a unit's share behind it
  const uint64_t z0 = STOCH ? rand_state(seed, uint64_t(q0) * 32 + uint64_t(tid) * VEC) : 0;
#pragma unroll
  for (int j = 0; j < SLOTS; ++j) {
    if (uint32_t(j) >= units) break;  // the same in all threads
    uint32_t* buf = pieces[j & 1];
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      if (uint32_t(j * kHeldBlock + u * (kHeldBlock / GV)) >= count) break;  // the same in all threads: nothing but stand-ins
      uint4 raw = kept[j][u];
      // (an empty asm: the values widened for the maximum would stay in registers from then to here)
      asm volatile("" : "+v"(raw.x), "+v"(raw.y), "+v"(raw.z), "+v"(raw.w));
      float f[VEC];
      widen(raw, f);
      const uint64_t z = z0 + uint64_t((j * LOADS + u) * kHeldBlock * VEC) * kRandStep;
#pragma unroll
      for (int h = 0; h < QPV; ++h)
        buf[(u * kHeldBlock + tid) * QPV + h] = quantize4<K, STOCH>(&f[4 * h], rv, z + uint64_t(4 * h) * kRandStep);
    }
    __syncthreads();  // double buffered: one barrier per unit
    constexpr int PARTS = CodeParts<K>::PARTS;
    const __amdgpu_buffer_rsrc_t codes = payload_buffer(payload32 + size_t(q0) * K, count * uint32_t(K * 4));
#pragma unroll
    for (int i = 0; i < PARTS; ++i) {
      const uint32_t part = uint32_t(i * kHeldBlock + tid);
      uint32_t out[CodeParts<K>::DWORDS];
      pack_part<K>(&buf[part * CodeParts<K>::PIECES], out);
      const uint32_t grp = uint32_t(j * kHeldBlock) + part / PARTS;
      if (grp < count) store_part<K>(codes, (grp * uint32_t(K) + part % PARTS * CodeParts<K>::DWORDS) * 4u, out);
    }
  }
  if (tid * 8 < tail)
    quantize_group8<T, K, STOCH>(x, reinterpret_cast<uint8_t*>(payload32), int64_t(total) * 4 + tid, N, payload_bytes, seed,
                                 [&](int64_t) { return r; });
}

}  // namespace

template <typename T>
hipError_t launch_whole(const accept_desc& d, const UPlan& p, const T* x, float* header, uint32_t* payload, ChipMail* mail,
                        int polls, hipStream_t s) {
  const uint32_t total = uint32_t(p.N / 32);
  const int grid = int((total + p.whole_per - 1) / p.whole_per);
  const int units = int((p.whole_per + kHeldBlock - 1) / kHeldBlock);
  const int64_t payload_bytes = (p.N * d.bits + 7) / 8;
  const bool stoch = d.rounding == ACCEPT_ROUND_STOCHASTIC;
  auto launch = [&](auto k, auto slots, auto st) {
    hipLaunchKernelGGL((quantize_whole_kernel<T, decltype(k)::value, decltype(slots)::value, decltype(st)::value>), dim3(grid),
                       dim3(kHeldBlock), 0, s, x, payload, header, mail, p.N, p.whole_per, payload_bytes, d.seed, polls);
  };
  auto sized = [&](auto k, auto st) {
    constexpr bool kOneUnit = sizeof(T) == 2 && decltype(st)::value;  // stochastic bfloat16 has no more
    static_assert(kWholeStochasticBf16 / 32 <= int64_t(kHeldGrid) * kHeldBlock, "one unit");
    if (units <= 1 || kOneUnit) launch(k, std::integral_constant<int, 1>{}, st);
    else if (units <= ChanSlots<T>::small) launch(k, std::integral_constant<int, kOneUnit ? 1 : ChanSlots<T>::small>{}, st);
    else launch(k, std::integral_constant<int, kOneUnit ? 1 : ChanSlots<T>::middle>{}, st);
  };
#define ACCEPT_WHOLE(KK)                                             \
  case KK:                                                           \
    if (stoch) sized(std::integral_constant<int, KK>{}, std::true_type{}); \
    else sized(std::integral_constant<int, KK>{}, std::false_type{}); \
    break;
  switch (d.bits) {
    ACCEPT_WHOLE(2) ACCEPT_WHOLE(3) ACCEPT_WHOLE(4) ACCEPT_WHOLE(5) ACCEPT_WHOLE(6) ACCEPT_WHOLE(7) ACCEPT_WHOLE(8)
    default: return hipErrorInvalidValue;
  }
#undef ACCEPT_WHOLE
  return hipGetLastError();
}

template <typename T>
hipError_t launch_held(const accept_desc& d, const UPlan& p, const T* x, float* header, uint32_t* payload,
                       ChipMail* mail, int polls, hipStream_t s) {
  const int64_t payload_bytes = (p.N * d.bits + 7) / 8;
#define ACCEPT_HELD(KK)                                                                                                 \
  case KK:                                                                                                              \
    hipLaunchKernelGGL((quantize_held_kernel<T, KK, kHeldUnits<T>>), dim3(kHeldGrid), dim3(kHeldBlock), 0, s, x, payload, \
                       header, mail, p.N, p.held_units, p.held_first, p.held_lds, payload_bytes, polls);                \
    break;
  switch (d.bits) {
    ACCEPT_HELD(2) ACCEPT_HELD(3) ACCEPT_HELD(4) ACCEPT_HELD(5) ACCEPT_HELD(6) ACCEPT_HELD(7) ACCEPT_HELD(8)
    default: return hipErrorInvalidValue;
  }
#undef ACCEPT_HELD
  return hipGetLastError();
}

template <typename T>
hipError_t launch_channels(const accept_desc& d, const UPlan& p, const T* x, float* header, uint32_t* payload,
                           ChipMail* mail, int polls, hipStream_t s) {
  ChanHeldGeom g{};
  g.seg_groups = uint32_t(p.seg_len / 32);
  g.rows = uint32_t(d.n);
  g.m_groups = uint32_t(p.m / 32);
  g.total = uint32_t(p.N / 32);
  g.per = p.chan_per;
  auto step = [&](uint32_t groups) {
    GroupPos st;
    const uint32_t segs = groups / g.seg_groups;
    st.pos = groups % g.seg_groups;
    const uint32_t chs = segs / g.rows;
    st.row = segs - chs * g.rows;
    st.at = st.row * g.m_groups + chs * g.seg_groups + st.pos;
    return st;
  };
  g.next_row = g.m_groups - g.seg_groups;
  g.next_channel = g.seg_groups - g.rows * g.m_groups;
  g.load_step = step(uint32_t(kHeldBlock * p.vec / 32));
  g.part_step = step(uint32_t(kHeldBlock / (d.bits == 6 || d.bits == 8 ? 2 : 1)));
  const uint32_t per_channel = g.rows * g.seg_groups;
  static_assert(kChanMaxUnits<T> * kHeldBlock * 32 / kChanMinChannel + 2 <= kChanMaxLocal, "channels of a workgroup");
  g.shared = g.per % per_channel != 0 ? 1u : 0u;
  const int grid = int((g.total + g.per - 1) / g.per);
  const int units = int((g.per + kHeldBlock - 1) / kHeldBlock);
  using S = ChanSlots<T>;
#define ACCEPT_CHAN(KK)                                                                                             \
  case KK:                                                                                                          \
    if (units <= S::small)                                                                                          \
      hipLaunchKernelGGL((quantize_channels_kernel<T, KK, S::small, 0>), dim3(grid), dim3(kHeldBlock), 0, s, x, payload, \
                         header, mail, g, polls);                                                             \
    else if (units <= S::middle)                                                                                    \
      hipLaunchKernelGGL((quantize_channels_kernel<T, KK, S::middle, 0>), dim3(grid), dim3(kHeldBlock), 0, s, x, payload, \
                         header, mail, g, polls);                                                             \
    else                                                                                                            \
      hipLaunchKernelGGL((quantize_channels_kernel<T, KK, S::large, kChanLdsUnits<T>>), dim3(grid), dim3(kHeldBlock), 0, s, \
                         x, payload, header, mail, g, polls);                                                 \
    break;
  switch (d.bits) {
    ACCEPT_CHAN(2) ACCEPT_CHAN(3) ACCEPT_CHAN(4) ACCEPT_CHAN(5) ACCEPT_CHAN(6) ACCEPT_CHAN(7) ACCEPT_CHAN(8)
    default: return hipErrorInvalidValue;
  }
#undef ACCEPT_CHAN
  return hipGetLastError();
}

}  // namespace accept
