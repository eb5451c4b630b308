// The kernels of uniform_chip.hpp.
#pragma once

#include <atomic>

#include "uniform_chip.hpp"

namespace accept {

// What the workgroups of calls with one workspace leave each other, in its control block.  A call's tag is one
// more than the number of calls before it, of which every workgroup has a word of its own: it reads the
// word when it starts and raises it when it ends (and those of the workgroups that this call does not have),
// so all of them agree.  So nothing has to be emptied: a value of an earlier call bears an earlier tag.
// (Counting the workgroups off on one counter, and the last one emptying everything, cost small tensors
// 1.5 us.)
struct ChanMail {
  uint64_t first[kHeldGrid], last[kHeldGrid];  // tag and the workgroup's maximum of its first, its last channel
  uint32_t calls[kHeldGrid];
};

namespace {

// U1, and U2 + U3 for the end of the tensor, in one kernel (one range for the tensor, rounding to
// nearest).  The range has to be known before the first element can be quantized, so the plain way
// reads the tensor twice, and the memory-side cache does not help: it delivers 7.4 TB/s, memory
// itself 7.2.  The registers and local memories of the chip hold 168 MiB, though.  Here one workgroup per compute unit
// reads units (16384 elements) b, b + 256, ..., keeps the last of them (float32: 7 units in registers
// and 2 in local memory, 151 MB over the chip; bfloat16: 12 and 4, 134 MB), hands its maximum to the
// other workgroups through a mailbox, waits for theirs, quantizes what it kept and reads the units
// before held_first once more.  quantize_pack_kernel does the up to 16383 elements behind the last
// whole unit; for the range every workgroup looks at 64 of them here.
//
// The wait is bounded: nothing says that all 256 workgroups run at the same time (another kernel may
// hold some compute units).  A workgroup that has not seen all mailboxes after `polls` looks gives
// up, says so in its record and ends; quantize_pack_kernel then takes its units too.  So every
// workgroup ends whatever else runs, and the result does not depend on it.
//
// Beside other work: a workgroup needs a whole compute unit (160 KiB of local memory, all registers), so
// next to a kernel whose workgroups keep filling the chip it starts late, and the early ones give up.
// Time of a call on one stream while another stream is busy, two reads / held (us): small elementwise
// kernels, 100 MB float32 43 / 32, 205 MB 85 / 70, 100 MB bfloat16 53 / 39; matrix products 155 / 149,
// 184 / 179, 160 / 155; copies of 512 MB without a pause 66 / 98, 130 / 161, 72 / 145.
//
// A mailbox is one 64-bit word, value and the call's mark together, written and read with device-scope
// accesses (they bypass the dies' second-level caches): no ordering between two words is needed.
// quantize_pack_kernel empties the mailboxes, so that a captured call finds none of its own mark when it
// is replayed; what a call left whose second kernel could not be launched bears another mark.
//
// 51.4 M float32 values (205 MB), k = 8: 59.4 us a call against 69.5 with two reads (range 32.8,
// quantize 38.0); here 32.7 us to the mailboxes, 15 us of quantizing, 4 us of kernel end, 4.5 us for
// the other kernel.  100 MB: 30.7 against 38.0; bfloat16 103 MB: 35.1 against 44.8.
// Stochastic rounding keeps the two reads: it is bound by its instructions, which the second read
// hides behind.
template <typename T, int K>
__global__ __launch_bounds__(kHeldBlock, 2) void quantize_held_kernel(const T* __restrict__ x,
                                                                      uint32_t* __restrict__ payload32,
                                                                      float2* __restrict__ records,
                                                                      uint64_t* __restrict__ mail, int64_t N,
                                                                      int64_t units, int64_t held_first, int lds_units,
                                                                      int polls, uint32_t mark) {
  constexpr int VEC = Elem<T>::VEC;
  constexpr int LOADS = kUnitElems / (kHeldBlock * VEC);  // vectors per thread and unit
  constexpr int SLOTS = kHeldUnits<T>;
  constexpr int RING = 32 / (4 * LOADS) * 2;  // units in flight while nothing is kept yet: 128 KiB per workgroup
  constexpr int WAVES = kHeldBlock / kWave;
  constexpr int LDS_UNITS = kHeldLdsUnits<T>;
  static_assert(SLOTS * LOADS == kHeldVecs<T> && RING >= 2 && RING < SLOTS, "registers");
  static_assert(LDS_UNITS % RING == 0 && LDS_UNITS < SLOTS, "units kept in local memory pass through the ring in whole turns");
  constexpr int PIECES = kUnitElems / 4;
  constexpr int QPV = VEC / 4;
  // local memory, all 160 KiB of it: what is kept, and two buffers of pieces (the first of which the
  // reductions use before)
  struct Local {
    uint4 kept[LDS_UNITS][LOADS][kHeldBlock];
    uint32_t pieces[2][PIECES];
  };
  static_assert(sizeof(Local) <= 160 * 1024, "local memory of a compute unit");
  __shared__ __attribute__((aligned(16))) Local local;
  float* const red = reinterpret_cast<float*>(local.pieces[0]);
  int* const red_up = reinterpret_cast<int*>(local.pieces[0]) + WAVES;
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

  c = wave_max(c);
  if (lane == 0) red[wave] = c;
  __syncthreads();
  c = red[0];
#pragma unroll
  for (int w = 1; w < WAVES; ++w) c = fmaxf(c, red[w]);
  const float mine = c;
  if (tid == 0)
    __hip_atomic_store(mail + blockIdx.x, (uint64_t(mark) << 32) | f32_as_u32(mine), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();  // red is free again
  if (tid < kHeldGrid) {  // wavefront w watches mailboxes 64w .. 64w+63
    uint64_t v = 0;
    bool all = false;
    for (int i = 0; i < polls; ++i) {
      v = __hip_atomic_load(mail + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      all = __ballot(uint32_t(v >> 32) != mark) == 0;
      if (all) break;
      __builtin_amdgcn_s_sleep(4);
    }
    const float cw = wave_max(u32_as_f32(uint32_t(v)));
    if (lane == 0) { red[wave] = cw; red_up[wave] = all ? 0 : 1; }
  }
  __syncthreads();
  int up = 0;
  c = 0.0f;
#pragma unroll
  for (int w = 0; w < kHeldGrid / kWave; ++w) { c = fmaxf(c, red[w]); up |= red_up[w]; }
  up = __builtin_amdgcn_readfirstlane(up);
  if (tid == 0) records[blockIdx.x] = make_float2(mine, up ? 0.0f : 1.0f);
  if (up) return;

  float s, r;
  scale_from_range(c, K, s, r);
  float rv[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) rv[e] = r;
  int buf_i = 0;
  auto quantize_unit = [&](int ordinal, auto vec_of) {
    uint32_t* buf = local.pieces[buf_i];
    buf_i ^= 1;
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      float f[VEC];
      widen(vec_of(u), f);
#pragma unroll
      for (int h = 0; h < QPV; ++h) buf[(u * kHeldBlock + tid) * QPV + h] = quantize4<K, false>(&f[4 * h], &rv[4 * h], 0);
    }
    __syncthreads();  // double buffered: one barrier per unit
    const uint4 a = *reinterpret_cast<const uint4*>(&buf[8 * tid]);
    const uint4 b = *reinterpret_cast<const uint4*>(&buf[8 * tid + 4]);
    const uint32_t P[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t out[K];
    pack8<K>(P, out);
    store_dwords<K>(payload32 + ((int64_t(ordinal) * kHeldGrid + blockIdx.x) * kHeldBlock + tid) * K, out);
  };
  __syncthreads();  // the reductions' words are free: pieces from here on
  // A slot that has been quantized takes a unit that was only looked at, the last of them first;
  // those loads are under way while the other kept units are quantized.  (Conditions are the same
  // in all threads.)
#pragma unroll
  for (int j = 0; j < SLOTS; ++j) {
    if (base + j < count) quantize_unit(base + j, [&](int u) { return kept[j][u]; });
    if (j < first) ask(first - 1 - j, kept[j]);
  }
  if (lds_units != 0) {
    for (int q = 0; q < LDS_UNITS; ++q) quantize_unit(first + q, [&](int u) { return local.kept[q][u][tid]; });
  }
  for (int o = first - 1; o >= 0; o -= SLOTS) {
#pragma unroll
    for (int j = 0; j < SLOTS; ++j) {
      if (o - j >= 0) {
        quantize_unit(o - j, [&](int u) { return kept[j][u]; });
        if (o - j - SLOTS >= 0) ask(o - j - SLOTS, kept[j]);
      }
    }
  }
}

// U1, U1b, U2 and U3 of a tensor with one range per channel, in one kernel and with one read: the
// tensor stays on the chip between the two steps.  The tensor's groups of 32 elements (k whole dwords
// of payload each; segments are whole groups) are numbered channel after channel, row after row inside a
// channel, and workgroup b has the groups b*per .. (b+1)*per - 1 of that order: most of its channels are
// its own altogether, and at most two, its first and its last, it shares with neighbours.  For these it
// leaves its maximum in a mailbox and looks for those of the others.  Workgroups are not sure to run at
// the same time; one that has looked `polls` times in vain reads the whole channel itself.  So every
// workgroup ends whatever else runs, with the same bits.
//
// A mailbox is one 64-bit word, value and the call's mark together, as in quantize_held_kernel.  Every
// workgroup counts itself off once it has all its ranges; the one that is counted last empties the
// mailboxes and the count.
//
// What bounds it: the read of the tensor (16 of 33 us at 103 MB of bfloat16, with the looking hidden behind
// it), then the instructions that quantize and pack, two wavefronts on a SIMD, and the payload's stores
// (38 MB there).  The places of a thread's vectors are stepped, not divided out, and only the loads and
// stores need them: which channel a unit belongs to is known from scalars (per element, as at first, the
// kernel took 42 us).  Streaming stores of the payload make a call alone 3 us faster and a decoder that
// reads it next 8 us slower.  Beside other work on another stream, two or three kernels / this one (us):
// matrix products 220 / 114 (100 x 8 x 12544 float32), small kernels 29.0 / 20.6 (64 x 100 x 3136 float32); 512 MB
// copies without a pause 42 / 23 there, but 60 / 80 to 105 for the large one, whose workgroups need a compute
// unit each.
// Place of a group of 32 elements: group inside its segment, batch row, and the group's number in the tensor.
struct GroupPos {
  uint32_t pos, row, at;
};
struct ChanHeldGeom {
  uint32_t seg_groups, rows;  // groups of a segment, batch rows
  uint32_t m_groups;          // groups of a row of the tensor
  uint32_t total, per;        // groups of the tensor, and of a workgroup
  GroupPos load_step;         // groups between two loads of a thread
  GroupPos unit_step;         // groups of a unit
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

static_assert(kChanMailOffset + sizeof(ChanMail) <= kCtrlBytes, "the control block holds them");

template <typename T, int K, int SLOTS, int LDS_UNITS>
__global__ __launch_bounds__(kHeldBlock, 2) void quantize_channels_kernel(const T* __restrict__ x,
                                                                          uint32_t* __restrict__ payload32,
                                                                          float* __restrict__ header,
                                                                          ChanMail* __restrict__ mail, ChanHeldGeom g,
                                                                          int polls) {
  constexpr int VEC = Elem<T>::VEC;
  constexpr int GV = 32 / VEC;                            // vectors of a group
  constexpr int LOADS = kUnitElems / (kHeldBlock * VEC);  // vectors per thread and unit
  static_assert(LOADS * (kHeldBlock / GV) == kHeldBlock && kUnitElems == 32 * kHeldBlock, "a unit is a group per thread");
  static_assert(LDS_UNITS <= SLOTS, "units kept in local memory pass through the first slots");
  constexpr int QPV = VEC / 4;
  struct Local {
    uint4 kept[LDS_UNITS > 0 ? LDS_UNITS : 1][LDS_UNITS > 0 ? LOADS : 1][LDS_UNITS > 0 ? kHeldBlock : 1];
    uint32_t pieces[2][kUnitElems / 4];
    uint32_t top[kChanMaxLocal];  // largest magnitude of the workgroup's channels, as bits
    float r[kChanMaxLocal];
    int up[2];
  };
  static_assert(sizeof(Local) <= 160 * 1024, "local memory of a compute unit");
  __shared__ __attribute__((aligned(16))) Local local;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);

  const uint32_t q0 = blockIdx.x * g.per;  // below total (host)
  const uint32_t count = g.total - q0 < g.per ? g.total - q0 : g.per;
  const uint32_t units = (count + kHeldBlock - 1) / kHeldBlock;
  const uint32_t tag = mail->calls[blockIdx.x] + 1u;
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
  const uint32_t per_channel = g.rows * g.seg_groups;
  const uint32_t ch_lo = q0 / per_channel;
  const uint32_t ch_hi = (q0 + count - 1) / per_channel;
  const uint32_t nloc = ch_hi - ch_lo + 1;
  if (tid < kChanMaxLocal) local.top[tid] = 0u;
  if (tid < 2) local.up[tid] = 0;
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
    uint64_t* const mail_first = mail->first;
    uint64_t* const mail_last = mail->last;
    const bool one = ch_lo == ch_hi;
    const bool watch_first = starts_inside || (one && ends_inside), watch_last = !one && ends_inside;
    auto post = [&](uint64_t* box, uint32_t v) {
      __hip_atomic_store(box, (uint64_t(tag) << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (tid == 0 && watch_first) post(mail_first + blockIdx.x, local.top[0]);
    if (tid == 0 && watch_last) post(mail_last + blockIdx.x, local.top[nloc - 1]);
    __syncthreads();
    // wavefront 0 watches the first channel's other workgroups, wavefront 1 the last one's
    if ((wave == 0 && watch_first) || (wave == 1 && watch_last)) {
      const uint32_t ch = wave == 0 ? ch_lo : ch_hi;
      const uint32_t from_wg = ch * per_channel / g.per, to_wg = (ch * per_channel + per_channel - 1) / g.per;
      const bool from_first = from_wg * g.per == ch * per_channel;  // it is the first channel of workgroup from_wg
      uint32_t top = 0;
      bool all = false;
      for (int i = 0; i < polls; ++i) {
        bool seen = true;
        top = 0;  // (a look may have met values of earlier calls)
        for (uint32_t w = from_wg + uint32_t(lane); w <= to_wg; w += kWave) {
          const uint64_t* box = (w != from_wg || from_first ? mail_first : mail_last) + w;
          const uint64_t v = __hip_atomic_load(box, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          seen = seen && uint32_t(v >> 32) == tag;
          top = max(top, uint32_t(v));
        }
        all = __ballot(!seen) == 0;
        if (all) break;
        __builtin_amdgcn_s_sleep(4);
      }
      const float t = wave_max(u32_as_f32(top));
      if (lane == 0) {
        if (all) local.top[ch - ch_lo] = f32_as_u32(t);
        else local.up[wave] = 1;
      }
    }
    __syncthreads();
    for (int e = 0; e < 2; ++e) {
      if (local.up[e] == 0) continue;  // the same in all threads
      const uint32_t ch = e == 0 ? ch_lo : ch_hi;
      float v = 0.0f;
      const uint32_t seg_vecs = g.seg_groups * GV, vecs = g.rows * seg_vecs;
      for (uint32_t i = tid; i < vecs; i += kHeldBlock) {
        const uint32_t row = i / seg_vecs;
        float f[VEC];
        load_vec(x + (size_t(row) * g.m_groups + size_t(ch) * g.seg_groups) * 32 + size_t(i - row * seg_vecs) * VEC, f);
#pragma unroll
        for (int q = 0; q < VEC; ++q) v = fmaxf(v, fabsf(f[q]));
      }
      v = wave_max(v);
      if (lane == 0) atomicMax(&local.top[ch - ch_lo], f32_as_u32(v));
    }
    __syncthreads();
    if (tid < kHeldGrid && uint32_t(tid) % gridDim.x == blockIdx.x) mail->calls[tid] = tag;
  }
  if (tid < int(nloc)) {
    float s, r;
    scale_from_range(u32_as_f32(local.top[tid]), K, s, r);
    local.r[tid] = r;
    if (tid > 0 || !starts_inside) header[ch_lo + tid] = s;
  }
  __syncthreads();

  GroupPos to = group_pos(g, q0 + uint32_t(tid));  // the group whose codes the thread writes
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
    const uint4 a = *reinterpret_cast<const uint4*>(&buf[8 * tid]);
    const uint4 b = *reinterpret_cast<const uint4*>(&buf[8 * tid + 4]);
    const uint32_t P[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint32_t out[K];
    pack8<K>(P, out);
    fresh(to);
    if (g0 + uint32_t(tid) < count) store_dwords<K>(payload32 + size_t(to.at) * K, out);
    group_advance(g, to, g.unit_step);
  };
  if constexpr (LDS_UNITS > 0) {
    for (int q = 0; q < LDS_UNITS; ++q)
      quantize_unit(q, [&](int u) { return local.kept[q][u][tid]; });
  }
#pragma unroll
  for (int j = 0; j < SLOTS; ++j)
    if (uint32_t(LDS_UNITS + j) < units) quantize_unit(LDS_UNITS + j, [&](int u) { return kept[(j + LDS_UNITS) % SLOTS][u]; });
}

// Mark of a call's mailboxes: a running number, never 0 (an empty mailbox).
uint32_t next_mark() {
  static std::atomic<uint32_t> calls{0};
  uint32_t mark = 0;
  while (mark == 0) mark = calls.fetch_add(1, std::memory_order_relaxed) + 1;
  return mark;
}

}  // namespace

template <typename T>
hipError_t launch_held(const accept_desc& d, const UPlan& p, const T* x, uint32_t* payload, float* partials,
                       uint64_t* mail, int polls, hipStream_t s) {
  float2* records = reinterpret_cast<float2*>(partials);
  const uint32_t mark = next_mark();
#define ACCEPT_HELD(KK)                                                                                          \
  case KK:                                                                                                       \
    hipLaunchKernelGGL((quantize_held_kernel<T, KK>), dim3(kHeldGrid), dim3(kHeldBlock), 0, s, x, payload, records, \
                       mail, p.N, p.held_units, p.held_first, p.held_lds, polls, mark);                              \
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
                           ChanMail* mail, int polls, hipStream_t s) {
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
  g.unit_step = step(kHeldBlock);
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
