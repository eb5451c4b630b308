// Scheme U's compressors that keep the tensor, or a part of it, on the chip between the range and the
// quantizer, and so read it once: which tensors take them (host).  One range per tensor: the held pass; one range
// per channel: the channels pass.  The kernels are compiled per input type (uniform_chip_f32.hip, uniform_chip_bf16.hip).
#pragma once

#include "uniform_quant.hpp"

namespace accept {

// The held pass (quantize_held_kernel): one workgroup per compute unit, two wavefronts per SIMD.
constexpr int kHeldBlock = 512;
constexpr int kUnitTiles = 2;
constexpr int kUnitElems = kUnitTiles * kTileElems;  // elements a workgroup takes at a time
template <typename T>
constexpr int kHeldVecs = 56;  // 16-byte vectors a thread keeps in registers (more would spill); 48: bfloat16 141 MB 38.6 / 37.1 us, 205 MB
                               // 64.4 / 60.8, 103 MB equal
constexpr int kHeldLdsVecs = 16;                     // and in local memory
template <typename T>
constexpr int kHeldUnits = kHeldVecs<T> * kHeldBlock * Elem<T>::VEC / kUnitElems;  // 7 (float32), 14 (bfloat16)
template <typename T>
constexpr int kHeldLdsUnits = kHeldLdsVecs * kHeldBlock * Elem<T>::VEC / kUnitElems;  // 2, 4
// Tensors that take the held pass.  Captured calls, two reads / held (us), when the held pass still had a second
// kernel (4 us) always: float32 51 MB 19.2 / 18.9 (15.5 now), 66 MB 23.3 / 21.1; bfloat16, whose values are twice as
// many, 51 MB 19.6 / 21.9, 72 MB 27.5 / 27.5 (22.8 now), 95 MB 35.2 / 32.8.  Above, the part that is kept gets small
// and the workgroups drift apart by more than they wait for each other: bfloat16 205 MB 75.9 / 67.7, 262 MB 96.1 /
// 94.2, 268 MB 98.3 / 95.2.  float32 gains beyond the line too (268 MB 89.6 / 79.5, 300 MB 110 / 97, 400 MB 149 /
// 150); it lies where both types do.
template <typename T>
constexpr int64_t kHeldMinBytes = int64_t(sizeof(T) == 4 ? 48 : 72) << 20;
constexpr int64_t kHeldMaxBytes = int64_t(256) << 20;
static_assert(kHeldMinBytes<float> / 4 >= int64_t(kHeldGrid) * kUnitElems, "every workgroup has a unit");
static_assert(kHeldMinBytes<bf16_t> / 2 >= int64_t(kHeldGrid) * kUnitElems, "every workgroup has a unit");

constexpr int kChanMaxLocal = 64;   // channels a workgroup may have a part of: at most 14 units of 512 groups, and
                                    // two parts, of channels of at least 128 groups
template <typename T>
constexpr int kChanLdsUnits = sizeof(T) == 4 ? 1 : 3;
// Registers for the units of a workgroup: three sizes, so that small tensors do not carry the large ones' loads.
template <typename T>
struct ChanSlots;
template <>
struct ChanSlots<float> {
  static constexpr int small = 2, middle = 4, large = 6;
};
template <>
struct ChanSlots<bf16_t> {
  static constexpr int small = 3, middle = 6, large = 11;
};
template <typename T>
constexpr int64_t kChanMaxUnits = ChanSlots<T>::large + kChanLdsUnits<T>;

// Groups of a workgroup of quantize_channels_kernel; 0: the tensor does not take it.  Segments have to be whole
// groups, and the tensor has to fit on the chip.  Against range and quantize kernels (two, or three with one
// that finishes the ranges between them; captured calls, us): 64 x 256 x 3136 bfloat16 k = 6 43.3 / 33.2, 32 x 256 x
// 3136 float32 38.4 / 26.8, 16 x 512 x 1024 15.5 / 10.4, 8 x 32 x 12544 10.7 / 6.5, 130 x 30 x 256 bfloat16 27.6 / 6.2,
// 64 x 5859 x 64 29.9 / 27.8.  Channels of fewer than 8192 elements are handed over often, which large tensors
// pay for: 4 x 5859 x 1024 bfloat16 26.2 / 27.9, 4 x 2441 x 1024 15.6 / 13.8; float32 35.7 / 37.3, 19.1 / 18.0.
constexpr int64_t kChanMinChannel = 4096;
constexpr int64_t kChanManyValues = int64_t(10) << 20;  // beyond, channels have twice that at least
// The fewest groups of a workgroup: 32 to 256 take the same time where channels are shared; fewer
// workgroups then have fewer mailboxes to look through.
constexpr int64_t kChanMinGroups = 128;
template <typename T>
inline uint32_t channel_groups(int64_t n, int64_t C, int64_t seg_len) {
  const int64_t groups = n * C * seg_len / 32, most = kChanMaxUnits<T> * kHeldBlock;
  if (seg_len % 32 != 0 || groups > most * kHeldGrid) return 0;
  if (n * seg_len < (groups * 32 > kChanManyValues ? 2 : 1) * kChanMinChannel) return 0;
  int64_t per = (groups + kHeldGrid - 1) / kHeldGrid;
  if (per < kChanMinGroups) per = kChanMinGroups;
  // Whole channels, if that is hardly more work for a workgroup: nothing is shared then, and nobody waits
  // (8 x 61 x 1024 bfloat16: 5.5 -> 4.1 us).
  const int64_t channel = n * seg_len / 32, whole = (per + channel - 1) / channel * channel;
  if (whole <= kHeldBlock || whole * 8 <= per * 9) per = whole;
  return uint32_t(per < most ? per : most);
}

template <typename T>
hipError_t launch_held(const accept_desc& d, const UPlan& p, const T* x, float* header, uint32_t* payload,
                       ChipMail* mail, int polls, hipStream_t s);
template <typename T>
hipError_t launch_channels(const accept_desc& d, const UPlan& p, const T* x, float* header, uint32_t* payload,
                           ChipMail* mail, int polls, hipStream_t s);

template <typename T>
hipError_t launch_whole(const accept_desc& d, const UPlan& p, const T* x, float* header, uint32_t* payload, ChipMail* mail,
                        int polls, hipStream_t s);

// Groups of a workgroup of quantize_whole_kernel; 0: the tensor does not take it.  Range and quantize kernels / this
// (us on the device, replayed graphs; a launch less is about 3 us of host time on top):
//   nearest, float32: 5 K 5.3 / 3.4, 16 K 4.6 / 2.8, 100 K 5.8 / 4.3, 262144 5.0 / 4.3, 0.5 M 5.1 / 4.8, 1.05 M 5.1 / 5.2, 2.1 M
//     5.3 / 5.6, 2.5 M 6.9 / 6.1, 4.2 M 8.2 / 7.1, 8.3 M 11.8 / 10.6, 12 M 16.3 / 13.7; bfloat16: 0.5 M 4.9 / 4.6, 2.1 M 5.2 /
//     5.0, 8.3 M 9.5 / 8.1, 25 M 21.8 / 18.9;
//   stochastic, float32: 20 K 7.5 / 4.5, 300 K 7.8 / 5.4, 1 M 6.6 / 6.1, 4 M 11.0 / 10.3, 12.6 M 25.0 / 23.7, 16.7 M 31.0 to 35 /
//     30 to 31.7; bfloat16: 20 K 7.1 / 4.4, 1 M 6.5 / 5.9, 2.1 M 6.6 / 6.7, 3.1 M 8.5 / 7.7.
// Where two kernels are ahead there (whole tiles of 8192 values, 1 to 2.1 M float32) the replays find the input in the second-level
// cache, which the range kernel's loads leave it in; inputs that nothing has read before: 1.05 M 8.05 / 8.0, 1.57 M 8.2 / 7.9,
// 2.1 M 8.05 / 8.2, 3.1 M 9.5 / 8.9.
// Above, nearest, float32 begins the held pass (12.6 M values, three units); bfloat16 would need nine units, whose loads take
// longer than two reads (26 M 19.0 / 42.5).
template <typename T>
constexpr int64_t kWholeNearestUnits = ChanSlots<T>::middle;
constexpr int64_t kWholeStochasticBf16 = int64_t(3) << 20;
// The fewest groups of a workgroup: fewer workgroups have fewer mailboxes to look through, one has none; the random
// numbers want more of them, and so do large float32 tensors.  128 / 512 groups: nearest, 16 K 3.9 / 3.0, 1 M 6.4 /
// 5.8; stochastic, 20 K 4.5 / 6.6, 1 M 7.1 / 8.8.  256 / 512 groups, nearest: float32 1.05 M 5.2 / 4.9, 1.5 M 5.5 / 5.3, 1.57 M
// 5.3 / 5.7, 2.1 M 5.3 / 5.7, 3.1 M 6.4 / 6.6; bfloat16 1.05 M 4.8 / 4.8, 2.1 M 5.1 / 5.0, 4.2 M 5.7 / 5.5.
constexpr int64_t kWholeMinGroups = kHeldBlock, kWholeMinGroupsStochastic = 128;
template <typename T>
constexpr int64_t kWholeSmallerParts = sizeof(T) == 4 ? int64_t(3) << 19 : INT64_MAX;  // values from which parts of half as many will do
template <typename T>
inline uint32_t whole_groups(int64_t N, bool stochastic) {
  const int64_t groups = N / 32;
  const int64_t units = stochastic ? ChanSlots<T>::middle : kWholeNearestUnits<T>;
  if (groups < 1 || groups > units * kHeldBlock * kHeldGrid) return 0;
  if (stochastic && sizeof(T) == 2 && N > kWholeStochasticBf16) return 0;
  const int64_t per = (groups + kHeldGrid - 1) / kHeldGrid;
  const int64_t least = stochastic ? kWholeMinGroupsStochastic : N >= kWholeSmallerParts<T> ? kWholeMinGroups / 2 : kWholeMinGroups;
  return uint32_t(per < least ? least : per);
}

}  // namespace accept
