// Scheme M on gfx950: multi-bit quantization x ~ B alpha with batch bit planes (paper
// paragraphs "Forward Quantizer", "Forward Encoder", "Forward Decoder", "Forward
// Dequantizer"; eqs. (MBQ), (alpha solution), (alpha update), (biased error)).
//
// Work item = 8 batch rows (one row group) x VEC adjacent columns.  The eight row loads of
// a wavefront are each contiguous across lanes; the 8 x k bit transpose the encoder needs
// happens in registers (a per-level table holds each sign pattern "spread" to one bit per
// byte, and eight shift-or steps build the k plane bytes of a column), so the encoder needs
// no LDS exchange and its k*VEC output bytes per lane are contiguous across lanes.  The
// least-squares sums ride along in the same pass: bit counts come from popcounts of the
// finished plane bytes, B^T x from multiply-adds with the 0/1 plane bits.
#include <type_traits>

#include "common.hpp"

namespace accept {

namespace {

// Launch shapes.  The bit-plane encoder runs one workgroup of 8 wavefronts per compute unit
// (256 on this chip): the wavefronts of a compute unit share one set of tables in local memory.
// The comparison-layout encoder and the residue pass are plain 256-thread kernels.
constexpr int kEncBlock = 512;
constexpr int kEncWaves = kEncBlock / kWave;
// Wavefronts draw their work from counters in device memory; the workgroups with block indices
// 8i .. 8i+7 (under round-robin dispatch one on each of the chip's eight dies) share counter i.
constexpr int kGroupBlocks = 8;
// Wave-items a group takes out of every sweep over the tensor (as a shift; the rule is at WorkQueue).
constexpr uint8_t kGroupSlotsShift = 2, kWaveSlotsShift = 6;
constexpr int kCounterStride = 64;  // uint32 words between two counters (256 bytes: their own cache lines)
constexpr int kEncodeGridMax = 256;
constexpr int kPlainGridMax = 768;
constexpr int kDecodeGridMax = 8192;
constexpr int kInitGrid = 1024;
constexpr int kMaxRecords = 2048;  // per-workgroup records the workspace has room for
constexpr int kMaxWaves = 16;      // wavefronts of the largest workgroup
constexpr int kMaxGroups = kEncodeGridMax / kGroupBlocks;
static_assert(size_t(kMaxGroups) * kCounterStride * sizeof(uint32_t) <= kMailOffset, "the first half of the control block holds the counters");
static_assert(kEncodeGridMax <= kMaxRecords && kPlainGridMax <= kMaxRecords && kInitGrid <= kMaxRecords, "records");

template <int NDW>
struct alignas((NDW % 4 == 0) ? 16 : (NDW % 2 == 0) ? 8 : 4) Dwords {
  uint32_t v[NDW];
};

__host__ __device__ constexpr int nstat_of(int k) { return k + 1 + k + k * (k - 1) / 2; }

// Position of a work item (row group g, column vector jv), advanced without divisions.
struct ItemPos {
  int64_t g, jv;
};
struct ItemStep {
  int64_t dg, dj;
};
__device__ __forceinline__ void item_advance(ItemPos& p, const ItemStep& st, int64_t ipg) {
  p.jv += st.dj;
  p.g += st.dg;
  if (p.jv >= ipg) { p.jv -= ipg; p.g += 1; }
}

// M1: the 2^k levels sum_j(+-alpha_j) (float32 sums in the order j = 0..k-1 from 0), sorted
// ascending with ties by pattern.  Thread `pat` computes its level and its rank; on return
// lv_sorted[rank] and pat_sorted[rank] are filled (after the caller's barrier).
template <int K>
__device__ __forceinline__ void build_levels(const float (&alpha)[K], float* lv_raw, float* lv_sorted,
                                             uint32_t* pat_sorted) {
  constexpr int P = 1 << K;
  const int pat = threadIdx.x;
  float lv = 0.0f;
  if (pat < P) {
#pragma unroll
    for (int j = 0; j < K; ++j) lv = __fadd_rn(lv, ((pat >> j) & 1) ? alpha[j] : -alpha[j]);
    lv_raw[pat] = lv;
  }
  __syncthreads();
  if (pat < P) {
    int rank = 0;
    for (int q = 0; q < P; ++q) {
      const float o = lv_raw[q];
      rank += (o < lv || (o == lv && q < pat)) ? 1 : 0;
    }
    lv_sorted[rank] = lv;
    pat_sorted[rank] = uint32_t(pat);
  }
  __syncthreads();
}

// ================================================================ encode + sums (M1..M4)
// M2 without a per-element binary search.  The top 12 bits of a float32 (sign, exponent, three
// mantissa bits) name a bucket, i.e. an interval of reals.  For every bucket a table holds
// lo = number of thresholds below the whole bucket; the element's position among the sorted
// levels is then lo + #{c < maxcnt : x > tau[lo + c]}, where maxcnt is the largest number of
// thresholds that fall inside any one bucket (1 for well separated levels) and tau is padded
// with +inf.  The float compares decide; the table only says where to start, so the result is
// exactly #{i : x > tau_i}.
constexpr int kLutBits = 12;
constexpr int kLutSize = 1 << kLutBits;

template <int K>
struct EncodeTables {
  static constexpr int P = 1 << K;
  static constexpr int NW = (K + 3) / 4;  // spread words per level
  static constexpr int SORT = (K <= 4) ? 1 : P;  // k <= 4 sorts in registers
  float lv_raw[SORT];
  float lv_sorted[SORT];
  uint32_t pat_sorted[SORT];
  float tau[3 * P];                        // P-1 thresholds, then +inf padding (the windowed search reads past them)
  uint32_t spread[P * NW];                 // per sorted level: bit p of the sign pattern at bit 8*(p%4) of word p/4
  // k <= 4 only: row lo = {tau[lo] (or +inf), spread[lo]}, so that one 8-byte read at lo*8 and one
  // 4-byte read at lo*8 + 12 (= spread[lo+1]) give everything an element needs (two 8-byte reads
  // and one 4-byte read when a bucket may hold two thresholds)
  alignas(8) uint32_t pair[2 * (P + 2)];
  static constexpr int LUT_SHIFT = (K <= 4) ? 3 : 0;  // bucket table entries are lo << LUT_SHIFT
  alignas(4) uint8_t lut[kLutSize];
  int maxcnt;
};

// Smallest value of bucket b (bit patterns b << shift .. (b << shift) | low-ones); buckets of
// negative values run backwards in bit order.
__device__ __forceinline__ float bucket_vmin(int b) {
  const uint32_t lo_bits = uint32_t(b) << (32 - kLutBits);
  const uint32_t hi_bits = lo_bits | ((1u << (32 - kLutBits)) - 1u);
  return u32_as_f32((b >> (kLutBits - 1)) ? hi_bits : lo_bits);
}


// The bucket table and the largest number of thresholds inside one bucket.
//   lo(b) = #{tau_i < smallest value of bucket b}, through `count_below(value)`;
//   thresholds inside bucket b = lo(value-order successor of b) - lo(b).  The successor is b+1 on
//   the positive side (b < kLutSize/2) and b-1 on the negative side, where bucket kLutSize/2 (-0)
//   is followed by bucket 0.  Buckets of NaN bit patterns give differences <= 0: ignored.
// A thread takes CH = 8 consecutive buckets (two dwords of the table; never across the sign
// boundary).  lo is monotone along a side, and with a few thresholds among 4096 buckets almost
// every chunk has the same lo at both ends: then every bucket of it has that lo and no threshold
// inside, and only the step to the chunk's successor bucket is left to look at.  The few chunks
// with a threshold inside are then redone one after the other by the whole wavefront, lane j
// taking bucket j of the chunk (one evaluation per chunk instead of eight in a row by one lane).
template <int SHIFT, typename F>
__device__ __forceinline__ int build_bucket_table(uint8_t* lut, F count_below) {
  constexpr int CH = 8;
  static_assert(kLutSize % (2 * CH) == 0, "chunks stay on one side of the sign boundary");
  static_assert((kLutSize / CH) % kWave == 0, "all lanes of a wavefront run the same number of rounds");
  uint32_t* lut32 = reinterpret_cast<uint32_t*>(lut);
  const int lane = threadIdx.x & (kWave - 1);
  int mymax = 0;
  // Chunk c goes to thread (c * 67) mod 512 of its round: the thresholds sit in a few
  // neighbouring chunks (values of similar magnitude), and this spreads those chunks over the
  // wavefronts instead of leaving them all to one.
  constexpr int NCH = kLutSize / CH;
  static_assert(NCH == 512, "the chunk permutation below is a bijection on 512 chunks");
#pragma nounroll
  for (int slot = threadIdx.x; slot < NCH; slot += blockDim.x) {
    const int b0 = ((slot * 67) & (NCH - 1)) * CH;
    const bool neg = b0 >= kLutSize / 2;
    // the chunk's first and last bucket in value order, and the bucket that follows the last
    const int b_first = neg ? b0 + CH - 1 : b0;
    const int b_last = neg ? b0 : b0 + CH - 1;
    int b_succ = neg ? b0 - 1 : b0 + CH;
    if (neg && b0 == kLutSize / 2) b_succ = 0;                  // -0's bucket is followed by +0's
    const bool has_succ = neg || b0 + CH < kLutSize / 2;        // the top positive buckets hold NaN patterns
    const int lo_first = count_below(bucket_vmin(b_first));
    const int lo_last = count_below(bucket_vmin(b_last));
    const int lo_succ = has_succ ? count_below(bucket_vmin(b_succ)) : lo_last;
    const bool steps_inside = lo_first != lo_last;
    if (!steps_inside) {
      const int cnt = lo_succ - lo_last;
      mymax = cnt > mymax ? cnt : mymax;
    }
    const uint32_t fill = (uint32_t(lo_first) * 0x01010101u) << SHIFT;  // lo < 32 when shifted by 3: no carry between bytes
    lut32[b0 / 4] = fill;
    lut32[b0 / 4 + 1] = fill;
    // chunks with a threshold inside (their entries were just filled with a placeholder)
    uint64_t pending = __ballot(steps_inside);
    while (pending != 0) {  // the same in every lane
      const int src = __ffsll((unsigned long long)pending) - 1;
      pending &= pending - 1;
      const int cb0 = __builtin_amdgcn_readlane(b0, src);
      const int c_succ = __builtin_amdgcn_readlane(lo_succ, src);
      const bool cneg = cb0 >= kLutSize / 2;
      const int j = lane & (CH - 1);  // lanes 8.. repeat the work of lanes 0..7 (and store the same bytes)
      const int lo_j = count_below(bucket_vmin(cb0 + j));
      lut[cb0 + j] = uint8_t(uint32_t(lo_j) << SHIFT);
      // thresholds inside bucket cb0 + j: lo of its successor (inside the chunk, else the chunk's) minus its own
      const int lo_up = __shfl(lo_j, (lane & ~(CH - 1)) | ((j + 1) & (CH - 1)), kWave);
      const int lo_down = __shfl(lo_j, (lane & ~(CH - 1)) | ((j + CH - 1) & (CH - 1)), kWave);
      const int next = cneg ? (j > 0 ? lo_down : c_succ) : (j < CH - 1 ? lo_up : c_succ);
      const int cnt = next - lo_j;
      mymax = cnt > mymax ? cnt : mymax;
    }
  }
  return mymax;
}

// M1 for k <= 4 by one wavefront, in registers: lane p holds pattern p's level (float32 sum in the
// order j = 0..k-1 from 0).  Its rank is the number of levels below its own (ties by pattern); a
// lane-to-lane push hands every level to the lane of its rank.  Afterwards lane i < 2^k has the
// i-th level and its pattern, and tau_i (+inf from lane 2^k - 1 on).
template <int K>
__device__ __forceinline__ void sort_levels(const float (&alpha)[K], float& lv_s, uint32_t& pat_s, float& tau) {
  constexpr int P = 1 << K;
  const int pat = threadIdx.x & (kWave - 1);
  float lv = 0.0f;
#pragma unroll
  for (int j = 0; j < K; ++j) lv = __fadd_rn(lv, ((pat >> j) & 1) ? alpha[j] : -alpha[j]);
  int rank = 0;
#pragma unroll
  for (int q = 0; q < P; ++q) {
    const float o = u32_as_f32(uint32_t(__builtin_amdgcn_readlane(int(f32_as_u32(lv)), q)));
    rank += (o < lv || (o == lv && q < pat)) ? 1 : 0;
  }
  if (pat >= P) rank = pat;  // idle lanes push to themselves
  lv_s = u32_as_f32(uint32_t(__builtin_amdgcn_ds_permute(rank * 4, int(f32_as_u32(lv)))));
  pat_s = uint32_t(__builtin_amdgcn_ds_permute(rank * 4, pat));
  const float lv_next = u32_as_f32(uint32_t(__builtin_amdgcn_ds_bpermute(((pat + 1) & (kWave - 1)) * 4,
                                                                        int(f32_as_u32(lv_s)))));
  tau = pat < P - 1 ? __fmul_rn(0.5f, __fadd_rn(lv_s, lv_next)) : __builtin_inff();
}

// M1 and the search tables.  alpha[0..K) = the previous coefficients, already in registers (the
// caller loads them first thing, so that their trip to memory overlaps its other set-up work).
template <int K>
__device__ __forceinline__ void build_encode_tables(const float (&alpha)[K], EncodeTables<K>& tb) {
  using TB = EncodeTables<K>;
  constexpr int P = TB::P;
  const int tid = threadIdx.x;
  const int nthr = blockDim.x;  // at least P = 256 for K = 8
  int mymax = 0;
  if (tid == 0) tb.maxcnt = 1;
  if constexpr (K <= 4) {
    // Few levels: the first wavefront sorts them in registers; thresholds, spread patterns and the
    // pair table follow without a barrier.
    if (tid < kWave) {
      float lv_s, tau;
      uint32_t pat_s;
      sort_levels<K>(alpha, lv_s, pat_s, tau);
      uint32_t sp = 0;
#pragma unroll
      for (int bb = 0; bb < K; ++bb) sp |= ((pat_s >> bb) & 1u) << (8 * bb);
      if (tid < 3 * P) tb.tau[tid] = tau;  // 3P <= 48 lanes: thresholds, then +inf padding
      if (tid < P) tb.spread[tid] = sp;
      if (tid <= P + 1) {
        tb.pair[2 * tid] = f32_as_u32(tau);  // tau[P-1], tau[P], tau[P+1] are +inf
        tb.pair[2 * tid + 1] = tid < P ? sp : 0u;
      }
    }
    __syncthreads();
    // bucket table: the P-1 thresholds sit in registers, a bucket's lo is P-1 compares
    float t[P - 1];
#pragma unroll
    for (int i = 0; i < P - 1; ++i) t[i] = tb.tau[i];
    mymax = build_bucket_table<TB::LUT_SHIFT>(tb.lut, [&](float vmin) {
      int l = 0;
#pragma unroll
      for (int i = 0; i < P - 1; ++i) l += (t[i] < vmin) ? 1 : 0;
      return l;
    });
  } else {
    build_levels<K>(alpha, tb.lv_raw, tb.lv_sorted, tb.pat_sorted);
    for (int i = tid; i < 3 * P; i += nthr)
      tb.tau[i] = (i < P - 1) ? __fmul_rn(0.5f, __fadd_rn(tb.lv_sorted[i], tb.lv_sorted[i + 1])) : __builtin_inff();
    if (tid < P) {
      const uint32_t pat = tb.pat_sorted[tid];
#pragma unroll
      for (int w = 0; w < TB::NW; ++w) {
        uint32_t sp = 0;
#pragma unroll
        for (int bb = 0; bb < 4; ++bb)
          if (4 * w + bb < K) sp |= ((pat >> (4 * w + bb)) & 1u) << (8 * bb);
        tb.spread[tid * TB::NW + w] = sp;
      }
    }
    __syncthreads();
    // bucket table: tau[0..P-1) is sorted and tau[P-1] = +inf, so a branch-free binary search over
    // P entries finds lo
    mymax = build_bucket_table<TB::LUT_SHIFT>(tb.lut, [&](float vmin) {
      int l = 0;
#pragma unroll
      for (int s = P >> 1; s >= 1; s >>= 1) l += (tb.tau[l + s - 1] < vmin) ? s : 0;
      return l;
    });
  }
  if (mymax > 1) atomicMax(&tb.maxcnt, mymax);
  __syncthreads();
}

// M2 for bfloat16 input and k <= 4: 16 bits name a value outright, so a table of 65536 bytes holds
// the position among the sorted levels (times 4, the byte offset of its flag word) of every value
// there is: one byte read and one word read per element, no compare, and any spacing of the levels.
//
// A flag word has one byte per plane, 0xBF where the plane is +1 and 0 where it is -1.  A byte
// selector turns the words of two neighbouring elements into the pair (-0.5 or 0, -0.5 or 0) of
// bfloat16 numbers of one plane (0xBF00 is -0.5), and one dot product of two adds both elements to the
// plane's sum: two instructions per plane and pair where widening, converting the flag and a
// multiply-add take four.  (The dot product rounds once, to within an ulp of its largest term,
// denormals included; the factor -2 is put back at the end of an item.  Against sums in 64 bits the
// header is as good as with multiply-adds for ReLU, normal, log-normal and Student-t values; where the
// terms of a sum differ by many powers of two the dot product's rounding leans to one side: over 40 powers
// m_q is off by 8e-9 of mean|x| instead of 3e-10, an eighth of the rounding of a level to float32.)
//
// What bounded the encoder was the number of vector instructions (at two wavefronts per SIMD each
// costs 4.3 cycles): 51.4 M values at k = 4: 36.9 -> 32.8 us a call, 18.5 -> 10.2 vector instructions
// per element (SQ_INSTS_VALU); the loop then runs at 7.0 TB/s.
constexpr uint32_t kFlagByte = 0xBFu;
template <int K>
struct ValueTables {
  static constexpr int P = 1 << K;
  float tau[P];
  uint32_t flags[P];
  alignas(16) uint8_t pos4[65536];
};

template <int K>
__device__ __forceinline__ void build_value_tables(const float (&alpha)[K], ValueTables<K>& tb) {
  constexpr int P = 1 << K;
  constexpr int CH = 128;  // values per block of the table; neighbours in bit order are neighbours in value order
  static_assert(kEncBlock * CH == 65536, "one block of the table per thread");
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  if (tid < kWave) {
    float lv_s, tau;
    uint32_t pat_s;
    sort_levels<K>(alpha, lv_s, pat_s, tau);
    uint32_t fl = 0;
#pragma unroll
    for (int bb = 0; bb < K; ++bb) fl |= ((pat_s >> bb) & 1u) * (kFlagByte << (8 * bb));
    if (tid < P) {
      tb.tau[tid] = tau;
      tb.flags[tid] = fl;
    }
  }
  __syncthreads();
  float t[P - 1];
#pragma unroll
  for (int i = 0; i < P - 1; ++i) t[i] = tb.tau[i];
  auto position4 = [&](uint32_t bits) {  // 4 * #{tau_i < value}; 0 for a NaN
    const float v = u32_as_f32(bits << 16);
    uint32_t l = 0;
#pragma unroll
    for (int i = 0; i < P - 1; ++i) l += (v > t[i]) ? 4u : 0u;
    return l;
  };
  // Positions are monotone along a block (one sign; the NaN patterns follow an infinity and give 0):
  // equal ends mean one byte throughout.  Blocks are dealt to threads so that the few with a
  // threshold inside spread over the wavefronts; these are then done by the whole wavefront, two
  // values per lane.  A block's eight 16-byte stores start at a place of the lane's own, so that
  // the lanes do not all write to the same banks.
  const uint32_t b0 = uint32_t((tid * 67) & (kEncBlock - 1)) * CH;
  const uint32_t first = position4(b0), last = position4(b0 + CH - 1);
  const uint32_t w = first * 0x01010101u;
  if (first == last) {
#pragma unroll
    for (int i = 0; i < CH / 16; ++i)
      *reinterpret_cast<uint4*>(&tb.pos4[b0 + 16 * ((i + lane) & (CH / 16 - 1))]) = make_uint4(w, w, w, w);
  }
  uint64_t pending = __ballot(first != last);
  while (pending != 0) {  // the same in every lane
    const int src = __ffsll((unsigned long long)pending) - 1;
    pending &= pending - 1;
    const uint32_t c0 = uint32_t(__builtin_amdgcn_readlane(int(b0), src)) + 2u * uint32_t(lane);
    *reinterpret_cast<uint16_t*>(&tb.pos4[c0]) = uint16_t(position4(c0) | (position4(c0 + 1) << 8));
  }
  __syncthreads();
}

// M2 by comparing with every threshold, in registers: for few levels, and no table to build before the first value can be looked up.
// Every wavefront sorts the levels itself.
template <int K>
struct DirectTables {
  static constexpr int P = 1 << K;
  float tau[P - 1];
  uint32_t spread[P];
};
template <int K>
__device__ __forceinline__ void build_direct_tables(const float (&alpha)[K], DirectTables<K>& tb) {
  constexpr int P = 1 << K;
  float lv_s, tau;
  uint32_t pat_s, sp = 0;
  sort_levels<K>(alpha, lv_s, pat_s, tau);
#pragma unroll
  for (int bb = 0; bb < K; ++bb) sp |= ((pat_s >> bb) & 1u) << (8 * bb);
#pragma unroll
  for (int i = 0; i < P; ++i) {
    if (i < P - 1) tb.tau[i] = u32_as_f32(uint32_t(__builtin_amdgcn_readlane(int(f32_as_u32(tau)), i)));
    tb.spread[i] = uint32_t(__builtin_amdgcn_readlane(int(sp), i));
  }
}

// Sum of NS per-thread float64 values over the threads of a workgroup, in a fixed order (so the
// result does not depend on timing): every wavefront adds its 64 lanes with register-to-register
// lane exchanges, lane 0 parks the NS wave totals in local memory, and thread s < NS adds the
// wavefronts' totals of statistic s in wavefront order.  On return thread s < NS holds total s
// (other threads: unspecified).  Ends with the buffer free for reuse after one more barrier.
struct WaveTotals {
  double v[kMaxWaves][48];  // nstat_of(8) = 45 statistics at most
};
template <int NS>
__device__ __forceinline__ double block_sum_stats(const double (&sv)[NS], WaveTotals& buf) {
  static_assert(NS <= 48, "statistics per record");
  const int tid = threadIdx.x;
  const int wave = tid / kWave, lane = tid & (kWave - 1);
  const int nwaves = (blockDim.x + kWave - 1) / kWave;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const double t = wave_sum(sv[s]);
    if (lane == 0) buf.v[wave][s] = t;
  }
  __syncthreads();
  double mine = 0.0;
  if (tid < NS) {
    mine = buf.v[0][tid];
    for (int w = 1; w < nwaves; ++w) mine += buf.v[w][tid];
  }
  return mine;
}

// Statistics carried by one thread.
template <int K>
struct EncodeStats {
  static constexpr int NPAIR = K * (K - 1) / 2;
  double H[K];      // sum of x over the +1 entries of plane p
  double Sx;        // 1^T x
  uint32_t cnt[K];  // +1 signs per plane
  uint32_t dis[NPAIR > 0 ? NPAIR : 1];  // elements whose planes p<q disagree
};

// M2 for one element, any K: sorted-level position via the bucket table, then the level's spread
// sign pattern.  Adds x to the running float32 sums: S_x always, A_p where plane p is +1
// (byte p of the spread word is 0 or 1; converting it to float and using a fused
// multiply-add gives x*1 or x*0 exactly, so each step rounds like a plain add).
template <int K>
__device__ __forceinline__ void accumulate_elem(float x, const uint32_t (&sp)[(K + 3) / 4], float (&a32)[K],
                                                float& sx32) {
  sx32 = __fadd_rn(sx32, x);
#pragma unroll
  for (int p = 0; p < K; ++p) a32[p] = __fmaf_rn(x, float((sp[p / 4] >> (8 * (p % 4))) & 0xFFu), a32[p]);
}

template <int K>
__device__ __forceinline__ void encode_elem(const EncodeTables<K>& tb, float x, int maxcnt,
                                            uint32_t (&sp)[(K + 3) / 4], float (&a32)[K], float& sx32) {
  using TB = EncodeTables<K>;
  const int lo = tb.lut[f32_as_u32(x) >> (32 - kLutBits)] >> TB::LUT_SHIFT;
  // #{c < maxcnt : x > tau[lo + c]}: the thresholds are sorted, so the true compares form a
  // prefix of tau[lo ..]; its length (at most maxcnt) is found by a branch-free binary search
  // over a window of 2*top - 1 >= maxcnt entries, top = the largest power of two <= maxcnt.
  // lo <= P-1 and the window is shorter than 2P: every read stays inside tau[3P).
  int cnt = 0;
#pragma nounroll
  for (int step = 1 << (31 - __clz(maxcnt)); step >= 1; step >>= 1)
    cnt += (x > tb.tau[lo + cnt + step - 1]) ? step : 0;
  const int idx = lo + cnt;
#pragma unroll
  for (int w = 0; w < TB::NW; ++w) sp[w] = tb.spread[idx * TB::NW + w];
  accumulate_elem<K>(x, sp, a32, sx32);
}

// M2 for NE elements.  MC = 1 or 2: no bucket holds more than MC thresholds (K <= 4 then takes
// everything an element needs from the pair table: the level is lo .. lo+MC); MC = 0: any
// number, maxcnt.  The pair-table form is written in three passes over the elements (bucket
// reads, row reads, selects and sums), so that the local-memory latencies of the NE elements
// overlap whatever order the instruction scheduler keeps.
template <int K, int MC, int NE>
__device__ __forceinline__ void encode_group(const EncodeTables<K>& tb, const float (&xs)[NE], int maxcnt,
                                             uint32_t (&sp)[NE][(K + 3) / 4], float (&a32)[K], float& sx32) {
  if constexpr (K <= 4 && (MC == 1 || MC == 2)) {
    const char* pair = reinterpret_cast<const char*>(tb.pair);
    uint32_t off[NE];  // lo * 8
#pragma unroll
    for (int e = 0; e < NE; ++e) off[e] = tb.lut[f32_as_u32(xs[e]) >> (32 - kLutBits)];
    uint2 t0[NE], t1[NE];  // {tau[lo], spread[lo]}, {tau[lo+1], spread[lo+1]}
    uint32_t top[NE];      // spread[lo+MC]
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const char* row = pair + off[e];
      t0[e] = *reinterpret_cast<const uint2*>(row);
      if constexpr (MC == 2) t1[e] = *reinterpret_cast<const uint2*>(row + 8);
      top[e] = *reinterpret_cast<const uint32_t*>(row + 8 * MC + 4);
    }
#pragma unroll
    for (int e = 0; e < NE; ++e) {
      const float x = xs[e];
      if constexpr (MC == 1) {
        sp[e][0] = (x > u32_as_f32(t0[e].x)) ? top[e] : t0[e].y;
      } else {  // tau[lo] <= tau[lo+1]
        const uint32_t s01 = (x > u32_as_f32(t0[e].x)) ? t1[e].y : t0[e].y;
        sp[e][0] = (x > u32_as_f32(t1[e].x)) ? top[e] : s01;
      }
      accumulate_elem<K>(x, sp[e], a32, sx32);
    }
  } else {
#pragma unroll
    for (int e = 0; e < NE; ++e) encode_elem<K>(tb, xs[e], MC == 1 ? 1 : maxcnt, sp[e], a32, sx32);
  }
}

// Bytes of two words: byte i of the result is byte s_i of {hi, lo} (0-3: lo, 4-7: hi).
template <int S0, int S1, int S2, int S3>
__device__ __forceinline__ uint32_t bytes_of(uint32_t hi, uint32_t lo) {
  return __builtin_amdgcn_perm(hi, lo, uint32_t(S0) | uint32_t(S1) << 8 | uint32_t(S2) << 16 | uint32_t(S3) << 24);
}
// The k <= 4 plane bytes of four columns (byte p of a[c]): as they lie in the payload (column after
// column, k bytes each), and plane by plane (byte c of planes[p]).  Written as byte selections: from
// shifts and masks the compiler makes two to three times as many instructions, and an item has
// only 32 or 64 elements to share them.
template <int K>
__device__ __forceinline__ void columns_to_payload(const uint32_t* a, uint32_t* out) {
  if constexpr (K == 1) {
    out[0] = bytes_of<0, 1, 4, 5>(bytes_of<0, 4, 0, 0>(a[3], a[2]), bytes_of<0, 4, 0, 0>(a[1], a[0]));
  } else if constexpr (K == 2) {
    out[0] = bytes_of<0, 1, 4, 5>(a[1], a[0]);
    out[1] = bytes_of<0, 1, 4, 5>(a[3], a[2]);
  } else if constexpr (K == 3) {
    out[0] = bytes_of<0, 1, 2, 4>(a[1], a[0]);
    out[1] = bytes_of<1, 2, 4, 5>(a[2], a[1]);
    out[2] = bytes_of<2, 4, 5, 6>(a[3], a[2]);
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c) out[c] = a[c];
  }
}
template <int K>
__device__ __forceinline__ void columns_to_planes(const uint32_t* a, uint32_t (&planes)[K]) {
  const uint32_t lo01 = bytes_of<0, 4, 1, 5>(a[1], a[0]), lo23 = bytes_of<0, 4, 1, 5>(a[3], a[2]);
  planes[0] = bytes_of<0, 1, 4, 5>(lo23, lo01);
  if constexpr (K > 1) planes[1] = bytes_of<2, 3, 6, 7>(lo23, lo01);
  if constexpr (K > 2) {
    const uint32_t hi01 = bytes_of<2, 6, 3, 7>(a[1], a[0]), hi23 = bytes_of<2, 6, 3, 7>(a[3], a[2]);
    planes[2] = bytes_of<0, 1, 4, 5>(hi23, hi01);
    if constexpr (K > 3) planes[3] = bytes_of<2, 3, 6, 7>(hi23, hi01);
  }
}

// The planes of a wavefront's items (float32, k <= 4: at most four dwords a lane, one lane's behind the other's), written
// through the cache.  The first lane's item is the first in memory.  64 x 802816, k = 4, streaming / written through:
// 46.9 / 46.2 us a call, 87.3 / 81.0 with the decoder behind it.  (bfloat16's eight dwords, two stores that
// leave gaps: 33.1 / 38.2 us; plain stores 33.6 and with the decoder 59.0 / 54.2: streaming ones are kept.)
// Of smaller tensors the reader gains as well, but the call itself loses up to 1 % (k = 2, streaming / written through, us):
// 64 x 200704 16.9 / 17.1 and with the decoder behind it 28.6 / 27.6, 300032 21.1 / 21.3, 38.3 / 36.3, 400384 25.4 / 25.6, 46.2 /
// 44.5, 458752 27.1 / 27.5, 49.7 / 47.7; from the line on it loses nothing: 524288 29.9 / 29.7, 55.5 / 52.6, 600064 33.8 / 33.6, 62.9 /
// 60.0 (k = 4 33.4 / 33.4, 60.8 / 56.8).
constexpr double kThroughValues = 1 << 25;
template <int NDW, int N>
__device__ __forceinline__ void store_planes(uint8_t* dst, const uint32_t (&out)[N]) {
  const uint64_t at = uint64_t(reinterpret_cast<uintptr_t>(dst));
  const uint64_t first = (uint64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(at >> 32))))) << 32) |
                         uint32_t(__builtin_amdgcn_readfirstlane(int(uint32_t(at))));
  uint32_t v[NDW];
#pragma unroll
  for (int i = 0; i < NDW; ++i) v[i] = out[i];
  store_through<NDW>(payload_buffer(reinterpret_cast<void*>(first), kWave * NDW * 4), uint32_t(at - first), v);
}

// End of an item: bit counts from the finished plane bytes, payload store, float32 partial
// sums (at most 8*VEC terms) folded into the thread's float64 sums.  A lane whose item lies
// beyond its row group (the ragged end of the last wave-item of a group) carries a copy of the
// group's last item: it stores the same bytes to the same place and counts nothing.
template <int K, int VEC, bool RAGGED = false>
__device__ __forceinline__ void finish_item(const uint32_t (&acc)[VEC][(K + 3) / 4], float (&h32)[K], float sx32,
                                            uint8_t* __restrict__ dst, bool counts, EncodeStats<K>& st,
                                            bool through = false) {
  constexpr int NDW = (VEC * K + 3) / 4;
  constexpr int CW = (VEC + 3) / 4;
  constexpr bool SELECT = VEC > 1 && K <= 4;  // by byte selections, four columns at a time
  uint32_t pw[K][CW];  // plane bytes of all VEC columns, plane-major
  // payload: byte ((g*m + j)*K + p); the item's VEC*K bytes are contiguous
  if constexpr (SELECT) {
    uint32_t out[NDW];
#pragma unroll
    for (int w = 0; w < CW; ++w) {
      const uint32_t a[4] = {acc[4 * w][0], acc[4 * w + 1][0], acc[4 * w + 2][0], acc[4 * w + 3][0]};
      columns_to_payload<K>(a, &out[K * w]);
      uint32_t planes[K];
      columns_to_planes<K>(a, planes);
#pragma unroll
      for (int p = 0; p < K; ++p) pw[p][w] = planes[p];
    }
    if constexpr (RAGGED) __builtin_memcpy(dst, out, sizeof(out));
    else if (NDW <= 4 && through) store_planes<(NDW <= 4 ? NDW : 1)>(dst, out);
    else store_dwords_stream<NDW>(reinterpret_cast<uint32_t*>(dst), out);
  } else {
    if constexpr (VEC > 1) {
      uint32_t out[NDW];
#pragma unroll
      for (int w = 0; w < NDW; ++w) out[w] = 0;
#pragma unroll
      for (int c = 0; c < VEC; ++c)
#pragma unroll
        for (int p = 0; p < K; ++p) {
          const int b = c * K + p;
          out[b / 4] |= ((acc[c][p / 4] >> (8 * (p % 4))) & 0xFFu) << (8 * (b % 4));
        }
      if constexpr (RAGGED) __builtin_memcpy(dst, out, sizeof(out));
      else store_dwords_stream<NDW>(reinterpret_cast<uint32_t*>(dst), out);
    } else {
#pragma unroll
      for (int p = 0; p < K; ++p) dst[p] = uint8_t(acc[0][p / 4] >> (8 * (p % 4)));
    }
#pragma unroll
    for (int p = 0; p < K; ++p) {
#pragma unroll
      for (int w = 0; w < CW; ++w) pw[p][w] = 0;
#pragma unroll
      for (int c = 0; c < VEC; ++c) pw[p][c / 4] |= ((acc[c][p / 4] >> (8 * (p % 4))) & 0xFFu) << (8 * (c % 4));
    }
  }
  if (__ballot(!counts) != 0) {  // a scalar branch, taken at the ragged end of a row group only
    const uint32_t keep = counts ? 0xFFFFFFFFu : 0u;
#pragma unroll
    for (int p = 0; p < K; ++p) {
      h32[p] = counts ? h32[p] : 0.0f;
#pragma unroll
      for (int w = 0; w < CW; ++w) pw[p][w] &= keep;
    }
    sx32 = counts ? sx32 : 0.0f;
  }
  {
    int pi = 0;
#pragma unroll
    for (int p = 0; p < K; ++p) {
#pragma unroll
      for (int w = 0; w < CW; ++w) st.cnt[p] += __popc(pw[p][w]);
#pragma unroll
      for (int q = p + 1; q < K; ++q) {
#pragma unroll
        for (int w = 0; w < CW; ++w) st.dis[pi] += __popc(pw[p][w] ^ pw[q][w]);
        ++pi;
      }
    }
  }
  st.Sx += double(sx32);
#pragma unroll
  for (int p = 0; p < K; ++p) st.H[p] += double(h32[p]);
}

// One row's share of an item as it comes from memory: VEC elements in a 16-byte vector, or a
// single element's bits.  Rows are kept in this form while they wait and widened to float32
// only when they are used, so that a load's result is not needed before then.
template <int VEC>
struct RawRow {
  uint4 v;
};
template <>
struct RawRow<1> {
  uint32_t v;
};
template <typename T, int VEC, bool RAGGED = false>
__device__ __forceinline__ RawRow<VEC> load_raw(const T* p) {
  RawRow<VEC> r;
  if constexpr (VEC > 1 && RAGGED) {
    r.v = load16_stream_any(p);
  } else if constexpr (VEC > 1) {
    r.v = load16_stream(p);  // every element of x is read once
  } else if constexpr (sizeof(T) == 4) {
    r.v = f32_as_u32(*reinterpret_cast<const float*>(p));
  } else {
    r.v = uint32_t(*reinterpret_cast<const uint16_t*>(p)) << 16;
  }
  return r;
}
template <int VEC>
__device__ __forceinline__ void widen_raw(const RawRow<VEC>& r, float (&f)[VEC]) {
  if constexpr (VEC > 1) {
    widen(r.v, f);
  } else {
    f[0] = u32_as_f32(r.v);
  }
}

// M2 and the sums, and M3, for rows r0 .. r0+GR-1 of an item: row r of the group lands at bit 7-r of
// each plane byte.  MC: see encode_group.
template <int K, int VEC, int MC, int GR>
__device__ __forceinline__ void encode_rows(const EncodeTables<K>& tb, const RawRow<VEC> (&rows)[8], int r0, int nrows,
                                            int maxcnt, uint32_t (&acc)[VEC][(K + 3) / 4], float (&a32)[K],
                                            float& sx32) {
  constexpr int NW = (K + 3) / 4;
  float xs[GR * VEC];
#pragma unroll
  for (int rr = 0; rr < GR; ++rr) {
    float row[VEC];
    widen_raw<VEC>(rows[r0 + rr], row);
#pragma unroll
    for (int c = 0; c < VEC; ++c) xs[rr * VEC + c] = row[c];
  }
  uint32_t sp[GR * VEC][NW];
  encode_group<K, MC, GR * VEC>(tb, xs, maxcnt, sp, a32, sx32);
#pragma unroll
  for (int rr = 0; rr < GR; ++rr)
#pragma unroll
    for (int c = 0; c < VEC; ++c)
#pragma unroll
      for (int w = 0; w < NW; ++w) acc[c][w] = (acc[c][w] << 1) | (r0 + rr < nrows ? sp[rr * VEC + c][w] : 0u);
}
// The same by value.  Two neighbouring elements (of a row, or of two rows if rows are single
// elements) make a pair.  The bits of a flag byte serve as the plane bit of any row but one: bit 6 of
// 0xBF is zero.
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c, false);
}
template <int K, int VEC, int MC, int GR>
__device__ __forceinline__ void encode_rows(const ValueTables<K>& tb, const RawRow<VEC> (&rows)[8], int r0, int nrows,
                                            int, uint32_t (&acc)[VEC][1], float (&a32)[K], float& sx32) {
  constexpr int NE = GR * VEC;
  static_assert(NE % 2 == 0, "pairs");
  uint32_t w[NE / 2];
#pragma unroll
  for (int rr = 0; rr < GR; ++rr) {
    if constexpr (VEC > 1) {
      const uint4 v = rows[r0 + rr].v;
      w[rr * 4] = v.x; w[rr * 4 + 1] = v.y; w[rr * 4 + 2] = v.z; w[rr * 4 + 3] = v.w;
    } else {
      if (rr % 2 == 0) w[rr / 2] = rows[r0 + rr].v >> 16; else w[rr / 2] |= rows[r0 + rr].v;
    }
  }
  uint32_t off[NE], fl[NE];
#pragma unroll
  for (int i = 0; i < NE / 2; ++i) {
    off[2 * i] = tb.pos4[w[i] & 0xFFFFu];
    off[2 * i + 1] = tb.pos4[w[i] >> 16];
  }
#pragma unroll
  for (int e = 0; e < NE; ++e) fl[e] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(tb.flags) + off[e]);
#pragma unroll
  for (int i = 0; i < NE / 2; ++i) {
    sx32 = dot2_bf16(w[i], 0x3F803F80u, sx32);  // a missing row reads as +0: it adds nothing to the sums
#pragma unroll
    for (int p = 0; p < K; ++p)
      a32[p] = dot2_bf16(w[i], __builtin_amdgcn_perm(fl[2 * i + 1], fl[2 * i], 0x040C000Cu + 0x01000100u * uint32_t(p)), a32[p]);
  }
#pragma unroll
  for (int rr = 0; rr < GR; ++rr)
#pragma unroll
    for (int c = 0; c < VEC; ++c) {
      const int bit = 7 - (r0 + rr);
      const uint32_t f = bit == 6 ? fl[rr * VEC + c] >> 1 : fl[rr * VEC + c];
      acc[c][0] |= (r0 + rr < nrows ? f : 0u) & (0x01010101u << bit);
    }
}
// The same by comparisons.
template <int K, int VEC, int MC, int GR>
__device__ __forceinline__ void encode_rows(const DirectTables<K>& tb, const RawRow<VEC> (&rows)[8], int r0, int nrows, int,
                                            uint32_t (&acc)[VEC][1], float (&a32)[K], float& sx32) {
#pragma unroll
  for (int rr = 0; rr < GR; ++rr) {
    float row[VEC];
    widen_raw<VEC>(rows[r0 + rr], row);
#pragma unroll
    for (int c = 0; c < VEC; ++c) {
      uint32_t sp[1] = {tb.spread[0]};
#pragma unroll
      for (int i = 0; i < DirectTables<K>::P - 1; ++i) sp[0] = row[c] > tb.tau[i] ? tb.spread[i + 1] : sp[0];
      accumulate_elem<K>(row[c], sp, a32, sx32);
      acc[c][0] = (acc[c][0] << 1) | (r0 + rr < nrows ? sp[0] : 0u);
    }
  }
}
// What the float32 sums of encode_rows have to be multiplied by.
template <int K>
__device__ __forceinline__ constexpr float sum_factor(const EncodeTables<K>&) { return 1.0f; }
template <int K>
__device__ __forceinline__ constexpr float sum_factor(const DirectTables<K>&) { return 1.0f; }
template <int K>
__device__ __forceinline__ constexpr float sum_factor(const ValueTables<K>&) { return -2.0f; }

// Plain (not pipelined) item of one column: any number of valid rows.
template <typename T, int K, typename Tables>
__device__ __forceinline__ void encode_column(const Tables& tb, const T* __restrict__ x,
                                              uint8_t* __restrict__ payload, int64_t n, int64_t m, int64_t g,
                                              int64_t j, int maxcnt, EncodeStats<K>& st) {
  constexpr int NW = (K + 3) / 4;
  const int64_t row0 = g * 8;
  const int nrows = (n - row0) < 8 ? int(n - row0) : 8;
  const T* xc = x + row0 * m + j;
  RawRow<1> rows[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) {  // all row loads first, so that they overlap
    rows[r].v = 0u;
    if (r < nrows) rows[r] = load_raw<T, 1>(xc + r * m);  // a missing row reads as +0: it adds nothing to the sums
  }
  float h32[K];
  float sx32 = 0.0f;
#pragma unroll
  for (int p = 0; p < K; ++p) h32[p] = 0.0f;
  uint32_t acc[1][NW];
#pragma unroll
  for (int w = 0; w < NW; ++w) acc[0][w] = 0;
  encode_rows<K, 1, 0, 8>(tb, rows, 0, nrows, maxcnt, acc, h32, sx32);  // missing rows give 0 bits
#pragma unroll
  for (int p = 0; p < K; ++p) h32[p] *= sum_factor(tb);
  finish_item<K, 1>(acc, h32, sx32, payload + ((g * m + j) * K), true, st);
}

// ---- the pipelined stream over complete row groups -------------------------------------------
// Unit of work = wave-item: 64 adjacent items (one per lane) of one row group, i.e. 8 rows x
// 64*VEC columns, every row a contiguous run in memory.  Wavefronts draw wave-items one at a
// time: a wavefront that is served faster (the instruction arbiter favours the oldest wavefront
// of a SIMD, some dies sit closer to the memory they happen to read) simply takes more of them,
// and the whole grid finishes together instead of waiting for its slowest compute unit.  The
// counters live in device memory, one per group of eight workgroups (one counter for the whole
// grid would see a request every nanosecond; an atomic on one address takes about twelve).
// Which wavefront ran which wave-item decides only the grouping of the float64 partial sums,
// never a payload bit.
//
// Queue position c of group i is wave-item (c / slots) * sweep + slots * i + c % slots, sweep = slots *
// groups: at any time the grid reads one contiguous stretch of each of eight rows (the pattern
// memory likes best), the groups advancing through the tensor side by side.  slots = 4: the groups' shares then differ by
// four wave-items at most.  (With 64, as many as a group has wavefronts, they differed by 64, a wave-item a
// wavefront, for which half of the chip waited at the end.  Whole call, 64 / 16 / 4 / 1 slots, us: 64 x 802816 float32, k = 4 43.5 /
// 42.7 / 42.7 / 43.2, bfloat16 30.8 / 29.4 / 29.3 / 29.3; 32 x 401408 float32, k = 3 16.5 / 15.5 / 15.4 / 15.4.)  A grid smaller
// than the chip has a wavefront for every wave-item, and its last group may be smaller than the others: there a
// sweep is all there is, and a group's share is its number of wavefronts (128 x 12544 float32, 98 workgroups, 64 / 4 slots
// 8.3 / 11.9).  So too for wave-items of one and an eighth to one and seven eighths times the wavefronts: nobody has more than two
// then, however they are shared out, and rows of any alignment pay for neighbours on other compute units (64 / 4 slots, six
// placements of the buffers each: 8000 x 1457 bfloat16, k = 2 12.5 / 13.6, k = 4 15.1 / 18.2, 3464 x 1457 float32, k = 4 14.4 / 16.8, 600 x
// 20001 bfloat16, k = 3 12.7 / 13.1, 15 x 390403 float32 11.2 / 11.7; aligned rows 40 x 400000 bfloat16, k = 4 13.7 / 13.8; but single columns,
// whose wave-items are short, 16 x 100003 float32, k = 1 6.3 / 6.0, 800 x 2051 6.4 / 6.1).
struct WorkQueue {
  uint32_t* counter;  // the group's counter: zero when the kernel starts, put back by the finalize kernel or the last workgroup
  uint32_t shift;     // slots = 1 << shift
  uint32_t first;     // slots * group
  uint32_t sweep;     // wave-items all groups take per sweep
  uint32_t count;     // queue positions 0 .. count-1 exist
  bool through;       // planes are written through the cache (see store_planes)
  uint32_t drawn;     // positions handed out without the counter: two per wavefront of the group
};
__device__ __forceinline__ uint32_t queue_to_wave_item(uint32_t c, const WorkQueue& q) {
  return (c >> q.shift) * q.sweep + q.first + (c & ((1u << q.shift) - 1u));
}

// Where a lane's item of a wave-item lives: the row group (the same in all lanes and kept in
// scalar registers, so that a row load is "scalar base + 32-bit lane offset" and costs no vector
// registers for its address) and the lane's own item number inside the group.
struct ItemAddr {
  uint32_t g;    // row group (scalar)
  uint32_t jv;   // item inside the group, clamped to the last one
  bool counts;   // false for the clamped copies that fill the ragged end of a row group
};
// Item of lane `lane` in wave-item w; wpg wave-items and ipg items per row group (both below
// 2^32, checked on the host, as are the byte lengths of a row of x and of a row group's planes).
__device__ __forceinline__ ItemAddr item_addr(uint32_t w, uint32_t wpg, uint32_t ipg, int lane) {
  ItemAddr a;
  a.g = uint32_t(__builtin_amdgcn_readfirstlane(int(w / wpg)));
  a.jv = (w - a.g * wpg) * uint32_t(kWave) + uint32_t(lane);
  a.counts = a.jv < ipg;
  if (!a.counts) a.jv = ipg - 1u;
  return a;
}
// Row 8g + r of the item: the base is formed from scalars only; lane_x = jv * VEC * sizeof(T).
template <typename T, int VEC, bool RAGGED>
__device__ __forceinline__ RawRow<VEC> load_row(const T* __restrict__ x, uint32_t g, uint64_t row_bytes, int r,
                                                uint32_t lane_x) {
  const char* base = reinterpret_cast<const char*>(x) + (uint64_t(g) * 8u + uint64_t(r)) * row_bytes;
  return load_raw<T, VEC, RAGGED>(reinterpret_cast<const T*>(base + lane_x));
}

// The partial row group (n % 8 != 0), behind the complete ones in the queue.
struct PartialGroup {
  uint32_t g;  // its number: that of the complete groups
  int rows;    // how many it has
  __device__ __forceinline__ int last_row(uint32_t group) const { return group == g ? rows - 1 : 7; }
};
// GR rows that are not there: their bits are 0.
template <int K, int VEC, int GR>
__device__ __forceinline__ void skip_rows(const EncodeTables<K>&, uint32_t (&acc)[VEC][(K + 3) / 4]) {
#pragma unroll
  for (int c = 0; c < VEC; ++c)
#pragma unroll
    for (int w = 0; w < (K + 3) / 4; ++w) acc[c][w] <<= GR;
}
template <int K, int VEC, int GR>
__device__ __forceinline__ void skip_rows(const DirectTables<K>&, uint32_t (&acc)[VEC][1]) {
#pragma unroll
  for (int c = 0; c < VEC; ++c) acc[c][0] <<= GR;
}
template <int K, int VEC, int GR>
__device__ __forceinline__ void skip_rows(const ValueTables<K>&, uint32_t (&)[VEC][1]) {}
// Rows r0 .. r0+GR-1 of an item of the partial group, of which the first `nrows` are there.
template <int K, int VEC, int MC, int GR, typename Tables>
__device__ __forceinline__ void encode_partial_rows(const Tables& tb, RawRow<VEC> (&rows)[8], int r0, int nrows, int maxcnt,
                                                    uint32_t (&acc)[VEC][(K + 3) / 4], float (&h32)[K], float& sx32) {
  if (r0 < nrows) {  // the same in all lanes
    if constexpr (GR > 1) {
#pragma unroll
      for (int r = r0; r < r0 + GR; ++r)
        if (r >= nrows) rows[r].v = 0u;
    }
    encode_rows<K, VEC, MC, GR>(tb, rows, r0, nrows, maxcnt, acc, h32, sx32);
  } else {
    skip_rows<K, VEC, GR>(tb, acc);
  }
}

// MIXED: behind the complete row groups there is a partial one; its wave-items are the last of the queue.  Rows beyond the
// last give 0 bits and add nothing: they are not worked through, and the last row is read in their place, so that
// the loads are unconditional.  (The partial group used to go in front of the stream or behind it, a wave-item at a time and with
// nothing in flight meanwhile, on workgroups that had their share of the others as well.  Whole call, beside / in the queue, us:
// 15 x 390403, k = 3, float32 15.1 / 13.1, bfloat16 15.0 / 12.0; 23 x 173913 13.9 / 10.8, k = 4 15.8 / 12.8; 15 x 20000, k = 2
// 9.1 / 7.7; 125 x 400000, k = 4 43.6 / 42.3, 29.4 / 29.2; 101 x 500000 bfloat16, k = 4 was 1 % slower by it, which shares of
// four wave-items (see WorkQueue) took back: 30.1 before both, 29.6 with both.)
template <typename T, int K, int VEC, bool RAGGED, int MC, bool MIXED, typename Tables>
__device__ __forceinline__ void encode_stream(const Tables& tb, const T* __restrict__ x,
                                              uint8_t* __restrict__ payload, uint64_t m, uint32_t ipg, uint32_t wpg,
                                              const WorkQueue& q, const PartialGroup& part, uint32_t cur, uint32_t nxt,
                                              ItemAddr ca, RawRow<VEC> (&fr)[8], EncodeStats<K>& st) {
  constexpr int NW = (K + 3) / 4;
  constexpr int GR = VEC >= 4 ? 1 : 4 / VEC;  // rows whose table lookups are issued together (at least 4 elements)
  const int lane = threadIdx.x & (kWave - 1);
  const uint64_t row_bytes = m * sizeof(T);
  // The first item's rows have had the whole table build to arrive.  Waiting for them here
  // (vmcnt 0, the other counters untouched) gives the loop an empty set of outstanding loads
  // on entry whatever code precedes it, so that the waits the compiler places inside the loop
  // are the ones its own steady state needs and no more.
  __builtin_amdgcn_s_waitcnt(0x0F70);
  auto items = [&](auto partial) {
    while (cur < q.count && (!MIXED || decltype(partial)::value || ca.g != part.g)) {
      // the wave-item after the next: asked for now, looked at when this item is done (the answer
      // comes back in line with the row loads issued below, well before it is needed)
      uint32_t after_v = 0;
      if (lane == 0) after_v = __hip_atomic_fetch_add(q.counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      // When there is no next wave-item every lane re-reads the first item of the tensor (valid,
      // one cache line per row for the whole wavefront), so that the loads stay unconditional and
      // the compiler can reuse the row registers in place.
      ItemAddr na;
      na.g = 0; na.jv = 0; na.counts = false;
      if (nxt < q.count) na = item_addr(queue_to_wave_item(nxt, q), wpg, ipg, lane);
      const char* na_row = reinterpret_cast<const char*>(x) + uint64_t(na.g) * 8u * row_bytes;
      const int na_last = MIXED ? part.last_row(na.g) : 7;
      uint32_t acc[VEC][NW];
      float h32[K];
      float sx32 = 0.0f;
#pragma unroll
      for (int p = 0; p < K; ++p) h32[p] = 0.0f;
#pragma unroll
      for (int c = 0; c < VEC; ++c)
#pragma unroll
        for (int w = 0; w < NW; ++w) acc[c][w] = 0;
#pragma unroll
      for (int r0 = 0; r0 < 8; r0 += GR) {
        if constexpr (decltype(partial)::value) encode_partial_rows<K, VEC, MC, GR>(tb, fr, r0, part.rows, MC, acc, h32, sx32);
        else encode_rows<K, VEC, MC, GR>(tb, fr, r0, 8, MC, acc, h32, sx32);
        // the sums pass through an empty asm: left alone, the compiler moves the whole chain of adds
        // to the end of the round, and every row's operands stay in registers until there
#pragma unroll
        for (int p = 0; p < K; ++p) asm volatile("" : "+v"(h32[p]));
        asm volatile("" : "+v"(sx32));
        // The loads of the next item's rows go where this group's rows were: they may not be
        // issued before the last use of those registers (else the compiler keeps a second set of
        // row registers and copies it over at the end of the round, which also means waiting for
        // all eight loads there).
        __builtin_amdgcn_sched_barrier(0);
        {
          // the lane offset passes through an empty asm, so that the addresses of this group's loads
          // are formed here and not, all eight of them, at the top of the round (and so that a last row
          // read in another's place stays a load: a branch round it cost a third of the rate)
          uint32_t lane_x = na.jv * uint32_t(VEC * sizeof(T));
#pragma unroll
          for (int r = r0; r < r0 + GR; ++r) {
            asm volatile("" : "+v"(lane_x));
            fr[r] = load_raw<T, VEC, RAGGED>(reinterpret_cast<const T*>(na_row + lane_x));
            if (!MIXED || r < na_last) na_row += row_bytes;
          }
        }
        // keep the instruction scheduler from mixing groups: it would otherwise hoist the table
        // reads of all 8*VEC elements and run out of registers
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int p = 0; p < K; ++p) h32[p] *= sum_factor(tb);
      finish_item<K, VEC, RAGGED>(acc, h32, sx32, payload + uint64_t(ca.g) * m * uint32_t(K) + ca.jv * uint32_t(VEC * K), ca.counts,
                                  st, q.through);
      cur = nxt;
      nxt = q.drawn + uint32_t(__builtin_amdgcn_readfirstlane(int(after_v)));
      ca = na;
    }
  };
  items(std::false_type{});
  if constexpr (MIXED) items(std::true_type{});
}

// A partial row group by itself: all there is of a tensor of fewer than eight rows (x and payload are the group's).  The next wave-item's rows are asked for before the
// current one's are used; its wavefronts otherwise wait for memory and work in turns (us a call,
// before / now: 1 x 12000000, k = 3, float32 56.7 / 39.7, bfloat16 42.8 / 29.7; 4 x 5416312, k = 4 38.3 / 33.3, 30.5 /
// 25.7; 3 x 2208816, k = 2 16.8 / 13.6).
template <typename T, int VEC, bool RAGGED>
__device__ __forceinline__ void load_few(const T* __restrict__ x, int n, int64_t m, const ItemAddr& ia,
                                         RawRow<VEC> (&rows)[8]) {
  const T* xc = x + int64_t(ia.jv) * VEC;
#pragma unroll
  for (int r = 0; r < 8; ++r) rows[r] = load_raw<T, VEC, RAGGED>(xc + (r < n ? r : n - 1) * m);
}
// rows: those of the first wave-item.
template <typename T, int K, int VEC, bool RAGGED, int MC, typename Tables>
__device__ __forceinline__ void encode_few(const Tables& tb, const T* __restrict__ x, uint8_t* __restrict__ payload,
                                           int n, int64_t m, uint32_t ipg, uint32_t wpg, int maxcnt,
                                           uint32_t first, uint32_t step, RawRow<VEC> (&rows)[8], EncodeStats<K>& st) {
  constexpr int NW = (K + 3) / 4;
  constexpr int GR = VEC >= 4 ? 1 : 4 / VEC;
  const int lane = threadIdx.x & (kWave - 1);
  if (first >= wpg) return;
  ItemAddr ia = item_addr(first, wpg, ipg, lane);
  auto work = [&] {
    float h32[K];
    float sx32 = 0.0f;
    uint32_t acc[VEC][NW];
#pragma unroll
    for (int p = 0; p < K; ++p) h32[p] = 0.0f;
#pragma unroll
    for (int c = 0; c < VEC; ++c)
#pragma unroll
      for (int v = 0; v < NW; ++v) acc[c][v] = 0;
#pragma unroll
    for (int r0 = 0; r0 < 8; r0 += GR) {
      encode_partial_rows<K, VEC, MC, GR>(tb, rows, r0, n, maxcnt, acc, h32, sx32);
#pragma unroll
      for (int p = 0; p < K; ++p) asm volatile("" : "+v"(h32[p]));  // as in the stream
      asm volatile("" : "+v"(sx32));
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int p = 0; p < K; ++p) h32[p] *= sum_factor(tb);
    finish_item<K, VEC, RAGGED>(acc, h32, sx32, payload + int64_t(ia.jv) * VEC * K, ia.counts, st);
  };
  if (first + step >= wpg) {  // one wave-item: nothing to ask for
    work();
    return;
  }
  for (uint32_t w = first; w < wpg; w += step) {
    const ItemAddr na = item_addr(w + step < wpg ? w + step : w, wpg, ipg, lane);
    RawRow<VEC> next[8];
    load_few<T, VEC, RAGGED>(x, n, m, na, next);
    work();
    ia = na;
#pragma unroll
    for (int r = 0; r < 8; ++r) rows[r] = next[r];
  }
}

// ========================================================================= finalize (M5)
// From the call's totals: alpha_cur = (B^T B)^-1 B^T x by Gaussian elimination with row
// pivoting, the moving average with beta = min(0.9, (1+t)/(10+t)), m_q = mean(B alpha_t - x);
// header = [alpha_t, m_q].  One thread; K is a template parameter so that the k x k system
// lives in registers.  tot: sums of x over the +1 entries of each plane, sum of x, +1 counts
// per plane, disagreement counts per plane pair.
template <int K>
__device__ __forceinline__ void solve_and_write_header(const double* tot, const float (&alpha_prev)[K], double n_elems,
                                                       double beta, float* __restrict__ header) {
  double G[K][K], b[K], Sb[K], a_prev[K], cur[K];
  const double Sx = tot[K];
  {
    int pi = 0;
#pragma unroll
    for (int p = 0; p < K; ++p) {
      a_prev[p] = double(alpha_prev[p]);
      b[p] = 2.0 * tot[p] - Sx;                 // B^T x = 2 * (sum over +1 entries) - sum(x)
      Sb[p] = 2.0 * tot[K + 1 + p] - n_elems;   // 1^T B
      G[p][p] = n_elems;
#pragma unroll
      for (int q = p + 1; q < K; ++q) {
        G[p][q] = G[q][p] = n_elems - 2.0 * tot[2 * K + 1 + pi];
        ++pi;
      }
    }
  }
  bool singular = false;
  double inv[K];
#pragma unroll
  for (int col = 0; col < K; ++col) {
    // bring the largest |entry| of the column to the diagonal (compare-and-swap keeps the
    // indices static, so the system stays in registers); in the first column it is there, n_elems
#pragma unroll
    for (int r = col + 1; r < K && col > 0; ++r) {
      if (fabs(G[r][col]) > fabs(G[col][col])) {
#pragma unroll
        for (int c = 0; c < K; ++c) { const double tmp = G[col][c]; G[col][c] = G[r][c]; G[r][c] = tmp; }
        const double tb_ = b[col]; b[col] = b[r]; b[r] = tb_;
      }
    }
    if (fabs(G[col][col]) < 1e-9 * n_elems) singular = true;
    inv[col] = 1.0 / G[col][col];  // one division per column; its products differ from quotients by an ulp
    if (!singular) {
#pragma unroll
      for (int r = col + 1; r < K; ++r) {
        const double fct = G[r][col] * inv[col];
#pragma unroll
        for (int c = col; c < K; ++c) G[r][c] -= fct * G[col][c];
        b[r] -= fct * b[col];
      }
    }
  }
#pragma unroll
  for (int r = K - 1; r >= 0; --r) {
    double acc = b[r];
#pragma unroll
    for (int c = r + 1; c < K; ++c) acc -= G[r][c] * cur[c];
    cur[r] = singular ? a_prev[r] : acc * inv[r];
  }
  double dot = 0.0;
#pragma unroll
  for (int p = 0; p < K; ++p) {
    const float a_t = float(beta * a_prev[p] + (1.0 - beta) * (singular ? a_prev[p] : cur[p]));
    header[p] = a_t;
    dot += double(a_t) * Sb[p];
  }
  header[K] = float((dot - Sx) / n_elems);
}

// What the kernels of one compress call share: the per-workgroup records in the workspace
// (stat-major: statistic s of workgroup b at records[s * nrec + b]), the previous coefficients
// and the header to write.
struct MbqCall {
  uint32_t* counters;  // work counters of the encode kernel (control block of the workspace)
  double* records;
  const float* alpha_prev;
  float* header;
  double n_elems;
  double beta;  // weight of the previous coefficients in the moving average: min(0.9, (1+t)/(10+t))
};
constexpr int kDoneCounter = 2;  // word of the counters (between two work counters) that counts off the workgroups

// The sums of N values (a power of two) over the 16 lanes of a row, in a fixed order: in every step a lane gives its partner one half of
// what it has left and takes the other half of the partner's, so that N - 1 additions and exchanges do, instead of 4 N.
// On return a lane has the sum number row_sum_index(lane).
template <int N, int CTRL>
__device__ __forceinline__ void row_sum_step(double* v, bool upper) {
  if constexpr (N > 1) {
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      const double keep = upper ? v[N / 2 + i] : v[i], give = upper ? v[i] : v[N / 2 + i];
      v[i] = keep + dpp_f64<CTRL>(give);
    }
  } else {
    v[0] += dpp_f64<CTRL>(v[0]);
  }
}
constexpr int kDppQuadReverse = 0x1B;  // quad_perm [3,2,1,0]
template <int N>
__device__ __forceinline__ double row_sums(double (&v)[N], int lane) {
  row_sum_step<N, kDppRowMirror>(v, (lane & 8) != 0);
  row_sum_step<(N > 1 ? N / 2 : 1), kDppRowHalfMirror>(v, (lane & 4) != 0);
  row_sum_step<(N > 2 ? N / 4 : 1), kDppQuadReverse>(v, (lane & 2) != 0);
  row_sum_step<(N > 4 ? N / 8 : 1), kDppQuadSwap1>(v, (lane & 1) != 0);
  return v[0];
}
template <int N>
__device__ __forceinline__ int row_sum_index(int lane) {
  return (lane & 15) * N / 16;
}

// Sum number i over the rows of nwaves wavefronts, which lie behind each other.
template <int N>
__device__ __forceinline__ double sum_of_rows(const double* rows, int i, int nwaves) {
  double part[4] = {0.0, 0.0, 0.0, 0.0};
  for (int j = 0; j < nwaves * (kWave / 16); j += 4)
#pragma unroll
    for (int u = 0; u < 4; ++u) part[u] += rows[(j + u) * N + i];
  return (part[0] + part[1]) + (part[2] + part[3]);
}

// End of an encode kernel (M4): the workgroup adds up its threads' statistics in a fixed order
// and stores one record.  (Up to 16 statistics, k <= 4; the wavefronts' sums one statistic after the other took
// 30 instructions each.  Whole call before / now, us: k = 4, 64 x 802816 float32 42.5 / 41.5, bfloat16 29.2 / 28.4, 32 x 401408 16.7 / 15.9,
// 64 x 8192 9.85 / 8.85, 128 x 160 8.6 / 7.4; k = 2, 4 x 65536 5.7 / 5.5.)
// FINISH: past the second-level cache, for a workgroup of another die that reads it in this kernel.
template <int K, bool FINISH = false>
__device__ __forceinline__ void store_record(const EncodeStats<K>& st, const MbqCall& call, WaveTotals& buf) {
  constexpr int NPAIR = K * (K - 1) / 2;
  constexpr int NSTAT = nstat_of(K);
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid & (kWave - 1);
  const int nwaves = (blockDim.x + kWave - 1) / kWave;
  double total = 0.0;
  if constexpr (NSTAT <= 16) {
    constexpr int N = NSTAT <= 4 ? 4 : NSTAT <= 8 ? 8 : 16;
    static_assert(sizeof(buf) >= kMaxWaves * (kWave / 16) / 2 * 16 * sizeof(double), "rows of half of the most wavefronts");
    static_assert(kEncWaves <= kMaxWaves / 2 && kBlock / kWave <= kMaxWaves / 2, "wavefronts of the kernels that store records");
    double v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = 0.0;
#pragma unroll
    for (int p = 0; p < K; ++p) {
      v[p] = st.H[p];
      v[K + 1 + p] = double(st.cnt[p]);
    }
    v[K] = st.Sx;
#pragma unroll
    for (int i = 0; i < NPAIR; ++i) v[2 * K + 1 + i] = double(st.dis[i]);
    double* const rows = &buf.v[0][0];
    rows[(tid / 16) * N + row_sum_index<N>(lane)] = row_sums<N>(v, lane);  // (N < 16: several lanes store the same)
    __syncthreads();
    if (tid < NSTAT) total = sum_of_rows<N>(rows, tid, nwaves);
  } else {
    double* mine = buf.v[wave];
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const double h = wave_sum(st.H[p]);
      const double c = double(wave_sum(st.cnt[p]));
      if (lane == 0) { mine[p] = h; mine[K + 1 + p] = c; }
    }
    const double sx = wave_sum(st.Sx);
    if (lane == 0) mine[K] = sx;
#pragma unroll
    for (int i = 0; i < NPAIR; ++i) {
      const double d = double(wave_sum(st.dis[i]));
      if (lane == 0) mine[2 * K + 1 + i] = d;
    }
    __syncthreads();
    if (tid < NSTAT) {
      total = buf.v[0][tid];
      for (int w = 1; w < nwaves; ++w) total += buf.v[w][tid];
    }
  }
  if (tid < NSTAT) {
    double* const rec = call.records + int64_t(tid) * gridDim.x + blockIdx.x;
    if constexpr (FINISH) __hip_atomic_store(rec, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *rec = total;
  }
}

// M5, one workgroup of 16 wavefronts: wavefront w takes the statistics w, w + 16, ... (their records
// lie together), lane l the records l, l + 64, ..., one wavefront sum per statistic; one thread
// solves and writes the header.  (With four wavefronts that each added up their share of every
// statistic the sums alone took 1.9 of the kernel's 3.7 us at k = 4.)
// k = 7 and 8 get 12 and 8 wavefronts: their solves keep 146 and 182 registers, and with 16 wavefronts the
// compiler has 128 (24 and 154 spilled; k = 8, 128 x 160: the whole call 27.0 -> 26.3 us).
constexpr int kFinalizeBlock = 1024;
constexpr int finalize_block(int k) { return k <= 6 ? kFinalizeBlock : k == 7 ? 768 : 512; }
// Sum of nrec records by one wavefront, four loads in flight; every lane has it.  FRESH: records that
// other workgroups have written in this kernel.
template <bool FRESH = false>
__device__ __forceinline__ double sum_records(const double* rec, int nrec, int lane) {
  auto one = [&](int b) {
    return FRESH ? __hip_atomic_load(rec + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : rec[b];
  };
  double a = 0.0;
  for (int b = lane; b < nrec; b += 4 * kWave) {
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = b + u * kWave < nrec ? one(b + u * kWave) : 0.0;
    a += (v[0] + v[1]) + (v[2] + v[3]);
  }
  return wave_sum(a);
}
template <int K>
__global__ __launch_bounds__(finalize_block(K)) void mbq_finalize_kernel(MbqCall call, int nrec) {
  constexpr int NSTAT = nstat_of(K);
  __shared__ double tot[48];
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid & (kWave - 1);
  float alpha_prev[K];  // asked for together with the records: the solve at the end would otherwise wait for them
#pragma unroll
  for (int p = 0; p < K; ++p) alpha_prev[p] = call.alpha_prev[p];
  for (int s = wave; s < NSTAT; s += finalize_block(K) / kWave) {
    const double a = sum_records(call.records + int64_t(s) * nrec, nrec, lane);
    if (lane == 0) tot[s] = a;
  }
  if (tid < kMaxGroups) call.counters[tid * kCounterStride] = 0u;  // the encode kernel's work counters, for the next call
  __syncthreads();
  if (tid == 0) solve_and_write_header<K>(tot, alpha_prev, call.n_elems, call.beta, call.header);
}

// The same at the end of an encode kernel of few workgroups: each counts itself off when its record is written, and
// the last one adds them up, in the finalize kernel's order, and solves.  No one waits for another.
// A launch less is about 3 us of host time; on the device, encode and finalize kernels / this (us, replayed graphs, float32,
// k = 2; 4): 16 x 2048 7.1 / 6.8; 9.9 / 10.0; 64 x 8448 (33 workgroups) 7.3 / 7.1; 10.2 / 10.4; 64 x 16384 (64) 7.5 / 7.4;
// 10.3 / 10.6; beyond the line, where the counter, one address, takes 12 ns each: 64 x 16640 (65) 7.6 / 7.5; 10.3 / 10.7, 64 x
// 20480 (80) 7.6 / 7.7; 10.3 / 10.9, 64 x 32768 (128) 7.9 / 8.3; 10.6 / 11.4, 64 x 50000 (196) 8.8 / 9.7; 11.2 / 12.6.
// The workgroups of a call add 64 to the count together, whatever their number is, and nothing puts it back: so it is
// a multiple of 64 whenever no call is under way, also after calls that overlapped on one workspace, which they must not
// (the last of all to end then finds it so, and clears the work counters behind all of them, whichever call it is of).
constexpr int kFinishGridMax = 64;
__device__ __forceinline__ bool last_workgroup(uint32_t* counters) {
  __shared__ int last;
  // This thread's part of the record is written: it has reached the memory that all dies read, where it was sent by a
  // device-scope store, and the compiler moves no access across.  So the count, which is raised behind the barrier, comes after
  // all of the record, and whoever finds the count full and then loads past its caches (sum_records<true>) finds the
  // records.  (A release and acquire by the count's own instruction also write back and empty the caches: 0.1 to
  // 0.3 us a call, 4 x 65536, k = 2 6.76 / 6.99.)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t share = blockIdx.x == 0 ? uint32_t(kFinishGridMax) + 1u - gridDim.x : 1u;
    const uint32_t before = __hip_atomic_fetch_add(counters + kDoneCounter, share, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = (before + share) % uint32_t(kFinishGridMax) == 0u ? 1 : 0;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(last) != 0;
}
// The work counters, for the next call; by the last workgroup, behind its loads of the records (which in front of them
// wait for these stores: 0.1 us).
__device__ __forceinline__ void clear_work_counters(uint32_t* counters) {
  if (threadIdx.x < uint32_t(kMaxGroups)) counters[threadIdx.x * kCounterStride] = 0u;
}
template <int K>
__device__ __forceinline__ void finish_in_last_workgroup(const MbqCall& call, const float (&alpha_prev)[K], WaveTotals& buf) {
  constexpr int NSTAT = nstat_of(K);
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid & (kWave - 1);
  const int nrec = int(gridDim.x);
  if (!last_workgroup(call.counters)) return;
  double* tot = buf.v[0];
  static_assert(kFinishGridMax <= kWave, "a record per lane");
  constexpr int EACH = (NSTAT + kEncWaves - 1) / kEncWaves;  // statistics of a wavefront, asked for together
  double v[EACH];
#pragma unroll
  for (int i = 0; i < EACH; ++i) {
    const int s = wave + i * kEncWaves;
    v[i] = s < NSTAT && lane < nrec
               ? __hip_atomic_load(call.records + int64_t(s) * nrec + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0.0;
  }
#pragma unroll
  for (int i = 0; i < EACH; ++i) {
    const int s = wave + i * kEncWaves;
    const double a = wave_sum(v[i]);
    if (s < NSTAT && lane == 0) tot[s] = a;
  }
  clear_work_counters(call.counters);
  __syncthreads();
  if (tid == 0) solve_and_write_header<K>(tot, alpha_prev, call.n_elems, call.beta, call.header);
}

// DIRECT: levels are found by comparisons (direct_levels below).
template <int K, bool DIRECT, typename S>
__device__ __forceinline__ decltype(auto) tables_of(S& shared) {
  if constexpr (DIRECT) return DirectTables<K>{};
  else return (shared);
}

// Which rows a tensor has (a kernel for each kind: what the others need costs 0.3 us): complete row groups only, complete ones
// and a partial one, fewer than eight rows.
enum Rows { kRowsComplete, kRowsMixed, kRowsFew };

// Fused M1..M4.  Row groups go through the pipelined stream: row r of the next
// wave-item is requested as soon as row r of the current one has been consumed, so a wavefront
// always has loads in flight while it works; the first wave-item's rows are requested before
// the tables are built.  The partial row group (n % 8 != 0) is the end of the same queue; the rare case of more
// than two thresholds per bucket takes the plain path, one
// column per thread.  RAGGED: m is not a multiple of VEC, so rows start at any alignment; vectors
// all the same, and the last m % VEC columns one per thread (15 x 390403 float32, k = 3: this kernel
// 12.0 us and the decoder 7.2, against 14.3 and 9.0 with single columns throughout).
// NARROW: too narrow for wave-items, so all columns one per thread, whatever the rows (VEC = 1, kRowsComplete).
template <typename T, int K, int VEC, bool RAGGED, bool FINISH, int ROWS, bool DIRECT, bool NARROW>
__global__ __launch_bounds__(kEncBlock) void mbq_encode_kernel(const T* __restrict__ x, uint8_t* __restrict__ payload,
                                                               MbqCall call, int64_t n, int64_t m, uint32_t ipg,
                                                               uint32_t wpg, uint32_t n_wave_items, bool wide,
                                                               uint8_t queue_shift) {
  constexpr int NPAIR = K * (K - 1) / 2;
  constexpr bool BY_VALUE = sizeof(T) == 2 && K <= 4 && !DIRECT;
  constexpr bool FEW = ROWS == kRowsFew, MIXED = ROWS == kRowsMixed;
  using SharedTables = std::conditional_t<DIRECT, char, std::conditional_t<BY_VALUE, ValueTables<K>, EncodeTables<K>>>;
  __shared__ SharedTables shared_tb;
  __shared__ WaveTotals red;
  std::conditional_t<DIRECT, DirectTables<K>, SharedTables&> tb = tables_of<K, DIRECT>(shared_tb);

  if constexpr (NARROW) {
    n_wave_items = 0;
    wide = false;
  }
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  float alpha[K];  // asked for first: nothing below needs them before the tables are built
#pragma unroll
  for (int j = 0; j < K; ++j) alpha[j] = call.alpha_prev[j];
  // this wavefront's place in its group's queue: the first two positions of every wavefront are
  // fixed (its index among the group's wavefronts, and that plus their number), the rest are drawn
  WorkQueue q;
  const uint32_t group = blockIdx.x / uint32_t(kGroupBlocks);
  const uint32_t groups = (gridDim.x + uint32_t(kGroupBlocks) - 1u) / uint32_t(kGroupBlocks);
  const uint32_t group_blocks =
      gridDim.x - group * uint32_t(kGroupBlocks) < uint32_t(kGroupBlocks) ? gridDim.x - group * uint32_t(kGroupBlocks)
                                                                        : uint32_t(kGroupBlocks);
  const uint32_t group_waves = group_blocks * uint32_t(kEncWaves);
  q.counter = call.counters + group * uint32_t(kCounterStride);
  q.shift = queue_shift;
  const uint32_t slots = 1u << q.shift;
  q.first = group << q.shift;
  q.sweep = groups << q.shift;
  {
    const uint32_t full_sweeps = n_wave_items / q.sweep;
    const uint32_t rest = n_wave_items - full_sweeps * q.sweep;
    const uint32_t extra = rest > q.first ? (rest - q.first < slots ? rest - q.first : slots) : 0u;
    q.count = (full_sweeps << q.shift) + extra;
  }
  q.through = sizeof(T) == 4 && call.n_elems >= kThroughValues;
  q.drawn = 2u * group_waves;
  const PartialGroup part{MIXED ? uint32_t(n / 8) : 0xFFFFFFFFu, int(n % 8)};
  const uint32_t cur = uint32_t(__builtin_amdgcn_readfirstlane(
      int((blockIdx.x - group * uint32_t(kGroupBlocks)) * uint32_t(kEncWaves) + uint32_t(tid) / uint32_t(kWave))));
  const uint32_t nxt = cur + group_waves;
  RawRow<VEC> fr[8];
  ItemAddr ca;
  ca.g = 0; ca.jv = 0; ca.counts = false;
  if (cur < q.count) {
    ca = item_addr(queue_to_wave_item(cur, q), wpg, ipg, lane);
    const int last = MIXED ? part.last_row(ca.g) : 7;
#pragma unroll
    for (int r = 0; r < 8; ++r)
      fr[r] = load_row<T, VEC, RAGGED>(x, ca.g, uint64_t(m) * sizeof(T), MIXED && r > last ? last : r, ca.jv * uint32_t(VEC * sizeof(T)));
  }

  const uint32_t wave_id = uint32_t(__builtin_amdgcn_readfirstlane(tid / kWave));
  const uint32_t few_first = wave_id * gridDim.x + blockIdx.x;  // wave-items are dealt to the workgroups first and to their wavefronts second
  if (FEW && wide && few_first < wpg)
    load_few<T, VEC, RAGGED>(x, int(n), m, item_addr(few_first, wpg, ipg, lane), fr);

  int maxcnt = 1;
  if constexpr (DIRECT) {
    build_direct_tables<K>(alpha, tb);
  } else if constexpr (BY_VALUE) {
    build_value_tables<K>(alpha, tb);
  } else {
    build_encode_tables<K>(alpha, tb);
    // the same value in every lane: read it into a scalar register, so that the choice of path
    // below is a scalar branch and not a divergent one whose sides run one after the other
    maxcnt = __builtin_amdgcn_readfirstlane(tb.maxcnt);
  }

  EncodeStats<K> st;
  st.Sx = 0.0;
#pragma unroll
  for (int p = 0; p < K; ++p) { st.H[p] = 0.0; st.cnt[p] = 0; }
#pragma unroll
  for (int i = 0; i < (NPAIR > 0 ? NPAIR : 1); ++i) st.dis[i] = 0;

  const int64_t stride = int64_t(gridDim.x) * kEncBlock;
  const int64_t gtid = int64_t(blockIdx.x) * kEncBlock + tid;
  // columns j0 .. j0 + rem - 1 of row groups 0 .. G - 1, one per thread
  auto single_columns = [&](int64_t G, int64_t j0, int64_t rem) {
    for (int64_t s = gtid; s < G * rem; s += stride) {
      const int64_t g = s / rem;
      encode_column<T, K>(tb, x, payload, n, m, g, j0 + s - g * rem, maxcnt, st);
    }
  };
  if constexpr (FEW) {
    int64_t col0 = 0;  // columns from here on go one per thread: all, where rows are too narrow or levels too close
    if (wide && maxcnt == 1) {
      encode_few<T, K, VEC, RAGGED, 1>(tb, x, payload, int(n), m, ipg, wpg, maxcnt, few_first,
                                       gridDim.x * uint32_t(kEncWaves), fr, st);
      col0 = int64_t(ipg) * VEC;
    }
    if constexpr (DIRECT || BY_VALUE) {  // a few columns, or a narrow tensor
      single_columns(1, col0, m - col0);
    } else if (col0 < m) {  // (in front of what the loop needs: 4 x 2000 float32, k = 4 7.83 / 7.74 us)
      // (Perhaps all, so without the division by which single_columns finds the row group: 1 x 12000000, k = 8, with / without, us:
      // float32 300 / 285, bfloat16 312 / 291; and n / 8 for 0: knowing it, the compiler puts a wait between the rows' loads.)
      for (int64_t j = col0 + gtid; j < m; j += stride) encode_column<T, K>(tb, x, payload, n, m, n / 8, j, maxcnt, st);
    }
  } else {
    const bool stream = n_wave_items != 0u;  // else: a geometry too narrow for wave-items
    auto row_groups = [&] {
      if (stream && maxcnt == 1) {
        encode_stream<T, K, VEC, RAGGED, 1, MIXED>(tb, x, payload, uint64_t(m), ipg, wpg, q, part, cur, nxt, ca, fr, st);
      } else if (stream && maxcnt == 2 && K <= 4 && !BY_VALUE && !DIRECT) {
        if constexpr (!BY_VALUE && !DIRECT)
          encode_stream<T, K, VEC, RAGGED, 2, MIXED>(tb, x, payload, uint64_t(m), ipg, wpg, q, part, cur, nxt, ca, fr, st);
      } else {
        // several thresholds share a bucket (levels closer than a bucket's width), or a very narrow
        // tensor: rare.  One column per thread keeps this path's register needs out of the kernel's
        // budget.
        single_columns((n + 7) / 8, 0, m);
      }
    };
    auto other_parts = [&] {
      // the up to VEC - 1 columns that no vector covers
      if (RAGGED && stream && maxcnt <= (K <= 4 && !BY_VALUE ? 2 : 1))
        single_columns((n + 7) / 8, int64_t(ipg) * VEC, m - int64_t(ipg) * VEC);
      if constexpr (VEC == 1 && !MIXED) {  // a partial row group that is not in the queue (kMixedColumnGroups)
        if (stream && n % 8 != 0) {
          const int64_t g = n / 8;
          if (maxcnt == 1) {
            RawRow<VEC> own[8];
            if (few_first < wpg) load_few<T, VEC, RAGGED>(x + g * 8 * m, int(n % 8), m, item_addr(few_first, wpg, ipg, lane), own);
            encode_few<T, K, VEC, RAGGED, 1>(tb, x + g * 8 * m, payload + g * m * K, int(n % 8), m, ipg, wpg, maxcnt, few_first,
                                             gridDim.x * uint32_t(kEncWaves), own, st);
          } else if (maxcnt == 2 && K <= 4) {
            for (int64_t j = gtid; j < m; j += stride) encode_column<T, K>(tb, x, payload, n, m, g, j, maxcnt, st);
          }
        }
      }
    };
    // What the stream does not cover takes two or three trips to memory one after the other.  Before the
    // stream (whose first rows are under way by then) they cost a few wavefronts items that others draw from
    // the queue; behind it, 2 to 4 us at the end of the kernel.  Whole call, float32, k = 2, behind / before:
    // 13113 x 1309 24.3 / 20.2 us, 3000 x 8193 27.0 / 23.1, 8315 x 1457 22.1 / 19.2.  Not so where values are
    // looked up in a table of their own (bfloat16, k = 4, 8315 x 1457: 18.6 / 20.6).
    if constexpr (BY_VALUE) {
      row_groups();
      other_parts();
    } else {
      other_parts();
      row_groups();
    }
  }
  store_record<K, FINISH>(st, call, red);
  if constexpr (FINISH) finish_in_last_workgroup<K>(call, alpha, red);
}

// ================================================ comparison layout: one byte per binary base
// ACCEPT_LAYOUT_UNENCODED: B itself, +1 / -1 as bytes, element-major with the k bases
// innermost ("w/o enc." in the paper's size table).  Same levels, same sums and the same
// finalize kernel as the bit-plane path; plain flat loops, four elements per thread and step.
template <typename T, int K>
__global__ __launch_bounds__(kBlock) void mbq_encode_plain_kernel(const T* __restrict__ x,
                                                                  uint8_t* __restrict__ payload, MbqCall call,
                                                                  int64_t N) {
  constexpr int NW = (K + 3) / 4;
  constexpr int NPAIR = K * (K - 1) / 2;
  __shared__ EncodeTables<K> tb;
  __shared__ WaveTotals red;
  const float* alpha_prev = call.alpha_prev;
  const int tid = threadIdx.x;
  float alpha[K];
#pragma unroll
  for (int j = 0; j < K; ++j) alpha[j] = alpha_prev[j];
  build_encode_tables<K>(alpha, tb);
  const int maxcnt = __builtin_amdgcn_readfirstlane(tb.maxcnt);
  EncodeStats<K> st;
  st.Sx = 0.0;
#pragma unroll
  for (int p = 0; p < K; ++p) { st.H[p] = 0.0; st.cnt[p] = 0; }
#pragma unroll
  for (int i = 0; i < (NPAIR > 0 ? NPAIR : 1); ++i) st.dis[i] = 0;

  // one element: level, sums, and its k bytes (+1 -> 0x01, -1 -> 0xFF) into bytes[0..K)
  auto element = [&](float v, uint8_t (&bytes)[K], float (&h32)[K], float& sx32) {
    uint32_t sp[NW];
    encode_elem<K>(tb, v, maxcnt, sp, h32, sx32);
    uint32_t bit[K];
#pragma unroll
    for (int p = 0; p < K; ++p) {
      bit[p] = (sp[p / 4] >> (8 * (p % 4))) & 1u;
      bytes[p] = bit[p] ? uint8_t(0x01) : uint8_t(0xFF);
      st.cnt[p] += bit[p];
    }
    int pi = 0;
#pragma unroll
    for (int p = 0; p < K; ++p)
#pragma unroll
      for (int q = p + 1; q < K; ++q) st.dis[pi++] += bit[p] ^ bit[q];
  };

  const int64_t quads = N / 4;
  const int64_t stride = int64_t(gridDim.x) * kBlock;
  const int64_t gtid = int64_t(blockIdx.x) * kBlock + tid;
  for (int64_t u = gtid; u < quads; u += stride) {
    float f[4];
    load_quad<T>(x + 4 * u, f);
    float h32[K];
    float sx32 = 0.0f;
#pragma unroll
    for (int p = 0; p < K; ++p) h32[p] = 0.0f;
    uint32_t out[K];  // 4 elements x K bytes = K dwords
#pragma unroll
    for (int w = 0; w < K; ++w) out[w] = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint8_t bytes[K];
      element(f[e], bytes, h32, sx32);
#pragma unroll
      for (int p = 0; p < K; ++p) {
        const int b = e * K + p;
        out[b / 4] |= uint32_t(bytes[p]) << (8 * (b % 4));
      }
    }
    store_dwords<K>(reinterpret_cast<uint32_t*>(payload) + u * K, out);
    st.Sx += double(sx32);
#pragma unroll
    for (int p = 0; p < K; ++p) st.H[p] += double(h32[p]);
  }
  {
    const int64_t i = quads * 4 + gtid;
    if (i < N) {
      float h32[K];
      float sx32 = 0.0f;
#pragma unroll
      for (int p = 0; p < K; ++p) h32[p] = 0.0f;
      uint8_t bytes[K];
      element(load_one(x + i), bytes, h32, sx32);
#pragma unroll
      for (int p = 0; p < K; ++p) payload[i * K + p] = bytes[p];
      st.Sx += double(sx32);
#pragma unroll
      for (int p = 0; p < K; ++p) st.H[p] += double(h32[p]);
    }
  }
  store_record<K>(st, call, red);
}

template <typename TO, int K>
__global__ __launch_bounds__(kBlock) void mbq_decode_plain_kernel(const uint8_t* __restrict__ payload,
                                                                  const float* __restrict__ header,
                                                                  TO* __restrict__ xhat, int64_t N) {
  constexpr int P = 1 << K;
  __shared__ float lut[P];
  const int tid = threadIdx.x;
  if (tid < P) {
    float v = 0.0f;
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const float a = header[p];
      v = __fadd_rn(v, ((tid >> p) & 1) ? a : -a);
    }
    lut[tid] = __fsub_rn(v, header[K]);
  }
  __syncthreads();
  const int64_t quads = N / 4;
  const int64_t stride = int64_t(gridDim.x) * kBlock;
  const int64_t gtid = int64_t(blockIdx.x) * kBlock + tid;
  for (int64_t u = gtid; u < quads; u += stride) {
    uint32_t w[K];
#pragma unroll
    for (int i = 0; i < K; ++i) w[i] = reinterpret_cast<const uint32_t*>(payload)[u * K + i];
    float f[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t pat = 0;
#pragma unroll
      for (int p = 0; p < K; ++p) {
        const int b = e * K + p;
        const uint32_t byte = (w[b / 4] >> (8 * (b % 4))) & 0xFFu;
        pat |= (((byte >> 7) & 1u) ^ 1u) << p;  // +1 (0x01) -> bit 1, -1 (0xFF) -> bit 0
      }
      f[e] = lut[pat];
    }
    store_quad<TO>(xhat + 4 * u, f);
  }
  const int64_t i = quads * 4 + gtid;
  if (i < N) {
    uint32_t pat = 0;
#pragma unroll
    for (int p = 0; p < K; ++p) pat |= (((uint32_t(payload[i * K + p]) >> 7) & 1u) ^ 1u) << p;
    store_one(xhat + i, lut[pat]);
  }
}

// ====================================================================== decode (D1 + D2)
// RAGGED: as in the encoder, vectors at any alignment and the last m % VEC columns one per thread: by the
// first rem_grid workgroups, beside the others and not behind them (7789 x 1027 float32, k = 2: 8.5 ->
// 8.2 us; 23 x 173913, k = 3, bfloat16 5.4 -> 4.9).
template <typename TO, int K, int VEC, bool RAGGED>
__global__ __launch_bounds__(kBlock) void mbq_decode_kernel(const uint8_t* __restrict__ payload,
                                                             const float* __restrict__ header,
                                                             TO* __restrict__ xhat, int64_t n, int64_t m,
                                                             int64_t ipg, int64_t items, ItemStep step, int rem_grid) {
  constexpr int P = 1 << K;
  __shared__ float lut[P];
  const int tid = threadIdx.x;
  if (tid < P) {
    // x_hat of a sign pattern: float32 sum of +-alpha_p, p = 0..k-1 from 0, minus m_q
    float v = 0.0f;
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const float a = header[p];
      v = __fadd_rn(v, ((tid >> p) & 1) ? a : -a);
    }
    lut[tid] = __fsub_rn(v, header[K]);
  }
  __syncthreads();

  // NC columns from column j of row group g, byte b of plane p of column c in byte c*K + p of w
  auto columns = [&](auto nc, int64_t g, int64_t j, const auto& w) {
    constexpr int NC = decltype(nc)::value;
    const int64_t row0 = g * 8;
    TO* dst = xhat + j;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      if (row0 + r < n) {
        float f[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          uint32_t pat = 0;
#pragma unroll
          for (int p = 0; p < K; ++p) {
            const int b = c * K + p;
            pat |= ((w[b / 4] >> (8 * (b % 4) + 7 - r)) & 1u) << p;
            // (or-ing in one bit after the other is one instruction a bit with its select; the wide
            // patterns' chains of ors the compiler regroups into one and a half)
            if constexpr (K >= 7) asm("" : "+v"(pat));
          }
          f[c] = lut[pat];
        }
        if constexpr (NC > 1 && RAGGED) store16_any(dst + (row0 + r) * m, narrow(f));
        else if constexpr (NC > 1) store_vec(dst + (row0 + r) * m, f);
        else store_one(dst + (row0 + r) * m, f[0]);
      }
    }
  };
  auto one_column = [&](int64_t g, int64_t j) {
    uint32_t w[(K + 3) / 4];
    const uint8_t* src = payload + (g * m + j) * K;
#pragma unroll
    for (int i = 0; i < (K + 3) / 4; ++i) w[i] = 0;
#pragma unroll
    for (int p = 0; p < K; ++p) w[p / 4] |= uint32_t(src[p]) << (8 * (p % 4));
    columns(std::integral_constant<int, 1>{}, g, j, w);
  };

  int block = blockIdx.x, grid = gridDim.x;
  if constexpr (RAGGED) {
    if (block < rem_grid) {
      const int64_t j0 = ipg * VEC, rem = m - j0, G = (n + 7) / 8;
      for (int64_t s = int64_t(block) * kBlock + tid; s < G * rem; s += int64_t(rem_grid) * kBlock) {
        const int64_t g = s / rem;
        one_column(g, j0 + s - g * rem);
      }
      return;
    }
    block -= rem_grid;
    grid -= rem_grid;
  }
  int64_t it = int64_t(block) * kBlock + tid;
  ItemPos pos;
  pos.g = it / ipg;
  pos.jv = it - pos.g * ipg;
  for (; it < items; it += int64_t(grid) * kBlock, item_advance(pos, step, ipg)) {
    if constexpr (VEC > 1) {
      constexpr int NDW = VEC * K / 4;
      const uint8_t* src = payload + ((pos.g * m + pos.jv * VEC) * K);
      uint32_t w[NDW];
      if constexpr (RAGGED) {
        __builtin_memcpy(w, src, sizeof(w));
      } else {
        const Dwords<NDW> in = *reinterpret_cast<const Dwords<NDW>*>(src);
#pragma unroll
        for (int i = 0; i < NDW; ++i) w[i] = in.v[i];
      }
      columns(std::integral_constant<int, VEC>{}, pos.g, pos.jv * VEC, w);
    } else {
      one_column(pos.g, pos.jv);
    }
  }
}

// ======================================================= residue initialisation (batch 0)
// rho_0 = x, b_j = sign(rho_j) (sign(0) = +1), alpha_j = mean|rho_j|, rho_(j+1) = rho_j - alpha_j b_j,
// carried in float64 like the definition.  alpha_j needs the whole tensor's |rho_j|, so the method
// is k passes over x.  Every workgroup of pass j adds up the records of pass j-1 itself, in the same
// order, and so has alpha_(j-1) without a kernel in between (that kernel took 4 us of each pass);
// workgroup 0 writes it down.  A batch-0 call on 32 x 401408 float32 at k = 2 / 3 / 4: 33.4 / 50.6 / 67.7
// -> 28.6 / 39.3 / 51.0 us; 64 x 802816: 85 / 128 / 176 -> 76 / 111 / 145 us.  (More workgroups for
// the last pass, 1024 to 2048 instead of 768, cost 1 to 3 us; fewer or more for the others as well.)
//
// Signs are taken from the sign bit (x + 0 has none for a zero, and no difference of two equal
// numbers has), so a step is a bit select and an add.  Where a residue is not a number all later ones
// and their mean are not, whatever sign is taken; only its plane bits need a compare
// (mbq_init_encode_kernel).

// Where pass j leaves its records (one double per workgroup and statistic, statistic-major).
constexpr int kInitPasses = 8;
static_assert(kInitPasses + kInitPasses + 2 <= nstat_of(8), "records of all passes, and k + 2 statistics of the last");

// alpha_j from the records of pass j, the same in every thread of every workgroup.
__device__ __forceinline__ float alpha_of_pass(const double* __restrict__ records, int nrec, double n_elems,
                                               WaveTotals& buf) {
  const int tid = threadIdx.x, wave = tid / kWave;
  double a = 0.0;
  for (int b = tid; b < nrec; b += kBlock) a += records[b];
  a = wave_sum(a);
  if ((tid & (kWave - 1)) == 0) buf.v[wave][0] = a;
  __syncthreads();
  a = 0.0;
#pragma unroll
  for (int w = 0; w < kBlock / kWave; ++w) a += buf.v[w][0];
  __syncthreads();  // the buffer is free again
  return float(a / n_elems);
}
// alpha_0 .. alpha_(J-1): the last from the records, which workgroup 0 also writes down, the others
// from where earlier passes left them.
template <int J>
__device__ __forceinline__ void alphas_of_passes(float* __restrict__ alpha_out, const double* __restrict__ records,
                                                 int nrec, double n_elems, WaveTotals& buf, double (&a)[J > 0 ? J : 1]) {
  if constexpr (J > 0) {
#pragma unroll
    for (int q = 0; q < J - 1; ++q) a[q] = double(alpha_out[q]);
    const float last = alpha_of_pass(records, nrec, n_elems, buf);
    if (blockIdx.x == 0 && threadIdx.x == 0) alpha_out[J - 1] = last;
    a[J - 1] = double(last);
  }
}
// rho <- rho - sign(rho) a
__device__ __forceinline__ double residue_step(double rho, double a) { return rho - __builtin_copysign(a, rho); }

// Pass J, sums only: sum of |rho_J| over tiles of 8192 elements (all of a thread's 16-byte loads of a
// tile in flight); one record per workgroup.
template <typename T, int J>
__global__ __launch_bounds__(kBlock) void mbq_init_pass_kernel(const T* __restrict__ x, int64_t N,
                                                                float* __restrict__ alpha_out,
                                                                const double* __restrict__ prev, int nprev,
                                                                double n_elems, double* __restrict__ records) {
  constexpr int VEC = Elem<T>::VEC;
  constexpr int LOADS = kTileElems / (kBlock * VEC);
  __shared__ WaveTotals red;
  const int tid = threadIdx.x;
  const int64_t tiles = N / kTileElems;
  uint4 raw[LOADS];
  auto ask = [&](int64_t tile) {
#pragma unroll
    for (int u = 0; u < LOADS; ++u) raw[u] = load16_stream(x + tile * kTileElems + (u * kBlock + tid) * VEC);
  };
  int64_t tile = blockIdx.x;
  if (tile < tiles) ask(tile);  // under way while alpha is formed
  double a[J > 0 ? J : 1];
  alphas_of_passes<J>(alpha_out, prev, nprev, n_elems, red, a);
  auto magnitude = [&](float v) {
    double rho = double(v + 0.0f);
#pragma unroll
    for (int q = 0; q < J; ++q) rho = residue_step(rho, a[q]);
    return fabs(rho);
  };
  double acc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) acc[e] = 0.0;
  while (tile < tiles) {
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      float f[VEC];
      widen(raw[u], f);
#pragma unroll
      for (int e = 0; e < VEC; ++e) acc[e] += magnitude(f[e]);
    }
    tile += gridDim.x;
    if (tile < tiles) ask(tile);
  }
  // behind the last whole tile
  for (int64_t i = tiles * kTileElems + int64_t(blockIdx.x) * kBlock + tid; i < N; i += int64_t(gridDim.x) * kBlock)
    acc[0] += magnitude(load_one(x + i));
#pragma unroll
  for (int e = 1; e < VEC; ++e) acc[0] += acc[e];
  const double sv[1] = {acc[0]};
  const double total = block_sum_stats<1>(sv, red);
  if (tid == 0) records[blockIdx.x] = total;
}

// Last pass (j = K-1) of a batch-0 compression: the signs b_0..b_(K-1) of every element need
// only alpha_0..alpha_(K-2), so the bit planes of B^0 are written in the same pass that adds up
// |rho_(K-1)| for alpha_(K-1).  Items as in the encoder (8 rows x VEC columns per lane, row loads
// contiguous across lanes), static grid-stride assignment.  Record per workgroup: sum|rho_(K-1)|,
// sum of x, +1 counts of the K planes.
template <typename T, int K, int VEC>
__global__ __launch_bounds__(kBlock) void mbq_init_encode_kernel(const T* __restrict__ x,
                                                                  float* __restrict__ alpha_out,
                                                                  const double* __restrict__ prev, int nprev,
                                                                  double n_elems, uint8_t* __restrict__ payload,
                                                                  double* __restrict__ records, int64_t n, int64_t m,
                                                                  int64_t ipg, int64_t items, ItemStep step) {
  constexpr int NW = (K + 3) / 4;
  constexpr int NDW = (VEC * K + 3) / 4;
  __shared__ WaveTotals red;
  const int tid = threadIdx.x;
  int64_t it = int64_t(blockIdx.x) * kBlock + tid;
  ItemPos pos;
  pos.g = it / ipg;
  pos.jv = it - pos.g * ipg;
  RawRow<VEC> fr[8];
  auto ask = [&]() {  // all row loads of an item, so that they overlap
    const int64_t row0 = pos.g * 8;
    const T* xc = x + row0 * m + pos.jv * VEC;
#pragma unroll
    for (int r = 0; r < 8; ++r)
      if (row0 + r < n) fr[r] = load_raw<T, VEC>(xc + r * m);
  };
  if (it < items) ask();  // under way while alpha is formed
  double a[K > 1 ? K - 1 : 1] = {};
  alphas_of_passes<K - 1>(alpha_out, prev, nprev, n_elems, red, a);
  // alpha_0 = mean|x| is finite exactly if every x is, and then every residue is.  Otherwise signs are
  // compared for: b_j = +1 where rho_j >= 0, which is false for what is not a number, whatever its sign
  // bit.  (One coefficient: nothing is known of x, and the pass is bound by its read of x either way.)
  const bool all_finite = __builtin_amdgcn_readfirstlane(fabs(a[0]) < double(__builtin_inff()) ? 1 : 0) != 0;
  double sum_abs = 0.0, sum_x = 0.0;
  uint32_t cnt[K];
#pragma unroll
  for (int p = 0; p < K; ++p) cnt[p] = 0;
  while (it < items) {
    const int64_t row0 = pos.g * 8;
    const int nrows = (n - row0) < 8 ? int(n - row0) : 8;
    uint32_t neg[VEC][K];  // sign bits, one row after the other entering at the bottom
#pragma unroll
    for (int c = 0; c < VEC; ++c)
#pragma unroll
      for (int q = 0; q < K; ++q) neg[c][q] = 0;
    float sx32 = 0.0f;
    auto rows = [&](auto finite) {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        if (r < nrows) {
          float row[VEC];
          widen_raw<VEC>(fr[r], row);
#pragma unroll
          for (int c = 0; c < VEC; ++c) {
            sx32 = __fadd_rn(sx32, row[c]);
            double rho = double(row[c] + 0.0f);
#pragma unroll
            for (int q = 0; q < K; ++q) {
              const uint32_t sign = decltype(finite)::value ? uint32_t(uint64_t(__double_as_longlong(rho)) >> 32)
                                                            : (rho >= 0.0 ? 0u : 0x80000000u);
              neg[c][q] = __builtin_amdgcn_alignbit(neg[c][q], sign, 31);
              if (q < K - 1) rho = residue_step(rho, a[q]);
            }
            sum_abs += fabs(rho);
          }
        }
      }
    };
    if (K > 1 && all_finite) rows(std::true_type{}); else rows(std::false_type{});
    // row r at bit 7-r; a missing row contributes 0 bits
    uint32_t acc[VEC][NW];
#pragma unroll
    for (int c = 0; c < VEC; ++c)
#pragma unroll
      for (int w = 0; w < NW; ++w) acc[c][w] = 0;
    const uint32_t valid = 0xFFu & (0xFFu << (8 - nrows));
#pragma unroll
    for (int c = 0; c < VEC; ++c)
#pragma unroll
      for (int q = 0; q < K; ++q) {
        const uint32_t plus = ~(neg[c][q] << (8 - nrows)) & valid;
        cnt[q] += __popc(plus);
        acc[c][q / 4] |= plus << (8 * (q % 4));
      }
    sum_x += double(sx32);
    uint8_t* dst = payload + ((pos.g * m + pos.jv * VEC) * K);
    if constexpr (VEC > 1 && K <= 4) {
      uint32_t out[NDW];
#pragma unroll
      for (int w = 0; w < VEC / 4; ++w) {
        const uint32_t q4[4] = {acc[4 * w][0], acc[4 * w + 1][0], acc[4 * w + 2][0], acc[4 * w + 3][0]};
        columns_to_payload<K>(q4, &out[K * w]);
      }
      store_dwords<NDW>(reinterpret_cast<uint32_t*>(dst), out);
    } else if constexpr (VEC > 1) {
      uint32_t out[NDW];
#pragma unroll
      for (int w = 0; w < NDW; ++w) out[w] = 0;
#pragma unroll
      for (int c = 0; c < VEC; ++c)
#pragma unroll
        for (int p = 0; p < K; ++p) {
          const int b = c * K + p;
          out[b / 4] |= ((acc[c][p / 4] >> (8 * (p % 4))) & 0xFFu) << (8 * (b % 4));
        }
      store_dwords<NDW>(reinterpret_cast<uint32_t*>(dst), out);
    } else {
#pragma unroll
      for (int p = 0; p < K; ++p) dst[p] = uint8_t(acc[0][p / 4] >> (8 * (p % 4)));
    }
    it += int64_t(gridDim.x) * kBlock;
    item_advance(pos, step, ipg);
    if (it < items) ask();
  }
  const int wave = tid / kWave, lane = tid & (kWave - 1);
  {
    const double sa = wave_sum(sum_abs), sx = wave_sum(sum_x);
    if (lane == 0) { red.v[wave][0] = sa; red.v[wave][1] = sx; }
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const double c = double(wave_sum(cnt[p]));
      if (lane == 0) red.v[wave][2 + p] = c;
    }
  }
  __syncthreads();
  if (tid < K + 2) {
    double total = red.v[0][tid];
    for (int w = 1; w < kBlock / kWave; ++w) total += red.v[w][tid];
    records[int64_t(tid) * gridDim.x + blockIdx.x] = total;
  }
}

// Batch 0 of a small tensor in one kernel instead of k + 1: an item of the encoder's kind per thread, its rows in registers for
// all k passes; between the passes the workgroups exchange their sums of |rho_j| through mailboxes, and the last one to
// end writes the rest of the header.
//
// The wait for the others is bounded as in scheme U's held pass: a workgroup that has looked `polls` times in
// vain adds up the missing parts itself, in the same order as their owners, so to the same bits, and posts them.
//
// A mailbox is two words, each with half of the float64 and the number of the exchange.  Every exchange of a call (k - 1,
// at most three) has a set of its own: a workgroup may be late for one that all others have left.
//
// What it saves is host time, about 3 us a launch; on the device it takes, k + 1 kernels / this (us, float32): 128 x 160, k = 2
// 8.4 / 6.6; 64 x 6144 k = 4 15.9 / 14.2; 64 x 16384 (64 workgroups) 9.4 / 9.2,
// 16.6 / 15.1; beyond the line mbq_first_held_kernel follows.
constexpr int kFirstBlock = 512, kFirstWaves = kFirstBlock / kWave;
struct SumExchange {
  double part[kHeldGrid / kWave];
  uint64_t missing[kHeldGrid / kWave];
};
struct SumBox {
  uint64_t *lo, *hi;
};
__device__ __forceinline__ SumBox sum_box(ChipMail* mail, int set, int b) {
  if (set == 0) return {mail->first + b, mail->last + b};
  if (set == 1) return {mail->more + b, between_box(mail, 0, b)};
  return {between_box(mail, 1, b), between_box(mail, 2, b)};
}
static_assert(kCounterStride * sizeof(uint32_t) == kBetweenStride * sizeof(uint64_t) && kMaxGroups * 8 == kHeldGrid && kDoneCounter < 16,
              "the boxes between the counters are behind the first eight of 32 words, which hold the counters");
__device__ __forceinline__ void post_sum(const SumBox& box, uint32_t tag, double v) {
  const uint64_t bits = uint64_t(__double_as_longlong(v)), t = uint64_t(tag) << 32;
  __hip_atomic_store(box.lo, t | uint32_t(bits), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(box.hi, t | uint32_t(bits >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Wavefronts 0 to 3 look for a lane's box each, at most `polls` times; `mine` is the lane's, `here` whether it is there.
// (Looking in vain holds up the others' posts, which go to the same lines: so the first look comes when most are there.  A
// first look at once / after 24 units of 64 cycles, 256 workgroups, k = 4, us: 64 x 20480 float32 19.3 / 13.2, 32 x 401408
// 37.4 / 31.8; after 12 34.2, after 48 33.3.  64 workgroups at once / after 16: 64 x 16384 17.0 / 15.5, 24: 15.5 / 14.2, two
// workgroups, k = 2 6.9 / 7.2.)
__device__ __forceinline__ void look_for_sums(ChipMail* mail, int set, uint32_t tag, int polls, double& mine, bool& here) {
  const SumBox at = sum_box(mail, set, threadIdx.x);
  if (gridDim.x > 64) __builtin_amdgcn_s_sleep(24);
  else if (gridDim.x >= 16) __builtin_amdgcn_s_sleep(16);
  for (int i = 0; i < polls && __ballot(!here) != 0; ++i) {
    if (i > 0) __builtin_amdgcn_s_sleep(4);
    if (here) continue;
    const uint64_t lo = __hip_atomic_load(at.lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t hi = __hip_atomic_load(at.hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    here = uint32_t(lo >> 32) == tag && uint32_t(hi >> 32) == tag;
    if (here) mine = __longlong_as_double((long long)((hi << 32) | uint32_t(lo)));
  }
}

// The sum of all workgroups' `total` (the same in all threads), in their order; part(b): workgroup b's, by all threads.
template <typename Part>
__device__ __forceinline__ double exchange_sums(ChipMail* mail, int set, uint32_t tag, int polls, double total, SumExchange& ex,
                                                Part part) {
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid & (kWave - 1);
  if (tid == 0) post_sum(sum_box(mail, set, blockIdx.x), tag, total);
  // threads 0 to 255 hold a workgroup's sum each, once it is there
  double one = 0.0;
  bool here = uint32_t(tid) >= gridDim.x;
  auto share = [&] {  // with the other wavefronts
    if (wave < kHeldGrid / kWave) {
      const uint64_t missing = __ballot(!here);
      const double t = wave_sum(one);
      if (lane == 0) {
        ex.missing[wave] = missing;
        ex.part[wave] = t;
      }
    }
    __syncthreads();
    int count = 0;
#pragma unroll
    for (int w = 0; w < kHeldGrid / kWave; ++w) count += __popcll((unsigned long long)ex.missing[w]);
    return __builtin_amdgcn_readfirstlane(count);
  };
  if (wave < kHeldGrid / kWave) look_for_sums(mail, set, tag, polls, one, here);
  for (int count = share(); count != 0; count = share()) {  // a workgroup less is missing after every turn, whatever becomes of its mailbox
    // one of the missing workgroups, another for neighbouring ones
    int skip = int(blockIdx.x) % count, found = 0;
#pragma unroll
    for (int w = 0; w < kHeldGrid / kWave; ++w) {
      uint64_t mw = ex.missing[w];
      const int number = __popcll((unsigned long long)mw);
      if (skip >= 0 && skip < number) {
        for (; skip > 0; --skip) mw &= mw - 1;
        found = w * kWave + __ffsll((unsigned long long)mw) - 1;
      }
      skip -= number;
    }
    const int b = __builtin_amdgcn_readfirstlane(found);
    const double t = part(b);  // (its barrier: ex has been read by all)
    if (tid == 0) post_sum(sum_box(mail, set, b), tag, t);
    if (tid == b) { one = t; here = true; }
    if (wave < kHeldGrid / kWave) look_for_sums(mail, set, tag, 1, one, here);
  }
  return (ex.part[0] + ex.part[1]) + (ex.part[2] + ex.part[3]);  // ex is free again behind the next barrier
}

template <typename T, int K, int VEC>
__global__ __launch_bounds__(kFirstBlock, 2) void mbq_first_kernel(const T* __restrict__ x, float* __restrict__ header,
                                                                   uint8_t* __restrict__ payload, uint32_t* ctrl,
                                                                   double* records, int64_t n, int64_t m, uint32_t ipg,
                                                                   uint32_t items, double n_elems, int polls) {
  constexpr int NDW = (VEC * K + 3) / 4;
  static_assert(K >= 1 && K <= 4, "plane bytes of a column in one word");
  __shared__ WaveTotals red;
  __shared__ SumExchange ex;
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid & (kWave - 1);
  ChipMail* mail = reinterpret_cast<ChipMail*>(reinterpret_cast<char*>(ctrl) + kMailOffset);
  // the thread's item in workgroup b: its first row and column, and how many rows it has (0: none)
  struct Place {
    int64_t row0, col;
    int rows;
  };
  auto place = [&](int b) {
    const uint32_t it = uint32_t(b) * kFirstBlock + uint32_t(tid);
    const uint32_t g = it / ipg;
    Place p;
    p.row0 = int64_t(g) * 8;
    p.col = int64_t(it - g * ipg) * VEC;
    p.rows = it < items ? (n - p.row0 < 8 ? int(n - p.row0) : 8) : 0;
    return p;
  };
  auto load = [&](const Place& p, RawRow<VEC> (&rows)[8]) {
    const T* xc = x + p.row0 * m + p.col;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      if constexpr (VEC > 1) rows[r].v = make_uint4(0u, 0u, 0u, 0u); else rows[r].v = 0u;
      if (r < p.rows) rows[r] = load_raw<T, VEC>(xc + r * m);
    }
  };
  const Place mine = place(blockIdx.x);
  RawRow<VEC> kept[8];
  load(mine, kept);
  const uint32_t calls = mail->calls[blockIdx.x];  // (behind the tensor's loads, which do not wait for it)

  double a[K > 1 ? K - 1 : 1] = {};
  // the sum of |rho_J| over the workgroup's items, whoever's items `rows` are; thread 0 has it
  auto add_item = [&](auto J, const RawRow<VEC> (&rows)[8], int nrows, double (&acc)[VEC]) {
    constexpr int j = decltype(J)::value;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      if (r < nrows) {
        float f[VEC];
        widen_raw<VEC>(rows[r], f);
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
          double rho = double(f[c] + 0.0f);
#pragma unroll
          for (int q = 0; q < j; ++q) rho = residue_step(rho, a[q]);
          acc[c] += fabs(rho);
        }
      }
    }
  };
  auto block_total = [&](double (&acc)[VEC]) {
#pragma unroll
    for (int c = 1; c < VEC; ++c) acc[0] += acc[c];
    const double t = wave_sum(acc[0]);
    if (lane == 0) red.v[wave][0] = t;
    __syncthreads();
    double total = red.v[0][0];
#pragma unroll
    for (int w = 1; w < kFirstWaves; ++w) total += red.v[w][0];
    return total;  // the buffer is free again behind the next barrier: one of exchange_sums
  };
  auto pass = [&](auto J) {
    constexpr int j = decltype(J)::value;
    double acc[VEC];
#pragma unroll
    for (int c = 0; c < VEC; ++c) acc[c] = 0.0;
    add_item(J, kept, mine.rows, acc);
    double total = block_total(acc);
    if (gridDim.x > 1)
      total = exchange_sums(mail, j, calls + 1u + uint32_t(j), polls, total, ex, [&](int b) {
        double other[VEC];
#pragma unroll
        for (int c = 0; c < VEC; ++c) other[c] = 0.0;
        RawRow<VEC> rows[8];
        const Place p = place(b);
        load(p, rows);
        add_item(J, rows, p.rows, other);
        return block_total(other);
      });
    else
      __syncthreads();
    const float alpha = float(total / n_elems);
    if (blockIdx.x == 0 && tid == 0) header[j] = alpha;
    a[j] = double(alpha);
  };
  if constexpr (K > 1) pass(std::integral_constant<int, 0>{});
  if constexpr (K > 2) pass(std::integral_constant<int, 1>{});
  if constexpr (K > 3) pass(std::integral_constant<int, 2>{});

  // last pass: signs, planes and sums, as in mbq_init_encode_kernel
  const bool all_finite = __builtin_amdgcn_readfirstlane(fabs(a[0]) < double(__builtin_inff()) ? 1 : 0) != 0;
  double sum_abs = 0.0, sum_x = 0.0;
  uint32_t cnt[K];
#pragma unroll
  for (int p = 0; p < K; ++p) cnt[p] = 0;
  {
    uint32_t neg[VEC][K];
#pragma unroll
    for (int c = 0; c < VEC; ++c)
#pragma unroll
      for (int q = 0; q < K; ++q) neg[c][q] = 0;
    float sx32 = 0.0f;
    auto rows = [&](auto finite) {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        if (r < mine.rows) {
          float row[VEC];
          widen_raw<VEC>(kept[r], row);
#pragma unroll
          for (int c = 0; c < VEC; ++c) {
            sx32 = __fadd_rn(sx32, row[c]);
            double rho = double(row[c] + 0.0f);
#pragma unroll
            for (int q = 0; q < K; ++q) {
              const uint32_t sign = decltype(finite)::value ? uint32_t(uint64_t(__double_as_longlong(rho)) >> 32)
                                                            : (rho >= 0.0 ? 0u : 0x80000000u);
              neg[c][q] = __builtin_amdgcn_alignbit(neg[c][q], sign, 31);
              if (q < K - 1) rho = residue_step(rho, a[q]);
            }
            sum_abs += fabs(rho);
          }
        }
      }
    };
    if (K > 1 && all_finite) rows(std::true_type{}); else rows(std::false_type{});
    uint32_t acc[VEC];
    const uint32_t valid = 0xFFu & (0xFFu << (8 - mine.rows));
#pragma unroll
    for (int c = 0; c < VEC; ++c) {
      acc[c] = 0;
#pragma unroll
      for (int q = 0; q < K; ++q) {
        const uint32_t plus = ~(neg[c][q] << (8 - mine.rows)) & valid;
        cnt[q] += __popc(plus);
        acc[c] |= plus << (8 * q);
      }
    }
    sum_x += double(sx32);
    if (mine.rows > 0) {
      uint8_t* dst = payload + ((mine.row0 / 8 * m + mine.col) * K);
      if constexpr (VEC > 1) {
        uint32_t out[NDW];
#pragma unroll
        for (int w = 0; w < VEC / 4; ++w) {
          const uint32_t q4[4] = {acc[4 * w], acc[4 * w + 1], acc[4 * w + 2], acc[4 * w + 3]};
          columns_to_payload<K>(q4, &out[K * w]);
        }
        store_dwords<NDW>(reinterpret_cast<uint32_t*>(dst), out);
      } else {
#pragma unroll
        for (int p = 0; p < K; ++p) dst[p] = uint8_t(acc[0] >> (8 * p));
      }
    }
  }
  double v[8] = {sum_abs, sum_x};
#pragma unroll
  for (int p = 0; p < K; ++p) v[2 + p] = double(cnt[p]);
  double* const rows = &red.v[0][0];
  rows[(tid / 16) * 8 + row_sum_index<8>(lane)] = row_sums<8>(v, lane);
  __syncthreads();
  if (tid < K + 2) {
    const double total = sum_of_rows<8>(rows, tid, kFirstWaves);
    double* const rec = records + int64_t(tid) * gridDim.x + blockIdx.x;
    __hip_atomic_store(rec, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  const bool last = last_workgroup(ctrl);
  if (K > 1 && gridDim.x > 1) count_exchanges(mail, calls, uint32_t(K - 1));
  if (!last) return;
  double* tot = red.v[0];
  const int nrec = int(gridDim.x);
  for (int s = wave; s < K + 2; s += kFirstWaves) {
    const double t = sum_records<true>(records + int64_t(s) * nrec, nrec, lane);
    if (lane == 0) tot[s] = t;
  }
  clear_work_counters(ctrl);
  __syncthreads();
  if (tid != 0) return;
  const float last_alpha = float(tot[0] / n_elems);
  header[K - 1] = last_alpha;
  double dot = 0.0;
#pragma unroll
  for (int p = 0; p < K; ++p) dot += (p == K - 1 ? double(last_alpha) : a[p < K - 1 ? p : 0]) * (2.0 * tot[2 + p] - n_elems);
  header[K] = float((dot - tot[1]) / n_elems);
}

// The same for larger tensors, up to SLOTS items per thread on 256 workgroups: the tensor is read once and stays in registers for
// all passes; the header's rest is left to mbq_init_finalize_kernel.  Items go by chunks of 64, one per wavefront: chunk
// (slot * 8 + wavefront) * 256 + workgroup, so that a last slot that is not full is spread over all workgroups.
// k kernels and their reads / this (whole call, us): 32 x 401408, k = 2, 3, 4 27.7 / 19.0, 39.2 / 25.0, 50.6 / 31.6, bfloat16 21.3 / 17.8,
// 30.8 / 25.7, 40.8 / 34.0; 64 x 40000, k = 3 17.6 / 12.1; 64 x 20480, k = 2 10.1 / 7.9; 3 x 800008 bfloat16 and the like as well.
// Of the 25 us at k = 3 the read takes 10 with the launch, an exchange about 2, a pass of float64 instructions 2 to 4.5 at two
// wavefronts per SIMD, the header's kernel 4.  Beside other work on another stream, kernels / this (us, 32 x 401408, k = 3, calls
// one behind the other): matrix products 326 / 160, small kernels 47 / 30, 512 MB copies without a pause 80 / 47.
template <typename T, int K, int SLOTS>
__global__ __launch_bounds__(kFirstBlock, 2) void mbq_first_held_kernel(const T* __restrict__ x, float* __restrict__ header,
                                                                        uint8_t* __restrict__ payload, uint32_t* ctrl,
                                                                        double* __restrict__ records, int64_t n, int64_t m,
                                                                        uint32_t ipg, uint32_t items, double n_elems,
                                                                        int polls) {
  constexpr int VEC = Elem<T>::VEC;
  constexpr int NDW = (VEC * K + 3) / 4;
  static_assert(K >= 2 && K <= 4, "plane bytes of a column in one word");
  __shared__ WaveTotals red;
  __shared__ SumExchange ex;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  ChipMail* mail = reinterpret_cast<ChipMail*>(reinterpret_cast<char*>(ctrl) + kMailOffset);
  const uint32_t chunks = (items + kWave - 1) / kWave;
  auto chunk_of = [&](int b, int slot) { return uint32_t((slot * kFirstWaves + wave) * kHeldGrid + b); };
  // the lane's item of a chunk: row group, place in it and rows (0: a copy of the last item, which counts nothing)
  struct Place {
    uint32_t g, jv;
    int rows;
  };
  auto place = [&](uint32_t chunk) {
    const uint32_t it = chunk * kWave + uint32_t(lane), at = it < items ? it : items - 1u;
    Place p;
    p.g = at / ipg;
    p.jv = at - p.g * ipg;
    const int64_t left = n - int64_t(p.g) * 8;
    p.rows = it < items ? (left < 8 ? int(left) : 8) : 0;
    return p;
  };
  // (the last row in the place of those that are not there: the loads are unconditional)
  auto load = [&](const Place& p, RawRow<VEC> (&rows)[8]) {
    const T* at = x + int64_t(p.g) * 8 * m + int64_t(p.jv) * VEC;
    const int64_t left = n - int64_t(p.g) * 8;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      rows[r] = load_raw<T, VEC>(at);
      if (r + 1 < left) at += m;
    }
  };
  // A row's values for one pass.  (An empty asm: widened, to 64 bits in the end, they would otherwise stay in registers from
  // one pass to the next, and be spilled.)
  auto widen_row = [](RawRow<VEC> row, float (&f)[VEC]) {
    asm volatile("" : "+v"(row.v.x), "+v"(row.v.y), "+v"(row.v.z), "+v"(row.v.w));
    widen_raw<VEC>(row, f);
  };
  RawRow<VEC> kept[SLOTS][8];
#pragma unroll
  for (int j = 0; j < SLOTS; ++j) {
    const uint32_t c = chunk_of(blockIdx.x, j);
    if (c < chunks) load(place(c), kept[j]);  // the same in all lanes
  }
  const uint32_t calls = mail->calls[blockIdx.x];

  double a[K - 1] = {};
  auto add_item = [&](auto J, const RawRow<VEC> (&rows)[8], int nrows, double (&acc)[VEC]) {
    constexpr int j = decltype(J)::value;
    auto add = [&](auto whole) {
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        if (!decltype(whole)::value && __ballot(r < nrows) == 0) break;
        float f[VEC];
        widen_row(rows[r], f);
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
          double rho = double(j > 0 ? f[c] + 0.0f : f[c]);
#pragma unroll
          for (int q = 0; q < j; ++q) rho = residue_step(rho, a[q]);
          acc[c] += decltype(whole)::value || r < nrows ? fabs(rho) : 0.0;
        }
      }
    };
    if (__ballot(nrows != 8) == 0) add(std::true_type{}); else add(std::false_type{});
  };
  auto block_total = [&](double (&acc)[VEC]) {
#pragma unroll
    for (int c = 1; c < VEC; ++c) acc[0] += acc[c];
    const double t = wave_sum(acc[0]);
    if (lane == 0) red.v[wave][0] = t;
    __syncthreads();
    double total = red.v[0][0];
#pragma unroll
    for (int w = 1; w < kFirstWaves; ++w) total += red.v[w][0];
    return total;  // the buffer is free again behind the next barrier: one of exchange_sums
  };
  auto pass = [&](auto J) {
    constexpr int j = decltype(J)::value;
    double acc[VEC];
#pragma unroll
    for (int c = 0; c < VEC; ++c) acc[c] = 0.0;
#pragma unroll
    for (int i = 0; i < SLOTS; ++i) {
      const uint32_t c = chunk_of(blockIdx.x, i);
      if (c < chunks) add_item(J, kept[i], place(c).rows, acc);
    }
    const double total = exchange_sums(mail, j, calls + 1u + uint32_t(j), polls, block_total(acc), ex, [&](int b) {
      double other[VEC];
#pragma unroll
      for (int c = 0; c < VEC; ++c) other[c] = 0.0;
#pragma nounroll
      for (int i = 0; i < SLOTS; ++i) {
        const uint32_t c = chunk_of(b, i);
        if (c >= chunks) break;
        const Place p = place(c);
        RawRow<VEC> rows[8];
        load(p, rows);
        add_item(J, rows, p.rows, other);
      }
      return block_total(other);
    });
    const float alpha = float(total / n_elems);
    if (blockIdx.x == 0 && tid == 0) header[j] = alpha;
    a[j] = double(alpha);
  };
  pass(std::integral_constant<int, 0>{});
  if constexpr (K > 2) pass(std::integral_constant<int, 1>{});
  if constexpr (K > 3) pass(std::integral_constant<int, 2>{});

  // last pass: signs, planes and sums, as in mbq_init_encode_kernel; by compares where a residue may not be finite
  const bool all_finite = __builtin_amdgcn_readfirstlane(fabs(a[0]) < double(__builtin_inff()) ? 1 : 0) != 0;
  double sum_abs = 0.0, sum_x = 0.0;
  uint32_t cnt[K];
#pragma unroll
  for (int p = 0; p < K; ++p) cnt[p] = 0;
#pragma unroll
  for (int i = 0; i < SLOTS; ++i) {
    const uint32_t chunk = chunk_of(blockIdx.x, i);
    if (chunk >= chunks) break;
    const Place p = place(chunk);
    uint32_t neg[VEC][K];
#pragma unroll
    for (int c = 0; c < VEC; ++c)
#pragma unroll
      for (int q = 0; q < K; ++q) neg[c][q] = 0;
    float sx32 = 0.0f;
    auto rows = [&](auto plain) {  // all rows there, all values finite
      constexpr bool PLAIN = decltype(plain)::value;
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        if (!PLAIN && __ballot(r < p.rows) == 0) {  // their bits are masked out
#pragma unroll
          for (int c = 0; c < VEC; ++c)
#pragma unroll
            for (int q = 0; q < K; ++q) neg[c][q] <<= 1;
          continue;
        }
        float row[VEC];
        widen_row(kept[i][r], row);
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
          sx32 = __fadd_rn(sx32, PLAIN || r < p.rows ? row[c] : 0.0f);
          double rho = double(row[c] + 0.0f);
#pragma unroll
          for (int q = 0; q < K; ++q) {
            const uint32_t sign = PLAIN ? uint32_t(uint64_t(__double_as_longlong(rho)) >> 32) : (rho >= 0.0 ? 0u : 0x80000000u);
            neg[c][q] = __builtin_amdgcn_alignbit(neg[c][q], sign, 31);
            if (q < K - 1) rho = residue_step(rho, a[q]);
          }
          sum_abs += PLAIN || r < p.rows ? fabs(rho) : 0.0;
        }
      }
    };
    if (all_finite && __ballot(p.rows != 8) == 0) rows(std::true_type{}); else rows(std::false_type{});
    uint32_t acc[VEC];
    const uint32_t valid = 0xFFu & (0xFFu << (8 - p.rows));
#pragma unroll
    for (int c = 0; c < VEC; ++c) {
      acc[c] = 0;
#pragma unroll
      for (int q = 0; q < K; ++q) {
        const uint32_t plus = ~neg[c][q] & valid;  // row r at bit 7 - r; rows that are not there give 0 bits
        cnt[q] += __popc(plus);
        acc[c] |= plus << (8 * q);
      }
    }
    sum_x += double(sx32);
    if (p.rows > 0) {
      uint32_t out[NDW];
#pragma unroll
      for (int w = 0; w < VEC / 4; ++w) {
        const uint32_t q4[4] = {acc[4 * w], acc[4 * w + 1], acc[4 * w + 2], acc[4 * w + 3]};
        columns_to_payload<K>(q4, &out[K * w]);
      }
      store_dwords<NDW>(reinterpret_cast<uint32_t*>(payload + (int64_t(p.g) * m + int64_t(p.jv) * VEC) * K), out);
    }
  }
  double v[8] = {sum_abs, sum_x};
#pragma unroll
  for (int p = 0; p < K; ++p) v[2 + p] = double(cnt[p]);
  double* const rows = &red.v[0][0];
  rows[(tid / 16) * 8 + row_sum_index<8>(lane)] = row_sums<8>(v, lane);
  __syncthreads();
  if (tid < K + 2) {
    const double total = sum_of_rows<8>(rows, tid, kFirstWaves);
    records[int64_t(tid) * gridDim.x + blockIdx.x] = total;
  }
  count_exchanges(mail, calls, uint32_t(K - 1));
}

// After the last pass: alpha_j = (sum of the workgroups' |rho_j| sums) / N, written to alpha_out[j]; of
// a batch-0 compression (nstat = k + 2) also the rest of the header:
// m_q = mean(B^0 alpha^0 - x) = (sum_p alpha_p (2 cnt_p - N) - sum x) / N  (eq. (biased error)),
// written behind the k coefficients that the earlier passes left in alpha_out.  A wavefront per
// statistic, as in mbq_finalize_kernel.
__global__ __launch_bounds__(kFinalizeBlock) void mbq_init_finalize_kernel(const double* __restrict__ records, int nrec,
                                                                            int nstat, double n_elems, int j,
                                                                            float* __restrict__ alpha_out) {
  __shared__ double tot[kInitPasses + 2];
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid & (kWave - 1);
  for (int s = wave; s < nstat; s += kFinalizeBlock / kWave) {
    const double t = sum_records(records + int64_t(s) * nrec, nrec, lane);
    if (lane == 0) tot[s] = t;
  }
  __syncthreads();
  if (tid != 0) return;
  const float a_j = float(tot[0] / n_elems);
  alpha_out[j] = a_j;
  if (nstat > 1) {
    const int k = nstat - 2;
    double dot = 0.0;
    for (int p = 0; p < k; ++p) {
      const double a_p = p == j ? double(a_j) : double(alpha_out[p]);
      dot += a_p * (2.0 * tot[2 + p] - n_elems);
    }
    alpha_out[k] = float((dot - tot[1]) / n_elems);
  }
}

// ============================================================================= host side
// Elements per vector: 16 bytes' worth; for the widths in use (k <= 4) at any alignment, where rows
// are long enough for wave-items and the tensor is large enough (ragged_columns).
//
// How large, in columns of all row groups: the columns that no vector covers take trips to memory of their own, where
// single columns all go at once; narrow rows have more such columns, and the ends of their rows are written in parts.
// Measured at 16 K to 54 M values, 4 to 101148 rows (us, single columns / vectors; encoder: k = 2; 3; 4):
//   decoder: 23 x 86957 4.4 / 4.8, 64 x 62501 6.2 / 5.4, 15 x 390403 9.0 / 7.2; float32 rows below 2048:
//     8315 x 1457 11.7 / 12.7, 10403 x 769 8.5 / 9.0, 16691 x 1519 21.2 / 20.0, 101148 x 535 42 / 40;
//   encoder, float32: 64 x 23437 6.8 / 6.9; 8.4 / 8.7; 9.6 / 10.1, 15 x 130003 7.4 / 7.15; 9.2 / 9.5; 10.0 / 10.35, 504 x 5003 7.3 / 7.3; 8.9 /
//     9.6; 10.1 / 10.6, 15 x 196613 8.5 / 7.8; 10.3 / 9.4; 11.1 / 10.5, 64 x 50001 8.0 / 7.9; 9.5 / 9.1; 10.8 / 10.2, 101 x 60001 11.3 / 9.8;
//     12.9 / 11.3; 13.9 / 12.2; rows below 4096 and a partial row group: 2614 x 1921 10.0 / 11.6; 11.5 / 13.6; 12.7 / 14.6, 8315 x 1457
//     18.2 / 19.4; 19.8 / 21.9; 21.1 / 23.1, 13113 x 1309 22.9 / 21.5; 24.5 / 23.5; 25.4 / 24.3, without one: 2000 x 3001 10.7 / 10.4;
//     12.3 / 12.2; 13.5 / 13.5; rows that leave a quarter or more of their wave-items' lanes idle: 55297 x 297 22.8 / 26.1; 24.4 / 29.5;
//     25.6 / 31.3, 19311 x 349 12.0 / 13.7; 13.5 / 16.6; 14.8 / 18.2;
//   encoder, bfloat16: 64 x 15625 7.25 / 7.95; 7.95 / 8.8; 8.9 / 9.8, 64 x 23437 8.1 / 8.0; 9.0 / 8.9; 9.75 / 10.0, 504 x 5003 8.8 / 8.4; 9.6 / 9.4; 10.2 /
//     10.5; with a partial row group 23 x 86957 8.4 / 8.4; 9.4 / 9.2; 10.05 / 10.4, 23 x 131073 9.7 / 8.9; 10.5 / 9.8; 10.9 / 11.1, 101 x
//     60001 12.6 / 9.3; 13.6 / 10.4; 13.8 / 11.5, 6001 x 1921 19.6 / 13.1; 20.5 / 14.3; 18.2 / 15.6; k = 1: 64 x 23437 6.9 / 6.9, 23 x 131073
//     7.9 / 7.9, 64 x 50001 8.1 / 7.85;
//   encoder, fewer than eight rows: float32 4 x 4001 4.65 / 5.4; 6.1 / 7.6; 6.9 / 8.5, 4 x 16383 5.0 / 5.4; 6.45 / 7.4; 7.3 / 8.5, and where
//     single columns are too many to finish by themselves 4 x 16387 5.3 / 5.2; 6.8 / 7.6; 7.9 / 8.5, 2 x 30001 5.4 / 4.95; 6.8 / 7.1; 7.9 /
//     8.2, 4 x 400001 7.3 / 6.5; 8.5 / 8.2; 9.6 / 9.2; bfloat16 4 x 4001 4.75 / 6.1; 6.2 / 6.9; 7.1 / 8.0, 4 x 16383 5.1 / 6.0; 6.6 / 7.0; 7.3 /
//     8.0, 2 x 30001 6.1 / 5.5; 6.8 / 6.65; 7.9 / 7.6, 4 x 400001 7.8 / 7.2; 8.6 / 7.7; 9.6 / 9.0.
int64_t ragged_columns(int dtype, int64_t n, int64_t m, int bits, bool encode) {
  const bool f32 = dtype == ACCEPT_F32;
  if (!encode) return f32 && m < 2048 ? int64_t(1) << 21 : int64_t(3) << 17;
  if (n < 8) return int64_t(kFinishGridMax) * 4 * kWave;  // (see tail_blocks in make_mplan)
  if (f32) {
    const int64_t ipg = m / Elem<float>::VEC, lanes = (ipg + kWave - 1) / kWave * kWave;
    if (4 * ipg < 3 * lanes) return INT64_MAX;
    return m < 4096 && n % 8 != 0 ? int64_t(3) << 19 : int64_t(3) << 17;
  }
  return n % 8 == 0 && bits > 1 ? int64_t(1) << 17 : int64_t(3) << 17;
}
int vec_for(int dtype, int64_t n, int64_t m, int bits, bool encode) {
  const int v = dtype == ACCEPT_BF16 ? 8 : 4;
  if (m % v == 0) return v;
  if (bits > 4 || m < v * kWave) return 1;
  return (n + 7) / 8 * m >= ragged_columns(dtype, n, m, bits, encode) ? v : 1;
}

int grid_for(int64_t items, int grid_max) {
  int64_t blocks = (items + kBlock - 1) / kBlock;
  if (blocks < 1) blocks = 1;
  return int(blocks < grid_max ? blocks : grid_max);
}

ItemStep step_for(int grid, int64_t ipg) {
  const int64_t stride = int64_t(grid) * kBlock;
  ItemStep st;
  st.dg = stride / ipg;
  st.dj = stride % ipg;
  return st;
}

MbqCall make_call(const accept_desc& d, const float* alpha_prev, void* header, void* ws) {
  MbqCall c;
  c.counters = static_cast<uint32_t*>(ws);
  c.records = reinterpret_cast<double*>(static_cast<char*>(ws) + kCtrlBytes);
  c.alpha_prev = alpha_prev;
  c.header = static_cast<float*>(header);
  c.n_elems = double(d.n) * double(d.m);
  const double beta = (1.0 + double(d.t)) / (10.0 + double(d.t));  // eq. (alpha update)
  c.beta = beta > 0.9 ? 0.9 : beta;
  return c;
}

template <typename T, int K, int VEC, bool RAGGED>
hipError_t launch_encode(const accept_desc& d, const MPlan& p, const T* x, uint8_t* payload, const MbqCall& call,
                         hipStream_t s) {
  // (only what direct_levels can ask for is compiled)
  constexpr bool F32 = sizeof(T) == 4;
  auto launch_narrow = [&](auto finish, auto direct) {
    hipLaunchKernelGGL((mbq_encode_kernel<T, K, 1, false, decltype(finish)::value, kRowsComplete, decltype(direct)::value, true>), dim3(p.grid),
                       dim3(kEncBlock), 0, s, x, payload, call, d.n, d.m, 1u, 1u, 0u, false, uint8_t(0));
    return hipGetLastError();
  };
  if constexpr (K == 1 && !F32) {
    if (!p.direct) return launch_narrow(std::false_type{}, std::false_type{});
  } else if constexpr (K == 3 || K == 4 || (K == 2 && !F32)) {
    if (p.direct && !p.wide) return launch_narrow(std::true_type{}, std::true_type{});
  }
  auto launch_one = [&](auto finish, auto rows, auto direct) {
    hipLaunchKernelGGL((mbq_encode_kernel<T, K, VEC, RAGGED, decltype(finish)::value, decltype(rows)::value, decltype(direct)::value, false>),
                       dim3(p.grid), dim3(kEncBlock), 0, s, x, payload, call, d.n, d.m, uint32_t(p.wide ? d.m / VEC : 1), p.wpg,
                       p.n_wave_items, p.wide, p.queue_shift);
  };
  auto launch_rows = [&](auto finish, auto rows) {
    constexpr bool kFinish = decltype(finish)::value, kFew = decltype(rows)::value == kRowsFew;
    if constexpr (K == 2 && F32 && !kFinish)
      p.direct ? launch_one(finish, rows, std::true_type{}) : launch_one(finish, rows, std::false_type{});
    else
      launch_one(finish, rows, std::bool_constant<K == 1 || (K == 2 && kFinish && (F32 || kFew))>{});
  };
  auto launch = [&](auto finish) {
    if (d.n < 8) launch_rows(finish, std::integral_constant<int, kRowsFew>{});
    else if (p.mixed) launch_rows(finish, std::integral_constant<int, kRowsMixed>{});
    else launch_rows(finish, std::integral_constant<int, kRowsComplete>{});
  };
  if constexpr (K <= 4) {
    if (p.finish) {
      launch(std::true_type{});
      return hipGetLastError();
    }
  }
  launch(std::false_type{});
  return hipGetLastError();
}

template <typename T, int VEC, bool RAGGED = false>
hipError_t encode_k(const accept_desc& d, const MPlan& p, const T* x, uint8_t* payload, const MbqCall& call,
                    hipStream_t s) {
  switch (d.bits) {
    case 1: return launch_encode<T, 1, VEC, RAGGED>(d, p, x, payload, call, s);
    case 2: return launch_encode<T, 2, VEC, RAGGED>(d, p, x, payload, call, s);
    case 3: return launch_encode<T, 3, VEC, RAGGED>(d, p, x, payload, call, s);
    case 4: return launch_encode<T, 4, VEC, RAGGED>(d, p, x, payload, call, s);
    default: break;
  }
  if constexpr (!RAGGED) {
    switch (d.bits) {
      case 5: return launch_encode<T, 5, VEC, false>(d, p, x, payload, call, s);
      case 6: return launch_encode<T, 6, VEC, false>(d, p, x, payload, call, s);
      case 7: return launch_encode<T, 7, VEC, false>(d, p, x, payload, call, s);
      case 8: return launch_encode<T, 8, VEC, false>(d, p, x, payload, call, s);
      default: break;
    }
  }
  return hipErrorInvalidValue;
}

template <typename TO, int K, int VEC, bool RAGGED>
hipError_t launch_decode(const accept_desc& d, const uint8_t* payload, const float* header, TO* xhat, hipStream_t s) {
  const int64_t ipg = d.m / VEC;
  const int64_t items = ((d.n + 7) / 8) * ipg;
  const int grid = grid_for(items, kDecodeGridMax);
  const int rem_grid = RAGGED ? grid_for(((d.n + 7) / 8) * (d.m - ipg * VEC), kDecodeGridMax) : 0;
  hipLaunchKernelGGL((mbq_decode_kernel<TO, K, VEC, RAGGED>), dim3(rem_grid + grid), dim3(kBlock), 0, s, payload, header,
                     xhat, d.n, d.m, ipg, items, step_for(grid, ipg), rem_grid);
  return hipGetLastError();
}

template <typename TO, int VEC, bool RAGGED = false>
hipError_t decode_k(const accept_desc& d, const uint8_t* payload, const float* header, TO* xhat, hipStream_t s) {
  switch (d.bits) {
    case 1: return launch_decode<TO, 1, VEC, RAGGED>(d, payload, header, xhat, s);
    case 2: return launch_decode<TO, 2, VEC, RAGGED>(d, payload, header, xhat, s);
    case 3: return launch_decode<TO, 3, VEC, RAGGED>(d, payload, header, xhat, s);
    case 4: return launch_decode<TO, 4, VEC, RAGGED>(d, payload, header, xhat, s);
    default: break;
  }
  if constexpr (!RAGGED) {
    switch (d.bits) {
      case 5: return launch_decode<TO, 5, VEC, false>(d, payload, header, xhat, s);
      case 6: return launch_decode<TO, 6, VEC, false>(d, payload, header, xhat, s);
      case 7: return launch_decode<TO, 7, VEC, false>(d, payload, header, xhat, s);
      case 8: return launch_decode<TO, 8, VEC, false>(d, payload, header, xhat, s);
      default: break;
    }
  }
  return hipErrorInvalidValue;
}

// What the passes of one initialisation share.
struct InitCall {
  float* alpha_out;
  const double* prev;  // records of the pass before
  int nprev;
  double* records;     // of this pass
  double n_elems;
};

template <typename T, int K, int VEC>
hipError_t launch_init_encode(const accept_desc& d, const T* x, const InitCall& c, uint8_t* payload, int grid,
                              hipStream_t s) {
  const int64_t ipg = d.m / VEC;
  const int64_t items = ((d.n + 7) / 8) * ipg;
  hipLaunchKernelGGL((mbq_init_encode_kernel<T, K, VEC>), dim3(grid), dim3(kBlock), 0, s, x, c.alpha_out, c.prev,
                     c.nprev, c.n_elems, payload, c.records, d.n, d.m, ipg, items, step_for(grid, ipg));
  return hipGetLastError();
}

template <typename T, int VEC>
hipError_t init_encode_k(const accept_desc& d, const T* x, const InitCall& c, uint8_t* payload, int grid, hipStream_t s) {
  switch (d.bits) {
    case 1: return launch_init_encode<T, 1, VEC>(d, x, c, payload, grid, s);
    case 2: return launch_init_encode<T, 2, VEC>(d, x, c, payload, grid, s);
    case 3: return launch_init_encode<T, 3, VEC>(d, x, c, payload, grid, s);
    case 4: return launch_init_encode<T, 4, VEC>(d, x, c, payload, grid, s);
    case 5: return launch_init_encode<T, 5, VEC>(d, x, c, payload, grid, s);
    case 6: return launch_init_encode<T, 6, VEC>(d, x, c, payload, grid, s);
    case 7: return launch_init_encode<T, 7, VEC>(d, x, c, payload, grid, s);
    case 8: return launch_init_encode<T, 8, VEC>(d, x, c, payload, grid, s);
    default: return hipErrorInvalidValue;
  }
}

// Batch 0 in one kernel: tensors of at most kFinishGridMax workgroups of an item per thread, the widths in use.
struct FirstPlan {
  int vec, grid;  // grid 0: not taken
  uint32_t ipg, items;
};
FirstPlan first_plan(const accept_desc& d, int vec) {
  FirstPlan f{};
  f.vec = d.m % vec == 0 ? vec : 1;
  const int64_t ipg = d.m / f.vec, items = (d.n + 7) / 8 * ipg;
  if (d.bits > 4 || items > int64_t(kFinishGridMax) * kFirstBlock) return f;
  f.ipg = uint32_t(ipg);
  f.items = uint32_t(items);
  f.grid = int((items + kFirstBlock - 1) / kFirstBlock);
  return f;
}
template <typename T, int K, int VEC>
hipError_t launch_first(const accept_desc& d, const FirstPlan& f, const T* x, float* header, uint8_t* payload, void* ws,
                        int polls, hipStream_t s) {
  double* records = reinterpret_cast<double*>(static_cast<char*>(ws) + kCtrlBytes);
  hipLaunchKernelGGL((mbq_first_kernel<T, K, VEC>), dim3(f.grid), dim3(kFirstBlock), 0, s, x, header, payload,
                     static_cast<uint32_t*>(ws), records, d.n, d.m, f.ipg, f.items, double(d.n) * double(d.m), polls);
  return hipGetLastError();
}
template <typename T, int VEC>
hipError_t first_k(const accept_desc& d, const FirstPlan& f, const T* x, float* header, uint8_t* payload, void* ws, int polls,
                   hipStream_t s) {
  switch (d.bits) {
    case 1: return launch_first<T, 1, VEC>(d, f, x, header, payload, ws, polls, s);
    case 2: return launch_first<T, 2, VEC>(d, f, x, header, payload, ws, polls, s);
    case 3: return launch_first<T, 3, VEC>(d, f, x, header, payload, ws, polls, s);
    case 4: return launch_first<T, 4, VEC>(d, f, x, header, payload, ws, polls, s);
    default: return hipErrorInvalidValue;
  }
}

// Batch 0 with the tensor kept in registers: items per thread of 256 workgroups; 0: not taken.
//
// Of fewer than eight rows an item has room for eight all the same, and its last pass goes by compares; kernels for every pass read and
// work through the rows that there are.  A kernel per pass / this, us, k = 2; 3; 4, float32: one row, 262144 items 10.1 / 9.65; 13.7 / 12.7;
// 17.8 / 15.8, 393000 10.8 / 11.45; 14.7 / 15.2; 19.3 / 19.2, 520000 11.6 / 13.2; 15.5 / 18.2; 20.4 / 22.2; two rows, 520000 13.6 / 14.4;
// 18.9 / 20.3; 24.1 / 24.8; from three on this is ahead everywhere (520000 15.9 / 15.4; 21.9 / 22.1; 28.0 / 27.8; seven 28.4 / 25.2; 39.1 /
// 33.1; 50.3 / 42.0).  bfloat16: one row, 180000 items 10.2 / 9.6; 14.3 / 12.6; 18.5 / 16.1, 524000 13.3 / 16.0; 18.9 / 22.6; 25.0 / 28.7;
// three, 180000 11.8 / 10.9; 16.9 / 15.1; 22.9 / 19.8, 205000 12.6 / 13.55; 18.0 / 20.0; 23.9 / 26.7; seven, 205000 17.8 / 18.7; 25.7 / 28.5;
// 34.4 / 38.5.  And just beyond half an item a thread, where one wavefront of five shares its SIMD: five rows, 76000 items 10.8 / 10.6;
// 15.0 / 14.9; 19.8 / 20.7, seven 11.7 / 11.7; 16.8 / 18.3; 22.5 / 24.9, but 84000 11.9 / 11.4; 17.0 / 16.1; 22.8 / 21.5.
constexpr int kFirstSlots = 4;
int first_slots(const accept_desc& d, int vec) {
  const int64_t items = d.m % vec == 0 ? (d.n + 7) / 8 * (d.m / vec) : INT64_MAX;
  constexpr int64_t kSlot = int64_t(kHeldGrid) * kFirstBlock;
  int64_t most = kFirstSlots * kSlot;
  if (d.n < 8) {
    most = vec == 8 ? kSlot / 2 * 3 : d.n <= 2 ? 2 * kSlot : most;
    if (vec == 8 && d.n >= 5 && items > kSlot / 2 && items <= kSlot / 8 * 5) return 0;
  }
  if (d.bits < 2 || d.bits > 4 || vec == 1 || items > most) return 0;
  return int((items + kHeldGrid * kFirstBlock - 1) / (kHeldGrid * kFirstBlock));
}
template <typename T, int K, int SLOTS>
hipError_t launch_first_held(const accept_desc& d, const T* x, float* header, uint8_t* payload, void* ws, double* records,
                             int polls, hipStream_t s) {
  const int64_t ipg = d.m / Elem<T>::VEC;
  hipLaunchKernelGGL((mbq_first_held_kernel<T, K, SLOTS>), dim3(kHeldGrid), dim3(kFirstBlock), 0, s, x, header, payload,
                     static_cast<uint32_t*>(ws), records, d.n, d.m, uint32_t(ipg), uint32_t((d.n + 7) / 8 * ipg),
                     double(d.n) * double(d.m), polls);
  return hipGetLastError();
}
template <typename T>
hipError_t first_held_k(const accept_desc& d, int slots, const T* x, float* header, uint8_t* payload, void* ws, double* records,
                        int polls, hipStream_t s) {
#define ACCEPT_FIRST(KK)                                                                                        \
  case KK:                                                                                                      \
    return slots == 1   ? launch_first_held<T, KK, 1>(d, x, header, payload, ws, records, polls, s)             \
           : slots == 2 ? launch_first_held<T, KK, 2>(d, x, header, payload, ws, records, polls, s)             \
                        : launch_first_held<T, KK, kFirstSlots>(d, x, header, payload, ws, records, polls, s);
  switch (d.bits) {
    ACCEPT_FIRST(2) ACCEPT_FIRST(3) ACCEPT_FIRST(4)
    default: return hipErrorInvalidValue;
  }
#undef ACCEPT_FIRST
}

template <typename T>
hipError_t launch_init_pass(int j, const T* x, int64_t N, const InitCall& c, int grid, hipStream_t s) {
#define ACCEPT_INIT(JJ)                                                                                        \
  case JJ:                                                                                                     \
    hipLaunchKernelGGL((mbq_init_pass_kernel<T, JJ>), dim3(grid), dim3(kBlock), 0, s, x, N, c.alpha_out, c.prev, \
                       c.nprev, c.n_elems, c.records);                                                         \
    break;
  switch (j) {
    ACCEPT_INIT(0) ACCEPT_INIT(1) ACCEPT_INIT(2) ACCEPT_INIT(3) ACCEPT_INIT(4) ACCEPT_INIT(5) ACCEPT_INIT(6) ACCEPT_INIT(7)
    default: return hipErrorInvalidValue;
  }
#undef ACCEPT_INIT
  return hipGetLastError();
}

}  // namespace

// Whether levels are found by comparing with every threshold, 2^k - 1 of them, instead of through tables that have to be built first
// (1.1 us; bfloat16's more).  Tables / comparisons (whole call, us): k = 1: 64 x 802816 float32 36.8 / 36.3, bfloat16 22.4 / 22.3, 15 x 20001
// 6.2 / 5.8; k = 2, float32: 4 x 65536 6.6 / 5.8, 64 x 32768 8.45 / 7.9, 15 x 390403 11.7 / 11.2, 64 x 400000 22.45 / 22.45, 64 x 802816
// 38.6 / 39.0; bfloat16: 4 x 65536 6.3 / 6.0, 64 x 16384 7.9 / 8.3, 64 x 400000 14.9 / 16.7; k = 3, float32: 64 x 8192 8.9 / 9.2, and
// bfloat16 9.5 / 11.7; but too narrow for wave-items, a column or less for a thread: 128 x 160, k = 2 6.8 / 5.7, k = 3
// 8.4 / 7.4, k = 4 9.8 / 9.05.  k = 1, bfloat16, too narrow for wave-items: 3000 x 256 6.45 / 5.95, 6000 x 256 7.4 / 7.2, 12000 x 256
// 8.3 / 8.6, 25000 x 128 9.1 / 9.75, 100000 x 256 48.7 / 72.4, 100000 x 504 90 / 136: tables beyond two columns for a thread.
bool direct_levels(const accept_desc& d, const MPlan& p) {
  constexpr int64_t kDirectColumns = 2 * int64_t(kEncodeGridMax) * kEncBlock;
  if (d.bits == 1) return d.in_dtype == ACCEPT_F32 || p.wide || p.G * d.m <= kDirectColumns;
  if (d.bits <= 4 && p.finish && !p.wide) return true;
  if (d.bits != 2) return false;
  return d.in_dtype == ACCEPT_BF16 ? d.n < 8 && p.finish : double(d.n) * double(d.m) < kThroughValues;
}

MPlan make_mplan(const accept_desc& d) {
  MPlan p{};
  p.vec = vec_for(d.in_dtype, d.n, d.m, d.bits, true);
  p.ragged = p.vec > 1 && d.m % p.vec != 0;
  p.G = (d.n + 7) / 8;
  // The encode kernel works on wave-items (64 items of one row group).  A row group needs at least
  // one full wave-item to be worth it, and numbers and row lengths have to fit 32 bits; other
  // geometries (very narrow tensors) go one column per thread.
  const int64_t ipg = d.m / p.vec;
  const int64_t wpg = (ipg + kWave - 1) / kWave;
  const int64_t full_groups = d.n / 8;
  // A partial row group behind complete ones is in the queue as well, except where items are single columns and complete
  // groups many: which rows a wave-item has costs scalar instructions for every one of them, a few percent of
  // that short work.  In the queue / beside it, float32, us: 15 x 20001, k = 2 7.2 / 7.6, 300 x 10001, k = 3 10.8 / 10.6, 8315 x
  // 1457, k = 2 20.2 / 19.6; vectors: 15 x 390403, k = 3 13.5 / 15.2, 23 x 173913 10.9 / 14.1, 101 x 500000, k = 4 42.6 / 43.9.
  constexpr int64_t kMixedColumnGroups = 16;
  p.mixed = d.n % 8 != 0 && full_groups > 0 && (p.vec > 1 || full_groups <= kMixedColumnGroups);
  const int64_t wave_items = (p.mixed ? p.G : full_groups) * wpg;
  p.wide = ipg >= kWave && wave_items < (int64_t(1) << 31) && d.m * 8 < (int64_t(1) << 32);
  p.stream = full_groups > 0 && p.wide;
  p.mixed = p.mixed && p.wide;
  p.wpg = p.wide ? uint32_t(wpg) : 1u;
  p.n_wave_items = p.stream ? uint32_t(wave_items) : 0u;
  {
    // one workgroup of 8 wavefronts per compute unit at most; fewer when there is less work
    int64_t blocks = p.stream ? (wave_items + kEncWaves - 1) / kEncWaves
                              : (full_groups * d.m + kEncBlock - 1) / kEncBlock;
    // The wave-items of fewer than eight rows are dealt to workgroups; where there are few of them, four to
    // a workgroup, which then are few enough to finish.  One to a workgroup and a finalize kernel / four (us, float32, n = 4,
    // k = 2; 4): 132 wave-items 6.9 / 6.5; 9.3 / 9.2, 256 6.9 / 6.7; 9.4 / 9.5, and with a line beyond, 260 6.9 / 6.8; 9.5 / 9.5,
    // 320 6.9 / 6.9; 9.4 / 9.7, 400 7.0 / 7.2; 9.4 / 9.9, 512 7.0 / 7.5; 9.4 / 10.2.
    const bool few = full_groups == 0 && wpg <= 4 * kFinishGridMax;
    // Where the partial row group is in the queue it has been counted; but of more than four bits several thresholds mostly
    // share a bucket, columns then go one per thread, and the grid is at least a row group's wave-items.  As many workgroups as the
    // queue needs / as this, k = 6, us: 9 x 100000 float32 20.5 / 17.1, bfloat16 30.3 / 17.8; 31 x 40000 20.7 / 17.1, 32.6 / 23.0.
    const bool counted = p.mixed && p.vec > 1 && d.bits <= 4;
    const int64_t tail_blocks = d.n % 8 == 0 || counted ? 0 : !p.wide ? (d.m + kEncBlock - 1) / kEncBlock : few ? (wpg + 3) / 4 : wpg;
    if (blocks < tail_blocks) blocks = tail_blocks;
    if (blocks < 1) blocks = 1;
    p.grid = int(blocks < kEncodeGridMax ? blocks : kEncodeGridMax);
  }
  // (see WorkQueue; in the kernel, which has this call's numbers later than its address, the coefficients' load waited for them:
  // 8 x 13488 bfloat16, k = 3 8.3 us, so 8.1)
  constexpr uint32_t kWavefronts = uint32_t(kEncodeGridMax) * uint32_t(kEncWaves);
  const bool two_sweeps = p.vec > 1 && p.n_wave_items > kWavefronts / 8u * 9u && p.n_wave_items <= kWavefronts / 8u * 15u;
  p.queue_shift = p.grid == kEncodeGridMax && !two_sweeps ? kGroupSlotsShift : kWaveSlotsShift;
  p.finish = d.layout == ACCEPT_LAYOUT_PACKED && d.bits <= 4 && p.grid <= kFinishGridMax;
  p.direct = direct_levels(d, p);
  // control block, then room for kMaxRecords records of the widest kind (k = 8)
  const size_t bytes = kCtrlBytes + size_t(nstat_of(8)) * kMaxRecords * sizeof(double);
  p.bytes = (bytes + 255) / 256 * 256;
  return p;
}

template <typename T>
hipError_t encode_plain_k(const accept_desc& d, int grid, const T* x, uint8_t* payload, const MbqCall& call,
                          hipStream_t s) {
  const int64_t N = d.n * d.m;
#define ACCEPT_ENC(KK)                                                                                         \
  case KK:                                                                                                     \
    hipLaunchKernelGGL((mbq_encode_plain_kernel<T, KK>), dim3(grid), dim3(kBlock), 0, s, x, payload, call, N); \
    break;
  switch (d.bits) {
    ACCEPT_ENC(1) ACCEPT_ENC(2) ACCEPT_ENC(3) ACCEPT_ENC(4) ACCEPT_ENC(5) ACCEPT_ENC(6) ACCEPT_ENC(7) ACCEPT_ENC(8)
    default: return hipErrorInvalidValue;
  }
#undef ACCEPT_ENC
  return hipGetLastError();
}

template <typename TO>
hipError_t decode_plain_k(const accept_desc& d, const uint8_t* payload, const float* header, TO* xhat,
                          hipStream_t s) {
  const int64_t N = d.n * d.m;
  const int grid = grid_for(N / 4 + 4, kDecodeGridMax);
#define ACCEPT_DEC(KK)                                                                                       \
  case KK:                                                                                                   \
    hipLaunchKernelGGL((mbq_decode_plain_kernel<TO, KK>), dim3(grid), dim3(kBlock), 0, s, payload, header, \
                       xhat, N);                                                                             \
    break;
  switch (d.bits) {
    ACCEPT_DEC(1) ACCEPT_DEC(2) ACCEPT_DEC(3) ACCEPT_DEC(4) ACCEPT_DEC(5) ACCEPT_DEC(6) ACCEPT_DEC(7) ACCEPT_DEC(8)
    default: return hipErrorInvalidValue;
  }
#undef ACCEPT_DEC
  return hipGetLastError();
}

hipError_t launch_mbq_compress(const accept_desc& d, const MPlan& p, const void* x, const float* alpha_prev,
                               void* header, void* payload, void* ws, hipStream_t s, StageTimer* tm) {
  const MbqCall call = make_call(d, alpha_prev, header, ws);
  uint8_t* pl = static_cast<uint8_t*>(payload);
  hipError_t e;
  mark(tm, s);
  int nrec = p.grid;
  if (d.layout == ACCEPT_LAYOUT_UNENCODED) {
    const int grid = nrec = grid_for(d.n * d.m / 4 + 4, kPlainGridMax);
    e = d.in_dtype == ACCEPT_BF16 ? encode_plain_k<bf16_t>(d, grid, static_cast<const bf16_t*>(x), pl, call, s)
                                  : encode_plain_k<float>(d, grid, static_cast<const float*>(x), pl, call, s);
  } else if (d.in_dtype == ACCEPT_BF16) {
    const bf16_t* xb = static_cast<const bf16_t*>(x);
    e = p.ragged     ? encode_k<bf16_t, 8, true>(d, p, xb, pl, call, s)
        : p.vec == 8 ? encode_k<bf16_t, 8>(d, p, xb, pl, call, s)
                     : encode_k<bf16_t, 1>(d, p, xb, pl, call, s);
  } else {
    const float* xf = static_cast<const float*>(x);
    e = p.ragged     ? encode_k<float, 4, true>(d, p, xf, pl, call, s)
        : p.vec == 4 ? encode_k<float, 4>(d, p, xf, pl, call, s)
                     : encode_k<float, 1>(d, p, xf, pl, call, s);
  }
  if (e != hipSuccess) return e;
  mark(tm, s);
  if (p.finish) return hipSuccess;
#define ACCEPT_FIN(KK)                                                                          \
  case KK:                                                                                      \
    hipLaunchKernelGGL(mbq_finalize_kernel<KK>, dim3(1), dim3(finalize_block(KK)), 0, s, call, nrec); \
    break;
  switch (d.bits) {
    ACCEPT_FIN(1) ACCEPT_FIN(2) ACCEPT_FIN(3) ACCEPT_FIN(4) ACCEPT_FIN(5) ACCEPT_FIN(6) ACCEPT_FIN(7) ACCEPT_FIN(8)
    default: return hipErrorInvalidValue;
  }
#undef ACCEPT_FIN
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  mark(tm, s);
  return hipSuccess;
}

hipError_t launch_mbq_decompress(const accept_desc& d, const void* header, const void* payload, void* xhat,
                                 hipStream_t s, StageTimer* tm) {
  const uint8_t* pl = static_cast<const uint8_t*>(payload);
  const float* hd = static_cast<const float*>(header);
  const int vec = vec_for(d.out_dtype, d.n, d.m, d.bits, false);
  hipError_t e;
  mark(tm, s);
  if (d.layout == ACCEPT_LAYOUT_UNENCODED) {
    e = d.out_dtype == ACCEPT_BF16 ? decode_plain_k<bf16_t>(d, pl, hd, static_cast<bf16_t*>(xhat), s)
                                   : decode_plain_k<float>(d, pl, hd, static_cast<float*>(xhat), s);
  } else if (d.out_dtype == ACCEPT_BF16) {
    bf16_t* o = static_cast<bf16_t*>(xhat);
    e = vec == 1         ? decode_k<bf16_t, 1>(d, pl, hd, o, s)
        : d.m % vec != 0 ? decode_k<bf16_t, 8, true>(d, pl, hd, o, s)
                         : decode_k<bf16_t, 8>(d, pl, hd, o, s);
  } else {
    float* o = static_cast<float*>(xhat);
    e = vec == 1         ? decode_k<float, 1>(d, pl, hd, o, s)
        : d.m % vec != 0 ? decode_k<float, 4, true>(d, pl, hd, o, s)
                         : decode_k<float, 4>(d, pl, hd, o, s);
  }
  if (e != hipSuccess) return e;
  mark(tm, s);
  return hipSuccess;
}

// Residue initialisation.  payload == nullptr: k sum passes, alpha^0 to alpha_out[0..k).
// Otherwise a batch-0 compression: k - 1 sum passes and one pass that also writes the bit planes
// of B^0 to payload; alpha_out is then the header, [alpha^0, m_q].
hipError_t launch_mbq_init(const accept_desc& d, const MPlan& p, const void* x, float* alpha_out, void* payload,
                           void* ws, hipStream_t s, int polls) {
  double* records = reinterpret_cast<double*>(static_cast<char*>(ws) + kCtrlBytes);
  const int64_t N = d.n * d.m;
  const int k = d.bits;
  const bool bf = d.in_dtype == ACCEPT_BF16;
  const bf16_t* xb = static_cast<const bf16_t*>(x);
  const float* xf = static_cast<const float*>(x);
  if (payload != nullptr) {
    const FirstPlan f = first_plan(d, p.vec);
    if (f.grid != 0) {
      uint8_t* pl = static_cast<uint8_t*>(payload);
      if (bf) return f.vec == 8 ? first_k<bf16_t, 8>(d, f, xb, alpha_out, pl, ws, polls, s) : first_k<bf16_t, 1>(d, f, xb, alpha_out, pl, ws, polls, s);
      return f.vec == 4 ? first_k<float, 4>(d, f, xf, alpha_out, pl, ws, polls, s) : first_k<float, 1>(d, f, xf, alpha_out, pl, ws, polls, s);
    }
  }
  hipError_t e;
  const int slots = payload != nullptr ? first_slots(d, bf ? Elem<bf16_t>::VEC : Elem<float>::VEC) : 0;
  if (slots != 0 && compute_units() >= kHeldGrid) {
    uint8_t* pl = static_cast<uint8_t*>(payload);
    e = bf ? first_held_k<bf16_t>(d, slots, xb, alpha_out, pl, ws, records, polls, s)
           : first_held_k<float>(d, slots, xf, alpha_out, pl, ws, records, polls, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(mbq_init_finalize_kernel, dim3(1), dim3(kFinalizeBlock), 0, s, records, kHeldGrid, k + 2, double(N),
                       k - 1, alpha_out);
    return hipGetLastError();
  }
  const int64_t tiles = (N + kTileElems - 1) / kTileElems;
  InitCall c{alpha_out, nullptr, 0, nullptr, double(N)};
  int nrec = 0, nstat = 1;
  for (int j = 0; j < k; ++j) {
    c.prev = c.records;
    c.nprev = nrec;
    c.records = records + int64_t(j) * kMaxRecords;
    if (payload != nullptr && j == k - 1) {
      uint8_t* pl = static_cast<uint8_t*>(payload);
      const int vec = d.m % p.vec == 0 ? p.vec : 1;
      nrec = grid_for(p.G * (d.m / vec), kPlainGridMax);
      nstat = k + 2;
      if (bf)
        e = vec == 8 ? init_encode_k<bf16_t, 8>(d, xb, c, pl, nrec, s) : init_encode_k<bf16_t, 1>(d, xb, c, pl, nrec, s);
      else
        e = vec == 4 ? init_encode_k<float, 4>(d, xf, c, pl, nrec, s) : init_encode_k<float, 1>(d, xf, c, pl, nrec, s);
    } else {
      nrec = int(tiles < kInitGrid ? tiles : kInitGrid);
      e = bf ? launch_init_pass<bf16_t>(j, xb, N, c, nrec, s) : launch_init_pass<float>(j, xf, N, c, nrec, s);
    }
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(mbq_init_finalize_kernel, dim3(1), dim3(kFinalizeBlock), 0, s, c.records, nrec, nstat, c.n_elems,
                     k - 1, alpha_out);
  return hipGetLastError();
}

}  // namespace accept
