// Order statistics of a short vector by one workgroup (gfx950): the keys (fp32 bits without the sign) at up to 32
// ranks are found together, by counts of 14, 9 and 8 bits.  The first count goes through the vector; the keys in the bins
// that hold a rank are then set aside in LDS and counted there.  Where they are too many, a sample names a key of every such
// bin, and the keys equal to it are counted instead of set aside (many equal keys, the usual reason); where that does not
// help, the further counts go through the vector again.  For vectors of up to kShortMax coordinates; the encoder's short_select
// (EncodeSelect) and the exponent fit's rank_short (FitSelect) use it.  Both read the counters of the bins of Inf and NaN between
// count_top and select_short, so that the first count's stay as they are up to there.
//
// All latency, and instructions where keys are many: one per key of 65 536 is 0.4 us.  (With the keys in registers, 64 a
// thread, and everything unrolled over them there were 73 KB of code, more than the instruction cache holds, and nothing
// was gained over reading the vector from L2 once more.)
#pragma once

#include <type_traits>

#include "cvlc_common.h"

namespace cvlc {
namespace {

constexpr uint32_t kShortBlock = 1024;
constexpr uint32_t kShortWaves = kShortBlock / kWave;
constexpr uint32_t kShortMax = 65536;
constexpr uint32_t kShortRanks = 32;
constexpr uint32_t kShortList = 640;                // keys that a wavefront sets aside
constexpr uint32_t kParts = 256;                    // a part of the vector: 256 coordinates, a wavefront's visit
constexpr uint32_t kPartShift = 8;
static_assert(kShortMax <= kParts << kPartShift && kParts == kShortWaves * 16u, "sixteen visits a wavefront at most");
constexpr uint32_t kTopShift = 17, kTopBins = 1u << (31 - kTopShift);    // first count: the 14 highest bits
constexpr uint32_t kMidShift = 8, kMidDigits = 1u << (kTopShift - kMidShift);
constexpr uint32_t kLowDigits = 1u << kMidShift;
constexpr uint32_t kNoKey = 0xFFFFFFFFu;            // past the vector's end: below 0 as a signed number, no key is
constexpr uint32_t kNoSame = 0xFFFFFFFEu;           // no key, and not past the end

// S.n_ranks and S.rank[0 .. n_ranks) are the caller's.
struct ShortSelect {
  union {
    alignas(16) uint32_t top[kTopBins];
    alignas(16) uint32_t mid[kShortRanks][kMidDigits];  // per bin of the first count that holds a rank
  };
  alignas(16) uint32_t low[kShortRanks][kLowDigits];    // per 23-bit prefix that holds a rank
  alignas(16) uint8_t tag[kTopBins];                    // 1 + the row of `mid` that counts this bin's keys, 0: none
  // Keys in the bins that hold a rank, every wavefront those it has come across, in order: row << 25 | the bits below the
  // bin's << 8 | place in the part.  Its visits' first places (0xFFFF: no such visit) and the last d mod 4 coordinates'.
  alignas(16) uint32_t list[kShortWaves][kShortList];
  uint16_t start[kParts], tail_start;
  uint32_t n_list[kShortWaves];
  uint32_t upto[kShortBlock];  // keys in the bins of threads 0 .. t (16 bins a thread, largest keys first)
  uint32_t scan_tmp[kShortWaves], members;
  uint32_t pooled;             // kPooled: entries in the common part of the lists
  uint32_t listed;             // 1: nobody's list ran over
  uint32_t counted;            // 1: the keys equal to same[] are not in the lists, their numbers by parts are in `tag` ...
  uint32_t same_bits;          // ... 1 << same_bits places a row
  uint32_t others;             // sampled keys that would be in the lists
  uint32_t same[kShortRanks];  // the keys that are counted, each row's share of the places (same_place); kNoSame: none
  uint32_t n_same[kShortRanks];
  uint32_t bin_row[kShortRanks];  // per rank: row of `mid`
  uint32_t n_ranks, extra, extra_bin, extra_rem;  // one more rank, or 0, whose bin of the first count is asked for
  // per rank (0: none); ranks ascend
  uint32_t rank[kShortRanks];
  uint32_t prefix[kShortRanks];  // the key's bits known so far, in the end all of them
  uint32_t rem[kShortRanks];     // rank among the keys with that prefix, in the end among the equal ones
  uint32_t row[kShortRanks];     // row of `low`
  uint32_t equal[kShortRanks];   // keys equal to the rank's
};

// What the two users differ in.
// kSpread: the bins of the first count lie so that powers of two, and whatever else differs in the exponent alone, are not all in
// one bank of LDS: a fit of 65 536 coordinates of 7, 16 and 32 magnitudes, 2^-k each, 61, 58 and 58 us and now 44, 37 and 36 (in the launches
// of long vectors 56, 50 and 46).  An instruction a key, 0.2 us of 25; the encoder has never had its bins otherwise.
// kPooled: the members are counted only, in whatever order: of the lists' room a fifth is common to all wavefronts, so that a
// sorted vector's members, which a few of them come across, find room as a rule (65 536 sorted normal ones 50 us and now 36, 45
// in the launches of long vectors).
struct EncodeSelect : ShortSelect {
  static constexpr bool kSpread = false, kPooled = false;
};
struct FitSelect : ShortSelect {
  static constexpr bool kSpread = true, kPooled = true;
};

// Where a bin of the first count is.  Aligned sixteens of bins stay together.
template <class Select>
__device__ __forceinline__ uint32_t top_at(uint32_t bin) {
  return Select::kSpread ? bin ^ (bin >> 6) : bin;
}

typedef float __attribute__((ext_vector_type(4))) ShortFloat4;
typedef const ShortFloat4 __attribute__((address_space(1))) * ShortFloat4Ptr;
typedef const float __attribute__((address_space(1))) * ShortFloatPtr;

// The workgroup's visit to a vector, whole wavefronts together: visit(position, keys of it and the three behind it), the
// positions of a visit being 256 neighbouring ones from a multiple of 256 on (kNoKey past the end).
template <class Visit>
__device__ __forceinline__ void visit_short(const float* update, uint32_t d, Visit visit) {
  constexpr uint32_t kDeep = 2;
  ShortFloat4Ptr quads = (ShortFloat4Ptr)update;
  const uint32_t whole = d / 4u, tid = threadIdx.x;
  // Two sets of registers in turn, and no branch around the loads (past the end the last ones again): with copies from
  // one set to the other, or a branch, every wait is for all loads.
  ShortFloat4 even[kDeep], odd[kDeep];
  auto load = [&](uint32_t base, ShortFloat4 (&v)[kDeep]) {
#pragma unroll
    for (uint32_t u = 0; u < kDeep; ++u) v[u] = quads[min(base + u * kShortBlock + tid, whole - 1u)];
  };
  auto visit_set = [&](uint32_t base, const ShortFloat4 (&v)[kDeep]) {
#pragma unroll
    for (uint32_t u = 0; u < kDeep; ++u) {
      const uint32_t q = base + u * kShortBlock + tid;
      if ((uint32_t)__builtin_amdgcn_readfirstlane(q) >= whole) break;
      uint32_t key[4];
#pragma unroll
      for (uint32_t c = 0; c < 4u; ++c) key[c] = q < whole ? __float_as_uint(v[u][c]) & 0x7FFFFFFFu : kNoKey;
      visit(q * 4u, key);
    }
  };
  if (whole) {  // uniform
    load(0, even);
    for (uint32_t base = 0; base < whole; base += 2u * kDeep * kShortBlock) {
      load(base + kDeep * kShortBlock, odd);
      visit_set(base, even);
      load(base + 2u * kDeep * kShortBlock, even);
      visit_set(base + kDeep * kShortBlock, odd);
    }
  }
  const uint32_t rest = d % 4u;
  if (rest && wave_id() == 0) {
    const uint32_t at = whole * 4u + min(lane_id(), rest - 1u);
    const uint32_t key[4] = {lane_id() < rest ? __float_as_uint(((ShortFloatPtr)update)[at]) & 0x7FFFFFFFu : kNoKey, kNoKey, kNoKey, kNoKey};
    visit(at, key);
  }
}

// counts[at] += 1 for the lanes that are `on`.  Lanes that share the first one's counter add together: a rank inside a
// large class of equal keys would have all 64 queue up at one counter.
__device__ __forceinline__ void add_together(uint32_t* counts, uint32_t at, bool on) {
  const uint64_t mask = __ballot(on);
  if (!mask) return;  // uniform
  const uint32_t leader = (uint32_t)__builtin_ctzll(mask), lead = __builtin_amdgcn_readlane(at, leader);
  const uint64_t same = __ballot(on && at == lead);
  const bool first = lane_id() == leader;
  if (first || (on && at != lead)) atomicAdd(&counts[at], first ? (uint32_t)__popcll(same) : 1u);
}

// counts[at[c]] += unit for the lanes that are on[c], keys of a visit.  The first of them tells whether a class of kLargeClass
// lanes or more is about: then its members add together, and a second one's.  What is left is added one by one, which costs what the
// largest class of a wavefront has lanes, several times over.  (Looked for among all keys, classes cost a vector of 65 536
// different magnitudes 8 us; in a loop, of which there is no need, 1 us.)
// SCALE: bytes that `at` counts in.
constexpr uint32_t kLargeClass = 16;
template <uint32_t SCALE = 4u>
__device__ __forceinline__ void add_visit(uint32_t* counts, const uint32_t (&at)[4], bool (&on)[4], uint32_t unit) {
  auto counter = [&](uint32_t i) { return SCALE == 4u ? counts + i : reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(counts) + i * SCALE); };
  auto one_by_one = [&]() {
#pragma unroll
    for (uint32_t c = 0; c < 4u; ++c)
      if (on[c]) atomicAdd(counter(at[c]), unit);
  };
  uint32_t lead, n;
  auto large_class = [&]() {
    const uint64_t mask = __ballot(on[0]);
    lead = __builtin_amdgcn_readlane(at[0], mask ? (uint32_t)__builtin_ctzll(mask) : 0u);
    n = (uint32_t)__popcll(__ballot(on[0] && at[0] == lead));
    return n >= kLargeClass;  // uniform
  };
  auto together = [&]() {
#pragma unroll
    for (uint32_t c = 1; c < 4u; ++c) n += (uint32_t)__popcll(__ballot(on[c] && at[c] == lead));
    if (lane_id() == 0u) atomicAdd(counter(lead), n * unit);
#pragma unroll
    for (uint32_t c = 0; c < 4u; ++c) on[c] = on[c] && at[c] != lead;
  };
  if (!large_class()) {
    one_by_one();
    return;
  }
  together();
  if (large_class()) together();
  one_by_one();
}

// The first count and its running sums.  Zeros, of which a vector may hold any number, are not counted one by one.
// Whole workgroup; S.top is all zeros (and a barrier lies behind that).  Ends with a barrier.
template <class Select>
__device__ __forceinline__ void count_top(Select& S, const float* update, uint32_t d) {
  visit_short(update, d, [&](uint32_t, const uint32_t (&key)[4]) {
    uint32_t at[4];
    bool on[4];
#pragma unroll
    for (uint32_t c = 0; c < 4u; ++c) {
      // top_at, in bytes: (a ^ b) & c in one instruction (three-operand bitwise op with its truth table)
      if (Select::kSpread) at[c] = __builtin_amdgcn_bitop3_b32(key[c] >> (kTopShift - 2u), key[c] >> (kTopShift + 4u), (kTopBins - 1u) * 4u, 0x28);
      else at[c] = key[c] >> kTopShift;
      on[c] = (int32_t)key[c] > 0;
    }
    add_visit<Select::kSpread ? 1u : 4u>(S.top, at, on, 1u);
  });
  __syncthreads();
  constexpr uint32_t kBins = kTopBins / kShortBlock;
  const uint4* mine = reinterpret_cast<const uint4*>(&S.top[top_at<Select>(kTopBins - kBins * (threadIdx.x + 1u)) & ~(kBins - 1u)]);
  uint32_t sum = 0, total;
#pragma unroll
  for (uint32_t i = 0; i < kBins / 4u; ++i) {
    const uint4 q = mine[i];
    sum += q.x + q.y + q.z + q.w;
  }
  const uint32_t above = block_excl_scan<kShortWaves>(sum, S.scan_tmp, &total);
  const bool last = threadIdx.x == kShortBlock - 1u;  // owns the smallest keys
  S.upto[threadIdx.x] = last ? d : above + sum;
  if (last) S.top[0] += d - total;
  __syncthreads();
}

// Bin of the first count that holds the rank-th largest key (1 <= rank <= d) and the rank inside it.
template <class Select>
__device__ __forceinline__ void find_top(const Select& S, uint32_t rank, uint32_t* bin, uint32_t* rem) {
  constexpr uint32_t kBins = kTopBins / kShortBlock;
  uint32_t t = 0;
#pragma unroll
  for (uint32_t step = kShortBlock / 2u; step; step >>= 1)
    if (S.upto[t + step - 1u] < rank) t += step;
  uint32_t left = rank - (t ? S.upto[t - 1u] : 0u), found = 0;
  const uint32_t largest = kTopBins - 1u - kBins * t;
#pragma unroll
  for (uint32_t i = 0; i < kBins; ++i) {  // the bin: as many of the thread's as the rank lies behind
    const uint32_t h = S.top[top_at<Select>(largest - i)];
    if (found == i && left > h && i + 1u < kBins) {
      left -= h;
      ++found;
    }
  }
  *bin = largest - found;
  *rem = left;
}

// Neighbouring ranks with the same prefix share a row.  Lanes 0 .. kShortRanks - 1 of one wavefront, called by all of it:
// the lane's row (ranks that are 0 have none), and whether the lane is its row's first.
__device__ __forceinline__ uint32_t short_row(bool valid, uint32_t prefix, bool* opens) {
  const uint32_t lane = lane_id();
  const uint32_t before = __shfl_up(prefix, 1, 64), was_valid = __shfl_up(valid ? 1u : 0u, 1, 64);
  *opens = valid && (lane == 0 || !was_valid || before != prefix);
  return lanes_below(__ballot(*opens)) + (*opens ? 1u : 0u) - 1u;
}

// The digit that holds the rem-th largest of what a row counted, for all ranks of the row.  Whole wavefront: lane l adds up
// digits PER * (63 - l) + PER - 1 down, then a lane per rank searches the sums.
template <uint32_t PER>
__device__ __forceinline__ void find_digits(ShortSelect& S, const uint32_t* counts, const uint32_t* row_of, uint32_t row, uint32_t bits) {
  const uint32_t lane = lane_id(), mine = PER * (kWave - 1u - lane), r = min(lane, kShortRanks - 1u);
  const uint32_t my_row = row_of[r], rem = S.rem[r], prefix = S.prefix[r];
  uint32_t sum = 0;
#pragma unroll
  for (uint32_t i = 0; i < PER; i += 4u) {
    const uint4 q = *reinterpret_cast<const uint4*>(counts + mine + i);
    sum += q.x + q.y + q.z + q.w;
  }
  const uint32_t incl = wave_incl_scan_u32(sum);
  uint32_t t = 0;  // lanes whose digits lie above the rank's
#pragma unroll
  for (uint32_t step = kWave / 2u; step; step >>= 1) {
    const uint32_t upto = __shfl(incl, (int)(t + step - 1u), kWave);
    t += upto < rem ? step : 0u;
  }
  const uint32_t above = __shfl(incl, (int)(max(t, 1u) - 1u), kWave), first = PER * (kWave - 1u - min(t, kWave - 1u));
  uint32_t h[PER], left = rem - (t ? above : 0u), found = PER - 1u;
#pragma unroll
  for (uint32_t i = 0; i < PER; i += 4u) {
    const uint4 q = *reinterpret_cast<const uint4*>(counts + first + i);
    h[i] = q.x; h[i + 1u] = q.y; h[i + 2u] = q.z; h[i + 3u] = q.w;
  }
#pragma unroll
  for (uint32_t i = PER - 1u; i > 0u; --i)
    if (found == i && left > h[i]) {
      left -= h[i];
      --found;
    }
  uint32_t equal = h[0];
#pragma unroll
  for (uint32_t i = 1; i < PER; ++i) equal = found == i ? h[i] : equal;
  if (lane < S.n_ranks && my_row == row) {  // ranks that are 0 have no row
    S.prefix[lane] = (prefix << bits) | (first + found);
    S.rem[lane] = left;
    S.equal[lane] = equal;
  }
}

// Counters of 16 bits per class and part, two parts a word: the word.  (One word more a class: a visit counts one part of every
// class, which would all be in the same bank.)
constexpr uint32_t kPartWords = kParts / 2u + 1u;
__device__ __forceinline__ uint32_t part_word(uint32_t cls, uint32_t part) { return cls * kPartWords + part / 2u; }

// Place in S.same of a key in a bin with this row (keys that share one are as a rule a few, far apart in their low bits).
__device__ __forceinline__ uint32_t same_place(uint32_t row, uint32_t key, uint32_t bits) {
  return ((row << bits) + ((key ^ key >> 6 ^ key >> 13) & ((1u << bits) - 1u))) % kShortRanks;
}

// What select_short needs all zeros: whole workgroup, a barrier before count_top.
__device__ __forceinline__ void clear_short(ShortSelect& S) {
  const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
  const uint32_t tid = threadIdx.x;
  for (uint32_t i = tid; i < kTopBins / 4u; i += kShortBlock) reinterpret_cast<uint4*>(S.top)[i] = zero;
  for (uint32_t i = tid; i < kShortRanks * kLowDigits / 4u; i += kShortBlock) reinterpret_cast<uint4*>(&S.low[0][0])[i] = zero;
  for (uint32_t i = tid; i < kTopBins / 16u; i += kShortBlock) reinterpret_cast<uint4*>(S.tag)[i] = zero;
  if (tid < kShortRanks) {  // no rank
    S.rank[tid] = S.prefix[tid] = S.rem[tid] = S.equal[tid] = 0;
    S.row[tid] = S.bin_row[tid] = kNoKey;
    S.same[tid] = kNoSame;
    S.n_same[tid] = 0;
  }
  if (tid < kParts) S.start[tid] = 0xFFFFu;
  if (tid == 0) {
    S.tail_start = 0xFFFFu;
    S.others = S.pooled = 0;
  }
}

// After count_top: the bins of the first count that hold the ranks, S.members keys in all, and the extra rank's.  Whole
// workgroup; ends with a barrier.
template <class Select>
__device__ __forceinline__ void locate_short(Select& S) {
  if (wave_id() == 0) {
    const uint32_t lane = lane_id(), n = S.n_ranks;
    const uint32_t rank = lane < n ? S.rank[lane] : (lane == kShortRanks ? S.extra : 0u);
    uint32_t bin = 0, rem = 0;
    if (rank) find_top(S, rank, &bin, &rem);
    bool opens;
    const uint32_t row = short_row(rank != 0u && lane < n, bin, &opens);
    if (opens) S.tag[bin] = (uint8_t)(row + 1u);
    const uint32_t members = wave_sum_u32(opens ? S.top[top_at<Select>(bin)] : 0u);
    if (rank && lane < n) {
      S.prefix[lane] = bin;
      S.rem[lane] = rem;
      S.bin_row[lane] = row;
    }
    if (lane == kShortRanks) {
      S.extra_bin = bin;
      S.extra_rem = rem;
    }
    if (lane == 0) S.members = members;
  }
  __syncthreads();
}

// After locate_short: S.prefix, S.rem and S.equal of every rank of S.rank.  Whole workgroup; ends with a barrier.
template <class Select>
__device__ __forceinline__ void select_short(Select& S, const float* update, uint32_t d) {
  const uint32_t tid = threadIdx.x, wave = wave_id(), lane = lane_id();
  // ranks ascend, so the last one's row is the last
  const uint32_t n = S.n_ranks, last = n ? n - 1u : 0u, members = S.members;
  if (members == 0u) return;  // uniform: no ranks
  const uint32_t n_rows = S.bin_row[last] + 1u;
  __syncthreads();  // the counts of the first step have been read, by the caller too
  for (uint32_t i = tid; i < n_rows * (kMidDigits / 4u); i += kShortBlock)
    reinterpret_cast<uint4*>(&S.mid[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
  auto tag_of = [&](uint32_t key) { return (uint32_t)S.tag[(key >> kTopShift) & (kTopBins - 1u)]; };  // kNoKey: anything
  // A wavefront's keys go to a list of its own, at places it counts by itself (places from a counter of the workgroup's: the
  // atomics queue up at it, 6 us for 65 536 coordinates).  Wavefronts take turns over the vector, so that four fifths of the room
  // is theirs alike as a rule; where one's list runs over, nobody's is used.
  constexpr uint32_t kRoom = kShortWaves * kShortList, kOwn = Select::kPooled ? kShortList / 5u * 4u : kShortList, kPool = kRoom - kShortWaves * kOwn;
  uint32_t* const mine = &S.list[0][0] + wave * kOwn;
  // Past the vector's end the tag is the last bin's.  Only NaN may give it one: such vectors have no lists, which saves the lists'
  // pass a look at every key (1 us of 41).
  const bool lists = S.tag[kTopBins - 1u] == 0u;  // uniform
  bool list = lists && members <= kRoom / 5u * 4u;  // uniform
  const bool counted = !list;
  const uint32_t same_bits = 31u - (uint32_t)__builtin_clz(kShortRanks / n_rows);
  if (counted) {
    // Sixteen parts spread over the vector: some of the rows' keys, as likely as they are frequent, and what would
    // remain for the lists.  (One client of 65 536, encode, us, first with three passes over the vector in such cases, now, and in
    // the launches of long vectors: half kept in 3 groups of seven magnitudes 121, 69, 74; in 15 groups of bfloat16 values 103,
    // 54, 66; nine tenths in 31 groups of one magnitude 188, 95, 115, of different ones 72, 50, 68.)
    const uint32_t n_parts = (d + (1u << kPartShift) - 1u) >> kPartShift, part = wave * n_parts / kShortWaves;
    uint32_t key[4], tag[4];
#pragma unroll
    for (uint32_t c = 0; c < 4u; ++c) {
      const uint32_t at = (part << kPartShift) + c * kWave + lane;
      key[c] = at < d ? __float_as_uint(((ShortFloatPtr)update)[min(at, d - 1u)]) & 0x7FFFFFFFu : kNoKey;
    }
#pragma unroll
    for (uint32_t c = 0; c < 4u; ++c) {
      tag[c] = key[c] != kNoKey ? tag_of(key[c]) : 0u;
      if (tag[c]) S.same[same_place(tag[c] - 1u, key[c], same_bits)] = key[c];  // whoever comes last
    }
    __syncthreads();
    uint32_t others = 0;
#pragma unroll
    for (uint32_t c = 0; c < 4u; ++c) others += (uint32_t)__popcll(__ballot(tag[c] && S.same[same_place(tag[c] - 1u, key[c], same_bits)] != key[c]));
    if (lane == 0) atomicAdd(&S.others, others);
    __syncthreads();
    list = lists && (uint64_t)S.others * n_parts <= (uint64_t)kRoom / 10u * 9u * kShortWaves;
  }
  uint32_t n_mine = 0;  // uniform per wavefront
  bool over = false;    // kPooled: ... and whether a visit's found no room
  auto set_aside = [&](auto some_counted) {
    constexpr bool kCounted = decltype(some_counted)::value;
    visit_short(update, d, [&](uint32_t first, const uint32_t (&key)[4]) {
      const uint32_t part = __builtin_amdgcn_readfirstlane(first >> kPartShift);
      const bool tail = (uint32_t)__builtin_amdgcn_readfirstlane(key[1]) == kNoKey;
      uint32_t tag[4];
      uint64_t m[4];
      bool kept[4];
#pragma unroll
      for (uint32_t c = 0; c < 4u; ++c) tag[c] = tag_of(key[c]);  // past the end: none, see above
      if constexpr (kCounted) {
        bool same[4];
        uint32_t at[4];
#pragma unroll
        for (uint32_t c = 0; c < 4u; ++c) at[c] = same_place(tag[c] - 1u, key[c], same_bits);
#pragma unroll
        for (uint32_t c = 0; c < 4u; ++c) same[c] = S.same[at[c]] == key[c];  // which has a tag, then
#pragma unroll
        for (uint32_t c = 0; c < 4u; ++c) {
          at[c] = part_word(at[c], part);
          kept[c] = tag[c] != 0u && !same[c];
        }
        add_visit(&S.low[0][0], at, same, 1u << ((part & 1u) * 16u));
      } else {
#pragma unroll
        for (uint32_t c = 0; c < 4u; ++c) kept[c] = tag[c] != 0u;
      }
#pragma unroll
      for (uint32_t c = 0; c < 4u; ++c) m[c] = __ballot(kept[c]);
      const uint32_t count = (uint32_t)(__popcll(m[0]) + __popcll(m[1]) + __popcll(m[2]) + __popcll(m[3]));
      if (lane == 0 && !Select::kPooled) {
        if (tail) S.tail_start = (uint16_t)min(n_mine, 0xFFFEu);
        else S.start[part] = (uint16_t)min(n_mine, 0xFFFEu);
      }
      uint32_t from_place = n_mine;
      bool fits = n_mine + count <= kOwn;  // uniform
      if constexpr (Select::kPooled) {
        if (!fits) {
          uint32_t from = 0;
          if (lane == 0) from = atomicAdd(&S.pooled, count);
          from = __builtin_amdgcn_readfirstlane(from);
          from_place = (kShortWaves - wave) * kOwn + from;  // counted from the wavefront's own list
          fits = from + count <= kPool;
          over = over || !fits;
        } else {
          n_mine += count;
        }
      }
      if (count && fits) {  // uniform
        uint32_t place = from_place;
#pragma unroll
        for (uint32_t c = 0; c < 4u; ++c) place = __builtin_amdgcn_mbcnt_hi((uint32_t)(m[c] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[c], place));
        const uint32_t within = first & ((1u << kPartShift) - 1u);
#pragma unroll
        for (uint32_t c = 0; c < 4u; ++c) {
          if (kept[c]) mine[place] = ((tag[c] - 1u) << 25) + ((key[c] << kPartShift) & ((1u << 25) - 1u)) + (within + c);
          place += kept[c] ? 1u : 0u;
        }
      }
      if constexpr (!Select::kPooled) n_mine += count;
    });
  };
  static_assert(25u == kTopShift + kPartShift && kShortRanks <= 128u, "row, bits below the bin's, place: a word");
  if (list) {
    if (counted) set_aside(std::true_type{});
    else set_aside(std::false_type{});
    if (lane == 0) S.n_list[wave] = n_mine;
  }
  if constexpr (!Select::kPooled) over = n_mine > kShortList;
  const bool listed = !__syncthreads_or(!list || over ? 1 : 0);
  if (tid == 0) {
    S.listed = listed ? 1u : 0u;
    S.counted = listed && counted ? 1u : 0u;
    S.same_bits = same_bits;
  }
  if (list && counted) {
    // The numbers of equal keys make room for the third count.  The lists' entries know their rows, so they take the tags' place.
    static_assert(sizeof(S.tag) == kShortRanks * kParts * 2u && sizeof(S.low) >= kShortRanks * kPartWords * 4u, "16 bits per class and part");
    for (uint32_t place = wave; place < kShortRanks; place += kShortWaves) {  // uniform per wavefront
      if (S.same[place] == kNoSame) continue;
      uint32_t* by_part = &S.low[0][0] + place * kPartWords;
      const uint32_t a = by_part[lane], b = by_part[lane + kWave];
      by_part[lane] = by_part[lane + kWave] = 0;
      if (!listed) continue;
      uint32_t* to = reinterpret_cast<uint32_t*>(S.tag) + place * (kParts / 2u);
      to[lane] = a;
      to[lane + kWave] = b;
      const uint32_t total = wave_sum_u32((a & 0xFFFFu) + (a >> 16) + (b & 0xFFFFu) + (b >> 16));
      if (lane == 0) {
        S.n_same[place] = total;
        if (total) atomicAdd(&S.mid[place >> same_bits][(S.same[place] >> kMidShift) & (kMidDigits - 1u)], total);
      }
    }
  }
  // every entry of the lists, whole wavefronts together: visit(entry, whether there is one)
  auto for_listed = [&](auto visit) {
    for (uint32_t i = lane; i - lane < n_mine; i += kWave) visit(i < n_mine ? mine[i] : 0u, i < n_mine);
    if (!Select::kPooled) return;
    const uint32_t pooled = S.pooled;
    for (uint32_t i = tid; i - lane < pooled; i += kShortBlock) visit(i < pooled ? (&S.list[0][0])[kShortWaves * kOwn + i] : 0u, i < pooled);
  };
  if (listed) {
    for_listed([&](uint32_t entry, bool on) { add_together(&S.mid[0][0], entry >> 16, on); });  // row * kMidDigits + digit
  } else {
    visit_short(update, d, [&](uint32_t, const uint32_t (&key)[4]) {
      uint32_t at[4];
      bool on[4];
#pragma unroll
      for (uint32_t c = 0; c < 4u; ++c) at[c] = tag_of(key[c]);
#pragma unroll
      for (uint32_t c = 0; c < 4u; ++c) {
        on[c] = (int32_t)key[c] >= 0 && at[c] != 0u;
        at[c] = (at[c] - 1u) * kMidDigits + ((key[c] >> kMidShift) & (kMidDigits - 1u));
      }
      add_visit(&S.mid[0][0], at, on, 1u);
    });
  }
  __syncthreads();
  for (uint32_t row = wave; row < n_rows; row += kShortWaves) {
    find_digits<kMidDigits / kWave>(S, S.mid[row], S.bin_row, row, kTopShift - kMidShift);
    // the row's counts give way to the rows of `low` (their number + 1) of the digits that hold a rank
    for (uint32_t i = lane; i < kMidDigits / 4u; i += kWave) reinterpret_cast<uint4*>(S.mid[row])[i] = make_uint4(0u, 0u, 0u, 0u);
  }
  __syncthreads();
  if (wave == 0) {
    const bool valid = lane < n && S.rank[min(lane, last)] != 0u;
    const uint32_t prefix = S.prefix[min(lane, last)], mid_row = S.bin_row[min(lane, last)];
    bool opens;
    const uint32_t row = short_row(valid, prefix, &opens);
    if (opens) S.mid[mid_row][prefix & (kMidDigits - 1u)] = row + 1u;
    if (valid) S.row[lane] = row;
  }
  __syncthreads();
  const uint32_t n_low = S.row[last] + 1u;
  if (listed) {
    for_listed([&](uint32_t entry, bool on) {
      const uint32_t u = on ? (&S.mid[0][0])[entry >> 16] : 0u;
      add_together(&S.low[0][0], (u - 1u) * kLowDigits + ((entry >> kPartShift) & (kLowDigits - 1u)), u != 0u);
    });
    if (counted && wave == 0 && lane < kShortRanks && S.n_same[lane]) {
      const uint32_t key = S.same[lane], u = S.mid[lane >> same_bits][(key >> kMidShift) & (kMidDigits - 1u)];
      if (u) atomicAdd(&S.low[u - 1u][key & (kLowDigits - 1u)], S.n_same[lane]);
    }
  } else {
    visit_short(update, d, [&](uint32_t, const uint32_t (&key)[4]) {
      uint32_t at[4];
      bool on[4];
#pragma unroll
      for (uint32_t c = 0; c < 4u; ++c) at[c] = (int32_t)key[c] >= 0 ? tag_of(key[c]) : 0u;
#pragma unroll
      for (uint32_t c = 0; c < 4u; ++c) at[c] = at[c] ? S.mid[at[c] - 1u][(key[c] >> kMidShift) & (kMidDigits - 1u)] : 0u;
#pragma unroll
      for (uint32_t c = 0; c < 4u; ++c) {
        on[c] = at[c] != 0u;
        at[c] = (at[c] - 1u) * kLowDigits + (key[c] & (kLowDigits - 1u));
      }
      add_visit(&S.low[0][0], at, on, 1u);
    });
  }
  __syncthreads();
  for (uint32_t row = wave; row < n_low; row += kShortWaves) find_digits<kLowDigits / kWave>(S, S.low[row], S.row, row, kMidShift);
  __syncthreads();
}

// After select_short, for the ranks that cut a class of equal keys (S.rem < S.equal): the position of the rem-th of them.
// The class's keys by parts of the vector, then a wavefront per rank searches its part.  Keys that were counted instead of set
// aside have been counted by parts; the others are now, every wavefront those of its list, or without lists in one more
// pass.  done(rank's index, position) is called by one thread.  Whole workgroup.
template <class Done>
__device__ __forceinline__ void visit_ties(EncodeSelect& S, const float* update, uint32_t d, Done done) {
  const uint32_t tid = threadIdx.x, wave = wave_id(), lane = lane_id();
  const uint32_t n_ranks = S.n_ranks, mine = min(lane, kShortRanks - 1u);
  const uint32_t my_equal = S.equal[mine], my_rem = S.rem[mine];  // every wavefront for itself: lane r = rank r
  const bool cut = lane < n_ranks && my_rem < my_equal;           // a rank that is 0: 0 < 0
  const uint64_t todo = __ballot(cut);
  if (!todo) return;  // uniform
  const bool listed = S.listed != 0u;
  const uint32_t my_key = S.prefix[mine];
  const uint32_t my_place = S.counted ? same_place(S.bin_row[mine], my_key, S.same_bits) : 0u;
  const bool known = cut && S.counted && S.same[my_place] == my_key;  // counted by parts, in `tag`
  const uint64_t known_ranks = __ballot(known);
  // The third count is done with: in its place the numbers + 1 of the classes by the digits that lead to them, and the classes'
  // counts by parts.
  constexpr uint32_t kMarks = kShortRanks * kLowDigits, kCounts = kShortRanks * kPartWords;
  static_assert(sizeof(S.low) >= kMarks + kCounts * 4u, "a byte per row and digit, 16 bits per class and part");
  uint8_t* marks = reinterpret_cast<uint8_t*>(&S.low[0][0]);
  uint32_t* counts = &S.low[0][0] + kMarks / 4u;
  bool opens;  // neighbouring ranks with equal keys share a class
  const uint32_t my_low = S.row[mine], cls = short_row(cut && !known, my_key, &opens);
  if (todo != known_ranks) {  // uniform
    __syncthreads();
    for (uint32_t i = tid; i < (kMarks / 4u + kCounts) / 4u; i += kShortBlock) reinterpret_cast<uint4*>(&S.low[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    if (wave == 0 && opens) marks[my_low * kLowDigits + (my_key & (kLowDigits - 1u))] = (uint8_t)(cls + 1u);
    __syncthreads();
    if (listed) {
      const uint32_t n_mine = S.n_list[wave];
      for (uint32_t i = lane; i - lane < n_mine; i += kWave) {
        const uint32_t entry = i < n_mine ? S.list[wave][i] : 0u, u = i < n_mine ? (&S.mid[0][0])[entry >> 16] : 0u;
        const uint32_t v = u ? marks[(u - 1u) * kLowDigits + ((entry >> kPartShift) & (kLowDigits - 1u))] : 0u;
        if (!__ballot(v != 0u)) continue;  // uniform
        uint32_t visit = 0;  // the wavefront's last one that starts at or before the entry
#pragma unroll
        for (uint32_t step = kParts / kShortWaves / 2u; step; step >>= 1)
          if (S.start[(visit + step) * kShortWaves + wave] <= i) visit += step;
        const uint32_t part = wave == 0u && S.tail_start <= i ? d / 4u * 4u >> kPartShift : visit * kShortWaves + wave;
        // One by one, ten rounds at most: lanes with the same word may count different halves of it (the last d mod 4 coordinates'
        // part can be the neighbour of one of the first wavefront's).
        if (v) atomicAdd(&counts[part_word(v - 1u, part)], 1u << ((part & 1u) * 16u));
      }
    } else {
      visit_short(update, d, [&](uint32_t first, const uint32_t (&key)[4]) {
        uint32_t at[4];
        bool on[4];
#pragma unroll
        for (uint32_t c = 0; c < 4u; ++c) at[c] = (int32_t)key[c] >= 0 ? (uint32_t)S.tag[(key[c] >> kTopShift) & (kTopBins - 1u)] : 0u;
#pragma unroll
        for (uint32_t c = 0; c < 4u; ++c) at[c] = at[c] ? S.mid[at[c] - 1u][(key[c] >> kMidShift) & (kMidDigits - 1u)] : 0u;
#pragma unroll
        for (uint32_t c = 0; c < 4u; ++c) at[c] = at[c] ? (uint32_t)marks[(at[c] - 1u) * kLowDigits + (key[c] & (kLowDigits - 1u))] : 0u;
        const uint32_t part = __builtin_amdgcn_readfirstlane(first >> kPartShift);
#pragma unroll
        for (uint32_t c = 0; c < 4u; ++c) {
          on[c] = at[c] != 0u;
          at[c] = part_word(at[c] - 1u, part);
        }
        add_visit(counts, at, on, 1u << ((part & 1u) * 16u));
      });
    }
    __syncthreads();
  }
  for (uint32_t r = wave; r < n_ranks; r += kShortWaves) {  // uniform per wavefront
    if (!(todo >> r & 1u)) continue;
    const uint32_t key = S.prefix[r];
    const bool from_tag = known_ranks >> r & 1u;
    const uint32_t of = __builtin_amdgcn_readlane(from_tag ? my_place : cls, r);
    const uint32_t* from = (from_tag ? reinterpret_cast<const uint32_t*>(S.tag) + of * (kParts / 2u) : counts + of * kPartWords) + 2u * lane;
    const uint32_t a = from[0], b = from[1];
    const uint32_t by_part[kParts / kWave] = {a & 0xFFFFu, a >> 16, b & 0xFFFFu, b >> 16};  // the class's keys in parts 4 * lane ...
    uint32_t rem = S.rem[r];
    // the rem-th lies in the first part up to which there are as many
    const uint32_t sum = by_part[0] + by_part[1] + by_part[2] + by_part[3], upto = wave_incl_scan_u32(sum);
    const uint64_t reached = __ballot(upto >= rem);
    const uint32_t at = reached ? (uint32_t)__builtin_ctzll(reached) : kWave - 1u;  // the parts add up to S.equal, more than rem
    uint32_t left = rem - (upto - sum), part = 4u * lane;
#pragma unroll
    for (uint32_t i = 0; i + 1u < kParts / kWave; ++i)
      if (part == 4u * lane + i && left > by_part[i]) {
        left -= by_part[i];
        ++part;
      }
    rem = __builtin_amdgcn_readlane(left, at);
    part = __builtin_amdgcn_readlane(part, at);
#pragma unroll
    for (uint32_t c = 0; c < 4u; ++c) {  // the part's 256 coordinates, 64 at a time
      const uint32_t pos = (part << kPartShift) + c * kWave + lane;
      const bool hit = pos < d && (__float_as_uint(((ShortFloatPtr)update)[min(pos, d - 1u)]) & 0x7FFFFFFFu) == key;
      const uint64_t hits = __ballot(hit);
      if (hit && lanes_below(hits) + 1u == rem) done(r, pos);
      const uint32_t n = (uint32_t)__popcll(hits);
      rem = rem > n ? rem - n : 0u;  // found: no lane has place 0
    }
  }
}

}  // namespace
}  // namespace cvlc
