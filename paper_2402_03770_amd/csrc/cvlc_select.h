// Order statistics of a short vector by one workgroup (gfx950): the keys (fp32 bits without the sign) at up to 32
// ranks are found together, by counts of 14, 9 and 8 bits.  The first count goes through the vector; the keys in the bins
// that hold a rank are then set aside in LDS and counted there, or, where they are too many (equal keys), in the
// vector again.  Part of the encoder and of the exponent fit, for vectors of up to kShortMax coordinates.
//
// All latency.  (With the keys in registers, 64 a thread, and everything unrolled over them there were 73 KB of code, more
// than the instruction cache holds, and nothing was gained over reading the vector from L2 once more.)
#pragma once

#include "cvlc_common.h"

namespace cvlc {
namespace {

constexpr uint32_t kShortBlock = 1024;
constexpr uint32_t kShortWaves = kShortBlock / kWave;
constexpr uint32_t kShortMax = 65536;
constexpr uint32_t kShortRanks = 32;
constexpr uint32_t kShortList = 256;                // keys that a wavefront sets aside
constexpr uint32_t kTopShift = 17, kTopBins = 1u << (31 - kTopShift);    // first count: the 14 highest bits
constexpr uint32_t kMidShift = 8, kMidDigits = 1u << (kTopShift - kMidShift);
constexpr uint32_t kLowDigits = 1u << kMidShift;
constexpr uint32_t kNoKey = 0xFFFFFFFFu;            // past the vector's end: below 0 as a signed number, no key is

// S.n_ranks and S.rank[0 .. n_ranks) are the caller's.
struct ShortSelect {
  union {
    alignas(16) uint32_t top[kTopBins];
    alignas(16) uint32_t mid[kShortRanks][kMidDigits];  // per bin of the first count that holds a rank
  };
  alignas(16) uint32_t low[kShortRanks][kLowDigits];    // per 23-bit prefix that holds a rank
  alignas(16) uint8_t tag[kTopBins];                    // 1 + the row of `mid` that counts this bin's keys, 0: none
  uint32_t list[kShortWaves][kShortList];  // keys in the bins that hold a rank, every wavefront those it has come across ...
  uint16_t at[kShortWaves][kShortList];    // ... their positions ...
  uint32_t n_list[kShortWaves];            // ... and how many they are
  uint32_t upto[kShortBlock];  // keys in the bins of threads 0 .. t (16 bins a thread, largest keys first)
  uint32_t scan_tmp[kShortWaves], members;
  uint32_t listed;             // 1: nobody's list ran over
  uint32_t n_ranks, extra, extra_bin, extra_rem;  // one more rank, or 0, whose bin of the first count is asked for
  // per rank (0: none); ranks ascend
  uint32_t rank[kShortRanks];
  uint32_t prefix[kShortRanks];  // the key's bits known so far, in the end all of them
  uint32_t rem[kShortRanks];     // rank among the keys with that prefix, in the end among the equal ones
  uint32_t row[kShortRanks];     // row of `mid`, then of `low`
  uint32_t equal[kShortRanks];   // keys equal to the rank's
};

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
  if (lane_id() == leader) atomicAdd(&counts[lead], (uint32_t)__popcll(same));
  else if (on && at != lead) atomicAdd(&counts[at], 1u);
}

// The first count and its running sums.  Zeros, of which a vector may hold any number, are not counted one by one.
// Whole workgroup; S.top is all zeros (and a barrier lies behind that).  Ends with a barrier.
__device__ __forceinline__ void count_top(ShortSelect& S, const float* update, uint32_t d) {
  visit_short(update, d, [&](uint32_t, const uint32_t (&key)[4]) {
#pragma unroll
    for (uint32_t c = 0; c < 4u; ++c)
      if ((int32_t)key[c] > 0) atomicAdd(&S.top[key[c] >> kTopShift], 1u);
  });
  __syncthreads();
  constexpr uint32_t kBins = kTopBins / kShortBlock;
  const uint4* mine = reinterpret_cast<const uint4*>(&S.top[kTopBins - kBins * (threadIdx.x + 1u)]);
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
__device__ __forceinline__ void find_top(const ShortSelect& S, uint32_t rank, uint32_t* bin, uint32_t* rem) {
  constexpr uint32_t kBins = kTopBins / kShortBlock;
  uint32_t t = 0;
#pragma unroll
  for (uint32_t step = kShortBlock / 2u; step; step >>= 1)
    if (S.upto[t + step - 1u] < rank) t += step;
  uint32_t left = rank - (t ? S.upto[t - 1u] : 0u), found = 0;
  const uint32_t largest = kTopBins - 1u - kBins * t;
#pragma unroll
  for (uint32_t i = 0; i < kBins; ++i) {  // the bin: as many of the thread's as the rank lies behind
    const uint32_t h = S.top[largest - i];
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
__device__ __forceinline__ void find_digits(ShortSelect& S, const uint32_t* counts, uint32_t row, uint32_t bits) {
  const uint32_t lane = lane_id(), mine = PER * (kWave - 1u - lane), r = min(lane, kShortRanks - 1u);
  const uint32_t my_row = S.row[r], rem = S.rem[r], prefix = S.prefix[r];
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

// What select_short needs all zeros: whole workgroup, a barrier before count_top.
__device__ __forceinline__ void clear_short(ShortSelect& S) {
  const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
  const uint32_t tid = threadIdx.x;
  for (uint32_t i = tid; i < kTopBins / 4u; i += kShortBlock) reinterpret_cast<uint4*>(S.top)[i] = zero;
  for (uint32_t i = tid; i < kShortRanks * kLowDigits / 4u; i += kShortBlock) reinterpret_cast<uint4*>(&S.low[0][0])[i] = zero;
  for (uint32_t i = tid; i < kTopBins / 16u; i += kShortBlock) reinterpret_cast<uint4*>(S.tag)[i] = zero;
  if (tid < kShortRanks) {  // no rank
    S.rank[tid] = S.prefix[tid] = S.rem[tid] = S.equal[tid] = 0;
    S.row[tid] = kNoKey;
  }
}

// After count_top: the bins of the first count that hold the ranks, S.members keys in all, and the extra rank's.  Whole
// workgroup; ends with a barrier.
__device__ __forceinline__ void locate_short(ShortSelect& S) {
  if (wave_id() == 0) {
    const uint32_t lane = lane_id(), n = S.n_ranks;
    const uint32_t rank = lane < n ? S.rank[lane] : (lane == kShortRanks ? S.extra : 0u);
    uint32_t bin = 0, rem = 0;
    if (rank) find_top(S, rank, &bin, &rem);
    bool opens;
    const uint32_t row = short_row(rank != 0u && lane < n, bin, &opens);
    if (opens) S.tag[bin] = (uint8_t)(row + 1u);
    const uint32_t members = wave_sum_u32(opens ? S.top[bin] : 0u);
    if (rank && lane < n) {
      S.prefix[lane] = bin;
      S.rem[lane] = rem;
      S.row[lane] = row;
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
__device__ __forceinline__ void select_short(ShortSelect& S, const float* update, uint32_t d) {
  const uint32_t tid = threadIdx.x, wave = wave_id(), lane = lane_id();
  // ranks ascend, so the last one's row is the last and its bin the lowest
  const uint32_t n = S.n_ranks, last = n ? n - 1u : 0u, members = S.members;
  if (members == 0u) return;  // uniform: no ranks
  const uint32_t n_rows = S.row[last] + 1u, floor_key = S.prefix[last] << kTopShift;
  __syncthreads();  // the counts of the first step have been read, by the caller too
  for (uint32_t i = tid; i < n_rows * (kMidDigits / 4u); i += kShortBlock)
    reinterpret_cast<uint4*>(&S.mid[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
  // A wavefront's keys go to a list of its own, at places it counts by itself (places from a counter of the workgroup's: the
  // atomics queue up at it, 6 us for 65 536 coordinates).  Wavefronts take turns over the vector, so that half the room is
  // theirs alike as a rule; where one's list runs over, nobody's is used.
  uint32_t n_mine = 0;  // uniform per wavefront
  if (members <= kShortWaves * kShortList / 2u) {
    visit_short(update, d, [&](uint32_t first, const uint32_t (&key)[4]) {
      uint32_t tag[4];
      uint64_t m[4];
#pragma unroll
      for (uint32_t c = 0; c < 4u; ++c) tag[c] = S.tag[(key[c] >> kTopShift) & (kTopBins - 1u)];
#pragma unroll
      for (uint32_t c = 0; c < 4u; ++c) m[c] = __ballot((int32_t)key[c] >= 0 && tag[c] != 0u);
      const uint32_t count = (uint32_t)(__popcll(m[0]) + __popcll(m[1]) + __popcll(m[2]) + __popcll(m[3]));
      if (count && n_mine + count <= kShortList) {  // uniform
        uint32_t place = n_mine + lanes_below(m[0]) + lanes_below(m[1]) + lanes_below(m[2]) + lanes_below(m[3]);
#pragma unroll
        for (uint32_t c = 0; c < 4u; ++c) {
          const bool kept = (int32_t)key[c] >= 0 && tag[c] != 0u;
          if (kept) {
            S.list[wave][place] = key[c];
            S.at[wave][place] = (uint16_t)(first + c);
          }
          place += kept ? 1u : 0u;
        }
      }
      n_mine += count;
    });
    if (lane == 0) S.n_list[wave] = n_mine;
  } else {
    n_mine = kNoKey;
  }
  const bool listed = !__syncthreads_or(n_mine > kShortList ? 1 : 0);
  if (tid == 0) S.listed = listed ? 1u : 0u;
  auto visit_members = [&](auto visit) {  // visit(row of mid, key, valid)
    auto tagged = [&](uint32_t key) {
      const uint32_t t = (int32_t)key >= (int32_t)floor_key ? S.tag[key >> kTopShift] : 0u;
      if (__ballot(t != 0u)) visit(t - 1u, key, t != 0u);
    };
    if (listed) {
      for (uint32_t i = lane; i - lane < n_mine; i += kWave) tagged(i < n_mine ? S.list[wave][i] : kNoKey);
    } else {
      visit_short(update, d, [&](uint32_t, const uint32_t (&key)[4]) {
#pragma unroll 1
        for (uint32_t c = 0; c < 4u; ++c) tagged(c == 0u ? key[0] : (c == 1u ? key[1] : (c == 2u ? key[2] : key[3])));
      });
    }
  };
  visit_members([&](uint32_t row, uint32_t key, bool on) {
    add_together(&S.mid[0][0], row * kMidDigits + ((key >> kMidShift) & (kMidDigits - 1u)), on);
  });
  __syncthreads();
  for (uint32_t row = wave; row < n_rows; row += kShortWaves) {
    find_digits<kMidDigits / kWave>(S, S.mid[row], row, kTopShift - kMidShift);
    // the row's counts give way to the rows of `low` (their number + 1) of the digits that hold a rank
    for (uint32_t i = lane; i < kMidDigits / 4u; i += kWave) reinterpret_cast<uint4*>(S.mid[row])[i] = make_uint4(0u, 0u, 0u, 0u);
  }
  __syncthreads();
  if (wave == 0) {
    const bool valid = lane < n && S.rank[min(lane, last)] != 0u;
    const uint32_t prefix = S.prefix[min(lane, last)], mid_row = S.row[min(lane, last)];
    bool opens;
    const uint32_t row = short_row(valid, prefix, &opens);
    if (opens) S.mid[mid_row][prefix & (kMidDigits - 1u)] = row + 1u;
    if (valid) S.row[lane] = row;
  }
  __syncthreads();
  const uint32_t n_low = S.row[last] + 1u;
  visit_members([&](uint32_t row, uint32_t key, bool on) {
    const uint32_t u = on ? S.mid[row][(key >> kMidShift) & (kMidDigits - 1u)] : 0u;
    add_together(&S.low[0][0], (u - 1u) * kLowDigits + (key & (kLowDigits - 1u)), u != 0u);
  });
  __syncthreads();
  for (uint32_t row = wave; row < n_low; row += kShortWaves) find_digits<kLowDigits / kWave>(S, S.low[row], row, kMidShift);
  __syncthreads();
}

// After select_short, for the ranks that cut a class of equal keys (S.rem < S.equal): the position of the rem-th of them.
// Small classes (two equal magnitudes at a boundary are nothing unusual) are looked for in the list, a wavefront per
// rank.  Otherwise one more pass counts every such class by parts of the vector, then a wavefront per rank searches its part.
// done(rank's index, position) is called by one thread.  Whole workgroup.
constexpr uint32_t kTieParts = 256;
template <class Done>
__device__ __forceinline__ void visit_ties(ShortSelect& S, const float* update, uint32_t d, Done done) {
  const uint32_t tid = threadIdx.x, wave = wave_id(), lane = lane_id();
  const uint32_t n_ranks = S.n_ranks, mine = min(lane, kShortRanks - 1u);
  const uint32_t my_equal = S.equal[mine], my_rem = S.rem[mine];  // every wavefront for itself: lane r = rank r
  const bool cut = lane < n_ranks && my_rem < my_equal;           // a rank that is 0: 0 < 0
  const uint64_t todo = __ballot(cut);
  if (!todo) return;  // uniform
  if (S.listed && !__ballot(cut && my_equal > kWave)) {
    for (uint32_t r = wave; r < n_ranks; r += kShortWaves) {  // uniform per wavefront
      if (!(todo >> r & 1u)) continue;
      const uint32_t key = S.prefix[r], rem = S.rem[r];
      uint32_t* found = S.low[r];  // the counts are done with
      uint32_t n = 0;
      for (uint32_t w = 0; w < kShortWaves; ++w) {
        const uint32_t n_list = S.n_list[w];
        for (uint32_t i = 0; i < n_list; i += kWave) {
          const bool hit = i + lane < n_list && S.list[w][i + lane] == key;
          const uint64_t hits = __ballot(hit);
          if (hit) found[n + lanes_below(hits)] = S.at[w][i + lane];
          n += (uint32_t)__popcll(hits);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      const uint32_t at = lane < n ? found[lane] : kNoKey;  // n = S.equal[r]
      uint32_t before = 0;
      for (uint32_t o = 0; o < n; ++o) before += __builtin_amdgcn_readlane(at, o) < at ? 1u : 0u;
      if (lane < n && before + 1u == rem) done(r, at);
    }
    return;
  }
  static_assert(kShortMax <= kTieParts * 256u && kShortRanks * kTieParts <= 2u * kShortWaves * kShortList, "a counter of 16 bits per class and part of 256 coordinates");
  uint32_t* counts = &S.list[0][0];  // of two neighbouring parts each
  bool opens;  // neighbouring ranks with equal keys share a class
  const uint32_t my_key = S.prefix[mine], my_low = S.row[mine], cls = short_row(cut, my_key, &opens);
  __syncthreads();
  for (uint32_t i = tid; i < kShortWaves * kShortList; i += kShortBlock) counts[i] = 0;
  for (uint32_t i = tid; i < kShortRanks * kLowDigits; i += kShortBlock) (&S.low[0][0])[i] = 0;
  __syncthreads();
  if (wave == 0 && opens) S.low[my_low][my_key & (kLowDigits - 1u)] = cls + 1u;  // the bins, then the digits, lead to it
  __syncthreads();
  const uint32_t floor_key = S.prefix[n_ranks - 1u];
  visit_short(update, d, [&](uint32_t first, const uint32_t (&keys)[4]) {
#pragma unroll 1
    for (uint32_t c = 0; c < 4u; ++c) {
      const uint32_t key = c == 0u ? keys[0] : (c == 1u ? keys[1] : (c == 2u ? keys[2] : keys[3]));
      const uint32_t t = (int32_t)key >= (int32_t)floor_key ? S.tag[key >> kTopShift] : 0u;
      if (!__ballot(t != 0u)) continue;  // uniform
      const uint32_t u = t ? S.mid[t - 1u][(key >> kMidShift) & (kMidDigits - 1u)] : 0u;
      const uint32_t v = u ? S.low[u - 1u][key & (kLowDigits - 1u)] : 0u;
      const uint64_t on = __ballot(v != 0u);
      if (!on) continue;  // uniform
      // one counter for most: the 64 coordinates lie in one part
      const uint32_t leader = (uint32_t)__builtin_ctzll(on), lead = __builtin_amdgcn_readlane(v, leader);
      const uint64_t same = __ballot(v == lead);
      const uint32_t part = first / 256u, word = ((v - 1u) * kTieParts + part) / 2u, shift = (part & 1u) * 16u;
      if (lane == leader) atomicAdd(&counts[word], (uint32_t)__popcll(same) << shift);
      else if (v && v != lead) atomicAdd(&counts[word], 1u << shift);
    }
  });
  __syncthreads();
  for (uint32_t r = wave; r < n_ranks; r += kShortWaves) {  // uniform per wavefront
    if (!(todo >> r & 1u)) continue;
    uint32_t rem = S.rem[r], part = 0;
    const uint32_t key = S.prefix[r], first = __builtin_amdgcn_readlane(cls, r) * kTieParts;
    for (uint32_t base = 0;; base += kWave) {  // the parts add up to S.equal, more than rem
      const uint32_t at = first + base + lane, n = (counts[at / 2u] >> ((at & 1u) * 16u)) & 0xFFFFu, upto = wave_incl_scan_u32(n);
      const uint64_t reached = __ballot(upto >= rem);
      if (reached || base + kWave >= kTieParts) {
        part = base + (reached ? (uint32_t)__builtin_ctzll(reached) : 0u);
        rem -= __builtin_amdgcn_readlane(upto - n, part - base);
        break;
      }
      rem -= __builtin_amdgcn_readlane(upto, kWave - 1u);
    }
#pragma unroll
    for (uint32_t c = 0; c < 4u; ++c) {  // the part's 256 coordinates, 64 at a time
      const uint32_t at = part * 256u + c * kWave + lane;
      const bool hit = at < d && (__float_as_uint(((ShortFloatPtr)update)[min(at, d - 1u)]) & 0x7FFFFFFFu) == key;
      const uint64_t hits = __ballot(hit);
      if (hit && lanes_below(hits) + 1u == rem) done(r, at);
      const uint32_t n = (uint32_t)__popcll(hits);
      rem = rem > n ? rem - n : 0u;  // found: no lane has place 0
    }
  }
}

}  // namespace
}  // namespace cvlc
