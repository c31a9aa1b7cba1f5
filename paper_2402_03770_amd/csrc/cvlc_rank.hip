// cvlc_rank.hip -- the first step of Algorithm 1: the decay exponent alpha_i of
// Definition 1, fitted on the GPU from each client's update vector.
//
// Definition 1 bounds the l-th largest magnitude by phi * l^alpha.  The fit is
// the least-squares slope of ln|U{l}| on ln l at the ranks l = 1, 2, 4, ... and
// l = d (zero magnitudes left out), so what the GPU must deliver is the exact
// magnitude at about log2(d) ranks that reach all the way to the smallest
// entry: order statistics of the whole vector, not only of its top k.
//
// Three radix levels over the 31-bit magnitude key (fp32 bits without the
// sign): 13 bits, then 9, then 9.  Every level is one streaming pass over the
// vectors (HBM bound) that counts digits in LDS, followed by a one-workgroup
// walk per client that turns counts into the next key prefix of every rank.
//
//   init        pointers of the vectors -> workspace; clears the counters
//   hist1       all keys: counts of key >> 18 (8192 bins, 32 KB of LDS)
//   walk<1>     per rank: its level-1 bin and its rank inside that bin; ranks
//               that share a prefix form a class (at most 32 classes)
//   pass<2>     keys whose level-1 bin belongs to a class: counts of the next
//               9 bits per class (32 x 512 bins, 64 KB of LDS)
//   walk<2>     22-bit prefixes, ranks inside, classes again
//   pass<3>     keys that match a 22-bit prefix: counts of the last 9 bits
//   walk<3>     the keys themselves; the fit (fp64, one thread per client)
//
// Vectors of up to 65 536 coordinates: one workgroup per client does all of it (rank_short).
//
// Only a few percent of a vector's keys lie in a level-1 bin that holds one of
// the ranks.  Given a workspace with room for them (cvlc_fit_workspace_bytes_for)
// the second pass writes those keys out, every wavefront to a stretch of its
// own, and the third pass never happens:
//   collect     (after hist1) the level-1 walk, by every workgroup for itself;
//               all keys: those whose level-1 bin belongs to a class go to the
//               wavefront's list (rows of 64 through LDS) and are counted on
//               their next 9 bits (level 2)
//   walk<2>, pass<3>, walk<3>   as above, the pass reading the lists
//
// Large calls do not even need the second pass: a sample says in which level-1
// bins the ranks can lie, give or take, and the first pass sets those bins' keys
// aside while it counts.
//   sample, guess   histograms of 4096 to 12288 pieces of 256 bytes in sixteen interleaved
//                   parts, and per rank the bins within 4.5 standard deviations
//                   of its place in their sum; the parts tell how far a place
//                   strays where the coordinates of a piece are alike
//   stream      all keys: counts of key >> 18; keys of the guessed bins go to
//               the wavefronts' lists
//   pass<2>, walk<2>, pass<3>, walk<3>   as above, the passes reading the lists, the
//               first after the level-1 walk; for a client with a rank outside the
//               guessed bins (known then, from the exact counts) collect
//               writes the lists anew
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "cvlc_common.h"
#include "cvlc_select.h"

namespace cvlc {
namespace {

constexpr uint32_t kRanksMax = CVLC_FIT_RANKS_MAX;
constexpr uint32_t kLevel1Bins = 8192;   // level 1: key >> 18
constexpr uint32_t kLevel1Shift = 18;
constexpr uint32_t kSubBits = 9;      // levels 2 and 3
constexpr uint32_t kSubBins = 1u << kSubBits;
constexpr uint32_t kRankBlock = 1024;
constexpr uint32_t kRankWaves = kRankBlock / kWave;
constexpr uint32_t kDeep = 4;         // float4 loads a thread keeps in flight
constexpr uint32_t kNoClass = 0xFFu;
static_assert(kRanksMax == 32, "one lane of half a wavefront per rank");

typedef const float __attribute__((address_space(1))) * GlobalFloatPtr;
typedef float __attribute__((ext_vector_type(4))) Float4V;
typedef const Float4V __attribute__((address_space(1))) * GlobalFloat4Ptr;

struct RankSet {  // the ranks of one call, ascending, as kernel arguments
  uint32_t n;
  uint32_t rank[kRanksMax];
};

// Per-client state; cleared by the init kernel.
struct RankCtl {
  uint32_t top[kLevel1Bins];               // level-1 counts of all d keys
  uint32_t sub[kRanksMax * kSubBins];   // per class: counts of the level's digit (cleared again by walk<2>)
  uint32_t prefix[kRanksMax];           // key prefix of rank j known so far (13, 22, 31 bits)
  uint32_t rem[kRanksMax];              // rank j counted inside its prefix class, 1-based from the largest key
  uint32_t cls[kRanksMax];              // class of rank j: classes number the distinct prefixes, largest first
  uint32_t cls_prefix[kRanksMax];
  uint32_t n_cls;
  uint32_t missed;                      // a rank lies outside the guessed bins: the lists do not hold its class
  uint32_t pad[2];
  uint8_t guess[kLevel1Bins / 8u];         // level-1 bins whose keys the lists hold, a bit each
};

struct RankLayout {
  size_t status, ptrs, ctl, list_cnt, lists, total;
  size_t zero_bytes;  // [status, ptrs) and the ctl array are cleared at the start of a call
  uint32_t blocks;    // workgroups per client in the collecting pass
  uint32_t wave_cap;  // keys a wavefront's list has room for (0: no lists, three passes)
};

size_t align256(size_t v) { return (v + 255u) & ~(size_t)255u; }

uint32_t pass_blocks_per_client(uint32_t d, uint32_t n, uint32_t per_cu);
uint32_t list_blocks_per_client(uint32_t d, uint32_t n);
uint32_t wave_cap_for(uint32_t d, uint32_t blocks);

// One pass fewer over the vectors for three small launches and longer lists, which are longest for vectors of rows with
// a scale of their own.  4 vectors of 25.6 M: 222 -> 217 us, of rows 211 -> 263; 12 of 11.2 M: 315 -> 254, of rows 290 ->
// 275; 32 of 11.2 M: 540 -> 431, of rows 528 -> 462.  For vectors that have the sample's pieces several times over.
bool one_pass_for(uint32_t n, uint32_t d) { return (uint64_t)n * d >= (7u << 24) && d >= (1u << 20); }

// d = 0: the layout without lists.  With lists, every wavefront of the collecting pass owns room for all
// the keys it reads (whole tiles, plus the last d % 4 coordinates), so nothing has to be counted first.
RankLayout rank_layout(uint32_t n, uint32_t d) {
  RankLayout L;
  size_t off = 0;
  L.status = off; off = align256(off + 256);
  L.ctl = off; off = align256(off + (size_t)n * sizeof(RankCtl));
  L.zero_bytes = off;
  L.ptrs = off; off = align256(off + (size_t)n * sizeof(const float*));
  L.list_cnt = L.lists = off;
  L.blocks = 0;
  L.wave_cap = 0;
  if (d) {
    L.blocks = list_blocks_per_client(d, n);
    L.wave_cap = wave_cap_for(d, L.blocks);
    const size_t n_lists = (size_t)n * L.blocks * kRankWaves;
    L.list_cnt = off; off = align256(off + n_lists * sizeof(uint32_t));
    L.lists = off; off = align256(off + n_lists * L.wave_cap * sizeof(uint32_t));
  }
  L.total = off;
  return L;
}

// ------------------------------------------------------------------ init
constexpr uint32_t kPtrChunk = 448;
struct PtrChunk {
  uint32_t first, count;
  const float* ptr[kPtrChunk];
};
static_assert(sizeof(PtrChunk) <= 3800, "kernel arguments are limited to 4 KB");

__global__ __launch_bounds__(256) void rank_init_kernel(const float** dst, PtrChunk c, uint4* zero, size_t zero_n16) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < zero_n16; i += (size_t)gridDim.x * blockDim.x)
    zero[i] = make_uint4(0u, 0u, 0u, 0u);
  if (blockIdx.x == 0)
    for (uint32_t i = threadIdx.x; i < c.count; i += blockDim.x) dst[c.first + i] = c.ptr[i];
}

// ------------------------------------------------------------------ the streaming passes
// A workgroup takes every gridDim.x-th tile of kRankBlock * kDeep float4; thread t
// reads the t-th, t+1024-th, ... float4 of the tile (clamped, so that no load sits
// under a branch) and hands every in-range key to `visit`.  The last d % 4
// coordinates go to the first threads of workgroup 0.
template <class Visit>
__device__ __forceinline__ void stream_keys(const float* update, uint32_t d, Visit visit) {
  const uint32_t n_quads = d / 4u;
  GlobalFloat4Ptr src = (GlobalFloat4Ptr)update;
  constexpr uint32_t kTileQuads = kRankBlock * kDeep;
  for (uint32_t q0 = blockIdx.x * kTileQuads; q0 < n_quads; q0 += gridDim.x * kTileQuads) {
    Float4V v[kDeep];
#pragma unroll
    for (uint32_t u = 0; u < kDeep; ++u) {
      const uint32_t q = q0 + u * kRankBlock + threadIdx.x;
      v[u] = __builtin_nontemporal_load(src + min(q, n_quads - 1u));
    }
#pragma unroll
    for (uint32_t u = 0; u < kDeep; ++u) {
      const uint32_t q = q0 + u * kRankBlock + threadIdx.x;
      if (q < n_quads) {
#pragma unroll
        for (int c = 0; c < 4; ++c) visit(__float_as_uint(v[u][c]) & 0x7FFFFFFFu);
      }
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < d - n_quads * 4u)
    visit(__float_as_uint(update[n_quads * 4u + threadIdx.x]) & 0x7FFFFFFFu);
}

__global__ __launch_bounds__(kRankBlock) void rank_hist1_kernel(const float* const* __restrict__ updates,
                                                                RankCtl* __restrict__ ctls, uint32_t d,
                                                                uint32_t* status) {
  __shared__ uint32_t hist[kLevel1Bins];
  RankCtl* ctl = ctls + blockIdx.y;
  for (uint32_t i = threadIdx.x; i < kLevel1Bins; i += kRankBlock) hist[i] = 0;
  __syncthreads();
  bool nonfinite = false;
  stream_keys(updates[blockIdx.y], d, [&](uint32_t key) {
    nonfinite |= key >= 0x7F800000u;
    atomicAdd(&hist[key >> kLevel1Shift], 1u);
  });
  const int any_nonfinite = __syncthreads_or((int)nonfinite);
  if (any_nonfinite && threadIdx.x == 0) atomicOr(status, CVLC_DEV_NONFINITE);
  for (uint32_t i = threadIdx.x; i < kLevel1Bins; i += kRankBlock) {
    const uint32_t h = hist[i];
    if (h) atomicAdd(&ctl->top[i], h);
  }
}

// LEVEL 2: prefix = level-1 bin, digit = bits 17..9.  LEVEL 3: prefix = top 22
// bits, digit = bits 8..0.  first_cls maps a level-1 bin to the first class whose
// prefix starts with it; classes are sorted, so the others follow it.
//
// LISTS: the keys come from the lists the collecting pass wrote (`lists`, `list_cnt`, `wave_cap`; a
// wavefront takes every (16 x workgroups)-th list of the client) instead of from the vectors.
struct KeyLists {
  const uint32_t* lists;
  const uint32_t* list_cnt;
  uint32_t per_client, wave_cap;
};

template <class Visit>
__device__ __forceinline__ void list_keys(const KeyLists& kl, Visit visit) {
  const uint32_t lane = lane_id();
  const uint32_t* __restrict__ cnts = kl.list_cnt + (size_t)blockIdx.y * kl.per_client;
  for (uint32_t l = blockIdx.x * kRankWaves + wave_id(); l < kl.per_client; l += gridDim.x * kRankWaves) {
    const uint32_t cnt = cnts[l];
    const uint32_t* __restrict__ keys = kl.lists + ((size_t)blockIdx.y * kl.per_client + l) * kl.wave_cap;
    for (uint32_t i0 = 0; i0 < cnt; i0 += kWave * 8u) {
      uint32_t k[8];
#pragma unroll
      for (uint32_t u = 0; u < 8; ++u) k[u] = keys[min(i0 + u * kWave + lane, cnt - 1u)];  // clamped: all in flight
#pragma unroll
      for (uint32_t u = 0; u < 8; ++u)
        if (i0 + u * kWave + lane < cnt) visit(k[u]);
    }
  }
}

// ------------------------------------------------------------------ the walks
// Ranks ascend, so their prefixes never increase: classes are runs of equal
// prefixes.  Called by the first 32 threads of a workgroup with the new prefix
// and inside-rank of rank `lane` (in LDS); writes the client's state.
// `ctl` may be null (nothing is written then).  Returns the number of classes; *cls_out / *opens_out: the
// caller's rank's class and whether that rank is the first of it.
__device__ __forceinline__ uint32_t write_classes(RankCtl* ctl, const uint32_t* s_prefix, const uint32_t* s_rem,
                                                  uint32_t n_ranks, uint32_t* cls_out = nullptr,
                                                  bool* opens_out = nullptr) {
  const uint32_t j = threadIdx.x;  // < 64, the first wavefront
  const bool live = j < n_ranks;
  const uint32_t mine = live ? s_prefix[j] : 0u;
  const bool opens = live && (j == 0 || s_prefix[j - 1] != mine);
  const uint64_t open_mask = __ballot(opens);
  const uint32_t c = lanes_below(open_mask) + (opens ? 1u : 0u) - 1u;  // classes opened up to and including j
  if (live && ctl) {
    ctl->prefix[j] = mine;
    ctl->rem[j] = s_rem[j];
    ctl->cls[j] = c;
    if (opens) ctl->cls_prefix[c] = mine;
  }
  const uint32_t n_cls = (uint32_t)__popcll(open_mask);
  if (j == 0 && ctl) ctl->n_cls = n_cls;
  if (cls_out) *cls_out = c;
  if (opens_out) *opens_out = opens;
  return n_cls;
}

// Level 1, whole workgroup: from the client's counts of key >> 18, the bin of every rank and the rank inside it
// (into LDS, valid after the next barrier, up to which `sums` is in use).  A wavefront per rank searches the running sums, the block
// of 128 bins first: most ranks lie in the bins of one or two wavefronts, so that threads that look for the ranks in their own
// bins leave them to those: pass<2> with its walk 28.0 us -> 23.9 at 32 x 11.2 M, the call 390.6 -> 384.5, 1 x 11.2 M 51.6 -> 44.9,
// 8 x 1.2 M 50.9 -> 41.9, 1 x 300 000 33.1 -> 26.6.
constexpr uint32_t kBlockBins = kLevel1Bins / kWave, kWalkSums = kLevel1Bins + 1u + kWave + 1u;
static_assert(kBlockBins == 2u * kWave && kWalkSums <= kRanksMax * kSubBins, "two bins of a block per lane; room where the level-2 counts will be");
__device__ __forceinline__ void level1_walk(const RankCtl* ctl, const RankSet& ranks, uint32_t* scan_tmp,
                                            uint32_t* s_prefix, uint32_t* s_rem, uint32_t* sums) {
  // thread t owns `per` bins ending at top = kLevel1Bins - 1 - per * t, largest keys first
  constexpr uint32_t per = kLevel1Bins / kRankBlock;
  static_assert(kBlockBins % per == 0, "a block begins with a thread's bins");
  const uint32_t top = kLevel1Bins - 1 - per * threadIdx.x;
  uint32_t h[per], mine = 0;
#pragma unroll
  for (uint32_t i = 0; i < per; ++i) {
    h[i] = ctl->top[top - i];
    mine += h[i];
  }
  uint32_t total;
  uint32_t above = block_excl_scan<kRankWaves>(mine, scan_tmp, &total);
  uint32_t* blocks = sums + kLevel1Bins + 1u;  // keys before every block, and all
  if (threadIdx.x * per % kBlockBins == 0) blocks[threadIdx.x * per / kBlockBins] = above;
#pragma unroll
  for (uint32_t i = 0; i < per; ++i) {
    sums[threadIdx.x * per + i] = above;
    above += h[i];
  }
  if (threadIdx.x == kRankBlock - 1u) sums[kLevel1Bins] = blocks[kWave] = above;
  __syncthreads();
  const uint32_t lane = lane_id();
  for (uint32_t j = wave_id(); j < ranks.n; j += kRankWaves) {
    const uint32_t target = ranks.rank[j];  // 1 .. d: inside some bin
    const uint32_t c = min((uint32_t)__popcll(__ballot(blocks[lane + 1u] < target)), kWave - 1u);
    const uint32_t* s = sums + c * kBlockBins + 2u * lane;
    const uint32_t k = min(c * kBlockBins + (uint32_t)__popcll(__ballot(s[1] < target)) + (uint32_t)__popcll(__ballot(s[2] < target)),
                           kLevel1Bins - 1u);
    if (lane == 0) {
      s_prefix[j] = kLevel1Bins - 1u - k;
      s_rem[j] = target - sums[k];
    }
  }
}

// WALK: the keys come from the lists of the guessed bins, and every workgroup does the level-1 walk for itself (a launch of
// its own for it takes 11 us), workgroup 0 of a client leaves its result, and whether a rank lies outside
// the guessed bins, where the later kernels look for them; a client whose guess missed has its level 2 counted by the
// collecting pass.
struct NoRanks {};  // (132 bytes of kernel arguments cost the small calls 0.3 us)
template <int LEVEL, bool LISTS, bool WALK>
__global__ __launch_bounds__(kRankBlock) void rank_pass_kernel(const float* const* __restrict__ updates,
                                                               RankCtl* __restrict__ ctls, uint32_t d, KeyLists kl,
                                                               std::conditional_t<WALK, RankSet, NoRanks> ranks) {
  __shared__ uint32_t hist[kRanksMax * kSubBins];
  __shared__ alignas(16) uint8_t first_cls[kLevel1Bins];
  __shared__ uint32_t cls_prefix[kRanksMax + 1];
  __shared__ uint32_t scan_tmp[kRankWaves], s_prefix[kRanksMax], s_rem[kRanksMax], s_n_cls, s_missed;  // WALK
  RankCtl* ctl = ctls + blockIdx.y;
  uint32_t n_cls;
  if constexpr (WALK) {
    if (threadIdx.x <= kRanksMax) cls_prefix[threadIdx.x] = 0xFFFFFFFFu;
    level1_walk(ctl, ranks, scan_tmp, s_prefix, s_rem, hist);
    __syncthreads();
    if (threadIdx.x < kWave) {
      const uint32_t bin = threadIdx.x < ranks.n ? s_prefix[threadIdx.x] : 0u;
      const bool outside = threadIdx.x < ranks.n && !((ctl->guess[bin >> 3] >> (bin & 7u)) & 1u);
      const uint32_t missed = __ballot(outside) ? 1u : 0u;
      uint32_t c;
      bool opens;
      const uint32_t n = write_classes(blockIdx.x == 0 ? ctl : nullptr, s_prefix, s_rem, ranks.n, &c, &opens);
      if (opens) cls_prefix[c] = bin;
      if (threadIdx.x == 0) {
        s_n_cls = n;
        s_missed = missed;
        if (blockIdx.x == 0) ctl->missed = missed;
      }
    }
    __syncthreads();
    if (s_missed) return;  // uniform
    n_cls = s_n_cls;
  } else {
    n_cls = ctl->n_cls;
    if (threadIdx.x <= kRanksMax) cls_prefix[threadIdx.x] = threadIdx.x < n_cls ? ctl->cls_prefix[threadIdx.x] : 0xFFFFFFFFu;
  }
  for (uint32_t i = threadIdx.x; i < n_cls * kSubBins; i += kRankBlock) hist[i] = 0;
  for (uint32_t i = threadIdx.x; i < kLevel1Bins / 4u; i += kRankBlock)
    reinterpret_cast<uint32_t*>(first_cls)[i] = 0xFFFFFFFFu;
  __syncthreads();
  if (threadIdx.x < n_cls) {
    const uint32_t c = threadIdx.x;
    const uint32_t bin = LEVEL == 2 ? cls_prefix[c] : cls_prefix[c] >> kSubBits;
    const uint32_t before = c == 0 ? 0xFFFFFFFFu : (LEVEL == 2 ? cls_prefix[c - 1] : cls_prefix[c - 1] >> kSubBits);
    if (bin != before) first_cls[bin] = (uint8_t)c;
  }
  __syncthreads();
  auto visit = [&](uint32_t key) {
    const uint32_t bin = key >> kLevel1Shift;
    uint32_t c = first_cls[bin];
    if (c == kNoClass) return;
    if (LEVEL == 2) {
      atomicAdd(&hist[c * kSubBins + ((key >> kSubBits) & (kSubBins - 1u))], 1u);
    } else {
      const uint32_t mine = key >> kSubBits;
      // the entry after the last class never starts with a level-1 bin, so the walk ends
      for (uint32_t p = cls_prefix[c]; (p >> kSubBits) == bin; p = cls_prefix[++c])
        if (p == mine) {
          atomicAdd(&hist[c * kSubBins + (key & (kSubBins - 1u))], 1u);
          break;
        }
    }
  };
  if (LISTS) list_keys(kl, visit); else stream_keys(updates[blockIdx.y], d, visit);
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < n_cls * kSubBins; i += kRankBlock) {
    const uint32_t h = hist[i];
    if (h) atomicAdd(&ctl->sub[i], h);
  }
}

// (The three-pass path; with room for the key lists the passes behind do this walk themselves.)
__global__ __launch_bounds__(kRankBlock) void rank_walk1_kernel(RankCtl* __restrict__ ctls, RankSet ranks) {
  __shared__ uint32_t scan_tmp[kRankWaves];
  __shared__ uint32_t s_prefix[kRanksMax], s_rem[kRanksMax];
  RankCtl* ctl = ctls + blockIdx.x;
  __shared__ uint32_t sums[kWalkSums];
  level1_walk(ctl, ranks, scan_tmp, s_prefix, s_rem, sums);
  __syncthreads();
  if (threadIdx.x < kWave) write_classes(ctl, s_prefix, s_rem, ranks.n);
}

// Ordinary least squares of ln(magnitude) on ln(rank) over the keys (in LDS) of the ranks: the logarithms
// side by side, the sums by one thread with the ranks in ascending order.  Whole workgroup.
__device__ __forceinline__ void fit_exponent(const uint32_t* s_keys, const RankSet& ranks, double* alpha_out) {
  __shared__ double s_x[kRanksMax], s_y[kRanksMax];
  if (threadIdx.x < ranks.n) {
    const double mag = (double)__uint_as_float(s_keys[threadIdx.x]);
    s_x[threadIdx.x] = log((double)ranks.rank[threadIdx.x]);
    s_y[threadIdx.x] = mag > 0.0 ? log(mag) : 0.0;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double sx = 0.0, sy = 0.0, sxx = 0.0, sxy = 0.0;
    uint32_t m = 0;
    for (uint32_t j = 0; j < ranks.n; ++j) {
      if (s_keys[j] == 0u) continue;  // a zero magnitude has no logarithm
      const double x = s_x[j], y = s_y[j];
      sx += x; sy += y; sxx += x * x; sxy += x * y; ++m;
    }
    *alpha_out = m < 2 ? -1.0 : ((double)m * sxy - sx * sy) / ((double)m * sxx - sx * sx);
  }
}

// A wavefront takes two classes: lane l holds the 8 digits ending at 511 - 8 l, and what is known of rank l.
// One workgroup per client, all latency: everything is asked for at once, before the number of classes is known, and a class goes
// through its own ranks only (all ranks' classes looked up in LDS for every class, the counts asked for class by class: level 2
// 7.8 us and level 3 9.6 for 32 clients, now 5.0 and 7.0).
template <int LEVEL>
__global__ __launch_bounds__(kRankBlock) void rank_walk_kernel(RankCtl* __restrict__ ctls, RankSet ranks,
                                                               uint32_t* __restrict__ keys_out,
                                                               double* __restrict__ alpha_out) {
  __shared__ uint32_t s_prefix[kRanksMax], s_rem[kRanksMax];
  RankCtl* ctl = ctls + blockIdx.x;
  constexpr uint32_t per = kSubBins / kWave, kTurns = kRanksMax / kRankWaves;
  typedef uint32_t __attribute__((ext_vector_type(4))) Words4;
  static_assert(per == 8u && sizeof(RankCtl) % 16u == 0 && offsetof(RankCtl, sub) % 16u == 0, "two 16-byte loads");
  const uint32_t lane = lane_id(), wave = wave_id(), top = kSubBins - 1 - per * lane, rank = min(lane, kRanksMax - 1u);
  Words4 counts[kTurns][2];
#pragma unroll
  for (uint32_t t = 0; t < kTurns; ++t) {
    const Words4* bins = reinterpret_cast<const Words4*>(ctl->sub + (wave + t * kRankWaves) * kSubBins + (top + 1u - per));
    counts[t][0] = bins[0];
    counts[t][1] = bins[1];
  }
  const uint32_t cls = ctl->cls[rank], old_rem = ctl->rem[rank], old_prefix = ctl->prefix[rank];
#pragma unroll
  for (uint32_t t = 0; t < kTurns; ++t) {
    const uint32_t c = wave + t * kRankWaves;
    uint64_t todo = __ballot(lane < ranks.n && cls == c);
    if (!todo) continue;  // uniform: no such class
    uint32_t h[per], mine = 0;
#pragma unroll
    for (uint32_t i = 0; i < per; ++i) {
      h[i] = counts[t][(per - 1u - i) / 4u][(per - 1u - i) % 4u];
      mine += h[i];
    }
    if (LEVEL == 2) {  // the next level counts into the same bins
      Words4* bins = reinterpret_cast<Words4*>(ctl->sub + c * kSubBins + (top + 1u - per));
      bins[0] = bins[1] = Words4{0u, 0u, 0u, 0u};
    }
    const uint32_t above = wave_incl_scan_u32(mine) - mine;
    while (todo) {
      const uint32_t j = (uint32_t)__builtin_ctzll(todo);
      const uint32_t target = (uint32_t)__builtin_amdgcn_readlane(old_rem, j), prefix = (uint32_t)__builtin_amdgcn_readlane(old_prefix, j);
      if (above < target && target <= above + mine) {  // one lane
        uint32_t acc = above;
#pragma unroll
        for (uint32_t i = 0; i < per; ++i) {
          if (acc < target && target <= acc + h[i]) {
            s_prefix[j] = (prefix << kSubBits) | (top - i);
            s_rem[j] = target - acc;
          }
          acc += h[i];
        }
      }
      todo &= todo - 1u;
    }
  }
  __syncthreads();
  if (LEVEL == 2) {
    if (threadIdx.x < kWave) write_classes(ctl, s_prefix, s_rem, ranks.n);
    return;
  }
  // level 3: s_prefix holds the keys
  if (keys_out && threadIdx.x < kRanksMax)
    keys_out[(size_t)blockIdx.x * kRanksMax + threadIdx.x] = threadIdx.x < ranks.n ? s_prefix[threadIdx.x] : 0u;
  fit_exponent(s_prefix, ranks, alpha_out + blockIdx.x);
}

// ------------------------------------------------------------------ two passes: collect, select
// The keys of the class bins, as the collecting pass leaves them: list (client, workgroup, wavefront) holds
// list_cnt[...] keys in no particular order.
constexpr uint32_t kCollectStage = 512;  // keys a wavefront stages in LDS; rows of 64 leave once 256 are there

//
// Every workgroup first does the level-1 walk for itself (the counts are in L2; a launch of its own for it costs
// more), workgroup 0 of a client also leaves the result where the later kernels look for it.  The keys it
// collects are counted on their next 9 bits as they pass (level 2, per class, 64 KB of LDS).  With its 104 KB
// of LDS one workgroup has a CU to itself, which suits a streaming pass (241 against 252 us with two).
// GUESSED: only the clients whose guess missed.
template <bool GUESSED>
__global__ __launch_bounds__(kRankBlock) void rank_collect_kernel(const float* const* __restrict__ updates,
                                                                  RankCtl* __restrict__ ctls, RankSet ranks,
                                                                  uint32_t d, uint32_t* __restrict__ lists,
                                                                  uint32_t* __restrict__ list_cnt, uint32_t wave_cap) {
  __shared__ alignas(16) uint8_t first_cls[kLevel1Bins];
  __shared__ uint32_t stage[kRankWaves][kCollectStage];
  __shared__ uint32_t s_fill[kRankWaves];  // keys a wavefront has staged
  __shared__ uint32_t level2[kRanksMax * kSubBins];
  __shared__ uint32_t scan_tmp[kRankWaves];
  __shared__ uint32_t s_prefix[kRanksMax], s_rem[kRanksMax];
  __shared__ uint32_t s_n_cls;
  RankCtl* ctl = ctls + blockIdx.y;
  if (GUESSED && !ctl->missed) return;  // uniform
  for (uint32_t i = threadIdx.x; i < kLevel1Bins / 4u; i += kRankBlock)
    reinterpret_cast<uint32_t*>(first_cls)[i] = 0xFFFFFFFFu;
  level1_walk(ctl, ranks, scan_tmp, s_prefix, s_rem, level2);
  __syncthreads();
  if (threadIdx.x < kWave) {
    uint32_t c;
    bool opens;
    const uint32_t n = write_classes(blockIdx.x == 0 ? ctl : nullptr, s_prefix, s_rem, ranks.n, &c, &opens);
    if (opens) first_cls[s_prefix[threadIdx.x]] = (uint8_t)c;  // level-1 classes: one per bin
    if (threadIdx.x == 0) s_n_cls = n;
  }
  __syncthreads();
  const uint32_t n_cls = s_n_cls;
  for (uint32_t i = threadIdx.x; i < n_cls * kSubBins; i += kRankBlock) level2[i] = 0;
  __syncthreads();
  const uint32_t lane = lane_id(), wave = wave_id();
  const size_t list = ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * kRankWaves + wave;
  uint32_t* __restrict__ out = lists + list * wave_cap;
  uint32_t* mine = stage[wave];
  uint32_t fill = 0, run = 0;  // staged keys as of the last look, keys already written (uniform over the wavefront)
  // LDS accesses of a wavefront complete in order; the fences keep the compiler from moving them.
  auto lds_fence = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
  if (lane == 0) s_fill[wave] = 0;
  lds_fence();
  // Class keys are few (a lane meets one in every sixteenth float4 or so): the lanes that hold some take
  // their places in the wavefront's stage with an LDS atomic; the order of the keys in a list is free.
  auto take = [&](const uint32_t* k, uint32_t n_keys, bool valid) {
    uint32_t hit = 0, cls[4];
    for (uint32_t c = 0; c < n_keys; ++c) {
      cls[c] = first_cls[k[c] >> kLevel1Shift];
      hit |= (cls[c] != kNoClass ? 1u : 0u) << c;
    }
    if (valid && hit) {
      uint32_t pos = atomicAdd(&s_fill[wave], (uint32_t)__popc(hit));
      for (uint32_t c = 0; c < n_keys; ++c)
        if ((hit >> c) & 1u) {
          mine[pos++] = k[c];
          atomicAdd(&level2[cls[c] * kSubBins + ((k[c] >> kSubBits) & (kSubBins - 1u))], 1u);
        }
    }
  };
  auto look = [&] {
    lds_fence();
    fill = __builtin_amdgcn_readfirstlane(s_fill[wave]);
  };
  auto flush = [&](bool all) {
    lds_fence();
    uint32_t g = 0;
    for (; g + kWave <= fill; g += kWave) out[run + g + lane] = mine[g + lane];
    const uint32_t left = fill - g;
    if (left) {
      const uint32_t k = lane < left ? mine[g + lane] : 0u;
      if (all) {
        if (lane < left) out[run + g + lane] = k;
        g += left;
      } else if (g) {  // the partial row moves to the front
        lds_fence();
        if (lane < left) mine[lane] = k;
      }
    }
    run += g;
    fill -= g;
    if (lane == 0) s_fill[wave] = fill;
    lds_fence();
  };
  const float* update = updates[blockIdx.y];
  const uint32_t n_quads = d / 4u;
  GlobalFloat4Ptr src = (GlobalFloat4Ptr)update;
  constexpr uint32_t kTileQuads = kRankBlock * kDeep;
  for (uint32_t q0 = blockIdx.x * kTileQuads; q0 < n_quads; q0 += gridDim.x * kTileQuads) {
    Float4V v[kDeep];
#pragma unroll
    for (uint32_t u = 0; u < kDeep; ++u) {
      const uint32_t q = q0 + u * kRankBlock + threadIdx.x;
      v[u] = __builtin_nontemporal_load(src + min(q, n_quads - 1u));
    }
#pragma unroll
    for (uint32_t u = 0; u < kDeep; ++u) {
      const uint32_t q = q0 + u * kRankBlock + threadIdx.x;
      uint32_t k[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) k[c] = __float_as_uint(v[u][c]) & 0x7FFFFFFFu;
      take(k, 4u, q < n_quads);
      look();
      if (fill >= kCollectStage - 4u * kWave) flush(false);  // room for the next four keys of every lane
    }
  }
  if (blockIdx.x == 0 && wave == 0) {  // the last d % 4 coordinates
    const bool valid = lane < d - n_quads * 4u;
    const uint32_t k = valid ? __float_as_uint(update[n_quads * 4u + lane]) & 0x7FFFFFFFu : 0u;
    take(&k, 1u, valid);
  }
  look();
  flush(true);
  if (lane == 0) list_cnt[list] = run;
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < n_cls * kSubBins; i += kRankBlock) {
    const uint32_t h = level2[i];
    if (h) atomicAdd(&ctl->sub[i], h);
  }
}

// ------------------------------------------------------------------ one pass: sample, guess, stream
constexpr uint32_t kPieceQuads = 16;       // a piece of the sample: 256 bytes
constexpr uint32_t kSamplePiecesMin = 4096, kSamplePiecesMax = 12288;  // by the length, see sample_pieces
constexpr uint32_t kSampleWgs = 16;        // workgroups per client

// Workgroup g takes pieces g, g + 16, ...: its counts are those of an evenly spread sample of its own.  The sum of the
// parts goes to `sub`, which the guess leaves cleared, the parts' counts of key >> 21 to parts, 16 a client and bin.
constexpr uint32_t kSampledPartShift = 21, kPartBins = 1u << (31u - kSampledPartShift), kPartStep = kLevel1Bins / kPartBins;
static_assert(kSamplePiecesMax / kSampleWgs * kPieceQuads * 4u < (1u << 16), "a part's counts and their sums fit 16 bits");
static_assert(kLevel1Bins <= kRanksMax * kSubBins, "the sample's counts fit where the second level's will stand");
// The more pieces, the nearer the margins (32 x 11.2 M: lists of 6 % of the keys instead of 8, of 9 % for vectors of rows
// instead of 17); an eighth of the vector is read at most.
constexpr uint32_t kSampleDeep = 4, kSampleTurn = kRankBlock * kSampleDeep;  // float4 a workgroup asks for together
uint32_t sample_pieces(uint32_t d) {
  const uint32_t eighth = d / (4u * kPieceQuads * 8u) / kSampleTurn * kSampleTurn;
  return std::min(kSamplePiecesMax, std::max(kSamplePiecesMin, eighth));
}
static_assert(kSampleWgs == kPieceQuads && kSamplePiecesMin % kSampleTurn == 0 && kSamplePiecesMax % kSampleTurn == 0, "whole turns");

__global__ __launch_bounds__(kRankBlock) void rank_sample_kernel(const float* const* __restrict__ updates, RankCtl* __restrict__ ctls,
                                                                 uint16_t* __restrict__ parts, uint32_t n_pieces, uint32_t sampled) {
  __shared__ uint32_t hist[kLevel1Bins];
  for (uint32_t i = threadIdx.x; i < kLevel1Bins; i += kRankBlock) hist[i] = 0;
  __syncthreads();
  GlobalFloat4Ptr src = (GlobalFloat4Ptr)updates[blockIdx.y];
  const uint32_t quads = sampled * kPieceQuads / kSampleWgs;
  for (uint32_t base = 0; base < quads; base += kSampleTurn) {
    Float4V v[kSampleDeep];
#pragma unroll
    for (uint32_t u = 0; u < kSampleDeep; ++u) {
      const uint32_t q = base + u * kRankBlock + threadIdx.x;
      const uint64_t piece = (uint64_t)(q / kPieceQuads * kSampleWgs + blockIdx.x) * n_pieces / sampled;  // evenly spread
      v[u] = src[piece * kPieceQuads + q % kPieceQuads];
    }
#pragma unroll
    for (uint32_t u = 0; u < kSampleDeep; ++u)
#pragma unroll
      for (int c = 0; c < 4; ++c) atomicAdd(&hist[(__float_as_uint(v[u][c]) & 0x7FFFFFFFu) >> kLevel1Shift], 1u);
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < kLevel1Bins; i += kRankBlock) {
    const uint32_t h = hist[i];
    if (h) atomicAdd(&ctls[blockIdx.y].sub[i], h);
  }
  static_assert(kPartBins == kRankBlock, "one bin of a part per thread");
  uint32_t sum = 0;
#pragma unroll
  for (uint32_t i = 0; i < kPartStep; ++i) sum += hist[threadIdx.x * kPartStep + i];
  parts[((size_t)blockIdx.y * kPartBins + threadIdx.x) * kSampleWgs + blockIdx.x] = (uint16_t)sum;
}

// A rank's place in the sample of n coordinates is binomial if they are drawn one by one: bins that hold a place within
// 4.5 standard deviations (and three more, for the ends) of the expected one are guessed.  They are drawn in pieces of
// 64 neighbours, though, and where neighbours are alike (a scale of its own per row, rows that are zero) a place
// strays up to eight times as far.  How far is measured: the variance of the sixteen parts' places over the
// binomial one, averaged over the bins of key >> 21 where that is not small.  (Binomial alone missed a rank in five of
// six vectors of rows of 64, and the call took 1.8 to 3 times as long; with the factor none of 66, the lists
// half as long again.)  Where the margins, beyond the bins of the expected places themselves, hold more than a seventh
// of the sample, the lists would cost more than the second pass they save: nothing is guessed.
// Wrong only costs time: the second pass.
// One workgroup per client, bound by the instructions of single wavefronts: nearly all keys lie in the bins of two of them, and
// a thread that compares its eight bins with every rank takes those 10 us.  A wavefront per rank that searches the running sums
// for the ends of its bins: 16.5 us -> 9.6 at 32 x 11.2 M, the call 396 -> 388.6.
__global__ __launch_bounds__(kRankBlock) void rank_guess_kernel(RankCtl* __restrict__ ctls, const uint16_t* __restrict__ parts,
                                                                RankSet ranks, uint32_t d, uint32_t sampled) {
  constexpr uint32_t per = kLevel1Bins / kRankBlock, kPairs = kSampleWgs / 2u;
  const float size = (float)(sampled * kPieceQuads * 4u);
  static_assert(per == 8u, "a byte of the bit set per thread");
  __shared__ uint32_t s_pair[kPairs][kRankWaves], scan_tmp[kRankWaves], s_extra[kRankWaves];
  __shared__ float s_factor[kRankWaves], s_bins[kRankWaves], s_place[kRanksMax], s_spread[kRanksMax], s_margin[kRanksMax];
  // keys in the bins before bin k and in the blocks of 128 bins before block c, largest keys first
  __shared__ alignas(16) uint32_t s_sum[kLevel1Bins + 1];
  __shared__ uint32_t s_block[kWave + 1], s_bits[kLevel1Bins / 32u], s_expected[kLevel1Bins / 32u];
  constexpr uint32_t kMarkWords = kLevel1Bins / 32u;
  static_assert(kBlockBins % per == 0 && 2u * kMarkWords <= kRankBlock, "a block begins with a thread's bins");
  RankCtl* ctl = ctls + blockIdx.x;
  const uint32_t lane = lane_id(), wave = wave_id();
  const uint32_t first = kLevel1Bins - per * (threadIdx.x + 1u);  // thread 0 owns the largest keys
  uint32_t h[per], mine = 0;
#pragma unroll
  for (uint32_t i = 0; i < per; ++i) h[i] = ctl->sub[first + i];
  const uint4* __restrict__ part = reinterpret_cast<const uint4*>(parts + ((size_t)blockIdx.x * kPartBins + (kPartBins - 1u - threadIdx.x)) * kSampleWgs);
  const uint4 p0 = part[0], p1 = part[1];
  if (threadIdx.x < ranks.n) {
    const double p = (double)ranks.rank[threadIdx.x] / (double)d;
    s_place[threadIdx.x] = (float)((double)size * p);
    s_spread[threadIdx.x] = (float)((double)size * p * (1.0 - p));
  }
#pragma unroll
  for (uint32_t i = 0; i < per; ++i) mine += h[i];
  uint32_t total;
  const uint32_t above = block_excl_scan<kRankWaves>(mine, scan_tmp, &total);
  if (threadIdx.x < kMarkWords)
    s_bits[threadIdx.x] = 0;
  else if (threadIdx.x < 2u * kMarkWords)
    s_expected[threadIdx.x - kMarkWords] = 0;
  {
    uint32_t sum = above;
    if (threadIdx.x * per % kBlockBins == 0) s_block[threadIdx.x * per / kBlockBins] = sum;
#pragma unroll
    for (uint32_t i = 0; i < per; ++i) {
      s_sum[threadIdx.x * per + i] = sum;
      sum += h[per - 1u - i];
    }
    if (threadIdx.x == kRankBlock - 1u) s_sum[kLevel1Bins] = s_block[kWave] = sum;
  }
  // the parts' places at the lower end of the thread's bin, two to a word
  uint32_t at[kPairs] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
#pragma unroll
  for (uint32_t j = 0; j < kPairs; ++j) {
    at[j] = wave_incl_scan_u32(at[j]);  // no carry between the halves
    if (lane == kWave - 1u) s_pair[j][wave] = at[j];
  }
  __syncthreads();
  if (threadIdx.x < kPairs * kRankWaves) {  // sixteen lanes per pair: the sums of the wavefronts before
    uint32_t* word = &s_pair[0][0] + threadIdx.x;
    const uint32_t own = *word;
    uint32_t sum = own;
#pragma unroll
    for (int o = 1; o < (int)kRankWaves; o <<= 1) {
      const uint32_t t = (uint32_t)__shfl_up((int)sum, o, (int)kRankWaves);
      if (threadIdx.x % kRankWaves >= (uint32_t)o) sum += t;
    }
    *word = sum - own;
  }
  __syncthreads();
  uint32_t place = 0;
#pragma unroll
  for (uint32_t j = 0; j < kPairs; ++j) {
    at[j] += s_pair[j][wave];
    place += (at[j] & 0xFFFFu) + (at[j] >> 16);
  }
  const float mean = (float)place * (1.0f / kSampleWgs), binomial = (float)place * (1.0f - (float)place / size);
  float squares = 0.0f;
#pragma unroll
  for (uint32_t j = 0; j < kPairs; ++j) {
    const float a = (float)(at[j] & 0xFFFFu) - mean, b = (float)(at[j] >> 16) - mean;
    squares += a * a + b * b;
  }
  const bool counts = binomial > 1024.0f;
  float factor = counts ? fminf(fmaxf(squares * ((float)kSampleWgs / (kSampleWgs - 1.0f)) / binomial, 1.0f), (float)(4u * kPieceQuads)) : 0.0f;
  float bins = counts ? 1.0f : 0.0f;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    factor += __shfl_xor(factor, o, kWave);
    bins += __shfl_xor(bins, o, kWave);
  }
  if (lane == 0) {
    s_factor[wave] = factor;
    s_bins[wave] = bins;
  }
  __syncthreads();
  factor = bins = 0.0f;
#pragma unroll
  for (uint32_t w = 0; w < kRankWaves; ++w) {
    factor += s_factor[w];
    bins += s_bins[w];
  }
  if (threadIdx.x < ranks.n) {
    factor = bins > 0.0f ? factor / bins : 1.0f;
    s_margin[threadIdx.x] = 4.5f * sqrtf(factor * s_spread[threadIdx.x]) + 3.0f * factor;
  }
  __syncthreads();
  // Bin k (0: the largest keys) holds the sample's places s_sum[k] .. s_sum[k + 1] + 1, the borders of both sides too: an empty
  // bin lies between two.  The bins that hold one of lo .. hi are neighbours: a wavefront per rank finds their ends.
  auto before = [&](float lo) {  // bins that end before place lo
    const uint32_t c = min((uint32_t)__popcll(__ballot((float)(s_block[lane + 1u] + 1u) < lo)), kWave - 1u);
    const uint32_t* s = s_sum + c * kBlockBins + 2u * lane;
    return c * kBlockBins + (uint32_t)__popcll(__ballot((float)(s[1] + 1u) < lo)) + (uint32_t)__popcll(__ballot((float)(s[2] + 1u) < lo));
  };
  auto up_to = [&](float hi) {  // bins that begin at place hi or before
    const uint32_t c = min((uint32_t)__popcll(__ballot((float)s_block[lane + 1u] <= hi)), kWave - 1u);
    const uint32_t* s = s_sum + c * kBlockBins + 2u * lane;
    return c * kBlockBins + (uint32_t)__popcll(__ballot((float)s[0] <= hi)) + (uint32_t)__popcll(__ballot((float)s[1] <= hi));
  };
  auto mark = [&](uint32_t* marks, uint32_t begin, uint32_t end) {
    for (uint32_t w = begin / 32u + lane; w * 32u < end; w += kWave) {
      const uint32_t from = max(begin, w * 32u) & 31u, to = min(end - w * 32u, 32u);
      if (from < to) atomicOr(&marks[w], (~0u << from) & (~0u >> (32u - to)));
    }
  };
  for (uint32_t j = wave; j < ranks.n; j += kRankWaves) {
    const float middle = s_place[j], margin = s_margin[j];
    const uint32_t b0 = before(middle - margin), b1 = up_to(middle + margin), e0 = before(middle), e1 = up_to(middle);
    if (b0 < b1) mark(s_bits, b0, b1);
    if (e0 < e1) mark(s_expected, e0, e1);
  }
  __syncthreads();
  // the thread's byte of the bit sets, its smallest bin in the lowest bit
  const uint32_t turn = 8u * (threadIdx.x & 3u);
  const uint32_t bits = __brev(s_bits[threadIdx.x >> 2] >> turn << 24), expected = __brev(s_expected[threadIdx.x >> 2] >> turn << 24);
  uint32_t extra = 0;
#pragma unroll
  for (uint32_t i = 0; i < per; ++i)
    if (((bits & ~expected) >> i) & 1u) extra += h[i];
  extra = wave_sum_u32(extra);
  if (lane == 0) s_extra[wave] = extra;
  __syncthreads();
  extra = 0;
#pragma unroll
  for (uint32_t w = 0; w < kRankWaves; ++w) extra += s_extra[w];
  ctl->guess[first / 8u] = (uint8_t)((float)extra > size / 7.0f ? 0u : bits);
#pragma unroll
  for (uint32_t i = 0; i < per; ++i) ctl->sub[first + i] = 0;  // last: a barrier waits for stores
}

// Counts all keys (level 1) and sets the keys of the guessed bins aside, in rows of 64 through LDS.  Bound by HBM:
// the vectors once, and the writes mixed into them (6 % of the keys).  32 vectors of 11.2 M: 290 us where the counting
// pass and the collecting pass took 223 + 272.
__global__ __launch_bounds__(kRankBlock) void rank_stream_kernel(const float* const* __restrict__ updates,
                                                                 RankCtl* __restrict__ ctls, uint32_t d,
                                                                 uint32_t* __restrict__ lists,
                                                                 uint32_t* __restrict__ list_cnt, uint32_t wave_cap,
                                                                 uint32_t* status) {
  __shared__ uint32_t hist[kLevel1Bins];
  __shared__ uint32_t guess[kLevel1Bins / 32u];
  __shared__ uint32_t stage[kRankWaves][kCollectStage];
  RankCtl* ctl = ctls + blockIdx.y;
  for (uint32_t i = threadIdx.x; i < kLevel1Bins; i += kRankBlock) hist[i] = 0;
  if (threadIdx.x < kLevel1Bins / 32u) guess[threadIdx.x] = reinterpret_cast<const uint32_t*>(ctl->guess)[threadIdx.x];
  __syncthreads();
  const uint32_t lane = lane_id(), wave = wave_id();
  const size_t list = ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * kRankWaves + wave;
  uint32_t* __restrict__ out = lists + list * wave_cap;
  uint32_t* mine = stage[wave];
  uint32_t fill = 0, run = 0;  // staged keys, keys already written (uniform over the wavefront)
  bool nonfinite = false;
  // LDS accesses of a wavefront complete in order; the fences keep the compiler from moving them.
  auto lds_fence = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
  auto flush = [&](bool all) {
    lds_fence();
    uint32_t g = 0;
    for (; g + kWave <= fill; g += kWave) out[run + g + lane] = mine[g + lane];
    const uint32_t left = fill - g;
    if (left) {
      const uint32_t k = lane < left ? mine[g + lane] : 0u;
      if (all) {
        if (lane < left) out[run + g + lane] = k;
        g += left;
      } else if (g) {  // the partial row moves to the front
        lds_fence();
        if (lane < left) mine[lane] = k;
      }
    }
    run += g;
    fill -= g;
    lds_fence();
  };
  auto take = [&](uint32_t key, bool valid) {
    const uint32_t bin = key >> kLevel1Shift;
    if (valid) atomicAdd(&hist[bin], 1u);
    nonfinite |= valid && key >= 0x7F800000u;
    const bool keep = valid && ((guess[bin >> 5] >> (bin & 31u)) & 1u);
    const uint64_t m = __ballot(keep);
    if (keep) mine[fill + lanes_below(m)] = key;
    fill += (uint32_t)__popcll(m);
  };
  const float* update = updates[blockIdx.y];
  const uint32_t n_quads = d / 4u;
  GlobalFloat4Ptr src = (GlobalFloat4Ptr)update;
  constexpr uint32_t kTileQuads = kRankBlock * kDeep;
  for (uint32_t q0 = blockIdx.x * kTileQuads; q0 < n_quads; q0 += gridDim.x * kTileQuads) {
    Float4V v[kDeep];
#pragma unroll
    for (uint32_t u = 0; u < kDeep; ++u) {
      const uint32_t q = q0 + u * kRankBlock + threadIdx.x;
      v[u] = __builtin_nontemporal_load(src + min(q, n_quads - 1u));
    }
#pragma unroll
    for (uint32_t u = 0; u < kDeep; ++u) {
      const bool valid = q0 + u * kRankBlock + threadIdx.x < n_quads;
#pragma unroll
      for (int c = 0; c < 4; ++c) take(__float_as_uint(v[u][c]) & 0x7FFFFFFFu, valid);
      if (fill > kCollectStage - 4u * kWave) flush(false);  // room for the next four keys of every lane
    }
  }
  if (blockIdx.x == 0 && wave == 0) {  // the last d % 4 coordinates
    const bool valid = lane < d - n_quads * 4u;
    take(valid ? __float_as_uint(update[n_quads * 4u + lane]) & 0x7FFFFFFFu : 0u, valid);
  }
  flush(true);
  if (lane == 0) list_cnt[list] = run;
  const int any_nonfinite = __syncthreads_or((int)nonfinite);
  if (any_nonfinite && threadIdx.x == 0) atomicOr(status, CVLC_DEV_NONFINITE);
  for (uint32_t i = threadIdx.x; i < kLevel1Bins; i += kRankBlock) {
    const uint32_t h = hist[i];
    if (h) atomicAdd(&ctl->top[i], h);
  }
}

// ------------------------------------------------------------------ short vectors: one launch
// A workgroup per client finds the keys at all ranks together (cvlc_select.h) and fits.  The pointers come as kernel arguments.
// The status word is written by the one workgroup of a single client; several add to what a launch before has cleared.
// us in six launches and in one or two: 1 x 2000 25.9 and 11.7, 1 x 20 000 30.5 and 15.6, 1 x 65 536 33.4 and 25.5, 32 x 65 536 37.7
// and 27.7, 100 x 65 536 54.9 and 26.7, 600 x 65 536 139 and 87, 2000 x 65 536 359 and 281; 65 536 of one magnitude 80.8 and 40.4, of five
// 61.6 and 49.3, bfloat16 33.6 and 26.1, nearly all zeros 75 and 36, sorted ones 46 and 36 (with both signs 44 and 41).
__global__ __launch_bounds__(kShortBlock) void rank_short_kernel(PtrChunk c, RankSet ranks, uint32_t d, uint32_t* __restrict__ keys_out,
                                                                 double* __restrict__ alpha_out, uint32_t* status, uint32_t single) {
  __shared__ FitSelect S;
  __shared__ uint32_t s_keys[kRanksMax];
  const uint32_t client = c.first + blockIdx.x, tid = threadIdx.x;
  const float* update = c.ptr[blockIdx.x];
  clear_short(S);
  __syncthreads();
  if (tid < ranks.n) S.rank[tid] = ranks.rank[tid];
  if (tid == 0) {
    S.n_ranks = ranks.n;
    S.extra = 0;
  }
  count_top(S, update, d);
  constexpr uint32_t kNonfinite = 0x7F800000u >> kTopShift;  // the first bin of Inf and NaN; the first wavefront looks at all of them
  static_assert(kTopBins - kNonfinite <= kWave && kRanksMax >= 17u && kRanksMax <= kShortRanks, "a bin per lane; all ranks of a short vector");
  const uint64_t flagged = __ballot(tid < kTopBins - kNonfinite && S.top[top_at<FitSelect>(kNonfinite + min(tid, kTopBins - kNonfinite - 1u))] != 0u);
  if (tid == 0) {
    if (single) *status = flagged ? CVLC_DEV_NONFINITE : 0u;
    else if (flagged) atomicOr(status, CVLC_DEV_NONFINITE);
  }
  locate_short(S);
  select_short(S, update, d);
  if (tid < kRanksMax) {
    s_keys[tid] = tid < ranks.n ? S.prefix[tid] : 0u;
    if (keys_out) keys_out[(size_t)client * kRanksMax + tid] = s_keys[tid];
  }
  __syncthreads();
  fit_exponent(s_keys, ranks, alpha_out + client);
}

uint32_t cu_count() {
  static int cus = 0;
  if (cus == 0) {
    int dev = 0, found = 0;
    cus = 256;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&found, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && found > 0)
      cus = found;
  }
  return (uint32_t)cus;
}

uint32_t tiles_of(uint32_t d) { return std::max(1u, (d / 4u + kRankBlock * kDeep - 1) / (kRankBlock * kDeep)); }

// Workgroups per client in a streaming pass: per_cu 1024-thread workgroups on every CU, never more than
// there are tiles.
uint32_t pass_blocks_per_client(uint32_t d, uint32_t n, uint32_t per_cu) {
  return std::max(1u, std::min((cu_count() * per_cu + n - 1) / n, tiles_of(d)));
}

// Keys that a wavefront reads of a client whose tiles are dealt round `blocks` workgroups: whole tiles, and the last d % 4.
uint32_t wave_cap_for(uint32_t d, uint32_t blocks) { return (tiles_of(d) + blocks - 1) / blocks * (kDeep * kWave * 4u) + kWave; }

// ... in the pass that writes the lists.  One pass: two for every CU.  Two passes: of the collecting one a CU holds one at a
// time, so as many as are held at once, that the prologue and the counters added up at the end (10 us of a small call) are paid
// once; twice as many where a client's whole number of them would leave more than an eighth of the CUs idle.  (Two for every CU,
// rounded up: 1 x 11.2 M 72 us instead of 59, 8 x 1.2 M 71 and 57, 8 x 11.2 M 181 and 164; one, rounded up: 12 x 9.6 M 256
// instead of 239, the last eight of 264 alone.)  Where few tiles a workgroup make such lists need more room than two for every CU
// do, it is those.
uint32_t list_blocks_per_client(uint32_t d, uint32_t n) {
  const uint32_t cus = cu_count(), twice = pass_blocks_per_client(d, n, 2u), once = cus / n;
  if (one_pass_for(n, d)) return twice;
  const uint32_t held = std::max(1u, std::min(once * n >= cus - cus / 8u ? once : 2u * cus / n, tiles_of(d)));
  return (uint64_t)held * wave_cap_for(d, held) <= (uint64_t)twice * wave_cap_for(d, twice) ? held : twice;
}

}  // namespace
}  // namespace cvlc

extern "C" {

uint32_t cvlc_fit_ranks(uint32_t d, uint32_t* ranks_out) {
  if (d == 0) return 0;
  uint32_t n = 0;
  for (uint64_t l = 1; l < d; l *= 2) {
    if (ranks_out) ranks_out[n] = (uint32_t)l;
    ++n;
  }
  if (ranks_out) ranks_out[n] = d;
  return n + 1;
}

size_t cvlc_fit_workspace_bytes(uint32_t n_clients) { return cvlc::rank_layout(n_clients, 0).total; }

size_t cvlc_fit_workspace_bytes_for(uint32_t n_clients, uint32_t d) {
  if (n_clients == 0 || d == 0 || d > 0x7FFFFFFFu) return 0;
  return cvlc::rank_layout(n_clients, d).total;
}

int cvlc_fit_alpha(uint32_t n, const float* const* d_updates, uint32_t d, double* d_alpha_out, uint32_t* d_keys_out,
                   void* d_workspace, size_t ws_bytes, void* hip_stream) {
  using namespace cvlc;
  if (n == 0 || !d_updates || !d_alpha_out || !d_workspace) return CVLC_ERR_ARG;
  if (d == 0 || d > 0x7FFFFFFFu || n > 65535u) return CVLC_ERR_ARG;
  if (reinterpret_cast<uintptr_t>(d_workspace) % 256u) return CVLC_ERR_ARG;
  for (uint32_t i = 0; i < n; ++i)
    if (!d_updates[i] || reinterpret_cast<uintptr_t>(d_updates[i]) % 16u) return CVLC_ERR_ARG;
  RankLayout L = rank_layout(n, d);  // with room for the collected keys: two passes
  if (ws_bytes < L.total) L = rank_layout(n, 0);
  if (ws_bytes < L.total) return CVLC_ERR_CAPACITY;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  char* base = static_cast<char*>(d_workspace);
  uint32_t* status = reinterpret_cast<uint32_t*>(base + L.status);
  RankCtl* ctls = reinterpret_cast<RankCtl*>(base + L.ctl);
  const float** ptrs = reinterpret_cast<const float**>(base + L.ptrs);
  RankSet ranks;
  for (uint32_t j = 0; j < kRanksMax; ++j) ranks.rank[j] = 0;
  ranks.n = cvlc_fit_ranks(d, ranks.rank);

  StageScope scope(CVLC_STAGE_FIT_ALPHA, stream);
  if (d <= kShortMax) {
    PtrChunk chunk;
    if (n > 1u) {
      chunk.first = chunk.count = 0;
      for (uint32_t i = 0; i < kPtrChunk; ++i) chunk.ptr[i] = nullptr;
      hipLaunchKernelGGL(rank_init_kernel, dim3(1), dim3(256), 0, stream, ptrs, chunk, reinterpret_cast<uint4*>(base), (size_t)1);
    }
    for (uint32_t first = 0; first < n; first += kPtrChunk) {
      chunk.first = first;
      chunk.count = std::min(n - first, kPtrChunk);
      for (uint32_t i = 0; i < kPtrChunk; ++i) chunk.ptr[i] = i < chunk.count ? d_updates[first + i] : nullptr;
      hipLaunchKernelGGL(rank_short_kernel, dim3(chunk.count), dim3(kShortBlock), 0, stream, chunk, ranks, d, d_keys_out, d_alpha_out, status,
                         n == 1u ? 1u : 0u);
    }
    return hip_check(hipGetLastError());
  }
  {
    PtrChunk chunk;
    for (uint32_t first = 0; first < n; first += kPtrChunk) {
      chunk.first = first;
      chunk.count = n - first < kPtrChunk ? n - first : kPtrChunk;
      for (uint32_t i = 0; i < kPtrChunk; ++i) chunk.ptr[i] = i < chunk.count ? d_updates[first + i] : nullptr;
      const size_t zero_n16 = first == 0 ? L.zero_bytes / 16u : 0u;
      size_t blocks = (zero_n16 + 2047u) / 2048u;  // eight pieces per thread, within 1..1024 workgroups
      blocks = blocks < 1 ? 1 : (blocks > 1024 ? 1024 : blocks);
      hipLaunchKernelGGL(rank_init_kernel, dim3((uint32_t)blocks), dim3(256), 0, stream, ptrs, chunk,
                         reinterpret_cast<uint4*>(base), zero_n16);
    }
  }
  const dim3 pass_grid(pass_blocks_per_client(d, n, 2u), n);
  KeyLists kl = {nullptr, nullptr, 0u, 0u};
  const bool one_pass = L.wave_cap && one_pass_for(n, d);
  if (one_pass) {
    // the parts' counts lie where the lists will: 32 KB a client of at least 4 MB
    uint16_t* parts = reinterpret_cast<uint16_t*>(base + L.lists);
    const uint32_t sampled = sample_pieces(d);
    hipLaunchKernelGGL(rank_sample_kernel, dim3(kSampleWgs, n), dim3(kRankBlock), 0, stream, ptrs, ctls, parts, d / (4u * kPieceQuads), sampled);
    hipLaunchKernelGGL(rank_guess_kernel, dim3(n), dim3(kRankBlock), 0, stream, ctls, parts, ranks, d, sampled);
  } else {
    hipLaunchKernelGGL(rank_hist1_kernel, pass_grid, dim3(kRankBlock), 0, stream, ptrs, ctls, d, status);
  }
  if (L.wave_cap) {  // two passes: the keys of the class bins are set aside, levels 2 and 3 count among those
    uint32_t* lists = reinterpret_cast<uint32_t*>(base + L.lists);
    uint32_t* list_cnt = reinterpret_cast<uint32_t*>(base + L.list_cnt);
    kl.lists = lists;
    kl.list_cnt = list_cnt;
    kl.per_client = L.blocks * kRankWaves;
    kl.wave_cap = L.wave_cap;
    // a few workgroups per client, whose cost is clearing and adding up the counters, and less so reading the keys; one
    // for every CU where 16 leave most CUs idle (16 and one for every CU: 1 x 11.2 M 99 -> 72 us, 4 x 11.2 M
    // 119 -> 112, 8 x 11.2 M 184 -> 181; 12 x 11.2 M 221 with 16, 225 with 32)
    const dim3 list_grid(std::min(L.blocks, n <= 8u ? std::max(16u, cu_count() / n) : 16u), n);
    if (one_pass) {
      hipLaunchKernelGGL(rank_stream_kernel, dim3(L.blocks, n), dim3(kRankBlock), 0, stream, ptrs, ctls, d, lists, list_cnt,
                         L.wave_cap, status);
      hipLaunchKernelGGL((rank_pass_kernel<2, true, true>), list_grid, dim3(kRankBlock), 0, stream, ptrs, ctls, d, kl, ranks);
    }
    auto collect = one_pass ? rank_collect_kernel<true> : rank_collect_kernel<false>;
    hipLaunchKernelGGL(collect, dim3(L.blocks, n), dim3(kRankBlock), 0, stream, ptrs, ctls, ranks, d, lists, list_cnt, L.wave_cap);
    hipLaunchKernelGGL(rank_walk_kernel<2>, dim3(n), dim3(kRankBlock), 0, stream, ctls, ranks, (uint32_t*)nullptr,
                       (double*)nullptr);
    hipLaunchKernelGGL((rank_pass_kernel<3, true, false>), list_grid, dim3(kRankBlock), 0, stream, ptrs, ctls, d, kl, NoRanks{});
    hipLaunchKernelGGL(rank_walk_kernel<3>, dim3(n), dim3(kRankBlock), 0, stream, ctls, ranks, d_keys_out, d_alpha_out);
    return hip_check(hipGetLastError());
  }
  hipLaunchKernelGGL(rank_walk1_kernel, dim3(n), dim3(kRankBlock), 0, stream, ctls, ranks);
  hipLaunchKernelGGL((rank_pass_kernel<2, false, false>), pass_grid, dim3(kRankBlock), 0, stream, ptrs, ctls, d, kl, NoRanks{});
  hipLaunchKernelGGL(rank_walk_kernel<2>, dim3(n), dim3(kRankBlock), 0, stream, ctls, ranks, (uint32_t*)nullptr,
                     (double*)nullptr);
  hipLaunchKernelGGL((rank_pass_kernel<3, false, false>), pass_grid, dim3(kRankBlock), 0, stream, ptrs, ctls, d, kl, NoRanks{});
  hipLaunchKernelGGL(rank_walk_kernel<3>, dim3(n), dim3(kRankBlock), 0, stream, ctls, ranks, d_keys_out, d_alpha_out);
  return hip_check(hipGetLastError());
}

}  // extern "C"
