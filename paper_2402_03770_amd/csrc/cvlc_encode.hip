// Encoder of libcvlc for gfx950: one client's update vector -> one
// variable-length stream (Sec. IV-B sparsification + quantisation, the final
// loop of Algorithm 1, packet format of Sec. IV-D).
//
// The paper ranks all d updates; here the ranking is never materialised.  The
// kernels find, for every group boundary Z_r, the exact Z_r-th largest
// magnitude (radix-histogram selection) and classify coordinates against those
// thresholds, which yields the same groups as a full sort with ties broken by
// position.  Launch chain per batch of clients (no kernel waits on another
// workgroup and none needs a memory fence; every dependency is a kernel
// boundary):
// (short vectors, up to 65 536 coordinates: short_select, count and emit only, unless they
// are very many; see short_pays)
//   upload        per-client parameters as kernel arguments; clears the
//                 call's control blocks
//   sample_hist   strided sample of |U| -> histogram of the top 13 key bits
//   sample_walk   conservative candidate threshold tau_lo from that histogram,
//                 and the selection bins: the range of keys above tau_lo cut
//                 into pieces of about a thousandth of the candidates each
//   filter        the one full pass over U.  Every wavefront owns regions of
//                 1024 to 8192 consecutive coordinates and writes the coordinates with
//                 key >= tau_lo to the front of the region's slot, in position
//                 order; it also counts the selection bins of what it keeps
//                 and sums the squares of what it drops
//   scan_l1       prefix over the region counts, list of the non-empty runs;
//                 selection bins of the boundaries (for a client whose sample
//                 misjudged, every coordinate becomes a candidate here)
//   gather        copies the runs into one dense, position-ordered candidate
//                 list, spans of 512 candidates per wavefront, and sets the
//                 members of the boundaries' bins aside
//   select        finds every boundary's element among the members of its bin (in
//                 the dense list where equal magnitudes make that a large part of
//                 it): its key, and its number in the dense list, which cuts a
//                 class of equal magnitudes
//   count         per span: group of every candidate and its number among the
//                 span's members of that group (left for emit, 16 bits per
//                 candidate), per-group count, min/max/sum of squares; for the
//                 QSGD quantiser also every group's exact sum of squares in
//                 integer limbs
//   layout        prefix of the per-span counts, headers (QSGD: the group norms
//                 from the exact sums), statistics; batches that keep much only, in
//                 others emit does that for itself
//   emit          per chunk of 8 spans: record number from prefix and span
//                 number, stochastic rounding (Philox4x32-10) and bit packing;
//                 on request the error energy of every group
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

#include "cvlc_common.h"
#include "cvlc_select.h"

namespace cvlc {
namespace {

constexpr uint32_t kWideBlock = 1024;
constexpr uint32_t kWideWaves = kWideBlock / kWave;
constexpr uint32_t kGatherBlock = 1024;  // threads of a gather workgroup
constexpr uint32_t kGatherWaves = kGatherBlock / kWave;
constexpr uint32_t kGatherResident = 512;   // gather workgroups the device holds
constexpr uint32_t kGatherBlocksMax = 64;   // ... and of one client's

constexpr uint32_t kHistCopiesMax = 8;

// ------------------------------------------------------------------ workspace layout
// Per-client, per-group constants of the last stages, written by the layout kernel.
struct GroupInfo {
  uint32_t payload[32];  // first stream word of the group's records
  uint32_t P[32], W[32], y[32];
  float m[32], inv[32];  // smallest value and reciprocal centroid spacing
  float step[32];        // centroid spacing, as the decoder derives it from the header
};

struct EncodeLayout {
  size_t status, ctl, params, region_cnt, region_sumsq, cand_idx, cand_val, dense_idx, dense_val, nz_off, nz_run, span_first, span_cnt, group_info,
      hist_bins, members, seg_cnt, norm_limbs, total;
  size_t zero_bytes;        // [status, params) is cleared at the start of a call
  uint32_t region_shift, n_regions, max_spans;
  uint32_t dense_cap;       // candidates the dense list of a client has room for
  uint32_t gather_blocks;   // workgroups per client in the gather
  uint32_t member_pool;     // entries of a member list
  uint32_t hist_copies;     // of a client's counts per selection bin
};

size_t align256(size_t v) { return (v + 255u) & ~(size_t)255u; }

// Workgroups per client in the filter pass: all of them resident at once
// (`resident` workgroups fit the device), every wavefront the same number of regions.
constexpr uint32_t kFilterBlocksCap = 2048;  // 8 workgroups on each of 256 CUs
uint32_t filter_blocks_per_client(uint32_t n_regions, uint32_t n, uint32_t resident) {
  const uint32_t max_blocks = resident / n > 0 ? resident / n : 1u;
  const uint32_t max_waves = max_blocks * kWavesPerBlock;
  const uint32_t rounds = (n_regions + max_waves - 1) / max_waves;
  const uint32_t waves = (n_regions + rounds - 1) / rounds;
  return (waves + kWavesPerBlock - 1) / kWavesPerBlock;
}

// Regions of 1 << region_shift coordinates.  A batch of several regions per resident wavefront takes the longest
// ones (long runs for the gather, few entries for the region scan).  A smaller batch leaves wavefronts without
// work, and the few that have some go through the eight sub-tiles of a long region one after the other, 2.5 us
// each: it takes the shortest regions, down to one sub-tile, that still give no wavefront a second one (32
// wavefronts fit a CU; 24 are counted on) and the region scan no fourth round.
// filter: 20.6 -> 5.8 us for one client of 65 536 coordinates, 20.6 -> 14.4 us for 8 of 1.2 M.  One client of
// 11.2 M: filter 27.8 -> 20.6 us with regions of 4096 (scan_l1 and the gather 1.5 and 1.2 us more); with regions of
// 2048 scan_l1 takes 13.1 us and more is lost than won.
uint32_t regions_of(uint32_t d, uint32_t shift) { return (uint32_t)(((uint64_t)d + (1u << shift) - 1u) >> shift); }

// Regions a client of n may have while they are shorter than the longest.
uint32_t short_regions_max(uint32_t n) {
  constexpr uint32_t kWavesCounted = 256u * 24u, kScanRounds = 3u * kWideBlock;
  return std::min(kScanRounds, kWavesCounted / n);
}

uint32_t region_shift_for(uint32_t d, uint32_t n) {
  uint32_t shift = kRegionShiftMax;
  while (shift > kRegionShiftMin && regions_of(d, shift - 1u) <= short_regions_max(n)) --shift;
  return shift;
}

// The most regions that a vector of up to d coordinates has.  The number itself falls by half wherever the length of
// a region doubles; the workspace is sized by this one, so that a workspace for one d holds every smaller one too.
uint32_t region_room_for(uint32_t d, uint32_t n) {
  return std::max(regions_of(d, kRegionShiftMax), std::min(regions_of(d, kRegionShiftMin), short_regions_max(n)));
}

// `cap`: candidates (coordinates at or above the sampled threshold) a client may have; the filter's own
// output is laid out by region and stays d long, everything behind it is as long as the candidates.
EncodeLayout encode_layout(uint32_t d, uint32_t n, uint32_t cap) {
  EncodeLayout L;
  L.region_shift = region_shift_for(d, n);
  L.n_regions = regions_of(d, L.region_shift);
  const uint32_t region_room = region_room_for(d, n);
  L.dense_cap = cap < d ? cap : d;
  L.max_spans = (uint32_t)(((uint64_t)L.dense_cap + kSpan - 1) / kSpan);
  {
    uint32_t b = (kGatherResident + n - 1) / n;
    L.gather_blocks = b < 2 ? 2u : (b > kGatherBlocksMax ? kGatherBlocksMax : b);
  }
  size_t off = 0;
  L.status = off; off = align256(off + 256);
  L.ctl = off; off = align256(off + (size_t)n * sizeof(ClientCtl));
  L.norm_limbs = off; off = align256(off + (size_t)n * 32 * kNormLimbs * sizeof(uint64_t));
  // The filter's workgroups add their counts to the client's by atomics, which queue up at each cache line: with few
  // clients, hundreds of workgroups on the same lines, so such a client has several copies, one for about 32 workgroups
  // (one client of 11.2 M: filter 30.6 -> 15.6 us; 8 of them: no difference).
  L.hist_copies = n >= kHistCopiesMax ? 1u : std::max(1u, std::min(kHistCopiesMax / n, region_room / (32u * kWavesPerBlock)));
  L.hist_bins = off; off = align256(off + (size_t)n * L.hist_copies * kSelBins * sizeof(uint32_t));
  L.zero_bytes = off;
  L.params = off; off = align256(off + (size_t)n * sizeof(ClientParams));
  L.region_cnt = off; off = align256(off + (size_t)n * region_room * sizeof(uint32_t));
  L.region_sumsq = off; off = align256(off + (size_t)n * region_room * sizeof(double));
  L.cand_idx = off; off = align256(off + (size_t)n * d * sizeof(uint16_t));
  L.cand_val = off; off = align256(off + (size_t)n * d * sizeof(uint32_t));
  L.dense_idx = off; off = align256(off + (size_t)n * L.dense_cap * sizeof(uint32_t));
  L.dense_val = off; off = align256(off + (size_t)n * L.dense_cap * sizeof(uint32_t));
  L.nz_off = off; off = align256(off + (size_t)n * (region_room + 1) * sizeof(uint32_t));
  L.nz_run = off; off = align256(off + (size_t)n * (region_room + 1) * sizeof(uint32_t));
  L.span_first = off; off = align256(off + (size_t)n * (L.max_spans + 1) * sizeof(uint32_t));
  L.span_cnt = off; off = align256(off + (size_t)n * (L.max_spans + 1) * 32 * sizeof(uint32_t));
  L.group_info = off; off = align256(off + (size_t)n * sizeof(GroupInfo));
  // Twice what a bin holds of up to 2 M candidates, give or take the sample's error; larger bins have their lists elsewhere.
  L.member_pool = std::min(kMemberPoolMin + L.dense_cap / 128u, kMemberPoolMax);
  L.members = off; off = align256(off + (size_t)n * kMemberSlots * L.member_pool * sizeof(uint64_t));
  L.seg_cnt = off; off = align256(off + (size_t)n * kMemberSlots * kGatherBlocksMax * sizeof(uint32_t));
  L.total = off;
  return L;
}

struct Workspace {  // device pointers into the caller's workspace
  uint32_t* status;
  ClientParams* params;
  ClientCtl* ctl;
  uint32_t* region_cnt;
  double* region_sumsq;
  uint16_t* cand_idx;  // positions of the kept coordinates inside their region: a run at the front of every region's slot
  uint32_t* cand_val;  // their value bits, same layout
  uint32_t* dense_idx; // the same candidates, contiguous per client, in position order: positions (read by emit only)
  uint32_t* dense_val;
  uint32_t* nz_off;      // the non-empty runs in position order: number of the run's first candidate ...
  uint32_t* nz_run;      // ... and its region; entry n_nz of nz_off holds the number of candidates
  uint32_t* span_first;  // index (into the non-empty runs) of the run that holds candidate 512 s, per span s
  uint32_t* span_cnt;  // per span of 512 candidates: members of every group, then their exclusive prefix
  GroupInfo* group_info;
  uint32_t* hist_bins; // per client, hist_copies times: candidates per selection bin (device-wide atomics from the filter, two counters each)
  unsigned long long* members;  // per (client, boundary): the candidates in the boundary's selection bin, as member_of() gives them
  uint32_t* seg_cnt;   // ... and how many of them each of the gather's workgroups has seen
  unsigned long long* norm_limbs;  // QSGD: per (client, group) the exact sum of squares in 32-bit limbs
  uint32_t d, region_shift, n_regions, max_spans, dense_cap, filter_blocks, gather_blocks, member_pool, hist_copies;
};

// Short vectors: their selection, count and emit work on the vector itself, its coordinates take the place of the
// candidates.  Less than any workspace that the general layout fits: that one has 6 bytes per coordinate and 500 KB per client more.
struct ShortLayout {
  size_t status, ctl, norm_limbs, params, places, span_cnt, total;
  uint32_t max_spans;
};

ShortLayout short_layout(uint32_t d, uint32_t n) {
  ShortLayout L;
  L.max_spans = (d + kSpan - 1u) / kSpan;
  size_t off = 0;
  L.status = off; off = align256(off + 256);
  L.ctl = off; off = align256(off + (size_t)n * sizeof(ClientCtl));
  L.norm_limbs = off; off = align256(off + (size_t)n * 32 * kNormLimbs * sizeof(uint64_t));
  L.params = off; off = align256(off + (size_t)n * sizeof(ClientParams));
  L.places = off; off = align256(off + (size_t)n * d * sizeof(uint16_t));
  L.span_cnt = off; off = align256(off + (size_t)n * (L.max_spans + 1) * 32 * sizeof(uint32_t));
  L.total = off;
  return L;
}
static_assert(kSpan >= 2u * 32u, "a span's counts take no more room than its candidates in the general layout");

// ------------------------------------------------------------------ parameter upload
// The per-client parameter blocks travel as kernel arguments (no pinned memory,
// no synchronisation).  Clients of a batch mostly share a plan, so a chunk holds
// every distinct block once, with pointers and client id left out ("template"),
// and six words per client: update pointer, stream pointer, client id, template.
constexpr uint32_t kUploadWords = 960;
constexpr uint32_t kParamWords = sizeof(ClientParams) / 4u;
constexpr uint32_t kRefWords = 6;
static_assert(sizeof(ClientParams) % 4 == 0 && offsetof(ClientParams, update) == 0 &&
                  offsetof(ClientParams, stream) == 8 && offsetof(ClientParams, client_id) == 16,
              "the upload kernel patches words 0..4 of a parameter block");
struct UploadChunk {
  uint32_t n_clients, first_client, n_templates, pad;
  uint32_t data[kUploadWords];  // n_templates parameter blocks, then n_clients references
};

// Word w of the parameter block of the chunk's client-th client.
__device__ __forceinline__ uint32_t param_word(const UploadChunk& c, uint32_t client, uint32_t w) {
  const uint32_t* ref = c.data + c.n_templates * kParamWords + client * kRefWords;
  return w < 5 ? ref[w] : c.data[ref[5] * kParamWords + w];
}

// Workgroup 0 expands the chunk into the clients' parameter blocks; all
// workgroups clear zero_n16 16-byte pieces from `zero` on (the call's state that
// starts at zero, in the call's first launch; a plain kernel, so that a caller
// may capture the call in a graph).
__global__ __launch_bounds__(256) void upload_kernel(uint32_t* dst, UploadChunk c, uint4* zero, uint32_t zero_n16) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < zero_n16; i += gridDim.x * blockDim.x)
    zero[i] = make_uint4(0u, 0u, 0u, 0u);
  if (blockIdx.x == 0) {
    for (uint32_t i = threadIdx.x; i < c.n_clients * kParamWords; i += blockDim.x) {
      const uint32_t client = i / kParamWords, w = i % kParamWords;
      dst[(size_t)(c.first_client + client) * kParamWords + w] = param_word(c, client, w);
    }
  }
}

// ------------------------------------------------------------------ small device helpers
// Number of set bits of the four masks in lanes below the caller's.
__device__ __forceinline__ uint32_t lanes_below4(uint64_t m0, uint64_t m1, uint64_t m2, uint64_t m3) {
  uint32_t acc = __builtin_amdgcn_mbcnt_lo((uint32_t)m0, 0u);
  acc = __builtin_amdgcn_mbcnt_hi((uint32_t)(m0 >> 32), acc);
  acc = __builtin_amdgcn_mbcnt_lo((uint32_t)m1, acc);
  acc = __builtin_amdgcn_mbcnt_hi((uint32_t)(m1 >> 32), acc);
  acc = __builtin_amdgcn_mbcnt_lo((uint32_t)m2, acc);
  acc = __builtin_amdgcn_mbcnt_hi((uint32_t)(m2 >> 32), acc);
  acc = __builtin_amdgcn_mbcnt_lo((uint32_t)m3, acc);
  acc = __builtin_amdgcn_mbcnt_hi((uint32_t)(m3 >> 32), acc);
  return acc;
}

// Pointers read from the parameter block are generic; the update vectors live in
// global memory, and saying so lets the loads be issued as global loads.
typedef const float __attribute__((address_space(1))) * GlobalFloatPtr;
typedef uint32_t __attribute__((address_space(1))) * GlobalWordPtr;
typedef const uint32_t __attribute__((address_space(1))) * GlobalConstWordPtr;
typedef float __attribute__((ext_vector_type(4))) Float4V;
typedef const Float4V __attribute__((address_space(1))) * GlobalFloat4Ptr;

// ------------------------------------------------------------------ 1. sample histogram
// Reads n_s 256-byte pieces spread evenly over the vector and histograms the
// magnitude keys on their top 13 bits.  kSampleBlocks workgroups per client each
// take a slice of the pieces, issue their loads four deep, and add their
// non-empty bins to the client's histogram.
// Small batches: latency, and the counters' clearing and adding up (workgroups of 256 threads, loads eight deep under a branch and
// behind the clearing, for 1, 8 and 32 clients 6.8, 8.0 and 13.6 us; now 4.2, 4.8 and 10.4).
__global__ __launch_bounds__(kWideBlock) void sample_hist_kernel(const ClientParams* __restrict__ params,
                                                             ClientCtl* __restrict__ ctls, uint32_t n_s,
                                                             uint64_t piece_step) {
  constexpr uint32_t kDeep = 4;  // the sample of 4096 pieces in one turn of 16 workgroups
  __shared__ uint32_t hist[kSampleBins];
  const uint32_t client = blockIdx.y;
  const ClientParams& p = params[client];
  ClientCtl* ctl = ctls + client;
  GlobalFloat4Ptr src = (GlobalFloat4Ptr)p.update;
  const uint32_t total_q = n_s * kSamplePieceQuads;
  const uint32_t per_block = (total_q + gridDim.x - 1) / gridDim.x;
  const uint32_t q_begin = min(total_q, blockIdx.x * per_block);
  const uint32_t q_end = min(total_q, q_begin + per_block);
  Float4V v[kDeep];
  auto ask = [&](uint32_t base) {  // no branch around the loads: a thread past the end reads the last piece again
#pragma unroll
    for (uint32_t u = 0; u < kDeep; ++u) {
      const uint32_t q = min(base + u * kWideBlock + threadIdx.x, total_q - 1u);
      const uint32_t j = q / kSamplePieceQuads, part = q % kSamplePieceQuads;
      const uint64_t piece = ((uint64_t)j * piece_step) >> 32;  // piece_step = 2^32 * pieces / n_s, rounded down
      v[u] = src[piece * kSamplePieceQuads + part];
    }
  };
  ask(q_begin);
  for (uint32_t i = threadIdx.x; i < kSampleBins; i += kWideBlock) hist[i] = 0;
  __syncthreads();
  for (uint32_t base = q_begin; base < q_end; base += kWideBlock * kDeep) {
    if (base != q_begin) ask(base);
#pragma unroll
    for (uint32_t u = 0; u < kDeep; ++u) {
      if (base + u * kWideBlock + threadIdx.x < q_end) {
#pragma unroll
        for (int c = 0; c < 4; ++c) atomicAdd(&hist[(__float_as_uint(v[u][c]) & 0x7FFFFFFFu) >> kSampleShift], 1u);
      }
    }
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < kSampleBins; i += kWideBlock) {
    const uint32_t h = hist[i];
    if (h) atomicAdd(&ctl->hist_sample[i], h);
  }
}

// A wavefront's visit to the keys begin .. end - 1 of a list of values: visit(number, key, valid), all lanes
// together.  One workgroup has a CU's share of the bandwidth at best, so eight 16-byte loads a lane go out together.
template <class Visit>
__device__ __forceinline__ void visit_keys(const uint32_t* __restrict__ val, uint32_t begin, uint32_t end, Visit visit) {
  typedef uint32_t __attribute__((ext_vector_type(4), aligned(4))) Words4;
  typedef const Words4 __attribute__((address_space(1))) * Words4Ptr;
  constexpr uint32_t kDeep = 8, kStep = kDeep * 4u * kWave;
  const uint32_t lane = lane_id();
  uint32_t base = begin;
  for (; base + kStep <= end; base += kStep) {
    Words4 v[kDeep];
#pragma unroll
    for (uint32_t u = 0; u < kDeep; ++u) v[u] = *((Words4Ptr)(val + base) + u * kWave + lane);
#pragma unroll
    for (uint32_t u = 0; u < kDeep; ++u)
#pragma unroll
      for (uint32_t c = 0; c < 4u; ++c) visit(base + (u * kWave + lane) * 4u + c, v[u][c] & 0x7FFFFFFFu, true);
  }
  for (; base < end; base += kWave) {
    const uint32_t i = base + lane;
    visit(i, val[min(i, end - 1u)] & 0x7FFFFFFFu, i < end);
  }
}

// ---- selection bins
constexpr uint32_t kNoBin = 0xFFFFFFFFu;

// Selection bin of a key; bins ascend with the keys.
__device__ __forceinline__ uint32_t selection_bin(const uint32_t* map, uint32_t anchor, uint32_t key) {
  const uint32_t top = key >> kSampleShift, t = top - anchor;  // keys below the window wrap to large values
  const uint32_t m = map[min(t, kMapBins - 1u)];
  const uint32_t fine = (m & 0xFFFFu) + ((key & ((1u << kSampleShift) - 1u)) >> (m >> 16));
  const uint32_t coarse = (key >> 23) + (top < anchor ? 0u : kOctaves + kFineBins);
  return t < kMapBins ? fine : coarse;
}

// The bin map for the window that begins at sample bin `anchor`: hist(b) of the `mass` keys at hand lie in sample
// bin b.  Whole workgroup of kWideBlock threads; thread w returns entry w (threads past the window: nothing of use).
template <class Hist>
__device__ __forceinline__ uint32_t build_bin_map(ClientCtl* ctl, uint32_t k, uint32_t anchor, uint32_t mass, uint32_t* scan_tmp, Hist hist) {
  const uint32_t aim = max(kFineMin, min(kFineMax, k / kFineShare));
  const uint32_t w = threadIdx.x;
  const bool mine = w < kMapBins;
  uint32_t bits = 0;
  if (mine && anchor + w < kSampleBins) {
    const uint32_t share = (uint32_t)((uint64_t)hist(anchor + w) * aim / (mass ? mass : 1u));
    if (share > 1u) bits = min(31u - (uint32_t)__builtin_clz(share), 10u);
  }
  uint32_t total;
  const uint32_t first = kOctaves + block_excl_scan<kWideWaves>(mine ? 1u << bits : 0u, scan_tmp, &total);
  const uint32_t entry = first | ((kSampleShift - bits) << 16);
  if (mine) ctl->bin_map[w] = entry;
  if (w == 0) ctl->anchor = anchor;
  return entry;
}
static_assert(kSelBins == 2u * kWideBlock, "two bins per thread in the scan");
static_assert(kMapBins <= kWideBlock && kOctaves + kFineBins < (1u << 16), "one thread per entry of the bin map, bins in 16 bits");

// Sample bins of a thread, largest keys first: thread t owns `kWalkBins` of them, ending at kSampleBins - 1 - kWalkBins * t.
constexpr uint32_t kWalkBins = kSampleBins / kWideBlock;

// The sample bin that holds the `target`-th largest of the keys counted in h (the caller's bins, `above` keys in
// larger ones), and how many keys lie in it or above it: written by the one thread that has it.
__device__ __forceinline__ void find_sample_bin(const uint32_t (&h)[kWalkBins], uint32_t above, uint32_t target,
                                                uint32_t* bin_out, uint32_t* reached_out) {
  const uint32_t top = kSampleBins - 1 - kWalkBins * threadIdx.x;
  uint32_t acc = above;
#pragma unroll
  for (uint32_t i = 0; i < kWalkBins; ++i) {
    if (acc < target && target <= acc + h[i]) {
      *bin_out = top - i;
      *reached_out = acc + h[i];
    }
    acc += h[i];
  }
}

// One workgroup per client walks the sample histogram from the large keys down
// to the sample rank the host derived from k/d plus a 6-sigma margin.  The
// lower edge of that bin becomes the candidate threshold and the window of fine
// selection bins begins there.  Without a threshold (every coordinate is a
// candidate) the window ends where the 4096th part of the sample with the
// largest keys begins: it reaches 16 octaves down from there.
__global__ __launch_bounds__(kWideBlock) void sample_walk_kernel(const ClientParams* __restrict__ params,
                                                                 ClientCtl* __restrict__ ctls) {
  __shared__ uint32_t scan_tmp[kWideWaves];
  __shared__ uint32_t s_bin[2], s_reached[2];
  const uint32_t client = blockIdx.x;
  const ClientParams& p = params[client];
  ClientCtl* ctl = ctls + client;
  const uint32_t target = p.sample_rank;
  const uint32_t top = kSampleBins - 1 - kWalkBins * threadIdx.x;
  uint32_t h[kWalkBins], mine = 0;
#pragma unroll
  for (uint32_t i = 0; i < kWalkBins; ++i) {
    h[i] = ctl->hist_sample[top - i];
    mine += h[i];
  }
  if (threadIdx.x < 2u) {
    s_bin[threadIdx.x] = 0;
    s_reached[threadIdx.x] = 0;
  }
  uint32_t total;
  const uint32_t above = block_excl_scan<kWideWaves>(mine, scan_tmp, &total);
  const bool sampled = target != 0u && target <= total;  // else tau_lo keeps its cleared value 0 (everything is a candidate)
  if (sampled) find_sample_bin(h, above, target, &s_bin[0], &s_reached[0]);
  else find_sample_bin(h, above, total / 4096u + 1u, &s_bin[1], &s_reached[1]);
  __syncthreads();
  if (sampled && threadIdx.x == 0) ctl->tau_lo = s_bin[0] << kSampleShift;
  const uint32_t anchor = sampled ? s_bin[0] : (s_bin[1] >= kMapBins ? s_bin[1] - (kMapBins - 1u) : 0u);
  build_bin_map(ctl, p.k, anchor, sampled ? s_reached[0] : total, scan_tmp, [&](uint32_t b) { return ctl->hist_sample[b]; });
}

// ------------------------------------------------------------------ 2. filter (the full pass)
// A wavefront streams a region in sub-tiles of 1024 coordinates, read as four
// float4 per lane (the j-th at j*256 + lane*4), so position order inside a
// sub-tile is (j, lane, component).  The next sub-tile's loads are issued
// before the current one is processed.
struct SubTile {
  float v[4][4];
};

__device__ __forceinline__ void load_subtile(SubTile& t, GlobalFloatPtr U, uint32_t sbase, uint32_t lane, uint32_t d) {
  if (sbase + kSubTile <= d) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      // read once, never again: keep the stream out of the way of what the caches hold
      const Float4V q = __builtin_nontemporal_load(reinterpret_cast<GlobalFloat4Ptr>(U + sbase + j * 256u + lane * 4u));
      t.v[j][0] = q.x; t.v[j][1] = q.y; t.v[j][2] = q.z; t.v[j][3] = q.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t e0 = sbase + j * 256u + lane * 4u;
#pragma unroll
      for (int c = 0; c < 4; ++c) t.v[j][c] = (e0 + c < d) ? U[e0 + c] : 0.0f;
    }
  }
}

// Kept coordinates are staged per wavefront in LDS and leave in rows of 64 (one
// coalesced 512-byte store each); a row also feeds the histogram over the selection bins.  Loads
// and stores share one outstanding-operation counter on this hardware, so a
// wavefront that has just stored must wait for the store's acknowledgement
// before it can consume its next loads: rows are therefore held back until the
// stage could not take another four float4 per lane, or the region ends.
constexpr uint32_t kStageCap = 448;
constexpr uint32_t kStageFlushAt = kStageCap - 256;  // more staged than this: flush

static_assert(kRegionShiftMax <= 16 && (1u << kRegionShiftMin) == kSubTile, "positions inside a region are kept in 16 bits; a sub-tile lies in one region");

struct FilterWave {
  uint2* stage;            // this wavefront's staging rows in LDS
  uint16_t* __restrict__ out_idx;  // the region's slot in global memory: positions inside the region (13 bits)
  uint32_t* __restrict__ out_val;  // ... and value bits
  uint32_t* hist;          // the workgroup's counts per selection bin, in LDS
  const uint32_t* map;     // the client's bin map, in LDS
  uint32_t anchor;
  uint32_t pos_mask;       // coordinates per region - 1
  uint32_t fill;           // staged entries (uniform)
  uint32_t run;            // entries already written to `out` (uniform)
  uint32_t nonfinite;      // a kept key was Inf or NaN (per lane)
};

// LDS accesses of one wavefront complete in order; this keeps the compiler from
// moving them across the point where lanes read what other lanes wrote.
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

__device__ __forceinline__ void flush_rows(FilterWave& w, uint32_t lane, bool all) {
  wave_lds_fence();
  uint32_t g = 0;
  for (; g + kWave <= w.fill; g += kWave) {
    const uint2 e = w.stage[g + lane];
    w.out_idx[w.run + g + lane] = (uint16_t)(e.x & w.pos_mask);
    w.out_val[w.run + g + lane] = e.y;
    atomicAdd(&w.hist[selection_bin(w.map, w.anchor, e.y & 0x7FFFFFFFu)], 1u);
    w.nonfinite |= (e.y & 0x7FFFFFFFu) >= 0x7F800000u ? 1u : 0u;
  }
  const uint32_t left = w.fill - g;  // < 64
  if (left) {
    uint2 e = make_uint2(0u, 0u);
    if (lane < left) e = w.stage[g + lane];
    if (all) {
      if (lane < left) {
        w.out_idx[w.run + g + lane] = (uint16_t)(e.x & w.pos_mask);
        w.out_val[w.run + g + lane] = e.y;
        atomicAdd(&w.hist[selection_bin(w.map, w.anchor, e.y & 0x7FFFFFFFu)], 1u);
        w.nonfinite |= (e.y & 0x7FFFFFFFu) >= 0x7F800000u ? 1u : 0u;
      }
      g += left;
    } else if (g) {  // move the partial row to the front
      wave_lds_fence();
      if (lane < left) w.stage[lane] = e;
    }
  }
  w.run += g;
  w.fill -= g;
  wave_lds_fence();
}

// Stages the coordinates of one sub-tile whose key reaches tau_lo, in position
// order.  The squares of the others go to *sq.  Inf and NaN have the largest
// keys, so they are always among the kept ones, where flush_rows sees them.
template <bool TAIL>
__device__ __forceinline__ void filter_subtile(const SubTile& t, uint32_t sbase, uint32_t lane, uint32_t d,
                                               uint32_t tau_lo, FilterWave& w, double* sq) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t e0 = sbase + j * 256u + lane * 4u;
    uint32_t bits[4];
    bool keep[4];
    uint64_t m[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      bits[c] = __float_as_uint(t.v[j][c]);
      const uint32_t key = bits[c] & 0x7FFFFFFFu;
      keep[c] = key >= tau_lo && (!TAIL || e0 + c < d);
      m[c] = __ballot(keep[c]);
      const double dropped = (double)(keep[c] ? 0.0f : t.v[j][c]);  // coordinates past d were loaded as 0
      *sq = fma(dropped, dropped, *sq);
    }
    if (m[0] | m[1] | m[2] | m[3]) {
      uint32_t pos = w.fill + lanes_below4(m[0], m[1], m[2], m[3]);
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if (keep[c]) {
          w.stage[pos] = make_uint2(e0 + c, bits[c]);
          ++pos;
        }
      }
      w.fill += (uint32_t)(__popcll(m[0]) + __popcll(m[1]) + __popcll(m[2]) + __popcll(m[3]));
      if (w.fill > kStageFlushAt) flush_rows(w, lane, false);
    }
  }
}

__global__ __launch_bounds__(kBlock) void filter_kernel(const ClientParams* __restrict__ params,
                                                        ClientCtl* __restrict__ ctls, Workspace ws) {
  __shared__ alignas(8) uint32_t s_hist[kSelBins];
  __shared__ uint32_t s_map[kMapBins];
  __shared__ uint2 s_stage[kWavesPerBlock][kStageCap];
  // workgroups start in the order of their number, and the older ones get ahead: every client gets its share of both
  const uint32_t lin = blockIdx.y * gridDim.x + blockIdx.x;
  const uint32_t client = lin % gridDim.y, block_x = lin / gridDim.y;
  const ClientParams& p = params[client];
  ClientCtl* ctl = ctls + client;
  const uint32_t tau_lo = ctl->tau_lo;
  const uint32_t d = ws.d, n_regions = ws.n_regions, region_len = 1u << ws.region_shift;
  GlobalFloatPtr U = (GlobalFloatPtr)p.update;
  const uint32_t lane = lane_id();
  for (uint32_t i = threadIdx.x; i < kSelBins; i += kBlock) s_hist[i] = 0;
  for (uint32_t i = threadIdx.x; i < kMapBins; i += kBlock) s_map[i] = ctl->bin_map[i];
  __syncthreads();

  double sq = 0.0;
  const uint32_t n_waves = gridDim.x * kWavesPerBlock;
  FilterWave w;
  w.stage = s_stage[wave_id()];
  w.hist = s_hist;
  w.map = s_map;
  w.anchor = ctl->anchor;
  w.pos_mask = region_len - 1u;
  w.nonfinite = 0;
  // Software pipeline over all sub-tiles of all of this wavefront's regions: the
  // loads of the next sub-tile (of the next region, at a region's end) are issued
  // before the current one is processed, so the rare row stores sit behind loads
  // that are already in flight.
  const uint32_t wave_global = block_x * kWavesPerBlock + wave_id();
  // Which regions a wavefront takes.  The first half of the rounds is dealt out (region = wavefront + round x
  // wavefronts: all wavefronts read one moving window); the rest is claimed from a counter of the client's, one
  // region at a time and one region ahead, so that the wavefronts that get ahead (the memory system serves
  // the oldest first) take over from those that fall behind and all end together: 285 -> 273 us.  (Claiming
  // every region: 278 us; a quarter of them: 276 us.)
  const uint32_t rounds = n_regions / n_waves;
  const uint32_t n_static = rounds >= 4u ? (rounds - rounds / 2u) * n_waves : n_regions;
  auto claim = [&]() {  // the next region nobody has taken yet (a per-lane value, lane 0's counts; not waited for here)
    uint32_t got = 0;
    if (lane == 0) got = atomicAdd(&ctl->claim, 1u);
    return got;
  };
  uint32_t region = wave_global;
  if (region >= n_static) region = n_static < n_regions ? n_static + (uint32_t)__builtin_amdgcn_readfirstlane(claim()) : n_regions;
  if (region < n_regions) {
    SubTile cur, nxt;
    bool upcoming_static = false;
    uint32_t claimed = 0;
    uint32_t sbase = region << ws.region_shift;
    load_subtile(cur, U, sbase, lane, d);
    while (true) {
      const uint32_t rbase = region << ws.region_shift;
      const uint32_t rend = (d - rbase < region_len) ? d : rbase + region_len;
      if (sbase == rbase) {
        w.out_idx = ws.cand_idx + (size_t)client * d + rbase;
        w.out_val = ws.cand_val + (size_t)client * d + rbase;
        w.fill = 0;
        w.run = 0;
        // the region after this one: the next of the wavefront's own, or one that is claimed now and known by the time this one ends
        upcoming_static = region < n_static && region + n_waves < n_static;
        if (!upcoming_static && n_static < n_regions) claimed = claim();
      }
      // where the pipeline goes next
      const bool last_of_region = sbase + kSubTile >= rend;
      uint32_t next_region = region;
      if (last_of_region)
        next_region = upcoming_static ? region + n_waves
                                      : (n_static < n_regions ? n_static + (uint32_t)__builtin_amdgcn_readfirstlane(claimed) : n_regions);
      const uint32_t next_sbase = last_of_region ? next_region << ws.region_shift : sbase + kSubTile;
      const bool more = next_region < n_regions;
      if (more) load_subtile(nxt, U, next_sbase, lane, d);
      if (sbase + kSubTile <= d) {
        filter_subtile<false>(cur, sbase, lane, d, tau_lo, w, &sq);
      } else {
        filter_subtile<true>(cur, sbase, lane, d, tau_lo, w, &sq);
      }
      if (last_of_region) {
        flush_rows(w, lane, true);
        const double total = wave_sum_f64(sq);
        sq = 0.0;
        if (lane == 0) {
          ws.region_cnt[(size_t)client * n_regions + region] = w.run;
          ws.region_sumsq[(size_t)client * n_regions + region] = total;
        }
      }
      if (!more) break;
      cur = nxt;
      region = next_region;
      sbase = next_sbase;
    }
  }
  // a threshold in the Inf/NaN range can only come from a sample that held such values
  if (w.nonfinite || tau_lo > 0x7F800000u) atomicOr(ws.status, CVLC_DEV_NONFINITE);
  __syncthreads();
  // two counters an atomic; no carry between them: a client has fewer than 2^32 candidates
  unsigned long long* mine = reinterpret_cast<unsigned long long*>(
      ws.hist_bins + ((size_t)client * ws.hist_copies + block_x % ws.hist_copies) * kSelBins);
  for (uint32_t i = threadIdx.x; i < kSelBins / 2u; i += kBlock) {
    const unsigned long long h = reinterpret_cast<const unsigned long long*>(s_hist)[i];
    if (h) atomicAdd(mine + i, h);
  }
}

// ---- member lists
// The gather sets the members of the boundaries' selection bins aside for the select kernel.  How many a bin has is
// known by then, so a list has room for all of them: a piece for every gather workgroup that has spans to go through,
// and behind the pieces room for what found its piece full, all members if need be.  Bins grow with the candidates
// (one to two 1024ths of them from 262 144 kept coordinates on): a list of up to half the boundary's pool lies there,
// a larger one in the client's own stream buffer, which nothing else is written to before the counting pass and which has
// three bytes and more for every kept coordinate.  For a client whose sample misjudged it lies in the filter's
// output, which is not looked at then.  Boundaries that share a bin share the list of the first of them.  A bin that
// holds a large part of all candidates (equal magnitudes) has no list, the select kernel walks the candidates for it.
constexpr uint32_t kWalkShare = 16;  // more than this part of the candidates: no list
typedef unsigned long long __attribute__((address_space(1))) * GlobalU64Ptr;

// A member as one number: members rank as the coordinates do (larger keys first, earlier positions first), no two are alike.
__device__ __forceinline__ unsigned long long member_of(uint32_t dense_i, uint32_t key) {
  return ((unsigned long long)key << 32) | (uint32_t)~dense_i;
}

// Workgroups of a client's gather that have spans to go through.
__device__ __forceinline__ uint32_t gather_workgroups(const Workspace& ws, uint32_t n_cand) {
  return max(1u, min(ws.gather_blocks, (n_cand + kSpan * kGatherWaves - 1u) / (kSpan * kGatherWaves)));
}

// One whole wavefront, lane b = boundary b: the list of its bin.
__device__ __forceinline__ MemberList place_member_list(const Workspace& ws, const ClientParams& p, uint32_t client, bool keep_all,
                                                        uint32_t n_cand, uint32_t bin, uint32_t members) {
  const uint32_t lane = lane_id();
  const uint32_t blocks = gather_workgroups(ws, n_cand);
  MemberList l = {0u, 0u, 0u, 0u, members};
  const bool valid = bin != kNoBin, large = valid && members > ws.member_pool / 2u;
  if (valid && !large) {
    l.entries = (uint64_t)(ws.members + ((size_t)client * kMemberSlots + lane) * ws.member_pool);
    l.cap = (ws.member_pool - members) / blocks;
    l.over_first = blocks * l.cap;
    l.over_room = ws.member_pool - l.over_first;
  }
  if (!__ballot(large)) return l;  // (a small list is looked for in the place of the first of its boundaries only)
  uint32_t first = lane;
#pragma unroll
  for (int j = (int)kMemberSlots - 1; j >= 0; --j)
    if ((uint32_t)j < lane && (uint32_t)__builtin_amdgcn_readlane(bin, j) == bin) first = (uint32_t)j;
  // the area of the larger lists, 8-byte aligned
  const uint64_t at = keep_all ? (uint64_t)(ws.cand_val + (size_t)client * ws.d) : (uint64_t)p.stream;
  const uint32_t words = keep_all ? ws.d : p.total_words, skip = (uint32_t)(at >> 2) & 1u;
  const uint32_t room = (max(words, skip) - skip) / 2u;
  uint32_t need = 0;
  if (large && members <= n_cand / kWalkShare) {
    l.cap = members / blocks + members / (4u * blocks) + 16u;  // a quarter more than the workgroups' equal shares
    l.over_first = blocks * l.cap;
    l.over_room = members;
    if (first == lane) need = l.over_first + l.over_room;  // below 2^29
  }
  uint32_t used = 0;
  for (uint32_t b = 0; b < kMemberSlots; ++b) {
    const uint32_t n = __builtin_amdgcn_readlane(need, b);
    if (n == 0 || n > room - used) continue;  // uniform
    if (first == b && large) l.entries = at + 4u * skip + 8ull * used;
    used += n;
  }
  return l;
}

// ------------------------------------------------------------------ 3. region prefix + the boundaries' selection bins
// One workgroup per client.  Turns the region counts into exclusive offsets
// and lists the non-empty runs with the number of their first candidate (the
// candidates' position-ordered numbering; the gather works in spans of 512
// candidates, and the run holding every span's first candidate is noted), then reads the counts per
// selection bin that the filter's workgroups accumulated and locates, for every boundary
// Z_r, the bin holding the Z_r-th largest key and the rank left inside it.
// Should the sampled threshold have kept fewer than k coordinates (the sample
// misjudged: six standard deviations, or a vector built against the sampling
// pattern), every coordinate becomes a candidate: the runs are then the regions
// themselves, read from the vector, and this workgroup draws up the bin map again, from
// the whole vector, and counts its selection bins on its own: slow, and next to never needed (1 x 11.2 M: 0.8 ms).
__global__ __launch_bounds__(kWideBlock) void scan_l1_kernel(const ClientParams* __restrict__ params,
                                                             ClientCtl* __restrict__ ctls, Workspace ws) {
  __shared__ uint32_t hist[kSelBins];
  __shared__ uint32_t incl[kSelBins];  // keys in bins >= b
  __shared__ uint32_t top_hist[kSampleBins];  // a misjudged sample: counts of key >> 18 of the whole vector
  __shared__ uint32_t s_bin, s_reached;
  __shared__ uint32_t scan_tmp[kWideWaves], scan_tmp2[kWideWaves];
  const uint32_t client = blockIdx.x, tid = threadIdx.x;
  const ClientParams& p = params[client];
  ClientCtl* ctl = ctls + client;
  const uint32_t n_regions = ws.n_regions;
  const uint32_t* cnt = ws.region_cnt + (size_t)client * n_regions;
  uint32_t* nz_off = ws.nz_off + (size_t)client * (n_regions + 1);
  uint32_t* nz_run = ws.nz_run + (size_t)client * (n_regions + 1);
  uint32_t* span_first = ws.span_first + (size_t)client * (ws.max_spans + 1);
  // One workgroup per client, all latency: everything that is read is asked for before anything is waited for, and a thread takes
  // one, two or four neighbouring regions, so that 4096 regions are one scan, of counts and non-empty regions together (a region
  // a thread, and two scans a round: 9.5 us for the 2735 regions of 1 x 11.2 M, 12.4 for the 3125 of 100 x 25.6 M, 7.3 and 9.9 now).
  const uint2* counted = reinterpret_cast<const uint2*>(ws.hist_bins + (size_t)client * ws.hist_copies * kSelBins);
  uint2 bins = counted[tid], more[kHistCopiesMax - 1u];
#pragma unroll
  for (uint32_t c = 1; c < kHistCopiesMax; ++c) more[c - 1u] = make_uint2(0u, 0u);
  uint32_t run = 0, n_nz = 0;
  auto scan_regions = [&](auto each) {
    constexpr uint32_t kEach = decltype(each)::value;
    uint32_t v[kEach];
    auto ask = [&](uint32_t base) {
#pragma unroll
      for (uint32_t i = 0; i < kEach; ++i) v[i] = cnt[min(base + tid * kEach + i, n_regions - 1u)];  // no branch around the loads
    };
    ask(0);
    if (ws.hist_copies > 1u) {  // a few clients at most
#pragma unroll
      for (uint32_t c = 1; c < kHistCopiesMax; ++c) more[c - 1u] = counted[min(c, ws.hist_copies - 1u) * (kSelBins / 2u) + tid];
    }
    for (uint32_t base = 0; base < n_regions; base += kWideBlock * kEach) {
      if (base) ask(base);
      uint32_t sum = 0, q = 0, total, total_nz;
#pragma unroll
      for (uint32_t i = 0; i < kEach; ++i) {
        v[i] = base + tid * kEach + i < n_regions ? v[i] : 0u;
        sum += v[i];
        q += v[i] ? 1u : 0u;
      }
      uint32_t begin = run + block_excl_scan2<kWideWaves>(sum, q, scan_tmp, scan_tmp2, &total, &total_nz);
      q += n_nz;
#pragma unroll
      for (uint32_t i = 0; i < kEach; ++i) {
        if (v[i]) {
          const uint32_t end = begin + v[i];
          nz_off[q] = begin;
          nz_run[q] = base + tid * kEach + i;
          // spans whose first candidate lies in this run (those the workspace has room for; more: see below)
          for (uint32_t sp = (begin + kSpan - 1) / kSpan; (uint64_t)sp * kSpan < end && sp <= ws.max_spans; ++sp)
            span_first[sp] = q;
          begin = end;
          ++q;
        }
      }
      run += total;
      n_nz += total_nz;
    }
  };
  if (n_regions <= kWideBlock) scan_regions(std::integral_constant<uint32_t, 1>());
  else if (n_regions <= 2u * kWideBlock) scan_regions(std::integral_constant<uint32_t, 2>());
  else scan_regions(std::integral_constant<uint32_t, 4>());
  const bool keep_all = run < p.k;  // uniform
  if (run > ws.dense_cap || (keep_all && ws.d > ws.dense_cap)) {  // the caller's workspace is too short for this vector: no stream, and say so
    if (tid == 0) {
      nz_off[0] = 0;
      ctl->n_cand = 0;
      ctl->n_nz = 0;
      ctl->dead = 1u;
      p.stream[0] = 0u;  // not a stream header
      atomicOr(ws.status, CVLC_DEV_WORKSPACE);
    }
    return;
  }
  if (!keep_all) {
    if (tid == 0) {
      nz_off[n_nz] = run;
      ctl->n_cand = run;
      ctl->n_nz = n_nz;
    }
#pragma unroll
    for (uint32_t c = 1; c < kHistCopiesMax; ++c) {
      bins.x += c < ws.hist_copies ? more[c - 1u].x : 0u;
      bins.y += c < ws.hist_copies ? more[c - 1u].y : 0u;
    }
    hist[2u * tid] = bins.x;
    hist[2u * tid + 1] = bins.y;
  } else {
    const uint32_t d = ws.d;
    __syncthreads();  // the runs written above are overwritten
    double* rsq = ws.region_sumsq + (size_t)client * n_regions;
    for (uint32_t j = tid; j < n_regions; j += kWideBlock) {
      nz_off[j] = j << ws.region_shift;
      nz_run[j] = j;
      rsq[j] = 0.0;  // nothing is dropped before the selection
    }
    for (uint32_t sp = tid; (uint64_t)sp * kSpan < d; sp += kWideBlock) span_first[sp] = sp >> (ws.region_shift - kSpanShift);
    if (tid == 0) {
      nz_off[n_regions] = d;
      ctl->n_cand = d;
      ctl->n_nz = n_regions;
      ctl->keep_all = 1u;
    }
    hist[2u * tid] = 0;
    hist[2u * tid + 1] = 0;
    for (uint32_t i = tid; i < kSampleBins; i += kWideBlock) top_hist[i] = 0;
    __syncthreads();
    // What one workgroup has of the memory's bandwidth bounds this (60 GB/s), and the LDS atomics, which hit few
    // counters: one pass, if it can be, of the keys at or above the sample's key of four times the rank that was too
    // low; all of them if they are fewer than k (at once all of them where the sample is wide of the mark).  The bins
    // are the sample bins themselves, from the one that holds the k-th key on: finer ones would take a second pass,
    // the longer member lists cost less.
    const uint32_t* __restrict__ bits = reinterpret_cast<const uint32_t*>(p.update);
    const uint32_t share = (d + kWideBlock - 1u) / kWideBlock * kWave;
    const uint32_t w_begin = min(tid / kWave * share, d), w_end = min(w_begin + share, d);
    uint32_t h[kWalkBins], mine = 0, all, above;
#pragma unroll
    for (uint32_t i = 0; i < kWalkBins; ++i) {
      h[i] = ctl->hist_sample[kSampleBins - 1 - kWalkBins * tid - i];
      mine += h[i];
    }
    if (tid == 0) s_bin = 0;
    above = block_excl_scan<kWideWaves>(mine, scan_tmp, &all);
    if (run >= p.k / 4u) find_sample_bin(h, above, 4u * p.sample_rank, &s_bin, &s_reached);
    __syncthreads();
    constexpr uint32_t kNonfiniteBin = 0x7F800000u >> kSampleShift;  // the first that only Inf and NaN lie in
    for (uint32_t floor_bin = min(s_bin, kNonfiniteBin);; floor_bin = 0) {
      auto count_top = [&](auto floored) {
        visit_keys(bits, w_begin, w_end, [&](uint32_t, uint32_t key, bool valid) {
          const uint32_t b = key >> kSampleShift;
          if (valid && (!floored.value || b >= floor_bin)) atomicAdd(&top_hist[b], 1u);
        });
      };
      if (floor_bin) count_top(std::true_type{}); else count_top(std::false_type{});
      __syncthreads();
      mine = 0;
#pragma unroll
      for (uint32_t i = 0; i < kWalkBins; ++i) {
        h[i] = top_hist[kSampleBins - 1 - kWalkBins * tid - i];
        mine += h[i];
      }
      above = block_excl_scan<kWideWaves>(mine, scan_tmp, &all);
      if (all >= p.k || floor_bin == 0) break;  // uniform
      __syncthreads();
      for (uint32_t i = tid; i < kSampleBins; i += kWideBlock) top_hist[i] = 0;
      __syncthreads();
    }
    if (tid < kSampleBins - kNonfiniteBin && top_hist[kNonfiniteBin + tid]) atomicOr(ws.status, CVLC_DEV_NONFINITE);
    find_sample_bin(h, above, p.k, &s_bin, &s_reached);  // 1 <= k <= d here: fewer than k were kept
    __syncthreads();
    const uint32_t anchor = s_bin;
    build_bin_map(ctl, p.k, anchor, 1u, scan_tmp, [](uint32_t) { return 0u; });
    if (tid < kMapBins && anchor + tid < kSampleBins) hist[kOctaves + tid] = top_hist[anchor + tid];
    for (uint32_t b = anchor + kMapBins + tid; b < kSampleBins; b += kWideBlock) {
      const uint32_t n = top_hist[b];
      if (n) atomicAdd(&hist[kOctaves + kFineBins + (b >> (23u - kSampleShift))], n);
    }
  }
  __syncthreads();
  const uint32_t top = kSelBins - 1 - 2u * tid;
  const uint32_t h0 = hist[top], h1 = hist[top - 1];
  uint32_t total;
  const uint32_t above = block_excl_scan<kWideWaves>(h0 + h1, scan_tmp, &total);
  incl[top] = above + h0;
  incl[top - 1] = above + h0 + h1;
  __syncthreads();
  if (tid < kWave) {  // lane b = boundary b
    uint32_t bin = kNoBin, rem = 0, members = 0;
    if (tid < p.R) {
      const uint32_t Z = p.Z[tid];
      if (Z > total) atomicOr(ws.status, CVLC_DEV_INTERNAL);  // cannot happen once the filter kept >= k
      if (Z != 0 && Z <= total) {
        uint32_t lo = 0, hi = kSelBins - 1;  // largest bin b with incl[b] >= Z
        while (lo < hi) {
          const uint32_t mid = (lo + hi + 1) >> 1;
          if (incl[mid] >= Z) lo = mid; else hi = mid - 1;
        }
        bin = lo;
        rem = Z - (incl[lo] - hist[lo]);
        members = hist[lo];
      }
    }
    const uint32_t n_cand = keep_all ? ws.d : run;
    const MemberList list = place_member_list(ws, p, client, keep_all, n_cand, bin, members);
    if (tid < 32) {
      ctl->sel_bin[tid] = bin;
      ctl->sel_rem[tid] = rem;
      ctl->list[tid] = list;
      ctl->tau[tid] = 0xFFFFFFFFu;  // boundaries with Z_r = 0 keep "nothing inside"
      ctl->iota[tid] = 0u;
    }
  }
}

// ------------------------------------------------------------------ 4. selection inside the boundaries' bins
// scan_l1 has left, for every boundary, the selection bin its key lies in and
// the boundary's rank inside that bin.  A bin holds about a thousandth of the
// candidates, so the gather, which reads every candidate anyway, sets the
// members of the boundaries' bins aside (key and number in the dense list), and
// the select kernel finds each boundary's element among them.  Its number in the
// dense list cuts a class of equal keys (ties rank by position, and that
// numbering preserves positions): keys above tau are inside, and so are those
// equal to it up to number iota.
// ---- walking the filter's output in position order
constexpr uint32_t kNoGroup = 0xFFFFFFFFu;
constexpr uint32_t kEmitBlock = kSpan * kChunkSpans / 8u;  // threads of a count/emit workgroup: 8 candidates each
constexpr uint32_t kEmitWaves = kEmitBlock / kWave;
constexpr uint32_t kPerLane = kSpan / kWave;              // candidates per lane per span
static_assert(kEmitWaves == kChunkSpans && kPerLane == 8, "one wavefront per span, eight rows of 64");

// The candidates of one client in position order, as the filter left them:
// candidate i is entry i - nz_off[q] of the run of region nz_run[q], q the last
// non-empty run with nz_off[q] <= i.
struct CandView {
  const uint32_t* __restrict__ val;         // region slots: value bits
  const uint16_t* __restrict__ idx;         // region slots: positions inside the region
  const uint32_t* __restrict__ nz_off;      // n_nz + 1 entries, the last = n
  const uint32_t* __restrict__ nz_run;
  const uint32_t* __restrict__ span_first;  // q of candidate 512 s
  uint32_t n_nz, n, region_shift;
};

__device__ __forceinline__ CandView cand_view(const Workspace& ws, const ClientCtl* ctl, uint32_t client) {
  CandView view;
  view.val = ws.cand_val + (size_t)client * ws.d;
  view.idx = ws.cand_idx + (size_t)client * ws.d;
  view.nz_off = ws.nz_off + (size_t)client * (ws.n_regions + 1);
  view.nz_run = ws.nz_run + (size_t)client * (ws.n_regions + 1);
  view.span_first = ws.span_first + (size_t)client * (ws.max_spans + 1);
  view.n_nz = ctl->n_nz;
  view.n = ctl->n_cand;
  view.region_shift = ws.region_shift;
  return view;
}

// Places of the candidates of span `span` in the region slots: row j of the
// span is candidate span*512 + j*64 + lane.  The runs that follow the span's
// first one are fetched 64 at a time, one per lane; every run that starts
// inside the span moves the rows at or after its first candidate on to it.
struct SpanWindow {  // the first 64 runs at or after a span's first candidate, one per lane
  uint32_t base, wo, wr;
};

__device__ __forceinline__ SpanWindow span_window(const CandView& cv, uint32_t span) {
  SpanWindow w;
  w.base = cv.span_first[span];
  w.wo = cv.nz_off[min(w.base + lane_id(), cv.n_nz)];
  w.wr = cv.nz_run[min(w.base + lane_id(), cv.n_nz)];  // entry n_nz is never selected: its offset is n >= end
  return w;
}

// A span that lies in a stretch of nearly empty regions crosses hundreds of runs (it has 512 candidates, so up
// to 512 of them): walking those one by one, a memory round trip per 63, made single wavefronts the last to
// finish by far.  So: few runs inside the window (the rule) are walked one by one; many are searched by every
// row at once (the window's 64 offsets ascend: six shuffle steps); the window after is asked for before
// the current one is worked on.
constexpr uint32_t kSerialRuns = 8;

__device__ __forceinline__ void span_slots(const CandView& cv, uint32_t span, const SpanWindow& win,
                                           uint32_t (&slot)[kPerLane]) {
  const uint32_t lane = lane_id();
  const uint32_t begin = span * kSpan;
  const uint32_t end = min(begin + kSpan, cv.n);
  uint32_t base = win.base, wo = win.wo, wr = win.wr;
  // slot of candidate i in run (region r, first candidate o): (r << region_shift) + (i - o); kept as i + shift
  const uint32_t shift0 = (__builtin_amdgcn_readlane(wr, 0) << cv.region_shift) - __builtin_amdgcn_readlane(wo, 0);
#pragma unroll
  for (uint32_t j = 0; j < kPerLane; ++j) slot[j] = shift0;
  while (true) {
    // entries 1..m of the window start inside the span (offsets ascend strictly; the entry after the last run holds n >= end)
    const uint32_t m = (uint32_t)__popcll(__ballot(wo < end) & ~1ull);
    const bool more = m == kWave - 1u;  // the window's last entry still starts inside: look at the next window too
    uint32_t nwo = 0, nwr = 0;
    if (more) {  // uniform
      nwo = cv.nz_off[min(base + (kWave - 1u) + lane, cv.n_nz)];
      nwr = cv.nz_run[min(base + (kWave - 1u) + lane, cv.n_nz)];
    }
    if (m <= kSerialRuns) {
      for (uint32_t t = 1; t <= m; ++t) {
        const uint32_t ot = __builtin_amdgcn_readlane(wo, t);
        const uint32_t shift = (__builtin_amdgcn_readlane(wr, t) << cv.region_shift) - ot;
#pragma unroll
        for (uint32_t j = 0; j < kPerLane; ++j) {
          const uint32_t i = begin + j * kWave + lane;
          if (i >= ot) slot[j] = shift;
        }
      }
    } else {
      const uint32_t first_here = __builtin_amdgcn_readlane(wo, 1);  // rows before it keep what they have
#pragma unroll
      for (uint32_t j = 0; j < kPerLane; ++j) {
        const uint32_t i = begin + j * kWave + lane;
        uint32_t pos = 0;  // last entry in 0..m whose offset is <= i
#pragma unroll
        for (uint32_t step = kWave / 2u; step; step >>= 1) {
          const uint32_t probe = (uint32_t)__shfl((int)wo, (int)min(pos + step, kWave - 1u), kWave);
          if (pos + step <= m && probe <= i) pos += step;
        }
        const uint32_t ro = (uint32_t)__shfl((int)wo, (int)pos, kWave), rr = (uint32_t)__shfl((int)wr, (int)pos, kWave);
        if (i >= first_here) slot[j] = (rr << cv.region_shift) - ro;
      }
    }
    if (!more) break;
    base += kWave - 1;  // entry 63 of this window is entry 0 of the next
    wo = nwo;
    wr = nwr;
  }
#pragma unroll
  for (uint32_t j = 0; j < kPerLane; ++j) slot[j] += begin + j * kWave + lane;  // meaningless for i >= n, never used there
}

// What the wavefronts of a gather workgroup share.
struct GatherShared {
  uint32_t map[kMapBins];
  uint8_t tag[kSelBins];       // per selection bin: 1 + the first boundary whose key lies in it, 0: none
  uint32_t bin[32];
  // per boundary
  uint32_t seen[32];           // members of its bin met by this workgroup
  uint4 list[32];              // the bin's list: address of its entries, cap, over_first
  uint32_t over_room[32];
};

// Every wavefront takes spans of 512 candidates (gw, gw + wavefronts, ...), collects
// them from the region runs they lie in, stores them at their place in the
// dense position-ordered candidate list and sets the members of the boundaries'
// bins aside.  Every span is the same amount of work wherever its candidates lie,
// and the wavefronts do not wait for each other.
// Bound by its mixed traffic (6 bytes read and 8 written per candidate).  A member takes its place in its workgroup's
// piece of the list with an LDS atomic; only what the piece has no room for takes one with a device-wide atomic,
// behind the pieces.
// (Past 80 scalar registers a CU takes one workgroup of 1024 threads instead of two, 565 us instead of 466 for
// 100 x 25.6 M: capped.)
__global__ __launch_bounds__(kGatherBlock) __attribute__((amdgpu_num_sgpr(80))) void gather_kernel(const ClientParams* __restrict__ params,
                                                              ClientCtl* __restrict__ ctls, Workspace ws) {
  __shared__ GatherShared S;
  const uint32_t client = blockIdx.y, tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const ClientParams& p = params[client];
  ClientCtl* ctl = ctls + client;
  const uint32_t R = p.R, anchor = ctl->anchor;
  const CandView cv = cand_view(ws, ctl, client);
  static_assert(kMapBins <= kGatherBlock && kSelBins / 4u <= kGatherBlock, "one entry per thread");
  // everything that is read from the control block is asked for together
  const uint32_t my_map = ctl->bin_map[min(tid, kMapBins - 1u)], b = min(tid, kMemberSlots - 1u);
  const uint32_t my_bin = tid < R ? ctl->sel_bin[b] : kNoBin;
  const uint64_t my_entries = ctl->list[b].entries;
  const uint32_t my_cap = ctl->list[b].cap, my_over_first = ctl->list[b].over_first, my_over_room = ctl->list[b].over_room;
  if (ctl->dead) return;  // the workspace was too short for this client (whole workgroup)
  if (tid < kMapBins) S.map[tid] = my_map;
  if (tid < kSelBins / 4u) reinterpret_cast<uint32_t*>(S.tag)[tid] = 0;
  if (tid < 32) {
    S.bin[tid] = my_bin;
    S.seen[tid] = 0;
    S.list[tid] = make_uint4((uint32_t)my_entries, (uint32_t)(my_entries >> 32), my_cap, my_over_first);
    S.over_room[tid] = my_over_room;
  }
  __syncthreads();
  if (tid < R) {
    bool first = my_entries != 0;
    for (uint32_t o = 0; o < tid; ++o) first = first && S.bin[o] != my_bin;
    if (first) S.tag[my_bin] = (uint8_t)(tid + 1u);
  }
  __syncthreads();
  const uint32_t blocks = gather_workgroups(ws, cv.n);
  if (blockIdx.x >= blocks) return;  // no span is left for this workgroup
  uint32_t* __restrict__ dst_idx = ws.dense_idx + (size_t)client * ws.dense_cap;
  uint32_t* __restrict__ dst_val = ws.dense_val + (size_t)client * ws.dense_cap;
  auto entries_of = [](const uint4& l) { return (GlobalU64Ptr)(((uint64_t)l.y << 32) | l.x); };
  // slot: 1 + boundary, 0: in no boundary's bin
  auto set_aside = [&](uint32_t slot, uint32_t dense_i, uint32_t key) {
    bool over = false;
    if (slot) {
      const uint32_t place = atomicAdd(&S.seen[slot - 1u], 1u);
      const uint4 l = S.list[slot - 1u];
      if (place < l.z) entries_of(l)[blockIdx.x * l.z + place] = member_of(dense_i, key);
      else over = true;
    }
    uint64_t todo = __ballot(over);
    while (todo) {  // one device-wide atomic per boundary and row
      const uint32_t leader = (uint32_t)__builtin_ctzll(todo), q = __builtin_amdgcn_readlane(slot, leader) - 1u;
      const uint64_t peers = __ballot(over && slot == q + 1u);
      uint32_t base = 0;
      if (lane == leader) base = atomicAdd(&ctl->over_cnt[q], (uint32_t)__popcll(peers));
      base = __builtin_amdgcn_readlane(base, leader);
      if (over && slot == q + 1u) {
        const uint32_t place = base + lanes_below(peers);
        if (place < S.over_room[q])  // always: a list has room for all members
          entries_of(S.list[q])[S.list[q].w + place] = member_of(dense_i, key);
      }
      todo &= ~peers;
    }
  };
  const uint32_t n_spans = (cv.n + kSpan - 1) / kSpan;
  // keep_all: a slot is a region of the vector itself and a candidate's place in it its position
  auto copy_spans = [&](auto keep_all) {
    const uint32_t* __restrict__ src_val = keep_all.value ? reinterpret_cast<const uint32_t*>(p.update) : cv.val;
    for (uint32_t span = blockIdx.x * kGatherWaves + wave; span < n_spans; span += blocks * kGatherWaves) {
      uint32_t slot[kPerLane], v[kPerLane], x[kPerLane];
      span_slots(cv, span, span_window(cv, span), slot);
#pragma unroll
      for (uint32_t j = 0; j < kPerLane; ++j) {
        // rows past the last candidate read some valid place instead of branching, so that the
        // sixteen loads of a span go out together
        const uint32_t sl = min(slot[j], ws.d - 1u);
        v[j] = src_val[sl];
        x[j] = keep_all.value ? sl : ((sl >> cv.region_shift) << cv.region_shift) + cv.idx[sl];  // a slot starts where its region starts
      }
      uint32_t tag[kPerLane];
#pragma unroll
      for (uint32_t j = 0; j < kPerLane; ++j) {
        const uint32_t i = span * kSpan + j * kWave + lane;
        if (i < cv.n) {
          dst_val[i] = v[j];
          dst_idx[i] = x[j];
        }
        tag[j] = i < cv.n ? S.tag[selection_bin(S.map, anchor, v[j] & 0x7FFFFFFFu)] : 0u;
      }
#pragma unroll
      for (uint32_t j = 0; j < kPerLane; ++j)
        if (__ballot(tag[j] != 0u)) set_aside(tag[j], span * kSpan + j * kWave + lane, v[j] & 0x7FFFFFFFu);
    }
  };
  if (ctl->keep_all) copy_spans(std::true_type{}); else copy_spans(std::false_type{});
  __syncthreads();
  if (tid < R) ws.seg_cnt[((size_t)client * kMemberSlots + tid) * kGatherBlocksMax + blockIdx.x] = S.seen[tid];
}

// One workgroup per (boundary, client); boundaries whose keys lie in one bin are
// all served by the first of them while the bin's list fits LDS, each by its own workgroup otherwise.  Members are
// 64-bit numbers of which no two are alike (see member_of).  Ten bits at a time below the highest bit in which the
// members differ are counted, until a wavefront's worth of them is left.  A bin without a list
// (equal keys) is looked for in the dense list (search_candidates), until LDS can hold what is left of it.
// All latency: one or two rounds of a handful of barriers each.
constexpr uint32_t kSelectBlock = 512;
constexpr uint32_t kSelectList = 2048;  // members kept in LDS; more are read again for every round
constexpr uint32_t kSelectWaves = kSelectBlock / kWave;
constexpr uint32_t kSelectDigits = 2u * kSelectBlock;  // two per thread
static_assert(kSelectDigits == 1024u, "ten bits a round");

struct SelectShared {
  unsigned long long list[kSelectList];
  uint32_t hist[kSelectDigits];
  uint32_t bin[32], rem[32], seg_first[kGatherBlocksMax + 1], scan_tmp[kSelectWaves];
  unsigned long long min, max, answer, few[kWave];
  uint32_t digit, left, in_digit, n_few;
  uint32_t lo, hi, larger, equal[kSelectWaves];  // search_candidates
};

// The digit that holds the rem-th largest of what is counted in S.hist: S.digit, how many it holds S.in_digit (cleared
// before, and left so if there are fewer), the rank among those S.left.  Whole workgroup; ends with a barrier.
__device__ __forceinline__ void find_digit(SelectShared& S, uint32_t rem) {
  const uint32_t digit = kSelectDigits - 1u - 2u * threadIdx.x;  // and the one below; larger digits first
  const uint32_t h0 = S.hist[digit], h1 = S.hist[digit - 1u];
  uint32_t total;
  const uint32_t above = block_excl_scan<kSelectWaves>(h0 + h1, S.scan_tmp, &total);
  if (above < rem && rem <= above + h0 + h1) {  // exactly one thread
    const bool second = rem > above + h0;
    S.digit = second ? digit - 1u : digit;
    S.left = rem - above - (second ? h0 : 0u);
    S.in_digit = second ? h1 : h0;
  }
  __syncthreads();
}

// Range of the keys that lie in a selection bin, into S.lo and S.hi.  Whole workgroup; ends with a barrier.
__device__ __forceinline__ void bin_keys(SelectShared& S, const ClientCtl* ctl, uint32_t bin) {
  static_assert(kMapBins <= kSelectBlock, "one entry per thread");
  const uint32_t anchor = ctl->anchor, t = threadIdx.x;
  if (bin < kOctaves || bin >= kOctaves + kFineBins) {
    if (t == 0) {
      const uint32_t octave = (bin < kOctaves ? bin : bin - (kOctaves + kFineBins)) << 23;
      S.lo = bin < kOctaves ? octave : max(octave, (anchor + kMapBins) << kSampleShift);
      S.hi = bin < kOctaves ? min(octave | 0x7FFFFFu, (anchor << kSampleShift) - 1u) : octave | 0x7FFFFFu;
    }
  } else if (t < kMapBins) {
    const uint32_t m = ctl->bin_map[t], first = m & 0xFFFFu, shift = m >> 16;
    if (bin >= first && bin - first < 1u << (kSampleShift - shift)) {  // exactly one thread
      S.lo = ((anchor + t) << kSampleShift) + ((bin - first) << shift);
      S.hi = S.lo + (1u << shift) - 1u;
    }
  }
  __syncthreads();
}

// The rem-th largest of the `count` candidates whose keys lie in bin `bin`, by going through the dense list, every
// wavefront an eighth of it: true with S.answer set, or false with at most kSelectList numbers in S.list, `count` and
// `rem` brought down to those.  A bin that holds a large part of all candidates holds equal keys as a rule: one of them, the
// first of 512 candidates spread over the list that lies in the range, is counted by itself, and where the boundary
// is among those no second pass is needed, only a search for its place by the wavefronts' counts.  Other keys are
// counted by the ten bits below the range's highest, equal ones of a row together, until the range is one key.
// 1 x 11.2 M of seven magnitudes, 45 % kept (6.4 M candidates, 1.6 M equal keys): 0.83 ms; 8.4 ms with two to four
// passes of 16 single loads a thread and an LDS atomic per key.
__device__ __forceinline__ bool search_candidates(SelectShared& S, const ClientCtl* ctl, const uint32_t* __restrict__ val,
                                                  uint32_t n, uint32_t bin, uint32_t& count, uint32_t& rem) {
  const uint32_t tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  bin_keys(S, ctl, bin);
  uint32_t lo = S.lo, hi = S.hi, tau = 0;
  bool counted = false;  // S.equal holds the wavefronts' counts of tau
  const uint32_t share = (n + kSelectBlock - 1u) / kSelectBlock * kWave;
  const uint32_t w_begin = min(wave * share, n), w_end = min(w_begin + share, n);
  while (true) {
    __syncthreads();  // the pass before is done with what is written below
    if (count <= kSelectList) {
      if (tid == 0) S.n_few = 0;
      __syncthreads();
      visit_keys(val, w_begin, w_end, [&](uint32_t i, uint32_t key, bool valid) {
        if (valid && key - lo <= hi - lo) {
          const uint32_t at = atomicAdd(&S.n_few, 1u);
          if (at < kSelectList) S.list[at] = member_of(i, key);  // always
        }
      });
      return false;
    }
    if (lo == hi) {
      tau = lo;
      break;
    }
    if (tid == 0) {
      S.digit = n;
      S.in_digit = 0;
      S.larger = 0;
    }
    S.hist[tid] = 0;
    S.hist[tid + kSelectBlock] = 0;
    __syncthreads();
    {
      const uint32_t i = (uint32_t)((uint64_t)tid * n / kSelectBlock);
      if ((val[i] & 0x7FFFFFFFu) - lo <= hi - lo) atomicMin(&S.digit, i);
    }
    __syncthreads();
    const uint32_t likely = S.digit < n ? val[S.digit] & 0x7FFFFFFFu : 0xFFFFFFFFu;
    const uint32_t bits = 32u - (uint32_t)__builtin_clz(hi - lo), shift = bits > 10u ? bits - 10u : 0u;
    uint32_t larger = 0, equal = 0;
    visit_keys(val, w_begin, w_end, [&](uint32_t, uint32_t key, bool valid) {
      const uint64_t same = __ballot(valid && key == likely);
      const bool other = valid && key != likely && key - lo <= hi - lo;
      equal += (uint32_t)__popcll(same);
      const uint64_t others = __ballot(other);
      if (!others) return;  // uniform
      larger += other && key > likely ? 1u : 0u;
      const uint32_t digit = (key - lo) >> shift, leader = (uint32_t)__builtin_ctzll(others);
      const uint32_t lead = __builtin_amdgcn_readlane(digit, leader);
      const uint64_t with_lead = __ballot(other && digit == lead);
      if (lane == leader) atomicAdd(&S.hist[lead], (uint32_t)__popcll(with_lead));
      else if (other && digit != lead) atomicAdd(&S.hist[digit], 1u);
    });
    larger = wave_sum_u32(larger);
    if (lane == 0) {
      if (larger) atomicAdd(&S.larger, larger);
      S.equal[wave] = equal;
    }
    __syncthreads();
    uint32_t equals = 0;
#pragma unroll
    for (uint32_t w = 0; w < kSelectWaves; ++w) equals += S.equal[w];
    if (S.larger < rem && rem <= S.larger + equals) {  // uniform
      tau = likely;
      rem -= S.larger;
      counted = true;
      break;
    }
    if (tid == 0 && equals) S.hist[(likely - lo) >> shift] += equals;
    __syncthreads();
    find_digit(S, rem);
    if (S.in_digit == 0) {  // uniform: fewer keys than the rank (cannot happen; reported by the caller)
      S.answer = ~0ull;
      return true;
    }
    lo += S.digit << shift;
    hi = min(hi, lo + ((1u << shift) - 1u));
    rem = S.left;
    count = S.in_digit;
  }
  // the rem-th candidate with key tau: which wavefront's share has it, again inside that share, and so on
  uint32_t begin = 0, end = n;
  while (end - begin > kWave) {  // uniform
    const uint32_t part = (end - begin + kSelectBlock - 1u) / kSelectBlock * kWave;
    if (!counted) {
      const uint32_t b = min(begin + wave * part, end), e = min(b + part, end);
      uint32_t equal = 0;
      visit_keys(val, b, e, [&](uint32_t, uint32_t key, bool valid) {
        equal += (uint32_t)__popcll(__ballot(valid && key == tau));
      });
      __syncthreads();  // the counts before have been read
      if (lane == 0) S.equal[wave] = equal;
      __syncthreads();
    }
    counted = false;
    uint32_t w = 0;
    while (w < kSelectWaves - 1u && rem > S.equal[w]) rem -= S.equal[w++];
    begin = min(begin + w * part, end);
    end = min(begin + part, end);
  }
  if (tid == 0) S.answer = ~0ull;
  __syncthreads();
  if (wave == 0) {
    const uint32_t i = begin + lane;
    const bool hit = i < end && (val[min(i, n - 1u)] & 0x7FFFFFFFu) == tau;
    const uint64_t hits = __ballot(hit);
    if (hit && lanes_below(hits) + 1u == rem) S.answer = member_of(i, tau);
  }
  __syncthreads();
  return true;
}

__global__ __launch_bounds__(kSelectBlock) void select_kernel(const ClientParams* __restrict__ params,
                                                              ClientCtl* __restrict__ ctls, Workspace ws) {
  __shared__ SelectShared S;
  const uint32_t r = blockIdx.x, client = blockIdx.y, tid = threadIdx.x, lane = lane_id(), wave = wave_id();
  const ClientParams& p = params[client];
  ClientCtl* ctl = ctls + client;
  // everything that is read from the control block is asked for together
  const uint32_t dead = ctl->dead, R = p.R, n_cand = ctl->n_cand;
  const uint32_t my_bin = tid < 32 ? ctl->sel_bin[tid] : kNoBin, my_rem = tid < 32 ? ctl->sel_rem[tid] : 0u;
  const uint32_t my_over = ctl->over_cnt[r];
  const MemberList l = ctl->list[r];
  const uint32_t blocks = gather_workgroups(ws, n_cand);
  auto seen_of = [&](uint32_t b) {
    return tid < blocks ? ws.seg_cnt[((size_t)client * kMemberSlots + b) * kGatherBlocksMax + tid] : 0u;
  };
  uint32_t seen = seen_of(r);
  if (dead || r >= R) return;  // uniform (dead: the workspace was too short for this client)
  if (tid < 32) {
    S.bin[tid] = my_bin;
    S.rem[tid] = my_rem;
  }
  __syncthreads();
  const uint32_t bin = S.bin[r];
  if (bin == kNoBin) return;
  uint32_t first = 0;  // the first boundary with this bin: the list is its
  while (S.bin[first] != bin) ++first;
  const bool listed = l.entries != 0, in_lds = !listed || l.members <= kSelectList;
  if (first != r && listed && in_lds) return;  // uniform: served by the workgroup of that boundary
  GlobalU64Ptr entries = (GlobalU64Ptr)l.entries;
  uint32_t m = 0, in_segs = 0;
  bool found = false;
  if (!listed) {
    uint32_t rem = S.rem[r];
    m = l.members;
    found = search_candidates(S, ctl, ws.dense_val + (size_t)client * ws.dense_cap, n_cand, bin, m, rem);
    if (tid == 0) S.rem[r] = rem;
  } else {
    uint32_t over = my_over;
    if (first != r) {  // the gather filled the list of the bin's first boundary
      entries = (GlobalU64Ptr)ctl->list[first].entries;
      seen = seen_of(first);
      over = ctl->over_cnt[first];
    }
    if (tid < kWave) {
      static_assert(kGatherBlocksMax <= kWave, "one lane per piece of a member list");
      const uint32_t here = min(seen, l.cap), incl = wave_incl_scan_u32(here);
      S.seg_first[tid] = incl - here;
      if (tid == kWave - 1u) S.seg_first[kWave] = incl;
    }
    __syncthreads();
    in_segs = S.seg_first[kWave];
    m = in_segs + min(over, l.over_room);
    if (in_lds) {
      m = min(m, kSelectList);  // m = l.members, no more than that
      for (uint32_t e = tid; e < m; e += kSelectBlock) {
        uint32_t at = l.over_first + e - in_segs;
        if (e < in_segs) {  // a thread finds its member's piece by the pieces' first places: six probes
          uint32_t s = 0;
#pragma unroll
          for (uint32_t step = kWave / 2u; step; step >>= 1)
            if (S.seg_first[s + step] <= e) s += step;
          at = s * l.cap + e - S.seg_first[s];
        }
        S.list[e] = entries[at];
      }
    }
  }
  auto each_member = [&](auto visit) {
    if (in_lds) {
      for (uint32_t e = tid; e < m; e += kSelectBlock) visit(S.list[e]);
    } else {
      // a wavefront takes piece after piece, then all of them go through what lies behind the pieces; eight rows are
      // asked for together
      constexpr uint32_t kRows = 8;
      auto visit_run = [&](uint32_t at, uint32_t count, uint32_t begin, uint32_t step) {
        for (uint32_t base = begin; base < count; base += step) {
          unsigned long long c[kRows];
#pragma unroll
          for (uint32_t u = 0; u < kRows; ++u) c[u] = entries[at + min(base + u * kWave + lane, count - 1u)];
#pragma unroll
          for (uint32_t u = 0; u < kRows; ++u)
            if (base + u * kWave + lane < count) visit(c[u]);
        }
      };
      for (uint32_t s = wave; s < blocks; s += kSelectWaves)
        visit_run(s * l.cap, S.seg_first[s + 1u] - S.seg_first[s], 0u, kRows * kWave);
      visit_run(l.over_first, m - in_segs, wave * kRows * kWave, kSelectWaves * kRows * kWave);
    }
  };
  const uint32_t b_end = listed && in_lds ? R : r + 1u;
  for (uint32_t b = r; b < b_end; ++b) {
    if (S.bin[b] != bin) continue;  // uniform
    __syncthreads();  // the list, and the rank that search_candidates leaves
    uint32_t rem = S.rem[b];
    unsigned long long prefix = 0;  // members at hand: those whose bits from `known` up are `prefix`
    uint32_t known = 63;            // keys have 31 bits
    while (!found && known != 0u) {  // no two members are alike: one is left at bit 0 at the latest
      __syncthreads();  // the round before is done with what is written below
      if (tid == 0) {
        S.min = ~0ull;
        S.max = 0;
        S.in_digit = 0;
        S.n_few = 0;
        S.answer = ~0ull;
      }
      S.hist[tid] = 0;
      S.hist[tid + kSelectBlock] = 0;
      __syncthreads();
      unsigned long long lo = ~0ull, hi = 0;
      each_member([&](unsigned long long c) {
        if ((c >> known) != prefix) return;
        lo = c < lo ? c : lo;
        hi = c > hi ? c : hi;
      });
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long lo2 = __shfl_xor(lo, o, 64), hi2 = __shfl_xor(hi, o, 64);
        lo = lo2 < lo ? lo2 : lo;
        hi = hi2 > hi ? hi2 : hi;
      }
      if (lane == 0 && lo <= hi) {
        atomicMin(&S.min, lo);
        atomicMax(&S.max, hi);
      }
      __syncthreads();
      lo = S.min;
      hi = S.max;
      if (lo > hi) break;  // uniform: no member at hand (cannot happen; reported below)
      const uint32_t top_bit = lo == hi ? 0u : 63u - (uint32_t)__builtin_clzll(lo ^ hi);
      const uint32_t shift = top_bit > 9u ? top_bit - 9u : 0u;
      each_member([&](unsigned long long c) {
        if ((c >> known) == prefix) atomicAdd(&S.hist[(uint32_t)(c >> shift) & (kSelectDigits - 1u)], 1u);
      });
      __syncthreads();
      find_digit(S, rem);
      if (S.in_digit == 0) break;  // uniform: fewer members than the rank (cannot happen; reported below)
      prefix = ((lo >> shift) & ~(unsigned long long)(kSelectDigits - 1u)) | S.digit;  // the bits above the digit are common to all
      known = shift;
      rem = S.left;
      if (S.in_digit <= kWave) {
        each_member([&](unsigned long long c) {
          if ((c >> known) == prefix) S.few[atomicAdd(&S.n_few, 1u)] = c;
        });
        __syncthreads();
        if (wave == 0) {
          const uint32_t n = S.in_digit;
          const unsigned long long mine = lane < n ? S.few[lane] : 0ull;
          uint32_t before = 0;
          for (uint32_t o = 0; o < n; ++o) before += S.few[o] > mine ? 1u : 0u;
          if (lane < n && before + 1u == rem) S.answer = mine;
        }
        __syncthreads();
        break;
      }
    }
    if (tid == 0) {
      if (S.answer == ~0ull) {
        atomicOr(ws.status, CVLC_DEV_INTERNAL);
      } else {
        ctl->tau[b] = (uint32_t)(S.answer >> 32);
        ctl->iota[b] = ~(uint32_t)S.answer;
      }
    }
  }
}

// ------------------------------------------------------------------ 4b. short vectors: the whole selection in one workgroup
// What the seven launches before this find for a long vector one workgroup per client finds for a short one
// (cvlc_select.h): exact keys of all boundaries, and where a boundary cuts a class of equal keys the position
// of the last one inside.  There are no candidates: the counting and packing passes go through the vector itself, a
// coordinate's number is its position.  The kernel also puts the client's parameters and control block in place.
// Latency, and the instructions that one CU issues for every coordinate (1 x 65 536, three groups: 21 us, of which the first count
// takes 6.5 and setting the boundaries' bins aside 8).

// The parameters come as kernel arguments, or have been uploaded before (batches of many different plans).
struct ParamsUploaded {
  const ClientParams* params;
};
__device__ __forceinline__ uint32_t short_client(const UploadChunk& c) { return c.first_client + blockIdx.x; }
__device__ __forceinline__ uint32_t short_client(const ParamsUploaded&) { return blockIdx.x; }
__device__ __forceinline__ uint32_t short_param(const UploadChunk& c, uint32_t w) { return param_word(c, blockIdx.x, w); }
__device__ __forceinline__ uint32_t short_param(const ParamsUploaded& u, uint32_t w) {
  return reinterpret_cast<const uint32_t*>(u.params + blockIdx.x)[w];
}

// Whether a vector would have more candidates than the caller's workspace has room for (`room` < d): what the
// general path refuses is refused here too.  Its candidates are the keys at or above the lower edge of the 13-bit bin that
// holds the sample's rank-th largest key, and the sample of a short vector is all of it but the last d mod kSamplePiece
// coordinates.  So that key lies between the vector's rank-th and (rank + missing)-th (the extra rank).  Whole
// workgroup, after locate_short; leaves S.top and S.upto as they were.
static_assert(kSampleShift == kTopShift + 1u && kShortMax <= kSampleChunksMax * kSamplePiece, "two bins to a sample bin, all pieces sampled");
__device__ __forceinline__ uint32_t short_missing(uint32_t d) { return d % kSamplePiece; }
__device__ __forceinline__ bool short_of_room(EncodeSelect& S, const float* update, uint32_t d, uint32_t room, uint32_t rank) {
  if (rank == 0u) return true;  // no threshold: all d are candidates
  const uint32_t missing = short_missing(d);
  const uint32_t upto = S.extra - S.extra_rem + S.top[S.extra_bin] + ((S.extra_bin & 1u) ? S.top[S.extra_bin - 1u] : 0u);
  if (upto <= room || missing == 0u) return upto > room;  // uniform
  // next to never: the counts without the last coordinates decide
  auto last_ones = [&](uint32_t by) {
    __syncthreads();
    if (threadIdx.x < missing) atomicAdd(&S.top[(__float_as_uint(((ShortFloatPtr)update)[d - missing + threadIdx.x]) & 0x7FFFFFFFu) >> kTopShift], by);
    __syncthreads();
  };
  last_ones(~0u);
  constexpr uint32_t kBins = kTopBins / kShortBlock;
  const uint32_t largest = kTopBins - 1u - kBins * threadIdx.x;
  uint32_t mine = 0, total;
  for (uint32_t i = 0; i < kBins; ++i) mine += S.top[largest - i];
  uint32_t above = block_excl_scan<kShortWaves>(mine, S.scan_tmp, &total);
  if (above < rank && rank <= above + mine) {  // one thread
    uint32_t bin = largest + 1u;
    while (above < rank) {
      bin -= 2u;
      above += S.top[bin] + S.top[bin + 1u];
    }
    S.extra_bin = bin;
  }
  last_ones(1u);
  const uint32_t from = S.extra_bin, t = (kTopBins - 1u - from) / kBins;
  uint32_t all = t ? S.upto[t - 1u] : 0u;
  for (uint32_t b = from; b < kTopBins - kBins * t; ++b) all += S.top[b];
  return all > room;
}

static_assert(sizeof(UploadChunk) + sizeof(Workspace) + 4u * sizeof(void*) <= 4096, "kernel arguments are limited to 4 KB");
template <class Params>
__global__ __launch_bounds__(kShortBlock) void short_select_kernel(Params source, ClientParams* params, ClientCtl* ctls, Workspace ws,
                                                                   cvlc_seg_stats_t* stats_out, uint32_t first_launch) {
  __shared__ EncodeSelect S;
  __shared__ uint32_t s_params[kParamWords];
  const uint32_t client = short_client(source), tid = threadIdx.x;
  const uint32_t d = ws.d;
  ClientCtl* ctl = ctls + client;
  if (tid < kParamWords) {
    const uint32_t word = short_param(source, tid);
    s_params[tid] = word;
    reinterpret_cast<uint32_t*>(params + client)[tid] = word;
  }
  if (first_launch && blockIdx.x == 0 && tid == 0) *ws.status = 0u;  // this kernel reports through ctl->flags
  clear_short(S);
  __syncthreads();
  const ClientParams& p = *reinterpret_cast<const ClientParams*>(s_params);
  const uint32_t R = p.R;
  const float* update = p.update;
  if (tid < R) S.rank[tid] = p.Z[tid];  // (cleared by the same thread)
  const bool check_room = ws.dense_cap < d;
  if (tid == 0) {
    S.n_ranks = R;
    S.extra = check_room && p.sample_rank ? p.sample_rank + short_missing(d) : 0u;
  }
  count_top(S, update, d);
  // the control block, as far as the later kernels read it, and what this kernel counts in
  static_assert(sizeof(SegPartial) * kSegCopies == kShortBlock * 4u, "a word per thread");
  reinterpret_cast<uint32_t*>(ctl->seg)[tid] = 0;
  for (uint32_t i = tid; i < 32u * kNormLimbs; i += kShortBlock) ws.norm_limbs[(size_t)client * 32u * kNormLimbs + i] = 0;
  const uint32_t flags = tid < kTopBins - (0x7F800000u >> kTopShift) ? S.top[(0x7F800000u >> kTopShift) + tid] : 0u;
  locate_short(S);
  const bool dead = check_room && short_of_room(S, update, d, ws.dense_cap, p.sample_rank);  // uniform
  const uint64_t flagged = __ballot(flags != 0u);  // the first wavefront looks at the bins of Inf and NaN
  static_assert(kTopBins - (0x7F800000u >> kTopShift) <= kWave, "a bin per lane");
  if (tid == 0) {
    ctl->n_cand = d;
    ctl->dead = dead ? 1u : 0u;
    ctl->flags = (flagged ? CVLC_DEV_NONFINITE : 0u) | (dead ? CVLC_DEV_WORKSPACE : 0u);
    ctl->emit_claim = 0;
    if (dead) p.stream[0] = 0u;  // not a stream header
  }
  if (dead) return;  // a refused client's statistics are not touched
  if (stats_out && tid < R) stats_out[(size_t)client * kStatsStride + tid].errsq = 0.0;  // the pack kernel adds to it when asked to
  select_short(S, update, d);
  if (tid < 32u) {
    const bool none = tid >= R || S.rank[tid] == 0u;
    ctl->tau[tid] = none ? 0xFFFFFFFFu : S.prefix[tid];
    if (none || S.rem[tid] == S.equal[tid]) ctl->iota[tid] = none ? 0u : 0xFFFFFFFFu;  // the whole class is inside
  }
  visit_ties(S, update, d, [&](uint32_t r, uint32_t at) {
    if (r < R) ctl->iota[r] = at;
  });
}

// ------------------------------------------------------------------ 5. classification of the candidates
struct Thresholds {  // group boundaries in LDS
  uint32_t tau[32];
  uint32_t iota[32];
  uint32_t cut[32];  // key < cut[r]  <=>  key <= tau[r] for r < R; 0 (never) for r >= R
  uint32_t above[33];  // the boundary key just above group g: tau[g - 1]; no key (all ones) above group 0
};

__device__ __forceinline__ void load_thresholds(Thresholds& t, const ClientCtl* ctl, uint32_t R) {
  if (threadIdx.x < 32) {
    const bool live = threadIdx.x < R;
    const uint32_t tau = live ? ctl->tau[threadIdx.x] : 0xFFFFFFFFu;
    t.tau[threadIdx.x] = tau;
    t.iota[threadIdx.x] = live ? ctl->iota[threadIdx.x] : 0u;
    t.cut[threadIdx.x] = live ? (tau == 0xFFFFFFFFu ? tau : tau + 1u) : 0u;  // keys stay below 2^31
    t.above[threadIdx.x + 1] = tau;
    if (threadIdx.x == 0) t.above[0] = 0xFFFFFFFFu;
  }
}

// Group of a candidate, 0-based: the first boundary r whose top-Z_r set holds
// it (key above tau_r, or equal and not after candidate iota_r); R if none (dropped).
// tau is non-increasing in r, so "key <= tau_r" holds for the first g boundaries
// and for no later one, g being the number of boundaries with tau_r >= key: a
// binary search over the boundaries (entries past R never hold) finds it in
// log2 R probes per candidate.  The position is only needed (and only read)
// when the key equals a boundary key.
template <uint32_t N>
__device__ __forceinline__ void classify_keys(const Thresholds& t, uint32_t R, const uint32_t (&key)[N],
                                              uint32_t (&grp)[N]) {
#pragma unroll
  for (uint32_t j = 0; j < N; ++j) grp[j] = 0;
  // largest power of two <= R: the probes reach entry 2 * top - 2 <= 30 at most, the result 2 * top - 1 >= R
  for (uint32_t step = R ? 1u << (31 - __builtin_clz(R)) : 0u; step; step >>= 1) {
    uint32_t probe[N];  // all N reads of a step before the first comparison: one LDS round trip per step
#pragma unroll
    for (uint32_t j = 0; j < N; ++j) probe[j] = t.cut[grp[j] + step - 1u];
#pragma unroll
    for (uint32_t j = 0; j < N; ++j) grp[j] += key[j] < probe[j] ? step : 0u;
  }
}

// Second step for a key that equals the boundary key just above its group:
// boundaries with that key decide by position, i.e. by the candidate's number
// in the position-ordered list against that of the last member inside.
__device__ __forceinline__ uint32_t classify_tie(const Thresholds& t, uint32_t key, uint32_t g, uint32_t dense_i) {
  while (g > 0 && t.tau[g - 1] == key && dense_i <= t.iota[g - 1]) --g;
  return g;
}

// Lanes that hold a candidate of the caller's group (group ids below 2^ID_BITS); lanes
// with g == kNoGroup match nobody.  Must be reached by the whole wavefront.
// Per bit of the id: the lanes that have it set, against an all-ones / all-zeros word of the
// caller's own bit; what differs in any bit is not the caller's group.
template <uint32_t ID_BITS>
__device__ __forceinline__ uint64_t same_group_lanes(uint32_t g) {
  const uint64_t coded = __ballot(g != kNoGroup);
  uint32_t differ_lo = 0, differ_hi = 0;
#pragma unroll
  for (uint32_t bit = 0; bit < ID_BITS; ++bit) {
    const uint32_t mine = (uint32_t)__builtin_amdgcn_sbfe((int32_t)g, bit, 1u);  // the bit, sign-extended
    const uint64_t set = __ballot(mine != 0u);
    differ_lo |= (uint32_t)set ^ mine;
    differ_hi |= (uint32_t)(set >> 32) ^ mine;
  }
  return coded & ~(((uint64_t)differ_hi << 32) | differ_lo);
}

// Loads span `span` of the dense list (kPerLane candidates per lane, row j at
// span*512 + j*64 + lane, i.e. in position order).  No branch around the loads (a lane past
// the end reads the last candidate again): all eight are in flight before the first is waited for.
__device__ __forceinline__ void load_span(const uint32_t* __restrict__ list, uint32_t n, uint32_t span,
                                          uint32_t (&out)[kPerLane]) {
  const uint32_t mine = span * kSpan + lane_id();
#pragma unroll
  for (uint32_t j = 0; j < kPerLane; ++j) out[j] = list[min(mine + j * kWave, n - 1u)];
}

// Classifies the loaded value bits of span `span`; grp[j] = kNoGroup past the end of the list.
__device__ __forceinline__ void classify_loaded(const Thresholds& thr, uint32_t R, uint32_t n, uint32_t span,
                                                const uint32_t (&v)[kPerLane], uint32_t (&grp)[kPerLane]) {
  const uint32_t mine = span * kSpan + lane_id();
  uint32_t key[kPerLane];
#pragma unroll
  for (uint32_t j = 0; j < kPerLane; ++j) key[j] = v[j] & 0x7FFFFFFFu;
  classify_keys<kPerLane>(thr, R, key, grp);
  // the boundary key just above every candidate's group, all eight read before the first is looked at:
  // only a key that equals it (next to none) goes on to the tie rule
  uint32_t above[kPerLane];
#pragma unroll
  for (uint32_t j = 0; j < kPerLane; ++j) above[j] = thr.above[grp[j]];
#pragma unroll
  for (uint32_t j = 0; j < kPerLane; ++j) {
    const uint32_t i = mine + j * kWave;
    uint32_t g = grp[j];
    if (above[j] == key[j]) g = classify_tie(thr, key[j], g, i);
    grp[j] = i < n ? g : kNoGroup;
  }
}

// ------------------------------------------------------------------ 6. group counts and statistics
// QSGD's header carries the group's l2-norm, and the stream must not depend on
// the order squares are added in: the sum of squares is kept exactly, as a
// fixed-point number in units of 2^-298 (the square of the smallest denormal)
// spread over 32-bit limbs, each limb summed in a 64-bit counter of its own.
// x = m * 2^(q - 149) with m < 2^24, so x^2 = m^2 << 2q: three limbs from 2q / 32.
struct SquareLimbs {
  uint32_t word;     // first limb
  uint32_t part[3];  // the pieces of m^2 << (2q mod 32), each below 2^32
};
__device__ __forceinline__ SquareLimbs square_limbs(uint32_t value_bits) {
  const uint32_t b = value_bits & 0x7FFFFFFFu, e = b >> 23, frac = b & 0x7FFFFFu;
  const uint64_t m = e ? (frac | 0x800000u) : frac;
  const uint32_t off = 2u * (e ? e - 1u : 0u), sh = off & 31u;
  const uint64_t sq = m * m, low = sq << sh;  // the top bits that leave `low` are part[2]
  SquareLimbs r;
  r.word = off >> 5;
  r.part[0] = (uint32_t)low;
  r.part[1] = (uint32_t)(low >> 32);
  r.part[2] = sh ? (uint32_t)(sq >> (64u - sh)) : 0u;
  return r;
}

// What the counting pass leaves for the packing pass, 16 bits per candidate of the dense list: its group
// (5 bits) and above it its number among the members of that group in its span of 512 (9 bits); kNoPlace
// for a dropped candidate.  The array takes the place of the filter's region-slot positions, which nothing
// reads once the gather has run (d entries per client, the dense list has at most as many).
constexpr uint32_t kPlaceShift = 5;
constexpr uint16_t kNoPlace = 0xFFFFu;
__device__ __forceinline__ uint16_t* span_places(const Workspace& ws, uint32_t client) {
  return ws.cand_idx + (size_t)client * ws.d;
}

// What the counting and the packing pass work on, and where a record's number inside its group comes from.
enum PassMode {
  kByLayout,  // dense candidates; the layout kernel turns the spans' counts into prefixes
  kByChunks,  // dense candidates; the counting pass also leaves every chunk's counts, from which a packing workgroup makes the prefixes it needs
  kShortVec,  // a short vector's coordinates; a packing workgroup adds up the spans' counts
};

// kByChunks: members of every group in every chunk of eight spans, 32 words a chunk, in the place of the region slots' values,
// which nothing reads once the boundaries are found (a chunk has 4096 candidates, a client d entries).
__device__ __forceinline__ uint32_t* chunk_totals(const Workspace& ws, uint32_t client) { return ws.cand_val + (size_t)client * ws.d; }
static_assert(kSpan * kChunkSpans >= 32u, "a chunk's counts take no more room than its candidates");
constexpr uint32_t kChunkSets = 16;  // chunks whose counts a counting workgroup holds in LDS

constexpr uint32_t kLimbBanks = 2;  // copies of a workgroup's limb counters, to thin out colliding LDS atomics

// Every wavefront takes spans of 512 candidates (gw, gw + wavefronts, ...) and
// writes, per span, the number of members of every group and, per candidate,
// its group and its number among the span's members of that group (together
// with the layout's prefix over the spans: its record's place in the stream;
// the packing pass neither classifies nor counts again).  Min, max and sum of
// squares of the groups go to LDS
// columns private to a lane id, so that the LDS atomics of one instruction never
// collide; they are reduced once at the end.  Wavefronts do not wait for each
// other before that.
// QSGD: also the exact sum of squares of every group (see above).
// kShortVec: the coordinates of a short vector take the candidates' place (short_select_kernel); most may be dropped, so
// those are neither numbered nor kept in the columns, their energy stays in a register.
// Without a layout kernel the pass also clears the stream, whose words the packing pass ORs into (45 MB of 32 x 11.2 M: 4 us;
// by workgroups of their own in the selection's launch, which leaves the memory idle: 8).
// kByChunks: a workgroup's eight wavefronts are on the eight spans of a chunk; the chunk's counts add up in LDS.
template <bool QSGD, PassMode MODE>
__global__ __launch_bounds__(kEmitBlock) void count_kernel(const ClientParams* __restrict__ params,
                                                           ClientCtl* __restrict__ ctls, Workspace ws,
                                                           cvlc_seg_stats_t* __restrict__ stats_out) {
  constexpr bool SHORT = MODE == kShortVec, CHUNKS = MODE == kByChunks;
  __shared__ Thresholds thr;
  __shared__ unsigned long long s_limb[QSGD ? kLimbBanks : 1][QSGD ? 32 : 1][kNormLimbs];  // bank = lane mod kLimbBanks
  __shared__ uint32_t s_max[33][kWave], s_negmin[33][kWave];
  __shared__ double s_sq[33][kWave];
  __shared__ uint32_t s_cnt[kEmitWaves][32];
  __shared__ uint32_t s_chunk[CHUNKS ? kChunkSets : 1u][32];
  const uint32_t client = blockIdx.y, tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const ClientParams& p = params[client];
  ClientCtl* ctl = ctls + client;
  if (ctl->dead) return;  // the workspace was too short for this client (whole workgroup)
  const uint32_t R = p.R, n = ctl->n_cand;
  const uint32_t n_spans = (n + kSpan - 1) / kSpan;
  const uint32_t* __restrict__ val = SHORT ? (const uint32_t*)(GlobalConstWordPtr)p.update : ws.dense_val + (size_t)client * ws.dense_cap;
  uint32_t* __restrict__ span_cnt = ws.span_cnt + (size_t)client * (ws.max_spans + 1) * 32;
  if (SHORT || CHUNKS)
    for (uint32_t i = blockIdx.x * kEmitBlock + tid; i < p.total_words; i += gridDim.x * kEmitBlock) ((GlobalWordPtr)p.stream)[i] = 0;
  if (CHUNKS) {
    if (stats_out && blockIdx.x == 0 && tid < R) stats_out[(size_t)client * kStatsStride + tid].errsq = 0.0;  // the pack kernel adds to it when asked to
    static_assert(kChunkSets * 32u == kEmitBlock, "a counter per thread");
    (&s_chunk[0][0])[tid] = 0;
  }
  load_thresholds(thr, ctl, R);
  if (tid < kEmitWaves * 32) (&s_cnt[0][0])[tid] = 0;
  for (uint32_t i = tid; i < 33 * kWave; i += kEmitBlock) {
    (&s_max[0][0])[i] = 0;
    (&s_negmin[0][0])[i] = 0;
    (&s_sq[0][0])[i] = 0.0;
  }
  if (QSGD)
    for (uint32_t i = tid; i < kLimbBanks * 32 * kNormLimbs; i += kEmitBlock) (&s_limb[0][0][0])[i] = 0;
  __syncthreads();
  uint16_t* __restrict__ place = span_places(ws, client);
  uint32_t* running = s_cnt[wave];  // members of every group (the dropped ones last) in the rows so far
  const uint32_t span_step = gridDim.x * kEmitWaves;
  double tail = 0.0;  // SHORT: energy of the dropped
  // kByChunks: the counts of the workgroup's chunks `first` .. `last` - 1 (its t-th chunk is blockIdx.x + t * gridDim.x)
  auto write_chunks = [&](uint32_t first, uint32_t last) {
    const uint32_t t = first + tid / 32u;
    if (t < last) chunk_totals(ws, client)[(size_t)(blockIdx.x + t * gridDim.x) * 32u + tid % 32u] = (&s_chunk[0][0])[tid];
  };
  uint32_t turn = 0;  // ... and the one at hand; wavefronts past the last span have an empty turn, so that all meet every kChunkSets turns
  uint32_t ahead[kPerLane];  // the next span's value bits, asked for before the current span is worked on
  if (blockIdx.x * kEmitWaves + wave < n_spans) load_span(val, n, blockIdx.x * kEmitWaves + wave, ahead);
  for (uint32_t span = blockIdx.x * kEmitWaves + wave; CHUNKS ? span - wave < n_spans : span < n_spans; span += span_step) {
    if (CHUNKS) {
      if (turn && turn % kChunkSets == 0u) {  // uniform over the workgroup
        __syncthreads();
        write_chunks(turn - kChunkSets, turn);
        (&s_chunk[0][0])[tid] = 0;  // the same thread's counter
        __syncthreads();
      }
      ++turn;
      if (span >= n_spans) continue;
    }
    uint32_t v[kPerLane], grp[kPerLane];
#pragma unroll
    for (uint32_t j = 0; j < kPerLane; ++j) v[j] = ahead[j];
    if (span + span_step < n_spans) load_span(val, n, span + span_step, ahead);
    classify_loaded(thr, R, n, span, v, grp);
    if (SHORT) {
#pragma unroll
      for (uint32_t j = 0; j < kPerLane; ++j) {
        const double x = grp[j] == R ? (double)__uint_as_float(v[j]) : 0.0;
        tail = fma(x, x, tail);
        if (grp[j] == R) grp[j] = kNoGroup;
      }
    }
    // Every candidate's number among the span's members of its group (row after row, lanes in order): a
    // row's members of a group read the group's running number and the lowest of them adds the row's
    // members to it.  This wavefront alone touches the counters and its LDS accesses complete in the order
    // they are issued, so no row waits for the one before.  What the counters hold after the last row are
    // the span's group sizes.
    uint32_t start[kPerLane], below[kPerLane];
    auto number_rows = [&](auto id_bits) {
#pragma unroll
      for (uint32_t j = 0; j < kPerLane; ++j) {
        start[j] = below[j] = 0;
        if (SHORT && !__ballot(grp[j] != kNoGroup)) continue;  // uniform
        const uint64_t same = same_group_lanes<decltype(id_bits)::value>(grp[j]);
        below[j] = lanes_below(same);
        if (grp[j] != kNoGroup) {
          start[j] = running[grp[j]];
          if (below[j] == 0) atomicAdd(&running[grp[j]], (uint32_t)__popcll(same));
        }
        asm volatile("" ::: "memory");  // the rows' LDS accesses stay in this order; nothing to wait for
      }
    };
    if (R < 8u) number_rows(std::integral_constant<uint32_t, 3>());  // ids 0 .. R, R for the dropped
    else if (R < 16u) number_rows(std::integral_constant<uint32_t, 4>());
    else number_rows(std::integral_constant<uint32_t, 5>());
#pragma unroll
    for (uint32_t j = 0; j < kPerLane; ++j) {
      const uint32_t i = span * kSpan + j * kWave + lane;
      if (i < n) place[i] = grp[j] < R ? (uint16_t)(grp[j] | ((start[j] + below[j]) << kPlaceShift)) : kNoPlace;
    }
    wave_lds_fence();
    if (lane < 32) {
      const uint32_t members = running[lane];
      span_cnt[(size_t)span * 32 + lane] = members;
      running[lane] = 0;
      if (CHUNKS) atomicAdd(&s_chunk[(turn - 1u) % kChunkSets][lane], members);
    }
    wave_lds_fence();
#pragma unroll
    for (uint32_t j = 0; j < kPerLane; ++j) {
      const uint32_t g = grp[j];
      if (g != kNoGroup) {
        const float x = __uint_as_float(v[j]);
        const uint32_t o = ordered_bits(x);
        atomicMax(&s_max[g][lane], o);
        atomicMax(&s_negmin[g][lane], ~o);
        atomicAdd(&s_sq[g][lane], (double)x * (double)x);
        if (QSGD && g < R) {
          const SquareLimbs sl = square_limbs(v[j]);  // word + 2 <= 17
          unsigned long long* mine = s_limb[lane % kLimbBanks][g] + sl.word;
          atomicAdd(mine, (unsigned long long)sl.part[0]);
          if (sl.part[1]) atomicAdd(mine + 1, (unsigned long long)sl.part[1]);
          if (sl.part[2]) atomicAdd(mine + 2, (unsigned long long)sl.part[2]);
        }
      }
    }
  }
  if (SHORT) {
    tail = wave_sum_f64(tail);
    if (lane == 0) atomicAdd(&ctl->seg[blockIdx.x % kSegCopies].sumsq[R], tail);
  }
  __syncthreads();
  if (CHUNKS && turn) write_chunks((turn - 1u) / kChunkSets * kChunkSets, turn);
  if (QSGD) {  // a workgroup sees fewer than 2^31 candidates, so no counter has wrapped
    unsigned long long* dst = ws.norm_limbs + (size_t)client * 32 * kNormLimbs;
    for (uint32_t i = tid; i < R * kNormLimbs; i += kEmitBlock) {
      unsigned long long t = 0;
      for (uint32_t b = 0; b < kLimbBanks; ++b) t += (&s_limb[b][0][0])[i];
      if (t) atomicAdd(&dst[i], t);
    }
  }
  // group g's columns are reduced by wavefront g mod 8; finite values never code to 0, so 0 = no member here
  for (uint32_t g = wave; SHORT ? g < R : g <= R; g += kEmitWaves) {
    const uint32_t mx = wave_max_u32(s_max[g][lane]);
    const uint32_t ng = wave_max_u32(s_negmin[g][lane]);
    const double sq = wave_sum_f64(s_sq[g][lane]);
    if (lane == 0 && mx != 0) {
      SegPartial* part = &ctl->seg[blockIdx.x % kSegCopies];
      atomicMax(&part->max_enc[g], mx);
      atomicMax(&part->negmin_enc[g], ng);
      atomicAdd(&part->sumsq[g], sq);
    }
  }
}

// ------------------------------------------------------------------ 7. layout: prefix, headers, statistics
// What the packing pass and the headers need to know of a group.
struct GroupValues {
  uint32_t P, y;
  float m, M, norm;    // smallest and largest value; QSGD: the l2-norm of the header
  float low, inv, step;  // first centroid, reciprocal spacing and spacing of the centroids
};

// One thread per group.  P, y: its size and code length (read from the parameters well before: a load in the middle of this
// is half a microsecond of a small call); enc_max, enc_negmin: as the counting pass leaves them; limbs: QSGD, the group's exact sum of
// squares in 64-bit counters; sum: room for it in LDS.  Status bits go to *flags.
__device__ __forceinline__ GroupValues group_values(uint32_t P, uint32_t y, uint32_t enc_max, uint32_t enc_negmin, uint32_t quant,
                                                    const unsigned long long* limbs, uint32_t (&sum)[kNormLimbs], uint32_t* flags) {
  GroupValues v;
  v.P = P;
  v.y = y;
  v.m = v.M = v.norm = 0.0f;
  if (v.P > 0 && enc_max != 0) {
    v.M = from_ordered_bits(enc_max);
    v.m = from_ordered_bits(~enc_negmin);
  } else if (v.P > 0) {
    *flags |= CVLC_DEV_INTERNAL;
  }
  if (!(fabsf(v.M - v.m) <= 3.4028234664e38f)) *flags |= CVLC_DEV_NONFINITE;
  if (quant == CVLC_QUANT_QSGD) {
    // carry the 64-bit counters into 32-bit limbs, then look for the smallest fp32 value whose
    // square reaches the sum: squares grow with the bit pattern, so a binary search over it
    unsigned long long carry = 0;
    int top = -1;  // highest limb that is not zero
    for (uint32_t i = 0; i < kNormLimbs; ++i) {
      const unsigned long long t = limbs[i] + carry;
      sum[i] = (uint32_t)t;
      if ((uint32_t)t) top = (int)i;
      carry = t >> 32;
    }
    auto reaches = [&](uint32_t key) {  // key^2 >= sum, compared limb by limb from the top
      const SquareLimbs sl = square_limbs(key);
      const int from = max(top, (int)sl.word + 2);
      for (int i = from; i >= 0; --i) {
        const uint32_t j = (uint32_t)i - sl.word;  // wraps to a large value below sl.word
        const uint32_t mine = j == 0u ? sl.part[0] : (j == 1u ? sl.part[1] : (j == 2u ? sl.part[2] : 0u));
        const uint32_t theirs = sum[i];
        if (mine != theirs) return mine > theirs;
      }
      return true;
    };
    uint32_t lo = 0, hi = 0x7F7FFFFFu;
    if (!reaches(hi)) {
      *flags |= CVLC_DEV_NONFINITE;  // the norm overflows fp32
      lo = hi;
    } else if (top >= 0) {
      // a floating-point estimate from the three top limbs brackets the answer within a few
      // patterns; the exact comparison decides, and the full range stays as the fallback
      double head = (double)sum[top];
      if (top >= 1) head = head * 4294967296.0 + (double)sum[top - 1];
      if (top >= 2) head = head * 4294967296.0 + (double)sum[top - 2];
      const float guess = (float)sqrt(ldexp(head, 32 * (top - (top >= 2 ? 2 : top)) - 298));
      const uint32_t g = min(__float_as_uint(guess), 0x7F7FFFFFu);
      const uint32_t glo = g > 2u ? g - 2u : 0u, ghi = g < 0x7F7FFFFDu ? g + 2u : 0x7F7FFFFFu;
      if (reaches(ghi) && (glo == 0u || !reaches(glo - 1u))) {
        lo = glo;
        hi = ghi;
      }
    } else {
      hi = 0;  // an all-zero group
    }
    while (lo < hi) {
      const uint32_t mid = lo + (hi - lo) / 2u;
      if (reaches(mid)) hi = mid; else lo = mid + 1u;
    }
    v.norm = __uint_as_float(lo);
  }
  if (quant == CVLC_QUANT_QSGD) {  // levels 0 .. s on [0, norm]: the same spacing rule with s = 2^(y-1) - 1 steps
    centroid_spacing(0.0f, v.norm, y == 32 ? 1u : y - 1u, &v.step, &v.inv);
    v.low = 0.0f;
  } else {
    centroid_spacing(v.m, v.M, y == 32 ? 1u : y, &v.step, &v.inv);
    v.low = v.m;
  }
  return v;
}

// A group's header, and its statistics but for the error energy, which the packing pass adds to.
__device__ __forceinline__ void write_group(const ClientParams& p, uint32_t client, uint32_t r, const GroupValues& v, double sumsq, uint32_t quant,
                                            cvlc_seg_stats_t* stats_out) {
  GlobalWordPtr hdr = (GlobalWordPtr)p.stream + kGlobalHeaderWords + kSegHeaderWords * r;
  hdr[0] = v.y;
  hdr[1] = v.P;
  hdr[2] = quant == CVLC_QUANT_QSGD ? __float_as_uint(v.norm) : __float_as_uint(v.m);
  hdr[3] = quant == CVLC_QUANT_QSGD ? 0u : __float_as_uint(v.M);
  if (stats_out) {
    cvlc_seg_stats_t* st = stats_out + (size_t)client * kStatsStride + r;
    st->min = v.m; st->max = v.M; st->sumsq = sumsq; st->count = v.P; st->reserved = 0;
  }
}

// One thread: the stream's header, and the statistics of what is dropped.  (sbits: counted bit by bit once more here, as the
// last thing that a launch waits for, it made layout_kernel 0.7 us longer.)
__device__ __forceinline__ void write_global(const ClientParams& p, uint32_t client, uint32_t d, uint32_t sbits, double dropped, uint32_t quant,
                                             cvlc_seg_stats_t* stats_out) {
  GlobalWordPtr stream = (GlobalWordPtr)p.stream;
  stream[0] = kMagic;
  stream[1] = kVersion | (quant << 16);
  stream[2] = d;
  stream[3] = p.R;
  stream[4] = sbits;
  stream[5] = __float_as_uint(p.B);
  stream[6] = p.client_id;
  stream[7] = p.total_words;
  if (stats_out) {
    cvlc_seg_stats_t* st = stats_out + (size_t)client * kStatsStride + p.R;
    st->min = 0.0f; st->max = 0.0f; st->sumsq = dropped; st->count = d - p.k; st->reserved = 0;
    st->errsq = dropped;  // dropped whole
  }
}

// One whole wavefront, lanes 0 .. 31: first stream word of a group's records, the exclusive prefix of the payload sizes.
__device__ __forceinline__ uint32_t group_payload(const ClientParams& p, uint32_t sbits) {
  const uint32_t r = lane_id();
  uint32_t words = 0;
  if (r < p.R) words = (uint32_t)payload_words(p.Z[r] - (r ? p.Z[r - 1] : 0u), sbits + p.y[r]);
  const uint32_t incl = wave_incl_scan_u32(words);
  return kGlobalHeaderWords + kSegHeaderWords * p.R + incl - words;
}

// One workgroup of 1024 threads per client.  Turns the per-span counts of the
// groups into exclusive prefixes (in place; the row after the last span
// receives the totals), checks the totals against the plan, and
// clears the first and the last stream word of every (chunk, group) record run,
// a chunk being 8 spans: those two words can be shared with the neighbouring
// chunks, which OR their bits in; all other payload words have one owner and are
// stored whole.  Then the headers and the statistics block.
__global__ __launch_bounds__(kWideBlock) void layout_kernel(const ClientParams* __restrict__ params,
                                                            ClientCtl* __restrict__ ctls, Workspace ws,
                                                            cvlc_seg_stats_t* __restrict__ stats_out, uint32_t quant) {
  __shared__ double s_tail[kWideWaves], s_dropped;
  __shared__ uint32_t s_sum[32][kNormLimbs];  // QSGD: a group's sum of squares, limbs below 2^32
  __shared__ uint32_t s_payload[32];
  __shared__ uint32_t s_tot[kWideWaves][32];
  const uint32_t client = blockIdx.x, tid = threadIdx.x;
  const ClientParams& p = params[client];
  ClientCtl* ctl = ctls + client;
  if (ctl->dead) return;  // the workspace was too short for this client (whole workgroup)
  const uint32_t R = p.R, sbits = position_bits(ws.d);
  const uint32_t n_spans = (ctl->n_cand + kSpan - 1) / kSpan;
  const uint32_t lane = lane_id(), wave = tid / kWave;
  GlobalWordPtr stream = (GlobalWordPtr)p.stream;
  uint32_t* cnt = ws.span_cnt + (size_t)client * (ws.max_spans + 1) * 32;
  // What the headers and the statistics at the end need from memory is asked for here: this kernel is one
  // workgroup per client and all latency.
  uint32_t enc_max = 0, enc_negmin = 0;
  double enc_sumsq = 0.0;
  if (tid <= R) {  // entry R: the candidates below the last boundary
#pragma unroll
    for (uint32_t c = 0; c < kSegCopies; ++c) {
      enc_max = max(enc_max, ctl->seg[c].max_enc[tid]);
      enc_negmin = max(enc_negmin, ctl->seg[c].negmin_enc[tid]);
      enc_sumsq += ctl->seg[c].sumsq[tid];
    }
    if (tid == R) s_dropped = enc_sumsq;
  }
  const double* rsq = ws.region_sumsq + (size_t)client * ws.n_regions;  // energy the filter dropped, region by region
  const double tail0 = tid < ws.n_regions ? rsq[tid] : 0.0;
  const double tail1 = tid + kWideBlock < ws.n_regions ? rsq[tid + kWideBlock] : 0.0;
  if (wave == 0) {
    const uint32_t payload = group_payload(p, sbits);
    if (lane < 32u) s_payload[lane] = payload;
  }
  __syncthreads();
  // Exclusive prefix of the per-span counts over the spans, per group, in place.
  // Wavefront w takes a contiguous range of spans (a whole number of chunks); a
  // lane takes group (lane & 31) of every second span, so that one load covers
  // two whole rows of the table.
  const uint32_t g = lane & 31u, half = lane >> 5;
  const uint32_t W = g < R ? sbits + p.y[g] : 0u;
  const uint32_t P = g < R ? p.Z[g] - (g ? p.Z[g - 1] : 0u) : 0u;
  const uint32_t per_wave = (((n_spans + kWideWaves - 1) / kWideWaves + kChunkSpans - 1) / kChunkSpans) * kChunkSpans;
  const uint32_t s0 = min(wave * per_wave, n_spans), s1 = min(s0 + per_wave, n_spans);
  constexpr uint32_t kBatch = 8;  // loads in flight per lane and batch
  // A lane's counts of one batch of 2 * kBatch spans from span c on (0 past the wavefront's range); the
  // loads are not branched around (a lane past the end reads the range's last row), so that they all go out
  // together.
  auto load_batch = [&](uint32_t c, uint32_t (&vs)[kBatch]) {
#pragma unroll
    for (uint32_t u = 0; u < kBatch; ++u) {
      const uint32_t cc = c + 2 * u + half;
      const uint32_t x = cnt[(size_t)min(cc, s1 - 1u) * 32 + g];
      vs[u] = cc < s1 ? x : 0u;
    }
  };
  // The counts are read twice, for the wavefronts' totals and for the prefix; the first kKeep batches of a
  // wavefront (all of them up to 768 spans per client) stay in registers in between: this kernel is one
  // workgroup per client and all latency.
  constexpr uint32_t kKeep = 3;
  uint32_t keep[kKeep][kBatch];
  {
    uint32_t acc = 0;
#pragma unroll
    for (uint32_t b = 0; b < kKeep; ++b) {
      if (s0 + b * 2 * kBatch < s1) {  // uniform
        load_batch(s0 + b * 2 * kBatch, keep[b]);
      } else {
#pragma unroll
        for (uint32_t u = 0; u < kBatch; ++u) keep[b][u] = 0;
      }
    }
#pragma unroll
    for (uint32_t b = 0; b < kKeep; ++b)
#pragma unroll
      for (uint32_t u = 0; u < kBatch; ++u) acc += keep[b][u];
    for (uint32_t c = s0 + kKeep * 2 * kBatch; c < s1; c += 2 * kBatch) {
      uint32_t vs[kBatch];
      load_batch(c, vs);
#pragma unroll
      for (uint32_t u = 0; u < kBatch; ++u) acc += vs[u];
    }
    acc += __shfl_xor(acc, 32, 64);
    if (half == 0) s_tot[wave][g] = acc;
  }
  __syncthreads();
  uint32_t run = 0, total = 0;
  for (uint32_t w = 0; w < kWideWaves; ++w) {
    const uint32_t t = s_tot[w][g];
    if (w < wave) run += t;
    total += t;
  }
  // The first and the last word of a (chunk, group) record run [b, e); a consistent selection
  // never passes the planned size, and the test keeps the two stores inside the group's
  // payload even if an internal check has failed.
  auto clear_edges = [&](uint32_t b, uint32_t e) {
    if (half == 0 && e > b && e <= P) {
      const uint64_t bit0 = (uint64_t)b * W, bit1 = (uint64_t)e * W;
      stream[s_payload[g] + (uint32_t)(bit0 >> 5)] = 0;
      stream[s_payload[g] + (uint32_t)((bit1 - 1) >> 5)] = 0;
    }
  };
  uint32_t chunk_begin = run;
  auto prefix_batch = [&](uint32_t c, const uint32_t (&vs)[kBatch]) {
#pragma unroll
    for (uint32_t u = 0; u < kBatch; ++u) {
      const uint32_t cp = c + 2 * u;  // the pair's first span
      if (cp >= s1) break;            // uniform
      if (cp % kChunkSpans == 0 && cp > s0) {
        clear_edges(chunk_begin, run);
        chunk_begin = run;
      }
      const uint32_t v = vs[u], other = __shfl_xor(v, 32, 64);
      if (cp + half < s1) cnt[(size_t)(cp + half) * 32 + g] = half ? run + other : run;
      run += v + other;
    }
  };
#pragma unroll
  for (uint32_t b = 0; b < kKeep; ++b)
    if (s0 + b * 2 * kBatch < s1) prefix_batch(s0 + b * 2 * kBatch, keep[b]);  // uniform
  for (uint32_t c = s0 + kKeep * 2 * kBatch; c < s1; c += 2 * kBatch) {
    uint32_t vs[kBatch];
    load_batch(c, vs);
    prefix_batch(c, vs);
  }
  if (s1 > s0) clear_edges(chunk_begin, run);
  if (wave == 0 && half == 0) {
    cnt[(size_t)n_spans * 32 + g] = total;
    if (g < R && total != P) atomicOr(ws.status, CVLC_DEV_INTERNAL);
  }
  // energy of the coordinates the filter dropped
  double acc = tail0 + tail1;
  for (uint32_t t = tid + 2u * kWideBlock; t < ws.n_regions; t += kWideBlock) acc += rsq[t];
  acc = wave_sum_f64(acc);
  if (lane == 0) s_tail[wave] = acc;
  __syncthreads();

  if (tid < R) {
    const uint32_t r = tid;
    uint32_t flags = 0;
    const GroupValues v = group_values(P, W - sbits, enc_max, enc_negmin, quant, ws.norm_limbs + ((size_t)client * 32 + r) * kNormLimbs, s_sum[r], &flags);  // g = r
    write_group(p, client, r, v, enc_sumsq, quant, stats_out);
    if (stats_out) stats_out[(size_t)client * kStatsStride + r].errsq = 0.0;  // the pack kernel adds the group's error energy when asked to
    GroupInfo* gi = ws.group_info + client;
    gi->payload[r] = s_payload[r];
    gi->P[r] = v.P;
    gi->W[r] = sbits + v.y;
    gi->y[r] = v.y;
    gi->m[r] = v.low;
    gi->inv[r] = v.inv;
    gi->step[r] = v.step;
    if (flags) atomicOr(ws.status, flags);
  }
  if (tid == 32) {
    double dropped = 0.0;
    for (uint32_t w = 0; w < kWideWaves; ++w) dropped += s_tail[w];
    write_global(p, client, ws.d, sbits, dropped + s_dropped, quant, stats_out);
  }
}

// ------------------------------------------------------------------ 8. emit: quantise + pack
// a ^ b ^ c in one instruction (three-operand bitwise op with the truth table of the parity).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Philox4x32-10 (Salmon et al., SC'11), first output word.
__device__ __forceinline__ uint32_t philox_word0(uint32_t c0, uint32_t c1, uint32_t k0, uint32_t k1) {
  uint32_t c2 = 0, c3 = 0;
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0, p1 = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
    const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    c0 = xor3(hi1, c1, k0);
    c1 = lo1;
    c2 = xor3(hi0, c3, k1);
    c3 = lo0;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  return c0;
}

// Unbiased rounding to one of 2^y uniform centroids on [m, M] (PQ): position
// t = (x - m) * inv in fp32, lower centroid floor(t), one up with probability
// frac(t) resolved against a 24-bit uniform.
__device__ __forceinline__ uint32_t quantise(float x, float m, float inv, uint32_t y, uint32_t u24) {
  const float top = (float)((1u << y) - 1u);
  float t = __fmul_rn(__fsub_rn(x, m), inv);
  if (!(t > 0.0f)) t = 0.0f;
  if (t > top) t = top;
  const float fl = floorf(t);
  const uint32_t j = (uint32_t)fl;
  const float frac = __fsub_rn(t, fl);
  const uint32_t thr = (uint32_t)__fmul_rn(frac, 16777216.0f);
  const uint32_t cid = j + (u24 < thr ? 1u : 0u);
  const uint32_t last = (1u << y) - 1u;
  return cid > last ? last : cid;
}




constexpr uint32_t kChunkCands = kSpan * kChunkSpans;         // 4096
constexpr uint32_t kShortSpans = kShortMax / kSpan;
constexpr uint32_t kBlocks = kEmitBlock / 32u;                // of spans or chunks whose counts a packing workgroup adds up, a thread per block and group
constexpr uint32_t kBlockShiftMin = 3;                        // a block has eight chunks at least
static_assert(kShortSpans % kBlocks == 0, "a short vector's spans are dealt out to the threads evenly");
constexpr uint32_t kEdgeChunks = 8;                           // chunks whose shared stream words a workgroup holds back
constexpr uint32_t kStageWords = kChunkCands * 2 + 2 * 32;    // every record is < 64 bits; two edge words per group

struct alignas(16) EmitGroup {  // per (chunk, group)
  uint32_t first, lim;   // the chunk's record run [first, lim) of the group
  uint32_t W, y;
  float m, inv;
  uint32_t stage_bit;    // bit of record `first` in the workgroup's staged image of the stream
  float step;            // centroid spacing (only read when the error energy is measured)
};

// One workgroup per chunk of 4096 candidates, one wavefront per span.  Every
// coded candidate gets its record number inside its group (members in earlier
// spans from the layout's prefix, plus its number inside the span, which the
// counting pass left with its group in 16 bits), is quantised and OR-ed into an
// LDS image of the stream words its group's run covers.  The image is then
// written out: a group's first and last word can be shared with a neighbouring
// chunk and are OR-ed into the (cleared) stream, all others are stored whole.
// ERR: every record also adds (xtilde / B - x)^2 to its group's error energy in
// the statistics block (Lemma 1's left side for this draw), xtilde being the
// centroid value the decoder will compute from the header.
// QSGD: the code is the level of |x| on [0, norm] with the sign bit above it.
// kShortVec: a short vector's coordinates in the candidates' place.
// kByChunks, kShortVec: there is no layout launch, every workgroup makes what it needs of the prefix from the chunks' or the spans'
// counts (at most 16 KB) and derives the groups' values for itself; a client's first one also writes its headers.
template <bool ERR, bool QSGD, PassMode MODE>
__global__ __launch_bounds__(kEmitBlock, MODE == kShortVec ? 4 : 6) void emit_kernel(const ClientParams* __restrict__ params,
                                                          ClientCtl* __restrict__ ctls, Workspace ws, uint64_t seed,
                                                          cvlc_seg_stats_t* __restrict__ stats_out) {
  constexpr bool SHORT = MODE == kShortVec, CHUNKS = MODE == kByChunks;
  __shared__ double s_err[ERR ? kEmitWaves : 1][32];  // per wavefront, per group
  __shared__ uint32_t s_stage[kStageWords];
  // A chunk's tables, two sets: the next chunk's are filled while the current one is written out.
  __shared__ uint32_t s_wrun[2][kEmitWaves][32];   // per wavefront, per group: record number of its span's first member
  __shared__ EmitGroup s_grp[2][32];               // what a record of the group needs, read as two 16-byte pieces
  __shared__ uint32_t s_word0[2][32];              // first stream word (group-relative) the chunk touches
  __shared__ uint32_t s_nwords[2][32];             // words the chunk touches in each group
  __shared__ uint32_t s_stage_off[2][33];
  __shared__ uint32_t s_payload[32];
  __shared__ uint32_t s_size[32];                  // records of every group
  __shared__ EmitGroup s_const[32];                // W, y, m, inv, step of every group
  __shared__ uint32_t s_next;                      // the chunk the workgroup takes after the current one
  // The first and the last word of a (chunk, group) run are OR-ed into the stream by device-wide atomics.
  // Whatever the wavefront loads next waits for their acknowledgement (the counter of outstanding memory
  // operations does not tell loads from atomics), so they are held back, kEdgeChunks chunks' worth, and
  // issued together.
  __shared__ uint32_t s_edge_word[kEdgeChunks][32][2];  // the bits; 0: nothing to OR
  __shared__ uint32_t s_edge_at[kEdgeChunks][32][2];    // the stream word they belong to
  // kShortVec: members of every group in the spans before; kByChunks: ... in the chunks before every 2^block_shift-th
  __shared__ uint32_t s_prefix[SHORT ? kShortSpans + 1u : CHUNKS ? kBlocks : 1u][32];
  __shared__ uint32_t s_part[SHORT || CHUNKS ? kBlocks : 1u][32];
  __shared__ uint32_t s_sum[(SHORT || CHUNKS) && QSGD ? 32 : 1][kNormLimbs];
  __shared__ double s_dropped[CHUNKS ? kEmitWaves : 1u];
  // Workgroups are dispatched in the order of their linear index and a CU serves its oldest first: the
  // clients' workgroups are interleaved in that order, so that every client has workgroups of every age.
  const uint32_t linear = blockIdx.y * gridDim.x + blockIdx.x;
  const uint32_t client = linear % gridDim.y, block_x = linear / gridDim.y;
  const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const ClientParams& p = params[client];
  ClientCtl* ctl = ctls + client;
  if (SHORT && block_x == 0 && tid == 0 && ctl->flags) atomicOr(ws.status, ctl->flags);
  if (ctl->dead) return;  // the workspace was too short for this client (whole workgroup)
  const uint32_t n = SHORT ? ws.d : ctl->n_cand;
  const uint32_t n_spans = (n + kSpan - 1) / kSpan;
  const uint32_t R = p.R, sbits = position_bits(ws.d);
  const uint32_t* __restrict__ val = SHORT ? (const uint32_t*)(GlobalConstWordPtr)p.update : ws.dense_val + (size_t)client * ws.dense_cap;
  const uint32_t* __restrict__ idx = ws.dense_idx + (size_t)client * ws.dense_cap;
  const uint16_t* __restrict__ place = span_places(ws, client);
  const uint32_t* __restrict__ prefix = ws.span_cnt + (size_t)client * (ws.max_spans + 1) * 32;
  GlobalWordPtr stream = (GlobalWordPtr)p.stream;
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32), client_id = p.client_id;

  // what thread r of the first 32 needs of group r for every chunk's tables (not in registers, where it would be every
  // thread's: as it is, three to eight of them spill where the prefix comes from the chunks' counts, none to three where it is the layout's)
  if (tid < 32u) {
    s_size[tid] = 0;
    s_const[tid] = EmitGroup{0u, 0u, 0u, 0u, 0.0f, 0.0f, 0u, 0.0f};
  }
  const uint32_t* __restrict__ totals = chunk_totals(ws, client);
  const uint32_t n_chunks = (n_spans + kChunkSpans - 1u) / kChunkSpans;
  uint32_t block_shift = kBlockShiftMin;
  if constexpr (SHORT || CHUNKS) {
    // The counts: a thread takes group tid mod 32 of eight neighbouring spans, or of a block of neighbouring chunks, eight
    // as a rule, more where there are more than 128 of them.
    constexpr uint32_t kSpansEach = kShortSpans / kBlocks;
    static_assert(kSpansEach == 1u << kBlockShiftMin, "eight loads together either way");
    const uint32_t g = tid % 32u, part = tid / 32u;
    uint32_t c[kSpansEach], sum = 0;
    if constexpr (SHORT) {
#pragma unroll
      for (uint32_t i = 0; i < kSpansEach; ++i) {
        const uint32_t span = part * kSpansEach + i;
        c[i] = prefix[(size_t)min(span, n_spans - 1u) * 32 + g];
        c[i] = span < n_spans ? c[i] : 0u;
      }
    } else {
      while ((n_chunks - 1u) >> block_shift >= kBlocks) ++block_shift;
      const uint32_t last = min((part + 1u) << block_shift, n_chunks);
      for (uint32_t from = part << block_shift; from < last; from += kSpansEach) {
#pragma unroll
        for (uint32_t i = 0; i < kSpansEach; ++i) c[i] = totals[(size_t)min(from + i, n_chunks - 1u) * 32 + g];
#pragma unroll
        for (uint32_t i = 0; i < kSpansEach; ++i) sum += from + i < last ? c[i] : 0u;
      }
    }
    const uint32_t my_group = min(tid, CVLC_MAX_CODED - 1u), y = p.y[my_group], P = p.Z[my_group] - (my_group ? p.Z[my_group - 1u] : 0u);
    uint32_t enc_max = 0, enc_negmin = 0, flags = 0;
    double sumsq = 0.0;
    if (tid <= R) {  // entry R: what is dropped
#pragma unroll
      for (uint32_t i = 0; i < kSegCopies; ++i) {
        enc_max = max(enc_max, ctl->seg[i].max_enc[tid]);
        enc_negmin = max(enc_negmin, ctl->seg[i].negmin_enc[tid]);
        sumsq += ctl->seg[i].sumsq[tid];
      }
    }
    if (CHUNKS && block_x == 0) {  // ... and by the filter, region by region
      const double* rsq = ws.region_sumsq + (size_t)client * ws.n_regions;
      double dropped = 0.0;
      for (uint32_t i = tid; i < ws.n_regions; i += kEmitBlock) dropped += rsq[i];
      dropped = wave_sum_f64(dropped);
      if (lane == 0) s_dropped[wave] = dropped;
    }
    if constexpr (SHORT) {
#pragma unroll
      for (uint32_t i = 0; i < kSpansEach; ++i) sum += c[i];
    }
    s_part[part][g] = sum;
    if (wave == 0) {
      const uint32_t payload = group_payload(p, sbits);
      if (lane < 32u) s_payload[lane] = payload;
    }
    __syncthreads();
    uint32_t run = 0, all = 0;
    if constexpr (SHORT) {
      for (uint32_t i = 0; i < part; ++i) run += s_part[i][g];
#pragma unroll
      for (uint32_t i = 0; i < kSpansEach; ++i) {
        s_prefix[part * kSpansEach + i][g] = run;
        run += c[i];
      }
      if (part == kBlocks - 1u) s_prefix[kShortSpans][g] = run;
    } else {
#pragma unroll
      for (uint32_t i = 0; i < kBlocks; ++i) {
        const uint32_t x = s_part[i][g];
        run += i < part ? x : 0u;
        all += x;
      }
      s_prefix[part][g] = run;
    }
    if (tid < R) {
      const GroupValues gv = group_values(P, y, enc_max, enc_negmin, QSGD ? CVLC_QUANT_QSGD : CVLC_QUANT_PQ,
                                          ws.norm_limbs + ((size_t)client * 32 + tid) * kNormLimbs, s_sum[QSGD ? tid : 0u], &flags);
      s_size[tid] = gv.P;
      s_const[tid] = EmitGroup{0u, 0u, sbits + y, y, gv.low, gv.inv, 0u, gv.step};
      if (block_x == 0) write_group(p, client, tid, gv, sumsq, QSGD ? CVLC_QUANT_QSGD : CVLC_QUANT_PQ, stats_out);
    }
    if (block_x == 0 && tid == R) {
      if constexpr (CHUNKS)
        for (uint32_t w = 0; w < kEmitWaves; ++w) sumsq += s_dropped[w];
      write_global(p, client, ws.d, sbits, sumsq, QSGD ? CVLC_QUANT_QSGD : CVLC_QUANT_PQ, stats_out);
    }
    __syncthreads();
    if constexpr (SHORT) all = s_prefix[kShortSpans][g];  // spans past the last are empty
    if (tid < R && all != P) flags |= CVLC_DEV_INTERNAL;  // g = tid
    if (block_x == 0 && flags) atomicOr(ws.status, flags);
  } else if (tid < 32 && tid < R) {
    const GroupInfo* gi = ws.group_info + client;
    s_size[tid] = gi->P[tid];
    s_const[tid] = EmitGroup{0u, 0u, gi->W[tid], gi->y[tid], gi->m[tid], gi->inv[tid], 0u, gi->step[tid]};
    s_payload[tid] = gi->payload[tid];
  }
  const double inv_B = ERR ? 1.0 / (double)p.B : 0.0;  // the scaling operation of Sec. IV-B
  if (ERR && lane < 32) s_err[wave][lane] = 0.0;       // touched by this wavefront only until the end
  auto chunk_exists = [&](uint32_t c) { return (uint64_t)c * kChunkSpans < n_spans; };
  // What a chunk needs of the layout's prefix: the record numbers the wavefront's span starts at (lanes
  // 0..31: one group each) and, for the first 32 threads, the chunk's record run of a group.
  uint32_t ahead_row = 0, ahead_first = 0, ahead_last = 0;
  // By chunks: the counts of the chunks between the block's first and this one, of the spans before the wavefront's in the
  // chunk, and of the chunk itself; the two halves of the wavefront take every second row.
  constexpr uint32_t kPairs = kChunkSpans / 2u;
  uint32_t ahead_chunk[CHUNKS ? kPairs : 1u], ahead_span[CHUNKS ? kPairs : 1u];
  static_assert(kChunkSpans == 1u << kBlockShiftMin, "as many spans in a chunk as chunks in a block at least");
  auto last_eight = [&](uint32_t c) {  // the first of the last eight chunks or fewer in the block before chunk c
    const uint32_t block = c >> block_shift << block_shift;
    return c > block ? block + (c - 1u - block) / kChunkSpans * kChunkSpans : block;
  };
  auto ask_prefix = [&](uint32_t c) {
    if (!chunk_exists(c)) return;  // uniform
    if constexpr (CHUNKS) {
      const uint32_t g = lane & 31u, half = lane >> 5, from = last_eight(c);
      ahead_row = 0;
      for (uint32_t x = (c >> block_shift << block_shift) + half; x < from; x += 2u) ahead_row += totals[(size_t)x * 32u + g];
#pragma unroll
      for (uint32_t u = 0; u < kPairs; ++u) {
        ahead_chunk[u] = totals[(size_t)min(from + 2u * u + half, c) * 32u + g];
        ahead_span[u] = prefix[(size_t)min(c * kChunkSpans + 2u * u + half, n_spans - 1u) * 32u + g];
      }
      if (wave == 0) ahead_last = totals[(size_t)c * 32u + g];
      return;
    }
    const uint32_t span = c * kChunkSpans + wave;
    auto row = [&](uint32_t sp, uint32_t g) { return SHORT ? s_prefix[sp][g] : prefix[(size_t)sp * 32 + g]; };
    if (lane < 32) ahead_row = span < n_spans ? row(span, lane) : 0u;
    if (tid < R && tid < 32) {
      const uint32_t last_span = min((c + 1) * kChunkSpans, n_spans);
      ahead_first = row(c * kChunkSpans, tid);
      ahead_last = row(last_span, tid);
    }
  };
  // Value bits, position and place of the candidates of the wavefront's span.  Unconditional loads (a
  // lane past the end reads the last candidate again), so that all of them are in flight together.
  uint32_t v[kPerLane], pid[kPerLane], plc[kPerLane];
  auto ask_candidates = [&](uint32_t c) {
    if (!chunk_exists(c)) return;  // uniform
#pragma unroll
    for (uint32_t j = 0; j < kPerLane; ++j) {
      const uint32_t i = (c * kChunkSpans + wave) * kSpan + j * kWave + lane;
      const uint32_t at = min(i, n - 1u);
      v[j] = val[at];
      pid[j] = SHORT ? i : idx[at];
      plc[j] = i < n ? (uint32_t)place[at] : (uint32_t)kNoPlace;
    }
  };
  // Fills set `to` of the chunk tables from what ask_prefix brought.
  auto set_up = [&](uint32_t to, uint32_t c) {
    if constexpr (CHUNKS) {
      if (!chunk_exists(c)) return;  // uniform
      const uint32_t half = lane >> 5, from = last_eight(c);
#pragma unroll
      for (uint32_t u = 0; u < kPairs; ++u) {
        ahead_row += from + 2u * u + half < c ? ahead_chunk[u] : 0u;
        ahead_row += 2u * u + half < wave ? ahead_span[u] : 0u;
      }
      ahead_row += (uint32_t)__shfl_xor((int)ahead_row, 32, 64);
      ahead_row += s_prefix[c >> block_shift][lane & 31u];
      ahead_first = ahead_row;  // read by the first wavefront, whose span is the chunk's first
      ahead_last += ahead_row;
    }
    if (lane < 32) s_wrun[to][wave][lane] = ahead_row;
    if (tid < 32) {
      const uint32_t r = tid;
      EmitGroup eg = s_const[r];
      uint32_t nwords = 0, first = 0, last = 0, bit_in_word = 0;
      if (r < R) {
        const uint32_t P = s_size[r], W = eg.W;
        // the chunk's record run of group r: [first, last), clamped so that every write stays inside
        // the group's payload even if an internal check has failed
        first = ahead_first;
        last = ahead_last;
        if (last > P) last = P;
        if (first > last) first = last;
        if (last > first) {
          const uint64_t bit0 = (uint64_t)first * W, bit1 = (uint64_t)last * W;
          s_word0[to][r] = (uint32_t)(bit0 >> 5);
          bit_in_word = (uint32_t)(bit0 & 31u);
          nwords = (uint32_t)(((bit1 - 1) >> 5) - (bit0 >> 5) + 1);
        }
      }
      s_nwords[to][r] = nwords;
      // exclusive prefix of the staged word counts over the groups
      const uint32_t incl = wave_incl_scan_u32(nwords);
      s_stage_off[to][r] = incl - nwords;
      if (r == 31) s_stage_off[to][32] = incl;
      eg.first = first;
      eg.lim = last;
      eg.stage_bit = (incl - nwords) * 32u + bit_in_word;  // bit of record `first` in the staged image
      s_grp[to][r] = eg;
    }
  };
  // Which chunks a workgroup takes: its own first, then whichever chunk of the client nobody has
  // taken yet (a counter of the client's), so that the workgroups of a CU, of which the oldest is served
  // first, all stay until the work runs out instead of leaving one after the other.  The next chunk is
  // claimed when the current one begins and known (through s_next) when its records are done.
  // A chunk goes through two phases with a barrier before each: the records (all wavefronts OR into the
  // staged image); write the image out, leaving zeros behind.  The next chunk's candidates and prefix
  // are requested before the current chunk is written out, its tables filled after.
  for (uint32_t i = tid; i < kEdgeChunks * 64u; i += kEmitBlock) (&s_edge_word[0][0][0])[i] = 0;  // groups past R stay 0
  uint32_t held = 0;  // chunks whose edge words are held back
  auto release_edges = [&]() {  // by the whole workgroup, after a barrier
    for (uint32_t i = tid; i < held * 64u; i += kEmitBlock) {
      const uint32_t word = (&s_edge_word[0][0][0])[i];
      if (word) atomicOr((uint32_t*)(stream + (&s_edge_at[0][0][0])[i]), word);
    }
  };
  ask_prefix(block_x);
  ask_candidates(block_x);
  for (uint32_t i = tid; i < kStageWords; i += kEmitBlock) s_stage[i] = 0;
  set_up(0, block_x);
  uint32_t cur = 0;
  for (uint32_t c = block_x; chunk_exists(c); cur ^= 1u) {
    uint32_t claimed = 0;
    if (tid == 0) claimed = atomicAdd(&ctl->emit_claim, 1u);
    __syncthreads();  // the chunk before is written out (and its image cleared); this chunk's tables are in place
    const uint32_t* wrun = s_wrun[cur][wave];
#pragma unroll
    for (uint32_t j = 0; j < kPerLane; ++j) {
      if (plc[j] != kNoPlace) {
        const uint32_t g = plc[j] & ((1u << kPlaceShift) - 1u);
        const uint32_t e = wrun[g] + (plc[j] >> kPlaceShift);
        const EmitGroup eg = s_grp[cur][g];
        if (e < eg.lim) {
          const uint32_t y = eg.y, W = eg.W;
          uint32_t cid;
          if (y == 32) {
            cid = v[j];
          } else {
            const uint32_t u24 = philox_word0(pid[j], client_id, k0, k1) >> 8;
            if (QSGD)
              cid = quantise(fabsf(__uint_as_float(v[j])), 0.0f, eg.inv, y - 1u, u24) | ((v[j] >> 31) << (y - 1u));
            else
              cid = quantise(__uint_as_float(v[j]), eg.m, eg.inv, y, u24);
          }
          if (ERR) {
            const float x = __uint_as_float(v[j]);
            float xt = x;
            if (y != 32) {
              if (QSGD) {
                const float mag = __fmaf_rn((float)(cid & ((1u << (y - 1u)) - 1u)), eg.step, 0.0f);
                xt = (cid >> (y - 1u)) ? -mag : mag;
              } else {
                xt = __fmaf_rn((float)cid, eg.step, eg.m);
              }
            }
            const double err = (double)xt * inv_B - (double)x;
            atomicAdd(&s_err[wave][g], err * err);
          }
          const uint64_t record = (uint64_t)pid[j] | ((uint64_t)cid << sbits);
          // a chunk's run of a group is at most 4096 records of at most 63 bits: 32 bits hold the offset
          const uint32_t bit = eg.stage_bit + __umul24(e - eg.first, W);
          const uint32_t w0 = bit >> 5, sh = bit & 31u;
          const uint64_t lo = record << sh;
          atomicOr(&s_stage[w0], (uint32_t)lo);
          if (sh + W > 32u) atomicOr(&s_stage[w0 + 1], (uint32_t)(lo >> 32));
          if (sh + W > 64u) atomicOr(&s_stage[w0 + 2], (uint32_t)(record >> (64u - sh)));
        }
      }
    }
    if (tid == 0) s_next = gridDim.x + claimed;
    __syncthreads();
    const uint32_t c_next = s_next;
    ask_prefix(c_next);
    ask_candidates(c_next);
    // A wavefront writes whole groups' runs, lane l the l-th, l+64-th, ... word (with all 512 threads on one
    // group after the other most lanes had nothing to write in every group).  A group's size changes steadily
    // with its number, so the groups are dealt out going up and coming down in turn (wavefront w: w, 15 - w,
    // 16 + w, 31 - w).
    for (uint32_t k = 0; k * kEmitWaves < R; ++k) {
      const uint32_t g = k * kEmitWaves + ((k & 1u) ? kEmitWaves - 1u - wave : wave);
      if (g >= R) continue;  // uniform per wavefront
      const uint32_t nwords = s_nwords[cur][g];
      uint32_t* staged_words = s_stage + s_stage_off[cur][g];
      const uint32_t first_word = s_payload[g] + s_word0[cur][g];
      GlobalWordPtr dst = stream + first_word;
      if (lane < 2) s_edge_word[held][g][lane] = 0;  // (this wavefront's LDS accesses complete in order)
      for (uint32_t rel = lane; rel < nwords; rel += kWave) {
        const uint32_t word = staged_words[rel];
        staged_words[rel] = 0;  // the image is all zeros again when the next chunk begins
        if (rel == 0 || rel == nwords - 1) {
          const uint32_t which = rel == 0 ? 0u : 1u;
          s_edge_word[held][g][which] = word;
          s_edge_at[held][g][which] = first_word + rel;
        } else {
          dst[rel] = word;
        }
      }
    }
    set_up(cur ^ 1u, c_next);  // the next chunk's tables (after the last chunk: tables nobody reads)
    c = c_next;
    if (++held == kEdgeChunks) {  // uniform
      __syncthreads();
      release_edges();
      held = 0;
    }
  }  // chunks
  __syncthreads();
  release_edges();
  if (ERR) {
    __syncthreads();
    if (tid < R) {
      double sum = 0.0;
      for (uint32_t w = 0; w < kEmitWaves; ++w) sum += s_err[w][tid];
      if (sum != 0.0) atomicAdd(&stats_out[(size_t)client * kStatsStride + tid].errsq, sum);
    }
  }
}

// ------------------------------------------------------------------ host side
// Candidates per client a workspace of ws_bytes has room for: the largest cap <= d whose layout fits (the
// layout grows with cap), 0 if not even one does.
uint32_t candidate_room(uint32_t d, uint32_t n, size_t ws_bytes) {
  if (encode_layout(d, n, 1u).total > ws_bytes) return 0u;
  uint32_t lo = 1u, hi = d;  // lo fits
  while (lo < hi) {
    const uint32_t mid = lo + (hi - lo + 1u) / 2u;
    if (encode_layout(d, n, mid).total <= ws_bytes) lo = mid; else hi = mid - 1u;
  }
  return lo;
}

int validate_batch(uint32_t n, const cvlc_plan_t* plans, const float* const* d_updates,
                   const uint32_t* client_ids, void* const* d_streams, const size_t* capacities,
                   void* d_workspace, size_t ws_bytes) {
  if (n == 0 || !plans || !d_updates || !client_ids || !d_streams || !capacities || !d_workspace) return CVLC_ERR_ARG;
  if (reinterpret_cast<uintptr_t>(d_workspace) % 256u) return CVLC_ERR_ARG;
  if (n > 65535u) return CVLC_ERR_ARG;  // clients index the grid's y dimension
  const uint32_t d = plans[0].d;
  for (uint32_t i = 0; i < n; ++i) {
    const int rc = cvlc_plan_validate(&plans[i]);
    if (rc) return rc;
    if (plans[i].d != d) return CVLC_ERR_ARG;
    if (!d_updates[i] || reinterpret_cast<uintptr_t>(d_updates[i]) % 16u) return CVLC_ERR_ARG;
    if (!d_streams[i] || reinterpret_cast<uintptr_t>(d_streams[i]) % 4u) return CVLC_ERR_ARG;
    if (capacities[i] < cvlc_stream_capacity(&plans[i])) return CVLC_ERR_CAPACITY;
    if (plans[i].total_bits / 32u > 0xFFFFFFFFull) return CVLC_ERR_PLAN;
  }
  uint32_t k_max = 0;
  for (uint32_t i = 0; i < n; ++i) {
    uint64_t k = 0;
    for (uint32_t r = 0; r < plans[i].n_coded; ++r) k += plans[i].count[r];
    if (k > k_max) k_max = (uint32_t)k;  // a valid plan keeps at most d
  }
  if (candidate_room(d, n, ws_bytes) < (k_max < 1 ? 1u : k_max)) return CVLC_ERR_CAPACITY;
  return CVLC_OK;
}

// Rank inside the sample at which the candidate threshold is read: the expected
// number of sampled coordinates inside the top k, plus six standard deviations
// of that count and a small constant.  0 = do not sample, keep every coordinate.
uint32_t sample_rank(uint32_t d, uint32_t k, uint32_t n_sampled) {
  if (n_sampled == 0) return 0u;
  const double expect = (double)k * (double)n_sampled / (double)d;
  const double want = std::ceil(expect + 6.0 * std::sqrt(expect) + 16.0);
  if (want >= (double)n_sampled) return 0u;
  return (uint32_t)want;
}

// Filter workgroups the current device holds at once, at most kFilterBlocksCap.
uint32_t filter_resident_blocks() {
  static uint32_t cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return kFilterBlocksCap / 2;
  if (cached[dev] == 0) {
    int cus = 0, per_cu = 0;
    uint32_t r = kFilterBlocksCap / 2;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, filter_kernel, kBlock, 0) == hipSuccess && cus > 0 &&
        per_cu > 0)
      r = (uint32_t)cus * (uint32_t)per_cu;
    cached[dev] = r > kFilterBlocksCap ? kFilterBlocksCap : r;
  }
  return cached[dev];
}

// Short vectors take three launches instead of ten: 1 x 2000 54 -> 26 us, 1 x 65 536 59 -> 41 (31 groups 68 -> 50), 32 x 65 536
// 76 -> 48, 100 x 65 536 of 31 groups 207 -> 122.  They go up to 65 536 coordinates because a place in one has 16 bits (a part of
// 256 coordinates and a byte): longer ones have not been tried.
// Of many long ones the general path reads all and then works on what it keeps, which is less than going through all of it
// again in the counting and the packing pass, unless next to nothing or a good part is kept.  us in ten launches and in
// three, 3 % kept: 144 x 65 536 104 and 90, 256 x 58 000 150 and 142, 300 x 65 536 191 and 203, 513 x 65 536 314 and 346, 2000 x 65 536
// 1244 and 1314, 2000 x 40 000 1247 and 1245; 30 % kept, 300 x 65 536 222 and 215; half a percent, 208 x 65 536 136 and 124.
constexpr uint64_t kShortAll = 9u << 20;      // coordinates of a batch: 144 of the longest
constexpr uint32_t kShortAnyNumber = 40960u;  // coordinates of a vector
bool short_pays(uint32_t n, const cvlc_plan_t* plans) {
  const uint64_t all = (uint64_t)n * plans[0].d;
  if (all <= kShortAll || plans[0].d <= kShortAnyNumber) return true;
  uint64_t kept = 0;
  for (uint32_t i = 0; i < n; ++i)
    for (uint32_t r = 0; r < plans[i].n_coded; ++r) kept += plans[i].count[r];
  return kept * 128u <= all || kept * 10u >= all * 3u;
}

// Whether the packing pass makes its prefixes from the chunks' counts (kByChunks) or a layout kernel does.  The layout is one
// workgroup per client: a launch of 5 us, and about 14 us for every million coordinates that the client with the most keeps.  In its
// place the counting pass clears the streams, not only the words at the runs' ends, which goes with all that is kept, and every
// packing workgroup goes through its client's chunks for every chunk of its own, beyond 128 of them one by one: that goes with all that
// is kept times what a client keeps.  Both sides were timed for 220 calls, of 1 to 300 clients that keep 1 % to all of 70 000 to
// 4e8 coordinates in 7, 15 and 31 groups; the line takes the slower side by more than 2 % in three of them, 5 % at most, and in
// two of these the difference is one of runs.  us with the layout and by chunks: 1 x 1.2 M 64 and 60, 1 x 11.2 M 79 and 72, half kept 257 and
// 188, 1 x 25.6 M all kept 957 and 717, 1 x 1e8 half kept 2042 and 1778, all kept 3843 and 4096, 1 x 2e8 all kept 7677 and 11 494; 8 x 1.2 M
// 77 and 73, 8 x 11.2 M 160 and 152, all kept 1157 and 1246; 32 x 11.2 M 453 and 450, a quarter kept 1261 and 1320, half kept 2247 and
// 2487; 100 x 300 000 125 and 122, 100 x 1.2 M half kept 837 and 870, 100 x 11.2 M 1330 and 1357 (where nothing else is said, 3 %).
bool chunks_pay(uint32_t n, const cvlc_plan_t* plans) {
  double all = 0.0, most = 0.0;  // millions of coordinates
  for (uint32_t i = 0; i < n; ++i) {
    uint64_t k = 0;
    for (uint32_t r = 0; r < plans[i].n_coded; ++r) k += plans[i].count[r];
    all += 1e-6 * (double)k;
    most = std::max(most, 1e-6 * (double)k);
  }
  return all * (3.0 + most) <= 60.0 * most + 80.0;
}

}  // namespace
}  // namespace cvlc

extern "C" {

size_t cvlc_encode_workspace_bytes(uint32_t d, uint32_t n_clients) {
  if (d < 1 || n_clients < 1) return 0;
  return cvlc::encode_layout(d, n_clients, d).total;
}

size_t cvlc_encode_workspace_bytes_for(uint32_t d, uint32_t n_clients, uint32_t max_candidates) {
  if (d < 1 || n_clients < 1) return 0;
  return cvlc::encode_layout(d, n_clients, max_candidates < 1 ? 1u : max_candidates).total;
}

uint32_t cvlc_plan_candidates_hint(const cvlc_plan_t* plan) {
  using namespace cvlc;
  if (!plan || cvlc_plan_validate(plan) != CVLC_OK) return 0;
  const uint32_t d = plan->d;
  uint64_t k = 0;
  for (uint32_t r = 0; r < plan->n_coded; ++r) k += plan->count[r];
  const uint32_t n_src = d / kSamplePiece;
  const uint32_t n_sampled = (n_src < kSampleChunksMax ? n_src : kSampleChunksMax) * kSamplePiece;
  const uint32_t rank = sample_rank(d, (uint32_t)k, n_sampled);
  if (rank == 0) return d;  // no threshold is sampled for this plan: every coordinate is a candidate
  // The share of the vector at or above the sample's rank-th largest key is rank / n_sampled give or take
  // sqrt(rank) / n_sampled; the threshold is that key rounded down to 13 bits, worth a few percent more.
  const double share = ((double)rank + 6.0 * std::sqrt((double)rank) + 16.0) / (double)n_sampled;
  const double want = std::ceil(1.25 * share * (double)d) + 4096.0;
  return want >= (double)d ? d : (uint32_t)want;
}

int cvlc_encode_batch(uint32_t n, const cvlc_plan_t* plans, const float* const* d_updates, uint64_t seed,
                      const uint32_t* client_ids, void* const* d_streams_out, const size_t* capacities,
                      void* d_workspace, size_t ws_bytes, cvlc_seg_stats_t* d_stats_out, uint32_t flags,
                      void* hip_stream) {
  using namespace cvlc;
  int rc = validate_batch(n, plans, d_updates, client_ids, d_streams_out, capacities, d_workspace, ws_bytes);
  if (rc) return rc;
  if (flags & ~CVLC_ENCODE_ERROR_STATS) return CVLC_ERR_ARG;
  const uint32_t quant = plans[0].quant;
  for (uint32_t i = 1; i < n; ++i)
    if (plans[i].quant != quant) return CVLC_ERR_ARG;
  if ((flags & CVLC_ENCODE_ERROR_STATS) && !d_stats_out) return CVLC_ERR_ARG;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const uint32_t d = plans[0].d;
  const EncodeLayout L = encode_layout(d, n, candidate_room(d, n, ws_bytes));
  const ShortLayout SL = short_layout(d, n);
  const bool is_short = d <= kShortMax && SL.total <= ws_bytes && short_pays(n, plans);
  char* base = static_cast<char*>(d_workspace);
  Workspace ws;
  ws.status = reinterpret_cast<uint32_t*>(base + L.status);
  ws.params = reinterpret_cast<ClientParams*>(base + L.params);
  ws.ctl = reinterpret_cast<ClientCtl*>(base + L.ctl);
  ws.region_cnt = reinterpret_cast<uint32_t*>(base + L.region_cnt);
  ws.region_sumsq = reinterpret_cast<double*>(base + L.region_sumsq);
  ws.cand_idx = reinterpret_cast<uint16_t*>(base + L.cand_idx);
  ws.cand_val = reinterpret_cast<uint32_t*>(base + L.cand_val);
  ws.dense_idx = reinterpret_cast<uint32_t*>(base + L.dense_idx);
  ws.dense_val = reinterpret_cast<uint32_t*>(base + L.dense_val);
  ws.nz_off = reinterpret_cast<uint32_t*>(base + L.nz_off);
  ws.nz_run = reinterpret_cast<uint32_t*>(base + L.nz_run);
  ws.span_first = reinterpret_cast<uint32_t*>(base + L.span_first);
  ws.span_cnt = reinterpret_cast<uint32_t*>(base + L.span_cnt);
  ws.group_info = reinterpret_cast<GroupInfo*>(base + L.group_info);
  ws.hist_bins = reinterpret_cast<uint32_t*>(base + L.hist_bins);
  ws.members = reinterpret_cast<unsigned long long*>(base + L.members);
  ws.seg_cnt = reinterpret_cast<uint32_t*>(base + L.seg_cnt);
  ws.norm_limbs = reinterpret_cast<unsigned long long*>(base + L.norm_limbs);
  ws.d = d;
  ws.region_shift = L.region_shift;
  ws.n_regions = L.n_regions;
  ws.max_spans = L.max_spans;
  ws.dense_cap = L.dense_cap;
  ws.filter_blocks = filter_blocks_per_client(L.n_regions, n, filter_resident_blocks());
  ws.gather_blocks = L.gather_blocks;
  ws.member_pool = L.member_pool;
  ws.hist_copies = L.hist_copies;
  if (is_short) {
    ws.status = reinterpret_cast<uint32_t*>(base + SL.status);
    ws.params = reinterpret_cast<ClientParams*>(base + SL.params);
    ws.ctl = reinterpret_cast<ClientCtl*>(base + SL.ctl);
    ws.norm_limbs = reinterpret_cast<unsigned long long*>(base + SL.norm_limbs);
    ws.cand_idx = reinterpret_cast<uint16_t*>(base + SL.places);
    ws.span_cnt = reinterpret_cast<uint32_t*>(base + SL.span_cnt);
    ws.max_spans = SL.max_spans;
  }

  // sample geometry: 256-byte pieces spread evenly; all of them when the vector is short
  const uint32_t n_src = d / kSamplePiece;
  const uint32_t n_s = n_src < kSampleChunksMax ? n_src : kSampleChunksMax;

  // the status word and the control blocks start every call at zero
  uint32_t zero_n16 = (uint32_t)((is_short ? SL.ctl : L.zero_bytes) / 16u);  // n <= 65535 clients: below 2^32 pieces
  auto short_select = [&](auto source, uint32_t clients, bool first) {
    StageScope scope(CVLC_STAGE_ENC_SELECT, stream);
    hipLaunchKernelGGL(short_select_kernel<decltype(source)>, dim3(clients), dim3(kShortBlock), 0, stream, source, ws.params, ws.ctl, ws,
                       d_stats_out, first ? 1u : 0u);
  };

  // per-client parameters, shipped as kernel arguments
  uint32_t max_R = 0;
  {
    UploadChunk chunk;
    chunk.n_clients = 0;
    chunk.first_client = 0;
    chunk.n_templates = 0;
    chunk.pad = 0;
    uint32_t refs[kUploadWords];  // the chunk's references, appended behind its templates when it is sent
    bool one_chunk = true;  // all clients' parameters fit one launch's arguments
    bool uploading = false;
    auto send = [&](bool last) {
      std::memcpy(&chunk.data[chunk.n_templates * kParamWords], refs, (size_t)chunk.n_clients * kRefWords * 4u);
      one_chunk = one_chunk && last;
      if (is_short && one_chunk) {
        short_select(chunk, chunk.n_clients, true);
        return;
      }
      if (!uploading) profile_mark(CVLC_STAGE_ENC_SETUP, true, stream);
      uploading = true;
      const uint32_t blocks = zero_n16 ? (zero_n16 + 1023u) / 1024u : 1u;
      hipLaunchKernelGGL(upload_kernel, dim3(blocks < 512u ? blocks : 512u), dim3(256), 0, stream,
                         reinterpret_cast<uint32_t*>(ws.params), chunk, reinterpret_cast<uint4*>(base + L.status),
                         zero_n16);
      zero_n16 = 0;  // cleared by the first launch
      chunk.first_client += chunk.n_clients;
      chunk.n_clients = 0;
      chunk.n_templates = 0;
    };
    for (uint32_t i = 0; i < n; ++i) {
      const cvlc_plan_t& pl = plans[i];
      ClientParams cp;
      std::memset(&cp, 0, sizeof(cp));  // pointers and client id stay out of the template
      cp.R = pl.n_coded;
      cp.total_words = (uint32_t)(pl.total_bits / 32u);
      cp.B = pl.B;
      uint32_t z = 0;
      for (uint32_t r = 0; r < pl.n_coded; ++r) {
        z += pl.count[r];
        cp.Z[r] = z;
        cp.y[r] = (uint8_t)pl.code_len[r];
      }
      cp.k = z;
      cp.sample_rank = sample_rank(d, z, n_s * kSamplePiece);
      if (pl.n_coded > max_R) max_R = pl.n_coded;
      for (int attempt = 0; attempt < 2; ++attempt) {
        uint32_t t = 0;
        while (t < chunk.n_templates && std::memcmp(&chunk.data[t * kParamWords], &cp, sizeof(cp)) != 0) ++t;
        const uint32_t templates = t == chunk.n_templates ? t + 1 : chunk.n_templates;
        if (templates * kParamWords + (chunk.n_clients + 1) * kRefWords > kUploadWords) {
          send(false);  // no room: this client opens the next chunk (which always has room for one)
          continue;
        }
        if (t == chunk.n_templates) {
          std::memcpy(&chunk.data[t * kParamWords], &cp, sizeof(cp));
          chunk.n_templates = templates;
        }
        uint32_t* ref = refs + chunk.n_clients * kRefWords;
        const uint64_t up = reinterpret_cast<uint64_t>(d_updates[i]), sp = reinterpret_cast<uint64_t>(d_streams_out[i]);
        ref[0] = (uint32_t)up;
        ref[1] = (uint32_t)(up >> 32);
        ref[2] = (uint32_t)sp;
        ref[3] = (uint32_t)(sp >> 32);
        ref[4] = client_ids[i];
        ref[5] = t;
        ++chunk.n_clients;
        break;
      }
    }
    if (chunk.n_clients) send(true);
    if (uploading) profile_mark(CVLC_STAGE_ENC_SETUP, false, stream);
    if (is_short && !one_chunk) short_select(ParamsUploaded{ws.params}, n, false);
  }

  if (!is_short) {
    {
      StageScope scope(CVLC_STAGE_ENC_SAMPLE, stream);
      // also for plans that keep everything: the selection bins are laid out by the sample.  n_src < 2^26 and n_s <= 2^12: the step is below 2^58 / n_s and j * step below 2^58
      if (n_s)
        hipLaunchKernelGGL(sample_hist_kernel, dim3(kSampleBlocks, n), dim3(kWideBlock), 0, stream, ws.params, ws.ctl, n_s,
                           ((uint64_t)n_src << 32) / n_s);
      hipLaunchKernelGGL(sample_walk_kernel, dim3(n), dim3(kWideBlock), 0, stream, ws.params, ws.ctl);
    }
    {
      StageScope scope(CVLC_STAGE_ENC_FILTER, stream);
      hipLaunchKernelGGL(filter_kernel, dim3(ws.filter_blocks, n), dim3(kBlock), 0, stream, ws.params, ws.ctl, ws);
    }
    {
      StageScope scope(CVLC_STAGE_ENC_REFILTER, stream);
      hipLaunchKernelGGL(scan_l1_kernel, dim3(n), dim3(kWideBlock), 0, stream, ws.params, ws.ctl, ws);
    }
    {
      StageScope scope(CVLC_STAGE_ENC_SELECT, stream);
      // the gather also builds the dense candidate list (also when nothing is coded)
      hipLaunchKernelGGL(gather_kernel, dim3(L.gather_blocks, n), dim3(kGatherBlock), 0, stream, ws.params, ws.ctl, ws);
      if (max_R)
        hipLaunchKernelGGL(select_kernel, dim3(max_R, n), dim3(kSelectBlock), 0, stream, ws.params, ws.ctl, ws);
    }
  }
  const PassMode mode = is_short ? kShortVec : (chunks_pay(n, plans) ? kByChunks : kByLayout);
  auto by_mode = [&](auto choose) {
    if (mode == kShortVec) return choose(std::integral_constant<PassMode, kShortVec>());
    if (mode == kByChunks) return choose(std::integral_constant<PassMode, kByChunks>());
    return choose(std::integral_constant<PassMode, kByLayout>());
  };
  // count: wavefronts walk the spans; about what the device holds at once (four workgroups per CU)
  uint32_t g_count = (1024u + n - 1) / n;
  if (g_count > (ws.max_spans + kEmitWaves - 1) / kEmitWaves) g_count = (ws.max_spans + kEmitWaves - 1) / kEmitWaves;
  {
    StageScope scope(CVLC_STAGE_ENC_CLASSIFY, stream);
    auto choose = [&](auto m) {
      return quant == CVLC_QUANT_QSGD ? count_kernel<true, decltype(m)::value> : count_kernel<false, decltype(m)::value>;
    };
    hipLaunchKernelGGL(by_mode(choose), dim3(g_count, n), dim3(kEmitBlock), 0, stream, ws.params, ws.ctl, ws, d_stats_out);
  }
  if (mode == kByLayout) {
    StageScope scope(CVLC_STAGE_ENC_LAYOUT, stream);
    hipLaunchKernelGGL(layout_kernel, dim3(n), dim3(kWideBlock), 0, stream, ws.params, ws.ctl, ws, d_stats_out, quant);
  }
  {
    // emit: workgroups walk the chunks; about what the device holds at once (three per CU)
    StageScope scope(CVLC_STAGE_ENC_EMIT, stream);
    uint32_t g_emit = (768u + n - 1) / n;
    const uint32_t max_chunks = (ws.max_spans + kChunkSpans - 1) / kChunkSpans;
    if (g_emit > max_chunks) g_emit = max_chunks;
    const bool err = flags & CVLC_ENCODE_ERROR_STATS, qsgd = quant == CVLC_QUANT_QSGD;
    auto choose = [&](auto m) {
      constexpr PassMode kMode = decltype(m)::value;
      return err ? (qsgd ? emit_kernel<true, true, kMode> : emit_kernel<true, false, kMode>)
                 : (qsgd ? emit_kernel<false, true, kMode> : emit_kernel<false, false, kMode>);
    };
    hipLaunchKernelGGL(by_mode(choose), dim3(g_emit, n), dim3(kEmitBlock), 0, stream, ws.params, ws.ctl, ws, seed, d_stats_out);
  }
  return hip_check(hipGetLastError());
}

int cvlc_encode(const cvlc_plan_t* plan, const float* d_update, uint64_t seed, uint32_t client_id,
                void* d_stream_out, size_t capacity, void* d_workspace, size_t ws_bytes,
                cvlc_seg_stats_t* d_stats_out, uint32_t flags, void* hip_stream) {
  if (!plan) return CVLC_ERR_ARG;
  const float* updates[1] = {d_update};
  void* streams[1] = {d_stream_out};
  return cvlc_encode_batch(1, plan, updates, seed, &client_id, streams, &capacity, d_workspace, ws_bytes,
                           d_stats_out, flags, hip_stream);
}

int cvlc_device_status(const void* d_workspace, void* hip_stream, uint32_t* status_out) {
  if (!d_workspace || !status_out) return CVLC_ERR_ARG;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  int rc = cvlc::hip_check(hipStreamSynchronize(stream));
  if (rc) return rc;
  return cvlc::hip_check(hipMemcpy(status_out, d_workspace, sizeof(uint32_t), hipMemcpyDeviceToHost));
}

}  // extern "C"
