// Parameter-server side of libcvlc for gfx950: decode n clients' streams and
// aggregate them into one dense fp32 vector (Sec. III step 3 with the 1/B
// scaling of Sec. IV-B):  out[j] = sum_i w_i * xhat_{i,j}.
//
// Records are stored per (client, group) in ascending position, so every such
// list is sorted.  Each workgroup owns a tile of output coordinates, pulls the
// slice of every list that falls into its tile, accumulates in LDS in fp64 and
// writes the tile once; nothing is scattered into global memory.
//   stream_table   validate headers (which must name the quantiser the caller
//                  expects), number the lists, and in one streaming pass over all
//                  records find, for every list, the first record of every output
//                  tile (and check order and range)
//   parse_headers, compact_lists, tile_table
//                  the same in three launches, for more than 112 streams
//   decode_tiles   fused decode + accumulate + single write of each tile (a second
//                  instance splits QSGD's sign bit from the level)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "cvlc_common.h"

namespace cvlc {
namespace {

constexpr uint32_t kListsPerClient = 32;   // descriptor slots per client (CVLC_MAX_CODED used)
constexpr uint32_t kTabChunk = 512;        // records per tile_table work item (one wavefront, eight a lane)

// LDS accesses of one wavefront complete in order; this keeps the compiler from
// moving them across the point where lanes read what other lanes wrote.
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

struct CompactDesc {  // one (client, group) record list, 32 bytes
  const uint32_t* payload;
  double weight;  // w_i
  uint32_t P;
  uint32_t wsy;   // W | s << 8 | y << 16
  float m, step;
};
static_assert(sizeof(CompactDesc) == 32, "CompactDesc is read as two 16-byte pieces");

struct DecodeCtl {  // written by stream_table or compact_lists
  uint32_t n_active;  // lists with records
  uint32_t n_items;   // compact_lists: tile_table work items in all
  uint32_t sparse;    // stream_table: some lists are empty; a list's row of the table is then not its number but row_of[number]
};

struct DecodeLayout {
  size_t status, ctl, stream_bad, desc, cdesc, item_start, table, total;
  uint32_t n_lists;
};

size_t align256(size_t v) { return (v + 255u) & ~(size_t)255u; }

struct StreamArg {  // per-stream inputs, passed as kernel arguments
  const uint32_t* words;
  uint64_t n_words;
  double weight;
  uint32_t has_weight;  // 0: derive 1/(n*B) from the header
  uint32_t pad;
};

uint32_t tiles_of(uint32_t d, uint32_t shift) { return (uint32_t)(((uint64_t)d + (1u << shift) - 1u) >> shift); }

uint32_t tile_shift_for(uint32_t d) { return d >= kDecLargeFrom ? kDecShiftMax : kDecShiftMin; }

DecodeLayout decode_layout(uint32_t d, uint32_t n) {
  DecodeLayout L;
  L.n_lists = n * kListsPerClient;
  size_t off = 0;
  L.status = off; off = align256(off + 256);
  L.ctl = off; off = align256(off + sizeof(DecodeCtl));
  L.stream_bad = off; off = align256(off + (size_t)n * sizeof(uint32_t));
  L.desc = off; off = align256(off + (size_t)L.n_lists * sizeof(ListDesc));
  L.cdesc = off; off = align256(off + (size_t)L.n_lists * sizeof(CompactDesc));
  L.item_start = off; off = align256(off + ((size_t)L.n_lists + 1) * sizeof(uint32_t));
  L.table = off; off = align256(off + (size_t)(tiles_of(d, kDecShiftMin) + 1) * L.n_lists * sizeof(uint32_t));
  L.total = off;
  return L;
}

// The streams' pointers, sizes and weights travel as kernel arguments of the
// header pass (no pinned memory, no synchronisation), up to kParseStreams a launch.
constexpr uint32_t kParseStreams = 112;
struct ParseChunk {
  uint32_t first, count, pad[2];
  StreamArg args[kParseStreams];
};
static_assert(sizeof(ParseChunk) <= 3800, "kernel arguments are limited to 4 KB");

// ------------------------------------------------------------------ 1. headers
// One wavefront per stream; lane r reads and checks the header of group r, so
// that the group headers are fetched together.  A stream that fails any check
// contributes nothing: all its lists are marked empty and the status bit is set.
typedef const uint32_t __attribute__((address_space(1))) * GlobalConstWordPtr;

__device__ __forceinline__ uint64_t wave_incl_scan_u64(uint64_t v) {
  const uint32_t lane = lane_id();
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t lo = __shfl_up((uint32_t)v, o, 64), hi = __shfl_up((uint32_t)(v >> 32), o, 64);
    if (lane >= (uint32_t)o) v += ((uint64_t)hi << 32) | lo;
  }
  return v;
}

// Whole wavefront: the headers of one stream.  Lane r gets list r (no records: P = 0, also past the last group and in a stream
// that fails a check); the result, the same for all lanes, is whether all checks held.
__device__ __forceinline__ bool parse_lists(const StreamArg& sa, uint32_t d, uint32_t n, uint32_t quant, ListDesc* list) {
  const uint32_t t = lane_id();
  GlobalConstWordPtr w = (GlobalConstWordPtr)sa.words;
  bool ok = sa.n_words >= kGlobalHeaderWords;  // everything about `ok` is uniform over the wavefront
  uint32_t g[kGlobalHeaderWords] = {0, 0, 0, 0, 0, 0, 0, 0};
  // The group headers are asked for together with the global header, before the number of groups is known
  // (lane r: where group r's header would be, clamped to the stream), so that one memory round trip serves both.
  uint32_t hw[kSegHeaderWords] = {0, 0, 0, 0};
  if (ok) {
#pragma unroll
    for (uint32_t i = 0; i < kGlobalHeaderWords; ++i) g[i] = w[i];
#pragma unroll
    for (uint32_t i = 0; i < kSegHeaderWords; ++i)
      hw[i] = w[min((uint64_t)(kGlobalHeaderWords + kSegHeaderWords * min(t, CVLC_MAX_CODED - 1u) + i), sa.n_words - 1u)];
  }
  const uint32_t R = g[3], s = g[4];
  const float B = __uint_as_float(g[5]);
  ok = ok && g[0] == kMagic && g[1] == (kVersion | (quant << 16)) && g[2] == d && R <= CVLC_MAX_CODED && s == position_bits(d) &&
       B > 0.0f && fabsf(B) <= 3.4028234664e38f;
  const uint64_t first_payload = kGlobalHeaderWords + (uint64_t)kSegHeaderWords * R;
  ok = ok && sa.n_words >= first_payload;
  const bool mine = ok && t < R;
  uint32_t y = 0, P = 0;
  float m = 0.0f, M = 0.0f;
  if (mine) {  // t < R <= 31 and the stream holds all R headers: the words read above are group t's
    y = hw[0];
    P = hw[1];
    m = __uint_as_float(hw[2]);
    M = __uint_as_float(hw[3]);
  }
  bool header_ok = !mine || (code_len_supported(y) && fabsf(m) <= 3.4028234664e38f &&
                             fabsf(M) <= 3.4028234664e38f && fabsf(M - m) <= 3.4028234664e38f);
  if (quant == CVLC_QUANT_QSGD && mine)  // {norm, 0}; a sign bit and at least one level bit
    header_ok = header_ok && y >= 2 && m >= 0.0f && __float_as_uint(M) == 0u;
  ok = ok && __ballot(header_ok) == ~0ull;
  // where every group's records start, and what the stream must add up to (sizes of groups with a bad header
  // do not matter: the stream is rejected)
  const uint64_t words = mine && header_ok ? payload_words(P, s + y) : 0u;
  const uint64_t incl = wave_incl_scan_u64(words);
  const uint64_t k_incl = wave_incl_scan_u64(mine ? P : 0u);
  const uint64_t total = first_payload + (((uint64_t)__shfl((uint32_t)(incl >> 32), 63, 64) << 32) | __shfl((uint32_t)incl, 63, 64));
  const uint64_t k = ((uint64_t)__shfl((uint32_t)(k_incl >> 32), 63, 64) << 32) | __shfl((uint32_t)k_incl, 63, 64);
  ok = ok && k <= d && total == g[7] && sa.n_words >= total;
  ListDesc ld;
  ld.payload = nullptr; ld.weight = 0.0; ld.P = 0; ld.W = 0; ld.s = 0; ld.y = 0; ld.m = 0.0f; ld.step = 0.0f;
  {
    if (ok && t < R) {
      float step = 0.0f, inv = 0.0f;
      if (y != 32) {
        if (quant == CVLC_QUANT_QSGD) {  // levels 0 .. 2^(y-1) - 1 on [0, norm]
          centroid_spacing(0.0f, m, y - 1u, &step, &inv);
          m = 0.0f;
        } else {
          centroid_spacing(m, M, y, &step, &inv);
        }
      }
      ld.payload = sa.words + (first_payload + incl - words);
      ld.weight = sa.has_weight ? sa.weight : 1.0 / ((double)n * (double)B);
      ld.P = P;
      ld.s = s;
      ld.y = y;
      ld.W = s + y;
      ld.m = m;
      ld.step = step;
    }
  }
  *list = ld;
  return ok;
}

__global__ __launch_bounds__(64) void parse_headers_kernel(ParseChunk chunk, ListDesc* descs, uint32_t d, uint32_t n,
                                                           uint32_t* __restrict__ stream_bad, uint32_t quant) {
  const uint32_t t = lane_id(), client = chunk.first + blockIdx.x;
  ListDesc list;
  const bool ok = parse_lists(chunk.args[blockIdx.x], d, n, quant, &list);
  if (t == 0) stream_bad[client] = ok ? 0u : 1u;  // gathered into the status word by the next kernel
  if (t < kListsPerClient) descs[(size_t)client * kListsPerClient + t] = list;
}

// ------------------------------------------------------------------ 1b. the non-empty lists
// One workgroup of 1024 threads.  Lists with records are numbered in (client,
// group) order; item_start is the exclusive prefix of their tile_table work items.
__global__ __launch_bounds__(1024) void compact_lists_kernel(const ListDesc* __restrict__ descs, uint32_t n_lists,
                                                             CompactDesc* __restrict__ cdesc,
                                                             uint32_t* __restrict__ item_start, DecodeCtl* ctl,
                                                             const uint32_t* __restrict__ stream_bad, uint32_t n,
                                                             uint32_t* status) {
  __shared__ uint32_t scan_tmp[16];
  const uint32_t tid = threadIdx.x;
  // the call's status word starts here: set if any stream failed its header checks
  uint32_t any_bad = 0;
  for (uint32_t i = tid; i < n; i += 1024) any_bad |= stream_bad[i];
  any_bad = __syncthreads_or((int)any_bad) ? 1u : 0u;
  if (tid == 0) *status = any_bad ? CVLC_DEV_STREAM : 0u;
  uint32_t lists_before = 0, items_before = 0;
  for (uint32_t base = 0; base < n_lists; base += 1024) {
    const uint32_t l = base + tid;
    ListDesc ld;
    ld.P = 0;
    if (l < n_lists) ld = descs[l];
    const uint32_t live = ld.P > 0 ? 1u : 0u;
    const uint32_t items = (ld.P + kTabChunk - 1) / kTabChunk;
    uint32_t tot_l, tot_i;
    const uint32_t pos = lists_before + block_excl_scan<16>(live, scan_tmp, &tot_l);
    const uint32_t first = items_before + block_excl_scan<16>(items, scan_tmp, &tot_i);
    if (live) {
      CompactDesc c;
      c.payload = ld.payload; c.weight = ld.weight; c.P = ld.P; c.wsy = ld.W | (ld.s << 8) | (ld.y << 16);
      c.m = ld.m; c.step = ld.step;
      cdesc[pos] = c;
      item_start[pos] = first;
    }
    lists_before += tot_l;
    items_before += tot_i;
  }
  if (tid == 0) {
    item_start[lists_before] = items_before;
    ctl->n_active = lists_before;
    ctl->n_items = items_before;
    ctl->sparse = 0;
  }
}

// ------------------------------------------------------------------ 2. tile table
// table[list][t] = index of the first record of `list` whose position lies in
// output tile t or later; entry n_tiles holds the list length.  (List-major: a
// list's entries are written in ascending t by neighbouring threads.)  A work
// item is a run of kTabChunk records of one list and belongs to one wavefront:
// lane l reads the position fields of records l, l + 64, ... of the run straight
// from the stream (neighbouring lanes, neighbouring words), all of them in flight
// together, and compares each with the one before it.  Wavefronts never wait for
// each other.  The pass also checks that positions ascend and stay below d.
// A position is one load of four bytes from the byte it starts in (two aligned words a record before: half of the
// kernel's loads): 24.5 -> 20.2 us for 32 streams of 11.2 M coordinates and, with the search below, 203 -> 142 us
// for 100 of 25.6 M.
constexpr uint32_t kTabTurns = kTabChunk / kWave;  // records of an item a lane looks at

// Fields at any bit: one load from the byte the field starts in (global loads need no alignment).
struct __attribute__((packed, aligned(1))) Bytes4 { uint32_t v; };
struct __attribute__((packed, aligned(1))) Bytes8 { uint64_t v; };
typedef const unsigned char __attribute__((address_space(1))) * GlobalBytePtr;
__device__ __forceinline__ uint32_t load4(GlobalBytePtr p) { return ((const Bytes4 __attribute__((address_space(1)))*)p)->v; }
__device__ __forceinline__ uint64_t load8(GlobalBytePtr p) { return ((const Bytes8 __attribute__((address_space(1)))*)p)->v; }

// The list that owns item q: the last one with item_start <= q; its first item and the next list's.
struct ItemOwner {
  uint32_t list, first_item, next_list;
};
// Whole wavefront, 64 probes a round: one round for up to 64 lists, two for up to 4096.  The last round's lanes hold the two starts.
// (A binary search by every lane costs log2 rounds: beyond 2048 lists it was twelve dependent loads per item and two thirds
// of the kernel.)
__device__ __forceinline__ ItemOwner owner_of(const uint32_t* __restrict__ item_start, uint32_t n_active, uint32_t q) {
  const uint32_t lane = lane_id();
  uint32_t a = 0, len = n_active;  // the owner is one of a .. a + len - 1
  while (len > kWave) {  // uniform
    const uint32_t step = (len + kWave - 1u) / kWave;
    const bool hit = lane * step < len && item_start[min(a + lane * step, n_active)] <= q;
    const uint32_t last = (uint32_t)__popcll(__ballot(hit)) - 1u;  // item_start ascends and its first entry is 0: the hits are a prefix
    a += last * step;
    len = min(step, len - last * step);
  }
  const uint32_t start = item_start[min(a + lane, n_active)];
  const uint32_t last = (uint32_t)__popcll(__ballot(lane < len && start <= q)) - 1u;
  ItemOwner o;
  o.list = __builtin_amdgcn_readfirstlane(a + last);
  o.first_item = __builtin_amdgcn_readlane(start, last);
  o.next_list = __builtin_amdgcn_readlane(start, min(last + 1u, kWave - 1u));
  if (last == kWave - 1u) o.next_list = item_start[o.list + 1u];  // uniform
  return o;
}
constexpr uint32_t kTableBlocks = 2048;  // workgroups of tile_table, eight per CU

// Item q of list a (descriptor d0, d1, its first item `first_item`), whole wavefront.  Returns whether a lane's record is out of
// order or of range.  WIDE: positions of more than 25 bits, which need not lie in the four bytes from the one they start in.
template <bool WIDE>
__device__ __forceinline__ bool table_item(uint4 d0, uint4 d1, uint32_t a, uint32_t first_item, uint32_t q, uint32_t* table,
                                           uint32_t d, uint32_t tile_shift, uint32_t n_tiles) {
  const uint32_t lane = lane_id();
  bool bad = false;
  // the list's descriptor is the same for all lanes: keeping it in scalar registers keeps the address
  // arithmetic of the loads below off the vector unit
  const uint64_t pay = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(d0.y) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane(d0.x);
  const uint32_t P = __builtin_amdgcn_readfirstlane(d1.x), wsy = __builtin_amdgcn_readfirstlane(d1.y);
  const uint32_t W = wsy & 0xFFu, s = (wsy >> 8) & 0xFFu;
  const uint32_t pid_mask = (1u << s) - 1u;  // s <= 31
  const uint32_t e0 = (q - first_item) * kTabChunk, cnt = min(P - e0, kTabChunk);
  uint32_t* row = table + (size_t)a * (n_tiles + 1);
  // The window of the item starts at the record before the run (the run's first record for the first
  // item of a list); records are addressed by their number in the window, bits by their offset from the
  // byte `src`, eight before the window's first word (a stream's headers lie in front of its first payload, so
  // the bytes are there): everything stays far below 2^24.
  const uint32_t lead = e0 ? 1u : 0u;
  const uint64_t bit0 = (uint64_t)(e0 - lead) * W;
  GlobalBytePtr src = (GlobalBytePtr)(pay + (bit0 >> 5) * 4u - 8u);
  const uint32_t sh0 = ((uint32_t)bit0 & 31u) + 64u;
  // the last place a whole load may start at: the list's payload ends there
  const uint64_t left = (((uint64_t)P * W + 31u) >> 5) * 4u - (bit0 >> 5) * 4u + 8u - (WIDE ? 8u : 4u);
  const uint32_t rel_last = left < (1u << 24) ? (uint32_t)left : 1u << 24;
  // position field of record r of the window
  auto request = [&](uint32_t r, uint32_t& sh) {
    const uint32_t bit = sh0 + __umul24(r, W), at = min(bit >> 3, rel_last);
    sh = bit - at * 8u;
    if constexpr (WIDE) return load8(src + at); else return load4(src + at);
  };
  decltype(request(0u, a)) w[kTabTurns], c_w;
  uint32_t sh[kTabTurns], c_sh;
  c_w = request(0u, c_sh);  // the record before the run (uniform)
#pragma unroll
  for (uint32_t i = 0; i < kTabTurns; ++i)  // no branch: a lane past the end reads the last record again
    w[i] = request(lead + min(i * kWave + lane, cnt - 1u), sh[i]);
  uint32_t carry = (uint32_t)(c_w >> c_sh) & pid_mask;
#pragma unroll
  for (uint32_t i = 0; i < kTabTurns; ++i) {
    if (i * kWave >= cnt) break;  // uniform
    const uint32_t j = i * kWave + lane;
    const bool live = j < cnt;
    const uint32_t e = e0 + j;
    const uint32_t pid = (uint32_t)(w[i] >> sh[i]) & pid_mask;
    // the record before mine sits in the lane below; lane 0 takes the last one of the turn before
    const uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp((int)carry, (int)pid, 0x138 /* wave_shr:1 */, 0xF, 0xF, false);
    carry = __builtin_amdgcn_readlane(pid, kWave - 1);
    // a position past the end (an error, reported below) counts as lying behind the last tile
    const uint32_t t_cur = min(pid >> tile_shift, n_tiles), t_prev = min(prev >> tile_shift, n_tiles);
    const bool first = e == 0, last = e == P - 1;
    bad |= live && ((!first && prev >= pid) || pid >= d);  // positions must ascend strictly and stay below d
    // entries (tile of record e-1, tile of record e] point at e; past the last record they hold P
    const bool starts = live && (first || last || t_cur != t_prev);
    if (!__ballot(starts)) continue;
    const uint32_t t_first = first ? 0u : t_prev + 1u;
    const bool single = starts && !last && t_first == t_cur;  // nearly always: the next tile, one entry
    if (single) row[t_cur] = e;
    if (!__ballot(starts && !single)) continue;
    const bool run = starts && !single && t_cur >= t_first;
    uint32_t tail_first = 1, tail_last = 0;
    if (starts && last) {
      tail_first = t_cur + 1;
      tail_last = n_tiles;
    }
    // short runs of entries are written by the lane that found them, long ones (the stretch before a
    // list's first record, after its last, or across a region it skips) by the whole wavefront
    constexpr uint32_t kLong = 16;
    const bool long_run = run && t_cur - t_first >= kLong;
    const bool long_tail = tail_last >= tail_first;
    if (run && !long_run)
      for (uint32_t t = t_first; t <= t_cur; ++t) row[t] = e;
    uint64_t todo = __ballot(long_run);
    while (todo) {
      const uint32_t from = (uint32_t)__builtin_ctzll(todo);
      const uint32_t a0 = __builtin_amdgcn_readlane(t_first, from), a1 = __builtin_amdgcn_readlane(t_cur, from);
      const uint32_t val = __builtin_amdgcn_readlane(e, from);
      for (uint32_t t = a0 + lane; t <= a1; t += kWave) row[t] = val;
      todo &= todo - 1;
    }
    todo = __ballot(long_tail);
    while (todo) {
      const uint32_t from = (uint32_t)__builtin_ctzll(todo);
      const uint32_t a0 = __builtin_amdgcn_readlane(tail_first, from), a1 = __builtin_amdgcn_readlane(tail_last, from);
      for (uint32_t t = a0 + lane; t <= a1; t += kWave) row[t] = P;
      todo &= todo - 1;
    }
  }
  return bad;
}

template <bool WIDE>
__global__ __launch_bounds__(kBlock, 8) void tile_table_kernel(const CompactDesc* __restrict__ cdesc,
                                                         const uint32_t* __restrict__ item_start,
                                                         const DecodeCtl* __restrict__ ctl, uint32_t* table,
                                                         uint32_t d, uint32_t tile_shift, uint32_t n_tiles, uint32_t* status) {
  const uint32_t tid = threadIdx.x;
  const uint32_t n_active = ctl->n_active, n_items = ctl->n_items;
  // A wavefront takes neighbouring items, so that it looks for the owner of the first one only and then walks on.
  constexpr uint64_t n_waves = kTableBlocks * kWavesPerBlock;
  const uint64_t me = blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(tid / kWave);
  // Few items go to the first workgroups, which start a microsecond before the last ones.
  uint32_t q_begin = (uint32_t)(me * n_items / n_waves), q_end = (uint32_t)((me + 1u) * n_items / n_waves);
  if (n_items <= n_waves) {
    q_begin = min((uint32_t)me, n_items);
    q_end = min((uint32_t)me + 1u, n_items);
  }
  if (q_begin >= q_end) return;  // uniform
  const ItemOwner owner = owner_of(item_start, n_active, q_begin);
  uint32_t a = owner.list, first_item = owner.first_item, next_list = owner.next_list;  // uniform
  bool bad = false;
  for (uint32_t q = q_begin; q < q_end; ++q) {  // uniform per wavefront
    while (q >= next_list) {  // every list has an item: one step at most
      ++a;
      first_item = next_list;
      next_list = item_start[a + 1u];
    }
    const uint4* dsrc = reinterpret_cast<const uint4*>(cdesc + a);
    bad |= table_item<WIDE>(dsrc[0], dsrc[1], a, first_item, q, table, d, tile_shift, n_tiles);
  }
  if (bad) atomicOr(status, CVLC_DEV_STREAM);
}

// ---- up to 112 streams: headers, list numbers and table in one launch
// A workgroup belongs to one stream: its first wavefront parses that stream's headers (and reads the other streams' numbers of
// groups, for the rows of its lists among all), its wavefronts share out the stream's items.  One of the stream's workgroups
// numbers its lists with records: its other wavefronts, which wait for the first one, count those of the streams before.
// (With the empty lists among the numbered ones, which decode_tiles then deals out and sweeps over, 100 x 11.2 M of one group with
// records and 30 without took 74.7 us for 50.4, 30 x 11.2 M of four and 27 53.5 for 46.2.)
// us of the launches before decode_tiles, headers, list numbers and items in launches of their own (up to eight streams: in one, whose
// workgroups each parsed all of them) and now: 32 x 11.2 M 27.0 and 20.9, 100 x 25.6 M 136 and 127, 8 x 1.2 M 8.3 and 7.4.  About
// 6 of them are the headers (every wavefront for itself: 9.6 with 32 streams, at whose few lines all of them queue up).
// What bounds the items is the read of the streams and, of 100 x 25.6 M, 39 MB of table written in between.  Level or slower
// (us of 100 x 25.6 M): a third of the vector instructions, by turns whose loads share one offset and one shift, 137; loads eight
// turns ahead 137; 16-byte loads an item ahead through LDS 135 (the loads alone 80, dwords 98); the items of neighbouring
// wavefronts side by side 129 (neighbouring stores of a list's row then come from two XCDs).
template <uint32_t STREAMS>
struct StreamArgs {
  uint32_t count, blocks;
  StreamArg args[STREAMS];
  uint16_t first[STREAMS];  // the stream's first workgroup
};
constexpr uint32_t kFewStreams = 8;  // whose arguments take 300 bytes instead of 3.8 KB
static_assert(sizeof(StreamArgs<kParseStreams>) <= 3840, "kernel arguments are limited to 4 KB");
struct TableShared {
  uint64_t payload[kWave];
  uint32_t P[kWave], wsy[kWave], first[kWave];
  uint32_t before, bad;
  uint32_t live_before[kWavesPerBlock];
};

// Whether the stream's header says that its group g has records, be the header right or wrong.
__device__ __forceinline__ bool names_records(const StreamArg& sa, uint32_t g) {
  GlobalConstWordPtr w = (GlobalConstWordPtr)sa.words;
  const uint32_t groups = w[3], P = w[min((uint64_t)(kGlobalHeaderWords + kSegHeaderWords * g + 1u), sa.n_words - 1u)];
  return g < min(groups, CVLC_MAX_CODED) && P != 0u;
}

template <bool WIDE, uint32_t STREAMS>
__global__ __launch_bounds__(kBlock, 8) void stream_table_kernel(StreamArgs<STREAMS> in, uint32_t quant, CompactDesc* __restrict__ cdesc,
                                                                 DecodeCtl* ctl, uint32_t* __restrict__ row_of, uint32_t* table, uint32_t d,
                                                                 uint32_t tile_shift, uint32_t n_tiles, uint8_t* __restrict__ found,
                                                                 uint32_t* status) {
  __shared__ TableShared S;
  const uint32_t lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  constexpr uint32_t kTurns = (STREAMS + kWave - 1u) / kWave;
  uint32_t client = 0, first_block = 0;
#pragma unroll
  for (uint32_t i = 0; i < kTurns; ++i) {
    const uint32_t c = i * kWave + lane, f = in.first[min(c, in.count - 1u)];
    const uint64_t at_or_before = __ballot(c < in.count && f <= blockIdx.x);  // firsts ascend: a prefix
    if (at_or_before) first_block = __builtin_amdgcn_readlane(f, 63u - (uint32_t)__builtin_clzll(at_or_before));
    client += (uint32_t)__popcll(at_or_before);
  }
  client = __builtin_amdgcn_readfirstlane(client - 1u);
  const uint32_t blocks = __builtin_amdgcn_readfirstlane((client + 1u < in.count ? in.first[client + 1u] : in.blocks) - first_block);
  // The stream's workgroup that numbers its lists: of as many streams as a power of two the first ones would all be on a few CUs of
  // one XCD (32 x 11.2 M: the launch 28 us instead of 22).
  const bool leads = blockIdx.x == first_block + client % blocks;  // uniform
  ListDesc list;
  uint32_t groups = 0;
  if (wave == 0) {
    // at most 31 lists a stream whatever its header says
    uint32_t before = 0;
#pragma unroll
    for (uint32_t i = 0; i < kTurns; ++i) {
      const uint32_t c = i * kWave + lane;
      const uint32_t g = c <= client ? min(((GlobalConstWordPtr)in.args[min(c, client)].words)[3], CVLC_MAX_CODED) : 0u;
      before += c < client ? g : 0u;
      groups += c == client ? g : 0u;
    }
    const bool ok = parse_lists(in.args[client], d, in.count, quant, &list);
    before = wave_sum_u32(before);
    groups = wave_sum_u32(groups);
    const uint32_t items = (list.P + kTabChunk - 1u) / kTabChunk;
    S.payload[lane] = (uint64_t)list.payload;
    S.P[lane] = list.P;
    S.wsy[lane] = list.W | (list.s << 8) | (list.y << 16);
    S.first[lane] = wave_incl_scan_u32(items) - items;  // lanes past the last list: the number of items
    if (lane == 0) {
      S.before = before;
      S.bad = ok ? 0u : 1u;
    }
  } else if (leads) {
    constexpr uint32_t kStep = 2u * (kWavesPerBlock - 1u), kDeep = 4u;  // streams looked at together, half a wavefront each, and times over
    uint32_t live = 0;
    for (uint32_t base = 0; base < client; base += kDeep * kStep) {
      bool names[kDeep];
#pragma unroll
      for (uint32_t u = 0; u < kDeep; ++u) {
        const uint32_t c = base + u * kStep + (wave - 1u) * 2u + (lane >> 5);
        names[u] = names_records(in.args[min(c, client)], lane & 31u) && c < client;  // no branch around the loads
      }
#pragma unroll
      for (uint32_t u = 0; u < kDeep; ++u) live += (uint32_t)__popcll(__ballot(names[u]));
    }
    if (lane == 0) S.live_before[wave] = live;
  }
  __syncthreads();
  if (leads && wave == 0) {
    uint32_t live = 0;
    for (uint32_t w = 1; w < kWavesPerBlock; ++w) live += S.live_before[w];
    const bool mine = names_records(in.args[client], min(lane, CVLC_MAX_CODED));
    const uint64_t mask = __ballot(mine);
    if (mine) {  // a refused stream's lists have no records
      const uint32_t number = live + lanes_below(mask);
      CompactDesc c;
      c.payload = list.payload; c.weight = list.weight; c.P = list.P; c.wsy = S.wsy[lane];
      c.m = list.m; c.step = list.step;
      cdesc[number] = c;
      row_of[number] = S.before + lane;
    }
    if (lane == 0 && client == in.count - 1u) {
      live += (uint32_t)__popcll(mask);
      ctl->n_active = live;
      ctl->sparse = live != S.before + groups;
      *status = 0;  // what the workgroups find goes to a byte of each, which decode_tiles adds to it
    }
  }
  const uint32_t first = S.first[lane], before = __builtin_amdgcn_readfirstlane(S.before);
  const uint32_t n_items = __builtin_amdgcn_readlane(first, kWave - 1u);
  const uint32_t n_waves = blocks * kWavesPerBlock, me = (blockIdx.x - first_block) * kWavesPerBlock + wave;
  bool bad = S.bad != 0u;
  // neighbouring items to a wavefront; few of them to the workgroups that start first
  uint32_t q = (uint32_t)((uint64_t)me * n_items / n_waves), q_end = (uint32_t)((uint64_t)(me + 1u) * n_items / n_waves);
  if (n_items <= n_waves) {
    q = min(me, n_items);
    q_end = min(me + 1u, n_items);
  }
  for (; q < q_end; ++q) {  // uniform per wavefront
    const uint32_t a = (uint32_t)__popcll(__ballot(first <= q)) - 1u;  // a list without records has no item of its own
    const uint64_t payload = S.payload[a];
    bad |= table_item<WIDE>(make_uint4((uint32_t)payload, (uint32_t)(payload >> 32), 0u, 0u), make_uint4(S.P[a], S.wsy[a], 0u, 0u), before + a,
                            __builtin_amdgcn_readlane(first, a), q, table, d, tile_shift, n_tiles);
  }
  const int any = __syncthreads_or((int)bad);
  if (threadIdx.x == 0) found[blockIdx.x] = any ? 1u : 0u;
}

// ------------------------------------------------------------------ 3. fused decode + accumulate
// Persistent workgroups walk the output tiles, neighbouring tiles at the same
// time on the same XCD (see tile_of below).  The lists are dealt out to the wavefronts, up to 64 each, lane i the
// list of one: lane i knows its list's descriptor and asks for the two table entries of its slice.  The
// records of the wavefront's slices are numbered 0..total-1 (an exclusive scan of the slice lengths), and
// the wavefront goes through them 64 at a time ("turn"), so that neighbouring lanes read neighbouring
// records.  Which slice a lane's record belongs to: the slices that start inside the turn set a bit at their
// first record's place in a 64-bit mask, and a lane counts the bits at or below its own place; what it needs of the
// slice it reads from LDS.  Wavefronts wait for each other twice a tile only: before it is written out, and
// before the next tile's first value is added.
// What bounds it: latencies, and cache lines.  A pair of table entries, a descriptor and a slice's records are a line each,
// however little of it is used, and a slice holds a handful of records.
// Hence tiles of 8192 coordinates, two workgroups a CU, where they are enough to go round: from 2^23 coordinates on, two
// tiles for every workgroup (us a call, tiles of 4096 and 8192: 100 x 25.6 M 550 and 407, 8 x 11.2 M 39.1 and 35.8, 32 x
// 11.2 M Gauss 61.9 and 57.0, layers 68 and 68; 32 x 5 M 44 and 53, 8 x 5 M 24.7 and 26.3).  With the records shared out evenly
// over all wavefronts, three barriers and a search a tile, and tiles of 4096: 600, 44.0, 69.3, 75, 48.5 and 28.7.
constexpr uint32_t kChunkTiles = 16; // consecutive tiles decoded side by side on one XCD (more: less refetching, less even load)

constexpr uint32_t kDecBlock = 512;  // threads of a decode workgroup
constexpr uint32_t kDecWaves = kDecBlock / kWave;
constexpr uint32_t kWaveLists = 60;  // lists a wavefront has in a sweep at most (64 would not fit twice into a CU with the large tile)
constexpr uint32_t kDecLists = kWaveLists * kDecWaves;  // ... and a workgroup

// Turns of 64 records a wavefront works on together, in two halves: as many as the registers hold with three workgroups a CU
// (small tiles) and with two (large ones, 64 KB of sums).
constexpr uint32_t half_turns(uint32_t tile_shift) { return tile_shift == kDecShiftMin ? 3u : 4u; }

// What the lanes need of a slice, set aside by the lane that owns its list.  `at` is a byte offset from `src`, eight
// bytes before the byte in which the slice's first record starts (a stream's headers lie in front of its first payload, so the
// bytes are there).
struct SliceInfo {
  uint4 where;  // src (two words); the bit offset from src of the record numbered 0; last `at` a load may use | W << 16 | y << 24
  uint4 value;  // weight (two words), m, step
};
template <uint32_t SHIFT>
struct DecodeShared {
  double acc[1u << SHIFT];
  SliceInfo slice[kDecWaves][kWaveLists];  // per wavefront: its non-empty slices, in order
  unsigned long long turn_mask[kDecWaves][2u * half_turns(SHIFT)];  // ... and the starts of slices inside each of its current turns
};
static_assert(((1u << kDecShiftMax) + kWave) * 63u / 8u + 8u < (1u << 16), "a slice's bytes are counted in 16 bits");
static_assert(((uint64_t)kWaveLists << kDecShiftMax) + kWave < (1u << 24), "a wavefront's records are numbered in 24 bits");

// Inclusive prefix sum over the 64 lanes, all of them active: adds within rows of sixteen, then across (no LDS round trips).
__device__ __forceinline__ uint32_t wave_incl_scan_rows(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111 /* row_shr:1 */, 0xF, 0xF, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112 /* row_shr:2 */, 0xF, 0xF, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114 /* row_shr:4 */, 0xF, 0xF, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118 /* row_shr:8 */, 0xF, 0xF, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142 /* row_bcast:15 */, 0xA, 0xF, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143 /* row_bcast:31 */, 0xC, 0xF, false);
  return v;
}

// SIGNED: the streams' codes hold a sign bit above the level (QSGD).
// WIDE: positions of more than 25 bits, which with a raw 32-bit code may not lie in eight bytes from the one they start in.
template <bool SIGNED, bool WIDE, uint32_t SHIFT>
__global__ __launch_bounds__(kDecBlock, SHIFT == kDecShiftMin ? 6 : 4) void decode_tiles_kernel(const CompactDesc* __restrict__ cdesc,
                                                              const DecodeCtl* __restrict__ ctl, const uint32_t* __restrict__ row_of,
                                                              const uint32_t* __restrict__ table, float* out,
                                                              uint32_t d, uint32_t n_tiles, uint32_t s, uint32_t accumulate,
                                                              const uint8_t* __restrict__ found, uint32_t n_found,
                                                              uint32_t* status) {
  constexpr uint32_t kTile = 1u << SHIFT, kHalf = half_turns(SHIFT), kTurns = 2u * kHalf;
  __shared__ DecodeShared<SHIFT> S;
  const uint32_t tid = threadIdx.x, lane = lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const uint32_t n_active = __builtin_amdgcn_readfirstlane(ctl->n_active), sparse = __builtin_amdgcn_readfirstlane(ctl->sparse);
  // Sweeps over the lists, of equal length.  In a sweep the lists are dealt out to 1, 2, 4 or 8 groups of wavefronts so that no
  // lane gets two, and wavefronts of the same group share out the records.  One by one where one sweep takes them all (clients
  // differ in what they keep of a layer: four neighbouring lists at a time make a 4 us longer call of 32 streams of 11.2 M
  // coordinates); in fours, a cache line of descriptors, where every sweep reads them anew.  The order turns by one from
  // hand to hand, so that a wavefront does not get the same groups of every client.
  const uint32_t n_sweeps = max((n_active + kDecLists - 1u) / kDecLists, 1u);
  const uint32_t per_sweep = (n_active + n_sweeps - 1u) / n_sweeps;
  const uint32_t group_bits = per_sweep <= kWaveLists ? 0u : per_sweep <= 2u * kWaveLists ? 1u : per_sweep <= 4u * kWaveLists ? 2u : 3u;
  const uint32_t group_mask = (1u << group_bits) - 1u, group = wave & group_mask, part = wave >> group_bits;
  const uint32_t part_records = kDecBlock >> group_bits;  // records of a turn of all the wavefronts of a group
  const uint32_t deal_bits = n_sweeps > 1u ? 2u : 0u, hand = lane >> deal_bits;
  const uint32_t mine = (((hand << group_bits) + ((group + hand) & group_mask)) << deal_bits) + (lane & ((1u << deal_bits) - 1u));  // the lane's list in a sweep
  static_assert(kDecWaves == 8u && kWaveLists % 4u == 0u, "three bits of groups, whole fours");
  bool bad = false;
  // What a lane needs of its list of the sweep at l0: the descriptor, and the two table entries for a tile.  Both
  // are asked for a sweep ahead (a sweep of few records is otherwise little but the chain of waits for descriptors,
  // then table entries, then records).
  auto request_desc = [&](uint32_t l0, uint4 (&dd)[2]) {
    const uint4* src = reinterpret_cast<const uint4*>(cdesc + min(l0 + mine, n_active - 1u));
    dd[0] = src[0];
    dd[1] = src[1];
  };
  auto row_of_mine = [&](uint32_t l0) { return sparse ? row_of[min(l0 + mine, n_active - 1u)] : l0 + mine; };  // uniform
  auto request_rows = [&](uint32_t tile, uint32_t l0, uint32_t row) {
    uint2 r = make_uint2(0u, 0u);
    if (tile < n_tiles && mine < per_sweep && l0 + mine < n_active) {
      const uint64_t two = load8((GlobalBytePtr)(table + (size_t)row * (n_tiles + 1) + tile));
      r.x = (uint32_t)two;
      r.y = (uint32_t)(two >> 32);
    }
    return r;
  };
  // Which tiles a workgroup takes.  Workgroup b runs on XCD b mod 8, and every XCD has an L2 of its own: a
  // tile's slice of a list shares its first and last cache line with the neighbouring tiles', so chunks of
  // kChunkTiles consecutive tiles are decoded at the same time by as many workgroups of one XCD, and the
  // chunks go round the XCDs (whole eighths of the vector per XCD would leave the XCD with the dense layers
  // behind).  Grids that do not divide into such chunks (fewer tiles than the device holds): tile b, b + grid, ...
  const bool chunked = gridDim.x % (8u * kChunkTiles) == 0;
  const uint32_t xcd = blockIdx.x & 7u, seat = blockIdx.x >> 3, chunks_at_once = gridDim.x / (8u * kChunkTiles);
  auto tile_of = [&](uint32_t r) {
    return chunked ? ((seat / kChunkTiles + chunks_at_once * r) * 8u + xcd) * kChunkTiles + seat % kChunkTiles
                   : blockIdx.x + r * gridDim.x;
  };
  uint32_t round = 0, l0 = 0;
  uint2 next_rows = make_uint2(0u, 0u);
  uint4 next_desc[2] = {make_uint4(0u, 0u, 0u, 0u), make_uint4(0u, 0u, 0u, 0u)};
  uint32_t next_row = 0;  // of the list whose table entries are asked for next
  if (n_active) {
    next_row = row_of_mine(0);
    next_rows = request_rows(tile_of(0), 0, next_row);
    request_desc(0, next_desc);
    if (n_sweeps > 1u) next_row = row_of_mine(per_sweep);
  }
  for (uint32_t i = tid; i < kTile; i += kDecBlock) S.acc[i] = 0.0;
  SliceInfo* slices = S.slice[wave];
  unsigned long long* masks = S.turn_mask[wave];
  bool open = false;  // all wavefronts have cleared their part of the tile (uniform)
  for (uint32_t tile = tile_of(0); tile < n_tiles;) {
    const uint32_t lo = tile << SHIFT;
    const uint32_t room = min(kTile, d - lo);  // coordinates of the tile
    const bool last_sweep = l0 + per_sweep >= n_active;  // of the tile
    const uint32_t next_tile = last_sweep ? tile_of(++round) : tile, next_l0 = last_sweep ? 0u : l0 + per_sweep;
    if (n_active) {  // uniform
      const uint2 rows = next_rows;
      const uint4 d0 = next_desc[0], d1 = next_desc[1];
      if (n_sweeps > 1u) request_desc(next_l0, next_desc);
      next_rows = request_rows(next_tile, next_l0, next_row);
      if (n_sweeps > 1u) next_row = row_of_mine(next_l0 + per_sweep >= n_active ? 0u : next_l0 + per_sweep);
      // this lane's list: its slice [begin, end) from two neighbouring table entries (none: both are 0)
      const uint32_t P = d1.x, W = d1.y & 0xFFu;
      const uint32_t begin = min(rows.x, P), end = min(rows.y, P);  // table entries of a malformed list may hold anything
      uint32_t len = end > begin ? end - begin : 0u;
      if (len > kTile) {  // positions ascend strictly: a tile holds at most one record per coordinate
        bad = true;
        len = 0;
      }
      const uint32_t incl = wave_incl_scan_rows(len), before = incl - len;
      const uint32_t total = __builtin_amdgcn_readlane(incl, kWave - 1);
      const uint64_t live = __ballot(len != 0u);
      if (len) {
        const uint64_t bit0 = (uint64_t)begin * W;
        const uint64_t src = (((uint64_t)d0.y << 32) | d0.x) + (bit0 >> 3) - 8u;
        const uint64_t left = payload_words(P, W) * 4u - (bit0 >> 3);  // bytes up to the payload's end: its last eight may be loaded
        SliceInfo& info = slices[lanes_below(live)];
        info.where = make_uint4((uint32_t)src, (uint32_t)(src >> 32), ((uint32_t)bit0 & 7u) + 64u - before * W,
                                (uint32_t)(left < 0xFFFFu ? left : 0xFFFFu) | (W << 16) | ((d1.y >> 16) << 24));
        info.value = make_uint4(d0.z, d0.w, d1.z, d1.w);
      }
      // the wavefront's share of the records, a multiple of 64
      const uint32_t share = ((total + part_records - 1u) / part_records) * kWave;
      const uint32_t q_begin = min(part * share, total), q_end = min(q_begin + share, total);
      // kTurns turns at a time.  First the start masks of all of them; then, half by half but without one
      // turn waiting for another, the slice from LDS and the record's place; then all record loads together, so that their
      // latencies overlap.  Nothing in a half branches on data or on the number of turns (a lane past the end reads the last
      // record again), so that no load has to be waited for before the next one is issued.  A record is read by one load of
      // eight bytes from the byte it starts in (from the payload's last eight bytes where it would reach past them).
      for (uint32_t q0 = q_begin; q0 < q_end; q0 += kWave * kTurns) {
        if (lane < kTurns) masks[lane] = 0ull;
        wave_lds_fence();
        const uint32_t f = before - q0;
        if (len && f < kWave * kTurns) atomicOr(&masks[f >> 6], 1ull << (f & 63u));
        uint32_t cur = (uint32_t)__popcll(__ballot(len && before < q0));  // slices that start before the turns at hand
        wave_lds_fence();
        uint64_t bits_of[kTurns];
        uint32_t tail_of[WIDE ? kTurns : 1];  // the byte behind those eight
        uint32_t at_of[kTurns];               // bits in front of the record, at most 63 | slice << 8 | y << 24
        auto request = [&](auto half) {
          constexpr uint32_t u0 = decltype(half)::value * kHalf;
          uint32_t a_of[kHalf];
          uint4 where[kHalf];
#pragma unroll
          for (uint32_t i = 0; i < kHalf; ++i) {
            const unsigned long long m = masks[u0 + i];
            const uint32_t m_lo = __builtin_amdgcn_readfirstlane((uint32_t)m), m_hi = __builtin_amdgcn_readfirstlane((uint32_t)(m >> 32));
            const uint64_t starts = ((uint64_t)m_hi << 32) | m_lo;
            // slices that start at or before the lane's record, less one; bit 0 counts for every lane
            const uint64_t above = starts >> 1;
            a_of[i] = __builtin_amdgcn_mbcnt_hi((uint32_t)(above >> 32),
                                                __builtin_amdgcn_mbcnt_lo((uint32_t)above, cur + (m_lo & 1u) - 1u));
            cur += (uint32_t)__popcll(starts);
          }
#pragma unroll
          for (uint32_t i = 0; i < kHalf; ++i) where[i] = slices[a_of[i]].where;
#pragma unroll
          for (uint32_t i = 0; i < kHalf; ++i) {
            const uint32_t u = u0 + i, last = where[i].w & 0xFFFFu;
            const uint32_t q = min(q0 + u * kWave + lane, q_end - 1u);
            const uint32_t bit = __umul24(q, (where[i].w >> 16) & 0xFFu) + where[i].z;
            const uint32_t at = min(bit >> 3, last);
            at_of[u] = ((bit - at * 8u) & 63u) | (a_of[i] << 8) | (where[i].w & 0xFF000000u);
            GlobalBytePtr src = (GlobalBytePtr)(((uint64_t)where[i].y << 32) | where[i].x);
            bits_of[u] = load8(src + at);
            if (WIDE) tail_of[u] = *(src + min(at + 8u, last + 7u));
          }
        };
        auto add_up = [&](auto half) {
          constexpr uint32_t u0 = decltype(half)::value * kHalf;
          uint32_t pos[kHalf];
          double val[kHalf];
#pragma unroll
          for (uint32_t i = 0; i < kHalf; ++i) {
            const uint32_t u = u0 + i;
            const uint4 v = slices[(at_of[u] >> 8) & 0xFFFFu].value;
            const uint32_t sh = at_of[u] & 63u, y = at_of[u] >> 24;
            uint64_t rec = bits_of[u] >> sh;
            if (WIDE && sh) rec |= (uint64_t)tail_of[u] << (64u - sh);
            pos[i] = ((uint32_t)rec & ((1u << s) - 1u)) - lo;  // s <= 31; a position below the tile wraps to a large value
            const uint32_t code = (uint32_t)(rec >> s);
            const uint32_t cid = __builtin_amdgcn_ubfe(code, 0u, y);  // a raw code, y = 32, is taken whole below
            float xhat;
            if (SIGNED) {
              const float mag = __fmaf_rn((float)__builtin_amdgcn_ubfe(code, 0u, y - 1u), __uint_as_float(v.w), __uint_as_float(v.z));
              xhat = __uint_as_float(__float_as_uint(mag) ^ ((cid >> ((y - 1u) & 31u)) << 31));
            } else {
              xhat = __fmaf_rn((float)cid, __uint_as_float(v.w), __uint_as_float(v.z));
            }
            if (y == 32u) xhat = __uint_as_float(code);
            val[i] = __hiloint2double((int)v.y, (int)v.x) * (double)xhat;
          }
#pragma unroll
          for (uint32_t i = 0; i < kHalf; ++i) {
            const bool live = q0 + (u0 + i) * kWave + lane < q_end, inside = pos[i] < room;
            if (live && inside) atomicAdd(&S.acc[pos[i]], val[i]);
            bad |= live && !inside;
          }
        };
        using First = std::integral_constant<uint32_t, 0>;
        using Second = std::integral_constant<uint32_t, 1>;
        const bool both = q_end - q0 > kWave * kHalf;  // uniform
        request(First{});
        if (both) request(Second{});
        if (!open) {  // uniform
          __syncthreads();
          open = true;
        }
        add_up(First{});
        if (both) add_up(Second{});
      }
      wave_lds_fence();  // the slices may be overwritten
    }
    if (last_sweep) {
      if (!open) __syncthreads();  // uniform
      open = false;
      __syncthreads();  // the tile's records are added up
    }
    if (last_sweep) {
      // pairs of coordinates, neighbouring lanes neighbouring pairs (LDS reads without bank conflicts, 512-byte
      // stores per wavefront): all reads first, then the stores.  The thread leaves zeros for the next tile.
      constexpr uint32_t kPairs = kTile / (2u * kDecBlock);
      double2 v[kPairs];
#pragma unroll
      for (uint32_t c = 0; c < kPairs; ++c) {
        double2* mine = reinterpret_cast<double2*>(&S.acc[c * (2u * kDecBlock) + tid * 2u]);
        v[c] = *mine;
        *mine = make_double2(0.0, 0.0);
      }
      const bool aligned = (reinterpret_cast<uintptr_t>(out + lo) & 7u) == 0;  // uniform
#pragma unroll
      for (uint32_t c = 0; c < kPairs; ++c) {
        const uint32_t j0 = lo + c * (2u * kDecBlock) + tid * 2u;
        if (aligned && j0 + 2u <= d) {
          float2* dst = reinterpret_cast<float2*>(out + j0);
          if (accumulate) {
            const float2 o = *dst;
            v[c].x += (double)o.x;
            v[c].y += (double)o.y;
          }
          *dst = make_float2((float)v[c].x, (float)v[c].y);
        } else {
          if (j0 < d) out[j0] = (float)(accumulate ? v[c].x + (double)out[j0] : v[c].x);
          if (j0 + 1u < d) out[j0 + 1u] = (float)(accumulate ? v[c].y + (double)out[j0 + 1u] : v[c].y);
        }
      }
    }
    tile = next_tile;
    l0 = next_l0;
  }
  if (blockIdx.x == 0)  // what the table's workgroups found, where the status word started in their launch
    for (uint32_t i = tid; i < n_found; i += kDecBlock) bad |= found[i] != 0u;
  if (bad) atomicOr(status, CVLC_DEV_STREAM);
}

// ------------------------------------------------------------------ scratch for callers that cannot allocate
// cvlc_decode_aggregate_static works in this array instead of a caller's
// workspace.  Every device the library runs on holds its own copy at its own
// address; host code never uses the array's name as an address, only what
// hipGetSymbolAddress returned for the current device.
static __device__ __align__(256) unsigned char scratch[CVLC_DECODE_STATIC_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {nullptr};

// Address of `scratch` on the current device, looked up once per device.
int static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return CVLC_ERR_DEVICE;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return CVLC_ERR_DEVICE;
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return CVLC_OK;
}

__global__ void copy_status_kernel(const uint32_t* __restrict__ status, uint32_t* __restrict__ dst) { *dst = *status; }

}  // namespace
}  // namespace cvlc

extern "C" {

size_t cvlc_decode_workspace_bytes(uint32_t d, uint32_t n_clients) {
  if (d < 1) return 0;
  return cvlc::decode_layout(d, n_clients < 1 ? 1 : n_clients).total;
}

int cvlc_decode_aggregate(uint32_t n, const void* const* d_streams, const size_t* stream_bytes,
                          const float* weights, float* d_out, uint32_t d, uint32_t flags, void* d_workspace,
                          size_t ws_bytes, void* hip_stream) {
  using namespace cvlc;
  if (!d_out || d < 1 || d > 0x7FFFFFFFu || !d_workspace) return CVLC_ERR_ARG;
  if (n > 65535u) return CVLC_ERR_ARG;  // streams index the grid's y dimension
  if (n > 0 && (!d_streams || !stream_bytes)) return CVLC_ERR_ARG;
  if (reinterpret_cast<uintptr_t>(d_workspace) % 256u || reinterpret_cast<uintptr_t>(d_out) % 4u) return CVLC_ERR_ARG;
  uint64_t items_bound = 0;  // tile_table work items are counted in 32 bits: a record takes two bits at least
  for (uint32_t i = 0; i < n; ++i) {
    if (!d_streams[i] || reinterpret_cast<uintptr_t>(d_streams[i]) % 4u) return CVLC_ERR_ARG;
    if (stream_bytes[i] < 4u * kGlobalHeaderWords) return CVLC_ERR_STREAM;
    items_bound += (uint64_t)stream_bytes[i] * 4u / kTabChunk + kListsPerClient;
  }
  if (items_bound > 0xFFFFFFFFull) return CVLC_ERR_ARG;
  if (ws_bytes < cvlc_decode_workspace_bytes(d, n)) return CVLC_ERR_CAPACITY;
  if (flags & ~(CVLC_DECODE_ACCUMULATE | CVLC_DECODE_QSGD)) return CVLC_ERR_ARG;
  const uint32_t quant = (flags & CVLC_DECODE_QSGD) ? CVLC_QUANT_QSGD : CVLC_QUANT_PQ;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  const DecodeLayout L = decode_layout(d, n < 1 ? 1 : n);
  char* base = static_cast<char*>(d_workspace);
  uint32_t* status = reinterpret_cast<uint32_t*>(base + L.status);
  uint32_t* stream_bad = reinterpret_cast<uint32_t*>(base + L.stream_bad);
  ListDesc* descs = reinterpret_cast<ListDesc*>(base + L.desc);
  CompactDesc* cdesc = reinterpret_cast<CompactDesc*>(base + L.cdesc);
  uint32_t* item_start = reinterpret_cast<uint32_t*>(base + L.item_start);
  DecodeCtl* ctl = reinterpret_cast<DecodeCtl*>(base + L.ctl);
  uint32_t* table = reinterpret_cast<uint32_t*>(base + L.table);
  const uint32_t n_lists = n * kListsPerClient;
  const bool wide = position_bits(d) > 25u;
  const uint32_t shift = tile_shift_for(d), n_tiles = tiles_of(d, shift);

  auto stream_arg = [&](uint32_t i) {
    StreamArg sa;
    sa.words = static_cast<const uint32_t*>(d_streams[i]);
    sa.n_words = stream_bytes[i] / 4u;
    sa.weight = weights ? (double)weights[i] : 0.0;
    sa.has_weight = weights ? 1u : 0u;
    sa.pad = 0;
    return sa;
  };
  // A byte for every workgroup of stream_table: in the place of the list descriptors, or where the table's rows end (a stream has
  // 31 at most, of the larger tiles if there are such) if that is more.
  uint8_t* found = reinterpret_cast<uint8_t*>(descs);
  uint32_t n_found = 0;
  if (n > 0 && n <= kParseStreams) {
    StageScope scope(CVLC_STAGE_DEC_TABLE, stream);
    const size_t rows_end = L.table + (size_t)n * CVLC_MAX_CODED * (n_tiles + 1u) * sizeof(uint32_t);
    size_t room = (size_t)n_lists * sizeof(ListDesc);
    if (L.total - rows_end > room) {
      found = reinterpret_cast<uint8_t*>(base + rows_end);
      room = L.total - rows_end;
    }
    // Workgroups by the streams' lengths, all resident, but no more than a wavefront for every item that a stream can hold (a
    // record has a code bit at least).  us a call with up to 320 workgroups a stream and up to 63 in all more than the device
    // holds, which start when others end, and now: 1 x 11.2 M all kept 57.5 and 42.9, 1 x 25.6 M all kept 111.6 and 78.9, half
    // kept 73.8 and 57.1 (1024 workgroups 59.0), 2 x 11.2 M half kept 50.5 and 45.2; 9 x 11.2 M half kept 132.8 and 126.7, 25 x 1.2 M half
    // kept 62.1 and 58.2, 100 x 11.2 M 121.9 and 115.9.
    uint64_t all = 0;
    for (uint32_t i = 0; i < n; ++i) all += stream_bytes[i];
    const uint64_t most = std::min<uint64_t>(kTableBlocks, room) - n;
    static_assert(kListsPerClient * sizeof(ListDesc) > kParseStreams, "room for a workgroup a stream at least");
    auto launch = [&](auto& in, auto kernel) {
      in.count = n;
      for (uint32_t i = 0; i < n; ++i) {
        const uint64_t items = (uint64_t)stream_bytes[i] * 8u / ((position_bits(d) + 1u) * kTabChunk) + CVLC_MAX_CODED;
        in.args[i] = stream_arg(i);
        in.first[i] = (uint16_t)n_found;
        n_found += (uint32_t)std::min(1u + most * stream_bytes[i] / all, (items + kWavesPerBlock - 1u) / kWavesPerBlock);
      }
      in.blocks = n_found;
      hipLaunchKernelGGL(kernel, dim3(n_found), dim3(kBlock), 0, stream, in, quant, cdesc, ctl, item_start, table, d, shift, n_tiles, found, status);
    };
    static_assert(kTableBlocks < (1u << 16), "the workgroups are numbered in 16 bits");
    if (n <= kFewStreams) {
      StreamArgs<kFewStreams> in;
      launch(in, wide ? stream_table_kernel<true, kFewStreams> : stream_table_kernel<false, kFewStreams>);
    } else {
      StreamArgs<kParseStreams> in;
      launch(in, wide ? stream_table_kernel<true, kParseStreams> : stream_table_kernel<false, kParseStreams>);
    }
  } else {
    profile_mark(CVLC_STAGE_DEC_SETUP, true, stream);
    {
      ParseChunk chunk;
      chunk.pad[0] = chunk.pad[1] = 0;
      for (uint32_t first = 0; first < n; first += kParseStreams) {
        chunk.first = first;
        chunk.count = (n - first < kParseStreams) ? n - first : kParseStreams;
        for (uint32_t i = 0; i < chunk.count; ++i) chunk.args[i] = stream_arg(first + i);
        hipLaunchKernelGGL(parse_headers_kernel, dim3(chunk.count), dim3(64), 0, stream, chunk, descs, d, n, stream_bad, quant);
      }
      // also for n = 0: writes the (empty) list counts and the status word
      hipLaunchKernelGGL(compact_lists_kernel, dim3(1), dim3(1024), 0, stream, descs, n_lists, cdesc, item_start, ctl, stream_bad, n, status);
    }
    profile_mark(CVLC_STAGE_DEC_SETUP, false, stream);
    if (n > 0) {
      StageScope scope(CVLC_STAGE_DEC_TABLE, stream);
      // the number of work items is only known on the device
      auto kernel = wide ? tile_table_kernel<true> : tile_table_kernel<false>;
      hipLaunchKernelGGL(kernel, dim3(kTableBlocks), dim3(kBlock), 0, stream, cdesc, item_start, ctl, table, d, shift, n_tiles,
                         status);
    }
  }
  {
    StageScope scope(CVLC_STAGE_DEC_TILES, stream);
    const bool large = shift == kDecShiftMax;
    const uint32_t g = std::min(n_tiles, large ? 512u : 768u);  // two or three workgroups per CU
    const bool qsgd = quant == CVLC_QUANT_QSGD;
    auto kernel = wide    ? (qsgd ? decode_tiles_kernel<true, true, kDecShiftMax> : decode_tiles_kernel<false, true, kDecShiftMax>)
                  : large ? (qsgd ? decode_tiles_kernel<true, false, kDecShiftMax> : decode_tiles_kernel<false, false, kDecShiftMax>)
                          : (qsgd ? decode_tiles_kernel<true, false, kDecShiftMin> : decode_tiles_kernel<false, false, kDecShiftMin>);
    hipLaunchKernelGGL(kernel, dim3(g), dim3(kDecBlock), 0, stream, cdesc, ctl, item_start, table, d_out, d, n_tiles, position_bits(d),
                       flags & CVLC_DECODE_ACCUMULATE, found, n_found, status);
  }
  return hip_check(hipGetLastError());
}

int cvlc_decode_aggregate_static(uint32_t n, const void* const* d_streams, const size_t* stream_bytes,
                                 const float* weights, float* d_out, uint32_t d, uint32_t flags,
                                 uint32_t* d_status_out, void* hip_stream) {
  using namespace cvlc;
  if (d < 1 || d > 0x7FFFFFFFu || n > 65535u) return CVLC_ERR_ARG;
  if (d_status_out && reinterpret_cast<uintptr_t>(d_status_out) % 4u) return CVLC_ERR_ARG;
  if (cvlc_decode_workspace_bytes(d, n) > (size_t)CVLC_DECODE_STATIC_BYTES) return CVLC_ERR_CAPACITY;
  void* ptr = nullptr;
  int rc = static_scratch(&ptr);
  if (rc) return rc;
  // everything the kernels read from the array they have written earlier in the same call, so what the
  // call before left there does not matter
  rc = cvlc_decode_aggregate(n, d_streams, stream_bytes, weights, d_out, d, flags, ptr, CVLC_DECODE_STATIC_BYTES,
                             hip_stream);
  if (rc) return rc;
  if (d_status_out) {
    hipLaunchKernelGGL(copy_status_kernel, dim3(1), dim3(1), 0, static_cast<hipStream_t>(hip_stream),
                       static_cast<const uint32_t*>(ptr), d_status_out);
    rc = hip_check(hipGetLastError());
  }
  return rc;
}

}  // extern "C"
