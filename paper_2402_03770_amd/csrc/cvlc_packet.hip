// cvlc_packet.hip -- packets (Sec. IV-C Eq. (3), Sec. IV-D): a client's stream
// is cut into packets of at most mtu bytes, each holding records of one group
// only and a header that lets the parameter server place and decode it on its
// own; the server puts the stream back together from the packets it received.
//
// Packet = little-endian 32-bit words:
//   0 "CVLP"   1 version | quantiser << 16   2 d   3 client   4 bits(B)
//   5 r | R << 8 | y_r << 16 | s << 24        6 P_r
//   7 e0, the number of the packet's first record inside its group
//   8, 9 the group's two centroid words ({min, max} or {norm, 0})
//   then c = min(cap_r, P_r - e0) records of W_r = s + y_r bits from bit 0,
//   zero padded to a word.  cap_r = floor((8 mtu - 320) / W_r) is the largest
//   record count that satisfies Eq. (3) with H = 320 bits.
// Packets are numbered group by group; an empty group sends one packet with no
// records so that its header fields survive.  In memory packets sit at a stride
// of mtu bytes.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "cvlc_common.h"

namespace cvlc {
namespace {

constexpr uint32_t kPktMagic = 0x504C5643u;  // "CVLP"
constexpr uint32_t kPktHeaderWords = CVLC_PACKET_HEADER_WORDS;
// The kernels that move records have a workgroup per packet, of THREADS threads that ask for DEEP words each together.  How many:
//   up to 128 words a packet    a wavefront, two words a lane: 25.6 M coordinates all kept, 241 757 packets of 512 bytes, packetize 65 us
//                               (four wavefronts 196), 5.1 M of 64 bytes 1203 us (4133); depacketize 1527 (1540) and 19 911 (21 515)
//   up to 384 words, where four wavefronts a packet are more than the device holds
//                               a wavefront, six words a lane: 8486 packets of 1500 bytes 7.3 us (10.5), 77 951 39 (72)
//   else                        four wavefronts, two words a lane: 973 packets of 1500 bytes are one wavefront for every SIMD, and one that
//                               goes through them by itself takes 7.1 us for 4.0; 3040 packets of 9000 bytes 13 us (six words a lane of one
//                               wavefront 13, two 17), 206 of 65 532 19 (38, 56)
// A grid has less than 2^32 threads (one of more is cut off without an error): more than 2^23 packets take several launches.
template <typename Launch>
void by_packet_shape(uint32_t n, uint32_t words, Launch launch) {
  using One = std::integral_constant<uint32_t, 64>;
  constexpr uint32_t kMost = 1u << 23;
  for (uint32_t first = 0, count; first < n; first += count) {
    count = n - first < kMost ? n - first : kMost;
    if (words <= 128u) launch(first, count, One(), std::integral_constant<uint32_t, 2>());
    else if (words <= 384u && n > 2048u) launch(first, count, One(), std::integral_constant<uint32_t, 6>());
    else launch(first, count, std::integral_constant<uint32_t, 256>(), std::integral_constant<uint32_t, 2>());
  }
}

typedef const uint32_t __attribute__((address_space(1))) * GlobalConstWordPtr;
typedef uint32_t __attribute__((address_space(1))) * GlobalWordPtr;

__host__ __device__ __forceinline__ bool mtu_supported(uint32_t mtu) {
  return mtu % 4u == 0 && mtu >= 64u && mtu <= 65532u;
}
__host__ __device__ __forceinline__ uint32_t packet_cap(uint32_t mtu, uint32_t W) {
  return (8u * mtu - 32u * kPktHeaderWords) / W;  // W <= 63 and mtu >= 64: at least 3
}
__host__ __device__ __forceinline__ uint32_t group_packets(uint32_t P, uint32_t cap) {
  return P == 0 ? 1u : (P + cap - 1u) / cap;
}

// ------------------------------------------------------------------ sender
struct PacketPlan {  // what the sender's kernel needs from the plan
  uint32_t R, s, mtu_words;
  uint32_t y[CVLC_MAX_CODED], P[CVLC_MAX_CODED];
  uint32_t first[CVLC_MAX_CODED], payload[CVLC_MAX_CODED];  // every group's first packet and first stream word
};

// One workgroup per packet: finds its (group, number inside the group) from the
// plan, copies the header fields from the stream's headers and moves its records
// down to bit 0 of the packet's payload; the rest of the packet's slot is zeroed.
// All latency: a lane per group finds the packet's (every lane in a loop over the groups, with two divisions each), and all loads
// are out before the first is waited for (the header's six one after the other, the words 64 at a time): 973 packets 7.1 -> 4.0 us.
template <uint32_t THREADS, uint32_t DEEP>
__global__ __launch_bounds__(THREADS) void packetize_kernel(PacketPlan plan, uint32_t first_packet, const uint32_t* __restrict__ stream,
                                                            uint32_t* __restrict__ packets) {
  const uint32_t mtu = plan.mtu_words * 4u, packet = first_packet + blockIdx.x;
  const uint32_t lane = lane_id(), tid = threadIdx.x;
  if (plan.R == 0) return;  // the grid has exactly one workgroup per packet; never taken
  const uint64_t from = __ballot(lane < plan.R && plan.first[min(lane, CVLC_MAX_CODED - 1u)] <= packet);  // a group has a packet at least: a prefix
  const uint32_t r = (uint32_t)__popcll(from) - 1u;
  const uint32_t P = plan.P[r], y = plan.y[r], W = plan.s + y, cap = packet_cap(mtu, W), e0 = (packet - plan.first[r]) * cap;
  const uint32_t c = P - e0 < cap ? P - e0 : cap;
  GlobalWordPtr out = (GlobalWordPtr)(packets + (size_t)packet * plan.mtu_words);
  // word `tid` of the header, where the stream has it
  const uint32_t at = tid == 1u || tid == 2u ? tid : tid == 3u ? 6u : tid == 4u ? 5u : kGlobalHeaderWords + kSegHeaderWords * r + (tid == 8u ? 2u : 3u);
  uint32_t field = ((GlobalConstWordPtr)stream)[at];
  // the packet's records are bits [e0 W, (e0 + c) W) of the group's payload
  const uint64_t bit0 = (uint64_t)e0 * W;
  const uint32_t group_words = (uint32_t)payload_words(P, W);
  const uint32_t w0 = (uint32_t)(bit0 >> 5), sh = (uint32_t)(bit0 & 31u);
  const uint32_t nbits = c * W, n_out = (nbits + 31u) >> 5, n_words = plan.mtu_words - kPktHeaderWords;
  GlobalConstWordPtr src = (GlobalConstWordPtr)(stream + plan.payload[r]);
  for (uint32_t base = 0; base < n_words; base += DEEP * THREADS) {
    uint32_t a[DEEP], b[DEEP];
    if (n_out) {  // uniform; an empty group has no words
#pragma unroll
      for (uint32_t u = 0; u < DEEP; ++u) {
        const uint32_t w = w0 + base + u * THREADS + tid;
        a[u] = src[min(w, group_words - 1u)];
        b[u] = src[min(w + 1u, group_words - 1u)];
      }
    }
#pragma unroll
    for (uint32_t u = 0; u < DEEP; ++u) {
      const uint32_t i = base + u * THREADS + tid;
      uint32_t v = 0;
      if (i < n_out) {
        v = sh ? (a[u] >> sh) | ((w0 + i + 1u < group_words ? b[u] : 0u) << (32u - sh)) : a[u];
        if (i == n_out - 1u && (nbits & 31u)) v &= (1u << (nbits & 31u)) - 1u;
      }
      if (i < n_words) out[kPktHeaderWords + i] = v;
    }
  }
  if (tid < kPktHeaderWords) {
    if (tid == 0u) field = kPktMagic;
    if (tid == 5u) field = r | (plan.R << 8) | (y << 16) | (plan.s << 24);
    if (tid == 6u) field = P;
    if (tid == 7u) field = e0;
    out[tid] = field;
  }
}

// ------------------------------------------------------------------ receiver
struct ReassemblyState {  // at the start of the workspace, after the status word's 256 bytes
  uint32_t valid;         // 1: the second kernel may copy
  uint32_t payload[32];   // every group's first stream word
};

constexpr uint32_t kGatherBlock = 1024;
constexpr uint32_t kSeenBits = 1u << 18;  // packets whose places are ticked off in LDS (more: in memory)

struct PktHeader {
  uint32_t w[kPktHeaderWords];
};
// All words of a header in one round trip, before any of them is looked at.
__device__ __forceinline__ PktHeader load_header(const uint32_t* __restrict__ packets, size_t p, uint32_t mtu_words) {
  PktHeader h;
#pragma unroll
  for (uint32_t i = 0; i < kPktHeaderWords; ++i) h.w[i] = packets[p * mtu_words + i];
  return h;
}

// Inclusive prefix sum over the 32 lanes of the first half of a wavefront.
__device__ __forceinline__ uint64_t half_incl_scan_u64(uint64_t v) {
#pragma unroll
  for (int o = 1; o < 32; o <<= 1) {
    const uint64_t t = (uint64_t)__shfl_up((unsigned long long)v, o, 64);
    if (lane_id() >= (uint32_t)o) v += t;
  }
  return v;
}

// One workgroup: reads every packet's header, takes each group's fields from
// the packet that holds its record 0, lays the stream out, writes its headers,
// checks every packet against that and that every place is taken exactly once,
// and clears the stream words that two packets share.
// All latency, so the round trips are what was cut: a thread keeps the header of its first packet between the two
// passes, a lane per group lays the stream out, and the places are ticked off in LDS (headers read field by field, the
// groups laid out one after the other by one thread, places in memory: 17.5 us for 973 packets, now 6.8).
__global__ __launch_bounds__(kGatherBlock) void reassemble_headers_kernel(const uint32_t* __restrict__ packets,
                                                                         uint32_t n, uint32_t mtu_words, uint32_t d,
                                                                         uint32_t* __restrict__ stream,
                                                                         uint64_t cap_words, uint32_t* status,
                                                                         ReassemblyState* st,
                                                                         uint32_t* __restrict__ seen) {
  __shared__ uint32_t g_y[32], g_P[32], g_c0[32], g_c1[32], g_have[32], g_payload[33], g_first[33];
  __shared__ uint32_t s_seen[kSeenBits / 32u];
  __shared__ uint32_t s_bad;
  const uint32_t tid = threadIdx.x, mtu = mtu_words * 4u;
  const PktHeader lead = load_header(packets, 0, mtu_words), mine = load_header(packets, min(tid, n - 1u), mtu_words);
  const bool seen_in_lds = n <= kSeenBits;
  if (tid < 32) g_have[tid] = 0;
  if (tid == 0) s_bad = 0;
  if (seen_in_lds) {
    for (uint32_t i = tid; i < (n + 31u) / 32u; i += kGatherBlock) s_seen[i] = 0;
  } else {
    for (uint32_t i = tid; i < n; i += kGatherBlock) seen[i] = 0;
  }
  const uint32_t f1 = lead.w[1], f3 = lead.w[3], f4 = lead.w[4], f5 = lead.w[5];
  const uint32_t R = (f5 >> 8) & 0xFFu, s = f5 >> 24;
  const float B = __uint_as_float(f4);
  const bool global_ok = lead.w[0] == kPktMagic && (f1 & 0xFFFFu) == kVersion && (f1 >> 16) <= CVLC_QUANT_QSGD &&
                         lead.w[2] == d && R <= CVLC_MAX_CODED && s == position_bits(d) && B > 0.0f &&
                         fabsf(B) <= 3.4028234664e38f;
  __syncthreads();
  if (global_ok) {
    for (uint32_t p = tid; p < n; p += kGatherBlock) {
      const PktHeader h = p == tid ? mine : load_header(packets, p, mtu_words);
      const uint32_t r = h.w[5] & 0xFFu;
      if (h.w[0] != kPktMagic || r >= R) {
        atomicOr(&s_bad, 1u);
      } else if (h.w[7] == 0) {  // holds the group's record 0: exactly one such packet per group
        if (atomicAdd(&g_have[r], 1u) == 0) {
          g_y[r] = (h.w[5] >> 16) & 0xFFu;
          g_P[r] = h.w[6];
          g_c0[r] = h.w[8];
          g_c1[r] = h.w[9];
        } else {
          atomicOr(&s_bad, 1u);
        }
      }
    }
  }
  __syncthreads();
  if (tid < kWave) {  // one wavefront, lane r = group r
    const bool group = tid < R && tid < 32u;
    bool ok = global_ok && !s_bad && (!group || (g_have[tid] == 1 && code_len_supported(g_y[tid]) && g_P[tid] <= d));
    ok = __ballot(ok) == ~0ull;
    uint64_t packets_here = 0, words_here = 0;
    if (ok && group) {
      const uint32_t W = s + g_y[tid];
      packets_here = group_packets(g_P[tid], packet_cap(mtu, W));
      words_here = payload_words(g_P[tid], W);
    }
    const uint64_t first_incl = half_incl_scan_u64(packets_here);
    const uint64_t payload_incl = kGlobalHeaderWords + (uint64_t)kSegHeaderWords * R + half_incl_scan_u64(words_here);
    // R <= 31: lane 31 holds the sums over all groups
    const uint64_t n_all = (uint64_t)__shfl((unsigned long long)first_incl, 31, 64);
    const uint64_t words_all = (uint64_t)__shfl((unsigned long long)payload_incl, 31, 64);
    ok = ok && n_all == n && words_all <= 0xFFFFFFFFull && words_all <= cap_words;
    if (ok) {
      if (tid < 32u) {
        g_first[tid] = (uint32_t)(first_incl - packets_here);
        g_payload[tid] = (uint32_t)(payload_incl - words_here);
      }
      if (tid == 0) {
        stream[0] = kMagic; stream[1] = f1; stream[2] = d; stream[3] = R; stream[4] = s; stream[5] = f4; stream[6] = f3;
        stream[7] = (uint32_t)words_all;
      }
      if (group) {
        uint32_t* gh = stream + kGlobalHeaderWords + kSegHeaderWords * tid;
        gh[0] = g_y[tid]; gh[1] = g_P[tid]; gh[2] = g_c0[tid]; gh[3] = g_c1[tid];
      }
    } else if (tid == 0) {
      s_bad = 1;
    }
  }
  __syncthreads();
  if (!s_bad) {
    for (uint32_t p = tid; p < n; p += kGatherBlock) {
      const PktHeader h = p == tid ? mine : load_header(packets, p, mtu_words);
      const uint32_t r = h.w[5] & 0xFFu;  // < R, checked above
      const uint32_t W = s + g_y[r], cap = packet_cap(mtu, W), P = g_P[r], e0 = h.w[7], place = e0 / cap;
      bool ok = h.w[1] == f1 && h.w[2] == d && h.w[3] == f3 && h.w[4] == f4 &&
                h.w[5] == (r | (R << 8) | (g_y[r] << 16) | (s << 24)) && h.w[6] == P && h.w[8] == g_c0[r] &&
                h.w[9] == g_c1[r] && e0 == place * cap && (e0 < P || (e0 == 0 && P == 0));
      if (ok) {  // n places, n packets, none twice: none missing
        const uint32_t at = g_first[r] + place;
        ok = seen_in_lds ? ((atomicOr(&s_seen[at >> 5], 1u << (at & 31u)) >> (at & 31u)) & 1u) == 0 : atomicAdd(&seen[at], 1u) == 0;
      }
      if (!ok) {
        atomicOr(&s_bad, 1u);
        continue;
      }
      const uint32_t c = P - e0 < cap ? P - e0 : cap;
      if (c) {  // the first and the last stream word of the packet's records may be shared with its neighbours
        const uint64_t bit0 = (uint64_t)e0 * W, bit1 = bit0 + (uint64_t)c * W;
        stream[g_payload[r] + (uint32_t)(bit0 >> 5)] = 0;
        stream[g_payload[r] + (uint32_t)((bit1 - 1) >> 5)] = 0;
      }
    }
  }
  __syncthreads();
  if (tid < 32) st->payload[tid] = tid < R ? g_payload[tid] : 0;
  if (tid == 0) {
    st->valid = s_bad ? 0u : 1u;
    *status = s_bad ? CVLC_DEV_STREAM : 0u;
    if (s_bad) stream[0] = 0;  // what is there is not a stream
  }
}

// One workgroup per packet: its records move up to their place in the group's
// payload.  Words wholly inside the packet's bit range are stored, the first
// and the last are OR-ed into the words the header kernel cleared.
// The packet's own header says all but where the group's payload begins (the header kernel has found them alike), so that
// the packet's words are asked for with it: 973 packets 5.3 -> 4.9 us.  A wavefront that has the packet to itself takes the word
// before a lane's from the lane below (314 328 packets of 128 bytes 152 us, loaded 158; 77 951 of 1500 93 and 99).
template <uint32_t THREADS, uint32_t DEEP>
__global__ __launch_bounds__(THREADS) void reassemble_payload_kernel(const uint32_t* __restrict__ packets, uint32_t first_packet,
                                                                       uint32_t mtu_words,
                                                                       const ReassemblyState* __restrict__ st,
                                                                       uint32_t* __restrict__ stream) {
  GlobalConstWordPtr pk = (GlobalConstWordPtr)(packets + (size_t)(first_packet + blockIdx.x) * mtu_words), src = pk + kPktHeaderWords;
  const uint32_t n_src = mtu_words - kPktHeaderWords, tid = threadIdx.x;
  uint32_t hi[DEEP], lo[DEEP];
  auto ask = [&](uint32_t base) {
#pragma unroll
    for (uint32_t u = 0; u < DEEP; ++u) {
      const uint32_t i = base + u * THREADS + tid;
      hi[u] = src[min(i, n_src - 1u)];
      if constexpr (THREADS != kWave) lo[u] = src[min(max(i, 1u) - 1u, n_src - 1u)];
    }
  };
  ask(0);
  const uint32_t h5 = pk[5], P = pk[6], e0 = pk[7], r = h5 & 31u;
  const uint32_t valid = st->valid, payload = st->payload[r];
  if (!valid) return;
  const uint32_t W = (h5 >> 24) + ((h5 >> 16) & 0xFFu), cap = packet_cap(mtu_words * 4u, W);
  const uint32_t c = P - e0 < cap ? P - e0 : cap;
  if (c == 0) return;
  const uint64_t bit0 = (uint64_t)e0 * W;
  const uint32_t nbits = c * W, sh = (uint32_t)(bit0 & 31u), full = nbits >> 5, part = (1u << (nbits & 31u)) - 1u;
  const uint32_t w0 = (uint32_t)(bit0 >> 5), last = (uint32_t)((bit0 + nbits - 1u) >> 5) - w0;
  GlobalWordPtr dst = (GlobalWordPtr)(stream + payload + w0);
  // word k of the packet's records, the bits beyond the last one cleared
  auto word = [&](uint32_t k, uint32_t v) { return k < full ? v : (k == full ? v & part : 0u); };
  uint32_t carry = 0;  // of a single wavefront: the last lane's word of the turn before
  for (uint32_t base = 0; base <= last; base += DEEP * THREADS) {
    if (base) ask(base);
    if constexpr (THREADS == kWave) {
#pragma unroll
      for (uint32_t u = 0; u < DEEP; ++u) {
        lo[u] = (uint32_t)__builtin_amdgcn_update_dpp((int)carry, (int)hi[u], 0x138 /* wave_shr:1 */, 0xF, 0xF, false);
        carry = __builtin_amdgcn_readlane(hi[u], kWave - 1);
      }
    }
#pragma unroll
    for (uint32_t u = 0; u < DEEP; ++u) {
      const uint32_t i = base + u * THREADS + tid;
      if (i > last) continue;
      const uint32_t below = i ? word(i - 1u, lo[u]) : 0u;
      const uint32_t v = sh ? (word(i, hi[u]) << sh) | (below >> (32u - sh)) : word(i, hi[u]);
      if (i == 0 || i == last) {
        if (v) atomicOr((uint32_t*)(dst + i), v);
      } else {
        dst[i] = v;
      }
    }
  }
}

size_t align256(size_t v) { return (v + 255u) & ~(size_t)255u; }

bool plan_packets(const cvlc_plan_t* plan, uint32_t mtu, uint64_t* count) {
  if (!plan || cvlc_plan_validate(plan) != CVLC_OK || !mtu_supported(mtu)) return false;
  uint64_t n = 0;
  for (uint32_t r = 0; r < plan->n_coded; ++r)
    n += group_packets(plan->count[r], packet_cap(mtu, plan->s + plan->code_len[r]));
  *count = n;
  return n <= 0xFFFFFFFFull;
}

}  // namespace
}  // namespace cvlc

extern "C" {

uint32_t cvlc_packet_count(const cvlc_plan_t* plan, uint32_t mtu_bytes) {
  uint64_t n = 0;
  return cvlc::plan_packets(plan, mtu_bytes, &n) ? (uint32_t)n : 0u;
}

uint32_t cvlc_packet_size(const cvlc_plan_t* plan, uint32_t mtu_bytes, uint32_t index) {
  using namespace cvlc;
  uint64_t n = 0;
  if (!plan_packets(plan, mtu_bytes, &n) || index >= n) return 0;
  uint32_t first = 0;
  for (uint32_t r = 0; r < plan->n_coded; ++r) {
    const uint32_t W = plan->s + plan->code_len[r], cap = packet_cap(mtu_bytes, W);
    const uint32_t npk = group_packets(plan->count[r], cap);
    if (index < first + npk) {
      const uint32_t e0 = (index - first) * cap;
      const uint32_t c = plan->count[r] - e0 < cap ? plan->count[r] - e0 : cap;
      return 4u * (kPktHeaderWords + (uint32_t)payload_words(c, W));
    }
    first += npk;
  }
  return 0;
}

int cvlc_packetize(const cvlc_plan_t* plan, const void* d_stream, uint32_t mtu_bytes, void* d_packets_out,
                   size_t capacity, void* hip_stream) {
  using namespace cvlc;
  if (!plan || !d_stream || !d_packets_out) return CVLC_ERR_ARG;
  if (reinterpret_cast<uintptr_t>(d_stream) % 4u || reinterpret_cast<uintptr_t>(d_packets_out) % 4u) return CVLC_ERR_ARG;
  if (!mtu_supported(mtu_bytes)) return CVLC_ERR_ARG;
  const int rc = cvlc_plan_validate(plan);
  if (rc) return rc;
  if (plan->total_bits / 32u > 0xFFFFFFFFull) return CVLC_ERR_PLAN;
  uint64_t n = 0;
  if (!plan_packets(plan, mtu_bytes, &n)) return CVLC_ERR_PLAN;
  if (capacity < n * (uint64_t)mtu_bytes) return CVLC_ERR_CAPACITY;
  if (n == 0) return CVLC_OK;  // no coded group: nothing to send
  PacketPlan pp;
  pp.R = plan->n_coded;
  pp.s = plan->s;
  pp.mtu_words = mtu_bytes / 4u;
  uint32_t first = 0, payload = kGlobalHeaderWords + kSegHeaderWords * plan->n_coded;
  for (uint32_t r = 0; r < CVLC_MAX_CODED; ++r) {
    const bool coded = r < plan->n_coded;
    pp.y[r] = coded ? plan->code_len[r] : 0;
    pp.P[r] = coded ? plan->count[r] : 0;
    pp.first[r] = first;
    pp.payload[r] = payload;
    if (coded) {
      first += group_packets(pp.P[r], packet_cap(mtu_bytes, pp.s + pp.y[r]));
      payload += (uint32_t)payload_words(pp.P[r], pp.s + pp.y[r]);
    }
  }
  by_packet_shape((uint32_t)n, pp.mtu_words - kPktHeaderWords, [&](uint32_t from, uint32_t count, auto threads, auto deep) {
    hipLaunchKernelGGL((packetize_kernel<threads.value, deep.value>), dim3(count), dim3(threads.value), 0,
                       static_cast<hipStream_t>(hip_stream), pp, from, static_cast<const uint32_t*>(d_stream), static_cast<uint32_t*>(d_packets_out));
  });
  return hip_check(hipGetLastError());
}

size_t cvlc_depacketize_workspace_bytes(uint32_t n_packets) {
  return 256u + cvlc::align256(sizeof(cvlc::ReassemblyState)) + cvlc::align256((size_t)n_packets * sizeof(uint32_t));
}

int cvlc_depacketize(const void* d_packets, uint32_t n_packets, uint32_t mtu_bytes, uint32_t d, void* d_stream_out,
                     size_t capacity, void* d_workspace, size_t ws_bytes, void* hip_stream) {
  using namespace cvlc;
  if (!d_packets || !d_stream_out || !d_workspace || n_packets == 0) return CVLC_ERR_ARG;
  if (d < 1 || d > 0x7FFFFFFFu || !mtu_supported(mtu_bytes)) return CVLC_ERR_ARG;
  if (reinterpret_cast<uintptr_t>(d_packets) % 4u || reinterpret_cast<uintptr_t>(d_stream_out) % 4u ||
      reinterpret_cast<uintptr_t>(d_workspace) % 256u)
    return CVLC_ERR_ARG;
  if (capacity < 4u * kGlobalHeaderWords) return CVLC_ERR_CAPACITY;
  if (ws_bytes < cvlc_depacketize_workspace_bytes(n_packets)) return CVLC_ERR_CAPACITY;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  char* base = static_cast<char*>(d_workspace);
  uint32_t* status = reinterpret_cast<uint32_t*>(base);
  ReassemblyState* st = reinterpret_cast<ReassemblyState*>(base + 256);
  uint32_t* seen = reinterpret_cast<uint32_t*>(base + 256 + align256(sizeof(ReassemblyState)));
  hipLaunchKernelGGL(reassemble_headers_kernel, dim3(1), dim3(kGatherBlock), 0, stream,
                     static_cast<const uint32_t*>(d_packets), n_packets, mtu_bytes / 4u, d,
                     static_cast<uint32_t*>(d_stream_out), (uint64_t)(capacity / 4u), status, st, seen);
  by_packet_shape(n_packets, mtu_bytes / 4u - kPktHeaderWords, [&](uint32_t from, uint32_t count, auto threads, auto deep) {
    hipLaunchKernelGGL((reassemble_payload_kernel<threads.value, deep.value>), dim3(count), dim3(threads.value), 0, stream,
                       static_cast<const uint32_t*>(d_packets), from, mtu_bytes / 4u, st, static_cast<uint32_t*>(d_stream_out));
  });
  return hip_check(hipGetLastError());
}

}  // extern "C"
