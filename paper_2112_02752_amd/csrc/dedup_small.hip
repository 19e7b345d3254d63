// ID dedup of a small batch in one workgroup (gfx950): bags, keys, the stable
// sort and the unique runs in one launch, with the batch in LDS.  The outputs
// are those of the general dedup (dedup.hip), bit for bit.
//
// What bounds it: one compute unit's vector instructions (a ballot per digit
// bit and 64 slots), so it is the faster form only for a few thousand keys.  The
// general passes spread such a batch over a few workgroups that meet through
// memory: a kernel boundary of about 3 us and two or three exchanges of 1.5 to
// 2.5 us a pass, 20 to 37 us for anything up to 60k keys.  A batch pays for the
// slots of its instance (2, 4 or 8 keys a thread).  Measured (us, general -> here;
// ids of a 17-bit and of a 26-bit table):
//    190 keys   20.6 -> 9.1   28.3 -> 9.1
//   1900        23.6 -> 9.2   32.6 -> 10.3
//   3900        25.5 -> 11.5  35.4 -> 14.9
//   4200                15.5          20.0
//   5800        25.6 -> 16.2  35.9 -> 21.2
//   7600        25.7 -> 18.0  35.8 -> 23.8
//   8190                18.5          24.2
// 8 keys a thread take 117 KB of the 160 KB of LDS; larger batches (12 keys, 157
// KB) were not tried.
#include "emb_common.h"
#include "kernels.h"

namespace emb {

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / kWave;

struct SmallArgs {
  const int32_t* offsets;
  const void* idx;
  int32_t idx64, T, B, M, N;
  uint32_t b_magic;  // bag_magic(B)
  int32_t passes, shift[kMaxPasses], bits[kMaxPasses];
  uint32_t* unique_keys;
  int32_t* counts;
  int32_t* seg;
  int32_t* perm;
  int32_t* num_unique;
  int32_t* sorted_bag;
  int32_t* chunk_seg;
  WsHeader* hdr;
  TableOffsets ro;
};

// Positions of a wavefront: w * 64 IT + i * 64 + lane, i < IT.
template <int IT>
__global__ __launch_bounds__(kThreads) void k_dedup_small(SmallArgs a) {
  constexpr int CAP = kThreads * IT;
  __shared__ uint32_t s_keys[CAP];
  __shared__ uint16_t s_pos[CAP];
  __shared__ int32_t s_bag[CAP];
  __shared__ uint16_t s_cnt[kWaves][kMaxDigits];  // later the heads' positions
  __shared__ uint32_t s_start[kMaxDigits];
  __shared__ uint32_t s_w[kWaves];
  __shared__ uint32_t s_toff[EMB_MAX_TABLES];
  static_assert(kWaves * kMaxDigits >= CAP, "the heads' positions fit the counters");
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wbase = w * (kWave * IT);

  // the ids' loads overlap the bag search
  uint32_t key[IT];
  int32_t pos[IT];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    pos[i] = wbase + i * kWave + lane;
    key[i] = pos[i] < a.N ? (uint32_t)load_id(a.idx, a.idx64, pos[i]) : 0u;
  }
  // bag of each position: every bag that holds ids writes its number plus one
  // at its first position, a running maximum carries it to the others
  for (int i = tid; i < CAP; i += kThreads) s_bag[i] = 0;
  for (int t = tid; t < a.T; t += kThreads) s_toff[t] = a.ro.off[t];
  __syncthreads();
  for (int m = tid; m < a.M; m += kThreads) {
    const int32_t st = a.offsets[m], en = a.offsets[m + 1];
    if (st < en && st >= 0 && st < a.N) s_bag[st] = m + 1;
  }
  __syncthreads();
  uint32_t carry = 0;
  uint32_t bag[IT];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const uint32_t m = wave_incl_max((uint32_t)s_bag[wbase + i * kWave + lane]);
    bag[i] = m > carry ? m : carry;
    const uint32_t last = (uint32_t)__builtin_amdgcn_readlane((int)m, kWave - 1);
    carry = last > carry ? last : carry;
  }
  if (lane == 0) s_w[w] = carry;
  __syncthreads();
  const uint32_t upto = wave_incl_max(lane < kWaves ? s_w[lane] : 0u);
  const uint32_t before = w > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)upto, w - 1) : 0u;
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const uint32_t m = (bag[i] > before ? bag[i] : before) - 1u;
    if (pos[i] < a.N) {
      s_bag[pos[i]] = (int32_t)m;
      if (a.T > 1) {
        const uint32_t t = table_of_bag(m, a.B, a.b_magic);
        key[i] += s_toff[t < (uint32_t)a.T ? t : 0u];
      }
    }
  }

  // stable radix passes
#pragma unroll 1
  for (int ps = 0; ps < a.passes; ++ps) {
    const int shift = a.shift[ps], bits = a.bits[ps], nd = 1 << bits;
    const uint32_t mask = (uint32_t)nd - 1u;
    for (int i = lane; i < nd / 2; i += kWave) reinterpret_cast<lds_word*>(s_cnt[w])[i] = 0u;
    wave_lds_order();
    uint32_t rank[IT];
    // rank of each key among its wavefront's earlier keys of its digit
    uint32_t lo[IT], hi[IT];
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const uint64_t all = __ballot(pos[i] < a.N);
      lo[i] = (uint32_t)all;
      hi[i] = (uint32_t)(all >> 32);
    }
#pragma unroll 1
    for (int b = 0; b < bits; ++b)
#pragma unroll
      for (int i = 0; i < IT; ++i) keep_peers(key[i] >> shift, b, lo[i], hi[i]);
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const uint32_t d = (key[i] >> shift) & mask;
      const bool valid = pos[i] < a.N;
      const uint64_t peers = ((uint64_t)hi[i] << 32) | lo[i];
      rank[i] = 0;
      if (valid) {
        const uint32_t r = lanes_below(peers);
        const uint32_t c = s_cnt[w][d];
        rank[i] = c + r;
        if (r == 0) s_cnt[w][d] = (uint16_t)(c + (uint32_t)__popcll(peers));
      }
      wave_lds_order();
    }
    __syncthreads();
    // per digit the wavefronts' offsets, then the digits' starts
    uint32_t total = 0;
    if (tid < nd) {
#pragma unroll
      for (int i = 0; i < kWaves; ++i) {
        const uint32_t c = s_cnt[i][tid];
        s_cnt[i][tid] = (uint16_t)total;
        total += c;
      }
    }
    const uint32_t incl = wave_incl_sum(total);
    if (lane == kWave - 1) s_w[w] = incl;
    __syncthreads();
    const uint32_t sums = wave_incl_sum(lane < kWaves ? s_w[lane] : 0u);
    if (tid < nd) s_start[tid] = incl - total + (w > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)sums, w - 1) : 0u);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < IT; ++i)
      if (wbase + i * kWave + lane < a.N) {
        const uint32_t d = (key[i] >> shift) & mask;
        const uint32_t dst = s_start[d] + s_cnt[w][d] + rank[i];
        s_keys[dst] = key[i];
        s_pos[dst] = (uint16_t)pos[i];
      }
    __syncthreads();
    // (slots past the last key keep a position past the last)
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int p = wbase + i * kWave + lane;
      if (p < a.N) {
        key[i] = s_keys[p];
        pos[i] = s_pos[p];
      }
    }
  }

  // the runs of equal keys
  uint32_t heads = 0, nheads = 0, rank[IT];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int p = wbase + i * kWave + lane;
    const bool head = p < a.N && (p == 0 || s_keys[p - 1] != key[i]);
    const uint64_t hb = __ballot(head);
    rank[i] = nheads + lanes_below(hb);
    heads |= head ? 1u << i : 0u;
    nheads += (uint32_t)__popcll(hb);
    if (p < a.N) {
      a.perm[p] = pos[i];
      a.sorted_bag[p] = s_bag[pos[i]];
    }
  }
  __syncthreads();  // (the last use of s_cnt as counters and of s_w is past)
  if (lane == 0) s_w[w] = nheads;
  __syncthreads();
  uint16_t* s_head = &s_cnt[0][0];
  const uint32_t sums = wave_incl_sum(lane < kWaves ? s_w[lane] : 0u);
  const uint32_t u0 = w > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)sums, w - 1) : 0u;
  const uint32_t U = (uint32_t)__builtin_amdgcn_readlane((int)sums, kWaves - 1);
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int p = wbase + i * kWave + lane;
    const uint32_t u = u0 + rank[i];
    const bool head = (heads >> i) & 1u;
    if (head) {
      a.unique_keys[u] = key[i];
      a.seg[u] = p;
      s_head[u] = (uint16_t)p;
    }
    // segment of every chunk's first position (lane 0: positions are taken 64 at a time)
    static_assert(kChunk == kWave, "a wavefront's 64 positions are a chunk");
    if (lane == 0 && p < a.N) a.chunk_seg[p / kChunk] = (int32_t)(u + (head ? 1u : 0u)) - 1;
  }
  __syncthreads();
  for (uint32_t u = tid; u < U; u += kThreads)
    a.counts[u] = (u + 1u < U ? (int32_t)s_head[u + 1u] : a.N) - (int32_t)s_head[u];
  if (tid == 0) {
    a.num_unique[0] = (int32_t)U;
    a.seg[U] = a.N;
    a.chunk_seg[(a.N + kChunk - 1) / kChunk] = (int32_t)U;
    // the call's generation (no wait of this call can fail)
    const uint32_t g = next_gen(a.hdr->gen);
    a.hdr->cur = g;
    a.hdr->gen = g;
  }
}

template <int IT>
hipError_t launch_t(const SmallArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_dedup_small<IT>, dim3(1), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}

}  // namespace

bool dedup_is_small(int64_t N, int64_t M) { return N <= kSmallKeys && M <= kSmallBags; }

hipError_t launch_dedup_small(const DedupLaunch& p, hipStream_t s) {
  char* ws = static_cast<char*>(p.ws);
  SmallArgs a{};
  a.offsets = p.offsets;
  a.idx = p.idx;
  a.idx64 = p.idx64;
  a.T = p.T;
  a.B = p.B;
  a.M = p.M;
  a.N = (int32_t)p.N;
  a.b_magic = bag_magic(p.B);
  a.passes = p.plan.passes;
  for (int i = 0; i < kMaxPasses; ++i) {
    a.shift[i] = p.plan.shift[i];
    a.bits[i] = p.plan.bits[i];
  }
  a.unique_keys = p.unique_keys;
  a.counts = p.counts;
  a.seg = p.seg_offsets;
  a.perm = p.sort_perm;
  a.num_unique = p.num_unique;
  a.sorted_bag = reinterpret_cast<int32_t*>(ws + p.lay.sorted_bag);
  a.chunk_seg = reinterpret_cast<int32_t*>(ws + p.lay.chunk_seg);
  a.hdr = reinterpret_cast<WsHeader*>(ws + p.lay.hdr);
  a.ro = p.ro;
  if (p.N <= 2 * kThreads) return launch_t<2>(a, s);
  if (p.N <= 4 * kThreads) return launch_t<4>(a, s);
  return launch_t<8>(a, s);
}

}  // namespace emb
