// Pooled embedding lookup, forward (gfx950).
//
//   out[m][d] = scale_m * sum_{j in bag m} W[row_offset[t(m)] + idx[j]][d]
//
// A row of D*sizeof(T) bytes is read as 16-byte vectors by a group of G lanes
// (G a power of two), so one wave instruction gathers R = 64/G rows.  A
// wavefront sums one bag: its ids are read 64 at a time, lane g*G + u taking
// id u*R + g, so that the ids of lane group g already sit in that group's own
// lanes and reach all of them by a lane broadcast within the group (DPP for
// groups of up to 16 lanes), with no trip through LDS.  Up to 8 rows per lane
// group are in flight; the groups are summed across the wavefront at the end
// (gfx950 row and half swaps).  Repeated ids of a bag are loaded again as a rule:
// a hot row is a cache hit, and finding the repeats costs more instructions than
// their loads.  Wide rows are the exception (merges_repeats): their repeats fill
// the vector cache's 64 bytes a cycle.
//
// The rows of a round are added pairwise, as many additions as one after
// another; rounds are added in double where a row takes 32 lanes or more, and in
// fp32 within a chunk of 64 ids and then across chunks where it takes fewer (in
// double 26 tables of 128 bf16 values take 140 us for 137).  One fp32 chain per
// lane group grows with the bag, and adding the same row over and over rounds the
// same way each time.  One id 4096 times in a bag, rows of 256 / 64 fp32 values:
// 3e-5 / 8e-6 off in the chain, exact / 5e-7 now; 4096 Zipf(1.2) ids, 64 values:
// 1.9e-6 and 6e-8.
//
// What bounds it: the rows the L2s miss, once the instructions per row are few
// enough.  Merging repeats by hash classes, LDS shuffles and a select per
// element, the kernel issued 640 vector instructions per bag of the 26-table
// bf16 workload (136M per call, about the kernel's whole 200 us on 1024 SIMDs
// at 4 cycles each); it issues 46M now and takes 134 us at 5.0 TB/s of L2 miss
// traffic (572 MB read, 109 MB written), the rate of a large device copy.  One
// 50M-row table, 16384 bags of 30 ids: 14-15 us either way (latency of four
// dependent loads); 8 tables of 1M rows: 22 -> 17 us (5.3 TB/s).
//
// Short bags: a wavefront per bag of one id leaves 63/64 of its loads unused
// and takes as long as a full one, so when the bags of a wavefront and its
// neighbours (four in all, or as many as there are lane groups) hold at most
// kShortBag ids each (one round of loads per lane group), the first of these
// wavefronts sums one bag per lane group and the others leave at once.
#include <type_traits>

#include "emb_common.h"
#include "kernels.h"

namespace emb {

namespace {

template <typename TW>
struct Vec;  // 16 bytes of table row

// (loaded raw, widened where it is used, so that every load of a round is
// issued before the first one is waited for)
template <>
struct Vec<float> {
  static constexpr int kElems = 4;
  __device__ __forceinline__ static void widen(const uint4& v, float (&o)[4]) {
    o[0] = __uint_as_float(v.x);
    o[1] = __uint_as_float(v.y);
    o[2] = __uint_as_float(v.z);
    o[3] = __uint_as_float(v.w);
  }
};

template <>
struct Vec<uint16_t> {
  static constexpr int kElems = 8;
  __device__ __forceinline__ static void widen(const uint4& v, float (&o)[8]) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = __uint_as_float(w[i] << 16);
      o[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
};

// value of lane (this lane's group)*G + u in every lane of the group
template <int G>
__device__ __forceinline__ uint32_t group_bcast(uint32_t v, int u, int g) {
  if constexpr (G == 64) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, u);
  } else {
    static_assert(G == 32, "narrower groups use DPP");
    const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)v, u);
    const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)v, u + 32);
    return g ? b : a;
  }
}
template <int G, int U>
__device__ __forceinline__ uint32_t group_bcast_dpp(uint32_t v) {
  static_assert(U < G, "lane of the group");
  const int x = (int)v;
  if constexpr (G == 16) {
    return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x150 + U, 0xf, 0xf, true);  // row_newbcast:U
  } else if constexpr (G == 8) {
    // lanes 0-7 of a row (banks 0 and 1) from lane U, lanes 8-15 from lane 8 + U
    const int lo = __builtin_amdgcn_mov_dpp(x, 0x150 + U, 0xf, 0xf, true);
    return (uint32_t)__builtin_amdgcn_update_dpp(lo, x, 0x150 + 8 + U, 0xf, 0xc, false);
  } else if constexpr (G == 4) {
    return (uint32_t)__builtin_amdgcn_mov_dpp(x, U * 0x55, 0xf, 0xf, true);  // quad_perm:[U,U,U,U]
  } else if constexpr (G == 2) {
    return (uint32_t)__builtin_amdgcn_mov_dpp(x, U == 0 ? 0xa0 : 0xf5, 0xf, 0xf, true);  // [U,U,2+U,2+U]
  } else {
    return v;
  }
}

template <int O, int NV, int E>
__device__ __forceinline__ void sum_groups(float (&acc)[NV][E]) {
  if constexpr (O < kWave) {
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int e = 0; e < E; ++e) acc[v][e] = add_across<O>(acc[v][e]);
    sum_groups<O * 2>(acc);
  }
}

// rows a lane group has in flight (for rows of NV vectors per lane)
constexpr int slots_in_flight(int g, int nv) { return 8 / nv < 1 ? 1 : (8 / nv < g ? 8 / nv : g); }
// bags short enough to be packed one per lane group
constexpr int kShortBag = 8;

// Bags whose repeated ids are merged: rows of 64 lanes, in bags of whole chunks
// of ids, or of enough ids to repeat the few rows of their table; rows of 32
// lanes in the latter only.  Measured (us, every id loaded -> merged), fp32:
//   512 values, 8192 bags of 100 ids of 10 rows     52   -> 17.9  (of 100 rows: 55 -> 47)
//   1024 values, 8192 bags of 64 ids of one row     62   -> 11.5
//   256 values, 4096 bags of 200 Zipf(1.2) ids      37.6 -> 32.5  (100 uniform ids: 63.2 -> 62.4)
//   256 values, 16384 bags of 20 ids of 3 rows      14.3 -> 10.1  (10 ids: 9.8 -> 10.1)
//   128 values, 16384 bags of 100 ids of 10 rows    29.4 -> 17.8  (40 ids of 40: 14.0 -> 14.4)
// With few repeats it loses: 128 values, bags of 30 Zipf(1.2) ids 14.2 -> 16.4,
// 512 bf16 values, bags of 20 Zipf(1.05) ids 9.6 -> 10.7.
__host__ __device__ constexpr bool merges_repeats(int g, int len, uint32_t rows) {
  const uint32_t n = (uint32_t)(len < kWave ? len : kWave);
  return g == 64 ? len >= kWave || (len >= 16 && rows <= 2 * n) : g == 32 && len >= 32 && rows <= n;
}

struct FwdArgs {
  const void* W;
  const int32_t* offsets;
  const void* idx;
  int32_t B, M, D, pool;
  uint32_t b_magic;  // bag_magic(B)
  float* out;
  TableOffsets ro;
};

// Slots [u0, u0 + UN) of every lane group (U0 the same number where it is a
// constant).  `row` holds, in lane g*G + u, the table row of group g's slot u;
// cnt is the group's number of slots.  Straight code: every load of the round
// is issued before the first is waited for.  Not FULL: slots the group lacks
// are read as zeros under a mask.
template <typename TW, int G, int NV, int UN, bool FULL, int U0, int U = 0>
__device__ __forceinline__ void load_slots(const char* const (&col)[NV], uint32_t rowbytes, uint32_t row, int u0,
                                           int cnt, int g, uint4 (&raw)[UN][NV]) {
  if constexpr (U < UN) {
    uint32_t r;
    if constexpr (G >= 32) r = group_bcast<G>(row, u0 + U, g);
    else r = group_bcast_dpp<G, U0 + U>(row);
    const uint64_t off = (uint64_t)r * (uint64_t)rowbytes;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if constexpr (FULL) {
        raw[U][v] = *reinterpret_cast<const uint4*>(col[v] + off);
      } else {
        raw[U][v] = make_uint4(0u, 0u, 0u, 0u);
        if (u0 + U < cnt) raw[U][v] = *reinterpret_cast<const uint4*>(col[v] + off);
      }
    }
    load_slots<TW, G, NV, UN, FULL, U0, U + 1>(col, rowbytes, row, u0, cnt, g, raw);
  }
}
// vector v of rows [U, U + N) of a round (N a power of two), added pairwise
template <typename TW, int U, int N, int UN, int NV>
__device__ __forceinline__ void sum_round(const uint4 (&raw)[UN][NV], int v, float (&o)[Vec<TW>::kElems]) {
  if constexpr (N == 1) {
    Vec<TW>::widen(raw[U][v], o);
  } else {
    float x[Vec<TW>::kElems];
    sum_round<TW, U, N / 2>(raw, v, o);
    sum_round<TW, U + N / 2, N / 2>(raw, v, x);
#pragma unroll
    for (int e = 0; e < Vec<TW>::kElems; ++e) o[e] += x[e];
  }
}
// (A: float for one or two rounds, else double)
template <typename TW, int G, int NV, int UN, bool FULL, int U0, typename A>
__device__ __forceinline__ void add_slots(const char* const (&col)[NV], uint32_t rowbytes, uint32_t row, int u0,
                                          int cnt, int g, A (&acc)[NV][Vec<TW>::kElems]) {
  uint4 raw[UN][NV];
  load_slots<TW, G, NV, UN, FULL, U0>(col, rowbytes, row, u0, cnt, g, raw);
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    float t[Vec<TW>::kElems];
    sum_round<TW, 0, UN>(raw, v, t);
#pragma unroll
    for (int e = 0; e < Vec<TW>::kElems; ++e) acc[v][e] += (A)t[e];
  }
}

// The slots of a chunk of ids from u0 on, nall of them present in every group
// and nmax in some group (both uniform): whole rounds without masks, then one
// masked round just long enough for what is left (a short bag does not pay
// for a long round).
template <typename TW, int G, int NV, int UN, int U0, typename A>
__device__ __forceinline__ void add_rest(const char* const (&col)[NV], uint32_t rowbytes, uint32_t row, int u0,
                                         int cnt, int nmax, int g, A (&acc)[NV][Vec<TW>::kElems]) {
  if constexpr (UN > 1) {
    if (nmax - u0 <= UN / 2) {
      add_rest<TW, G, NV, UN / 2, U0>(col, rowbytes, row, u0, cnt, nmax, g, acc);
      return;
    }
  }
  add_slots<TW, G, NV, UN, false, U0>(col, rowbytes, row, u0, cnt, g, acc);
}
template <typename TW, int G, int NV, int U0 = 0, typename A>
__device__ __forceinline__ void add_chunk(const char* const (&col)[NV], uint32_t rowbytes, uint32_t row, int cnt,
                                          int nall, int nmax, int g, A (&acc)[NV][Vec<TW>::kElems]) {
  constexpr int UN = slots_in_flight(G, NV);
  if constexpr (G >= 32) {
    int u0 = 0;
    for (; u0 + UN <= nall; u0 += UN) add_slots<TW, G, NV, UN, true, 0>(col, rowbytes, row, u0, cnt, g, acc);
    for (; u0 < nmax; u0 += UN) add_rest<TW, G, NV, UN, 0>(col, rowbytes, row, u0, cnt, nmax, g, acc);
  } else if constexpr (U0 < G) {
    if (U0 + UN <= nall) add_slots<TW, G, NV, UN, true, U0>(col, rowbytes, row, U0, cnt, g, acc);
    else if (U0 < nmax) add_rest<TW, G, NV, UN, U0>(col, rowbytes, row, U0, cnt, nmax, g, acc);
    if (U0 + UN < nmax) add_chunk<TW, G, NV, U0 + UN>(col, rowbytes, row, cnt, nall, nmax, g, acc);
  }
}

// A chunk's distinct rows and how often each occurs, dealt to the lane groups
// (`key`: the row of position `lane`, of n); returns their number.  Lanes are
// classed by an 8-bit hash of the row, one ballot a bit; a lane whose row is that
// of its class's lowest lane repeats it (a hash collision leaves a row twice).
template <int G>
__device__ __forceinline__ int merge_repeats(int lane, int n, uint32_t key, uint32_t& row, float& weight) {
  constexpr int R = kWave / G;
  const bool valid = lane < n;
  const uint64_t all = __ballot(valid);
  uint32_t lo = (uint32_t)all, hi = (uint32_t)(all >> 32);
  const uint32_t h = (key * 0x9e3779b1u) >> 24;
#pragma unroll
  for (int b = 0; b < 8; ++b) keep_peers(h, b, lo, hi);
  const uint64_t peers = ((uint64_t)hi << 32) | lo;
  const int lead = valid ? (int)__builtin_ctzll(peers) : lane;
  // (the shuffle runs on every lane: a lane switched off does not supply its value)
  const uint32_t lead_key = (uint32_t)__shfl((int)key, lead, kWave);
  const bool dup = valid && lead != lane && lead_key == key;
  const uint64_t dups = __ballot(dup);
  const bool keep = valid && !dup;
  const uint64_t kept = __ballot(keep);
  const int nk = (int)__popcll(kept);
  const int rank = keep ? (int)lanes_below(kept) : nk + (int)lanes_below(~kept);
  const int dst = rank % R * G + rank / R;
  const int times = keep ? 1 + (lead == lane ? (int)__popcll(dups & peers) : 0) : 0;
  row = (uint32_t)__builtin_amdgcn_ds_permute(dst << 2, (int)key);
  weight = __int_as_float(__builtin_amdgcn_ds_permute(dst << 2, __float_as_int((float)times)));
  return nk;
}

// A bag whose chunks' repeated rows are merged: rounds of multiply-adds, one chain
// each, the rounds in double.  Slots past a group's last hold rows that stand in
// and are dropped.
template <typename TW, int G, int NV, typename TI>
__device__ __forceinline__ void sum_merged(const char* const (&col)[NV], uint32_t rowbytes, const TI* idx, int start,
                                           int end, uint32_t base, int lane, float (&acc)[NV][Vec<TW>::kElems]) {
  constexpr int R = kWave / G, UN = slots_in_flight(G, NV), E = Vec<TW>::kElems;
  const int g = lane / G;
  double sum[NV][E] = {};
#pragma unroll 1
  for (int j0 = start; j0 < end; j0 += kWave) {
    const int n = min(kWave, end - j0);
    uint32_t row;
    float weight;
    // (lanes past the chunk stand in with the table's first row)
    const int nk = merge_repeats<G>(lane, n, base + (lane < n ? (uint32_t)(int32_t)idx[j0 + lane] : 0u), row, weight);
    const int cnt = (nk - g + R - 1) / R, nall = nk / R, nmax = (nk + R - 1) / R;
#pragma unroll 1
    for (int u0 = 0; u0 < nmax; u0 += UN) {
      uint4 raw[UN][NV];
      load_slots<TW, G, NV, UN, true, 0>(col, rowbytes, row, u0, cnt, g, raw);
      if (u0 + UN > nall) {
#pragma unroll
        for (int u = 0; u < UN; ++u)
#pragma unroll
          for (int v = 0; v < NV; ++v)
            if (u0 + u >= cnt) raw[u][v] = make_uint4(0u, 0u, 0u, 0u);
      }
      float t[NV][E] = {};
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const float w = __uint_as_float(group_bcast<G>(__float_as_uint(weight), u0 + u, g));
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          float x[E];
          Vec<TW>::widen(raw[u][v], x);
#pragma unroll
          for (int e = 0; e < E; ++e) t[v][e] = __builtin_fmaf(w, x[e], t[v][e]);
        }
      }
#pragma unroll
      for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int e = 0; e < E; ++e) sum[v][e] += (double)t[v][e];
    }
  }
#pragma unroll
  for (int v = 0; v < NV; ++v)
#pragma unroll
    for (int e = 0; e < E; ++e) acc[v][e] = (float)sum[v][e];
}

template <typename TW, int G, int NV, typename TI>
__global__ __launch_bounds__(256) void k_pool_fwd(FwdArgs a) {
  constexpr int R = kWave / G;
  constexpr int E = Vec<TW>::kElems;
  constexpr int P = R < 4 ? R : 4;  // bags a wavefront packs
  const int lane = threadIdx.x & (kWave - 1);
  // the bag is uniform across the wavefront: keep its bookkeeping scalar
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = (int)blockIdx.x * 4 + w;
  if (m >= a.M) return;
  const int g = lane / G, sub = lane % G;
  const TI* idx = static_cast<const TI*>(a.idx);
  const uint32_t rowbytes = (uint32_t)a.D * (uint32_t)sizeof(TW);

  // (rows wider than NV * G vectors: the row's part blockIdx.y)
  const int part = (int)blockIdx.y * (NV * G * E);
  const char* col[NV];  // this lane's columns (lanes past the row's end stand in at column 0, stored by none)
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int c0 = part + (v * G + sub) * E;
    col[v] = static_cast<const char*>(a.W) + (size_t)(c0 < a.D ? c0 : 0) * sizeof(TW);
  }

  int first, last;  // the bag's ids
  // the P bags of this wavefront and its neighbours, when they are all there
  const int m0 = m - w % P;
  if (P > 1 && a.B >= P && m0 + P <= a.M) {
    int o[P + 1];
#pragma unroll
    for (int i = 0; i <= P; ++i) o[i] = a.offsets[m0 + i];
    if constexpr (P > 1) {
      int lmax = 0, lmin = kShortBag;
#pragma unroll
      for (int i = 0; i < P; ++i) {
        lmax = max(lmax, o[i + 1] - o[i]);
        lmin = min(lmin, o[i + 1] - o[i]);
      }
      if (lmax <= (kShortBag < G ? kShortBag : G)) {
        if (w % P) return;
        // one bag per lane group (groups past P have none)
        int start = o[0], len = o[1] - o[0];
#pragma unroll
        for (int i = 1; i < P; ++i) {
          start = g == i ? o[i] : start;
          len = g == i ? o[i + 1] - o[i] : len;
        }
        if (g >= P) len = 0;
        const int t = (int)table_of_bag((uint32_t)m0, a.B, a.b_magic);
        // P bags lie in at most two tables
        const uint32_t base = m0 + g < (t + 1) * a.B ? a.ro.off[t] : a.ro.off[t + 1];
        const uint32_t row = sub < len ? base + (uint32_t)(int32_t)idx[start + sub] : 0u;
        static_assert(kShortBag <= 8 && NV == 1, "a short bag is one round");
        float acc[NV][E] = {};
        add_chunk<TW, G, NV>(col, rowbytes, row, len, R > P ? 0 : lmin, lmax, g, acc);
        const float scale = (a.pool == EMB_POOL_MEAN && len > 0) ? 1.0f / (float)len : 1.0f;
        float* op = a.out + (size_t)(m0 + g) * (size_t)a.D;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const int c0 = (v * G + sub) * E;
          if (g < P && c0 < a.D) {
#pragma unroll
            for (int e = 0; e < E; e += 4)
              *reinterpret_cast<float4*>(op + c0 + e) = make_float4(acc[v][e] * scale, acc[v][e + 1] * scale,
                                                                    acc[v][e + 2] * scale, acc[v][e + 3] * scale);
          }
        }
        return;
      }
    }
    first = o[0];
    last = o[1];
#pragma unroll
    for (int i = 1; i < P; ++i) {
      first = w % P == i ? o[i] : first;
      last = w % P == i ? o[i + 1] : last;
    }
  } else {
    first = a.offsets[m];
    last = a.offsets[m + 1];
  }

  // one bag: group g takes ids g, g + R, g + 2R, ... of every 64
  const int start = __builtin_amdgcn_readfirstlane(first), end = __builtin_amdgcn_readfirstlane(last);
  const int t = (int)table_of_bag((uint32_t)m, a.B, a.b_magic);
  const uint32_t base = a.ro.off[t];
  float acc[NV][E];
  if (merges_repeats(G, end - start, a.ro.off[t + 1] - base)) {
    if constexpr (G >= 32) sum_merged<TW, G, NV, TI>(col, rowbytes, idx, start, end, base, lane, acc);
  } else {
    // (chunks of one or two rounds: their sums, and the bag's of these, in fp32)
    typename std::conditional<(G >= 32), double, float>::type sum[NV][E] = {};
    for (int j0 = start; j0 < end; j0 += kWave) {
      const int n = min(kWave, end - j0);
      const int k = sub * R + g;
      const uint32_t row = k < n ? base + (uint32_t)(int32_t)idx[j0 + k] : 0u;
      if constexpr (G >= 32) {
        add_chunk<TW, G, NV>(col, rowbytes, row, (n - g + R - 1) / R, n / R, (n + R - 1) / R, g, sum);
      } else {
        float t[NV][E] = {};
        add_chunk<TW, G, NV>(col, rowbytes, row, (n - g + R - 1) / R, n / R, (n + R - 1) / R, g, t);
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll
          for (int e = 0; e < E; ++e) sum[v][e] += t[v][e];
      }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int e = 0; e < E; ++e) acc[v][e] = (float)sum[v][e];
  }
  sum_groups<G>(acc);

  const int L = end - start;
  const float scale = (a.pool == EMB_POOL_MEAN && L > 0) ? 1.0f / (float)L : 1.0f;
  float* op = a.out + (size_t)m * (size_t)a.D;
  if (g == 0) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int c0 = part + (v * G + sub) * E;
      if (c0 < a.D) {
#pragma unroll
        for (int e = 0; e < E; e += 4)
          *reinterpret_cast<float4*>(op + c0 + e) = make_float4(acc[v][e] * scale, acc[v][e + 1] * scale,
                                                                acc[v][e + 2] * scale, acc[v][e + 3] * scale);
      }
    }
  }
}

template <typename TW, int G, int NV>
hipError_t launch_t(const FwdLaunch& p, hipStream_t s) {
  constexpr int kPart = NV * G * Vec<TW>::kElems;
  dim3 grid((unsigned)((p.M + 3) / 4), (unsigned)((p.D + kPart - 1) / kPart)), block(256);
  FwdArgs a;
  a.W = p.W;
  a.offsets = p.offsets;
  a.idx = p.idx;
  a.B = p.B;
  a.M = p.M;
  a.D = p.D;
  a.pool = p.pool;
  a.b_magic = bag_magic(p.B);
  a.out = p.out;
  a.ro = p.ro;
  // the index type (int32 or int64) is a template argument: no per-load branch
  if (p.idx64) hipLaunchKernelGGL((k_pool_fwd<TW, G, NV, int64_t>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((k_pool_fwd<TW, G, NV, int32_t>), grid, block, 0, s, a);
  return hipGetLastError();
}

template <typename TW>
hipError_t launch_dtype(const FwdLaunch& p, hipStream_t s) {
  const int vecs = p.D * (int)sizeof(TW) / 16;  // 16-byte vectors per row
  if (vecs <= 1) return launch_t<TW, 1, 1>(p, s);
  if (vecs <= 2) return launch_t<TW, 2, 1>(p, s);
  if (vecs <= 4) return launch_t<TW, 4, 1>(p, s);
  if (vecs <= 8) return launch_t<TW, 8, 1>(p, s);
  if (vecs <= 16) return launch_t<TW, 16, 1>(p, s);
  if (vecs <= 32) return launch_t<TW, 32, 1>(p, s);
  if (vecs <= 64) return launch_t<TW, 64, 1>(p, s);
  // wider rows in parts of 128 vectors, a wavefront each: the sums of a whole row
  // leave registers for one to three wavefronts per SIMD (2048 bags of 20 ids,
  // 2048 fp32 values: 86 us whole, 28 in parts; 4096 bf16 values: 60 and 31)
  if (vecs <= 512) return launch_t<TW, 64, 2>(p, s);
  return hipErrorInvalidValue;
}

}  // namespace

int fwd_max_row_vectors() { return 512; }

hipError_t launch_pool_fwd(const FwdLaunch& p, hipStream_t s) {
  if (p.M == 0) return hipSuccess;
  return p.dtype == EMB_FP32 ? launch_dtype<float>(p, s) : launch_dtype<uint16_t>(p, s);
}

}  // namespace emb
