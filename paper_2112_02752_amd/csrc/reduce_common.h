// What the two forms of the gradient reduce share: arguments, rounding of
// stored rows, and the pieces of long segments within a chunk.
#pragma once

#include "emb_common.h"
#include "kernels.h"

namespace emb {

struct Upd {
  void* W;
  float* state;
  int32_t D, opt, fuse;
  float lr, eps;
  int32_t rounding;  // bf16 stores: 0 nearest even, 1 stochastic
  uint64_t seed;
};

struct RArgs {
  const float* G;
  const int32_t* seg;
  const uint32_t* ukeys;
  const int32_t* num_unique;
  const int32_t* sorted_bag;  // bag of every sorted position
  const int32_t* offsets;     // bag offsets (mean pooling scales by 1 / bag length)
  const int32_t* chunk_seg;
  float* grad_rows;
  float* partials;
  uint64_t* level2;     // [ncomb][2][D] tagged rows, cleared by the main kernel
  uint32_t* arrivals;   // [ncomb] arrival counters, cleared by the main kernel
  int32_t ncomb;        // combine blocks
  void* hdr;            // workspace header (error bits)
  int32_t N, D, pool, nchunks;
  int32_t split;        // wave form: 2^split wavefronts share a chunk (a block is one chunk, or four if they do not)
  Upd up;
};

struct UArgs {
  const float* grad_rows;
  const uint32_t* ukeys;
  const int32_t* num_unique;
  int32_t max_unique;
  uint32_t rows;
  Upd up;
};

// the wave form (reduce_wave.hip), for rows of more than kLaneGroupDim values
constexpr int kLaneGroupDim = 32;
hipError_t launch_reduce_wave(const RArgs& ra, int dtype, hipStream_t s);
hipError_t launch_update_wave(const UArgs& ua, int dtype, hipStream_t s);

// splitmix64 (Steele, Lea and Flood 2014): the output for generator state x
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
  uint64_t z = x + 0x9e3779b97f4a7c15ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

// One stored value with stochastic rounding to bf16: the top 16 bits of
// splitmix64(seed ^ splitmix64(c)), c the element's counter, are added to the
// 16 bits below the bf16 mantissa, which are then cut off (the magnitude
// rounds up with probability dropped / 2^16); non-finite values round to
// nearest even.
__device__ __forceinline__ uint16_t bf16_stochastic(float x, uint64_t seed, uint64_t c) {
  const uint32_t u = __float_as_uint(x);
  const uint32_t r16 = (uint32_t)(splitmix64(seed ^ splitmix64(c)) >> 48);
  return (u & 0x7f800000u) == 0x7f800000u ? f32_to_bf16_rne(x) : (uint16_t)((u + r16) >> 16);
}

// whether the dedup this reduce follows flagged an error: its unique scan made
// its generation the header's, so its error bits are those of that generation
__device__ __forceinline__ bool dedup_failed(const RArgs& a) {
  const WsHeader* h = reinterpret_cast<const WsHeader*>(a.hdr);
  return (call_errors(h, h->gen) & kDedupErrors) != 0u;
}

// 1 / bag length for mean pooling (a position's bag is never empty), else 1
__device__ __forceinline__ float bag_scale(const RArgs& a, int bag) {
  return a.pool == EMB_POOL_MEAN ? 1.0f / (float)(a.offsets[bag + 1] - a.offsets[bag]) : 1.0f;
}

// Metadata of one heavy-segment check: the pieces of heavy segments that
// lie in chunk c.  Slot 0: the segment holding the chunk's first position
// (if heavy); slot 1: a different heavy segment holding its last position.
struct ChunkPieces {
  int lo[2], hi[2];
  int u0, s0, e0;  // the segment holding the chunk's first position
  int u1, s1, e1;  // the segment holding the chunk's last position
};

__device__ __forceinline__ ChunkPieces chunk_pieces(const RArgs& a, int c, int U) {
  ChunkPieces r;
  const int p0 = c * kChunk, p1 = min(a.N, p0 + kChunk);
  const int u0 = a.chunk_seg[c], cs1 = a.chunk_seg[c + 1];
  // all needed offsets in one round of independent loads
  const int s0 = a.seg[u0], e0 = a.seg[u0 + 1];
  const int sc = a.seg[cs1];
  const int scm = cs1 > 0 ? a.seg[cs1 - 1] : 0;
  const int scp = cs1 < U ? a.seg[cs1 + 1] : a.N;
  if (sc == p1) {  // position p1 starts segment cs1: the chunk ends with segment cs1 - 1
    r.u1 = cs1 - 1;
    r.s1 = scm;
    r.e1 = sc;
  } else {
    r.u1 = cs1;
    r.s1 = sc;
    r.e1 = scp;
  }
  r.u0 = u0;
  r.s0 = s0;
  r.e0 = e0;
  r.lo[0] = r.hi[0] = r.lo[1] = r.hi[1] = 0;
  if (e0 - s0 > kChunk) {
    r.lo[0] = p0;
    r.hi[0] = min(p1, e0);
  }
  if (r.u1 != u0 && r.e1 - r.s1 > kChunk) {
    r.lo[1] = r.s1;
    r.hi[1] = p1;
  }
  return r;
}

// level-2 rows carry this tag (rows and counters are cleared by the main kernel)
constexpr uint32_t kLevel2Tag = 1u;

}  // namespace emb
