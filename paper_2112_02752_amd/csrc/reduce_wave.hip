// Backward segment-reduce and sparse optimizer step for rows of more than 32
// values (gfx950): a row is held by the whole wavefront.
//
//   g_u = sum over sorted positions k of segment u of scale_{m(k)} * G[m(k)]
//   W_r <- opt(W_r, g_u), r = unique_keys[u]
//
// Each lane holds EL columns (1 for rows of up to 64 values, 2 up to 128, ...)
// and a wavefront walks the 64 sorted positions of one chunk in order.  What
// is walked is uniform across the wavefront, so bags, keys, row addresses and
// the decision where a segment ends live in scalar registers, and a position
// costs one row load and EL multiply-adds, whatever the segments' lengths.
// The gradient rows of a batch of positions, and the table rows (and state) of
// the segments that end in it, are loaded together before any is used.
//  - A segment of at most kChunk positions belongs to the chunk it starts in,
//    whose wavefront walks on into the next chunk for its last positions and
//    applies the optimizer.  Each row has exactly one owner.
//  - A longer one leaves a partial row per chunk it crosses; k_combine_wave
//    adds them in chunk order and applies the optimizer.
// Every sum runs in a fixed order, so results are bitwise reproducible.
//
// What bounds it: the L2s' misses (gradient rows, and table rows read and
// written).  200M-row-like long tail (64 fp32 values, 3.3M lookups, SGD): 337
// -> 234 us, 1.6 GB of L2 misses at 6.9 TB/s; there lane groups (reduce.hip)
// wait for the longest of a wavefront's 16 segments and load stand-in rows for
// the rest.  26 tables of 128 bf16 values, 5.5M lookups, row-wise Adagrad: 510
// -> 321 us: neighbouring chunks run at the same time on all of the chip, so
// one table's gradient rows (4 MB) are used while they are in the L2s (2.53 ->
// 1.27 GB read); with light and heavy segments on wavefronts of their own,
// several tables' rows were live at once.  It is then bound by instruction
// issue (1350 vector and 750 scalar a chunk) as much as by misses (4.8 TB/s).
// Element-wise Adagrad, 104 bf16 values, 277k lookups: 99 -> 65 us (stochastic
// rounding's 64-bit products are half of its instructions).
// Measured and not kept: chunks dealt to the XCDs in runs of 16 to 4096
// (nothing gained, the largest lose), the next batch's rows loaded during the
// sums (20 more registers: 5 to 8% slower), batches of 4 or 16 positions.
#include "reduce_common.h"

namespace emb {

namespace {

// optimizer of a kernel instance; kReduceOnly writes gradient rows alone
constexpr int kReduceOnly = 3;

template <int EL>
struct Cols {
  static constexpr int VW = EL < 4 ? EL : 4;  // consecutive columns per vector
  static constexpr int NV = EL / VW;
  uint32_t at[NV];  // this lane's first column of each vector (0 stands in past the row's end)
  bool ok[NV];
  __device__ __forceinline__ Cols(int lane, int D) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int c = v * kWave * VW + lane * VW;
      ok[v] = c < D;
      at[v] = ok[v] ? (uint32_t)c : 0u;
    }
  }
};

// Rows are addressed by 64-bit addresses that are uniform across the
// wavefront (a lane computes each row's address once, for all rows of a chunk
// together) and the lane's column offset: a load then needs no address
// arithmetic.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef double f64x2 __attribute__((ext_vector_type(2)));
template <typename T>
__device__ __forceinline__ T load_at(uint64_t row, uint32_t off) {
  return *reinterpret_cast<const __attribute__((address_space(1))) T*>(
      reinterpret_cast<const __attribute__((address_space(1))) char*>(row) + off);
}
template <typename T>
__device__ __forceinline__ void store_at(uint64_t row, uint32_t off, T v) {
  *reinterpret_cast<__attribute__((address_space(1))) T*>(
      reinterpret_cast<__attribute__((address_space(1))) char*>(row) + off) = v;
}
__device__ __forceinline__ uint64_t addr_of(const void* p) { return reinterpret_cast<uint64_t>(p); }

// row of floats -> this lane's columns
template <int EL>
__device__ __forceinline__ void load_f32(uint64_t row, const Cols<EL>& cl, float (&x)[EL]) {
  constexpr int VW = Cols<EL>::VW;
#pragma unroll
  for (int v = 0; v < Cols<EL>::NV; ++v) {
    if constexpr (VW == 1) {
      x[v] = load_at<float>(row, cl.at[v] * 4u);
    } else if constexpr (VW == 2) {
      const f32x2 t = load_at<f32x2>(row, cl.at[v] * 4u);
      x[2 * v] = t.x;
      x[2 * v + 1] = t.y;
    } else {
      const f32x4 t = load_at<f32x4>(row, cl.at[v] * 4u);
      x[4 * v] = t.x;
      x[4 * v + 1] = t.y;
      x[4 * v + 2] = t.z;
      x[4 * v + 3] = t.w;
    }
  }
}
template <int EL>
__device__ __forceinline__ void store_f32(uint64_t row, const Cols<EL>& cl, const float (&x)[EL]) {
  constexpr int VW = Cols<EL>::VW;
#pragma unroll
  for (int v = 0; v < Cols<EL>::NV; ++v) {
    if (!cl.ok[v]) continue;
    if constexpr (VW == 1) store_at<float>(row, cl.at[v] * 4u, x[v]);
    else if constexpr (VW == 2) store_at<f32x2>(row, cl.at[v] * 4u, f32x2{x[2 * v], x[2 * v + 1]});
    else store_at<f32x4>(row, cl.at[v] * 4u, f32x4{x[4 * v], x[4 * v + 1], x[4 * v + 2], x[4 * v + 3]});
  }
}

// a table row's columns, as stored
template <typename TW, int EL>
struct WRow;
template <int EL>
struct WRow<float, EL> {
  float x[EL];
  __device__ __forceinline__ void load(uint64_t row, const Cols<EL>& cl) { load_f32<EL>(row, cl, x); }
  __device__ __forceinline__ float get(int e) const { return x[e]; }
  __device__ __forceinline__ static void store(const Upd&, uint64_t row, uint32_t, const Cols<EL>& cl,
                                               const float (&o)[EL]) {
    store_f32<EL>(row, cl, o);
  }
};
template <int EL>
struct WRow<uint16_t, EL> {
  static constexpr int VW = Cols<EL>::VW, NV = Cols<EL>::NV, RV = VW == 4 ? 2 : 1;
  uint32_t r[NV * RV];
  __device__ __forceinline__ void load(uint64_t row, const Cols<EL>& cl) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if constexpr (VW == 1) {
        r[v] = load_at<uint16_t>(row, cl.at[v] * 2u);
      } else if constexpr (VW == 2) {
        r[v] = load_at<uint32_t>(row, cl.at[v] * 2u);
      } else {
        const u32x2 t = load_at<u32x2>(row, cl.at[v] * 2u);
        r[2 * v] = t.x;
        r[2 * v + 1] = t.y;
      }
    }
  }
  __device__ __forceinline__ float get(int e) const {
    if constexpr (VW == 1) return __uint_as_float(r[e] << 16);
    else return __uint_as_float(e % 2 ? r[e / 2] & 0xffff0000u : r[e / 2] << 16);
  }
  __device__ __forceinline__ static void store(const Upd& up, uint64_t row, uint32_t key, const Cols<EL>& cl,
                                               const float (&o)[EL]) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      uint32_t b[VW];
      if (up.rounding) {
#pragma unroll
        for (int e = 0; e < VW; ++e)
          b[e] = bf16_stochastic(o[v * VW + e], up.seed, (uint64_t)key * (uint64_t)up.D + cl.at[v] + (uint64_t)e);
      } else {
#pragma unroll
        for (int e = 0; e < VW; ++e) b[e] = f32_to_bf16_rne(o[v * VW + e]);
      }
      if (!cl.ok[v]) continue;
      if constexpr (VW == 1) store_at<uint16_t>(row, cl.at[v] * 2u, (uint16_t)b[0]);
      else if constexpr (VW == 2) store_at<uint32_t>(row, cl.at[v] * 2u, b[0] | (b[1] << 16));
      else store_at<u32x2>(row, cl.at[v] * 2u, u32x2{b[0] | (b[1] << 16), b[2] | (b[3] << 16)});
    }
  }
};

// what an update reads of a row it owns besides the row-wise accumulator,
// loaded ahead
template <typename TW, int EL, int OPT>
struct Owned {
  WRow<TW, EL> w;
  float h[EL];  // element-wise Adagrad
  __device__ __forceinline__ void load(const Upd& up, uint64_t row, uint32_t key, const Cols<EL>& cl) {
    if constexpr (OPT != kReduceOnly) w.load(row, cl);
    if constexpr (OPT == EMB_OPT_ADAGRAD_ELEMENTWISE) load_f32<EL>(state_row(up, key), cl, h);
  }
  // element-wise Adagrad: the row's accumulators
  __device__ __forceinline__ static uint64_t state_row(const Upd& up, uint32_t key) {
    return addr_of(up.state) + (uint64_t)key * (uint64_t)up.D * 4u;
  }
};

// value of lane l ^ O
template <int O>
__device__ __forceinline__ float lane_xor(float x) {
  const int v = __float_as_int(x);
  if constexpr (O == 1) return __int_as_float(__builtin_amdgcn_mov_dpp(v, 0xb1, 0xf, 0xf, true));  // quad_perm:[1,0,3,2]
  else if constexpr (O == 2) return __int_as_float(__builtin_amdgcn_mov_dpp(v, 0x4e, 0xf, 0xf, true));  // [2,3,0,1]
  else if constexpr (O == 4) return __int_as_float(__builtin_amdgcn_ds_swizzle(v, 0x101f));  // xor 4
  else return __int_as_float(__builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true));  // O == 8: row_ror:8
}
// N rows (a power of two, at most 8), one value per lane each, summed over the
// wavefront: lane l gets row l % N's sum.  The order of the additions (lanes 1
// apart, then 2, 4, ... 32) is that of any other N.
template <int N, int O = 1, int BT>
__device__ __forceinline__ float rows_sum(float (&r)[BT], int lane) {
#pragma clang fp contract(off)
  if constexpr (N > 1) {
    const bool hi = (lane & O) != 0;
#pragma unroll
    for (int i = 0; i < N / 2; ++i) {
      const float keep = hi ? r[2 * i + 1] : r[2 * i], give = hi ? r[2 * i] : r[2 * i + 1];
      r[i] = keep + lane_xor<O>(give);
    }
    return rows_sum<N / 2, O * 2>(r, lane);
  } else if constexpr (O < 16) {
    r[0] += lane_xor<O>(r[0]);
    return rows_sum<1, O * 2>(r, lane);
  } else {
    return add_across<32>(add_across<16>(r[0]));
  }
}

__device__ __forceinline__ uint32_t lane_value(uint32_t v, int l) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}
__device__ __forceinline__ float lane_value(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ uint64_t lane_value(uint64_t v, int l) {
  return ((uint64_t)lane_value((uint32_t)(v >> 32), l) << 32) | lane_value((uint32_t)v, l);
}
__device__ __forceinline__ uint64_t lane_shfl(uint64_t v, int l) {
  return ((uint64_t)(uint32_t)__shfl((int)(v >> 32), l, kWave) << 32) | (uint32_t)__shfl((int)(uint32_t)v, l, kWave);
}

// x summed over the wavefront, in every lane, in the order of rows_sum
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
#pragma clang fp contract(off)
  return x + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float wave_sum(float x) {
  // (lanes of a quad, then of half a row, hold equal sums: a mirror is as good as an xor)
  float r[1] = {dpp_add<0x140>(dpp_add<0x141>(dpp_add<0x4e>(dpp_add<0xb1>(x))))};
  return rows_sum<1, 16>(r, 0);
}

// The rows q of a batch whose bit is set in `mask`: g_u written out (if asked)
// and the optimizer applied.  Lane l holds the key, the segment, the table
// row's address and the row-wise accumulator of row l % BT; the scalars of
// row-wise Adagrad are computed for all rows of the batch at once, one row per
// lane.  The arithmetic does not depend on the batch, so the unfused update
// equals the fused one.
template <typename TW, int EL, int OPT, int BT>
__device__ __forceinline__ void apply_rows(const Upd& up, float* grad_rows, uint32_t mask, int u, uint32_t key,
                                           uint64_t row, float h, const float (&g)[BT][EL],
                                           const Owned<TW, EL, OPT> (&own)[BT], const Cols<EL>& cl, int lane) {
  // (which products are fused into sums is written out: it must not depend on the batch)
#pragma clang fp contract(off)
  if (grad_rows) {
    const uint64_t grow = addr_of(grad_rows) + (uint64_t)(uint32_t)u * (uint64_t)up.D * 4u;
#pragma unroll
    for (int q = 0; q < BT; ++q)
      if ((mask >> q) & 1u) store_f32<EL>(lane_value(grow, q), cl, g[q]);
  }
  if constexpr (OPT != kReduceOnly) {
    float step = up.lr;
    if constexpr (OPT == EMB_OPT_ADAGRAD_ROWWISE) {
      auto squares = [&](int q) {
        float sq = 0.f;
#pragma unroll
        for (int v = 0; v < Cols<EL>::NV; ++v) {
          float s = 0.f;
#pragma unroll
          for (int e = 0; e < Cols<EL>::VW; ++e)
            s = __builtin_fmaf(g[q][v * Cols<EL>::VW + e], g[q][v * Cols<EL>::VW + e], s);
          sq += cl.ok[v] ? s : 0.f;
        }
        return sq;
      };
      float total = 0.f;
      // one row at a time costs about 13 instructions a row, all together 67
      if (BT <= 4 || __popc(mask) <= 4) {
#pragma unroll
        for (int q = 0; q < BT; ++q)
          if ((mask >> q) & 1u) {
            const float t = wave_sum(squares(q));
            total = lane % BT == q ? t : total;
          }
      } else {
        float sq[BT];
#pragma unroll
        for (int q = 0; q < BT; ++q) sq[q] = squares(q);
        total = rows_sum<BT>(sq, lane);
      }
      h += total / (float)up.D;
      if (lane < BT && ((mask >> lane) & 1u)) up.state[key] = h;
      step = up.lr / (sqrtf(h) + up.eps);
    }
#pragma unroll
    for (int q = 0; q < BT; ++q)
      if ((mask >> q) & 1u) {
        float o[EL];
        if constexpr (OPT == EMB_OPT_ADAGRAD_ELEMENTWISE) {
          float hn[EL];
#pragma unroll
          for (int e = 0; e < EL; ++e) {
            hn[e] = __builtin_fmaf(g[q][e], g[q][e], own[q].h[e]);
            o[e] = own[q].w.get(e) - up.lr * g[q][e] / (sqrtf(hn[e]) + up.eps);
          }
          store_f32<EL>(Owned<TW, EL, OPT>::state_row(up, lane_value(key, q)), cl, hn);
        } else {
          const float st = OPT == EMB_OPT_ADAGRAD_ROWWISE ? lane_value(step, q) : step;
#pragma unroll
          for (int e = 0; e < EL; ++e) o[e] = __builtin_fmaf(-st, g[q][e], own[q].w.get(e));
        }
        WRow<TW, EL>::store(up, lane_value(row, q), lane_value(key, q), cl, o);
      }
  }
}

// Positions whose rows are loaded together.  The gradient rows and the owned
// rows of a batch then take, for rows of up to 256 values, 34 to 78 vector
// registers: 8 wavefronts per SIMD for gradient rows alone, 6 to 8 with an
// optimizer (row-wise Adagrad 7 up to 64 values, 6 fp32 and 7 bf16 up to 128, 6
// up to 256; up to 128 values its scalar registers are the limit as well, and
// some of them live in lanes of a vector register).
constexpr int batch_for(int el, int opt) {
  const int b = el <= 2 ? 8 : (el == 4 ? 4 : 2);
  return opt == EMB_OPT_ADAGRAD_ELEMENTWISE && b > 2 ? b / 2 : b;
}
// Positions summed apart from what came before them (shorter chains of
// roundings): the same for every optimizer, so that fused and unfused
// gradient rows are the same.
constexpr int sum_block(int el) { return batch_for(el, EMB_OPT_SGD); }

// OR over the wavefront of one bit per lane (uniform result)
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_or(uint32_t x) {
  return x | (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xf, 0xf, true);
}
__device__ __forceinline__ uint32_t wave_or(uint32_t x) {
  x = dpp_or<0x140>(dpp_or<0x141>(dpp_or<0x4e>(dpp_or<0xb1>(x))));
  return lane_value(x, 0) | lane_value(x, 16) | lane_value(x, 32) | lane_value(x, 48);
}

// zeros in place of the rows from n on (which stand-in loads brought)
template <int EL, int BT>
__device__ __forceinline__ void drop_rows(float (&x)[BT][EL], int n) {
#pragma unroll
  for (int q = 0; q < BT; ++q)
#pragma unroll
    for (int v = 0; v < EL; ++v) x[q][v] = q < n ? x[q][v] : 0.f;
}

// Within a segment the positions of one bag are consecutive (positions ascend
// and so do their bags): each run of one bag is one gradient row, weighted by
// its length.  From the bags and scales of n positions, one per lane, and the
// positions at which a segment ends: the runs' bags (lane i the i-th run's,
// with its last position's end flag in the top bit; 0 past the last run) and
// weights; returns the number of runs.  With R > 1 lane groups the i-th run
// goes to lane (i % R) * (64 / R) + i / R: group i % R, its slot i / R.
template <int R = 1>
__device__ __forceinline__ int bag_runs(int lane, int n, int bag, float scale, uint64_t pos_ends, uint32_t& run,
                                        float& weight) {
  const int before = __shfl_up(bag, 1, kWave);
  const bool head = lane < n && (lane == 0 || bag != before || ((pos_ends >> (lane - 1)) & 1u));
  const uint64_t heads = __ballot(head);
  const int nruns = (int)__popcll(heads);
  const uint64_t above = lane == kWave - 1 ? 0ull : heads >> (lane + 1);
  const int next = above ? lane + 1 + __builtin_ctzll(above) : n;
  const int rank = head ? (int)lanes_below(heads) : nruns + (int)lanes_below(~heads);
  const int dst = rank % R * (kWave / R) + rank / R;
  const uint32_t flag = head && ((pos_ends >> (next - 1)) & 1u) ? 0x80000000u : 0u;
  run = (uint32_t)__builtin_amdgcn_ds_permute(dst << 2, head ? (int)((uint32_t)bag | flag) : 0);
  weight = __int_as_float(
      __builtin_amdgcn_ds_permute(dst << 2, __float_as_int(head ? (float)(next - lane) * scale : 0.f)));
  return nruns;
}

// Runs in slots [U0, 16) of the four lane groups of 16 (lane 16 g + u: run
// 4 u + g), added to this lane's four columns at `col`, in double: a hot id's row
// is the sum of thousands of chunks', and what they are rounded by is most of
// its error (50M-row workload, 90k positions: 8e-5 with fp32 sums, partial rows
// and range rows, where the row's values are about 300).  Four slots, 16 rows, are
// loaded together; slots past the last run are read as zeros under a mask.
template <int U0, int U, bool FULL>
__device__ __forceinline__ void load_quad(uint64_t col, uint32_t rowbytes, uint32_t run, float weight, int nruns, int g,
                                          f32x4 (&x)[4], float (&wt)[4]) {
  if constexpr (U < 4) {
    const uint32_t r = (uint32_t)__builtin_amdgcn_mov_dpp((int)run, 0x150 + U0 + U, 0xf, 0xf, true);  // row_newbcast
    wt[U] = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(weight), 0x150 + U0 + U, 0xf, 0xf, true));
    x[U] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (FULL || (U0 + U) * 4 + g < nruns) x[U] = load_at<f32x4>(col + (uint64_t)r * rowbytes, 0u);
    load_quad<U0, U + 1, FULL>(col, rowbytes, run, weight, nruns, g, x, wt);
  }
}
template <int U0 = 0>
__device__ __forceinline__ void add_quads(uint64_t col, uint32_t rowbytes, uint32_t run, float weight, int nruns, int g,
                                          double (&sum)[4]) {
  if constexpr (U0 < 16) {
    if (nruns <= U0 * 4) return;
    f32x4 x[4];
    float wt[4];
    if (nruns >= (U0 + 4) * 4) load_quad<U0, 0, true>(col, rowbytes, run, weight, nruns, g, x, wt);
    else load_quad<U0, 0, false>(col, rowbytes, run, weight, nruns, g, x, wt);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) sum[i] = __builtin_fma((double)wt[u], (double)x[u][i], sum[i]);
    add_quads<U0 + 4>(col, rowbytes, run, weight, nruns, g, sum);
  }
}

// s_waitcnt of all loads (vmcnt 0, the other counters not waited for)
constexpr int kWaitLoads = 0x0f70;

template <typename TW, int EL, int OPT>
__global__ __launch_bounds__(256) void k_reduce_wave(RArgs a) {
  constexpr int BT = batch_for(EL, OPT), SB = sum_block(EL);
  __shared__ float s_part[4 * 2][EL][kWave];  // long segments' rows of a split chunk's parts (part, slot)
  const int lane = threadIdx.x & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // a block is four chunks, or the parts of one
  const int threads = a.split == 1 ? 2 * kWave : 4 * kWave;
  const int D = a.D;
  const Cols<EL> cl(lane, D);
  const int U = *a.num_unique;
  if (dedup_failed(a)) {
    // The dedup this reduce follows flagged an error: its outputs are
    // undefined, so no table row is written.  Unfused, the gradient rows of
    // the unique ids it reported are zeroed, so that the optimizer step
    // applied to them afterwards leaves every row as it is (for SGD, and for
    // Adagrad with eps > 0).
    if (a.grad_rows) {
      const int64_t n = (int64_t)min(max(U, 0), a.N) * D;
      for (int64_t i = (int64_t)blockIdx.x * threads + threadIdx.x; i < n; i += (int64_t)gridDim.x * threads)
        a.grad_rows[i] = 0.f;
    }
    return;
  }
  // the combine that follows starts from cleared level-2 rows and counters
  {
    const int nw = a.ncomb * 2 * D;
    for (int i = (int)blockIdx.x * threads + (int)threadIdx.x; i < nw + a.ncomb; i += (int)gridDim.x * threads) {
      if (i < nw) a.level2[i] = 0;
      else a.arrivals[i - nw] = 0u;
    }
  }
  // this wavefront's positions [q0, q1): a chunk's, or its part `sw` of them
  // (parts of one chunk are the wavefronts of one block)
  const int c = a.split ? (int)blockIdx.x : (int)blockIdx.x * 4 + w;
  if (c >= a.nchunks) return;
  const int sw = a.split ? w : 0, P = kChunk >> a.split;
  const int p0 = c * kChunk, p1 = min(a.N, p0 + kChunk);
  const int q0 = p0 + sw * P, q1 = min(a.N, q0 + P), n = q1 - q0;  // n <= 0 past the last position

  const int cs0 = __builtin_amdgcn_readfirstlane(a.chunk_seg[c]);
  const int cs1 = __builtin_amdgcn_readfirstlane(a.chunk_seg[c + 1]);
  // the bags of these positions, and of the ones after them
  const int bag = q0 + lane < a.N ? a.sorted_bag[q0 + lane] : 0;
  // A long segment's partial row: slot 0 if the segment holds the chunk's
  // first position, else slot 1.  The parts' rows meet in LDS.
  auto store_part = [&](int slot, const float (&v)[EL]) {
    if (a.split) {
#pragma unroll
      for (int e = 0; e < EL; ++e) s_part[sw * 2 + slot][e][lane] = v[e];
    } else {
      store_f32<EL>(addr_of(a.partials) + ((uint64_t)c * 2 + slot) * (uint64_t)D * 4u, cl, v);
    }
  };
  // the parts' rows of slot `slot`, parts [i0, i1), added in order by one wavefront
  auto join_parts = [&](int slot, int i0, int i1) {
    float sum[EL];
#pragma unroll
    for (int v = 0; v < EL; ++v) sum[v] = 0.f;
    for (int i = i0; i < i1; ++i)
#pragma unroll
      for (int v = 0; v < EL; ++v) sum[v] += s_part[i * 2 + slot][v][lane];
    store_f32<EL>(addr_of(a.partials) + ((uint64_t)c * 2 + slot) * (uint64_t)D * 4u, cl, sum);
  };
  if (cs0 == cs1) {
    // The whole chunk, and the position after it, lie in one segment (a long
    // one): its sum is the segment's partial row.  Most chunks of a skewed
    // batch are of this kind, and need no segment's bounds, keys or rows: one
    // wavefront does all of it.
    if (sw) return;
    uint32_t run;
    float weight;
    if constexpr (EL == 1) {
      // rows of up to 64 values: four at a time, 16 lanes to a row (a row a
      // wavefront load would take twice the instructions per row)
      const int nruns = bag_runs<4>(lane, kChunk, bag, bag_scale(a, bag), 0ull, run, weight);
      const int sub = lane % 16;
      const uint64_t col = addr_of(a.G) + (sub * 4 < D ? (uint64_t)sub * 16u : 0ull);
      double sum[4] = {0., 0., 0., 0.};
      add_quads(col, (uint32_t)D * 4u, run, weight, nruns, lane / 16, sum);
#pragma unroll
      for (int i = 0; i < 4; ++i) sum[i] = add_across<32>(add_across<16>(sum[i]));
      // (in double, over the place of both of the chunk's partial rows)
      if (lane < 16 && sub * 4 < D) {
        const uint64_t dst = addr_of(a.partials) + (uint64_t)c * 2 * (uint64_t)D * 4u;
        store_at<f64x2>(dst, (uint32_t)sub * 32u, f64x2{sum[0], sum[1]});
        store_at<f64x2>(dst, (uint32_t)sub * 32u + 16u, f64x2{sum[2], sum[3]});
      }
      return;
    }
    const int nruns = bag_runs(lane, kChunk, bag, bag_scale(a, bag), 0ull, run, weight);
    const uint64_t row = addr_of(a.G) + (uint64_t)run * ((uint64_t)D * 4u);
    constexpr int LB = EL <= 2 ? 16 : (EL == 4 ? 8 : 4);
    float acc[EL];
#pragma unroll
    for (int v = 0; v < EL; ++v) acc[v] = 0.f;
    for (int b = 0; b < nruns; b += LB) {
      float x[LB][EL];
#pragma unroll
      for (int q = 0; q < LB; ++q) load_f32<EL>(lane_value(row, b + q), cl, x[q]);
      if (nruns - b < LB) drop_rows<EL, LB>(x, nruns - b);
      float t[EL];
#pragma unroll
      for (int v = 0; v < EL; ++v) t[v] = 0.f;
#pragma unroll
      for (int q = 0; q < LB; ++q) {
        const float wt = lane_value(weight, b + q);
#pragma unroll
        for (int v = 0; v < EL; ++v) t[v] = __builtin_fmaf(wt, x[q][v], t[v]);
      }
#pragma unroll
      for (int v = 0; v < EL; ++v) acc[v] += t[v];
    }
    store_f32<EL>(addr_of(a.partials) + (uint64_t)c * 2 * (uint64_t)D * 4u, cl, acc);
    return;
  }
  const int bag_next = q1 + lane < a.N ? a.sorted_bag[q1 + lane] : 0;
  // lane i: the i-th segment with a position in the chunk
  const int i0 = cs0 + lane;
  int s = 0x7fffffff, e = 0x7fffffff;
  uint32_t key = 0;
  if (i0 < U && i0 <= cs1) {
    s = a.seg[i0];
    e = a.seg[i0 + 1];
    key = a.ukeys[i0];
  }
  const uint64_t wrow = addr_of(a.up.W) + (uint64_t)key * ((uint64_t)D * sizeof(TW));
  // (each segment's row-wise accumulator; those not owned are not written)
  const float hseg = OPT == EMB_OPT_ADAGRAD_ROWWISE && e <= a.N ? a.up.state[key] : 0.f;
  const float scale = lane < n ? bag_scale(a, bag) : 0.f;
  const int f = (int)__popcll(__ballot(s <= q0)) - 1, l = (int)__popcll(__ballot(s < q1)) - 1;  // first, last segment
  const int s0 = (int)lane_value((uint32_t)s, f), e0 = (int)lane_value((uint32_t)e, f);
  const int sl = (int)lane_value((uint32_t)s, l), el = (int)lane_value((uint32_t)e, l);
  const bool long0 = e0 - s0 > kChunk, longl = el - sl > kChunk;
  // nothing to do: no positions, or all of them in a segment of an earlier part
  if (n > 0 && !(s0 < q0 && e0 > q1 && !long0)) {
  // positions at which a segment ends
  const int ep = e > q0 && e <= q1 ? e - 1 - q0 : -1;
  const uint64_t pos_ends = (uint64_t)wave_or(ep >= 0 && ep < 32 ? 1u << ep : 0u) |
                            (uint64_t)wave_or(ep >= 32 ? 1u << (ep & 31) : 0u) << 32;
  uint32_t run;
  float weight;
  const int nruns = bag_runs(lane, n, bag, scale, pos_ends, run, weight);
  const uint64_t ends = __ballot((run >> 31) != 0u);
  // address of each run's gradient row (row 0 stands in past the last run)
  const uint64_t row = addr_of(a.G) + (uint64_t)(run & 0x7fffffffu) * ((uint64_t)D * 4u);
  // All of the ends are owned by this wavefront, except that of a first
  // segment that started before: its row is the last partial of a long
  // segment, or belongs to the wavefront where it started.
  const bool head_in = s0 < q0 && e0 <= q1;
  const uint64_t owned = head_in ? ends & (ends - 1) : ends;

  float acc[EL], t[EL];
#pragma unroll
  for (int v = 0; v < EL; ++v) acc[v] = t[v] = 0.f;
  // the runs of a first segment that belongs to an earlier wavefront are walked over
  const int k0 = head_in && !long0 ? __builtin_ctzll(ends) + 1 : 0;
  float x[BT][EL];
  Owned<TW, EL, OPT> own[BT];
  for (int b = k0 / SB * SB; b < nruns; b += BT) {
    const uint32_t eb = (uint32_t)(ends >> b) & ((1u << BT) - 1u), ob = (uint32_t)(owned >> b) & ((1u << BT) - 1u);
    const int jb = f + (int)__popcll(ends & ((1ull << b) - 1ull));
    // the batch's gradient rows (row 0 stands in past the last run) and the
    // rows of the segments that end in it, all in flight together
#pragma unroll
    for (int q = 0; q < BT; ++q) load_f32<EL>(lane_value(row, b + q), cl, x[q]);
    if constexpr (OPT != kReduceOnly) {
      int j = jb;
#pragma unroll
      for (int q = 0; q < BT; ++q) {
        if ((ob >> q) & 1u) own[q].load(a.up, lane_value(wrow, j), lane_value(key, j), cl);
        j += (int)((eb >> q) & 1u);
      }
    }
    if (nruns - b < BT) drop_rows<EL, BT>(x, nruns - b);
    // Running sums replace the rows: x[q] is the sum up to run q of its
    // segment within the block, where a segment ends with what came before.
#pragma unroll
    for (int q = 0; q < BT; ++q) {
      const float wt = lane_value(weight, b + q);
#pragma unroll
      for (int v = 0; v < EL; ++v) x[q][v] = __builtin_fmaf(wt, x[q][v], t[v]);
      if ((eb >> q) & 1u) {
#pragma unroll
        for (int v = 0; v < EL; ++v) {
          x[q][v] += acc[v];
          acc[v] = t[v] = 0.f;
        }
      } else {
#pragma unroll
        for (int v = 0; v < EL; ++v) t[v] = x[q][v];
      }
    }
    if (BT == SB || (b + BT) % SB == 0 || b + BT >= nruns) {
#pragma unroll
      for (int v = 0; v < EL; ++v) {
        acc[v] += t[v];
        t[v] = 0.f;
      }
    }
    // every load of the batch has arrived: nothing that follows waits for the
    // stores below on a load's account
    __builtin_amdgcn_s_waitcnt(kWaitLoads);
    if (long0 && eb != ob) {
#pragma unroll
      for (int q = 0; q < BT; ++q)
        if (((eb & ~ob) >> q) & 1u) store_part(0, x[q]);
    }
    if (ob) {
      // lane l: the segment that ends at run l % BT of the batch, if one does
      const int jl = min(jb + (int)__popc(eb & ((1u << (lane % BT)) - 1u)), kWave - 1);
      const uint32_t kl = (uint32_t)__shfl((int)key, jl, kWave);
      const float hl = OPT == EMB_OPT_ADAGRAD_ROWWISE ? __shfl(hseg, jl, kWave) : 0.f;
      apply_rows<TW, EL, OPT, BT>(a.up, a.grad_rows, ob, cs0 + jl, kl, lane_shfl(wrow, jl), hl, x, own, cl, lane);
    }
  }
  // the last segment goes on past these positions
  if (el > q1) {
    if (longl) {
      store_part(l == 0 ? 0 : 1, acc);
    } else {
      const int rest = el - q1;
      const uint32_t lkey = lane_value(key, l);
      Owned<TW, EL, OPT> lown[1];
      lown[0].load(a.up, lane_value(wrow, l), lkey, cl);
      const float scale_next = lane < rest ? bag_scale(a, bag_next) : 0.f;
      const uint64_t row_next = addr_of(a.G) + (uint64_t)(uint32_t)bag_next * ((uint64_t)D * 4u);
      for (int b = 0; b < rest; b += BT) {
#pragma unroll
        for (int q = 0; q < BT; ++q)
          load_f32<EL>(lane_value(row_next, b + q), cl, x[q]);
        if (rest - b < BT) drop_rows<EL, BT>(x, rest - b);
#pragma unroll
        for (int q = 0; q < BT; ++q) {
          const float sc = lane_value(scale_next, b + q);
#pragma unroll
          for (int v = 0; v < EL; ++v) t[v] = __builtin_fmaf(sc, x[q][v], t[v]);
        }
        if (BT == SB || (b + BT) % SB == 0 || b + BT >= rest) {
#pragma unroll
          for (int v = 0; v < EL; ++v) {
            acc[v] += t[v];
            t[v] = 0.f;
          }
        }
      }
      float g[1][EL];
#pragma unroll
      for (int v = 0; v < EL; ++v) g[0][v] = acc[v];
      apply_rows<TW, EL, OPT, 1>(a.up, a.grad_rows, 1u, cs0 + l, lkey, lane_value(wrow, l), lane_value(hseg, l), g,
                                     lown, cl, lane);
    }
  }
  }
  if (a.split) {
    // the parts' rows of the chunk's long segments, added in order: slot 0 by
    // the first wavefront, slot 1 by the second (all wavefronts of the block
    // see the same chunk, so all or none reach the barrier)
    const int fs = (int)lane_value((uint32_t)s, 0), fe = (int)lane_value((uint32_t)e, 0);
    const int cl1 = (int)__popcll(__ballot(s < p1)) - 1;
    const int ls = (int)lane_value((uint32_t)s, cl1), le = (int)lane_value((uint32_t)e, cl1);
    const bool slot0 = fe - fs > kChunk, slot1 = cl1 > 0 && le - ls > kChunk;
    if (slot0 || slot1) {
      __syncthreads();
      // slot 0 lies in the parts that start before its end, slot 1 in those
      // that end after its start
      if (sw == 0 && slot0) join_parts(0, 0, min(1 << a.split, (fe - p0 + P - 1) / P));
      if (sw == 1 && slot1) join_parts(1, (ls - p0) / P, 1 << a.split);
    }
  }
}

// rows summed by a combine wavefront in one round.  (Not more: a combine is a
// few microseconds of dependent loads, and what it unrolls has to be fetched
// as instructions first; rows of 128 values: 64 a round took 16 us where 16 take
// less than 10, with 33 KB of code instead of 8.  Rows of up to 64 values, 50M-row
// workload: 16 a round 9.4 us, 32 8.7, and 7.5 with addresses of less code.)
constexpr int combine_rows(int el) { return el == 1 ? 32 : (el == 2 ? 16 : (el == 4 ? 8 : (el == 8 ? 4 : 2))); }
constexpr int level2_rows(int el) { return combine_rows(el) / 2; }

// Long segments.  The block of a range of kCombineChunks chunks lists (one
// lane per chunk) the pieces of long segments in its range: the segments
// that start in it and the one that holds its first position, if that one
// started earlier.  One wavefront per piece sums the piece's chunk partials
// in chunk order.  A segment that lies in the range is finished at once; a
// segment that crosses ranges leaves one row per range (slot 1 in the range
// where it starts, slot 0 in the others) as tagged words, and the block
// that arrives last at the segment's counter adds those rows in range order
// and applies the optimizer.  The order of every sum is fixed, so the result
// does not depend on which block arrives last; no block ever waits for
// another to arrive.  Rows are added in double: the partials of a hot id's
// thousands of positions are many and large, and their roundings in fp32 would
// be most of its row's error.
//
// Level-2 rows are words whose tag tells that they have arrived (the main kernel
// clears them): doubles whose last bit is set for rows of up to 64 values, a tag
// above a float for wider ones.
template <int EL>
__device__ __forceinline__ uint64_t level2_word(double x) {
  if constexpr (EL == 1) return (uint64_t)__double_as_longlong(x) | 1ull;
  else return ((uint64_t)kLevel2Tag << 32) | __float_as_uint((float)x);
}
template <int EL>
__device__ __forceinline__ double level2_value(uint64_t w) {
  if constexpr (EL == 1) return __longlong_as_double((int64_t)(w & ~1ull));
  else return (double)__uint_as_float((uint32_t)w);
}
template <int EL>
__device__ __forceinline__ void level2_sum(const RArgs& a, int g0, int g1, WsHeader* h, const Cols<EL>& cl,
                                           double (&sum)[EL]) {
  constexpr int RR = level2_rows(EL);
  constexpr int VW = Cols<EL>::VW;
#pragma unroll
  for (int v = 0; v < EL; ++v) sum[v] = 0.;
#pragma unroll 1
  for (int r0 = g0; r0 < g1; r0 += RR) {
    uint64_t x[RR][EL];
    uint32_t spins = 0;
    const uint64_t t0 = wait_clock();
    // the rows of a round are loaded together until all carry their tags
    // (rows past the last stand in with it)
    const uint64_t* src = a.level2 + (size_t)r0 * 2 * a.D;
#pragma unroll 1
    for (;;) {
      uint32_t tags = kLevel2Tag;
      uint32_t off = 0;
#pragma unroll
      for (int q = 0; q < RR; ++q) {
        // (the segment's first range left its row in slot 1)
        const uint64_t* row = src + off + (q == 0 && r0 == g0 ? a.D : 0);
#pragma unroll
        for (int v = 0; v < EL; ++v) x[q][v] = ld_relaxed_u64(row + cl.at[v / VW] + v % VW);
        off += r0 + q + 1 < g1 ? 2u * (uint32_t)a.D : 0u;
        asm("" : "+v"(off));
      }
#pragma unroll
      for (int q = 0; q < RR; ++q)
#pragma unroll
        for (int v = 0; v < EL; ++v) tags &= (uint32_t)(EL == 1 ? x[q][v] : x[q][v] >> 32);
      if (__ballot(tags != kLevel2Tag) == 0ull) break;
      if (wait_over(h, h->gen, t0, ++spins)) {
        flag_timeout(h, h->gen, kSiteCombine, kCombineError);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
#pragma unroll
    for (int q = 0; q < RR; ++q)
      if (r0 + q < g1) {
#pragma unroll
        for (int v = 0; v < EL; ++v) sum[v] += level2_value<EL>(x[q][v]);
      }
  }
}

template <typename TW, int EL, int OPT>
__global__ __launch_bounds__(kCombineThreads) void k_combine_wave(RArgs a) {
  constexpr int NWv = kCombineThreads / kWave;
  constexpr int CU = combine_rows(EL);
  constexpr int VW = Cols<EL>::VW;
  __shared__ int4 s_piece[kCombineChunks + 1];  // (segment, first chunk in range, start, end)
  __shared__ int s_n;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int D = a.D;
  const Cols<EL> cl(lane, D);
  const int U = *a.num_unique;
  if (dedup_failed(a)) return;  // as in k_reduce_wave
  const int blk = blockIdx.x;
  const int c0 = blk * kCombineChunks, c1 = min(a.nchunks, c0 + kCombineChunks);
  if (tid == 0) s_n = 0;
  __syncthreads();
  if (tid < c1 - c0) {
    const int c = c0 + tid;
    const ChunkPieces cp = chunk_pieces(a, c, U);
    if (cp.e1 - cp.s1 > kChunk && cp.s1 >= c * kChunk) s_piece[atomicAdd(&s_n, 1)] = make_int4(cp.u1, c, cp.s1, cp.e1);
    if (c == c0 && cp.hi[0] > cp.lo[0] && cp.s0 < c * kChunk)
      s_piece[atomicAdd(&s_n, 1)] = make_int4(cp.u0, c, cp.s0, cp.e0);
  }
  __syncthreads();
  const int n = s_n;
  for (int k = w; k < n; k += NWv) {
    const int4 pc = s_piece[k];
    const int u = __builtin_amdgcn_readfirstlane(pc.x), cf = __builtin_amdgcn_readfirstlane(pc.y);
    const int st = __builtin_amdgcn_readfirstlane(pc.z), en = __builtin_amdgcn_readfirstlane(pc.w);
    const int cs = st / kChunk, ce = (en - 1) / kChunk;  // chunks of the whole segment
    const int cl1 = min(c1 - 1, ce);                     // last chunk of this piece
    const int np = cl1 - cf + 1;
    const uint32_t key = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.ukeys[u]);
    Owned<TW, EL, OPT> own[1];
    const uint64_t wrow = addr_of(a.up.W) + (uint64_t)key * ((uint64_t)D * sizeof(TW));
    own[0].load(a.up, wrow, key, cl);
    const float h = OPT == EMB_OPT_ADAGRAD_ROWWISE ? a.up.state[key] : 0.f;
    double sum[EL];
#pragma unroll
    for (int v = 0; v < EL; ++v) sum[v] = 0.;
    if constexpr (EL == 1) {
      // The piece's whole chunks (that lie, with the position after them, in the
      // segment) left doubles; its first chunk, if the segment starts within it,
      // and its last, if the segment ends in it, floats.
      const bool part0 = st > cf * kChunk, part1 = en <= (cl1 + 1) * kChunk;
      const int w0 = cf + (part0 ? 1 : 0), w1 = cl1 + (part1 ? 0 : 1);
      const uint64_t stride = (uint64_t)D * 8u, rows = addr_of(a.partials);
      const float x0 = load_at<float>(rows + (uint64_t)cf * stride + (uint64_t)D * 4u, cl.at[0] * 4u);
      const float x1 = load_at<float>(rows + (uint64_t)cl1 * stride, cl.at[0] * 4u);
      // (rounds of 32 rows, whole ranges' in two; what is left, and short pieces, in
      // rounds of 8.  Addresses are the piece's first row and a 32-bit offset: a
      // 64-bit scalar for each of a round's rows is more than there are.)
      const uint64_t first = rows + (uint64_t)w0 * stride;
      const uint32_t step = (uint32_t)D * 8u;
      const int nw = w1 - w0;
      uint32_t off = cl.at[0] * 8u;
      int i0 = 0;
#pragma unroll 1
      for (; i0 + CU <= nw; i0 += CU) {
        double x[CU];
#pragma unroll
        for (int q = 0; q < CU; ++q) {
          x[q] = load_at<double>(first, off);
          off += step;
          asm("" : "+v"(off));  // (not 32 multiples of the step in scalars)
        }
#pragma unroll
        for (int q = 0; q < CU; ++q) sum[0] += x[q];
      }
#pragma unroll 1
      for (; i0 < nw; i0 += 8) {
        double x[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          x[q] = load_at<double>(first, off);
          off += i0 + q + 1 < nw ? step : 0u;
          asm("" : "+v"(off));
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) sum[0] += i0 + q < nw ? x[q] : 0.;
      }
      sum[0] += (part0 ? (double)x0 : 0.) + (part1 ? (double)x1 : 0.);
    } else {
      // lane i: the address of the piece's i-th partial (the last one's past it)
      const int ci = cf + min(lane, np - 1);
      const uint64_t prow =
          addr_of(a.partials) + ((uint64_t)ci * 2 + (ci == cs && st != ci * kChunk ? 1 : 0)) * ((uint64_t)D * 4u);
#pragma unroll 1
      for (int i0 = 0; i0 < np; i0 += CU) {
        float x[CU][EL];
#pragma unroll
        for (int q = 0; q < CU; ++q) load_f32<EL>(lane_value(prow, i0 + q), cl, x[q]);
        if (np - i0 < CU) drop_rows<EL, CU>(x, np - i0);
#pragma unroll
        for (int q = 0; q < CU; ++q)
#pragma unroll
          for (int v = 0; v < EL; ++v) sum[v] += (double)x[q][v];
      }
    }
    const int bs = cs / kCombineChunks, be = ce / kCombineChunks;  // combine blocks of the segment
    bool done = bs == be;
    if (!done) {
      // publish this range's row, then arrive
      uint64_t* dst = a.level2 + ((size_t)blk * 2 + (blk == bs ? 1 : 0)) * D;
#pragma unroll
      for (int v = 0; v < EL; ++v)
        if (cl.ok[v / VW]) st_u64(dst + cl.at[v / VW] + v % VW, level2_word<EL>(sum[v]));
      uint32_t old = 0;
      if (lane == 0) old = atomic_add_u32(&a.arrivals[bs], 1u);
      done = lane_value(old, 0) == (uint32_t)(be - bs);
      if (done) level2_sum<EL>(a, bs, be + 1, reinterpret_cast<WsHeader*>(a.hdr), cl, sum);
    }
    float acc1[1][EL];
#pragma unroll
    for (int v = 0; v < EL; ++v) acc1[0][v] = (float)sum[v];
    if (done) apply_rows<TW, EL, OPT, 1>(a.up, a.grad_rows, 1u, u, key, wrow, h, acc1, own, cl, lane);
  }
}

// rows a wavefront of the unfused update takes at a time
constexpr int kUpdateRows = 16;

template <typename TW, int EL, int OPT>
__global__ __launch_bounds__(256) void k_update_wave(UArgs a) {
  constexpr int BT = batch_for(EL, OPT);
  const int lane = threadIdx.x & (kWave - 1);
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Cols<EL> cl(lane, a.up.D);
  const int U = min(__builtin_amdgcn_readfirstlane(*a.num_unique), a.max_unique);
  for (int u0 = ((int)blockIdx.x * 4 + w) * kUpdateRows; u0 < U; u0 += (int)gridDim.x * 4 * kUpdateRows) {
    const int n = min(kUpdateRows, U - u0);
    // keys that are no rows (of a failed dedup) are never written through
    const uint32_t key = lane < n ? a.ukeys[u0 + lane] : 0xffffffffu;
    const bool is_row = lane < n && key < a.rows;
    const uint32_t rows = (uint32_t)__ballot(is_row);
    const uint64_t wrow = addr_of(a.up.W) + (uint64_t)key * ((uint64_t)a.up.D * sizeof(TW));
    const float hrow = OPT == EMB_OPT_ADAGRAD_ROWWISE && is_row ? a.up.state[key] : 0.f;
    for (int b = 0; b < n; b += BT) {
      float x[BT][EL];
      Owned<TW, EL, OPT> own[BT];
      const uint32_t mask = (rows >> b) & ((1u << BT) - 1u);
#pragma unroll
      for (int q = 0; q < BT; ++q) {
        if ((mask >> q) & 1u) {
          load_f32<EL>(addr_of(a.grad_rows) + (uint64_t)(u0 + b + q) * (uint64_t)a.up.D * 4u, cl, x[q]);
          own[q].load(a.up, lane_value(wrow, b + q), lane_value(key, b + q), cl);
        } else {
#pragma unroll
          for (int v = 0; v < EL; ++v) x[q][v] = 0.f;
        }
      }
      const int l = b + lane % BT;
      const uint32_t kl = (uint32_t)__shfl((int)key, l, kWave);
      const float hl = OPT == EMB_OPT_ADAGRAD_ROWWISE ? __shfl(hrow, l, kWave) : 0.f;
      apply_rows<TW, EL, OPT, BT>(a.up, nullptr, mask, u0 + l, kl, lane_shfl(wrow, l), hl, x, own, cl, lane);
    }
  }
}

// Chunks of a batch up to which four, and two, wavefronts share each.  One
// wavefront to a chunk fills the device once with 7000 to 8000 chunks (7 or 8 to
// a SIMD), and a few chunks more are a second round of few wavefronts; the parts
// of a chunk cost its bounds again.  Gradient rows alone take fewer instructions
// and registers, and gain less (they are summed by the same parts, so that they
// are those of the fused step).  Main kernel and combine, six batches in turn, one
// / two / four wavefronts to a chunk (us):
//   64 fp32 values       row-wise Adagrad,      the same,              gradient rows alone,
//                        Zipf 1.2               Zipf 0.9               8 tables, Zipf 1.1
//     3.7k chunks        28.6 / 25.8 / 24.8     42.8 / 42.8 / 42.5     22.9 / 21.8 / 21.9
//     5.7k               33.5 / 28.7 / 30.3     54.8 / 51.9 / 54.5     25.6 / 24.6 / 25.4
//     9.5k               39.3 / 36.2 / 39.1     76.9 / 71.9 / 78.9     31.7 / 31.2 / 33.7
//    13.4k               47.8 / 45.0 / 50.6     93.5 / 90.9 / 102      39.6 / 41.4 / 46.1
//    17.2k               57.3 / 55.5 / 64.2      113 / 110 / 125       48.3 / 50.4 / 57.1
//   256 fp32 values      row-wise Adagrad, Zipf 1.1
//     3.7k / 9.5k        61.9 / 56.4 / 54.3      124 / 115 / 112
//    17.2k                200 / 194 / 192
constexpr int split_four(int el) { return el == 1 ? 5000 : 8192; }
constexpr int split_two(int el) { return el == 1 ? 16384 : 20480; }

template <typename TW, int EL, int OPT>
hipError_t launch_reduce_t(const RArgs& ra, hipStream_t s) {
  const int blocks = ra.split ? ra.nchunks : (ra.nchunks + 3) / 4;
  const int waves = ra.split == 1 ? 2 : 4;
  hipLaunchKernelGGL((k_reduce_wave<TW, EL, OPT>), dim3((unsigned)blocks), dim3((unsigned)(waves * kWave)), 0, s, ra);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_combine_wave<TW, EL, OPT>), dim3((unsigned)ra.ncomb), dim3(kCombineThreads), 0, s, ra);
  return hipGetLastError();
}

template <typename TW, int EL>
hipError_t launch_reduce_opt(const RArgs& ra, hipStream_t s) {
  if (!ra.up.fuse) return launch_reduce_t<TW, EL, kReduceOnly>(ra, s);
  switch (ra.up.opt) {
    case EMB_OPT_SGD: return launch_reduce_t<TW, EL, EMB_OPT_SGD>(ra, s);
    case EMB_OPT_ADAGRAD_ROWWISE: return launch_reduce_t<TW, EL, EMB_OPT_ADAGRAD_ROWWISE>(ra, s);
    default: return launch_reduce_t<TW, EL, EMB_OPT_ADAGRAD_ELEMENTWISE>(ra, s);
  }
}

template <typename TW>
hipError_t launch_reduce_dt(const RArgs& ra, hipStream_t s) {
  if (ra.D <= 64) return launch_reduce_opt<TW, 1>(ra, s);
  if (ra.D <= 128) return launch_reduce_opt<TW, 2>(ra, s);
  if (ra.D <= 256) return launch_reduce_opt<TW, 4>(ra, s);
  if (ra.D <= 512) return launch_reduce_opt<TW, 8>(ra, s);
  if (ra.D <= 1024) return launch_reduce_opt<TW, 16>(ra, s);
  return hipErrorInvalidValue;
}

template <typename TW, int EL>
hipError_t launch_update_t(const UArgs& ua, hipStream_t s) {
  int64_t want = ((int64_t)ua.max_unique + 4 * kUpdateRows - 1) / (4 * kUpdateRows);
  const dim3 grid((unsigned)(want > 4096 ? 4096 : want)), block(256);
  switch (ua.up.opt) {
    case EMB_OPT_SGD: hipLaunchKernelGGL((k_update_wave<TW, EL, EMB_OPT_SGD>), grid, block, 0, s, ua); break;
    case EMB_OPT_ADAGRAD_ROWWISE:
      hipLaunchKernelGGL((k_update_wave<TW, EL, EMB_OPT_ADAGRAD_ROWWISE>), grid, block, 0, s, ua);
      break;
    default: hipLaunchKernelGGL((k_update_wave<TW, EL, EMB_OPT_ADAGRAD_ELEMENTWISE>), grid, block, 0, s, ua);
  }
  return hipGetLastError();
}

template <typename TW>
hipError_t launch_update_dt(const UArgs& ua, hipStream_t s) {
  if (ua.up.D <= 64) return launch_update_t<TW, 1>(ua, s);
  if (ua.up.D <= 128) return launch_update_t<TW, 2>(ua, s);
  if (ua.up.D <= 256) return launch_update_t<TW, 4>(ua, s);
  if (ua.up.D <= 512) return launch_update_t<TW, 8>(ua, s);
  if (ua.up.D <= 1024) return launch_update_t<TW, 16>(ua, s);
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_reduce_wave(const RArgs& args, int dtype, hipStream_t s) {
  RArgs ra = args;
  const int el = ra.D <= 64 ? 1 : 2;
  ra.split = ra.nchunks <= split_four(el) ? 2 : (ra.nchunks <= split_two(el) ? 1 : 0);
  return dtype == EMB_FP32 ? launch_reduce_dt<float>(ra, s) : launch_reduce_dt<uint16_t>(ra, s);
}

hipError_t launch_update_wave(const UArgs& ua, int dtype, hipStream_t s) {
  return dtype == EMB_FP32 ? launch_update_dt<float>(ua, s) : launch_update_dt<uint16_t>(ua, s);
}

}  // namespace emb
