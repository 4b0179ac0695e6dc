// libsmfg consumer kernels: GraphSAGE mean aggregation over one MFG block, alone and fused into
// the layer's linear transform on the matrix cores.
#ifndef SMFG_KERNELS_AGGREGATE_H_
#define SMFG_KERNELS_AGGREGATE_H_

#include "device_common.h"

namespace smfg_dev {

// A group of 16 lanes walks the samples of SPAN consecutive destinations, which are one
// contiguous range of the block's indices array; a lane owns V consecutive columns per round of
// 16 * V columns.  kAggDepth source rows are requested before the first is used, whichever
// destination they belong to, so a short destination (fanout 5) does not limit the loads in
// flight; their ids come in one read of the group, an id per lane, those of the next ten while these are added (96 K
// destinations x 5 of 200 bytes 27.8 -> 27.2 us).  Each destination's rows are added in float, in slot order, then divided once.
// Offsets are clamped to [0, max_edges] and source ids outside [0, max_src) read row 0, so the
// arrays of a batch that ended with a status (contents unspecified) cannot cause a stray read.
constexpr int kAggLanes = 16;
constexpr int kAggSpan = 2;
constexpr int kAggDepth = 10;
constexpr int kAggGroups = kThreads / kAggLanes;
constexpr int kAggRows = kAggGroups * kAggSpan;  // destinations per block of k_mean_aggregate

// ALIGNED: the vectors of a row lie at multiples of their size.  Else they lie at any element (the target
// reads vectors from any address) and the last one of a row ends with it: it overlaps the one before,
// and both lanes compute and write the same means there.  Rows of 100 halfs in 13 vectors of 8 are one
// column round of the 16 lanes; in vectors of 4, the widest aligned ones, they were two, the second
// with 9 lanes in use (96 K destinations x 5: 36 -> 28 us; 203 halfs 142 -> 54, 33 floats 32 -> 16).
template <typename T, int V, bool ALIGNED>
struct alignas(ALIGNED ? sizeof(T) * V : sizeof(T)) RowVec {
  T v[V];
};

__device__ __forceinline__ float to_float(_Float16 h) { return static_cast<float>(h); }
__device__ __forceinline__ float to_float(float f) { return f; }

// Offset of a destination.  The array has max_dst + 1 of them, so they can be on their way together with the number of
// destinations; what lies past its end is not used.
__device__ __forceinline__ int load_offset(const int32_t* __restrict__ indptr, int64_t i, int64_t max_dst, int64_t max_edges) {
  const int o = indptr[i < max_dst ? i : max_dst];
  return o < 0 ? 0 : o > max_edges ? static_cast<int>(max_edges) : o;
}

// The boundaries of a group's destinations from its lanes (lane q <= SPAN that of destination q), never decreasing, those
// past its last destination the end of it.
template <int LANES, int SPAN>
__device__ __forceinline__ void group_offsets(int mine, int rows_here, int (&off)[SPAN + 1]) {
#pragma unroll
  for (int q = 0; q <= SPAN; ++q) {
    const int o = __shfl(mine, q, LANES);
    off[q] = q == 0 || (q <= rows_here && o > off[q - 1]) ? o : off[q - 1];
  }
}

// Source ids of the group's samples from e on, one per lane; the last one again past e_end.
__device__ __forceinline__ uint32_t load_id(const int32_t* __restrict__ indices, int e, int e_end, int lane) {
  return e < e_end ? static_cast<uint32_t>(indices[e + lane < e_end ? e + lane : e_end - 1]) : 0u;
}

// Means of the group's rows_here (<= SPAN) destinations, off[0 .. rows_here] their boundaries.  emit(r, c, mean) receives, once
// per destination r and column round, the V means of columns c .. c + V (zeros for an empty row).  All lanes of the
// group call, and stay together: they hold each other's ids.
template <typename T, int V, bool ALIGNED, int LANES, int DEPTH, int SPAN, typename Emit>
__device__ __forceinline__ void walk_group_means(const int (&off)[SPAN + 1], int rows_here, const int32_t* __restrict__ indices,
                                                 const T* __restrict__ x, uint32_t nsrc, int dim, int lane, Emit emit) {
  typedef RowVec<T, V, ALIGNED> Vec;
  static_assert(DEPTH <= LANES, "a lane per id");
  const int e_begin = off[0], e_end = off[SPAN];
  const uint32_t first = load_id(indices, e_begin, e_end, lane);
  for (int cb = 0; cb < dim; cb += LANES * V) {
    const int c0 = cb + lane * V;
    const int c = c0 + V <= dim ? c0 : dim - V;
    float acc[V];
#pragma unroll
    for (int t = 0; t < V; ++t) acc[t] = 0.f;
    int r = 0;               // destination being summed
    int r_begin = e_begin;   // its first sample
    int r_end = off[1];
    // closes destination r (mean or zeros) and moves to the next one
    auto close_row = [&]() {
      const float k = static_cast<float>(r_end - r_begin);
      float mean[V];
#pragma unroll
      for (int t = 0; t < V; ++t) {
        mean[t] = r_end > r_begin ? acc[t] / k : 0.f;
        acc[t] = 0.f;
      }
      if (c0 < dim) emit(r, c, mean);
      ++r;
      r_begin = r_end;
#pragma unroll
      for (int q = 2; q <= SPAN; ++q)
        if (q == r + 1) r_end = off[q];
    };
    uint32_t ids = first;
    for (int e = e_begin; e < e_end; e += DEPTH) {
      Vec rows[DEPTH];
      ids = ids < nsrc ? ids : 0u;
#pragma unroll
      for (int u = 0; u < DEPTH; ++u)
        rows[u] = *reinterpret_cast<const Vec*>(x + static_cast<int64_t>(static_cast<uint32_t>(__shfl(static_cast<int>(ids), u, LANES))) * dim + c);
      ids = load_id(indices, e + DEPTH, e_end, lane);
#pragma unroll
      for (int u = 0; u < DEPTH; ++u) {
        if (e + u < e_end) {
          while (e + u >= r_end && r < rows_here) close_row();
#pragma unroll
          for (int t = 0; t < V; ++t) acc[t] += to_float(rows[u].v[t]);
        }
      }
    }
    while (r < rows_here) close_row();
  }
}

template <typename T, int V, bool ALIGNED>
__global__ void __launch_bounds__(kThreads) k_mean_aggregate(const int32_t* __restrict__ indptr,
                                                             const int32_t* __restrict__ indices,
                                                             int64_t max_edges,
                                                             const int64_t* __restrict__ num_dst, int64_t max_dst,
                                                             const T* __restrict__ x, int64_t max_src, int dim,
                                                             float* __restrict__ out) {
  const int grp = threadIdx.x / kAggLanes, lane = threadIdx.x & (kAggLanes - 1);
  const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kAggRows + static_cast<int64_t>(grp) * kAggSpan;
  const int mine = load_offset(indptr, i0 + (lane < kAggSpan ? lane : kAggSpan), max_dst, max_edges);
  int64_t n = *num_dst;
  if (n > max_dst) n = max_dst;
  if (i0 >= n) return;
  const int rows_here = static_cast<int>(n - i0 < kAggSpan ? n - i0 : kAggSpan);
  int off[kAggSpan + 1];
  group_offsets<kAggLanes, kAggSpan>(mine, rows_here, off);
  walk_group_means<T, V, ALIGNED, kAggLanes, kAggDepth, kAggSpan>(off, rows_here, indices, x, static_cast<uint32_t>(max_src), dim, lane,
                                                                  [&](int r, int c, const float* mean) {
                                                                    float* o = out + (i0 + r) * dim + c;
#pragma unroll
                                                                    for (int t = 0; t < V; ++t) o[t] = mean[t];
                                                                  });
}

// ---- one GraphSAGE layer: out = act([x_dst | mean] W^T + b) -------------------------------------
//
// A persistent block takes tiles of consecutive destinations, one after the other.  A lane group of
// 8, 16 or 32 lanes fetches the rows of a destination's samples, a vector of 8 columns per lane; their mean,
// rounded to half, and the destination's own row (destination i is source i) make a row of the tile in LDS, which eight
// waves then multiply, each by its 32 columns of W^T, with v_mfma_f32_32x32x16_f16.  A wave keeps its part of W in
// registers for all tiles of the block: read for every tile of 64 rows it was 0.3 GB from the L2 for 154 K destinations of
// 128 -> 256, as much as the rows, and took half as long again.
//
// dim <= 128 (k_sage_layer): eight more waves do the fetching, two tiles ahead of the one that is being multiplied, so that
// rows are on their way all the time; what is left is the HBM's.  154 K destinations x 5, 128 -> 256, half: 80 -> 61 us, 4.8 TB/s of what
// the layer cannot do without (68 us while waits for a tile's rows were waits for the next one's as well); 96 K x 5 of 104 columns 51 -> 40, 47 K
// of 96 26 -> 19, 150 K x 10, 64 -> 128 63 -> 54.  With all waves doing both, a tile ahead, 78 us for the first.  Where a block has a tile or less, a
// chain of dependent reads remains: 12.5 K x 10, 128 -> 256 20 -> 12 us, 1 K x 15 19 -> 10.  Blocks of whole neighbourhoods, 128 -> 256: 12 K
// destinations with 5.1 M samples, 17 000 the most, 3.51 ms by k_sage_layer_cols, 3.67 with a range of destinations per block and 5 rows
// of a destination at a time, 2.63 with tiles dealt and 10; 11 K with 2.9 M, 50 000 the most, 6.6, 7.9 and 4.2.
// dim > 128 (k_sage_layer_wide): W takes 128 registers of a wave, which leaves room for eight waves in a compute unit, and all
// of them fetch, a tile ahead.  300 K x 5, 256 -> 256 283 -> 226 us, 60 K x 15 113 -> 107, 13 K x 10 24 -> 21.5, 1 K x 15 20 -> 10;
// with four waves that only fetch and eight that only multiply 244, 123, 22 and 15.
// Such a block takes a compute unit for itself, so beside another stream's gather it waits for one: a layer of an epoch's
// consumer can stand still for as long as the gather of the next set takes, which then is that much faster (16 batches
// with three layers each 3.60 -> 3.46 ms; with blocks of 256 threads that read W for every tile 3.52, for the second layer only 3.68).
constexpr int kLayerPad = 8;  // halfs of padding per LDS row
constexpr int kLayerMaxDim = 256;
constexpr int kLayerMaxCols = 256;  // of W in the registers of kLayerWaves waves
constexpr int kLayerWaves = 8;   // that multiply
constexpr int kLayerLoaders = 8;
constexpr int kLayerThreads = (kLayerWaves + kLayerLoaders) * 64, kLayerWideThreads = kLayerWaves * 64;
constexpr int kLayerWideRows = 32;
constexpr int kLayerBlocks = 256;   // one to a compute unit
constexpr int kLayerMinRows = 16;   // of a block
constexpr int layer_rows(int lanes) { return kLayerLoaders * 64 / lanes; }
constexpr int layer_lda(int dim) { return 2 * dim + kLayerPad; }
// a wave's results, 32 x 32 of them, on their way through the LDS to consecutive memory
template <typename OutT>
constexpr int layer_ldo() { return 32 + 16 / static_cast<int>(sizeof(OutT)); }
template <typename OutT>
constexpr size_t layer_lds_bytes(int rows, int dim) { return sizeof(_Float16) * 2 * rows * layer_lda(dim) + sizeof(OutT) * kLayerWaves * 32 * layer_ldo<OutT>(); }
static_assert(layer_lds_bytes<float>(layer_rows(8), 64) <= 160 * 1024 && layer_lds_bytes<float>(layer_rows(16), 128) <= 160 * 1024 &&
              layer_lds_bytes<float>(kLayerWideRows, kLayerMaxDim) <= 160 * 1024, "LDS of a compute unit");

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float4_t __attribute__((ext_vector_type(4)));
typedef float float16_t __attribute__((ext_vector_type(16)));

// Weights in the order the layer kernel's lanes consume them: for column slice sl (32 output
// columns), vector q (16 reduction indices) and lane (hi, col): the 8 halfs
// w[32 sl + col][16 q + 8 hi .. + 8), zeros for columns past out_dim.
__global__ void __launch_bounds__(kThreads) k_sage_pack_weights(const _Float16* __restrict__ w, int K, int out_dim,
                                                                half8_t* __restrict__ packed, int64_t vectors) {
  const int nq = K / 16;
  for (int64_t v = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; v < vectors;
       v += static_cast<int64_t>(gridDim.x) * kThreads) {
    const int l = static_cast<int>(v & 63);
    const int64_t sq = v >> 6;
    const int q = static_cast<int>(sq % nq);
    const int sl = static_cast<int>(sq / nq);
    const int row = sl * 32 + (l & 31);
    half8_t o = {0, 0, 0, 0, 0, 0, 0, 0};
    if (row < out_dim) o = *reinterpret_cast<const half8_t*>(w + static_cast<int64_t>(row) * K + q * 16 + (l >> 5) * 8);
    packed[v] = o;
  }
}

struct LayerArgs {
  const int32_t* indptr;
  const int32_t* indices;
  int64_t max_edges;
  const int64_t* num_dst;
  int64_t max_dst;
  const _Float16* x;
  int64_t max_src;
  int dim;
  const _Float16* w;
  const float* bias;
  int out_dim, relu;
  void* out;
};

__device__ __forceinline__ int64_t layer_rows_in_all(const LayerArgs& P) {
  int64_t n = *P.num_dst;
  if (n > P.max_dst) n = P.max_dst;
  if (n > P.max_src) n = P.max_src;  // a destination's own row is row i of x
  if (n < 0) n = 0;
  return n;
}
// An even share of consecutive destinations, so that no block has a tile more than the others to do.
__device__ __forceinline__ void layer_range(const LayerArgs& P, int& b0, int& b1) {
  const int64_t n = layer_rows_in_all(P);
  b0 = static_cast<int>(n * blockIdx.x / gridDim.x);
  b1 = static_cast<int>(n * (blockIdx.x + 1) / gridDim.x);
}
// A block's tiles of at most MOST destinations: an even share in one piece where that is two of them at most, else dealt to the blocks in
// turn, as many in each.  In blocks of whole neighbourhoods the destinations with the most samples are neighbours of each other; one range per
// block left them all to a few.  In one piece the second tile is the shorter one, and with it the last product, which nothing hides (12 K x 7, 128 -> 256
// 9.3 us; 10.1 with two even tiles); over more turns the even share is ahead (50 K x 20, 64 -> 128 23.1 us; 24.9 with full tiles).
template <int MOST>
struct LayerTiles {
  uint32_t n, rows, first, step, end;  // destinations in all and of a tile; first one of the block's first tile, from there to the next tile's, end
  __device__ __forceinline__ explicit LayerTiles(const LayerArgs& P) : n(static_cast<uint32_t>(layer_rows_in_all(P))) {
    const uint32_t share = (n + gridDim.x - 1u) / gridDim.x;
    if (share <= 2u * MOST) {
      rows = step = MOST;
      first = blockIdx.x * share;
      end = first + share < n ? first + share : n;
    } else {
      const uint32_t turns = (share + MOST - 1u) / MOST;
      rows = (share + turns - 1u) / turns;
      step = gridDim.x * rows;
      first = blockIdx.x * rows;
      end = n;
    }
  }
  __device__ __forceinline__ uint32_t count(uint32_t i0) const { return i0 >= end ? 0u : end - i0 < rows ? end - i0 : rows; }
};

// What a lane reads: vectors of 8 columns of rows of x; lanes past the last column read it once more.
struct LayerColumns {
  const char* at;
  uint32_t row_bytes, nsrc;
  bool own;  // the lane has columns
  __device__ __forceinline__ LayerColumns(const LayerArgs& P, int lane)
      : at(reinterpret_cast<const char*>(P.x) + (lane * 8 < P.dim ? lane * 8 : P.dim - 8) * sizeof(_Float16)),
        row_bytes(static_cast<uint32_t>(P.dim) * sizeof(_Float16)), nsrc(static_cast<uint32_t>(P.max_src)), own(lane * 8 < P.dim) {}
  __device__ __forceinline__ half8_t row(uint32_t i) const {
    return *reinterpret_cast<const half8_t*>(at + static_cast<uint64_t>(i) * row_bytes);
  }
  // the rows that DEPTH lanes of the group name, from the first-th on
  template <int LANES, int DEPTH>
  __device__ __forceinline__ void rows(uint32_t ids, half8_t (&v)[DEPTH], int first = 0) const {
    ids = ids < nsrc ? ids : 0u;
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) v[u] = row(static_cast<uint32_t>(__shfl(static_cast<int>(ids), first + u, LANES)));
  }
};

__device__ __forceinline__ void layer_add(float (&acc)[8], const half8_t v) {
#pragma unroll
  for (int t = 0; t < 8; ++t) acc[t] += to_float(v[t]);
}
// Sums / k, zeros if k is 0.  The quotient, rounded once, is that of the sum and the rounded reciprocal, corrected by its remainder
// (Markstein): for k < 2^20 what a division gives, in 4 instructions instead of 10 (2 of the 80 us above).
__device__ __forceinline__ half8_t layer_mean(const float (&acc)[8], int samples) {
  const float k = static_cast<float>(samples > 0 ? samples : 1), inv = 1.f / k;
  half8_t h;
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const float q = acc[t] * inv;
    h[t] = static_cast<_Float16>(__builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-q, k, acc[t]), inv, q), k, acc[t]));
  }
  return h;
}

// A wave's part of the multiplication: a slice of 32 columns, in tiles of 64 destinations of every other 32 where there are as many waves as
// that takes.
template <typename OutT, int STEPS, int ROWS>  // steps of 16 reduction indices and destinations of a tile, at most
struct LayerProduct {
  const LayerArgs& P;
  const int parts, part, slice, lane, col, hi, nq, lda;
  const bool vectors;
  OutT* const res;  // [32][layer_ldo], the wave's own
  half8_t w[STEPS];

  __device__ __forceinline__ half8_t weights(int q) const {
    return reinterpret_cast<const half8_t*>(P.w)[(static_cast<int64_t>(slice) * nq + (q < nq ? q : 0)) * 64 + lane];
  }
  __device__ __forceinline__ LayerProduct(const LayerArgs& p, int wv, OutT* all_res)
      : P(p), parts(ROWS == 32 || p.out_dim > 128 ? 1 : 2), part(ROWS == 32 ? 0 : wv * parts / kLayerWaves), slice(ROWS == 32 ? wv : wv - part * (kLayerWaves / parts)),
        lane(threadIdx.x & 63), col(lane & 31), hi(lane >> 5), nq(p.dim / 8), lda(layer_lda(p.dim)),
        vectors(p.out_dim % (16 / static_cast<int>(sizeof(OutT))) == 0 && reinterpret_cast<uintptr_t>(p.out) % 16 == 0),
        res(all_res + wv * 32 * layer_ldo<OutT>()) {
    if (slice * 32 < P.out_dim) {
#pragma unroll
      for (int q = 0; q < STEPS; ++q) w[q] = weights(q);
    }
  }
  // destinations tile0 .. tile0 + here, their inputs in a
  __device__ __forceinline__ void tile(const _Float16* a, int tile0, int here) const {
    constexpr int kVec = 16 / static_cast<int>(sizeof(OutT)), kRowLanes = 32 / kVec, ldo = layer_ldo<OutT>();
    if (slice * 32 >= P.out_dim) return;
    const int j = slice * 32 + col;
    const float bias = P.bias && j < P.out_dim ? P.bias[j] : 0.f;
    for (int rb = 32 * part; rb < here; rb += 32 * parts) {
      const _Float16* ap = a + (rb + col) * lda + hi * 8;
      float16_t acc;
#pragma unroll
      for (int t = 0; t < 16; ++t) acc[t] = 0.f;
      // lane half hi supplies reduction indices 16 q + 8 hi .. + 8 of both operands (any assignment works as
      // long as it is the same on both sides); rows past the tile's last only reach results that are not stored
      const auto step = [&](int q, const half8_t b) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(*reinterpret_cast<const half8_t*>(ap + q * 16), b, acc, 0, 0, 0);
      };
#pragma unroll
      for (int q = 0; q < STEPS; ++q)
        if (q < nq) step(q, w[q]);
      // element t of a lane's accumulator: row 8 (t / 4) + 4 hi + t % 4, column col
      OutT* o = res + 4 * hi * ldo + col;
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        float v = acc[t] + bias;
        if (P.relu) v = v > 0.f ? v : 0.f;
        o[(8 * (t / 4) + t % 4) * ldo] = static_cast<OutT>(v);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      OutT* to = static_cast<OutT*>(P.out) + static_cast<int64_t>(tile0 + rb) * P.out_dim + slice * 32;
      const int rows = here - rb < 32 ? here - rb : 32, cols = P.out_dim - slice * 32 < 32 ? P.out_dim - slice * 32 : 32;
      if (vectors) {
        const int c = lane % kRowLanes * kVec;
#pragma unroll
        for (int r0 = 0; r0 < 32; r0 += 64 / kRowLanes) {
          const int r = r0 + lane / kRowLanes;
          if (r < rows && c < cols) *reinterpret_cast<float4_t*>(to + static_cast<int64_t>(r) * P.out_dim + c) = *reinterpret_cast<const float4_t*>(res + r * ldo + c);
        }
      } else if (col < cols) {
        // as many reads of the LDS at a time, while W leaves the registers for it: 50 K x 3, 64 -> 47, float 16.6 -> 11.7 us
        constexpr int kRead = STEPS <= 16 ? 8 : 1;
        if constexpr (kRead == 1) {
          for (int r = hi; r < rows; r += 2) to[static_cast<int64_t>(r) * P.out_dim + col] = res[r * ldo + col];
        } else {
          OutT* at = to + static_cast<int64_t>(hi) * P.out_dim + col;
#pragma unroll 1
          for (int r = hi; r < rows; r += 2 * kRead) {
            OutT v[kRead];
#pragma unroll
            for (int u = 0; u < kRead; ++u) v[u] = res[(r + 2 * u) * ldo + col];
#pragma unroll
            for (int u = 0; u < kRead; ++u, at += 2 * P.out_dim)
              if (r + 2 * u < rows) *at = v[u];
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
};

// dim <= 8 * LANES <= 128.  A lane group of the fetching waves has a destination per tile; the rows of two tiles, the ids of
// a third and the offsets of a fourth are on their way.  Of a destination with more than kDepth samples the first kDepth are
// fetched ahead (8 of them: 1 % more for a fanout of 5, 2 % less for 64), the others while those before them are added, up to 2 kDepth at a time.
template <typename OutT, int LANES>
__global__ void __launch_bounds__(kLayerThreads) k_sage_layer(const LayerArgs P) {
  constexpr int ROWS = layer_rows(LANES), kDepth = 5, kAhead = 2;
  constexpr bool kHeld = LANES >= 2 * kDepth;  // a group's lanes hold the ids of the second kDepth samples, too
  static_assert(ROWS == 32 || ROWS == 64, "one or two accumulators");
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int lda = layer_lda(P.dim);
  _Float16* buf = reinterpret_cast<_Float16*>(lds_raw);  // [2][ROWS][lda]
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const LayerTiles<ROWS> T(P);
  if (T.first >= T.end) return;
  const bool one = T.end - T.first <= T.step;  // tile: with code of its own, since in a small call every line of code has to be fetched
  if (wv < kLayerLoaders) {
    const uint32_t grp = threadIdx.x / LANES;
    const int lane = threadIdx.x & (LANES - 1);
    const LayerColumns x(P, lane);
    struct Ahead {
      half8_t rows[kDepth], own;
      uint32_t ids, more;  // of the samples from begin on, as many as the group has lanes; unless kHeld, of those behind the first kDepth
      int begin, end;
    } s[kAhead];
    int begin, end, next_begin, next_end;
    uint32_t id, id_more = 0;
    // the group's destination of the tile whose offsets are read next; past the end where a tile has none for it, and then the last one of
    // all without samples stands in
    uint32_t i = grp < T.rows ? T.first + grp : T.end;
    const auto read_offsets = [&]() {
      const uint32_t at = i < T.end ? i : T.n - 1u;
      next_begin = load_offset(P.indptr, at, P.max_dst, P.max_edges);
      next_end = load_offset(P.indptr, at + (i < T.end ? 1u : 0u), P.max_dst, P.max_edges);
      i += T.step;
    };
    const auto read_ids = [&]() {
      begin = next_begin;
      end = next_end > begin ? next_end : begin;
      id = load_id(P.indices, begin, end, lane);
      if (!kHeld) id_more = load_id(P.indices, begin < end - kDepth ? begin + kDepth : end, end, lane);
    };
    // rows of a tile; ids and offsets of those behind it first, since waiting for them must not be waiting for the rows
    const auto issue = [&](Ahead& t) {
      const uint32_t at = i - 2u * T.step;
      t.ids = id;
      t.more = id_more;
      t.begin = begin;
      t.end = end;
      read_ids();
      read_offsets();
      x.rows<LANES>(t.ids, t.rows);
      t.own = x.row(at < T.end ? at : T.n - 1u);
    };
    const auto finish = [&](Ahead& t, _Float16* a) {
      float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      const int samples = t.end - t.begin;
      const auto add = [&](const half8_t (&v)[kDepth], int count) {
#pragma unroll
        for (int u = 0; u < kDepth; ++u)
          if (u < count) layer_add(acc, v[u]);
      };
      add(t.rows, samples);
      if (samples > kDepth) {
        const uint32_t last = static_cast<uint32_t>(t.end) - 1u;
        uint32_t at = static_cast<uint32_t>(t.begin + lane);
        const auto ids_at = [&](int ahead) {  // past the end that of the last sample
          const uint32_t e = at + static_cast<uint32_t>(ahead);
          return static_cast<uint32_t>(P.indices[e < last ? e : last]);
        };
        half8_t (&here)[kDepth] = t.rows, next[kDepth];
        int left = samples - kDepth;
        uint32_t id0 = ids_at(2 * kDepth), id1 = ids_at(3 * kDepth);
        if constexpr (kHeld) x.rows<LANES>(t.ids, here, kDepth);
        else x.rows<LANES>(t.more, here);
        if (left > kDepth) {
          x.rows<LANES>(id0, next);
          id0 = ids_at(4 * kDepth);
          while (left > 2 * kDepth) {
            add(here, kDepth);
            x.rows<LANES>(id1, here);
            id1 = ids_at(5 * kDepth);
            add(next, kDepth);
            x.rows<LANES>(id0, next);
            id0 = ids_at(6 * kDepth);
            at += 2 * kDepth;
            left -= 2 * kDepth;
          }
        }
        add(here, left);
        add(next, left - kDepth);
        // Nothing under way where the ways meet again, or the waits behind would be for the next tile's rows as well.
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
      }
      const half8_t mean = layer_mean(acc, samples);
      if (x.own) {
        *reinterpret_cast<half8_t*>(a + grp * lda + lane * 8) = t.own;
        *reinterpret_cast<half8_t*>(a + grp * lda + P.dim + lane * 8) = mean;
      }
    };
    read_offsets();
    read_ids();
    read_offsets();
    static_assert(kAhead == 2, "the halves of buf");
    issue(s[0]);
    if (one) {
      finish(s[0], buf);
      __syncthreads();
      __syncthreads();
      return;
    }
    issue(s[1]);
    // Two tiles a turn, the last of an odd number with one of no destinations: a way past the second to the next turn would make every
    // wait for rows one for the tile's behind them.
    for (uint32_t i0 = T.first; i0 < T.end; i0 += 2u * T.step) {
      finish(s[0], buf);
      issue(s[0]);
      __syncthreads();
      finish(s[1], buf + ROWS * lda);
      issue(s[1]);
      __syncthreads();
    }
    __syncthreads();
    return;
  }
  const LayerProduct<OutT, LANES, ROWS> product(P, wv - kLayerLoaders, reinterpret_cast<OutT*>(buf + 2 * ROWS * lda));
  __syncthreads();
  for (uint32_t i0 = T.first; i0 < T.end; i0 += 2u * T.step) {
    product.tile(buf, static_cast<int>(i0), static_cast<int>(T.count(i0)));
    __syncthreads();
    if (one) return;
    product.tile(buf + ROWS * lda, static_cast<int>(i0 + T.step), static_cast<int>(T.count(i0 + T.step)));
    __syncthreads();
  }
}

// 128 < dim <= 256.  A lane group has up to kSpan consecutive destinations per tile, fewer where the block has few; the first rows of
// the next tile are on their way while the present one is multiplied.
template <typename OutT>
__global__ void __launch_bounds__(kLayerWideThreads, 2) k_sage_layer_wide(const LayerArgs P) {
  constexpr int LANES = 32, kGroups = kLayerWideThreads / LANES, kSpan = kLayerWideRows / kGroups, kDepth = 10;
  extern __shared__ __align__(16) unsigned char lds_raw[];
  const int lda = layer_lda(P.dim);
  _Float16* buf = reinterpret_cast<_Float16*>(lds_raw);  // [2][kLayerWideRows][lda]
  const LayerProduct<OutT, LANES, kLayerWideRows> product(P, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), reinterpret_cast<OutT*>(buf + 2 * kLayerWideRows * lda));
  int b0, b1;
  layer_range(P, b0, b1);
  if (b0 == b1) return;
  const int want = (b1 - b0 + kGroups - 1) / kGroups, per = want < kSpan ? want : kSpan, rows_tile = kGroups * per;
  const int grp = threadIdx.x / LANES, lane = threadIdx.x & (LANES - 1);
  const LayerColumns x(P, lane);
  const uint32_t past = static_cast<uint32_t>(b1);
  const auto rows_of = [&](uint32_t i0) { return i0 < past ? (past - i0 < static_cast<uint32_t>(per) ? static_cast<int>(past - i0) : per) : 0; };
  const auto offset_of = [&](uint32_t i0) { return load_offset(P.indptr, static_cast<int64_t>(i0) + (lane < kSpan ? lane : kSpan), P.max_dst, P.max_edges); };
  half8_t rows[kDepth], own[kSpan];
  const auto read_own = [&](uint32_t i0) {
#pragma unroll
    for (uint32_t r = 0; r < kSpan; ++r) own[r] = x.row(i0 + r < past ? i0 + r : past - 1u);
  };
  uint32_t i0 = static_cast<uint32_t>(b0 + grp * per);
  int off[kSpan + 1], mine = offset_of(i0);
  group_offsets<LANES, kSpan>(mine, rows_of(i0), off);
  uint32_t id = load_id(P.indices, off[0], off[kSpan], lane);
  mine = offset_of(i0 + static_cast<uint32_t>(rows_tile));
  x.rows<LANES>(id, rows);
  read_own(i0);
  _Float16* a = buf;
  for (int tile0 = b0; tile0 < b1; tile0 += rows_tile) {
    int next[kSpan + 1];
    group_offsets<LANES, kSpan>(mine, rows_of(i0 + static_cast<uint32_t>(rows_tile)), next);
    id = load_id(P.indices, next[0], next[kSpan], lane);
    mine = offset_of(i0 + 2u * static_cast<uint32_t>(rows_tile));
    const int rows_here = rows_of(i0), e_end = off[kSpan];
    _Float16* ag = a + grp * per * lda + lane * 8;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    int r = 0, r_begin = off[0], r_end = off[1];
    const auto close_row = [&]() {
      const half8_t mean = layer_mean(acc, r_end - r_begin);
      if (x.own) *reinterpret_cast<half8_t*>(ag + r * lda + P.dim) = mean;
#pragma unroll
      for (int t = 0; t < 8; ++t) acc[t] = 0.f;
      ++r;
      r_begin = r_end;
#pragma unroll
      for (int q = 2; q <= kSpan; ++q)
        if (q == r + 1) r_end = off[q];
    };
    uint32_t ids = load_id(P.indices, off[0] + kDepth, e_end, lane);
    for (int e = off[0]; e < e_end; e += kDepth) {
#pragma unroll
      for (int u = 0; u < kDepth; ++u) {
        if (e + u < e_end) {
          while (e + u >= r_end && r < rows_here) close_row();
          layer_add(acc, rows[u]);
        }
      }
      if (e + kDepth < e_end) {
        x.rows<LANES>(ids, rows);
        ids = load_id(P.indices, e + 2 * kDepth, e_end, lane);
      }
    }
    while (r < rows_here) close_row();
#pragma unroll
    for (int q = 0; q < kSpan; ++q)
      if (x.own && q < rows_here) *reinterpret_cast<half8_t*>(ag + q * lda) = own[q];
#pragma unroll
    for (int q = 0; q <= kSpan; ++q) off[q] = next[q];
    i0 += static_cast<uint32_t>(rows_tile);
    if (tile0 + rows_tile < b1) {
      x.rows<LANES>(id, rows);
      read_own(i0);
    }
    // the other half of buf is written next, by waves that may be a tile ahead of those still multiplying this one
    __syncthreads();
    product.tile(a, tile0, b1 - tile0 < rows_tile ? b1 - tile0 : rows_tile);
    a = a == buf ? buf + kLayerWideRows * lda : buf;
  }
}

// More than kLayerMaxCols output columns, where W does not fit the registers of a block, and more than 128 columns in with a small W
// (layer_reads_w): every tile reads W from the L2.  A block of four waves builds the inputs of ROWS destinations and multiplies them, a wave the column slices 4 apart.  100 K destinations x 5, 200 -> 300, half: 102 us
// (150 by k_sage_layer_wide with the columns from 256 on read for every tile); 64 -> 300 47 us (63 by k_sage_layer).
constexpr int layer_cols_rows(int dim) { return dim <= 128 ? 64 : 32; }  // at most 34 KB of LDS, four blocks to a compute unit
constexpr int kLayerColsAhead = 8;  // vectors of W requested ahead of their use
template <typename OutT, int ROWS>
__global__ void __launch_bounds__(kThreads, 4) k_sage_layer_cols(const LayerArgs P) {
  static_assert(ROWS == 32 || ROWS == 64, "one or two 32-row accumulators");
  constexpr int kLayerRows = ROWS;
  constexpr int kLayerSpan = ROWS / kAggGroups;  // destinations per lane group
  extern __shared__ __align__(16) unsigned char lds_raw[];
  _Float16* a_lds = reinterpret_cast<_Float16*>(lds_raw);  // [ROWS][2 dim + kLayerPad]
  const _Float16* x = P.x;
  const int dim = P.dim, out_dim = P.out_dim;
  OutT* out = static_cast<OutT*>(P.out);
  int64_t n = *P.num_dst;
  if (n > P.max_dst) n = P.max_dst;
  if (n > P.max_src) n = P.max_src;  // a destination's own row is row i of x
  const int64_t tile0 = static_cast<int64_t>(blockIdx.x) * kLayerRows;
  if (tile0 >= n) return;
  const int rows_tile = static_cast<int>(n - tile0 < kLayerRows ? n - tile0 : kLayerRows);
  const int K = 2 * dim;
  const int lda = K + kLayerPad;
  const int grp = threadIdx.x / kAggLanes, lane = threadIdx.x & (kAggLanes - 1);
  const int64_t i0 = tile0 + static_cast<int64_t>(grp) * kLayerSpan;
  const int mine = load_offset(P.indptr, i0 + (lane < kLayerSpan ? lane : kLayerSpan), P.max_dst, P.max_edges);

  // own rows -> columns [0, dim); rows past the end of the block become zeros (both halves)
  {
    const int vec_per_row = dim / 8;
    const half8_t zero = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int idx = threadIdx.x; idx < kLayerRows * vec_per_row; idx += kThreads) {
      const int r = idx / vec_per_row, cv = idx - r * vec_per_row;
      half8_t v = zero;
      if (r < rows_tile) v = *reinterpret_cast<const half8_t*>(x + (tile0 + r) * dim + cv * 8);
      *reinterpret_cast<half8_t*>(a_lds + r * lda + cv * 8) = v;
      if (r >= rows_tile) *reinterpret_cast<half8_t*>(a_lds + r * lda + dim + cv * 8) = zero;
    }
  }
  __syncthreads();
  if (i0 < n) {
    const int rows_here = static_cast<int>(n - i0 < kLayerSpan ? n - i0 : kLayerSpan);
    int off[kLayerSpan + 1];
    group_offsets<kAggLanes, kLayerSpan>(mine, rows_here, off);
    _Float16* a_grp = a_lds + (grp * kLayerSpan) * lda + dim;
    walk_group_means<_Float16, 8, true, kAggLanes, kAggDepth, kLayerSpan>(off, rows_here, P.indices, x, static_cast<uint32_t>(P.max_src), dim, lane,
                                                                          [&](int r, int c, const float* mean) {
                                                                            half8_t h;
#pragma unroll
                                                                            for (int t = 0; t < 8; ++t) h[t] = static_cast<_Float16>(mean[t]);
                                                                            *reinterpret_cast<half8_t*>(a_grp + r * lda + c) = h;
                                                                          });
  }
  __syncthreads();

  // tile [ROWS x K] times W^T: wave wv takes the column slices wv, wv + 4, ...  The packed
  // weights hold, for every slice and every 16 reduction indices, the 64 lanes' operands side by
  // side, so one load instruction of the wave reads 1 KB of consecutive memory (W stays in the L2);
  // kLayerColsAhead such vectors are always on their way.
  const int wv = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int col = l & 31, hi = l >> 5;
  const int nq = K / 16;
  for (int n0 = wv * 32; n0 < out_dim; n0 += 4 * 32) {
    const half8_t* wp = reinterpret_cast<const half8_t*>(P.w) + static_cast<int64_t>(n0 / 32) * nq * 64 + l;
    const _Float16* ap0 = a_lds + col * lda + hi * 8;
    const _Float16* ap1 = ap0 + 32 * lda;
    float16_t acc0, acc1;
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      acc0[t] = 0.f;
      acc1[t] = 0.f;
    }
    half8_t bq[kLayerColsAhead];
#pragma unroll
    for (int u = 0; u < kLayerColsAhead; ++u) bq[u] = wp[(u < nq ? u : 0) * 64];
    // one v_mfma_f32_32x32x16_f16 per vector: lane half hi supplies reduction indices 16 q + 8 hi .. + 8
    // of both operands (any assignment works as long as it is the same on both sides)
    // The body is free of branches (a vector past the end multiplies zeros), so the LDS reads of
    // the unrolled steps can be issued ahead of the MFMAs that use them.
    for (int qb = 0; qb < nq; qb += kLayerColsAhead) {
#pragma unroll
      for (int u = 0; u < kLayerColsAhead; ++u) {
        const int q = qb + u;
        const half8_t zero = {0, 0, 0, 0, 0, 0, 0, 0};
        const half8_t b = q < nq ? bq[u] : zero;
        const int qn = q + kLayerColsAhead;
        bq[u] = wp[(qn < nq ? qn : 0) * 64];
        const int k0 = (q < nq ? q : 0) * 16;
        const half8_t a0 = *reinterpret_cast<const half8_t*>(ap0 + k0);
        acc0 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0, b, acc0, 0, 0, 0);
        if constexpr (ROWS == 64) {
          const half8_t a1 = *reinterpret_cast<const half8_t*>(ap1 + k0);
          acc1 = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1, b, acc1, 0, 0, 0);
        }
      }
    }
    // element t of a lane's accumulator: row 8 (t / 4) + 4 hi + t % 4, column col.  The row term
    // that depends on t is the same for all lanes, so a store is one lane pointer plus a uniform
    // offset.
    if (n0 + col < out_dim) {
      const float bj = P.bias ? P.bias[n0 + col] : 0.f;
      OutT* o0 = out + (tile0 + 4 * hi) * out_dim + n0 + col;
      const int rows_left = rows_tile - 4 * hi;  // rows of the tile at or after the lane's first
      OutT r0[16], r1[16];
#pragma unroll
      for (int t = 0; t < 16; ++t) {
        float v0 = acc0[t] + bj, v1 = acc1[t] + bj;
        if (P.relu) {
          v0 = v0 > 0.f ? v0 : 0.f;
          v1 = v1 > 0.f ? v1 : 0.f;
        }
        r0[t] = static_cast<OutT>(v0);
        r1[t] = static_cast<OutT>(v1);
      }
      if (rows_tile == ROWS) {  // full tile: all stores in one go, nothing to test
#pragma unroll
        for (int t = 0; t < 16; ++t) {
          const int rt = 8 * (t / 4) + (t % 4);
          o0[static_cast<int64_t>(rt) * out_dim] = r0[t];
          if (ROWS == 64) o0[static_cast<int64_t>(rt + 32) * out_dim] = r1[t];
        }
      } else {
#pragma unroll
        for (int t = 0; t < 16; ++t) {
          const int rt = 8 * (t / 4) + (t % 4);
          if (rt < rows_left) o0[static_cast<int64_t>(rt) * out_dim] = r0[t];
          if (ROWS == 64 && rt + 32 < rows_left) o0[static_cast<int64_t>(rt + 32) * out_dim] = r1[t];
        }
      }
    }
  }
}

}  // namespace smfg_dev

#endif  // SMFG_KERNELS_AGGREGATE_H_
