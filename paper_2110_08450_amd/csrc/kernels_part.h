// libsmfg partition strategy for the dedup of a hop (fanouts up to SMFG_MAX_FANOUT).
//
// Procedure OneHopMFG keeps one map from global to local ids and gives a node its local id at the
// first encounter.  Here the map never exists as one structure in memory.  Per hop:
//   sample_part   a block of destinations draws its neighbours into gsrc and sorts its records by hash bucket
//                 in LDS; a record is (node, value): one per known node (value = its local id) and one per
//                 sample (value = tag | scan position).  The sorted records, a segment, and where each
//                 bucket begins within it go to memory side by side with the other blocks';
//   split_buckets only for hops with more records than 2^kPartMaxLgB buckets of the target size hold (such
//                 a hop starts with fewer, larger buckets, see part_levels): one block per bucket
//                 collects the bucket's records from all segments and orders them by further hash bits into
//                 sub-buckets (`rec2`), which then take the place of the buckets;
//   dedup_buckets one block per bucket collects the bucket's records from all segments and builds a hash table
//                 of its nodes in LDS, keeping
//                 the smallest value per node (a known node's local id always wins, else the
//                 earliest scan position).  A sample that is its node's first appearance keeps
//                 its gsrc entry (the node id, bit 31 clear); every other sample's entry is
//                 overwritten with kResolved | final local id (known node) or kPointer | position
//                 of the first appearance.  In the outer hops most samples are first appearances,
//                 so few entries are rewritten.
// flag_rows_part / assemble_part then number the first appearances in scan order (with scan_tiles between
// them in hops of more than kAssembleTiles tiles), exactly the ids the serial first-encounter rule gives.  Which thread inserts first never
// matters: only minima are kept.  All global traffic but the neighbour reads and those scattered
// 4-byte rewrites is streaming, and there are no global atomics.
#ifndef SMFG_KERNELS_PART_H_
#define SMFG_KERNELS_PART_H_

#include <type_traits>

#include "device_common.h"
#include "kernels_fast.h"

namespace smfg_dev {

constexpr int kPartMaxLgB = 11;                     // at most 2048 buckets per hop ...
constexpr int kPartMaxLg2 = 10;                     // ... each split into at most 1024 sub-buckets
constexpr int kPartTableLg = 11;                    // LDS table: 2048 slots
constexpr int kPartBucketRecords = 1024;            // buckets are sized for at most this many on average ...
constexpr int kPartFewRecords = 256;                // ... in hops that leave the chip idle for half or a quarter of it,
constexpr int kPartBuckets = 512;                   // as long as a launch has fewer buckets than this
constexpr int kPartMostRecords = 1228;              // before a second level begins
constexpr int64_t kPartOneLevel = int64_t(kPartMostRecords + 1) << kPartMaxLgB;  // one level of buckets holds fewer
constexpr int64_t kPartMaxRecords = static_cast<int64_t>(kPartBucketRecords) << (kPartMaxLgB + kPartMaxLg2);
constexpr uint32_t kPartHash = 0x9E3779B1u;         // odd: node -> node * kPartHash is a bijection on 32 bits
constexpr uint32_t kResolved = 0x80000000u;         // gsrc entry: low 30 bits = final local id of a known node
constexpr uint32_t kPointer = 0xC0000000u;          // gsrc entry: low 30 bits = position of the first appearance

__device__ __forceinline__ uint32_t part_bucket(uint32_t node, int lgB) {
  return lgB == 0 ? 0u : (node * kPartHash) >> (32 - lgB);
}

// Buckets (2^lgB) and sub-buckets per bucket (2^lg2) of the current hop, settled on the device: the host's figures
// come from the most destinations and samples a hop can have and only bound them (whole neighbourhoods: far
// less than all edges of the graph).  Grids are sized for the bound and surplus blocks leave.
// A block of k_dedup_buckets takes about as long for a bucket of 256 records as for one of 1024, some 7 us of dependent
// reads and barriers, so a hop has as few buckets as fill the chip, and as large ones as the registers of a
// block hold: 1.0 M records in each of eight batches 69 us with buckets of 1000, 77 with 500; 410 K records in
// four batches 7 us with 512 buckets, 14 with 64.  One level ends where the parts of a bucket become so short, two
// records of a segment of 4096, that beside another set's gather every one of them is a line from memory: 5.6 M
// records per batch, pipelined, 326 us per batch with two levels and 400 with 4096 buckets (alone 113 and 124 us); for 2.4 M
// it is 180 us with 2048 buckets and 177 with two levels, alone 115 and 168 per set of four.
struct HopShape {
  int lgB, lg2;
};
// 2^lg buckets in all: one level up to 2^kPartMaxLgB of them; beyond that two levels, the first of
// 2^kPartSplitLgB buckets (more if the second would exceed 2^kPartMaxLg2), of which a segment of 4096 records
// has a part of 16, a line of 128 bytes, to be read by k_split_buckets.
constexpr int kPartSplitLgB = 8;
__host__ __device__ inline void part_levels(int lg, int& lgB, int& lg2) {
  if (lg <= kPartMaxLgB) {
    lgB = lg;
    lg2 = 0;
    return;
  }
  lgB = lg - kPartMaxLg2 > kPartSplitLgB ? lg - kPartMaxLg2 : kPartSplitLgB;
  lg2 = lg - lgB;
}
// log2 of the buckets for that many records of a batch, `most` at most.
__host__ __device__ inline int part_buckets_lg(long long records, int batches, int most) {
  int lg = 0;
  while (lg < most && ((records >> lg) > (lg < kPartMaxLgB ? kPartBucketRecords : kPartMostRecords) || ((records >> lg) > kPartFewRecords && (batches << lg) < kPartBuckets))) ++lg;
  return lg;
}
// The shape for that many records of a batch: 2^lg buckets at most in all, and in one level 2^one_level, what the batch's
// workspace has offsets for.
__host__ __device__ inline HopShape hop_levels(long long records, int batches, int lg, int one_level) {
  HopShape s;
  part_levels(part_buckets_lg(records, batches, lg), s.lgB, s.lg2);
  if (s.lg2 == 0 && s.lgB > one_level) s.lgB = one_level;
  return s;
}
// Records: known nodes and sample positions, or samples where their number is known (P.flat); both are
// final before the first kernel that asks.
__device__ __forceinline__ HopShape hop_shape(const Launch& P, const BatchCtx& B, long long n) {
  return hop_levels(P.flat ? n + B.counts[P.L + 1 + P.h] : n * (1 + P.d), P.G, P.lg, B.one_level);
}

// ---- segments ------------------------------------------------------------------------------------
// The records of one block sorted by bucket: segment g is rec[g * cap ..), bucket b's part of it
// [offs[b], offs[b + 1]) of its row of `hist`, offsets within the segment.  A bucket is the union of its parts
// of all segments.  So no block has to know what the others hold before it writes.  With buckets of one
// contiguous range each, the counts of all blocks had to be scanned between a kernel that counted and one that
// read the samples back and moved the records: 1.0 M records in each of eight batches 168 us for
// the three, 107 of them for the one that drew, 114 us for k_sample_part, which sorts beside its scattered reads; its buckets'
// many short parts cost k_dedup_buckets some us (59 -> 68).  29 M records of one batch (two levels, with the split):
// 549 -> 339 us, k_dedup_buckets 164 -> 210.
// Blocks are of 256 threads, whose places a gather beside them leaves free often enough (whole neighbourhoods,
// pipelined: k_part_flat with 1024 threads 780 us, 56 alone).  Segments of 4096 records, 16 per thread, instead of 2048
// where a hop has more than 512 of those: k_dedup_buckets 78 -> 67 us, k_sample_part the same; 8192 records gain
// nothing more, and cost fanout 20 its occupancy (230 -> 293 us).
constexpr int kSegPer = 16;                       // most records of a segment per thread of its block
constexpr int kSegMax = kSegPer * kThreads;
__host__ __device__ constexpr uint32_t offs_stride(int lgB) { return ((1u << lgB) + 3u) & ~1u; }  // whole 4-byte words
// Most destinations of fanout d in a segment of `per` records per thread, and the least that a full one holds.
__host__ __device__ constexpr int seg_rows(int per, int d) {
  return per * kThreads / (1 + d) < per / 4 * kThreads ? per * kThreads / (1 + d) : per / 4 * kThreads;
}
__host__ __device__ constexpr int seg_least(int d) { return seg_rows(kSegPer, d) * (1 + d); }
// Exact offsets: records per segment, a multiple of 1024 settled on the device from the hop's record count, so
// that a launch has some 512 segments where it can.
__host__ __device__ inline uint32_t flat_seg(uint32_t batches, uint32_t records) {
  const uint32_t per = (records / 512u * batches + 1023u) & ~1023u;
  return per < 1024u ? 1024u : per > static_cast<uint32_t>(kSegMax) ? static_cast<uint32_t>(kSegMax) : per;
}
struct Segments {
  uint32_t count, cap;
};
__device__ __forceinline__ Segments hop_segments(const Launch& P, const BatchCtx& B, uint32_t n) {
  Segments s;
  if (P.flat) {
    const uint32_t records = n + static_cast<uint32_t>(B.counts[P.L + 1 + P.h]);
    s.cap = flat_seg(static_cast<uint32_t>(P.G), records);
    s.count = (records + s.cap - 1u) / s.cap;
  } else {
    s.cap = static_cast<uint32_t>(P.block_rows) * static_cast<uint32_t>(1 + P.d);
    s.count = (n + static_cast<uint32_t>(P.block_rows) - 1u) / static_cast<uint32_t>(P.block_rows);
  }
  return s;
}

// Buckets are dealt to blocks so that neighbouring buckets, whose parts share lines in every segment, run on
// the same XCD (workgroups go to the XCDs in turn, a batch's to 8 / gcd(8, batches) of them).
constexpr uint32_t kXcds = 8;
__device__ __forceinline__ uint32_t bucket_of_block(const Launch& P, uint32_t i, uint32_t buckets) {
  const uint32_t g = static_cast<uint32_t>(P.G);
  const uint32_t ways = g % 8u == 0u ? 1u : g % 4u == 0u ? 2u : g % 2u == 0u ? 4u : kXcds;
  if (buckets < ways) return i;
  return (i % ways) * (buckets / ways) + i / ways;
}

// counts <- (n_0, 0, ..., status 0), by a whole block.  A batch of more
// seeds than the graph has nodes holds a stray or a repeated one; it ends here, since grids, rows and
// positions of a hop are bounded by the number of nodes.
__device__ __forceinline__ void begin_counts(const Launch& P, const BatchCtx& B) {
  int64_t status = SMFG_ST_OK;
  if (B.num_seeds > P.num_nodes) {
    int stray = 0;
    for (int i = threadIdx.x; i < B.num_seeds; i += kThreads) {
      const int32_t v = B.seeds[i];
      stray |= v < 0 || static_cast<int64_t>(v) >= P.num_nodes;
    }
    status = __syncthreads_or(stray) ? SMFG_ST_SEED_OUT_OF_RANGE : SMFG_ST_DUPLICATE_SEED;
  }
  const int m = 2 * P.L + 2;
  for (int q = threadIdx.x; q < m; q += kThreads) B.counts[q] = q == 0 ? B.num_seeds : q == m - 1 ? status : 0;
}
// ... and node_ids[i] <- seed i, with its label.
__device__ __forceinline__ int32_t begin_seed(const Launch& P, const BatchCtx& B, int i) {
  const int32_t v = B.seeds[i];
  B.node_ids[i] = v;
  if (B.labels && v >= 0 && static_cast<int64_t>(v) < P.num_nodes) copy_label(P, B, i, v);
  return v;
}
// Both, for calls whose first hop is k_sample_part, which range-checks the seeds when the status word is zero.
__global__ void __launch_bounds__(kThreads) k_begin(const Launch P) {
  const BatchCtx& B = P.b[batch_of_block(P)];
  if (block_in_batch(P) == 0) begin_counts(P, B);
  const int stride = blocks_per_batch(P) * kThreads;
  for (int i = block_in_batch(P) * kThreads + threadIdx.x; i < B.num_seeds; i += stride) begin_seed(P, B, i);
}

// Exclusive scan of the counts cnt[0, nB) of a block's buckets in place, the total at cnt[nB], which is returned as
// well.  All threads of the block call, and all find cnt complete on return.
template <int NT>
__device__ __forceinline__ uint32_t scan_counts(uint32_t* cnt, uint32_t nB, uint32_t* scan) {
  const uint32_t per = nB > NT ? nB / NT : 1u;
  uint32_t sum = 0;
  for (uint32_t u = 0; u < per; ++u) {
    const uint32_t b = threadIdx.x * per + u;
    if (b < nB) sum += cnt[b];
  }
  uint32_t total;
  uint32_t pre = block_exscan<NT>(sum, scan, total);
  for (uint32_t u = 0; u < per; ++u) {
    const uint32_t b = threadIdx.x * per + u;
    if (b < nB) {
      const uint32_t c = cnt[b];
      cnt[b] = pre;
      pre += c;
    }
  }
  if (threadIdx.x == 0) cnt[nB] = total;
  __syncthreads();
  return total;
}
// Counts of a segment's buckets, two to a word: a record's rank in its bucket, then where its bucket begins.
__device__ __forceinline__ uint32_t count_packed(uint32_t* cnt, uint32_t b) {
  const uint32_t shift = (b & 1u) * 16u;
  return atomicAdd(&cnt[b >> 1], 1u << shift) >> shift & 0xFFFFu;
}
__device__ __forceinline__ uint32_t packed(const uint32_t* cnt, uint32_t b) { return cnt[b >> 1] >> ((b & 1u) * 16u) & 0xFFFFu; }
// Exclusive scan of such counts in place, with the total behind them, and to the segment's row of hist.
template <int NT>
__device__ __forceinline__ uint32_t segment_offsets(uint32_t* cnt, int lgB, uint16_t* __restrict__ row, uint32_t* scan) {
  const uint32_t words = lgB == 0 ? 1u : 1u << (lgB - 1);
  const uint32_t per = words > NT ? words / NT : 1u;
  uint32_t sum = 0, total;
  for (uint32_t u = 0; u < per; ++u) {
    const uint32_t w = threadIdx.x * per + u;
    if (w < words) sum += (cnt[w] & 0xFFFFu) + (cnt[w] >> 16);
  }
  uint32_t pre = block_exscan<NT>(sum, scan, total);
  for (uint32_t u = 0; u < per; ++u) {
    const uint32_t w = threadIdx.x * per + u;
    if (w < words) {
      const uint32_t c = cnt[w];
      cnt[w] = pre | (pre + (c & 0xFFFFu)) << 16;
      pre += (c & 0xFFFFu) + (c >> 16);
    }
  }
  if (lgB > 0 && threadIdx.x == 0) cnt[words] = total;
  __syncthreads();
  for (uint32_t q = threadIdx.x; q < offs_stride(lgB) / 2u; q += NT) reinterpret_cast<uint32_t*>(row)[q] = cnt[q];
  return total;
}

// Samples of the block's destinations -> gsrc, rowk; their records and the destinations' -> a segment.
// D: the fanout rounded up to 8, 16 or 32.  Segments of up to 4096 records are sorted by 256 threads, 16 records each, or by 512 in
// launches of at most kPartWideBlocks blocks, which leave most of the chip's waves unused otherwise: 85 K destinations x 5, 265 blocks, 24.6 ->
// 21.3 us; 442 blocks of 7 destinations x 20 24.7 -> 23.3; 2120 blocks 114 -> 119; with 1024 threads 21.0, 31.9 and 122.
constexpr int kPartWideThreads = 2 * kThreads, kPartWideBlocks = 512;
template <int D, int PER, int NT>
__global__ void __launch_bounds__(NT) k_sample_part(const Launch P) {
  constexpr int kRows = PER / 4;  // at most so many destinations per thread
  __shared__ union {
    DrawLds<kRows * NT, PER * NT> draw;
    unsigned long long stage[PER * NT];
  } S;
  __shared__ uint32_t scan[NT / 64];
  extern __shared__ uint32_t cnt[];  // offs_stride / 2 words
  const BatchCtx& B = P.b[batch_of_block(P)];
  const int blk = block_in_batch(P);
  const int n = static_cast<int>(B.counts[P.h]);  // on its way with the status
  if (block_has_status(B, P.L)) return;
  const int r0 = blk * P.block_rows;
  if (r0 >= n) return;
  const int rows = n - r0 < P.block_rows ? n - r0 : P.block_rows;
  const uint32_t d = static_cast<uint32_t>(P.d);
  const int lgB = hop_shape(P, B, n).lgB;
  for (uint32_t b = threadIdx.x; b < offs_stride(lgB) / 2u; b += NT) cnt[b] = 0u;
  draw_positions<D, NT>(
      P, B, P.h, d, B.node_ids, S.draw, r0, rows, [&] { set_status(B, P.L, SMFG_ST_SEED_OUT_OF_RANGE); },
      [&](int i, uint32_t, uint32_t k) { B.rowk[i] = static_cast<int32_t>(k); });
  const uint32_t samples = static_cast<uint32_t>(rows) * d;
  const uint32_t pos0 = static_cast<uint32_t>(r0) * d;
  uint32_t g[PER], rk[PER], v[kRows], rv[kRows];
  read_neighbours<NT>(P, DivD(d), S.draw, threadIdx.x, samples, g);
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    const int r = u * NT + static_cast<int>(threadIdx.x);
    v[u] = r < rows ? S.draw.node[r] : kNoSample;
    rv[u] = r < rows ? count_packed(cnt, part_bucket(v[u], lgB)) : 0u;
  }
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    rk[u] = 0u;
    if (g[u] != kNoSample) {
      B.gsrc[pos0 + u * NT + threadIdx.x] = static_cast<int32_t>(g[u]);
      rk[u] = count_packed(cnt, part_bucket(g[u], lgB));
    }
  }
  __syncthreads();
  const uint32_t total = segment_offsets<NT>(cnt, lgB, B.hist + static_cast<size_t>(blk) * offs_stride(lgB), scan);
#pragma unroll
  for (int u = 0; u < kRows; ++u) {
    const uint32_t r = u * NT + threadIdx.x;
    if (r < static_cast<uint32_t>(rows))
      S.stage[packed(cnt, part_bucket(v[u], lgB)) + rv[u]] = (static_cast<unsigned long long>(v[u]) << 32) | (static_cast<uint32_t>(r0) + r);
  }
#pragma unroll
  for (int u = 0; u < PER; ++u)
    if (g[u] != kNoSample)
      S.stage[packed(cnt, part_bucket(g[u], lgB)) + rk[u]] =
          (static_cast<unsigned long long>(g[u]) << 32) | (kPend | (pos0 + u * NT + threadIdx.x));
  __syncthreads();
  uint64_t* __restrict__ out = B.rec + static_cast<size_t>(blk) * (static_cast<uint32_t>(P.block_rows) * (1u + d));
  for (uint32_t t = threadIdx.x; t < total; t += NT) out[t] = S.stage[t];
}

// ---- second level ------------------------------------------------------------------------------
// A block takes a bucket's parts of `range` consecutive segments and sorts their records by the lg2 hash bits below the
// bucket's, so that a sub-bucket lies in parts as well, one per range: those of (range, bucket) go to the
// place in rec2 that the records of lower buckets of the range leave free in front of it, and bstart2 keeps
// where each of its sub-buckets begins.  range is such that a block's records fit its registers unless they are
// far from evenly spread.
// It reads every record once; a block per bucket, which counted the whole bucket before it moved anything, took 154 us
// for 29 M records, and 130 us so.
constexpr int kSplitThreads = kThreads;
constexpr uint32_t kSplitMax = kSegPer * kSplitThreads;
constexpr uint32_t kSplitAim = kSplitMax / 8u * 7u;  // some 8 standard deviations below
__host__ __device__ inline uint32_t split_range(uint32_t cap, int lgB) {
  const uint32_t per = static_cast<uint32_t>((static_cast<uint64_t>(kSplitAim) << lgB) / cap);
  return per < 1u ? 1u : per;
}

__global__ void __launch_bounds__(kSplitThreads) k_split_buckets(const Launch P) {
  constexpr int NT = kSplitThreads;
  __shared__ union {
    uint32_t list[kSplitMax];
    unsigned long long stage[kSplitMax];
  } S;
  __shared__ uint32_t cnt[(1 << kPartMaxLg2) + 1], scan[NT / 64];
  const BatchCtx& B = P.b[batch_of_block(P)];
  const int64_t n = B.counts[P.h];  // on its way with the status
  if (block_has_status(B, P.L)) return;
  const HopShape hs = hop_shape(P, B, n);
  if (hs.lg2 == 0) return;
  const Segments segs = hop_segments(P, B, static_cast<uint32_t>(n));
  const uint32_t nB = 1u << hs.lgB, n2 = 1u << hs.lg2, stride = offs_stride(hs.lgB);
  const uint32_t range = split_range(segs.cap, hs.lgB);
  const uint32_t ranges = (segs.count + range - 1u) / range;
  const int shift = 32 - hs.lgB - hs.lg2;
  const auto sub_of = [&](unsigned long long rec) { return ((static_cast<uint32_t>(rec >> 32) * kPartHash) >> shift) & (n2 - 1u); };
  for (uint32_t i = static_cast<uint32_t>(block_in_batch(P)); i < ranges * nB; i += static_cast<uint32_t>(blocks_per_batch(P))) {
    const uint32_t bucket = bucket_of_block(P, i % nB, nB);
    const uint32_t s0 = i / nB * range, s1 = segs.count - s0 < range ? segs.count : s0 + range;
    __syncthreads();  // the previous bucket is done with the LDS
    for (uint32_t b = threadIdx.x; b < n2; b += NT) cnt[b] = 0u;
    // how many records there are, how many of lower buckets, and where each is, while they fit
    uint32_t total = 0, lower = 0, longest = 0;
    for (uint32_t c0 = s0; c0 < s1; c0 += NT) {
      const uint32_t s = c0 + threadIdx.x;
      const uint16_t* at = B.hist + static_cast<size_t>(s) * stride + bucket;
      const uint32_t start = s < s1 ? at[0] : 0u, size = s < s1 ? at[1] - start : 0u;
      uint32_t turn, below;
      const uint32_t to = total + block_exscan<NT>(size, scan, turn);
      block_exscan<NT>(start, scan, below);
      total += turn;
      lower += below;
      longest = longest > size ? longest : size;
      if (total <= kSplitMax)
        for (uint32_t j = 0; j < size; ++j) S.list[to + j] = s * segs.cap + start + j;
    }
    __syncthreads();
    const uint32_t rec0 = s0 * segs.cap + lower;
    uint32_t* starts = B.bstart2 + static_cast<size_t>(i / nB * nB + bucket) * (n2 + 1u);
    if (total <= kSplitMax) {
      unsigned long long r[kSegPer];
      uint32_t rk[kSegPer];
#pragma unroll
      for (int u = 0; u < kSegPer; ++u) {
        const uint32_t q = u * NT + threadIdx.x;
        r[u] = q < total ? B.rec[S.list[q]] : kEmpty;
      }
#pragma unroll
      for (int u = 0; u < kSegPer; ++u) rk[u] = r[u] != kEmpty ? atomicAdd(&cnt[sub_of(r[u])], 1u) : 0u;
      __syncthreads();
      scan_counts<NT>(cnt, n2, scan);
      for (uint32_t b = threadIdx.x; b <= n2; b += NT) starts[b] = rec0 + cnt[b];
#pragma unroll
      for (int u = 0; u < kSegPer; ++u)
        if (r[u] != kEmpty) S.stage[cnt[sub_of(r[u])] + rk[u]] = r[u];
      __syncthreads();
      for (uint32_t t = threadIdx.x; t < total; t += NT) B.rec2[rec0 + t] = S.stage[t];
    } else {  // read twice, written one by one
      longest = block_max<NT>(longest, scan);
      const auto each = [&](auto use) {
        for (uint32_t q = threadIdx.x; q < (s1 - s0) * longest; q += NT) {
          const uint32_t s = s0 + q / longest, j = q % longest;
          const uint16_t* at = B.hist + static_cast<size_t>(s) * stride + bucket;
          if (at[0] + j < at[1]) use(B.rec[static_cast<size_t>(s) * segs.cap + at[0] + j]);
        }
      };
      each([&](unsigned long long rec) { atomicAdd(&cnt[sub_of(rec)], 1u); });
      __syncthreads();
      scan_counts<NT>(cnt, n2, scan);
      for (uint32_t b = threadIdx.x; b <= n2; b += NT) starts[b] = rec0 + cnt[b];
      __syncthreads();
      each([&](unsigned long long rec) { B.rec2[rec0 + atomicAdd(&cnt[sub_of(rec)], 1u)] = rec; });
    }
  }
}

// ---- dedup -----------------------------------------------------------------------------------------
// All records of a node are in one (sub-)bucket, so the bucket's table in LDS sees every occurrence of its nodes.
// The table in LDS: a node and the smallest value of its records per slot, in arrays of their own, since LDS atomics on
// 32 bits and reads of half the width make up for the second access (1.0 M records in eight batches 100 us with
// 64-bit words, 88 so).
template <int LG>
struct DedupTable {
  static constexpr uint32_t kSlots = 1u << LG;
  uint32_t node[kSlots], least[kSlots];
};
constexpr uint32_t kNoNode = 0xFFFFFFFFu;

template <int NT, int LG>
__device__ __forceinline__ void dedup_clear(DedupTable<LG>& T) {
  uint4* words = reinterpret_cast<uint4*>(&T);
  for (uint32_t q = threadIdx.x; q < sizeof(T) / 16; q += NT) words[q] = make_uint4(kNoNode, kNoNode, kNoNode, kNoNode);
}

// One record into the bucket's table: the slot of its node keeps the smallest value.  False if none of
// the first PROBES slots is free.
template <uint32_t PROBES, int LG>
__device__ __forceinline__ bool dedup_insert(DedupTable<LG>& T, unsigned long long rec, uint32_t& sl) {
  const uint32_t node = static_cast<uint32_t>(rec >> 32);
  // A plain read first: a node sampled thousands of times (a hub) would otherwise queue thousands of
  // compare-and-swaps on one LDS word.  Slots never lose their node, values only fall.
  for (uint32_t probes = 0; probes < PROBES; ++probes) {
    uint32_t old = T.node[sl];
    if (old == kNoNode) old = atomicCAS(&T.node[sl], kNoNode, node);
    if (old == kNoNode || old == node) {
      atomicMin(&T.least[sl], static_cast<uint32_t>(rec));
      return true;
    }
    sl = (sl + 1u) & (T.kSlots - 1u);
  }
  return false;
}

// What the smallest value of a record's node says about it: a sample that is not its node's smallest value learns the
// node's local id or the position of its first appearance.  kRepeated for a known node that is not alone with its
// id: two of them with one id can only be a repeated seed.
constexpr uint32_t kRepeated = 1u, kLost = 2u;
__device__ __forceinline__ uint32_t settle_record(int32_t* gsrc, uint32_t val, uint32_t least) {
  if (least == val) return 0u;  // a known node, or a first appearance, whose entry stays
  // least < kPend: the node's final local id; else least names the position of the first appearance
  if (val >= kPend)
    gsrc[val & ~kTagMask] =
        static_cast<int32_t>(least < kPend ? (kResolved | least) : (kPointer | (least & ~kTagMask)));
  return val < kPend ? kRepeated : 0u;
}
template <typename Batch>
__device__ __forceinline__ void report(const Batch& B, int L, uint32_t wrong) {
  if (wrong != 0u) set_status(B, L, (wrong & kLost) != 0u ? SMFG_ST_INTERNAL : SMFG_ST_DUPLICATE_SEED);
}

// What the filled table says about one record.
template <int LG>
__device__ __forceinline__ uint32_t dedup_settle(int32_t* gsrc, const DedupTable<LG>& T, unsigned long long rec, uint32_t sl) {
  const uint32_t node = static_cast<uint32_t>(rec >> 32);
  for (uint32_t probes = 0; probes < T.kSlots; ++probes) {
    if (T.node[sl] == node) return settle_record(gsrc, static_cast<uint32_t>(rec), T.least[sl]);
    sl = (sl + 1u) & (T.kSlots - 1u);
  }
  return kLost;  // every inserted node is found again, unless the scratch is disturbed meanwhile
}

// All records of a set that holds every record of its nodes, which fit the registers of the block: U per
// thread (kEmpty: none).  They stay there between the two passes, with the slot that the first one found; there
// are no more than 2^LG of them, so that the table cannot overflow.  `free_bits` hash bits are not
// yet spoken for.  All threads of the block (NT) call, none of which uses the table's LDS any more.
template <int NT, int LG, int U>
__device__ __forceinline__ uint32_t dedup_in_registers(int32_t* gsrc, DedupTable<LG>& T, int free_bits,
                                                       const unsigned long long (&mine)[U]) {
  const int down = free_bits > LG ? free_bits - LG : 0;
  uint32_t sl[U];
#pragma unroll
  for (int u = 0; u < U; ++u) sl[u] = ((static_cast<uint32_t>(mine[u] >> 32) * kPartHash) >> down) & (T.kSlots - 1u);
  dedup_clear<NT>(T);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (mine[u] != kEmpty) dedup_insert<(1u << LG)>(T, mine[u], sl[u]);
  __syncthreads();
  uint32_t wrong = 0u;
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (mine[u] != kEmpty) wrong |= settle_record(gsrc, static_cast<uint32_t>(mine[u]), T.least[sl[u]]);
  __syncthreads();
  return wrong;
}

// The records of a (sub-)bucket that lies in parts: part_of(p, from, size) tells where the p-th of them is in recs and
// how much it holds.  A thread per part, then a thread per record, which finds it through a list in the LDS:
// that of the usual bucket then becomes its table, of a larger one (hubs among its nodes, as a rule, so few nodes for
// its size) it stays in the upper half, a window of kList records at a time, and the records are read in both
// passes.  Nodes that do not fit half the table are taken in 2^lgR rounds, round i those whose next lgR hash bits equal i; should a round still
// overflow, the bucket starts over with one more bit.  With no more hash bits left than the slots have,
// every node of a round has a slot of its own (the hash is a bijection), so the retries end.
// U records per thread are kept in registers: 5 are what 64 of them hold, with which eight blocks share a compute unit
// (with 8, and 88 registers, 1.0 M records in each of eight batches took 78 us instead of 69), and enough for
// buckets of 1024 whatever their spread; 6 for those of 1228.
template <int U, typename PartOf>
__device__ __forceinline__ void dedup_parts(const Launch& P, const BatchCtx& B, DedupTable<kPartTableLg>& T, int& overflow,
                                            uint32_t* scan, const uint64_t* __restrict__ recs, uint32_t parts, int free_bits,
                                            PartOf part_of) {
  constexpr int NT = kThreads;
  constexpr int kPer = 4;  // parts per thread and turn
  constexpr uint32_t kList = DedupTable<kPartTableLg>::kSlots;
  static_assert(sizeof(T) == 2 * kList * sizeof(uint32_t), "the list takes the upper half");
  uint32_t* list = reinterpret_cast<uint32_t*>(&T) + kList;
  // few, longer parts: several threads to each, of which the first counts it
  uint32_t lanes = 64u;
  while (lanes > 1u && NT / lanes < parts) lanes /= 2u;
  const uint32_t lane = threadIdx.x & (lanes - 1u);
  // where the records w0 .. w0 + kList of the bucket are; returns how many it has in all
  const auto find = [&](uint32_t w0) {
    uint32_t cnt = 0;
    for (uint32_t p0 = 0; p0 < parts; p0 += NT * kPer / lanes) {
      uint32_t from[kPer], size[kPer], mine = 0, turn;
#pragma unroll
      for (int u = 0; u < kPer; ++u) {  // every read on its way before the first is used
        const uint32_t p = p0 + (u * NT + threadIdx.x) / lanes;
        part_of(p < parts ? p : 0u, from[u], size[u]);
      }
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        if (p0 + (u * NT + threadIdx.x) / lanes >= parts) size[u] = 0u;
        mine += lane == 0u ? size[u] : 0u;
      }
      uint32_t to = cnt + block_exscan<NT>(mine, scan, turn) - w0;
      if (lane != 0u) to -= size[0] + size[1] + size[2] + size[3];
      cnt += turn;
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        for (uint32_t j = lane; j < size[u]; j += lanes)
          if (to + j < kList) list[to + j] = from[u] + j;
        to += size[u];
      }
    }
    __syncthreads();
    return cnt;
  };
  const uint32_t cnt = find(0u);
  if (cnt <= NT * U) {
    unsigned long long mine[U];
#pragma unroll
    for (int u = 0; u < U; ++u) mine[u] = u * NT + threadIdx.x < cnt ? recs[list[u * NT + threadIdx.x]] : kEmpty;
    __syncthreads();
    if (cnt != 0u) report(B, P.L, dedup_in_registers<NT>(B.gsrc, T, free_bits, mine));
    return;
  }
  constexpr int kHalf = kPartTableLg - 1, kAhead = 4;
  DedupTable<kHalf>& H = *reinterpret_cast<DedupTable<kHalf>*>(&T);
  const int max_lgR = free_bits > kHalf ? free_bits - kHalf : 0;
  uint32_t wrong = 0u;
#pragma unroll 1
  for (int lgR = 0; lgR <= max_lgR; ++lgR) {
    const int rem = free_bits - lgR, down = rem > kHalf ? rem - kHalf : 0;
    const uint32_t rounds = 1u << lgR;
    bool failed = false;
#pragma unroll 1
    for (uint32_t round = 0; round < rounds && !failed; ++round) {
      dedup_clear<NT>(H);
      if (threadIdx.x == 0) overflow = 0;
#pragma unroll 1
      for (int pass = 0; pass < 2 && !failed; ++pass) {  // insert, then settle
#pragma unroll 1
        for (uint32_t w0 = 0; w0 < cnt; w0 += kList) {
          __syncthreads();
          if (cnt > kList) find(w0);
          const uint32_t here = cnt - w0 < kList ? cnt - w0 : kList;
#pragma unroll 1
          for (uint32_t r = threadIdx.x; r < here; r += NT * kAhead) {
            unsigned long long mine[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) mine[u] = r + u * NT < here ? recs[list[r + u * NT]] : kEmpty;
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
              const uint32_t hash = static_cast<uint32_t>(mine[u] >> 32) * kPartHash;
              if (mine[u] == kEmpty || (lgR != 0 && ((hash >> rem) & (rounds - 1u)) != round)) continue;
              uint32_t sl = (hash >> down) & (H.kSlots - 1u);
              if (pass == 1) wrong |= dedup_settle(B.gsrc, H, mine[u], sl);
              else if (!dedup_insert<64>(H, mine[u], sl)) overflow = 1;
            }
          }
        }
        __syncthreads();
        failed = overflow != 0;
      }
      __syncthreads();  // every thread has read the overflow word, and is done with the table
    }
    if (!failed) break;
    if (lgR == max_lgR) wrong |= kLost;  // cannot overflow with a slot per node
  }
  report(B, P.L, wrong);
}

// LARGE: the hop may have two levels, or the largest buckets of one (the host's bound says so); then a block takes
// several (sub-)buckets one after the other.
template <bool LARGE>
__global__ void __launch_bounds__(kThreads, LARGE ? 7 : 8) k_dedup_buckets(const Launch P) {
  __shared__ __align__(16) DedupTable<kPartTableLg> T;
  __shared__ uint32_t scan[kThreads / 64];
  __shared__ int overflow_lds;
  const BatchCtx& B = P.b[batch_of_block(P)];
  const int64_t n = B.counts[P.h];  // on its way with the status
  if (block_has_status(B, P.L)) return;
  const HopShape hs = hop_shape(P, B, n);
  const Segments segs = hop_segments(P, B, static_cast<uint32_t>(n));
  const bool two = LARGE && hs.lg2 != 0;
  const uint32_t nB = 1u << hs.lgB, n2 = 1u << hs.lg2, all = nB << hs.lg2, stride = offs_stride(hs.lgB);
  const uint32_t range = split_range(segs.cap, hs.lgB), parts = two ? (segs.count + range - 1u) / range : segs.count;
  for (uint32_t i = static_cast<uint32_t>(block_in_batch(P)); i < all; i += static_cast<uint32_t>(blocks_per_batch(P))) {
    const uint32_t bucket = bucket_of_block(P, i, all);
    dedup_parts<LARGE ? 6 : 5>(P, B, T, overflow_lds, scan, two ? B.rec2 : B.rec, parts, 32 - hs.lgB - hs.lg2,
                [&](uint32_t p, uint32_t& from, uint32_t& size) {
                  if (two) {
                    const uint32_t* at = B.bstart2 + static_cast<size_t>(p * nB + (bucket >> hs.lg2)) * (n2 + 1u) + (bucket & (n2 - 1u));
                    from = at[0];
                    size = at[1] - at[0];
                  } else {
                    const uint16_t* at = B.hist + static_cast<size_t>(p) * stride + bucket;
                    from = p * segs.cap + at[0];
                    size = static_cast<uint32_t>(at[1]) - at[0];
                  }
                });
    __syncthreads();
  }
}

// A tile's destinations and, a turn ahead of their use, its entries: flag_rows asks for a tile's first entries together with
// the samples of its destinations, and for the others before it looks at those before them.  29 M positions 42.6 -> 25.1 us, 77 K
// destinations x 20 10.2 -> 5.9, 11 K x 10 6.4 -> 4.3.  The same in assemble costs it registers: 24 -> 28 us for 1.2 M x 5.
struct Tile {
  int i0, rows;         // its first destination, and how many there are
  uint32_t pos0, cnt;   // the same of its positions
  __device__ __forceinline__ Tile(int tile, int n, uint32_t d)
      : i0(tile * kTileRows), rows(n - i0 < kTileRows ? n - i0 : kTileRows), pos0(static_cast<uint32_t>(i0) * d),
        cnt(rows > 0 ? static_cast<uint32_t>(rows) * d : 0u) {}
};
template <int U>
struct TileEntries {
  uint32_t e[U];  // of positions at, at + kThreads, ... of a tile
  __device__ __forceinline__ void fetch(const BatchCtx& B, const Tile& t, uint32_t at) {
#pragma unroll
    for (int u = 0; u < U; ++u) e[u] = at + u * kThreads < t.cnt ? static_cast<uint32_t>(B.gsrc[t.pos0 + at + u * kThreads]) : kResolved;
  }
};

// flag_rows for the entries dedup_buckets leaves: a valid sample whose entry still is a node id
// (bit 31 clear) is a first appearance.  Per destination: bit mask of its first appearances; in-tile
// exclusive scan of (samples, new nodes); per-tile totals.  Streaming: a wave's ballot is the bits of 64 positions,
// from which each destination then takes its own.  With an LDS atomicOr per first appearance, 20 consecutive
// ones of which hit one word, 29 M positions took 54 us; 43 so, and 25, 4.7 TB/s of entries, with the entries a turn ahead.
__global__ void __launch_bounds__(kThreads) k_flag_rows_part(const Launch P) {
  __shared__ unsigned long long lds[kThreads / 64];
  __shared__ unsigned long long bits[kTileRows * SMFG_MAX_FANOUT / 64 + 1];  // of the tile's positions
  const BatchCtx& B = P.b[batch_of_block(P)];
  const int nblocks = blocks_per_batch(P);
  const int n = static_cast<int>(B.counts[P.h]);  // on its way with the status
  if (block_has_status(B, P.L)) return;
  const uint32_t d = static_cast<uint32_t>(P.d);
  const int tiles = (n + kTileRows - 1) / kTileRows;
  if (block_in_batch(P) >= tiles) return;
  const int tr = threadIdx.x;
  constexpr int U = 4;
  TileEntries<U> ahead;
  int next_k = 0;
  const auto ask = [&](const Tile& t) {
    ahead.fetch(B, t, tr);
    next_k = tr < t.rows ? B.rowk[t.i0 + tr] : 0;
  };
  ask(Tile(block_in_batch(P), n, d));
  for (int tile = block_in_batch(P); tile < tiles; tile += nblocks) {
    const Tile t(tile, n, d);
    const int k = next_k;
    __syncthreads();  // the previous tile's bits have been read
    for (uint32_t base = tr & ~63; base < t.cnt; base += kThreads * U) {  // whole waves
      const TileEntries<U> here = ahead;
      ahead.fetch(B, t, base + kThreads * U + (tr & 63));
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const unsigned long long b = __ballot((here.e[u] & kResolved) == 0u);
        if ((tr & 63) == 0 && base + u * kThreads < t.cnt) bits[(base + u * kThreads) >> 6] = b;
      }
    }
    if (tile + nblocks < tiles) ask(Tile(tile + nblocks, n, d));
    __syncthreads();
    uint32_t m = 0u;
    if (k > 0) {
      const uint32_t at = static_cast<uint32_t>(tr) * d, sh = at & 63u;
      unsigned long long own = bits[at >> 6] >> sh;
      if (sh + d > 64u) own |= bits[(at >> 6) + 1u] << (64u - sh);
      m = static_cast<uint32_t>(own & ((1ull << k) - 1ull));
    }
    const unsigned long long x = (static_cast<unsigned long long>(k) << 32) | static_cast<unsigned long long>(__popc(m));
    unsigned long long total;
    const unsigned long long pre = block_exscan(x, lds, total);
    if (tr < t.rows) {
      B.rowmn[t.i0 + tr] = make_uint2(m, static_cast<uint32_t>(pre & 0xFFFFFFFFull));
      B.rowoff[t.i0 + tr] = static_cast<int32_t>(pre >> 32);
    }
    if (tr == 0) B.tile_sums[tile] = total;
  }
}

// assemble for those entries: block indptr; block indices = final local ids; node ids of the
// first appearances.  A pointer always names a first appearance, so one lookup of that
// destination's record settles it.  SCAN (hops of at most kAssembleTiles tiles, one per block): every block
// scans the tile totals for itself, a few kilobytes from the L2, instead of k_scan_tiles before it -
// 3 to 5 us of a launch that does nothing else, for less than 1 us here.  Where that leaves compute units idle (SHARED), P.parts blocks share a
// tile, a run of kThreads U positions each in turn: 11 K destinations x 10 8.6 -> 5.9 us, 77 K x 20 14.1 -> 12.1, 4 K x 20 10.5 -> 6.1.
// In a variant of its own: the one more count costs the other an eighth of its waves (1.2 M destinations x 5 24 -> 26 us).
constexpr int kAssembleTiles = 1024;
template <bool SCAN, bool SHARED>
__global__ void __launch_bounds__(kThreads) k_assemble_part(const Launch P) {
  constexpr int kPer = kAssembleTiles / kThreads;
  __shared__ uint32_t tile_new[SCAN ? kAssembleTiles : 1];  // new nodes before each tile
  __shared__ unsigned long long own_lds, scan_lds[kThreads / 64];
  // per destination: samples, first-appearance bits, block offset, local id of the first new node
  __shared__ uint4 row_lds[kTileRows];
  const BatchCtx& B = P.b[batch_of_block(P)];
  const int n = static_cast<int>(B.counts[P.h]);  // on its way with the status
  if (block_has_status(B, P.L)) return;
  const uint32_t d = static_cast<uint32_t>(P.d);
  const DivD div(d);
  const double inv_d = 1.0 / static_cast<double>(d);
  const int tiles = (n + kTileRows - 1) / kTileRows;
  const int nblocks = blocks_per_batch(P);
  constexpr int U = 4;
  const int parts = SHARED ? P.parts : 1, own = block_in_batch(P) / parts, part = block_in_batch(P) - own * parts;
  if (SCAN) {
    if (own >= (tiles > 0 ? tiles : 1)) return;  // the first block also closes an empty hop
    unsigned long long x[kPer], mine = 0, total;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int t = threadIdx.x * kPer + u;
      x[u] = t < tiles ? B.tile_sums[t] : 0ull;
      mine += x[u];
    }
    unsigned long long pre = block_exscan(mine, scan_lds, total);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int t = threadIdx.x * kPer + u;
      tile_new[t] = static_cast<uint32_t>(pre);
      if (t == own) own_lds = pre;
      pre += x[u];
    }
    if (!close_hop(P, B, n, total, block_in_batch(P) == 0 && threadIdx.x == 0)) return;
    __syncthreads();
  }
  const auto tile_before = [&](uint32_t t) { return SCAN ? tile_new[t] : static_cast<uint32_t>(B.tile_sums[t] & 0xFFFFFFFFull); };
  for (int tile = own; tile < tiles; tile += nblocks) {
    const int i0 = tile * kTileRows;
    const int nrows = n - i0 < kTileRows ? n - i0 : kTileRows;
    const int tr = threadIdx.x;
    const unsigned long long tpre = SCAN ? own_lds : B.tile_sums[tile];
    __syncthreads();
    if (tr < nrows) {
      const uint32_t off = static_cast<uint32_t>(tpre >> 32) + static_cast<uint32_t>(B.rowoff[i0 + tr]);
      const uint2 mn = B.rowmn[i0 + tr];
      row_lds[tr] = make_uint4(static_cast<uint32_t>(B.rowk[i0 + tr]), mn.x, off,
                               static_cast<uint32_t>(n) + static_cast<uint32_t>(tpre & 0xFFFFFFFFull) + mn.y);
      if (part == 0) B.blk_indptr[i0 + tr] = static_cast<int32_t>(off);
    }
    __syncthreads();
    const uint32_t pos0 = static_cast<uint32_t>(i0) * d;
    const uint32_t cnt = static_cast<uint32_t>(nrows) * d;
    for (uint32_t base = static_cast<uint32_t>(part * kThreads * U) + threadIdx.x; base < cnt; base += parts * kThreads * U) {
      uint32_t e[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t idx = base + u * kThreads;
        e[u] = idx < cnt ? static_cast<uint32_t>(B.gsrc[pos0 + idx]) : 0u;
      }
      // the records of the destinations that pointers name are fetched for all U samples of the
      // thread before any is used (other samples fetch the tile's first record), so the scattered
      // reads of a thread overlap
      uint32_t sl[U], q[U], qi[U];
      uint4 row[U];
      bool live[U], dup[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t idx = base + u * kThreads;
        uint32_t r = 0u;
        sl[u] = 0u;
        if (idx < cnt) div.split(idx, r, sl[u]);
        row[u] = row_lds[r];
        live[u] = idx < cnt && sl[u] < row[u].x;
        dup[u] = live[u] && (e[u] & kPointer) == kPointer;
        q[u] = dup[u] ? (e[u] & ~kPointer) : pos0;
        // q / d: positions have 30 bits, so half of 1 / d is far more than what the product is off
        qi[u] = static_cast<uint32_t>((static_cast<double>(q[u]) + 0.5) * inv_d);
      }
      uint2 mn[U];
      uint32_t ts[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        mn[u] = B.rowmn[qi[u]];
        ts[u] = tile_before(qi[u] / kTileRows);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (!live[u]) continue;
        uint32_t local;
        if ((e[u] & kResolved) == 0u) {  // first appearance: rank among the new nodes of this hop
          local = row[u].w + __popc(row[u].y & ((1u << sl[u]) - 1u));
          B.node_ids[local] = static_cast<int32_t>(e[u]);
        } else if (dup[u]) {
          const uint32_t qs = q[u] - qi[u] * d;
          local = static_cast<uint32_t>(n) + ts[u] + mn[u].y + __popc(mn[u].x & ((1u << qs) - 1u));
          if (((mn[u].x >> qs) & 1u) == 0u) {  // the named sample is not a first appearance: scratch disturbed
            set_status(B, P.L, SMFG_ST_INTERNAL);
            local = 0u;
          }
        } else {
          local = e[u] & ~kPointer;
        }
        B.blk_indices[row[u].z + sl[u]] = static_cast<int32_t>(local);
      }
    }
  }
}

}  // namespace smfg_dev

#endif  // SMFG_KERNELS_PART_H_
