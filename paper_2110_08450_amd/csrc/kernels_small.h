// libsmfg small hops: two launches per hop, or one, whatever is in it, and at most one before the first.
//
// A hop of fewer than kSmallRecords records keeps no kernel busy for much longer than its launch and a
// chain of dependent reads take (about 5 us together), so what counts is how many there are:
//   draw    of the first hop, unless finish does it: many blocks, since its scattered reads need many compute units to be in flight at once;
//   dedup   unless finish does it: 2^kSmallLgB blocks per batch, each reads all records, keeps those of its hash bucket and
//           settles them in an LDS table: no histogram, no scatter;
//   finish  blocks of consecutive destinations; each reads all entries of the hop, which gives it the
//           first-appearance bits and their prefix sums in its own LDS, and then writes the final ids of
//           its own destinations: no flags, no scan of tiles in between, no block waits for another.  It then
//           knows the ids and local ids of its destinations and of the new nodes among their samples, and goes on
//           with these: the draw of the next small hop, or, after the last hop of a call, their feature rows.
// Reading everything in every block costs up to 128 KB from the L2, a few us at most.  Measured, one batch
// per call, whole call with its gather, against the table strategy's four launches per hop: (10, 5) with
// 256 seeds 62 -> 34 us, (15, 10, 5) with 16 seeds 78 -> 52 us; with a dedup for every hop 38 and 60, and with the draw and the
// gather in launches of their own 41 and 65 us.  One block for a
// whole batch was slower (16 seeds: 172 us): a single compute unit has too few reads in flight.
#ifndef SMFG_KERNELS_SMALL_H_
#define SMFG_KERNELS_SMALL_H_

#include <type_traits>

#include "device_common.h"
#include "kernels_fast.h"
#include "kernels_part.h"

namespace smfg_dev {

constexpr int kSmallThreads = 1024;
constexpr int64_t kSmallRecords = 32768;  // known nodes + positions of a hop: fewer than this
constexpr int kSmallLgB = 4;              // 16 buckets
constexpr int kSmallTableLg = 13;         // of 8192 slots
constexpr uint32_t kSmallList = 1u << (kSmallTableLg - 1);
// Destinations per block of finish for a hop of at most max_rows: some 32 blocks per batch, fewer where there are
// many batches, since a block takes a compute unit for itself.
constexpr int kSmallMinBlocks = 256 / SMFG_MAX_BATCHES, kSmallMaxBlocks = 32, kSmallMinTile = 1;
constexpr int small_tile(int64_t max_rows, int batches) {
  const int most = 256 / batches, blocks = most > kSmallMaxBlocks ? kSmallMaxBlocks : most;
  const int64_t tile = (max_rows + blocks - 1) / blocks;
  return static_cast<int>(tile < kSmallMinTile ? kSmallMinTile : tile);
}
// The most destinations and new nodes of a block.
constexpr int kSmallNodes = static_cast<int>(kSmallRecords) / kSmallMinBlocks + kSmallMinTile * (1 + SMFG_MAX_FANOUT);
static_assert(kSmallRecords / 2 / kSmallMinBlocks <= kSmallThreads, "a thread per destination");
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(1)));  // a vector at any byte address

struct SmallBatch {
  const int32_t* seeds;
  int64_t* counts;
  int32_t* node_ids;
  uint8_t* labels;
  uint8_t* features;
  int32_t* gsrc;  // per (destination, slot): node id, settled state, or kNoSample
  int32_t* rowk;  // samples per destination
  int32_t* blk_indptr[SMFG_MAX_LAYERS];
  int32_t* blk_indices[SMFG_MAX_LAYERS];
  int32_t edge_capacity[SMFG_MAX_LAYERS];
  int32_t node_capacity;
  int32_t num_seeds;
  uint32_t key0, key1;
  // Odd hops have arrays of their own, so many times 256 bytes behind these: finish writes what the next hop starts with
  // while other blocks of it still read the present one's.
  uint32_t gsrc_odd, rowk_odd;
};

struct SmallLaunch {
  const int64_t* indptr;
  const int32_t* indices;
  const uint8_t* labels;
  int64_t num_nodes;
  int32_t label_bytes;
  int32_t L;
  int32_t G;
  int32_t fanouts[SMFG_MAX_LAYERS];
  int32_t rows;                    // destinations per block of the draw
  int32_t tile[SMFG_MAX_LAYERS];   // destinations per block of finish, at most kSmallThreads
  const uint8_t* feat;             // rows to be gathered by the last hop, or null
  int64_t row_bytes, row_stride;
  SmallBatch b[SMFG_MAX_BATCHES];
};
static_assert(sizeof(SmallLaunch) <= 4096, "kernel arguments are limited to 4 KB");

__device__ __forceinline__ int32_t* small_array(int32_t* even, uint32_t odd, int h) {
  return (h & 1) == 0 ? even : even + static_cast<size_t>(odd) * 64u;
}
__device__ __forceinline__ int32_t* small_gsrc(const SmallBatch& B, int h) { return small_array(B.gsrc, B.gsrc_odd, h); }
__device__ __forceinline__ int32_t* small_rowk(const SmallBatch& B, int h) { return small_array(B.rowk, B.rowk_odd, h); }

__device__ __forceinline__ int small_batch(const SmallLaunch& P) { return static_cast<int>(blockIdx.x % static_cast<unsigned>(P.G)); }
__device__ __forceinline__ int small_block(const SmallLaunch& P) { return static_cast<int>(blockIdx.x / static_cast<unsigned>(P.G)); }
// Destinations of hop h, or -1 if the batch has a status (the same for the whole block).  Hop 0 starts
// the counts, so its draw does not look at them.
__device__ __forceinline__ int small_rows(const SmallLaunch& P, const SmallBatch& B, int h) {
  const int n = h == 0 ? B.num_seeds : static_cast<int>(B.counts[h]);  // on its way with the status
  return block_has_status(B, P.L) ? -1 : n;
}

// Hop 0 of more than finish draws: every position gets a node id or kNoSample.  Reads the seeds, copies them to the node ids and starts the
// counts; k_small_dedup, or finish, looks for seeds that are no nodes.
template <int D>
__global__ void __launch_bounds__(kThreads) k_small_draw(const SmallLaunch P) {
  __shared__ DrawLds<kThreads, 512> S;  // kThreads / d rows of at most d + 1 words
  const SmallBatch& B = P.b[small_batch(P)];
  const int n = B.num_seeds;
  const int i0 = small_block(P) * P.rows;
  if (i0 == 0)
    for (int q = threadIdx.x; q < 2 * P.L + 2; q += kThreads) B.counts[q] = q == 0 ? n : 0;
  if (i0 >= n) return;
  const uint32_t d = static_cast<uint32_t>(P.fanouts[0]);
  const int rows = n - i0 < P.rows ? n - i0 : P.rows;
  draw_positions<D, kThreads>(
      P, B, 0, d, B.seeds, S, i0, rows, [] {},
      [&](int i, uint32_t v, uint32_t k) {
        B.rowk[i] = static_cast<int32_t>(k);
        B.node_ids[i] = static_cast<int32_t>(v);
        if (B.labels && v < P.num_nodes) copy_label(P, B, i, static_cast<int32_t>(v));
      });
  const uint32_t cnt = static_cast<uint32_t>(rows) * d;
  uint32_t g[1];  // a sample per thread
  read_neighbours<kThreads>(P, DivD(d), S, threadIdx.x, cnt, g);
  if (threadIdx.x < cnt) B.gsrc[static_cast<uint32_t>(i0) * d + threadIdx.x] = static_cast<int32_t>(g[0]);
}

// All records of a set that holds every record of its nodes: record(i) for i in [0, cnt) one of them or
// kEmpty; `free_bits` hash bits are not yet spoken for.  More than half the table are handled in 2^lgR rounds, as
// in dedup_parts.  overflow: one LDS word.  What was wrong, if anything.  All threads of the block (NT) call.
template <int NT, int LG, typename Record>
__device__ __forceinline__ uint32_t dedup_records(int32_t* gsrc, DedupTable<LG>& T, int& overflow, uint32_t cnt, int free_bits,
                                                  Record record) {
  constexpr int U = 8;  // records in flight per thread
  const int max_lgR = free_bits > LG ? free_bits - LG : 0;
  if (cnt <= NT * U && cnt <= T.kSlots / 2) {
    unsigned long long mine[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t r = u * NT + threadIdx.x;
      mine[u] = r < cnt ? record(r) : kEmpty;
    }
    return dedup_in_registers<NT>(gsrc, T, free_bits, mine);
  }
  uint32_t wrong = 0u;
  int lgR = 0;
  while (lgR < max_lgR && (cnt >> lgR) > T.kSlots / 2) ++lgR;
  for (;;) {
    bool failed = false;
    const int rem = free_bits - lgR;  // hash bits below the round's
    const int down = rem > LG ? rem - LG : 0;
    const uint32_t rounds = 1u << lgR;
    for (uint32_t round = 0; round < rounds && !failed; ++round) {
      dedup_clear<NT>(T);
      if (threadIdx.x == 0) overflow = 0;
      __syncthreads();
      for (int pass = 0; pass < 2 && !failed; ++pass) {  // insert, then settle
        for (uint32_t c0 = 0; c0 < cnt; c0 += NT * U) {
          unsigned long long mine[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const uint32_t r = c0 + u * NT + threadIdx.x;
            mine[u] = r < cnt ? record(r) : kEmpty;
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            if (mine[u] == kEmpty) continue;
            const uint32_t hsh = static_cast<uint32_t>(mine[u] >> 32) * kPartHash;
            if (lgR != 0 && ((hsh >> rem) & (rounds - 1u)) != round) continue;
            uint32_t sl = (hsh >> down) & (T.kSlots - 1u);
            if (pass == 0) {
              if (!dedup_insert<(1u << LG)>(T, mine[u], sl)) overflow = 1;
            } else {
              wrong |= dedup_settle(gsrc, T, mine[u], sl);
            }
          }
        }
        __syncthreads();
        failed = overflow != 0;
      }
    }
    if (!failed) break;
    if (lgR >= max_lgR) {  // cannot overflow with a slot per node
      wrong |= kLost;
      break;
    }
    __syncthreads();  // every thread has read the overflow word before the next attempt clears it
    ++lgR;
  }
  return wrong;
}

// One block per (batch, bucket).  Blocks of other buckets rewrite entries while this one reads them; such
// an entry is of no interest before (another bucket's node) nor after (bit 31 set).
__global__ void __launch_bounds__(kSmallThreads) k_small_dedup(const SmallLaunch P, int h) {
  constexpr int NT = kSmallThreads;
  __shared__ __align__(16) DedupTable<kSmallTableLg> T;
  __shared__ unsigned long long list[kSmallList];
  __shared__ uint32_t listed;
  __shared__ int overflow;
  const SmallBatch& B = P.b[small_batch(P)];
  const uint32_t bucket = static_cast<uint32_t>(small_block(P));
  if (threadIdx.x == 0) listed = 0u;
  const int rows = small_rows(P, B, h);
  if (rows < 0) return;
  const uint32_t n = static_cast<uint32_t>(rows);
  const uint32_t cnt = n + n * static_cast<uint32_t>(P.fanouts[h]);
  // an entry is of interest if it is a node of this bucket (bit 31: no sample, or settled in an earlier
  // round - its node's smallest value never is).  The bucket comes from a full-rate 24-bit
  // multiplication, since every record is tested by all 16 blocks
  const auto wanted = [&](uint32_t node) {
    const uint32_t x = (node ^ (node >> 15)) & 0xFFFFFFu;
    return (node & kResolved) == 0u && ((__umul24(x, 0x79B1B5u) >> 20) & ((1u << kSmallLgB) - 1u)) == bucket;
  };
  const auto as_record = [&](uint32_t node, uint32_t i) {
    return (static_cast<unsigned long long>(node) << 32) | (i < n ? i : (kPend | (i - n)));
  };
  if (h == 0 && bucket == 0u)
    for (uint32_t i = threadIdx.x; i < n; i += NT)
      if (static_cast<uint32_t>(B.node_ids[i]) >= P.num_nodes) set_status(B, P.L, SMFG_ST_SEED_OUT_OF_RANGE);
  const uint32_t positions = cnt - n;
  int32_t* gsrc = small_gsrc(B, h);
  // a turn: K known nodes and 4 U positions per thread, every read on its way before the first is used
  // (the entries are padded to whole 256 bytes); a wave reserves room for all it found at once (a thread each, 16 waves of 64 atomics
  // on one word: 256 seeds x 10 and then x 5 8.5 -> 7.0 us, 1024 x 15 9.8 -> 7.7)
  constexpr int K = 4, U = 4;
  for (uint32_t c = 0; c * NT * K < n || c * NT * 4u * U < positions; ++c) {
    uint32_t e[K + 4 * U];
    const uint32_t i0 = c * NT * K + threadIdx.x, q0 = (c * NT * U + threadIdx.x) * 4u;
#pragma unroll
    for (int u = 0; u < K; ++u) e[u] = i0 + u * NT < n ? static_cast<uint32_t>(B.node_ids[i0 + u * NT]) : kNoSample;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t q = q0 + u * NT * 4u;
      const uint4 x = q < positions ? *reinterpret_cast<const uint4*>(gsrc + q) : make_uint4(kNoSample, kNoSample, kNoSample, kNoSample);
      e[K + 4 * u] = x.x; e[K + 4 * u + 1] = x.y; e[K + 4 * u + 2] = x.z; e[K + 4 * u + 3] = x.w;
    }
    uint32_t found = 0;
#pragma unroll
    for (int t = 0; t < K + 4 * U; ++t) {
      const bool there = t < K || q0 + static_cast<uint32_t>((t - K) / 4) * NT * 4u + static_cast<uint32_t>((t - K) % 4) < positions;
      found |= (there && wanted(e[t]) ? 1u : 0u) << t;
    }
    const uint32_t own = static_cast<uint32_t>(__popc(found)), upto = wave_inscan(own);
    uint32_t at = 0;
    if ((threadIdx.x & 63u) == 63u) at = atomicAdd(&listed, upto);
    at = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(at), 63)) + upto - own;
#pragma unroll
    for (int t = 0; t < K + 4 * U; ++t)
      if (found >> t & 1u) {
        const uint32_t i = t < K ? i0 + t * NT : n + q0 + static_cast<uint32_t>((t - K) / 4) * NT * 4u + static_cast<uint32_t>((t - K) % 4);
        if (at < kSmallList) list[at] = as_record(e[t], i);
        ++at;
      }
  }
  __syncthreads();
  const bool fits = listed <= kSmallList;
  const uint32_t wrong = dedup_records<NT>(gsrc, T, overflow, fits ? listed : cnt, 32, [&](uint32_t i) {
    if (fits) return list[i];
    const uint32_t node = static_cast<uint32_t>(i < n ? B.node_ids[i] : gsrc[i - n]);
    return wanted(node) ? as_record(node, i) : kEmpty;
  });
  report(B, P.L, wrong);
}

// Where finish finds the entries of its hop: settled by k_small_dedup, drawn by the launch before, or nowhere yet.
enum { kSettled, kDrawn, kSeeds };
// A hop of at most kOneRecords records is settled in the blocks of finish themselves, each of which has a table of all its nodes,
// and a first hop of at most kOneDraw records and kOneSamples samples, one per thread, is drawn there as well: every block does all of it
// again, but there is a launch less.  Only the first block tells what is wrong.  Calls of one hop with each in a launch of its own /
// settled in finish / drawn there too, 1 batch and 16 batches, microseconds:
//   16 seeds x 15      17.1 13.8 12.7   22.4 15.0 12.8        128 x 31 (4096 records)   24.9 23.2    26.6 26.3
//   68 x 15            17.8 14.9 13.4   22.8 15.2 14.3        512 x 7 (4096)            19.2 18.8    22.6 21.3
//   128 x 7            16.5 13.4 12.5   22.7 14.7 13.3        1024 x 3 (4096)           19.0 19.0    22.7 22.2
//   1024 x 1 (2048)    17.5 15.0 17.2   22.7 17.2 18.8
constexpr int64_t kOneRecords = 4096, kOneDraw = 1280, kOneSamples = 1024;
template <int FROM>
struct SmallTable {
  DedupTable<kSmallTableLg> T;
  uint32_t entry[kOneRecords];  // per position what k_small_dedup leaves in gsrc
};
template <>
struct SmallTable<kSettled> {};

// The entries of a batch's hop -> A.entry; e: those of positions 4 tid .. 4 tid + 3, known(i): known node i.  All
// threads call; true if a known node is there twice.
template <int NT, typename Known, typename Table>
__device__ __forceinline__ bool settle_in_block(Table& A, uint32_t n, uint32_t positions, const uint32_t (&e)[4], Known known) {
  constexpr int K = static_cast<int>(kOneRecords / 2 / NT);
  static_assert(kOneRecords <= 4 * NT && kOneRecords <= 1 << (kSmallTableLg - 1), "positions of a thread, half the table");
  const int tid = threadIdx.x;
  const auto home = [](uint32_t node) { return (node * kPartHash) >> (32 - kSmallTableLg); };
  uint32_t known_slot[K], slot[4];
  dedup_clear<NT>(A.T);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < K; ++u) {
    const uint32_t i = u * NT + tid;
    const uint32_t v = i < n ? known(i) : 0u;
    known_slot[u] = home(v);
    if (i < n) dedup_insert<(1u << kSmallTableLg)>(A.T, static_cast<unsigned long long>(v) << 32 | i, known_slot[u]);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    slot[u] = home(e[u]);
    if (e[u] != kNoSample) dedup_insert<(1u << kSmallTableLg)>(A.T, static_cast<unsigned long long>(e[u]) << 32 | (kPend | (4u * tid + u)), slot[u]);
  }
  __syncthreads();
  bool twice = false;
#pragma unroll
  for (int u = 0; u < K; ++u) {
    const uint32_t i = u * NT + tid;
    twice = twice || (i < n && A.T.least[known_slot[u]] != i);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const uint32_t q = 4u * tid + u;
    if (q >= positions) continue;
    const uint32_t least = e[u] != kNoSample ? A.T.least[slot[u]] : 0u;
    A.entry[q] = e[u] == kNoSample || least == (kPend | q) ? e[u] : least < kPend ? (kResolved | least) : (kPointer | (least & ~kTagMask));
  }
  return __syncthreads_or(twice ? 1 : 0) != 0;
}

// Blocks of P.tile[h] destinations.  What follows goes on in the same block, which has the nodes in its LDS: its own
// destinations and the new nodes among their samples.  D > 0: the draw of the next hop for them, D its fanout rounded
// up to 8, 16 or 32.  GATHER: the last hop; their feature rows.
template <int D, bool GATHER, int FROM>
__global__ void __launch_bounds__(kSmallThreads) k_small_finish(const SmallLaunch P, int h) {
  constexpr int NT = kSmallThreads;
  constexpr bool kGoesOn = D > 0 || GATHER;
  constexpr int kWords = static_cast<int>(kSmallRecords / 64);
  static_assert(kWords <= NT, "a thread per word of the scan");
  __shared__ unsigned long long first[kWords];  // bit q % 64 of word q / 64: position q is a first appearance
  __shared__ uint32_t before[kWords];           // first appearances before the word
  __shared__ uint32_t off[NT];                  // block offsets of the own destinations
  __shared__ unsigned long long scan[NT / 64];
  __shared__ int32_t ids[kGoesOn ? kSmallNodes : 1];  // the own destinations, then the new nodes
  __shared__ __align__(16) SmallTable<FROM> A;
  __shared__ typename std::conditional<(D > 0 || FROM == kSeeds), DrawLds<NT, 4 * NT>, int>::type S;
  const SmallBatch& B = P.b[small_batch(P)];
  const int n = FROM == kSeeds ? B.num_seeds : small_rows(P, B, h);
  const int i0 = small_block(P) * P.tile[h];
  if (n < 0 || (i0 >= n && i0 > 0)) return;  // the first block also closes an empty hop
  const int rows = n - i0 < P.tile[h] ? n - i0 : P.tile[h];
  const uint32_t d = static_cast<uint32_t>(P.fanouts[h]);
  const uint32_t positions = static_cast<uint32_t>(n) * d;
  const int tid = threadIdx.x;
  const int32_t* rowk = small_rowk(B, h);
  const int32_t* gsrc = small_gsrc(B, h);
  int64_t wrong = SMFG_ST_OK;
  if constexpr (FROM == kSeeds) {
    int stray = 0;
    draw_positions<32, NT>(
        P, B, 0, d, B.seeds, S, 0, n, [&] { stray = 1; },
        [&](int i, uint32_t v, uint32_t) {
          if (i < i0 || i >= i0 + rows) return;
          B.node_ids[i] = static_cast<int32_t>(v);
          if (B.labels && v < P.num_nodes) copy_label(P, B, i, static_cast<int32_t>(v));
        });
    uint32_t g[1];  // a sample per thread
    read_neighbours<NT>(P, DivD(d), S, tid, positions, g);
    A.entry[tid] = g[0];
    if (__syncthreads_or(stray)) wrong = SMFG_ST_SEED_OUT_OF_RANGE;
  }
  const auto samples_of = [&](int i) {
    if constexpr (FROM == kSeeds) return S.deg[i] < d ? S.deg[i] : d;
    else return static_cast<uint32_t>(rowk[i]);
  };
  const uint32_t k = tid < rows ? samples_of(i0 + tid) : 0u;
  if (kGoesOn && tid < rows) ids[tid] = FROM == kSeeds ? B.seeds[i0 + tid] : B.node_ids[i0 + tid];
  // samples of the destinations before the own ones, and of all
  unsigned long long sums = 0;
  for (int i = tid; i < n; i += NT) {
    const unsigned long long x = samples_of(i);
    sums += i < i0 ? (x << 32 | x) : x;
  }
  // bit 31 clear: a first appearance; the four bits of 16 threads make a word
  const auto flag = [&](uint32_t q, const uint4 e) {
    uint32_t nibble = (~e.x >> 31) | (~e.y >> 31) << 1 | (~e.z >> 31) << 2 | (~e.w >> 31) << 3;
    if (q + 4u > positions) nibble &= q < positions ? (1u << (positions - q)) - 1u : 0u;
    unsigned long long bits = static_cast<unsigned long long>(nibble) << (4 * (tid & 15));
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) bits |= __shfl_xor(bits, o, 64);
    if ((tid & 15) == 0 && q < positions) first[q >> 6] = bits;
  };
  if constexpr (FROM == kSettled) {
    constexpr int U = 4;
    for (uint32_t q0 = tid * 4u; q0 < ((positions + 63u) & ~63u); q0 += NT * 4u * U) {
      uint4 e[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t q = q0 + u * NT * 4u;
        e[u] = q < positions ? *reinterpret_cast<const uint4*>(gsrc + q) : make_uint4(kNoSample, kNoSample, kNoSample, kNoSample);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) flag(q0 + u * NT * 4u, e[u]);
    }
  } else {
    const uint32_t q = 4u * tid;
    const uint4 x = q >= positions ? make_uint4(kNoSample, kNoSample, kNoSample, kNoSample)
                    : *reinterpret_cast<const uint4*>(FROM == kSeeds ? reinterpret_cast<const int32_t*>(A.entry) + q : gsrc + q);
    const uint32_t e[4] = {x.x, q + 1u < positions ? x.y : kNoSample, q + 2u < positions ? x.z : kNoSample, q + 3u < positions ? x.w : kNoSample};
    int stray = 0;
    const bool twice = settle_in_block<NT>(A, static_cast<uint32_t>(n), positions, e, [&](uint32_t i) {
      if constexpr (FROM == kSeeds) return S.node[i];
      const uint32_t v = static_cast<uint32_t>(B.node_ids[i]);
      if (h == 0 && v >= P.num_nodes) stray = 1;
      return v;
    });
    if (FROM == kDrawn && h == 0 && __syncthreads_or(stray)) wrong = SMFG_ST_SEED_OUT_OF_RANGE;
    if (twice && wrong == SMFG_ST_OK) wrong = SMFG_ST_DUPLICATE_SEED;
    flag(q, q < positions ? *reinterpret_cast<const uint4*>(A.entry + q) : make_uint4(kNoSample, kNoSample, kNoSample, kNoSample));
  }
  unsigned long long total, all;
  block_exscan<NT>(sums, scan, all);
  __syncthreads();
  const uint32_t words = (positions + 63u) >> 6;
  const uint32_t mine = static_cast<uint32_t>(tid) < words ? static_cast<uint32_t>(__popcll(first[tid])) : 0u;
  const unsigned long long pre = block_exscan<NT>(static_cast<unsigned long long>(k) << 32 | mine, scan, total);
  const uint32_t edges = static_cast<uint32_t>(all), nodes = static_cast<uint32_t>(n) + static_cast<uint32_t>(total);
  const uint32_t own = static_cast<uint32_t>(all >> 32) + static_cast<uint32_t>(pre >> 32);
  if (tid < kWords) before[tid] = static_cast<uint32_t>(n) + static_cast<uint32_t>(pre);
  off[tid] = own;
  const bool nodes_fit = nodes <= static_cast<uint32_t>(B.node_capacity);
  const bool edges_fit = edges <= static_cast<uint32_t>(B.edge_capacity[h]);
  const bool bad_seeds = wrong != SMFG_ST_OK;  // as elsewhere, nothing but the seeds is counted then
  if (wrong == SMFG_ST_OK) wrong = !nodes_fit ? SMFG_ST_NODE_CAPACITY : !edges_fit ? SMFG_ST_EDGE_CAPACITY : SMFG_ST_OK;
  if (tid == 0 && i0 == 0) {
    if constexpr (FROM == kSeeds) {  // starts the counts
      for (int q = 0; q < 2 * P.L + 2; ++q)
        B.counts[q] = q == 0 ? n : q == 2 * P.L + 1 ? wrong : bad_seeds ? 0 : q == 1 ? nodes : q == P.L + 1 ? edges : 0;
    } else {
      if (!bad_seeds) {
        B.counts[P.L + 1 + h] = edges;
        B.counts[h + 1] = nodes;
      }
      if (wrong != SMFG_ST_OK) set_status(B, P.L, wrong);
    }
    if (wrong == SMFG_ST_OK) B.blk_indptr[h][n] = static_cast<int32_t>(edges);
  }
  if (wrong != SMFG_ST_OK) return;
  if (tid < rows) B.blk_indptr[h][i0 + tid] = static_cast<int32_t>(own);
  __syncthreads();
  const DivD div(d);
  const uint32_t pos0 = static_cast<uint32_t>(i0) * d;
  const uint32_t own_cnt = static_cast<uint32_t>(rows) * d;
  const auto id_of = [&](uint32_t q) { return before[q >> 6] + static_cast<uint32_t>(__popcll(first[q >> 6] & ((1ull << (q & 63u)) - 1ull))); };
  const uint32_t first_new = own_cnt > 0u ? id_of(pos0) : 0u;
  for (uint32_t idx = tid; idx < own_cnt; idx += NT) {
    uint32_t e;
    if constexpr (FROM == kSettled) e = static_cast<uint32_t>(gsrc[pos0 + idx]);
    else e = A.entry[pos0 + idx];
    if (e == kNoSample) continue;
    uint32_t r, s, local;
    div.split(idx, r, s);
    if ((e & kResolved) == 0u) {
      local = id_of(pos0 + idx);
      B.node_ids[local] = static_cast<int32_t>(e);
      if (kGoesOn) ids[static_cast<uint32_t>(rows) + local - first_new] = static_cast<int32_t>(e);
    } else if ((e & kPointer) == kPointer) {
      local = id_of(e & ~kPointer);  // a pointer always names a first appearance
    } else {
      local = e & ~kPointer;
    }
    B.blk_indices[h][off[r] + s] = static_cast<int32_t>(local);
  }
  if constexpr (kGoesOn) {
    __syncthreads();
    // id_of counts the bits below a position, so the end of the own positions tells how many new nodes they have
    const uint32_t end = pos0 + own_cnt;
    const uint32_t after = own_cnt == 0u ? first_new : end < positions ? id_of(end) : nodes;
    const int known = rows, count = rows + static_cast<int>(after - first_new);
    const auto index_of = [&](int j) { return j < known ? i0 + j : static_cast<int>(first_new) + j - known; };
    if constexpr (D > 0) {
      const uint32_t next_d = static_cast<uint32_t>(P.fanouts[h + 1]);
      int32_t* next_gsrc = small_gsrc(B, h + 1);
      int32_t* next_rowk = small_rowk(B, h + 1);
      const int most = 4 * NT / static_cast<int>(draw_stride(next_d)), turn = most < NT ? most : NT;
      const DivD next_div(next_d);
      for (int j0 = 0; j0 < count; j0 += turn) {
        const int here = count - j0 < turn ? count - j0 : turn;
        draw_positions<D, NT>(P, B, h + 1, next_d, ids, S, j0, here, [] {},
                              [&](int j, uint32_t, uint32_t samples) { next_rowk[index_of(j)] = static_cast<int32_t>(samples); });
        const uint32_t cnt = static_cast<uint32_t>(here) * next_d;
        for (uint32_t base = tid; base < cnt; base += 2u * NT) {
          uint32_t g[2];
          read_neighbours<NT>(P, next_div, S, base, cnt, g);
#pragma unroll
          for (int u = 0; u < 2; ++u)
            if (base + u * NT < cnt) {
              uint32_t r, s;
              next_div.split(base + u * NT, r, s);
              next_gsrc[static_cast<uint32_t>(index_of(j0 + static_cast<int>(r))) * next_d + s] = static_cast<int32_t>(g[u]);
            }
        }
        __syncthreads();  // the next turn's rows replace these
      }
    }
    if constexpr (GATHER) {
      const uint32_t vecs = static_cast<uint32_t>((P.row_bytes + 15) / 16), all = static_cast<uint32_t>(count) * vecs;
      for (uint32_t base = tid; base < all; base += 4u * NT) {
        u32x4u v[4];
        uint8_t* to[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t q = base + u * NT < all ? base + u * NT : all - 1u;
          const uint32_t j = q / vecs;
          int64_t id = ids[j];
          if (id < 0 || id >= P.num_nodes) id = 0;  // no id can cause a read outside x
          // a row's last vector ends with it and may overlap the one before (see AnyRow)
          const int64_t byte = q - j * vecs == vecs - 1u ? P.row_bytes - 16 : static_cast<int64_t>(q - j * vecs) * 16;
          v[u] = *reinterpret_cast<const u32x4u*>(P.feat + id * P.row_stride + byte);
          to[u] = B.features + static_cast<int64_t>(index_of(static_cast<int>(j))) * P.row_bytes + byte;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (base + u * NT < all) *reinterpret_cast<u32x4u*>(to[u]) = v[u];
      }
    }
  }
}

}  // namespace smfg_dev

#endif  // SMFG_KERNELS_SMALL_H_
