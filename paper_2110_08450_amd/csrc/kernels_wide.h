// libsmfg wide path: fanouts above SMFG_MAX_FANOUT and SMFG_FANOUT_ALL, samples at exact block offsets.
// count_rows / scan_count_tiles fix the offsets; then either the table strategy (sample_wide<true>,
// flag_flat, scan_flat_tiles, assemble_flat) or the partition strategy (sample_wide<false>, part_flat,
// [split_buckets], dedup_buckets, flag_flat_part, scan_flat_tiles,
// assemble_flat_part) turns the samples into local ids.
#ifndef SMFG_KERNELS_WIDE_H_
#define SMFG_KERNELS_WIDE_H_

#include "device_common.h"
#include "kernels_part.h"

namespace smfg_dev {

// Samples sit at their exact block offsets (pos = block indptr[i] + s), so a count + scan pass
// comes first and the later passes walk the samples flat, four consecutive samples per thread.
constexpr int kWideTile = 4 * kThreads;  // samples per flat tile

// Degree, sample count and row start per destination; in-tile scan of the sample counts.
__global__ void __launch_bounds__(kThreads) k_count_rows(const Launch P) {
  __shared__ unsigned long long lds[kThreads / 64];
  const BatchCtx& B = P.b[batch_of_block(P)];
  if (block_has_status(B, P.L)) return;
  const int n = static_cast<int>(B.counts[P.h]);
  const int d = P.d;
  const int tiles = (n + kTileRows - 1) / kTileRows;
  for (int tile = block_in_batch(P); tile < tiles; tile += blocks_per_batch(P)) {
    const int i = tile * kTileRows + threadIdx.x;
    uint32_t k = 0;
    if (i < n) {
      const int32_t id = B.node_ids[i];
      int64_t a = 0;
      uint32_t deg = 0;
      // the seeds are caller data: none may index the graph unchecked (later hops only hold
      // neighbour ids read from the graph)
      if (P.h == 0 && (id < 0 || static_cast<int64_t>(id) >= P.num_nodes)) {
        set_status(B, P.L, SMFG_ST_SEED_OUT_OF_RANGE);
      } else {
        a = P.indptr[id];
        deg = static_cast<uint32_t>(P.indptr[id + 1] - a);
      }
      k = (d < 0 || deg <= static_cast<uint32_t>(d)) ? deg : static_cast<uint32_t>(d);
      B.rowstart[i] = a;
      B.rowdeg[i] = deg;
      B.rowk[i] = static_cast<int32_t>(k);
    }
    unsigned long long total;
    const unsigned long long pre = block_exscan(static_cast<unsigned long long>(k), lds, total);
    if (i < n) B.rowoff[i] = static_cast<int32_t>(pre);
    if (threadIdx.x == 0) B.tile_sums[tile] = total;
    __syncthreads();
  }
}

// Exclusive scan of the per-tile sample counts; E_h and its capacity checks.
__global__ void __launch_bounds__(kTileScanThreads) k_scan_count_tiles(const Launch P) {
  const BatchCtx& B = P.b[batch_of_block(P)];
  if (block_has_status(B, P.L)) return;
  const int n = static_cast<int>(B.counts[P.h]);
  const unsigned long long edges = scan_tile_sums(B.tile_sums, static_cast<uint32_t>((n + kTileRows - 1) / kTileRows));
  if (threadIdx.x == 0) {
    const bool fits = edges <= static_cast<unsigned long long>(B.edge_capacity) &&
                      edges <= static_cast<unsigned long long>(B.lostto_entries);
    B.counts[P.L + 1 + P.h] = static_cast<int64_t>(edges);
    if (fits) B.blk_indptr[n] = static_cast<int32_t>(edges);
    else set_status(B, P.L, SMFG_ST_EDGE_CAPACITY);
  }
}

// A wave takes up to kWideRows consecutive destinations (fewer when the hop has fewer destinations
// than that per wave of the grid: a hop of few, long rows then still spreads over the chip): lane l
// first fetches the row record of destination l (start, degree, sample count, block offset:
// coalesced, once per group of rows), then the wave walks the rows, lane l of round r owning slot
// s = 64 r + l: first the rows that are one plain round (whole row taken, at most 64 samples; several
// in flight), then the others one by one - a row taken whole kWideCopyRounds rounds at a time, a
// row with drawn positions after Floyd's rule has settled them in the wave's part of the LDS
// (per wave two arrays of the fanout rounded up to 64 words and a hash table of at least twice that, sized
// by the launch; none for SMFG_FANOUT_ALL, where nothing is drawn).  INSERT: the sample goes into
// the dedup table at once (table strategy); else only its node id is stored (partition strategy).
constexpr int kWideRows = 16;
constexpr int kWideCopyRounds = 8;
constexpr uint32_t wide_lds_words(int d) { return d < 0 ? 0u : (static_cast<uint32_t>(d) + 63u) & ~63u; }
constexpr uint32_t wide_table_words(int d) {
  uint32_t w = d < 0 ? 0u : 128u;
  while (w < 2u * wide_lds_words(d)) w *= 2u;
  return w;
}
constexpr size_t wide_lds_bytes(int d) {
  return sizeof(uint32_t) * (kThreads / 64) * (2 * wide_lds_words(d) + wide_table_words(d));
}
static_assert(wide_lds_bytes(SMFG_MAX_WIDE_FANOUT) <= 65536, "LDS of a block");

// What happens to a drawn sample: recorded (partition strategy), or also inserted into the dedup
// table right away (table strategy; see k_sample_insert for the three cases).
template <bool INSERT>
__device__ __forceinline__ void wide_emit(const Launch& P, const BatchCtx& B, uint32_t g, uint32_t pos) {
  if (INSERT) {
    uint32_t slot;
    bool full;
    const uint32_t prev = table_insert_min(B, g, kPend | pos, slot, full);
    if (full) set_status(B, P.L, SMFG_ST_TABLE_FULL);
    uint32_t e = prev;
    if (prev > (kPend | pos)) {
      e = kSlot | slot;
      if (prev != 0xFFFFFFFFu) B.lostto[prev & ~kTagMask] = kPend | pos;
    }
    B.ent[pos] = e;
  }
  B.gsrc[pos] = static_cast<int32_t>(g);
}

// Floyd's subset algorithm for one destination with k > 32 slots, by one wave (lane l owns slots
// l, l + 64, ...).  Slot s draws t_s in [0, j_s], j_s = deg - k + s, and takes t_s unless an
// earlier slot holds that position, else j_s.  Settled without walking the slots one by one:
// an earlier slot holds t_s exactly if (a) an earlier slot drew the same value - whether that slot
// kept it or not, the value was in the set by then - or (b) t_s is the j of an earlier slot q (only
// q = t_s - (deg - k) can be) and slot q took its j, i.e. was itself refused.  (a) needs no other
// slot's outcome; (b) refers to one earlier slot.  So every slot is refused outright, accepted
// outright, or "as slot q": chains of such references are shortcut by pointer jumping, at most
// log2 k + 1 passes.  (a) is settled by a hash table that keeps the first slot of every value; a scan over
// all earlier draws, four per LDS read, kept the wave issuing k^2 / 256 rounds of compares (k_sample_wide
// of a launch set of four batches with fanouts (100, 100) 136 us against 88 us, a call of 1024
// destinations x 1000 185 against 84 us, (40, 40) 203 against 200 us).  `draws` keeps the t_s, `picks` the
// states and in the end the positions p_s, `table` the first slots (all LDS, private to the wave).
__device__ __forceinline__ void floyd_positions(const Launch& P, const BatchCtx& B, uint32_t v, uint32_t deg,
                                                uint32_t k, uint32_t* picks, uint32_t* draws, uint32_t* table,
                                                uint32_t table_mask) {
  constexpr uint32_t kNone = 0xFFFFFFFFu;
  constexpr uint32_t kKnown = 0x80000000u, kRefused = 0x40000000u, kRefMask = 0x3FFFFFFFu;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t j0 = deg - k;
  for (uint32_t q = lane; q <= table_mask; q += 64u) table[q] = kNone;
  // a lane draws for four slots at a time; the arrays are rounded up to a multiple of 64 words, and what
  // lies at or beyond slot k is not looked at
  for (uint32_t s = 4u * lane; s < k; s += 4u * 64u) {
    uint32_t w[4];
    philox_block(v, static_cast<uint32_t>(P.h), s >> 2, B.key0, B.key1, w);
    uint4 t;  // an index in [0, j_s] each
    t.x = __umulhi(w[0], j0 + s + 1u);
    t.y = __umulhi(w[1], j0 + s + 2u);
    t.z = __umulhi(w[2], j0 + s + 3u);
    t.w = __umulhi(w[3], j0 + s + 4u);
    *reinterpret_cast<uint4*>(draws + s) = t;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (uint32_t s = lane; s < k; s += 64u) {
    const uint32_t t = draws[s];
    uint32_t at = (t * kPartHash) >> 16;
    for (;;) {  // ends: more words than slots, and a word once taken keeps its value
      at &= table_mask;
      const uint32_t old = atomicCAS(&table[at], kNone, s);
      if (old == kNone) break;
      if (draws[old] == t) {
        atomicMin(&table[at], s);
        break;
      }
      ++at;
    }
    picks[s] = at;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (uint32_t s = lane; s < k; s += 64u) {
    const uint32_t t = draws[s];
    const bool dup = table[picks[s]] < s;
    const bool refers = !dup && t >= j0 && t - j0 < s;
    picks[s] = dup ? (kKnown | kRefused) : (refers ? t - j0 : kKnown);
  }
  for (;;) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    bool open = false;
    for (uint32_t s = lane; s < k; s += 64u) {
      const uint32_t st = picks[s];
      if ((st & kKnown) == 0u) {
        // as slot q: take its outcome if it has one, else refer to what it refers to (a word is read
        // and written whole, and a state only ever moves forward along its chain, so the order in
        // which lanes get here does not matter)
        const uint32_t sq = picks[st & kRefMask];
        picks[s] = (sq & kKnown) ? sq : (sq & kRefMask);
        open = open || (sq & kKnown) == 0u;
      }
    }
    if (__ballot(open) == 0ull) break;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (uint32_t s = lane; s < k; s += 64u) picks[s] = (picks[s] & kRefused) ? j0 + s : draws[s];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

template <bool INSERT>
__global__ void __launch_bounds__(kThreads) k_sample_wide(const Launch P) {
  extern __shared__ __align__(16) uint32_t wide_lds[];
  const BatchCtx& B = P.b[batch_of_block(P)];
  if (__any(status_of(B, P.L) != 0)) return;  // whole waves only: the lanes below cooperate
  const int n = static_cast<int>(B.counts[P.h]);
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const uint32_t words = wide_lds_words(P.d), table_words = wide_table_words(P.d);
  uint32_t* draws = wide_lds + wave * (2 * words + table_words);
  uint32_t* picks = draws + words;
  uint32_t* table = picks + words;
  const int waves_total = blocks_per_batch(P) * (kThreads / 64);
  int per = (n + waves_total - 1) / waves_total;  // destinations per wave and turn
  per = per < 1 ? 1 : (per > kWideRows ? kWideRows : per);
  for (int i0 = (block_in_batch(P) * (kThreads / 64) + wave) * per; i0 < n; i0 += waves_total * per) {
    const int il = i0 + lane;
    uint32_t v_l = 0, deg_l = 0, k_l = 0, base_l = 0, a_lo = 0, a_hi = 0;
    if (lane < per && il < n) {
      v_l = static_cast<uint32_t>(B.node_ids[il]);
      const int64_t a = B.rowstart[il];
      a_lo = static_cast<uint32_t>(a);
      a_hi = static_cast<uint32_t>(static_cast<uint64_t>(a) >> 32);
      deg_l = static_cast<uint32_t>(B.rowdeg[il]);
      k_l = static_cast<uint32_t>(B.rowk[il]);
      base_l = static_cast<uint32_t>(B.tile_sums[il / kTileRows]) + static_cast<uint32_t>(B.rowoff[il]);
      B.blk_indptr[il] = static_cast<int32_t>(base_l);
    }
    const int rows = n - i0 < per ? n - i0 : per;
    static_assert(kWideRows % 4 == 0 && kWideRows <= 64, "rows are walked four at a time, a lane per row record");
    for (int r0 = 0; r0 < rows; r0 += 4) {  // lanes beyond the last row hold k = 0
      uint32_t g[4], pos[4];
      bool on[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = r0 + u;
        const int64_t a = static_cast<int64_t>((static_cast<uint64_t>(__shfl(a_hi, r, 64)) << 32) | __shfl(a_lo, r, 64));
        const uint32_t deg = __shfl(deg_l, r, 64);
        const uint32_t k = __shfl(k_l, r, 64);
        pos[u] = __shfl(base_l, r, 64) + static_cast<uint32_t>(lane);
        on[u] = deg == k && k <= 64u && static_cast<uint32_t>(lane) < k;
        g[u] = on[u] ? static_cast<uint32_t>(__builtin_nontemporal_load(P.indices + (a + lane))) : 0u;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (on[u]) wide_emit<INSERT>(P, B, g[u], pos[u]);
    }
    for (int r = 0; r < rows; ++r) {
      const uint32_t v = __shfl(v_l, r, 64);
      const int64_t a = static_cast<int64_t>((static_cast<uint64_t>(__shfl(a_hi, r, 64)) << 32) | __shfl(a_lo, r, 64));
      const uint32_t deg = __shfl(deg_l, r, 64);
      const uint32_t k = __shfl(k_l, r, 64);
      const uint32_t base = __shfl(base_l, r, 64);
      const bool floyd = deg > k;  // only then are positions drawn (k = fanout <= SMFG_MAX_WIDE_FANOUT)
      if (!floyd && k <= 64u) continue;  // done above
      if (!floyd) {  // the whole row in CSR order; every read of a turn leaves before a result is used
        for (uint32_t s0 = static_cast<uint32_t>(lane); s0 < k; s0 += 64u * kWideCopyRounds) {
          uint32_t gv[kWideCopyRounds];
#pragma unroll
          for (int u = 0; u < kWideCopyRounds; ++u) {
            const uint32_t sl = s0 + 64u * u;
            gv[u] = sl < k ? static_cast<uint32_t>(__builtin_nontemporal_load(P.indices + (a + sl))) : 0u;
          }
#pragma unroll
          for (int u = 0; u < kWideCopyRounds; ++u) {
            const uint32_t sl = s0 + 64u * u;
            if (sl < k) wide_emit<INSERT>(P, B, gv[u], base + sl);
          }
        }
        continue;
      }
      floyd_positions(P, B, v, deg, k, picks, draws, table, table_words - 1u);
      for (uint32_t s0 = 0; s0 < k; s0 += 128) {  // two rounds at a time
        const uint32_t sa = s0 + static_cast<uint32_t>(lane), sb = sa + 64u;
        uint32_t ga = 0, gb = 0;
        if (sa < k) ga = static_cast<uint32_t>(__builtin_nontemporal_load(P.indices + (a + picks[sa])));
        if (sb < k) gb = static_cast<uint32_t>(__builtin_nontemporal_load(P.indices + (a + picks[sb])));
        if (sa < k) wide_emit<INSERT>(P, B, ga, base + sa);
        if (sb < k) wide_emit<INSERT>(P, B, gb, base + sb);
      }
      // the next row's draws must not overwrite picks a lane has yet to read
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// ---- partition strategy over exact offsets ----------------------------------------------------
// The records of a hop as one stream: element e < n is known node e, element n + pos the sample
// at position pos.
__device__ __forceinline__ unsigned long long flat_record(const BatchCtx& B, uint32_t e, uint32_t n) {
  if (e < n) return (static_cast<unsigned long long>(static_cast<uint32_t>(B.node_ids[e])) << 32) | e;
  const uint32_t pos = e - n;
  return (static_cast<unsigned long long>(static_cast<uint32_t>(B.gsrc[pos])) << 32) | (kPend | pos);
}

// The stream's segments, sorted by bucket.
constexpr int kFlatThreads = kThreads;
__global__ void __launch_bounds__(kFlatThreads) k_part_flat(const Launch P) {
  constexpr int NT = kFlatThreads;
  __shared__ unsigned long long stage[kSegMax];
  __shared__ uint32_t scan[NT / 64];
  extern __shared__ uint32_t cnt[];  // offs_stride / 2 words
  const BatchCtx& B = P.b[batch_of_block(P)];
  if (block_has_status(B, P.L)) return;
  const uint32_t n = static_cast<uint32_t>(B.counts[P.h]);
  const uint32_t total_e = n + static_cast<uint32_t>(B.counts[P.L + 1 + P.h]);
  const int lgB = hop_shape(P, B).lgB;
  const Segments segs = hop_segments(P, B);
  for (uint32_t seg = static_cast<uint32_t>(block_in_batch(P)); seg < segs.count; seg += static_cast<uint32_t>(blocks_per_batch(P))) {
    const uint32_t e0 = seg * segs.cap;
    const uint32_t e1 = total_e - e0 < segs.cap ? total_e : e0 + segs.cap;
    unsigned long long r[kSegPer];
    uint32_t rk[kSegPer];
#pragma unroll
    for (int u = 0; u < kSegPer; ++u) {
      const uint32_t e = e0 + u * NT + threadIdx.x;
      r[u] = e < e1 ? flat_record(B, e, n) : kEmpty;
    }
    __syncthreads();  // the previous segment has been written out
    for (uint32_t b = threadIdx.x; b < offs_stride(lgB) / 2u; b += NT) cnt[b] = 0u;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSegPer; ++u) rk[u] = r[u] != kEmpty ? count_packed(cnt, part_bucket(static_cast<uint32_t>(r[u] >> 32), lgB)) : 0u;
    __syncthreads();
    segment_offsets<NT>(cnt, lgB, B.hist + static_cast<size_t>(seg) * offs_stride(lgB), scan);
#pragma unroll
    for (int u = 0; u < kSegPer; ++u)
      if (r[u] != kEmpty) stage[packed(cnt, part_bucket(static_cast<uint32_t>(r[u] >> 32), lgB)) + rk[u]] = r[u];
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < e1 - e0; t += NT) B.rec[e0 + t] = stage[t];
  }
}

// flag_flat for the entries dedup_buckets leaves (a sample whose gsrc entry still is a node id is a
// first appearance).  Instead of a rank per sample, every group of 64 consecutive samples gets one
// 16-byte record: the 64 first-appearance bits and the number of new nodes of the tile before the
// group.  For a hop of millions of samples that is about a megabyte, which stays in the L2, so the
// lookups of the samples that repeat a node (scattered over the hop) do not go to memory.
// A wave takes four groups one after the other, a sample per lane, so that its reads are consecutive and a ballot is
// a group's bits.  Bound by the stream of entries and, in launches with far more blocks than tiles, by the blocks that leave:
// 9.7 M samples of four batches 18.5 -> 17.6 us, 5.5 M of one 9.9 -> 9.3, against four consecutive samples per thread.
__global__ void __launch_bounds__(kThreads) k_flag_flat_part(const Launch P) {
  constexpr int kWaves = kThreads / 64;
  __shared__ uint32_t lds[2][kWaves];
  const BatchCtx& B = P.b[batch_of_block(P)];
  if (block_has_status(B, P.L)) return;
  const uint32_t E = static_cast<uint32_t>(B.counts[P.L + 1 + P.h]);
  const uint32_t tiles = (E + kWideTile - 1) / kWideTile;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int turn = 0;  // a wave writes the sums of the next tile while others may still read the present one's
  for (uint32_t tile = block_in_batch(P); tile < tiles; tile += blocks_per_batch(P), turn ^= 1) {
    const uint32_t p0 = tile * kWideTile + static_cast<uint32_t>(wave) * 256u;
    uint32_t e[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t pos = p0 + u * 64 + lane;
      e[u] = pos < E ? static_cast<uint32_t>(B.gsrc[pos]) : kResolved;
    }
    unsigned long long own = 0;  // lane u < 4: the bits of group u, and the new nodes of the wave before it
    uint32_t before = 0, sum = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const unsigned long long bits = __ballot((e[u] & kResolved) == 0u);
      if (lane == u) {
        own = bits;
        before = sum;
      }
      sum += static_cast<uint32_t>(__popcll(bits));
    }
    if (lane == 0) lds[turn][wave] = sum;
    __syncthreads();
    uint32_t total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      if (w < wave) before += lds[turn][w];
      total += lds[turn][w];
    }
    if (lane < 4 && p0 + static_cast<uint32_t>(lane) * 64u < E)
      B.grp[(p0 >> 6) + lane] = make_uint4(static_cast<uint32_t>(own), static_cast<uint32_t>(own >> 32), before, 0u);
    if (threadIdx.x == 0) B.stile_sums[tile] = total;
  }
}

// New nodes of the hop before the sample at position q (a first appearance or not).
__device__ __forceinline__ uint32_t flat_rank(const uint4 g, uint32_t tile_before, uint32_t q) {
  const unsigned long long bits = (static_cast<unsigned long long>(g.y) << 32) | g.x;
  return tile_before + g.z + __popcll(bits & ((1ull << (q & 63u)) - 1ull));
}

// assemble_flat for those entries, a wave's samples as in flag_flat_part: its reads and writes are consecutive.
// What is left is bound by the scattered lookups of what pointers name: 9.7 M samples of four batches 43 -> 34 us, 5.5 M of one
// 28 -> 23.5, against four consecutive samples per thread, whose stores took every fourth word of a line.
__global__ void __launch_bounds__(kThreads) k_assemble_flat_part(const Launch P) {
  const BatchCtx& B = P.b[batch_of_block(P)];
  if (status_of(B, P.L) != 0) return;
  const uint32_t n = static_cast<uint32_t>(B.counts[P.h]);
  const uint32_t E = static_cast<uint32_t>(B.counts[P.L + 1 + P.h]);
  const uint32_t tiles = (E + kWideTile - 1) / kWideTile;
  for (uint32_t tile = block_in_batch(P); tile < tiles; tile += blocks_per_batch(P)) {
    const uint32_t tpre = static_cast<uint32_t>(B.stile_sums[tile]);
    const uint32_t p0 = tile * kWideTile + (threadIdx.x >> 6) * 256u + (threadIdx.x & 63u);
    uint4 own[4];
    uint32_t e[4], q[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t pos = p0 + u * 64;
      e[u] = pos < E ? static_cast<uint32_t>(B.gsrc[pos]) : kResolved;
      own[u] = B.grp[(pos < E ? pos : tile * kWideTile) >> 6];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) q[u] = (e[u] & kPointer) == kPointer ? (e[u] & ~kPointer) : tile * kWideTile;
    // what the pointers name is fetched for all four samples before any is used
    uint4 qg[4];
    uint32_t qtile[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      qg[u] = B.grp[q[u] >> 6];
      qtile[u] = static_cast<uint32_t>(B.stile_sums[q[u] / kWideTile]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t pos = p0 + u * 64;
      if (pos >= E) continue;
      uint32_t local;
      if ((e[u] & kResolved) == 0u) {  // first appearance
        local = n + flat_rank(own[u], tpre, pos);
        B.node_ids[local] = static_cast<int32_t>(e[u]);
      } else if ((e[u] & kPointer) == kPointer) {
        local = n + flat_rank(qg[u], qtile[u], q[u]);  // a pointer always names a first appearance
      } else {
        local = e[u] & ~kPointer;
      }
      B.blk_indices[pos] = static_cast<int32_t>(local);
    }
  }
}

// ---- table strategy over exact offsets ---------------------------------------------------------
// Flat over the samples: first appearances, their in-tile ranks, per-tile totals.
__global__ void __launch_bounds__(kThreads) k_flag_flat(const Launch P) {
  __shared__ unsigned long long lds[kThreads / 64];
  const BatchCtx& B = P.b[batch_of_block(P)];
  if (block_has_status(B, P.L)) {
    for (int64_t q = static_cast<int64_t>(block_in_batch(P)) * kThreads + threadIdx.x; q < B.lostto_entries;
         q += static_cast<int64_t>(blocks_per_batch(P)) * kThreads)
      B.lostto[q] = 0u;
    return;
  }
  const uint32_t E = static_cast<uint32_t>(B.counts[P.L + 1 + P.h]);
  const uint32_t tiles = (E + kWideTile - 1) / kWideTile;
  for (uint32_t tile = block_in_batch(P); tile < tiles; tile += blocks_per_batch(P)) {
    const uint32_t p0 = tile * kWideTile + threadIdx.x * 4;
    uint32_t first[4];
    uint32_t mine = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      first[u] = 0;
      const uint32_t pos = p0 + u;
      if (pos < E) {
        const uint32_t lost = B.lostto[pos];
        if (lost != 0u) {
          B.ent[pos] = lost;
          B.lostto[pos] = 0u;
        } else {
          first[u] = (B.ent[pos] & kTagMask) == kSlot ? 1u : 0u;
        }
      }
      mine += first[u];
    }
    unsigned long long total;
    uint32_t pre = static_cast<uint32_t>(block_exscan(static_cast<unsigned long long>(mine), lds, total));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (p0 + u < E) B.rank[p0 + u] = pre;
      pre += first[u];
    }
    if (threadIdx.x == 0) B.stile_sums[tile] = total;
    __syncthreads();
  }
}

// Exclusive scan of the per-tile counts of new nodes; n_{h+1} and its capacity check.
__global__ void __launch_bounds__(kTileScanThreads) k_scan_flat_tiles(const Launch P) {
  const BatchCtx& B = P.b[batch_of_block(P)];
  if (block_has_status(B, P.L)) return;
  const int n = static_cast<int>(B.counts[P.h]);
  const uint32_t E = static_cast<uint32_t>(B.counts[P.L + 1 + P.h]);
  const unsigned long long fresh = scan_tile_sums(B.stile_sums, (E + kWideTile - 1) / kWideTile);
  if (threadIdx.x == 0) {
    const int64_t nodes = static_cast<int64_t>(n) + static_cast<int64_t>(fresh);
    B.counts[P.h + 1] = nodes;
    if (nodes > B.node_capacity) set_status(B, P.L, SMFG_ST_NODE_CAPACITY);
  }
}

// Flat over the samples: final local ids -> block indices; first appearances publish themselves.
__global__ void __launch_bounds__(kThreads) k_assemble_flat(const Launch P) {
  const BatchCtx& B = P.b[batch_of_block(P)];
  if (status_of(B, P.L) != 0) return;
  const uint32_t n = static_cast<uint32_t>(B.counts[P.h]);
  const uint32_t E = static_cast<uint32_t>(B.counts[P.L + 1 + P.h]);
  const bool last = P.h == P.L - 1;
  const uint32_t tiles = (E + kWideTile - 1) / kWideTile;
  for (uint32_t tile = block_in_batch(P); tile < tiles; tile += blocks_per_batch(P)) {
    const uint32_t tpre = n + static_cast<uint32_t>(B.stile_sums[tile]);
    const uint32_t p0 = tile * kWideTile + threadIdx.x * 4;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t pos = p0 + u;
      if (pos >= E) continue;
      const uint32_t e = B.ent[pos];
      const uint32_t tag = e & kTagMask;
      uint32_t local = e;
      if (tag == kSlot) {
        local = tpre + B.rank[pos];
        const uint32_t g = static_cast<uint32_t>(B.gsrc[pos]);
        B.node_ids[local] = static_cast<int32_t>(g);
        if (!last) B.table[e & ~kTagMask] = (static_cast<uint64_t>(g) << 32) | local;
      } else if (tag != 0u) {  // kPend: same node as the sample at position q < pos
        uint32_t q = e & ~kTagMask;
        for (;;) {
          const uint32_t eq = B.ent[q];
          if ((eq & kTagMask) == kSlot) {  // q is the node's first appearance
            local = n + static_cast<uint32_t>(B.stile_sums[q / kWideTile]) + B.rank[q];
            break;
          }
          const uint32_t nxt = eq & ~kTagMask;  // strictly smaller position, or the scratch was disturbed
          if (nxt >= q) {
            set_status(B, P.L, SMFG_ST_INTERNAL);
            local = 0u;
            break;
          }
          q = nxt;
        }
      }
      B.blk_indices[pos] = static_cast<int32_t>(local);
    }
  }
}

}  // namespace smfg_dev

#endif  // SMFG_KERNELS_WIDE_H_
