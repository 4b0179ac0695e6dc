// libsmfg wide path: fanouts above SMFG_MAX_FANOUT and SMFG_FANOUT_ALL, samples at exact block offsets.
// count_rows counts the samples; then either the table strategy (sample_wide<true>,
// flag_flat, scan_flat_tiles, assemble_flat) or the partition strategy (sample_wide<false>, part_flat,
// [split_buckets], dedup_buckets, flag_flat_part, assemble_flat_part) turns them into local ids.  No launch of the latter only
// scans: two hops of fanouts (100, 100), four batches, 772 -> 742 us without the scans of either side and without k_begin, whole
// neighbourhoods of two hops 401 -> 381, two hops of some 100 samples 79 -> 64.
#ifndef SMFG_KERNELS_WIDE_H_
#define SMFG_KERNELS_WIDE_H_

#include "device_common.h"
#include "kernels_part.h"

namespace smfg_dev {

// Samples sit at their exact block offsets (pos = block indptr[i] + s), so a count + scan pass
// comes first and the later passes walk the samples flat, four consecutive samples per thread.
constexpr int kWideTile = 4 * kThreads;  // samples per flat tile

// The block offset of a destination is rowoff, the samples of its tile of kTileRows before it, and the sums of the tiles before
// that.  The first wave of a block of k_sample_wide adds these up while the row records are on their way: up to kDirectTiles totals, or,
// in hops of more destinations (131 K), totals of kSuperTiles tiles, which k_count_rows adds to with one atomic per tile, and the last
// few.  A launch in between that scanned the totals took 4.6 us, whatever a hop had.  With every wave adding up for itself the
// kernel was bound by instruction issue (28 K destinations x 100 in each of four batches 85 -> 104 us).
// The totals of tiles of tiles are in the memory of rowmn and hist, of which neither holds anything between two hops; the end of a
// hop clears them for the next.  A first hop has none, nor has one behind small hops, whose nodes are too few.
constexpr uint32_t kDirectTiles = 512, kSuperTiles = 64;
static_assert((kSmallRecords + kTileRows - 1) / kTileRows <= kDirectTiles, "nodes known after small hops");
__device__ __forceinline__ bool has_supers(const Launch& P, uint32_t tiles) { return P.h > 0 && tiles > kDirectTiles; }
__device__ __forceinline__ unsigned long long* super_sums(const BatchCtx& B) { return reinterpret_cast<unsigned long long*>(B.rowmn); }
__device__ __forceinline__ void clear_supers(const Launch& P, const BatchCtx& B) {
  if (P.h + 1 == P.L) return;
  const uint32_t supers = static_cast<uint32_t>(B.node_capacity) / (kTileRows * kSuperTiles) + 1u;
  for (uint32_t q = block_in_batch(P) * kThreads + threadIdx.x; q < supers; q += blocks_per_batch(P) * kThreads) super_sums(B)[q] = 0ull;
}

// Degree, sample count and row start per destination; in-tile scan of the sample counts.  BEGIN: the first hop under the
// partition strategy, which starts the counts and node ids as k_begin does; that no seed is stray is for k_sample_wide to
// tell, since the status word is being cleared.
template <bool BEGIN>
__global__ void __launch_bounds__(kThreads) k_count_rows(const Launch P) {
  __shared__ unsigned long long lds[kThreads / 64];
  const BatchCtx& B = P.b[batch_of_block(P)];
  const int n = BEGIN ? B.num_seeds : static_cast<int>(B.counts[P.h]);  // on its way with the status
  if (BEGIN ? false : block_has_status(B, P.L)) return;
  if (BEGIN && block_in_batch(P) == 0) begin_counts(P, B);
  const bool rows = !BEGIN || n <= P.num_nodes;
  const int d = P.d;
  const int tiles = (n + kTileRows - 1) / kTileRows;
  for (int tile = block_in_batch(P); tile < tiles; tile += blocks_per_batch(P)) {
    const int i = tile * kTileRows + threadIdx.x;
    uint32_t k = 0;
    if (i < n) {
      const int32_t id = BEGIN ? begin_seed(P, B, i) : B.node_ids[i];
      int64_t a = 0;
      uint32_t deg = 0;
      // the seeds are caller data: none may index the graph unchecked (later hops only hold
      // neighbour ids read from the graph)
      if (P.h > 0 || (id >= 0 && static_cast<int64_t>(id) < P.num_nodes)) {
        a = P.indptr[id];
        deg = static_cast<uint32_t>(P.indptr[id + 1] - a);
      }
      k = (d < 0 || deg <= static_cast<uint32_t>(d)) ? deg : static_cast<uint32_t>(d);
      if (rows) {
        B.rowstart[i] = a;
        B.rowdeg[i] = deg;
        B.rowk[i] = static_cast<int32_t>(k);
      }
    }
    unsigned long long total;
    const unsigned long long pre = block_exscan(static_cast<unsigned long long>(k), lds, total);
    if (rows && i < n) B.rowoff[i] = static_cast<int32_t>(pre);
    if (rows && threadIdx.x == 0) {
      B.tile_sums[tile] = total;
      if (has_supers(P, static_cast<uint32_t>(tiles))) atomicAdd(&super_sums(B)[static_cast<uint32_t>(tile) / kSuperTiles], total);
    }
    __syncthreads();
  }
}

// Samples of the hop's tiles before `tile`, the same for every lane of the wave, all of which call.
__device__ __forceinline__ unsigned long long samples_before(const Launch& P, const BatchCtx& B, uint32_t tiles, uint32_t tile) {
  const uint32_t lane = threadIdx.x & 63u;
  const bool supers = has_supers(P, tiles);
  const uint64_t* sums = supers ? reinterpret_cast<const uint64_t*>(super_sums(B)) : B.tile_sums;
  const uint32_t count = supers ? tile / kSuperTiles : tile;
  static_assert(kSuperTiles == 64, "a lane per tile");
  unsigned long long before = 0;
  if (supers && lane < tile % kSuperTiles) before = B.tile_sums[(tile & ~(kSuperTiles - 1u)) + lane];
  constexpr int U = 4;
  for (uint32_t q0 = lane; q0 - lane < count; q0 += 64u * U) {  // every read of a turn on its way before the first is used
    unsigned long long x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = sums[q0 + 64u * u < count ? q0 + 64u * u : count - 1u];
#pragma unroll
    for (int u = 0; u < U; ++u) before += q0 + 64u * u < count ? x[u] : 0ull;
  }
  const unsigned long long inc = wave_inscan(before);
  return static_cast<unsigned long long>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(inc >> 32), 63))) << 32 |
         static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(inc), 63));
}

// E_h, or what is wrong with the hop, by one wave.
__device__ __forceinline__ void close_samples(const Launch& P, const BatchCtx& B, int n, uint32_t tiles, unsigned long long room) {
  const unsigned long long edges = tiles == 0u ? 0ull : samples_before(P, B, tiles, tiles - 1u) + B.tile_sums[tiles - 1u];
  // a stray seed comes first, as it does where seeds are checked before anything is counted
  bool stray = false;
  for (int i = threadIdx.x & 63; edges > room && P.h == 0 && i < n; i += 64) stray = stray || static_cast<uint32_t>(B.node_ids[i]) >= P.num_nodes;
  stray = __any(stray);
  if ((threadIdx.x & 63) != 0) return;
  B.counts[P.L + 1 + P.h] = static_cast<int64_t>(edges);
  if (edges <= room) B.blk_indptr[n] = static_cast<int32_t>(edges);
  else set_status(B, P.L, stray ? SMFG_ST_SEED_OUT_OF_RANGE : SMFG_ST_EDGE_CAPACITY);
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
static_assert(wide_lds_bytes(SMFG_MAX_WIDE_FANOUT) + 2 * sizeof(uint2) <= 160 * 1024, "LDS of a compute unit, with the offsets of two turns");

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
  __shared__ uint2 turn_lds[2];  // .x samples of the tiles before the turn's first one, .y whether the batch ends here
  const BatchCtx& B = P.b[batch_of_block(P)];
  // A batch that had a status when the block started may count more nodes than its arrays hold; those below are read, and nothing
  // is done with them.  The first wave's answer is the block's: others may set a status meanwhile.
  const bool stopped = __any(status_of(B, P.L) != 0);
  const int64_t known = B.counts[P.h];
  const int n = static_cast<int>(known < B.node_capacity ? known : B.node_capacity);
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const uint32_t words = wide_lds_words(P.d), table_words = wide_table_words(P.d);
  uint32_t* draws = wide_lds + wave * (2 * words + table_words);
  uint32_t* picks = draws + words;
  uint32_t* table = picks + words;
  const int waves_total = blocks_per_batch(P) * (kThreads / 64);
  int per = (n + waves_total - 1) / waves_total;  // destinations per wave and turn
  per = per < 1 ? 1 : (per > kWideRows ? kWideRows : per);
  static_assert(kThreads / 64 * kWideRows <= kTileRows, "a block's destinations are in two tiles at most");
  const uint32_t tiles = static_cast<uint32_t>(n + kTileRows - 1) / kTileRows;
  const unsigned long long room = static_cast<unsigned long long>(B.edge_capacity < B.lostto_entries ? B.edge_capacity : B.lostto_entries);
  // Nothing of a hop with too many samples goes into the table: it may not have as many slots as they have nodes, and that would be told instead.
  const bool none = INSERT && wave == 0 && n > 0 && samples_before(P, B, tiles, tiles - 1u) + B.tile_sums[tiles - 1u] > room;
  int turn = 0;  // wave 0 writes the next turn's offset while others may still read the present one's
  for (int b0 = block_in_batch(P) * (kThreads / 64) * per; b0 < n; b0 += waves_total * per, turn ^= 1) {
    const int i0 = b0 + wave * per;
    const int il = i0 + lane;
    uint32_t v_l = 0, deg_l = 0, k_l = 0, base_l = 0, a_lo = 0, a_hi = 0;
    const bool mine = lane < per && il < n;
    if (mine) {
      v_l = static_cast<uint32_t>(B.node_ids[il]);
      const int64_t a = B.rowstart[il];
      a_lo = static_cast<uint32_t>(a);
      a_hi = static_cast<uint32_t>(static_cast<uint64_t>(a) >> 32);
      deg_l = static_cast<uint32_t>(B.rowdeg[il]);
      k_l = static_cast<uint32_t>(B.rowk[il]);
      base_l = static_cast<uint32_t>(B.rowoff[il]);
      if (il / kTileRows != b0 / kTileRows) base_l += static_cast<uint32_t>(B.tile_sums[b0 / kTileRows]);
    }
    if (wave == 0) {
      const uint32_t before = static_cast<uint32_t>(samples_before(P, B, tiles, static_cast<uint32_t>(b0 / kTileRows)));
      if (lane == 0) turn_lds[turn] = make_uint2(before, stopped || none ? 1u : 0u);
    }
    __syncthreads();
    if (turn_lds[turn].y != 0u) break;
    base_l += turn_lds[turn].x;
    if (mine) {
      if (P.h == 0 && v_l >= P.num_nodes) set_status(B, P.L, SMFG_ST_SEED_OUT_OF_RANGE);
      B.blk_indptr[il] = static_cast<int32_t>(base_l);
    }
    // nothing is written past the room of a hop that has too many samples, whatever the offsets come to
    if (static_cast<unsigned long long>(base_l) + k_l > room) k_l = deg_l = 0u;
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
  if (block_in_batch(P) == blocks_per_batch(P) - 1 && wave == 0 && !stopped) close_samples(P, B, n, tiles, room);
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
  const uint32_t n = static_cast<uint32_t>(B.counts[P.h]);  // both on their way with the status
  const uint32_t total_e = n + static_cast<uint32_t>(B.counts[P.L + 1 + P.h]);
  if (block_has_status(B, P.L)) {
    // k_sample_wide counts while it looks for stray seeds; as elsewhere, nothing but the seeds is counted with one
    if (P.h == 0 && block_in_batch(P) == 0 && threadIdx.x == 0 && status_of(B, P.L) == SMFG_ST_SEED_OUT_OF_RANGE) B.counts[P.L + 1] = 0;
    return;
  }
  const int lgB = hop_shape(P, B, n).lgB;
  const Segments segs = hop_segments(P, B, n);
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
// 9.7 M samples of four batches 18.5 -> 17.6 us, 5.5 M of one 9.9 -> 9.3, against four consecutive samples per thread;
// 12.3 and 8.3 with the larger tiles below and half the blocks.
// Tiles are of as many groups as leave at most kFlatTiles of them, so that every block of k_assemble_flat_part can scan their totals
// for itself.
constexpr uint32_t kFlatTiles = 2048;
__device__ __forceinline__ uint32_t flat_tile_lg(uint32_t samples) {  // log2 of the samples of a tile, for at most 2^30 of them
  uint32_t lg = 10;
  static_assert(kWideTile == 1 << 10, "the smallest tile");
  while (samples > kFlatTiles << lg) ++lg;
  return lg;
}
__global__ void __launch_bounds__(kThreads) k_flag_flat_part(const Launch P) {
  constexpr int kWaves = kThreads / 64;
  __shared__ uint32_t lds[2][kWaves];
  const BatchCtx& B = P.b[batch_of_block(P)];
  const uint32_t E = static_cast<uint32_t>(B.counts[P.L + 1 + P.h]);  // on its way with the status
  if (block_has_status(B, P.L)) return;
  const uint32_t lg = flat_tile_lg(E), tiles = (E + (1u << lg) - 1u) >> lg;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int turn = 0;  // a wave writes the next sums while others may still read the present ones
  for (uint32_t tile = block_in_batch(P); tile < tiles; tile += blocks_per_batch(P)) {
    const uint32_t end = E - (tile << lg) < 1u << lg ? E : (tile + 1u) << lg;
    uint32_t total = 0;  // new nodes of the tile so far
    uint32_t next[4];
    const auto fetch = [&](uint32_t p0) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t pos = p0 + u * 64 + lane;
        next[u] = pos < end ? static_cast<uint32_t>(B.gsrc[pos]) : kResolved;
      }
    };
    uint32_t p0 = (tile << lg) + static_cast<uint32_t>(wave) * 256u;
    fetch(p0);
    for (uint32_t c0 = tile << lg; c0 < end; c0 += kWideTile, p0 += kWideTile, turn ^= 1) {
      uint32_t e[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) e[u] = next[u];
      fetch(p0 + kWideTile);
      unsigned long long own = 0;  // lane u < 4: the bits of group u, and the new nodes of the tile before it
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
      before += total;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        if (w < wave) before += lds[turn][w];
        total += lds[turn][w];
      }
      if (lane < 4 && p0 + static_cast<uint32_t>(lane) * 64u < end)
        B.grp[(p0 >> 6) + lane] = make_uint4(static_cast<uint32_t>(own), static_cast<uint32_t>(own >> 32), before, 0u);
    }
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
// Every block scans the totals of the tiles for itself, 16 KB from the L2 at most, and then takes several runs of kWideTile samples.
constexpr unsigned kAssembleFlatBlocks = 2048;  // of a launch: what the chip holds at a time
__global__ void __launch_bounds__(kThreads) k_assemble_flat_part(const Launch P) {
  constexpr int kPer = kFlatTiles / kThreads;
  __shared__ uint32_t tile_new[kFlatTiles];  // new nodes of the tiles before
  __shared__ uint32_t scan[kThreads / 64];
  const BatchCtx& B = P.b[batch_of_block(P)];
  const uint32_t n = static_cast<uint32_t>(B.counts[P.h]);  // both on their way with the status
  const uint32_t E = static_cast<uint32_t>(B.counts[P.L + 1 + P.h]);
  if (block_has_status(B, P.L)) return;
  const uint32_t lg = flat_tile_lg(E), tiles = (E + (1u << lg) - 1u) >> lg, chunks = (E + kWideTile - 1) / kWideTile;
  clear_supers(P, B);
  if (static_cast<uint32_t>(block_in_batch(P)) >= (chunks > 0u ? chunks : 1u)) return;  // the first block also closes an empty hop
  {
    uint32_t x[kPer], mine = 0, fresh;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const uint32_t t = threadIdx.x * kPer + u;
      x[u] = t < tiles ? static_cast<uint32_t>(B.stile_sums[t]) : 0u;
      mine += x[u];
    }
    uint32_t pre = block_exscan<kThreads>(mine, scan, fresh);
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      tile_new[threadIdx.x * kPer + u] = pre;
      pre += x[u];
    }
    const int64_t nodes = static_cast<int64_t>(n) + static_cast<int64_t>(fresh);
    if (block_in_batch(P) == 0 && threadIdx.x == 0) {
      B.counts[P.h + 1] = nodes;
      if (nodes > B.node_capacity) set_status(B, P.L, SMFG_ST_NODE_CAPACITY);
    }
    if (nodes > B.node_capacity) return;
    __syncthreads();
  }
  for (uint32_t chunk = block_in_batch(P); chunk < chunks; chunk += blocks_per_batch(P)) {
    const uint32_t c0 = chunk * kWideTile, tpre = tile_new[c0 >> lg];
    const uint32_t p0 = c0 + (threadIdx.x >> 6) * 256u + (threadIdx.x & 63u);
    uint4 own[4];
    uint32_t e[4], q[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t pos = p0 + u * 64;
      e[u] = pos < E ? static_cast<uint32_t>(B.gsrc[pos]) : kResolved;
      own[u] = B.grp[(pos < E ? pos : c0) >> 6];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) q[u] = (e[u] & kPointer) == kPointer ? (e[u] & ~kPointer) : c0;
    // what the pointers name is fetched for all four samples before any is used
    uint4 qg[4];
    uint32_t qtile[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      qg[u] = B.grp[q[u] >> 6];
      qtile[u] = tile_new[q[u] >> lg];
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
  clear_supers(P, B);
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
