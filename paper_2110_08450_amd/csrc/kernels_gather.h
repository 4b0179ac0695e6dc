// libsmfg feature gather xs = x[ids] (Listing 1).
#ifndef SMFG_KERNELS_GATHER_H_
#define SMFG_KERNELS_GATHER_H_

#include <type_traits>

#include "device_common.h"

namespace smfg_dev {

// Rows are moved as vectors of sizeof(V) bytes.  A block copies ROWS consecutive output rows (32,
// or 64 when a row has fewer than 256 bytes: the 200-byte rows of the products-shaped workload
// copy 6 % faster that way, 256- and 512-byte rows 2-5 % slower) and exits: many short-lived blocks
// reach a higher copy rate on this chip than a persistent grid-stride loop.  Inside a block the output chunk is addressed as one flat vector array, so
// stores are fully coalesced and the lanes that share a row read one contiguous span of it.
// A row id outside [0, num_nodes) is read as row 0, so that no id can cause a read outside x.
// Rows of more than 512 MiB go one to a block, as AnyRow with 64-bit indices: 32 of them would outgrow
// the 32-bit ones.
constexpr int gather_rows_per_block(int64_t row_bytes) { return row_bytes < 256 ? 64 : row_bytes <= (int64_t(1) << 29) ? 32 : 1; }

// The copy's loads and stores are written out as instructions, for two reasons.  Cache policy:
// rows are read once and written once, and the compiler's non-temporal builtins set `nt` alone.
// `nt` keeps the rows from displacing what the sampling kernels beside the copy have in the
// caches (without it the whole path loses 8-13 %); stores with `sc0` on top measured +2.5 to +3 %
// on the papers100M-, arxiv- and products-shaped workloads, loads at system scope (`sc0 sc1`)
// another +1.4 % on the first (means of six interleaved runs).  Issue order: the two loads of a
// round leave together and its two stores leave back to back after one wait; the compiler put a
// wait between the stores, which cost the 200-byte rows of the products-shaped workload 3 %.
// Which level a line is kept in does not change what is copied: the table is read-only, and the
// kernel's end makes every store visible to what follows.  The wait is part of the load
// statements because the compiler does not track loads it did not emit; for the same reason a
// store is followed by two idle cycles: the hardware reads a wide store's data registers a
// moment after issue and wants no vector write to them in between, a gap the compiler only
// inserts after stores of its own.
template <typename V>
__device__ __forceinline__ void store_streaming(V v, V* p) {
  if constexpr (sizeof(V) == 16) {
    asm volatile("global_store_dwordx4 %0, %1, off sc0 nt\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
  } else if constexpr (sizeof(V) == 8) {
    asm volatile("global_store_dwordx2 %0, %1, off sc0 nt\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
  } else if constexpr (sizeof(V) == 4) {
    asm volatile("global_store_dword %0, %1, off sc0 nt\n\ts_nop 1" : : "v"(p), "v"(v) : "memory");
  } else {
    __builtin_nontemporal_store(v, p);
  }
}
template <typename V>
__device__ __forceinline__ V load_streaming(const V* p) {
  V v;
  if constexpr (sizeof(V) == 16) {
    asm volatile("global_load_dwordx4 %0, %1, off sc0 sc1 nt\n\ts_waitcnt vmcnt(0)" : "=&v"(v) : "v"(p) : "memory");
  } else if constexpr (sizeof(V) == 8) {
    asm volatile("global_load_dwordx2 %0, %1, off sc0 sc1 nt\n\ts_waitcnt vmcnt(0)" : "=&v"(v) : "v"(p) : "memory");
  } else if constexpr (sizeof(V) == 4) {
    asm volatile("global_load_dword %0, %1, off sc0 sc1 nt\n\ts_waitcnt vmcnt(0)" : "=&v"(v) : "v"(p) : "memory");
  } else {
    v = __builtin_nontemporal_load(p);
  }
  return v;
}
template <typename V>
__device__ __forceinline__ void load_pair_streaming(const V* p0, const V* p1, V& v0, V& v1) {
  if constexpr (sizeof(V) == 16) {
    asm volatile(
        "global_load_dwordx4 %0, %2, off sc0 sc1 nt\n\t"
        "global_load_dwordx4 %1, %3, off sc0 sc1 nt\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(v0), "=&v"(v1)
        : "v"(p0), "v"(p1)
        : "memory");
  } else if constexpr (sizeof(V) == 8) {
    asm volatile(
        "global_load_dwordx2 %0, %2, off sc0 sc1 nt\n\t"
        "global_load_dwordx2 %1, %3, off sc0 sc1 nt\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(v0), "=&v"(v1)
        : "v"(p0), "v"(p1)
        : "memory");
  } else if constexpr (sizeof(V) == 4) {
    asm volatile(
        "global_load_dword %0, %2, off sc0 sc1 nt\n\t"
        "global_load_dword %1, %3, off sc0 sc1 nt\n\t"
        "s_waitcnt vmcnt(0)"
        : "=&v"(v0), "=&v"(v1)
        : "v"(p0), "v"(p1)
        : "memory");
  } else {
    v0 = __builtin_nontemporal_load(p0);
    v1 = __builtin_nontemporal_load(p1);
  }
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
// A row as 16-byte vectors from its own first byte on, whatever its address and length (at least 16): the
// last one ends with the row and overlaps the one before, and both write the same bytes there.  The
// target reads and writes vectors at any byte address.  Used where nothing wider than 4 bytes is
// aligned; vectors as narrow as that cost instructions (400 K rows of 602 bytes 133 -> 102 us, 800 K
// of 77 bytes 64 -> 40, 800 K of 66 bytes 42 -> 36, 300 K of 404 bytes 56 -> 52), while rows of 200 bytes
// stay with 8-byte vectors (420 against 431 us).  Putting an aligned vector together from the end of one
// row and the beginning of the next instead of overlapping took 109 us for the 602-byte rows.
struct AnyRow {};

// The id of the thread's row of the block, if the array has as many.
template <int ROWS>
__device__ __forceinline__ int32_t row_id(const int32_t* __restrict__ ids, int64_t size) {
  const int64_t r = static_cast<int64_t>(blockIdx.x) * ROWS + threadIdx.x;
  return threadIdx.x < ROWS && r < size ? ids[r] : 0;
}
template <typename V, int ROWS>
__device__ __forceinline__ void gather_rows(const uint8_t* __restrict__ feat, int64_t row_stride,
                                            int64_t row_bytes, int64_t num_nodes,
                                            int32_t own, int64_t n,
                                            uint8_t* __restrict__ out) {
  static_assert(ROWS <= kThreads, "a thread per row has its id");
  constexpr bool kAny = __is_same(V, AnyRow);
  using W = typename std::conditional<kAny, u32x4, V>::type;
  using Index = typename std::conditional<ROWS == 1, uint64_t, uint32_t>::type;
  const Index vec_per_row = static_cast<Index>((row_bytes + (kAny ? 15 : 0)) / static_cast<int64_t>(sizeof(W)));
  __shared__ int64_t row_byte[ROWS];  // byte offset of each source row
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * ROWS;
  if (r0 >= n) return;
  const uint32_t rows = static_cast<uint32_t>(n - r0 < ROWS ? n - r0 : ROWS);
  const Index cnt = rows * vec_per_row;
  if (threadIdx.x < ROWS) {
    int64_t id = threadIdx.x < rows ? own : 0;
    if (id < 0 || id >= num_nodes) id = 0;
    row_byte[threadIdx.x] = id * row_stride;
  }
  __syncthreads();
  uint8_t* __restrict__ o = out + r0 * row_bytes;
  // (row, column) of a vector of the chunk by multiplication: ceil(2^32 / vec_per_row) gives the
  // exact quotient as long as index * vec_per_row < 2^32, which holds for every index of a chunk
  // when a row has at most 8192 vectors; longer rows divide
  const bool by_mul = vec_per_row <= 8192u;
  const uint64_t inv = 0xFFFFFFFFull / vec_per_row + 1ull;
  const auto place = [&](Index idx, const W*& from, W*& to) {
    const uint32_t jrow = ROWS == 1 ? 0u : static_cast<uint32_t>(by_mul ? (idx * inv) >> 32 : idx / vec_per_row);
    Index byte = (idx - jrow * vec_per_row) * static_cast<Index>(sizeof(W));
    if (kAny && idx - jrow * vec_per_row == vec_per_row - 1u) byte = static_cast<Index>(row_bytes) - 16u;
    from = reinterpret_cast<const W*>(feat + row_byte[jrow] + byte);
    to = kAny ? reinterpret_cast<W*>(o + jrow * row_bytes + byte) : reinterpret_cast<W*>(o) + idx;
  };
  // a round: two independent row reads per thread, then the two stores; the last round of a
  // thread may hold one vector only
  for (Index base = threadIdx.x; base < cnt; base += kThreads * 2) {
    const W *f0, *f1;
    W *t0, *t1;
    place(base, f0, t0);
    if (base + kThreads < cnt) {
      W v0, v1;
      place(base + kThreads, f1, t1);
      load_pair_streaming(f0, f1, v0, v1);
      store_streaming(v0, t0);
      store_streaming(v1, t1);
    } else {
      store_streaming(load_streaming(f0), t0);
    }
  }
}

template <typename V, int ROWS>
__global__ void __launch_bounds__(kThreads) k_gather(const Launch P) {
  const BatchCtx& B = P.b[blockIdx.y];
  // The number of rows, the status and the ids, as far as the array goes, on their way together: a block is four reads that
  // wait for each other otherwise, and two so.
  int64_t n = B.counts[P.L];
  const int32_t own = row_id<ROWS>(B.node_ids, B.node_capacity);
  if (B.features == nullptr || status_of(B, P.L) != 0) return;
  if (n > B.node_capacity) n = B.node_capacity;
  gather_rows<V, ROWS>(P.feat, P.row_stride, P.row_bytes, P.num_nodes, own, n, B.features);
}

template <typename V, int ROWS>
__global__ void __launch_bounds__(kThreads) k_gather_plain(const uint8_t* feat, int64_t row_bytes,
                                                           int64_t row_stride, int64_t num_nodes,
                                                           const int32_t* ids, const int64_t* num_rows,
                                                           int64_t max_rows, uint8_t* out) {
  int64_t n = *num_rows;
  if (n > max_rows) n = max_rows;
  if (n < 0) n = 0;
  const int32_t own = row_id<ROWS>(ids, n);  // there need not be more
  gather_rows<V, ROWS>(feat, row_stride, row_bytes, num_nodes, own, n, out);
}

}  // namespace smfg_dev

#endif  // SMFG_KERNELS_GATHER_H_
