"""Host logic of a sampling call (workspace plans, the path a call takes), run without a GPU: the
library's source is compiled together with a few exports of the functions that decide."""
import ctypes
import os
import random
import subprocess

import pytest

from paper_2110_08450_amd import build

SMALL_RECORDS = 32768   # a hop of the small path has fewer known nodes + sample positions than this
MAX_LAYERS = 8
I32P, I64P = ctypes.POINTER(ctypes.c_int32), ctypes.POINTER(ctypes.c_int64)

EXPORTS = r"""
#include "smfg.hip"
extern "C" {
void* plan(int64_t num_nodes, int32_t max_seeds, int32_t L, const int32_t* fanouts, int64_t node_capacity, int64_t sample_capacity) {
  smfg_graph g;
  std::memset(&g, 0, sizeof(g));
  g.num_nodes = num_nodes;
  smfg_workspace* ws = new smfg_workspace;
  if (plan_workspace(ws, &g, max_seeds, L, fanouts, node_capacity, sample_capacity) == SMFG_OK) return ws;
  delete ws;
  return nullptr;
}
void drop(void* ws) { delete static_cast<smfg_workspace*>(ws); }
int32_t is_part(const void* ws) { return static_cast<const smfg_workspace*>(ws)->part ? 1 : 0; }
int64_t slots(const void* ws) { return static_cast<const smfg_workspace*>(ws)->slot_entries; }
int32_t row_bounds(int32_t num_seeds, int32_t L, const int32_t* fanouts, int64_t num_nodes, int64_t node_capacity, int64_t* rows) {
  return hop_row_bounds(num_seeds, L, fanouts, num_nodes, node_capacity, rows) ? 1 : 0;
}
// lgB, lg2 and the least lgB of a hop of two levels
void levels(int32_t lg, int32_t* out) {
  part_levels(lg, out[0], out[1]);
  out[2] = kPartSplitLgB;
}
int32_t buckets(int64_t records, int32_t batches) { return buckets_log2(records, batches); }
int64_t one_level_records() { return kPartOneLevel; }
int32_t max_levels(int32_t which) { return which == 0 ? kPartMaxLgB : kPartMaxLg2; }
int32_t gather_block(int64_t row_bytes) { return gather_rows_per_block(row_bytes); }
int32_t gather_vector(int64_t address, int64_t row_bytes) {
  const int v = vec_bytes(static_cast<uintptr_t>(address), 0, row_bytes, 0);
  return v == kAnyRow ? 16 : v;
}
int32_t crowded(int64_t row_stride, int32_t gathers, int32_t num_batches) {
  smfg_graph g;
  std::memset(&g, 0, sizeof(g));
  g.row_stride = row_stride;
  g.feat = row_stride > 0 ? reinterpret_cast<const uint8_t*>(256) : nullptr;
  return crowded_by_a_gather(&g, gathers != 0, num_batches) ? 1 : 0;
}
int64_t hist_entries(const void* ws) { return static_cast<const smfg_workspace*>(ws)->hist_entries; }
// row_blocks << lgB of a hop and the rows its blocks cover, or -1 if a workspace has no room for it
int64_t part_hop(void** ws, int32_t num_batches, int64_t max_rows, int32_t d, int64_t* covered) {
  HopPlan hp;
  if (!plan_part_hop(reinterpret_cast<const smfg_workspace* const*>(ws), num_batches, max_rows, d, &hp)) return -1;
  *covered = hp.row_blocks * hp.block_rows;
  return hp.row_blocks << hp.lgB;
}
int32_t small_hops(void** ws, const int32_t* num_seeds, int64_t num_nodes, const int64_t* rows, const int32_t* fanouts, int32_t L,
                   int32_t num_batches, int32_t crowded) {
  return small_hops_of(reinterpret_cast<const smfg_workspace* const*>(ws), num_seeds, num_nodes,
                       reinterpret_cast<const int64_t (*)[SMFG_MAX_LAYERS + 1]>(rows), fanouts, L, num_batches, crowded != 0);
}
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("host")
    src, lib = d / "host.hip", d / "host.so"
    src.write_text(EXPORTS)
    subprocess.run([build.hipcc(), "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC", "-shared",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.dirname(build.SRC), "-I", build.INCLUDE, str(src), "-o", str(lib)],
                   check=True, capture_output=True, timeout=300)
    h = ctypes.CDLL(str(lib))
    i32, i64, vp = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p
    h.plan.argtypes, h.plan.restype = [i64, i32, i32, I32P, i64, i64], vp
    h.drop.argtypes = h.is_part.argtypes = h.slots.argtypes = [vp]
    h.slots.restype = i64
    h.crowded.argtypes = [i64, i32, i32]
    h.levels.argtypes = [i32, I32P]
    h.buckets.argtypes = [i64, i32]
    h.one_level_records.restype = i64
    h.gather_block.argtypes, h.gather_vector.argtypes = [i64], [i64, i64]
    h.hist_entries.argtypes, h.hist_entries.restype = [vp], i64
    h.part_hop.argtypes, h.part_hop.restype = [ctypes.POINTER(vp), i32, i64, i32, I64P], i64
    h.row_bounds.argtypes = [i32, i32, I32P, i64, i64, I64P]
    h.small_hops.argtypes = [ctypes.POINTER(vp), I32P, i64, I64P, I32P, i32, i32, i32]
    return h


def fan_array(fanouts):
    return (ctypes.c_int32 * len(fanouts))(*fanouts)


def rows_of(host, seeds, fanouts, num_nodes, node_capacity=1 << 29):
    rows = (ctypes.c_int64 * len(fanouts))()
    assert host.row_bounds(seeds, len(fanouts), fan_array(fanouts), num_nodes, node_capacity, rows)
    return list(rows)


def small_hops(host, ws, seeds, num_nodes, rows, fanouts, crowded=False):
    """rows[b][h]: the most destinations of hop h of batch b."""
    flat = [x for r in rows for x in list(r) + [0] * (MAX_LAYERS + 1 - len(r))]
    return host.small_hops((ctypes.c_void_p * len(ws))(*ws), fan_array(seeds), num_nodes, (ctypes.c_int64 * len(flat))(*flat),
                           fan_array(fanouts), len(fanouts), len(ws), crowded)


@pytest.mark.parametrize("sizes", [(256, 100), (300, 100), (256, 250), (31, 30, 1), (300, 17, 1, 100)])
def test_set_of_own_sized_table_workspaces_takes_the_small_path(host, sizes):
    """A workspace per batch, planned for that batch: every hop of every batch is small and has room."""
    fan = (10, 5)
    ws = [host.plan(1 << 20, n, 2, fan_array(fan), 0, 0) for n in sizes]
    assert not any(host.is_part(w) for w in ws)
    assert small_hops(host, ws, sizes, 1 << 20, [rows_of(host, n, fan, 1 << 20) for n in sizes], fan) == 2
    for w in ws:
        host.drop(w)


def test_small_hops_of_ragged_sets(host):
    """Random launch sets of batches and workspaces of different sizes.  With device tables a call takes
    the small path for all hops or for none (a hop on the table after one off it would find the table
    uncleared and without the nodes so far); a hop on the small path is below its limit and has room for
    its padded positions in every batch's own workspace."""
    rnd = random.Random(5)
    seen = {"table": set(), "part": set()}
    for _ in range(4000):
        L = rnd.randint(1, 4)
        fan = [rnd.choice([rnd.randint(1, 32), rnd.randint(1, 8), rnd.randint(33, 200) if rnd.random() < 0.3 else 3])
               for _ in range(L)]
        num_nodes = int(10 ** rnd.uniform(0, 7))
        top = int(10 ** rnd.uniform(0, 3.2)) + 1
        seeds = [rnd.randint(max(1, top // rnd.choice([2, 10, 100])), top) for _ in range(rnd.randint(1, 9))]
        sized = lambda n: n if rnd.random() < 0.7 else top
        capacity = rnd.choice([0, 0, rnd.randint(top, 40 * top)])
        samples = rnd.randint(1, 20 * top) if max(fan) > 32 and rnd.random() < 0.5 else 0
        ws = [host.plan(num_nodes, sized(n), L, fan_array(fan), capacity, samples) for n in seeds]
        if all(ws) and len({host.is_part(w) for w in ws}) == 1:
            rows = [rows_of(host, n, fan, num_nodes, capacity or 1 << 29) for n in seeds]
            hops = small_hops(host, ws, seeds, num_nodes, rows, fan)
            assert 0 <= hops <= L
            # beside another set's gather: the same, but a call with larger hops has no small ones
            crowded = small_hops(host, ws, seeds, num_nodes, rows, fan, crowded=True)
            assert crowded == (hops if hops == L else 0)
            if not host.is_part(ws[0]):
                assert hops in (0, L), (fan, seeds)
            for w, r, n in zip(ws, rows, seeds):
                for h in range(hops):
                    # the kernels read the seeds as the destinations of hop 0, all of them
                    assert max(r[h], n if h == 0 else 0) * fan[h] <= host.slots(w)
                    assert fan[h] <= 32 and r[h] * (1 + fan[h]) < SMALL_RECORDS and r[h] * fan[h] <= host.slots(w)
            seen["part" if host.is_part(ws[0]) else "table"].add("none" if hops == 0 else "all" if hops == L else "some")
        for w in ws:
            if w:
                host.drop(w)
    assert seen["table"] >= {"all"} and seen["part"] >= {"none", "some"}


def test_which_calls_run_beside_a_gather(host):
    """Only sets of five batches and more that leave the gather to another call."""
    assert [host.crowded(256, 0, n) for n in (1, 2, 4, 5, 16)] == [0, 0, 0, 1, 1]
    assert not host.crowded(256, 1, 8)      # gathers itself
    assert not host.crowded(0, 0, 8)        # no features: nobody gathers


@pytest.mark.parametrize("num_nodes", [1 << 28, 500_000])
@pytest.mark.parametrize("fanouts", [(15, 10, 5), (12, 7), (25, 10), (20, 20, 20), (3, 3, 3, 3)])
def test_a_workspace_takes_fewer_seeds_than_it_was_made_for(host, fanouts, num_nodes):
    """Every number of seeds up to a partition workspace's own, alone or in a launch set, fits it: a
    hop's rows are covered by row blocks that the workspace has counters for."""
    rnd = random.Random(1)
    covered = ctypes.c_int64()
    planned = 0
    for top in [515, 600, 1000, 1024] + [int(10 ** rnd.uniform(1.5, 3.8)) for _ in range(60)]:
        w = host.plan(num_nodes, top, len(fanouts), fan_array(fanouts), 0, 0)
        if not w or not host.is_part(w):
            continue
        planned += 1
        for n in {top, top - 1, top - top // 7, top // 2 + 1, *(rnd.randint(1, top) for _ in range(40))}:
            for d, rows in zip(fanouts, rows_of(host, n, fanouts, num_nodes)):
                for batches in (1, 2, 8, 9, 16):
                    got = host.part_hop((ctypes.c_void_p * batches)(*[w] * batches), batches, rows, d, covered)
                    assert 0 < got <= host.hist_entries(w), (top, n, d, batches)
                    assert covered.value >= rows
        host.drop(w)
    assert planned > 10


def test_gather_blocks_stay_within_their_indices(host):
    """A block of several rows counts vectors and bytes of a row in 32 bits; the last round of a thread
    may look 2 x 256 vectors beyond the block's last one."""
    sizes = {x for e in range(37) for x in range((1 << e) - 9, (1 << e) + 10) if x > 0}
    for row_bytes in sizes | {x * 16 for x in sizes} | {(1 << 31) - 8192, 600_000_003 * 8}:
        for address in (0, 8, 4, 2, 1):
            rows, vec = host.gather_block(row_bytes), host.gather_vector(address, row_bytes)
            if rows > 1:
                assert rows * -(-row_bytes // vec) + 512 < 1 << 32 and row_bytes < 1 << 32
            if rows != 64:      # the rows per block for which vectors of 4 bytes and less are not built
                assert vec >= 8


def test_bucket_levels(host):
    """How 2^lg hash buckets are laid out in one or two levels: within what the kernels' LDS arrays hold, together
    always 2^lg; a hop of two levels starts with 256 buckets or more."""
    most_b, most_2 = host.max_levels(0), host.max_levels(1)
    out = (ctypes.c_int32 * 3)()
    for lg in range(most_b + most_2 + 1):
        host.levels(lg, out)
        assert out[0] + out[1] == lg and 0 <= out[0] <= most_b and 0 <= out[1] <= most_2
        assert out[1] == 0 if lg <= most_b else (out[1] > 0 and out[0] >= out[2] == 8)


def test_bucket_levels_for_every_number_of_batches(host):
    """Two levels begin at the same number of records however many batches share a launch, so that the capacity of a
    workspace does not depend on the launch set; a batch never has more buckets for being one of several, and has the
    same ones from 512 in all."""
    most_b, one_level = host.max_levels(0), host.one_level_records()
    rnd = random.Random(3)
    for records in [1, one_level - 1, one_level] + [int(10 ** rnd.uniform(0, 9)) for _ in range(2000)]:
        alone = host.buckets(records, 1)
        assert (alone > most_b) == (records >= one_level)
        for batches in range(2, 17):
            lg = host.buckets(records, batches)
            assert lg <= alone and (lg == alone or batches << lg >= 512)
            assert lg == alone or alone <= most_b
