"""Room for the segments of a hop: whatever number of destinations and samples a batch turns out to have, the
offsets of its segments and sub-buckets fit what its workspace was made for.  The library's source is
compiled together with a few exports, so this runs without a GPU."""
import ctypes
import os
import random
import subprocess

import pytest

from paper_2110_08450_amd import build

EXPORTS = r"""
#include "smfg.hip"
extern "C" {
void* plan(int64_t num_nodes, int32_t max_seeds, int32_t L, const int32_t* fanouts, int64_t samples) {
  smfg_graph g;
  std::memset(&g, 0, sizeof(g));
  g.num_nodes = num_nodes;
  smfg_workspace* ws = new smfg_workspace;
  if (plan_workspace(ws, &g, max_seeds, L, fanouts, 0, samples) == SMFG_OK && ws->part) return ws;
  delete ws;
  return nullptr;
}
void drop(void* ws) { delete static_cast<smfg_workspace*>(ws); }
int64_t records(const void* ws) { return static_cast<const smfg_workspace*>(ws)->rec_entries; }
// the levels that `records` of a hop's batch b take, if they have room in its workspace and in the LDS of the hop's blocks
static int64_t room(const smfg_workspace* w, int64_t count, int64_t cap, int64_t records, int batches, const HopPlan& hp, int b) {
  const HopShape hs = hop_levels(records, batches, hp.lgB + hp.lg2, hp.one_level[b]);
  const int lgB = hs.lgB, lg2 = hs.lg2;
  if (count * offs_stride(lgB) > (lg2 > 0 ? w->hist_two : w->hist_entries)) return -1;
  if (offs_stride(lgB) * 2 > offsets_lds_bytes(hp.most_lgB)) return -4;
  if (lg2 == 0) return 1;
  if (lgB > kPartMaxLgB || lg2 > kPartMaxLg2) return -2;
  const int64_t range = split_range(static_cast<uint32_t>(cap), lgB);
  if (((count + range - 1) / range << lgB) * ((1 << lg2) + 1) * 4 > w->b_bstart2) return -3;
  return 2;
}
// rows of a hop that were bounded by max_rows: 1 or 2 levels, or negative where something does not fit
int64_t drawn(void* ws, int32_t batches, int64_t max_rows, int32_t d, int64_t rows) {
  const smfg_workspace* w = static_cast<const smfg_workspace*>(ws);
  const smfg_workspace* all[SMFG_MAX_BATCHES];
  for (int b = 0; b < batches; ++b) all[b] = w;
  HopPlan hp;
  if (!plan_part_hop(all, batches, max_rows, d, &hp)) return -10;
  if (hp.block_rows > seg_rows(hp.per, d) || hp.block_rows * (1 + d) > hp.per * kThreads || hp.block_rows > hp.per / 4 * kThreads) return -11;
  if (hp.block_rows * static_cast<int64_t>(draw_stride(d)) > hp.per * kThreads) return -12;
  if (hp.row_blocks * hp.block_rows < max_rows) return -13;
  const int64_t cap = static_cast<int64_t>(hp.block_rows) * (1 + d);
  if ((rows + hp.block_rows - 1) / hp.block_rows * cap > w->rec_entries + cap) return -14;
  const HopShape hs = hop_levels(rows * (1 + d), batches, hp.lgB + hp.lg2, hp.one_level[0]);
  if (rows * (1 + d) >> (hs.lgB + hs.lg2) > kPartMostRecords) return -15;
  return room(w, (rows + hp.block_rows - 1) / hp.block_rows, cap, rows * (1 + d), batches, hp, 0);
}
// Whether the arrays of a workspace, with hist as long as hops of one and of two levels may take it, lie one behind the
// other, but for those that take turns; its size.
int64_t layout(void* ws) {
  smfg_workspace* w = static_cast<smfg_workspace*>(ws);
  const uint64_t base = 1ull << 32;
  bind_workspace(w, reinterpret_cast<void*>(base));
  const int64_t n = w->node_capacity;
  const auto end = [&](const void* p, int64_t bytes) { return reinterpret_cast<uint64_t>(p) + static_cast<uint64_t>(bytes); };
  const auto at = [&](const void* p) { return reinterpret_cast<uint64_t>(p); };
  const int64_t tiles = (n + kTileRows - 1) / kTileRows;
  if (end(w->gsrc, w->slot_entries * 4) > at(w->rowk) || end(w->rowk, n * 4) > at(w->rowoff)) return -1;
  if (end(w->rowoff, n * 4) > at(w->tile_sums) || end(w->tile_sums, tiles * 8) > at(w->rowmn) || at(w->hist) != at(w->rowmn)) return -2;
  if (end(w->rowmn, n * 8) > at(w->split_lg > 0 ? static_cast<void*>(w->bstart2) : w->rec)) return -3;
  if (end(w->hist, w->hist_two * 2) > at(w->split_lg > 0 ? static_cast<void*>(w->bstart2) : w->rec)) return -4;
  if (end(w->hist, w->hist_entries * 2) > at(w->rec)) return -5;
  if (w->split_lg > 0 && (end(w->bstart2, split_entries_for(w->rec_entries) * 4) > at(w->rec2) || end(w->rec2, w->rec_entries * 8) > at(w->rec))) return -6;
  uint64_t last = end(w->rec, w->rec_entries * 8);
  if (w->flat) {
    if (last > at(w->grp) || end(w->grp, (w->slot_entries / 64 + 1) * 16) > at(w->rowstart) || end(w->rowstart, n * 8) > at(w->rowdeg) ||
        end(w->rowdeg, n * 4) > at(w->stile_sums))
      return -7;
    last = end(w->stile_sums, (w->slot_entries / kWideTile + 1) * 8);
  }
  for (const void* p : {static_cast<void*>(w->gsrc), static_cast<void*>(w->rowk), static_cast<void*>(w->rowoff), static_cast<void*>(w->tile_sums),
                        static_cast<void*>(w->rowmn), static_cast<void*>(w->bstart2), static_cast<void*>(w->rec2), static_cast<void*>(w->rec)})
    if (at(p) % 256 != 0) return -8;
  return last <= base + static_cast<uint64_t>(w->bytes) ? w->bytes : -9;
}
// `records` of a hop over exact offsets that was bounded by `bound`: 1 or 2 levels, 0 if the call is refused
int64_t flat(void* ws, int32_t batches, int64_t bound, int64_t records) {
  const smfg_workspace* w = static_cast<const smfg_workspace*>(ws);
  const smfg_workspace* all[SMFG_MAX_BATCHES];
  for (int b = 0; b < batches; ++b) all[b] = w;
  HopPlan hp;
  if (!plan_flat_hop(all, batches, bound, &hp)) return 0;
  const int64_t cap = flat_seg(batches, static_cast<uint32_t>(records));
  return room(w, (records + cap - 1) / cap, cap, records, batches, hp, 0);
}
// The same for every batch of a set whose workspaces differ, records[b] of each; `share`: the most records to a bucket in a
// batch whose workspace was not cut.
int64_t flat_set(void** ws, int32_t batches, int64_t bound, const int64_t* records, int64_t* share) {
  const smfg_workspace* const* w = reinterpret_cast<const smfg_workspace* const*>(ws);
  HopPlan hp;
  if (!plan_flat_hop(w, batches, bound, &hp)) return 0;
  *share = 0;
  for (int b = 0; b < batches; ++b) {
    const int64_t cap = flat_seg(batches, static_cast<uint32_t>(records[b]));
    const int64_t got = room(w[b], (records[b] + cap - 1) / cap, cap, records[b], batches, hp, b);
    if (got < 0) return got;
    const HopShape hs = hop_levels(records[b], batches, hp.lgB + hp.lg2, hp.one_level[b]);
    if (records[b] >> (hs.lgB + hs.lg2) > *share) *share = records[b] >> (hs.lgB + hs.lg2);
  }
  return 1;
}
}
"""


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    d = tmp_path_factory.mktemp("segments")
    src, lib = d / "host.hip", d / "host.so"
    src.write_text(EXPORTS)
    subprocess.run([build.hipcc(), "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC", "-shared",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.dirname(build.SRC), "-I", build.INCLUDE, str(src), "-o", str(lib)],
                   check=True, capture_output=True, timeout=300)
    h = ctypes.CDLL(str(lib))
    i32, i64, vp = ctypes.c_int32, ctypes.c_int64, ctypes.c_void_p
    h.plan.argtypes, h.plan.restype = [i64, i32, i32, ctypes.POINTER(i32), i64], vp
    h.drop.argtypes, h.drop.restype = [vp], None
    h.records.argtypes, h.records.restype = [vp], i64
    h.drawn.argtypes, h.drawn.restype = [vp, i32, i64, i32, i64], i64
    h.flat.argtypes, h.flat.restype = [vp, i32, i64, i64], i64
    h.flat_set.argtypes, h.flat_set.restype = [ctypes.POINTER(vp), i32, i64, ctypes.POINTER(i64), ctypes.POINTER(i64)], i64
    h.layout.argtypes, h.layout.restype = [vp], i64
    return h


def _sizes(rnd, most):
    return {most, most - 1, most // 2 + 1, 1, *(int(most ** rnd.random()) for _ in range(30)), *(rnd.randint(1, most) for _ in range(20))}


@pytest.mark.parametrize("wide", [False, True])
def test_offsets_of_every_hop_fit_the_workspace(host, wide):
    """Own fanouts or others, fewer seeds, fewer rows than the bound, any number of batches."""
    rnd = random.Random(4)
    levels = set()
    for _ in range(250):
        nodes = int(10 ** rnd.uniform(4, 8.6))
        fan = [rnd.choice([1, 2, 3, 5, 10, 20, 32, rnd.randint(1, 32)]) for _ in range(rnd.randint(1, 3))]
        if wide:
            fan.append(rnd.choice([40, 100, 1000]))
        seeds = int(10 ** rnd.uniform(2, 6.3))
        w = host.plan(nodes, seeds, len(fan), (ctypes.c_int32 * len(fan))(*fan), 0)
        if not w:
            continue
        most = host.records(w)
        assert host.layout(w) > 0, (host.layout(w), nodes, fan, seeds)
        for batches in (1, 2, 4, 8, 16):
            if wide:
                for bound in {most, rnd.randint(1, most)}:
                    for r in _sizes(rnd, bound):
                        got = host.flat(w, batches, bound, r)
                        assert got > 0, (got, nodes, fan, seeds, batches, bound, r)
                        levels.add(("flat", got))
            for d in {1, 2, 3, 5, 20, 32, *[x for x in fan if x <= 32]}:
                top = min(most // (1 + d), nodes)
                if top < 1:
                    continue
                for bound in {top, rnd.randint(1, top)}:
                    for rows in _sizes(rnd, bound):
                        got = host.drawn(w, batches, bound, d, rows)
                        assert got > 0, (got, nodes, fan, seeds, batches, d, bound, rows)
                        levels.add(("drawn", got))
        host.drop(w)
    assert levels == {("drawn", 1), ("drawn", 2)} | ({("flat", 1), ("flat", 2)} if wide else set())


def test_static_calls_near_the_limit_of_their_scratch(host):
    """Calls that once took nearly all of the 64 MiB fit them with all the buckets that their records take."""
    share = ctypes.c_int64()
    for nodes, fan, seeds in [(100_000, [100], 29_893), (95_101, [327, 3, 3], 9_174), (717_948, [32], 82_705), (481_513, [32, 1000], 65),
                              (524_879, [1000], 2_044), (311_627, [32], 92_402), (242_211, [5, 32, 10], 15_676), (35_837, [806, 40, 40], 3_874)]:
        w = host.plan(nodes, seeds, len(fan), (ctypes.c_int32 * len(fan))(*fan), 0)
        assert 0 < host.layout(w) <= 64 << 20, (nodes, fan, seeds)
        most = host.records(w)
        if max(fan) > 32:
            for r in {most, min(most, (1229 << 11) - 1), min(most, 1229 << 11)}:
                assert host.flat_set((ctypes.c_void_p * 1)(w), 1, most, (ctypes.c_int64 * 1)(r), share) == 1 and share.value <= 1228
        host.drop(w)


def test_wide_sets_of_workspaces_of_any_size(host):
    """A launch set over exact offsets: every batch has the buckets that its own records take, 1228 of them to a bucket at
    most, whatever the workspaces beside its own were made for, and a block has LDS for them."""
    rnd = random.Random(11)
    fan = (ctypes.c_int32 * 2)(100, 100)
    seen = set()
    for turn in range(300):
        nodes = 2_450_000 if turn < 20 else int(10 ** rnd.uniform(3, 7))
        tops = [2048, 1] if turn < 20 else [int(10 ** rnd.uniform(0, 3.6)) for _ in range(rnd.randint(2, 16))]
        ws = [host.plan(nodes, top, 2, fan, 0) for top in tops]
        if all(ws):
            most = [host.records(w) for w in ws]
            bound = max(most) if turn < 20 else rnd.randint(1, max(most))
            share = ctypes.c_int64()
            for _ in range(40):
                recs = [rnd.choice([min(bound, m), int(min(bound, m) ** rnd.random()), rnd.randint(1, min(bound, m))]) for m in most]
                got = host.flat_set((ctypes.c_void_p * len(ws))(*ws), len(ws), bound, (ctypes.c_int64 * len(ws))(*recs), share)
                assert got == 1 and share.value <= 1228, (got, share.value, nodes, tops, bound, recs)
                seen.add(max(recs) >= 1229 << 11)
        for w in ws:
            if w:
                host.drop(w)
    assert seen == {False, True}
