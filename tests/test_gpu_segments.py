"""Hops of the partition strategy at the sizes where their segments, buckets and sub-buckets change, against the
CPU oracle (needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2110_08450_amd import binding as smfg
from test_gpu_parity import DEV, GpuGraph, assert_same, fetch
from test_gpu_variants import random_graph, sample

pytestmark = pytest.mark.gpu


def segment_rows(d):
    """Destinations of a full segment of 8 records per thread of a block of 256."""
    return min(2048 // (1 + d), 512)


@pytest.mark.parametrize("more", [0, 1])
@pytest.mark.parametrize("d", [1, 2, 3, 7, 16, 20, 32])
def test_segments_of_either_size(d, more, monkeypatch):
    """512 full segments of 8 records per thread, and one destination more, which makes them segments of 16 with a
    short last one; each with another batch of a few rows, down to one."""
    monkeypatch.setenv("SMFG_DEDUP", "partition")
    n = 270_000
    gg = random_graph(n, 2 * d, d)
    perm = np.random.default_rng(d).permutation(n).astype(np.int32)
    batches = [perm[:512 * segment_rows(d) + more], perm[-1 - 40 * more:]]
    ws = [smfg.workspace_create(gg.g, len(batches[0]), (d,)) for _ in batches]
    outs = [smfg.alloc_output(gg.g, len(b), (d,)) for b in batches]
    smfg.sample_mfg_many(gg.g, ws, [torch.from_numpy(b).to(DEV) for b in batches], (d,), [5, 6], outs)
    for b, key, out in zip(batches, (5, 6), outs):
        assert_same(fetch(out, 1), gg.oracle.sample_mfg(b, (d,), key), 1)


@pytest.mark.parametrize("fanout", [4, 3, -1])
@pytest.mark.parametrize("hubs", [0, 3])
def test_two_levels_with_and_without_hubs(hubs, fanout):
    """More records than one level takes; with the neighbours of half the destinations among three nodes, whose
    buckets hold far more than a block of the second level keeps in registers."""
    n = 2_000_000
    rng = np.random.default_rng(hubs)
    rows = rng.integers(0, n, size=(n, 4)).astype(np.int32)
    if hubs:
        rows[::2] = rng.integers(0, hubs, size=(n // 2, 4)) * 600_001 + 17
    gg = GpuGraph(np.arange(n + 1, dtype=np.int64) * 4, rows.ravel(), None)
    s = rng.permutation(n)[:1_950_000].astype(np.int32)
    ws = smfg.workspace_create(gg.g, len(s), (fanout,), 0, 4 * n if fanout < 0 else 0)
    out = smfg.alloc_output(gg.g, len(s), (fanout,), edge_capacity=[4 * n])
    smfg.sample_mfg(gg.g, ws, torch.from_numpy(s).to(DEV), (fanout,), 9, out)
    assert_same(fetch(out, 1), gg.oracle.sample_mfg(s, (fanout,), 9), 1)


def test_segments_of_other_fanouts_than_planned(monkeypatch):
    """A workspace made for fanout 20 and used with 1 and 2, whose segments are smaller and so more."""
    monkeypatch.setenv("SMFG_DEDUP", "partition")
    n = 1_500_000
    gg = random_graph(n, 4, 2)
    perm = np.random.default_rng(0).permutation(n).astype(np.int32)
    ws = smfg.workspace_create(gg.g, 140_000, (20,))
    for d, seeds in [(1, 140_000), (2, 139_999)]:
        out = smfg.alloc_output(gg.g, seeds, (d,))
        smfg.sample_mfg(gg.g, ws, torch.from_numpy(perm[:seeds]).to(DEV), (d,), 3, out)
        assert_same(fetch(out, 1), gg.oracle.sample_mfg(perm[:seeds], (d,), 3), 1)


@pytest.mark.parametrize("batches", [1, 3, 16])
@pytest.mark.parametrize("fanouts,seeds,dim,dtype", [
    ((10, 5), 256, 32, np.float32), ((1, 32), 300, 9, np.float16), ((31, 3), 200, 8, np.float16), ((32, 1), 990, 4, np.float32),
    ((15, 10, 5), 16, 100, np.float16), ((2, 2, 2, 17), 30, 101, np.float16), ((1,), 16383, 7, np.float32), ((3,), 0, 16, np.float32),
    ((10, 5), 290, 700, np.float32)])
def test_small_hops_that_go_on(fanouts, seeds, dim, dtype, batches):
    """Small calls whose blocks draw for the next hop, in one turn or several, and copy the feature rows, of 16 bytes
    and more and up to the size that is left to the gather; the odd hops' arrays of table and partition workspaces."""
    gg = random_graph(40_000, 40, 13, dim=dim, dtype=dtype)
    rng = np.random.default_rng(seeds)
    sizes = [seeds] + [int(x) for x in rng.integers(0, seeds + 1, size=batches - 1)]
    s = [rng.permutation(40_000)[:k].astype(np.int32) for k in sizes]
    ws = [smfg.workspace_create(gg.g, seeds, fanouts) for _ in s]
    outs = [smfg.alloc_output(gg.g, seeds, fanouts) for _ in s]
    for turn in range(2):
        keys = [100 * turn + b for b in range(batches)]
        smfg.sample_mfg_many(gg.g, ws, [torch.from_numpy(x).to(DEV) for x in s], fanouts, keys, outs)
        for x, key, out in zip(s, keys, outs):
            assert_same(fetch(out, len(fanouts)), gg.oracle.sample_mfg(x, fanouts, key), len(fanouts))


@pytest.mark.parametrize("samples", [1, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 4097])
def test_flat_groups_and_tiles(samples, monkeypatch):
    """Whole neighbourhoods of two destinations at the edges of groups of 64 samples, of a wave's 256 and of tiles of
    1024; a third of the samples repeat nodes, the destinations among them."""
    monkeypatch.setenv("SMFG_DEDUP", "partition")
    n = 6000
    rng = np.random.default_rng(samples)
    first = rng.permutation(n)[:samples - samples // 3]
    indices = np.concatenate([first, rng.choice(np.append(first, [0, 1]), samples // 3)]).astype(np.int32)
    indptr = np.full(n + 1, samples, dtype=np.int64)
    indptr[:2] = [0, len(first)]
    gg = GpuGraph(indptr, indices, None)
    s = np.array([0, 1], dtype=np.int32)
    ws = smfg.workspace_create(gg.g, 2, (-1,), 0, samples)
    out = smfg.alloc_output(gg.g, 2, (-1,), edge_capacity=[samples])
    smfg.sample_mfg(gg.g, ws, torch.from_numpy(s).to(DEV), (-1,), 3, out)
    assert_same(fetch(out, 1), gg.oracle.sample_mfg(s, (-1,), 3), 1)


@pytest.mark.parametrize("n,fan,most,others", [(100_000, (100,), 30_907, (24_000, 29_894, 30_717, 30_876)), (300_000, (32,), 94_834, (75_000, 94_238))])
def test_static_calls_up_to_the_limit_of_their_scratch(n, fan, most, others):
    """Hops of one level and of two whose scratch takes nearly all of the 64 MiB, up to the last that a workspace of that
    size would serve; the next one is refused."""
    rng = np.random.default_rng(3)
    deg = fan[0] + 10
    gg = GpuGraph(np.arange(n + 1, dtype=np.int64) * deg, rng.integers(0, n, size=deg * n).astype(np.int32), None)
    perm = rng.permutation(n).astype(np.int32)
    out = smfg.alloc_output(gg.g, most + 1, fan)
    dev = torch.from_numpy(perm).to(DEV)
    for seeds in (*others, most):
        assert smfg.workspace_create(gg.g, seeds, fan).nbytes <= smfg.STATIC_SCRATCH_BYTES
        smfg.sample_mfg_static(gg.g, dev[:seeds], fan, 11, out)
        assert_same(fetch(out, 1), gg.oracle.sample_mfg(perm[:seeds], fan, 11), 1)
    assert smfg.workspace_create(gg.g, most + 1, fan).nbytes > smfg.STATIC_SCRATCH_BYTES
    with pytest.raises(smfg.SmfgError) as e:
        smfg.sample_mfg_static(gg.g, dev[:most + 1], fan, 11, out)
    assert e.value.code == smfg.ERR_CAPACITY


@pytest.mark.parametrize("fanouts,sizes", [((100,), (26_000, 16)), ((100,), (20_000, 1)), ((100,), (1, 26_000, 300, 12_000)),
                                           ((40, 40), (2000, 1)), ((-1,), (3, 24_000))])
def test_wide_set_of_one_large_and_one_small_workspace(fanouts, sizes):
    """A workspace made for each batch: the small one has offsets for a few buckets only, the large batch takes 2048, or two
    levels beyond 2.5 M records, beside it."""
    n = 150_000
    rng = np.random.default_rng(5)
    gg = GpuGraph(np.arange(n + 1, dtype=np.int64) * 110, rng.integers(0, n, size=110 * n).astype(np.int32), None)
    s = [rng.permutation(n)[:k].astype(np.int32) for k in sizes]
    samples = [110 * k if fanouts[0] < 0 else 0 for k in sizes]
    ws = [smfg.workspace_create(gg.g, k, fanouts, 0, e) for k, e in zip(sizes, samples)]
    outs = [smfg.alloc_output(gg.g, k, fanouts, edge_capacity=[e] if e else None) for k, e in zip(sizes, samples)]
    for turn in range(2):
        smfg.sample_mfg_many(gg.g, ws, [torch.from_numpy(x).to(DEV) for x in s], fanouts, [turn + 10 * b for b in range(len(s))], outs)
        for b, (x, out) in enumerate(zip(s, outs)):
            assert_same(fetch(out, len(fanouts)), gg.oracle.sample_mfg(x, fanouts, turn + 10 * b), len(fanouts))


def test_stages_of_launches_that_do_two():
    """A hop of the partition strategy draws and partitions in one launch, counted in both stages, with its time in the
    sampling; one of two levels is split in another."""
    gg = random_graph(400_000, 40, 21)
    for seeds, fan, splits in [(20_000, (10,), 0), (150_000, (20,), 1)]:
        s = torch.arange(seeds, dtype=torch.int32, device=DEV)
        ws = smfg.workspace_create(gg.g, seeds, fan)
        out = smfg.alloc_output(gg.g, seeds, fan)
        smfg.profile_begin(2, 100)
        try:
            smfg.sample_mfg(gg.g, ws, s, fan, 1, out)
        finally:
            prof = smfg.profile_end()
        assert prof["sample_insert"][1] == 1 and prof["sample_insert"][0] > 0
        assert prof["partition"][1] == 1 + splits


@pytest.mark.parametrize("strategy", ["partition", "table"])
@pytest.mark.parametrize("seeds,fanouts", [(131_072, (33, 33)), (131_073, (33, 33)), (70_000, (33, 5, 40))])
def test_wide_hops_of_many_tiles(seeds, fanouts, strategy, monkeypatch):
    """More destinations than a block adds up tile by tile (131072) in first and later hops, more samples (2 M) than 2048
    tiles of 1024 hold, and the same workspace again."""
    monkeypatch.setenv("SMFG_DEDUP", strategy)
    gg = random_graph(200_000, 30, 31)
    s = np.random.default_rng(seeds).permutation(200_000)[:seeds].astype(np.int32)
    ws = smfg.workspace_create(gg.g, seeds, fanouts)
    out = smfg.alloc_output(gg.g, seeds, fanouts)
    for key in (7, 8):
        smfg.sample_mfg(gg.g, ws, torch.from_numpy(s).to(DEV), fanouts, key, out)
        assert_same(fetch(out, len(fanouts)), gg.oracle.sample_mfg(s, fanouts, key), len(fanouts))


@pytest.mark.parametrize("strategy", ["partition", "table"])
@pytest.mark.parametrize("room,stray,status", [(-10, False, smfg.ST_EDGE_CAPACITY), (-10, True, smfg.ST_SEED_OUT_OF_RANGE),
                                               (0, True, smfg.ST_SEED_OUT_OF_RANGE), (0, False, 0)])
def test_wide_first_hop_that_does_not_fit(room, stray, status, strategy, monkeypatch):
    """Samples beyond the room of a batch, a stray seed, or both: nothing lies behind the buffers' ends, the stray seed is
    what is reported, and a call that fits is as ever."""
    monkeypatch.setenv("SMFG_DEDUP", strategy)
    gg = random_graph(5_000, 40, 32)
    s = np.random.default_rng(32).permutation(5_000)[:600].astype(np.int32)
    drawn = s[:599] if stray else s  # a stray seed has no samples
    edges = gg.oracle.sample_mfg(drawn, (-1,), 1).num_edges[0]
    capacity = edges + room
    bad = s.copy()
    if stray:
        bad[599] = 5_000
    ws = smfg.workspace_create(gg.g, 600, (-1,), 0, edges)
    out = smfg.alloc_output(gg.g, 600, (-1,), edge_capacity=[edges])
    out.indices[0].fill_(-7)
    out.c.edge_capacity[0] = capacity
    smfg.sample_mfg(gg.g, ws, torch.from_numpy(bad).to(DEV), (-1,), 1, out)
    assert fetch(out, 1)["status"] == status
    assert (out.indices[0][capacity:] == -7).all()
    smfg.sample_mfg(gg.g, ws, torch.from_numpy(s[:500]).to(DEV), (-1,), 1, out)
    assert_same(fetch(out, 1), gg.oracle.sample_mfg(s[:500], (-1,), 1), 1)


@pytest.mark.parametrize("later", [False, True])
def test_wide_hop_of_more_samples_than_room_and_nodes_than_slots(later, monkeypatch):
    """The table strategy, a hop whose samples do not fit, and which hold more nodes than the table has slots: nothing is looked up in a
    full table (0.1 ms; 30 with the samples that have room looked up), the samples are what is reported, and the next call on the workspace does not notice."""
    monkeypatch.setenv("SMFG_DEDUP", "table")
    gg = random_graph(200_000, 60, 33)
    perm = np.random.default_rng(33).permutation(200_000).astype(np.int32)
    fanouts, few, many = ((3, -1), 30, 1500) if later else ((-1,), 100, 6000)
    nodes, room = 8000, 60_000  # 16384 slots
    ref = gg.oracle.sample_mfg(perm[:many], fanouts, 1)
    assert ref.num_edges[-1] > room and (not later or ref.num_nodes[1] < nodes)
    ws = smfg.workspace_create(gg.g, many, fanouts, nodes, room)
    out = smfg.alloc_output(gg.g, many, fanouts, node_capacity=nodes, edge_capacity=[room] * len(fanouts))
    took = {}
    for seeds, status in ((few, 0), (many, smfg.ST_EDGE_CAPACITY), (few, 0), (many, smfg.ST_EDGE_CAPACITY)):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        smfg.sample_mfg(gg.g, ws, torch.from_numpy(perm[:seeds]).to(DEV), fanouts, 1, out)
        b.record()
        b.synchronize()
        took[seeds] = a.elapsed_time(b)
        got = fetch(out, len(fanouts))
        assert got["status"] == status
        if status == 0:
            assert_same(got, gg.oracle.sample_mfg(perm[:seeds], fanouts, 1), len(fanouts))
    assert took[many] < 1


@pytest.mark.parametrize("fanouts,seeds", [((15,), 68), ((15,), 69), ((1,), 640), ((1,), 641), ((4, 2), 256), ((4, 2), 257), ((31,), 33), ((31,), 34),
                                           ((1,), 2048), ((1,), 2049), ((31, 1), 128), ((31, 1), 129), ((3,), 1024), ((32, 3, 1), 1), ((7, 7), 0)])
def test_small_hops_settled_in_one_launch(fanouts, seeds):
    """First hops on both sides of 1280 records, 1024 samples and 4096 records, and hops behind them, one batch and several."""
    gg = random_graph(3_000, 40, 5, dim=9)
    keys = [3, 4, 5]
    s = [np.random.default_rng(k).permutation(3_000)[:n].astype(np.int32) for k, n in zip(keys, [seeds, (seeds + 1) // 2, min(seeds, 1)])]
    ws = [smfg.workspace_create(gg.g, len(x), fanouts) for x in s]
    outs = [smfg.alloc_output(gg.g, max(len(x), 1), fanouts) for x in s]
    for count in (1, 3):
        smfg.sample_mfg_many(gg.g, ws[:count], [torch.from_numpy(x).to(DEV) for x in s[:count]], fanouts, keys[:count], outs[:count])
        for x, key, out in list(zip(s, keys, outs))[:count]:
            assert_same(fetch(out, len(fanouts)), gg.oracle.sample_mfg(x, fanouts, key), len(fanouts))


@pytest.mark.parametrize("seeds", [40, 200])
def test_small_hops_settled_in_one_launch_that_fail(seeds):
    """Repeated and stray seeds and outputs too small, of first hops drawn in the same launch or before; the batches beside them and
    the next call do not notice."""
    gg = random_graph(5_000, 30, 8, dim=5)
    fan, perm = (10, 5), np.random.default_rng(4).permutation(5_000).astype(np.int32)
    s = [perm[i * 200:i * 200 + seeds].copy() for i in range(6)]
    s[1][seeds - 1] = s[1][0]
    s[2][seeds // 2], s[3][0] = 5_000, -1
    outs = [smfg.alloc_output(gg.g, seeds, fan) for _ in s]
    outs[4] = smfg.alloc_output(gg.g, seeds, fan, node_capacity=seeds + 1)
    outs[5] = smfg.alloc_output(gg.g, seeds, fan, edge_capacity=[seeds, 100_000])
    ws = [smfg.workspace_create(gg.g, seeds, fan) for _ in s]
    for _ in range(2):
        smfg.sample_mfg_many(gg.g, ws, [torch.from_numpy(x).to(DEV) for x in s], fan, range(6), outs)
        assert_same(fetch(outs[0], 2), gg.oracle.sample_mfg(s[0], fan, 0), 2)
        assert [fetch(o, 2)["status"] for o in outs[1:]] == [smfg.ST_DUPLICATE_SEED, smfg.ST_SEED_OUT_OF_RANGE, smfg.ST_SEED_OUT_OF_RANGE,
                                                            smfg.ST_NODE_CAPACITY, smfg.ST_EDGE_CAPACITY]


@pytest.mark.parametrize("d,seeds,batches", [(4, 257, 1), (5, 1, 1), (5, 513, 1), (8, 256, 2), (9, 255, 1), (9, 769, 16), (17, 300, 1), (32, 257, 1),
                                             (32, 4_000, 16), (20, 70_000, 1), (20, 140_000, 1)])
def test_tiles_shared_by_blocks(d, seeds, batches, monkeypatch):
    """Tiles of assemble whose positions one, two, four or eight blocks write, the last tile short, with and without a block's
    worth of positions for each."""
    monkeypatch.setenv("SMFG_DEDUP", "partition")
    gg = random_graph(150_000, 2 * d, d)
    s = [np.random.default_rng(b).permutation(150_000)[:seeds - 3 * b].astype(np.int32) for b in range(min(batches, seeds))]
    ws = [smfg.workspace_create(gg.g, seeds, (d,)) for _ in s]
    outs = [smfg.alloc_output(gg.g, seeds, (d,)) for _ in s]
    smfg.sample_mfg_many(gg.g, ws, [torch.from_numpy(x).to(DEV) for x in s], (d,), range(len(s)), outs)
    for b in range(0, len(s), 5):
        assert_same(fetch(outs[b], 1), gg.oracle.sample_mfg(s[b], (d,), b), 1)


@pytest.mark.parametrize("level", [1, 2])
@pytest.mark.parametrize("dim,folded", [(32, True), (3, False)])
def test_a_gather_without_a_launch_has_no_time(dim, folded, level):
    """Rows that the last hop's launch copies itself are counted as a gather; its time is that launch's."""
    gg = random_graph(20_000, 30, 17, dim=dim, dtype=np.float32)
    s = torch.arange(100, dtype=torch.int32, device=DEV)
    ws = smfg.workspace_create(gg.g, 100, (10, 5))
    out = smfg.alloc_output(gg.g, 100, (10, 5))
    smfg.profile_begin(level, 100)
    try:
        for key in range(3):
            smfg.sample_mfg(gg.g, ws, s, (10, 5), key, out)
    finally:
        prof = smfg.profile_end()
    assert prof["gather"][1] == 3 and (prof["gather"][0] == 0) == folded
    assert prof["assemble"][1] == (6 if level == 2 else 0) == prof["sample_insert"][1]
    again = smfg.profile_end()
    assert all(n == 0 for _, n in again.values())


@pytest.mark.parametrize("bad", ["stray", "twice"])
@pytest.mark.parametrize("strategy", ["", "partition", "table"])
@pytest.mark.parametrize("seeds,fanouts", [(60, (10, 5)), (200, (10, 5)), (1000, (7, 3)), (60, (40, 3)), (700, (33, 34)), (700, (-1,))])
def test_bad_seeds_leave_nothing_counted(seeds, fanouts, strategy, bad, monkeypatch):
    """Whatever draws the first hop: a batch with a stray or repeated seed counts its seeds and no node, nor a stray one's batch a sample."""
    monkeypatch.setenv("SMFG_DEDUP", strategy)
    gg = random_graph(5_000, 60, 34)
    s = np.random.default_rng(34).permutation(5_000)[:seeds].astype(np.int32)
    s[seeds // 2] = 5_000 if bad == "stray" else s[0]
    L, room = len(fanouts), 400_000 if min(fanouts) < 0 else 0
    ws = smfg.workspace_create(gg.g, seeds, fanouts, 0, room)
    out = smfg.alloc_output(gg.g, seeds, fanouts)
    smfg.sample_mfg(gg.g, ws, torch.from_numpy(s).to(DEV), fanouts, 1, out)
    want = [seeds] + [0] * (2 * L) + [smfg.ST_SEED_OUT_OF_RANGE if bad == "stray" else smfg.ST_DUPLICATE_SEED]
    got = fetch(out, L)["counts"]
    if bad == "twice" and max(fanouts[0], 64 * (fanouts[0] < 0)) > 32 and ws.strategy == "partition":
        got[L + 1] = 0  # told behind the draw, whose samples are counted
    assert got == want
