"""HIP library vs CPU oracle at the sizes where a kernel variant begins or ends (needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2110_08450_amd import binding as smfg
from test_gpu_parity import DEV, GpuGraph, assert_same, fetch

pytestmark = pytest.mark.gpu


def random_graph(n, max_deg, seed, dim=None, dtype=np.float16):
    """CSR rows of 0 .. max_deg neighbours each, a few of them popular; rows may repeat a neighbour."""
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, max_deg + 1, size=n)
    indptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(deg, out=indptr[1:])
    indices = (rng.random(int(indptr[-1])) ** 2 * n).astype(np.int32)
    feat = rng.standard_normal((n, dim)).astype(dtype) if dim else None
    return GpuGraph(indptr, indices, feat)


def sample(gg, seeds, fanouts, key):
    ws = smfg.workspace_create(gg.g, len(seeds), fanouts)
    out = smfg.alloc_output(gg.g, len(seeds), fanouts)
    smfg.sample_mfg(gg.g, ws, torch.from_numpy(seeds).to(DEV), fanouts, key, out)
    return fetch(out, len(fanouts)), ws.strategy


def launches(call):
    """Launches per stage of a call.  On the small path a hop counts once as sample_insert (a launch of its own for the
    first, done by the hop before for the others), dedup_buckets and assemble, the last of which may do the gather, and
    nothing comes before the first one."""
    smfg.profile_begin(2, 200)
    try:
        call()
    finally:
        prof = smfg.profile_end()
    return {stage: n for stage, (_, n) in prof.items() if n}


def small_launches(hops, features=True):
    return dict(sample_insert=hops, dedup_buckets=hops, assemble=hops, **({"gather": 1} if features else {}))


@pytest.mark.parametrize("fanout,seeds", [(8, 140_000), (9, 70_000), (16, 131_072), (17, 131_073), (32, 70_001)])
def test_draw_over_several_turns(fanout, seeds):
    """Row blocks of more destinations than one turn of the draw takes, fanouts on both sides of the
    register variants (8, 16, 32), degrees around the fanout."""
    gg = random_graph(150_000, 2 * fanout, fanout)
    s = np.random.default_rng(seeds).permutation(150_000)[:seeds].astype(np.int32)
    res, strategy = sample(gg, s, (fanout,), 0xABCDEF0123)
    assert strategy == "partition"
    assert_same(res, gg.oracle.sample_mfg(s, (fanout,), 0xABCDEF0123), 1)


@pytest.mark.parametrize("fanouts,planned,seeds", [((15, 10, 5), 600, 515), ((20, 20, 20), 515, 133), ((12, 7), 2060, 1295)])
def test_partition_workspace_made_for_more_seeds(fanouts, planned, seeds):
    """Fewer rows that would be cut into more row blocks than the workspace has counters for."""
    gg = random_graph(1_300_000, 30, 14)
    s = np.random.default_rng(seeds).permutation(1_300_000)[:seeds].astype(np.int32)
    ws = smfg.workspace_create(gg.g, planned, fanouts)
    assert ws.strategy == "partition"
    out = smfg.alloc_output(gg.g, seeds, fanouts)
    smfg.sample_mfg(gg.g, ws, torch.from_numpy(s).to(DEV), fanouts, 7, out)
    assert_same(fetch(out, len(fanouts)), gg.oracle.sample_mfg(s, fanouts, 7), len(fanouts))


@pytest.mark.parametrize("fanouts,seeds", [
    ((15, 10, 5), 31), ((15, 10, 5), 1), ((1,), 16383), ((1,), 16384), ((32,), 992), ((32,), 993), ((31, 3), 200),
    ((2,) * 8, 4), ((10, 5), 256), ((9, 8), 300), ((5,), 0), ((15, 10, 5), 1024), ((5, 100), 60), ((3, 40, 2), 900)])
def test_small_calls_and_hops(fanouts, seeds):
    """Calls and first hops on both sides of the small path's limit (32768 records of a hop), rows with
    and without a draw, several tiles of destinations, several rounds of the dedup, empty batches, hops
    of the other paths after a small one."""
    gg = random_graph(40_000, 40, 3, dim=6)
    s = np.random.default_rng(seeds).permutation(40_000)[:seeds].astype(np.int32)
    res, _ = sample(gg, s, fanouts, 5)
    assert_same(res, gg.oracle.sample_mfg(s, fanouts, 5), len(fanouts))


def small_bucket(node):
    """The bucket of 16 that k_small_dedup deals a node to (a 24-bit product, bits 20 to 23)."""
    x = (node ^ (node >> np.uint64(15))) & np.uint64(0xFFFFFF)
    return (x * np.uint64(0x79B1B5) >> np.uint64(20)) & np.uint64(15)


def test_small_call_with_a_hub_beyond_the_list():
    """6000 rows that all hold one hub: its bucket has more records than the list of 4096 that a block keeps
    of what it found, so the block reads the hop again in every round, with entries settled meanwhile."""
    n, hub = 60_000, 12_345
    rng = np.random.default_rng(21)
    rows = rng.integers(0, n, size=(n, 3)).astype(np.int32)
    rows[np.arange(n), rng.integers(0, 3, size=n)] = hub
    gg = GpuGraph(np.arange(n + 1, dtype=np.int64) * 3, rows.ravel(), None)
    for s in (rng.permutation(n)[:6_000].astype(np.int32), np.append(rng.permutation(hub)[:5_999], hub).astype(np.int32)):
        ws, out = smfg.workspace_create(gg.g, len(s), (3,)), smfg.alloc_output(gg.g, len(s), (3,))
        seeds = torch.from_numpy(s).to(DEV)
        assert launches(lambda: smfg.sample_mfg(gg.g, ws, seeds, (3,), 9, out)) == small_launches(1, features=False)
        assert_same(fetch(out, 1), gg.oracle.sample_mfg(s, (3,), 9), 1)


def test_small_call_table_overflows_and_retries():
    """20 000 distinct nodes of one bucket that share the three leading bits of the other hash: eight rounds
    are planned (20 000 / 8 records each, at most half a table of 8192 slots), but one gets all records and
    overflows the table; 16 rounds leave 10 000 nodes in one, 32 rounds 5000, which fit."""
    n = 1 << 22
    node = np.arange(n, dtype=np.uint64)
    h = (node * np.uint64(0x9E3779B1)) & np.uint64(0xFFFFFFFF)
    same = node[(small_bucket(node) == 5) & (h >> np.uint64(29) == 3)]
    assert len(same) >= 20_000
    same, h = same[:20_000], h[same[:20_000].astype(np.int64)]
    most = [np.bincount((h >> np.uint64(32 - lg)).astype(np.int64)).max() for lg in (3, 4, 5)]
    assert most[0] > 8192 and most[1] > 8192 > most[2]
    seeds, others = same[:10_000].astype(np.int32), same[10_000:]
    indptr = np.zeros(n + 1, dtype=np.int64)
    deg = np.zeros(n, dtype=np.int64)
    deg[seeds] = 1
    np.cumsum(deg, out=indptr[1:])
    gg = GpuGraph(indptr, others.astype(np.int32), None)
    s = np.random.default_rng(1).permutation(seeds)
    ws, out = smfg.workspace_create(gg.g, len(s), (1,)), smfg.alloc_output(gg.g, len(s), (1,))
    on_device = torch.from_numpy(s).to(DEV)
    assert launches(lambda: smfg.sample_mfg(gg.g, ws, on_device, (1,), 9, out)) == small_launches(1, features=False)
    assert_same(fetch(out, 1), gg.oracle.sample_mfg(s, (1,), 9), 1)


def test_small_launch_set_labels_and_status():
    """Ragged batches in one call, with labels; a batch with a repeated seed, one with a seed out of
    range and two whose output is too small end with their status and leave the others alone."""
    gg = random_graph(5_000, 30, 8, dim=5)
    labels = torch.arange(5_000, device=DEV, dtype=torch.int16) * 3
    smfg.graph_set_labels(gg.g, labels)
    fan = (10, 5)
    perm = np.random.default_rng(4).permutation(5_000).astype(np.int32)
    batches = [perm[:300], perm[300:317], perm[400:401], perm[500:600].copy(), perm[600:700].copy(), perm[700:800], perm[800:900]]
    batches[3][40] = batches[3][7]
    batches[4][11] = 5_000
    outs = [smfg.alloc_output(gg.g, len(b), fan) for b in batches]
    outs[5] = smfg.alloc_output(gg.g, 100, fan, node_capacity=400)
    outs[6] = smfg.alloc_output(gg.g, 100, fan, edge_capacity=[100, 100_000])
    wss = [smfg.workspace_create(gg.g, len(b), fan) for b in batches]
    keys = list(range(70, 77))
    for _ in range(2):  # the workspaces are as good after a status as before
        seeds = [torch.from_numpy(b).to(DEV) for b in batches]
        assert launches(lambda: smfg.sample_mfg_many(gg.g, wss, seeds, fan, keys, outs)) == small_launches(2)
        for i in range(3):
            assert_same(fetch(outs[i], 2), gg.oracle.sample_mfg(batches[i], fan, keys[i]), 2)
            assert torch.equal(outs[i].labels[:len(batches[i])].cpu(), labels.cpu()[torch.from_numpy(batches[i]).long()])
        assert [fetch(o, 2)["status"] for o in outs[3:]] == [smfg.ST_DUPLICATE_SEED, smfg.ST_SEED_OUT_OF_RANGE,
                                                            smfg.ST_NODE_CAPACITY, smfg.ST_EDGE_CAPACITY]


@pytest.mark.parametrize("sizes", [(256, 100), (256, 250), (31, 30, 1)])
def test_small_set_with_a_workspace_per_batch(sizes):
    """Workspaces planned for their own batch each, none with room for the largest one; twice, with other
    seeds, so that the second call finds what the first one left."""
    gg = random_graph(8_000, 30, 9, dim=5)
    fan = (10, 5)
    wss = [smfg.workspace_create(gg.g, n, fan) for n in sizes]
    assert all(w.strategy == "table" for w in wss)
    outs = [smfg.alloc_output(gg.g, n, fan) for n in sizes]
    for turn in range(2):
        rng = np.random.default_rng(turn)
        batches = [rng.permutation(8_000)[:n].astype(np.int32) for n in sizes]
        keys = [100 * turn + i for i in range(len(sizes))]
        seeds = [torch.from_numpy(b).to(DEV) for b in batches]
        assert launches(lambda: smfg.sample_mfg_many(gg.g, wss, seeds, fan, keys, outs)) == small_launches(2)
        for b, key, out in zip(batches, keys, outs):
            assert_same(fetch(out, 2), gg.oracle.sample_mfg(b, fan, key), 2)


@pytest.mark.parametrize("num_batches,own_gather,small", [(16, True, True), (16, False, False), (5, False, False), (4, False, True)])
def test_small_first_hop_of_a_larger_set(num_batches, own_gather, small):
    """Ragged sets whose first hop is small and whose second one is not, gathered by the call or by another one."""
    n, fan = 60_000, (6, 12)
    gg = random_graph(n, 24, 15)
    feat = torch.arange(n, dtype=torch.int32, device=DEV)[:, None].expand(n, 600).contiguous()
    g = smfg.graph_create(gg.indptr, gg.indices, feat)
    rng = np.random.default_rng(num_batches)
    batches = [rng.permutation(n)[:k].astype(np.int32) for k in rng.integers(500, 2_000, size=num_batches)]
    wss = [smfg.workspace_create(g, 2_000, fan) for _ in batches]
    assert all(w.strategy == "partition" for w in wss)
    outs = [smfg.alloc_output(g, 2_000, fan, with_features=own_gather) for _ in batches]
    seeds, keys = [torch.from_numpy(b).to(DEV) for b in batches], list(range(num_batches))
    for _ in range(2):
        ran = launches(lambda: smfg.sample_mfg_many(g, wss, seeds, fan, keys, outs, with_features=own_gather))
        assert ran["partition"] == (1 if small else 2) and ("seeds" in ran) == (not small)
        for b, key, out in zip(batches, keys, outs):
            ref = gg.oracle.sample_mfg(b, fan, key)
            got = fetch(out, 2)
            got.pop("features", None)
            assert_same(got, ref, 2)
            if own_gather:
                assert torch.equal(out.features[:got["n"][2]], feat[out.node_ids[:got["n"][2]].long()])


@pytest.mark.parametrize("forced", ["", "table", "partition"])
@pytest.mark.parametrize("fan", [(32,), (5, 3), (40, 2)])
def test_more_seeds_than_nodes(fan, forced, monkeypatch):
    """Such a batch holds a repeated seed or one that is no node, if only after every node was there once;
    it ends with that status, and the other batch of the call is as it should be."""
    monkeypatch.setenv("SMFG_DEDUP", forced)
    n = 100
    gg = random_graph(n, 60, 12, dim=5)
    perm = np.random.default_rng(6).permutation(n).astype(np.int32)
    good = perm[:40].copy()
    for seeds, status in [(np.append(perm, perm[3]), smfg.ST_DUPLICATE_SEED),
                          (np.append(perm, np.int32(n)), smfg.ST_SEED_OUT_OF_RANGE),
                          (np.append(np.int32(-1), perm), smfg.ST_SEED_OUT_OF_RANGE),
                          (np.tile(perm, 50), smfg.ST_DUPLICATE_SEED)]:
        batches = [good, seeds]
        wss = [smfg.workspace_create(gg.g, len(seeds), fan) for _ in batches]
        outs = [smfg.alloc_output(gg.g, len(b), fan, node_capacity=max(n, len(b))) for b in batches]
        smfg.sample_mfg_many(gg.g, wss, [torch.from_numpy(b).to(DEV) for b in batches], fan, [1, 2], outs)
        assert_same(fetch(outs[0], len(fan)), gg.oracle.sample_mfg(good, fan, 1), len(fan))
        assert fetch(outs[1], len(fan))["status"] == status


@pytest.mark.parametrize("strategy", ["table", "partition"])
def test_static_scratch_under_a_forced_strategy(strategy, monkeypatch):
    """The library's own scratch array, left by one strategy and shape and used by the next."""
    gg = random_graph(8_000, 30, 10, dim=5)
    rng = np.random.default_rng(3)
    for forced, fan, n in [(strategy, (10, 5), 200), ("", (6, 4), 150), (strategy, (10, 5), 120), (strategy, (40, 3), 50)]:
        monkeypatch.setenv("SMFG_DEDUP", forced)
        s = rng.permutation(8_000)[:n].astype(np.int32)
        out = smfg.alloc_output(gg.g, n, fan)
        ran = launches(lambda: smfg.sample_mfg_static(gg.g, torch.from_numpy(s).to(DEV), fan, n, out))
        assert (ran == small_launches(2)) == (forced == "")
        assert_same(fetch(out, 2), gg.oracle.sample_mfg(s, fan, n), 2)


def test_small_hop_of_a_wide_call_needs_room_for_padded_positions():
    """A wide call's workspace holds the samples that are drawn, not destinations x fanout: with room for
    1000 samples, 500 destinations of one neighbour each must not be laid out 20 apart."""
    n = 3_000
    rng = np.random.default_rng(2)
    gg = GpuGraph(np.arange(n + 1, dtype=np.int64), rng.integers(0, n, size=n).astype(np.int32), None)
    s, fan = rng.permutation(n)[:500].astype(np.int32), (20, 100)
    ws = smfg.workspace_create(gg.g, 500, fan, sample_capacity=1_000)
    out = smfg.alloc_output(gg.g, 500, fan)
    smfg.sample_mfg(gg.g, ws, torch.from_numpy(s).to(DEV), fan, 3, out)
    assert_same(fetch(out, 2), gg.oracle.sample_mfg(s, fan, 3), 2)


@pytest.mark.parametrize("dim", [8, 9, 15, 16, 17, 24, 31, 33, 100, 301, 12_345])
@pytest.mark.parametrize("shift", [0, 1, 3])
def test_gather_rows_at_any_address(dim, shift):
    """2-byte elements from a wider table at an odd column, into an output that starts `shift` elements
    after an aligned address: every alignment of source and output, rows shorter than, equal to and
    just beyond whole 16-byte vectors, a partial last block, nothing written outside."""
    n, rows = 300, 131
    table = torch.randint(-30_000, 30_000, (n, dim + 5), dtype=torch.int16, device=DEV)
    feat = table[:, shift:shift + dim]
    g = smfg.graph_create(torch.zeros(n + 1, dtype=torch.int64, device=DEV), torch.zeros(1, dtype=torch.int32, device=DEV)[:0], feat)
    ids = torch.randint(0, n, (rows,), dtype=torch.int32, device=DEV)
    flat = torch.full((shift + (rows + 2) * dim,), 31_000, dtype=torch.int16, device=DEV)
    out = flat[shift:].view(rows + 2, dim)
    smfg.gather_rows(g, ids, torch.tensor([rows], device=DEV), rows + 2, out)
    torch.cuda.synchronize()
    assert torch.equal(out[:rows], feat[ids.long()])
    assert (out[rows:] == 31_000).all() and (flat[:shift] == 31_000).all()


@pytest.mark.parametrize("dim,dtype,rows", [(600_000_003, torch.int64, 2), ((1 << 30) + 5, torch.int16, 33)])
def test_gather_rows_beyond_32_bits(dim, dtype, rows):
    """Rows of 4.8 GB, and more rows of 2 GiB than a block of ordinary rows takes."""
    table = torch.empty((2, dim), dtype=dtype, device=DEV).random_()
    indptr = torch.tensor([0, 1, 1], dtype=torch.int64, device=DEV)
    g = smfg.graph_create(indptr, torch.ones(1, dtype=torch.int32, device=DEV), table)
    ids = (torch.arange(rows, dtype=torch.int32, device=DEV) + 1) % 2
    out = torch.zeros((rows, dim), dtype=dtype, device=DEV)
    smfg.gather_rows(g, ids, torch.tensor([rows], device=DEV), rows, out)
    for i in range(rows):
        assert torch.equal(out[i], table[(i + 1) % 2])
    del out
    sampled = smfg.alloc_output(g, 2, (1,))
    smfg.sample_mfg(g, smfg.workspace_create(g, 2, (1,)), ids[:2].contiguous(), (1,), 1, sampled)
    assert smfg.read_counts(sampled)[:2] == [2, 2]
    assert torch.equal(sampled.features[0], table[1]) and torch.equal(sampled.features[1], table[0])
    del sampled, table, g
    torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
@pytest.mark.parametrize("dim,shift", [(3, 1), (4, 1), (7, 0), (8, 1), (9, 0), (128, 1), (129, 0), (131, 3)])
def test_mean_aggregate_at_any_address(dim, shift, dtype):
    """Rows of any width from any element on; columns that two lanes compute; nothing written outside.
    Small whole numbers and row lengths of 1, 2 and 4: every sum and quotient is exact."""
    gen = torch.Generator().manual_seed(dim)
    src, lens = 90, torch.tensor([0, 1, 2, 4] * 16 + [4])
    flat = torch.randint(-50, 50, (shift + src * dim,), generator=gen).to(dtype).to(DEV)
    x = flat[shift:].view(src, dim)
    indptr = torch.cat([torch.zeros(1, dtype=torch.int64), torch.cumsum(lens, 0)])
    indices = torch.randint(0, src, (int(indptr[-1]),), generator=gen)
    out = torch.full((len(lens) + 1, dim), 7.5, dtype=torch.float32, device=DEV)
    smfg.mean_aggregate(indptr.to(torch.int32).to(DEV), indices.to(torch.int32).to(DEV), torch.tensor([len(lens)], device=DEV),
                        len(lens), x, out)
    torch.cuda.synchronize()
    h = x.float().cpu()
    want = torch.stack([h[indices[a:b]].sum(0) / max(1, b - a) for a, b in zip(indptr[:-1].tolist(), indptr[1:].tolist())])
    assert torch.equal(out[:-1].cpu(), want) and (out[-1] == 7.5).all()


@pytest.mark.parametrize("seeds", [262_144, 262_145])
def test_assemble_with_and_without_its_own_scan(seeds):
    """1024 tiles of 256 destinations, the most that every block scans for itself, and one more."""
    gg = random_graph(300_000, 4, 11)
    s = np.random.default_rng(seeds).permutation(300_000)[:seeds].astype(np.int32)
    res, _ = sample(gg, s, (2,), 17)
    assert_same(res, gg.oracle.sample_mfg(s, (2,), 17), 1)


@pytest.mark.parametrize("fanout", [33, 64, 65, 128, 129, 1000, 1024])
def test_wide_draw_with_its_hash_table(fanout):
    """Both sides of the sizes at which a row's table of drawn values grows, degrees just above the
    fanout, where many draws repeat or refer to an earlier slot, and far above it."""
    rng = np.random.default_rng(fanout)
    n = 6_000
    deg = np.concatenate([rng.integers(fanout - 3, fanout + 40, size=40), rng.integers(0, 5 * fanout, size=40),
                          np.zeros(n - 80, dtype=np.int64)])
    indptr = np.zeros(n + 1, dtype=np.int64)
    np.cumsum(deg, out=indptr[1:])
    gg = GpuGraph(indptr, rng.integers(0, n, size=int(indptr[-1])).astype(np.int32), None)
    s = rng.permutation(80).astype(np.int32)
    res, _ = sample(gg, s, (fanout,), 31)
    assert_same(res, gg.oracle.sample_mfg(s, (fanout,), 31), 1)
