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


@pytest.mark.parametrize("fanout,seeds", [(8, 140_000), (9, 70_000), (16, 131_072), (17, 131_073), (32, 70_001)])
def test_draw_over_several_turns(fanout, seeds):
    """Row blocks of more destinations than one turn of the draw takes, fanouts on both sides of the
    register variants (8, 16, 32), degrees around the fanout."""
    gg = random_graph(150_000, 2 * fanout, fanout)
    s = np.random.default_rng(seeds).permutation(150_000)[:seeds].astype(np.int32)
    res, strategy = sample(gg, s, (fanout,), 0xABCDEF0123)
    assert strategy == "partition"
    assert_same(res, gg.oracle.sample_mfg(s, (fanout,), 0xABCDEF0123), 1)
