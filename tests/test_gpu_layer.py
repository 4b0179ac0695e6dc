"""The layer kernels at the edges of their tiles, lane groups and column slices."""
import numpy as np
import pytest
import torch

import oracle
from paper_2110_08450_amd import binding as smfg

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def block_of(rng, n_dst, fanout, n_src):
    k = rng.integers(0, fanout + 1, n_dst)
    k[rng.integers(0, n_dst)] = 0
    indptr = np.zeros(n_dst + 1, np.int32)
    indptr[1:] = np.cumsum(k)
    return indptr, rng.integers(0, n_src, max(1, int(indptr[-1])), dtype=np.int32)[:int(indptr[-1])]


def layer(indptr, indices, x, w, b, relu, out_dtype, spare=3):
    """The first n of n + spare rows of the block's arrays are destinations; the others' offsets are garbage."""
    n = len(indptr) - 1
    ip = torch.from_numpy(np.concatenate([indptr, np.full(spare, 2 ** 31 - 1, np.int32)])).to(DEV)
    ix = torch.from_numpy(indices if len(indices) else np.zeros(1, np.int32)).to(DEV)  # never without an address
    y = torch.full((n + spare, w.shape[0]), float("nan"), dtype=out_dtype, device=DEV)
    smfg.sage_layer(ip, ix, torch.tensor([n], device=DEV), n + spare, torch.from_numpy(x).to(DEV),
                    smfg.sage_pack_weights(torch.from_numpy(w).to(DEV)), torch.from_numpy(b).to(DEV), relu, y)
    assert torch.isnan(y[n:]).all()  # nothing written past the destinations
    return y[:n].float().cpu().numpy().astype(np.float64)


# tiles are of 64 (dim <= 64), 32 and up to 32 destinations; a block has 16 or more of them, 256 blocks
@pytest.mark.parametrize("n_dst,fanout,dim,out_dim,dtype", [
    (1, 1, 8, 1, torch.float32), (15, 4, 8, 31, torch.float16), (17, 5, 56, 33, torch.float16), (65, 6, 64, 256, torch.float16),
    (33, 5, 72, 32, torch.float32), (600, 11, 128, 255, torch.float16), (257, 16, 120, 256, torch.float32), (9001, 17, 128, 8, torch.float16),
    (16, 10, 136, 40, torch.float16), (4111, 21, 136, 256, torch.float32), (8229, 4, 256, 172, torch.float16), (300, 33, 248, 17, torch.float16),
    (130, 7, 16, 257, torch.float16), (70, 40, 128, 300, torch.float32), (33, 12, 256, 512, torch.float16), (20000, 3, 24, 24, torch.float16),
    (9001, 3, 64, 47, torch.float32), (12100, 2, 40, 65, torch.float16), (8500, 4, 128, 33, torch.float16), (8500, 4, 64, 129, torch.float32)])
def test_layer_edges(n_dst, fanout, dim, out_dim, dtype):
    """Bound: S (2^-11 + (2 dim + k + 2) 2^-24), S = sum of |w| |input| + |bias|: the mean rounded to half, then
    float sums; half an ulp of a half result."""
    check_layer(n_dst, fanout, dim, out_dim, dtype)


@pytest.mark.parametrize("max_dst,dim,out_dim", [(20_479, 136, 33), (20_480, 136, 33), (20_480, 256, 129), (65_535, 136, 129), (65_536, 136, 129),
                                                 (65_536, 256, 128), (65_536, 256, 129), (65_536, 128, 40)])
@pytest.mark.parametrize("n_dst", [1, 700])
def test_layer_either_side_of_reading_w_for_every_tile(max_dst, dim, out_dim, n_dst):
    check_layer(n_dst, 9, dim, out_dim, torch.float16, max_dst - n_dst)


def check_layer(n_dst, fanout, dim, out_dim, dtype, spare=3):
    rng = np.random.default_rng(n_dst + dim)
    n_src = n_dst + 50
    indptr, indices = block_of(rng, n_dst, fanout, n_src)
    x = rng.standard_normal((n_src, dim)).astype(np.float16)
    w = (rng.standard_normal((out_dim, 2 * dim)) / np.sqrt(dim)).astype(np.float16)
    b = rng.standard_normal(out_dim).astype(np.float32)
    relu = n_dst % 2 == 0
    got = layer(indptr, indices, x, w, b, relu, dtype, spare)
    want, mag = oracle.sage_layer(indptr, indices, x, w.astype(np.float64), b.astype(np.float64), relu)
    tol = mag * (2.0 ** -11 + (2 * dim + np.diff(indptr)[:, None] + 2) * 2.0 ** -24)
    if dtype == torch.float16:
        tol = tol + np.abs(want) * 2.0 ** -11 + 2.0 ** -24
    assert (np.abs(got - want) <= tol).all()


@pytest.mark.parametrize("dim", [8, 128, 136])
def test_layer_means_are_rounded_quotients(dim):
    """W picks one column of the mean, so the float result is the mean itself: the float sum in slot order,
    divided, rounded to half, bit for bit; an infinite sum stays infinite."""
    rng = np.random.default_rng(dim)
    n_dst, n_src = 2000, 3000
    indptr, indices = block_of(rng, n_dst, 70, n_src)
    x = (rng.standard_normal((n_src, dim)) * 10.0 ** rng.uniform(-6, 3, (n_src, 1))).astype(np.float16)
    w = np.zeros((dim, 2 * dim), np.float16)
    w[np.arange(dim), dim + np.arange(dim)] = 1
    got = layer(indptr, indices, x, w, np.zeros(dim, np.float32), False, torch.float32)
    for i in range(n_dst):
        s = np.zeros(dim, np.float32)
        for e in range(indptr[i], indptr[i + 1]):
            s = s + x[indices[e]].astype(np.float32)
        k = np.float32(max(1, indptr[i + 1] - indptr[i]))
        assert np.array_equal(got[i], (s / k).astype(np.float16).astype(np.float64))
    x[:] = np.inf
    got = layer(indptr, indices, x, np.ones((3, 2 * dim), np.float16), np.zeros(3, np.float32), False, torch.float32)
    assert np.isposinf(got).all()


def rows_of(deg, n_src, seed):
    indptr = np.zeros(len(deg) + 1, np.int32)
    indptr[1:] = np.cumsum(deg)
    return indptr, np.random.default_rng(seed).integers(0, n_src, int(indptr[-1]), dtype=np.int32)


# turns of 5 and 10 rows of a destination, ids of 8, 16 and 32 lanes, tiles with and without one, and a block's second tile
@pytest.mark.parametrize("dim", [16, 64, 72, 128, 144, 256])
def test_long_rows(dim):
    """As above for destinations of some thousand samples between short and empty ones: means bit for bit."""
    deg = np.concatenate([np.arange(64), np.repeat([0, 3, 4099, 1], 30), np.random.default_rng(dim).permutation(np.arange(20, 84)), [2500, 0, 6001]])
    deg = np.concatenate([deg, np.tile([1, 0, 2], 6000), deg])
    n_src = len(deg) + 100
    indptr, indices = rows_of(deg, n_src, dim)
    x = np.random.default_rng(dim + 1).standard_normal((n_src, dim)).astype(np.float16)
    w = np.zeros((dim, 2 * dim), np.float16)
    w[np.arange(dim), dim + np.arange(dim)] = 1
    got = layer(indptr, indices, x, w, np.zeros(dim, np.float32), False, torch.float32)
    rows = x[indices].astype(np.float32)
    for i in range(len(deg)):
        s = np.add.accumulate(rows[indptr[i]:indptr[i + 1]], axis=0, dtype=np.float32)[-1] if deg[i] else np.zeros(dim, np.float32)
        assert np.array_equal(got[i], (s / np.float32(max(1, deg[i]))).astype(np.float16).astype(np.float64)), (i, deg[i])


@pytest.mark.parametrize("dim,out_dim", [(64, 128), (128, 256)])
def test_long_rows_side_by_side(dim, out_dim):
    """Whole neighbourhoods: the destinations met first are the popular ones.  Twelve of 5000 samples, 32 apart, were the work of one
    block, one after the other, and took 5.6 and 10.8 times as long as 8000 apart; a block each, they take what they take anywhere."""
    n_dst, n_src = 100_000, 150_000
    x = torch.randn((n_src, dim), device=DEV).half()
    w = smfg.sage_pack_weights(torch.randn((out_dim, 2 * dim), device=DEV).half())
    num = torch.tensor([n_dst], device=DEV)
    y = torch.empty((n_dst, out_dim), dtype=torch.float16, device=DEV)
    took = []
    for apart in (32, 8000):
        deg = np.full(n_dst, 2)
        deg[np.arange(12) * apart] = 5000
        ip, ix = [torch.from_numpy(a).to(DEV) for a in rows_of(deg, n_src, 1)]
        best = float("inf")
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            smfg.sage_layer(ip, ix, num, n_dst, x, w, None, True, y)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        took.append(best)
    assert took[0] < 3 * took[1], took
