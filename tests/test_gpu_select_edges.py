"""Top-k and column slice at the sizes where their launches change: tiles per
thread block, counts added tile by tile or by groups of tiles, the small
forms, and searches that end before the last digit. Bit for bit against torch
or the oracle; everything here is integer or copied."""
import ctypes
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2210_10737_amd as rsc
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu):
    yield


def check_topk(key, k):
    n = key.numel()
    idx, mask = rsc.topk_select(key, k)
    # keys are below 2^63 here, so int64 order is their order; stable: ties by index
    want = torch.sort(torch.sort(key, descending=True, stable=True).indices[:k]).values
    assert torch.equal(idx.long(), want), (n, k)
    bits = torch.zeros((n + 31) // 32 * 32, dtype=torch.int64, device="cuda")
    bits[want] = 1
    words = (bits.view(-1, 32) << torch.arange(32, device="cuda")).sum(1)
    assert torch.equal(mask.long() & 0xFFFFFFFF, words), (n, k)


@pytest.mark.parametrize("n", [1, 31, 33, 4095, 4096, 4097, 16383, 16384, 16385, 17409, (1 << 20) - 1, 1 << 20,
                               (1 << 20) + 1, 3_000_001])
@pytest.mark.parametrize("kind", ["spread", "ties", "low_bits", "equal"])
def test_topk_sizes(n, kind):
    g = torch.Generator(device="cuda").manual_seed(n)
    if kind == "spread":      # ends after a few digits
        key = torch.rand(n, generator=g, dtype=torch.float64, device="cuda").view(torch.int64) + 1
    elif kind == "ties":      # few distinct keys: the wanted bin is never whole
        key = torch.randint(0, 5, (n,), generator=g, device="cuda") * (1 << 40) + 3
    elif kind == "low_bits":  # differ in the last digit only
        key = torch.randint(0, 1 << 10, (n,), generator=g, device="cuda") + (1 << 61)
    else:
        key = torch.full((n,), 77, dtype=torch.int64, device="cuda")
    for k in sorted({1, n // 3, n - 1, n} - {0}):
        check_topk(key, k)


def test_topk_many_tiles():
    """More tiles than the emit's blocks add one by one."""
    n = 8193 * 4096
    g = torch.Generator(device="cuda").manual_seed(1)
    check_topk(torch.randint(0, 1 << 62, (n,), generator=g, device="cuda") >> 20, n // 3)


@pytest.mark.parametrize("n_cols", [31, 131_072, 131_073])
@pytest.mark.parametrize("nnz", [1, 4096, 4097, 256 * 4096, 256 * 4096 + 1, 2048 * 4096, 2048 * 4096 + 1])
def test_slice_sizes(n_cols, nnz):
    row = min(n_cols, 700)
    lens = np.full((nnz + row - 1) // row, row)
    lens[-1] -= lens.sum() - nnz
    lens = np.concatenate([[0], lens, [0, 0]])
    A = synth.bucket_csr(lens, n_cols, seed=nnz % 1000)
    X = rsc.DeviceCsr.from_host(A.rowptr, A.col, A.val, n_cols)
    rng = np.random.default_rng(nnz)
    keep = rng.random(n_cols) < 0.4
    words = np.zeros((n_cols + 31) // 32, np.uint32)
    np.bitwise_or.at(words, np.arange(n_cols) // 32, keep.astype(np.uint32) << (np.arange(n_cols) % 32).astype(np.uint32))
    S, nnz_out = rsc.slice_csr(X, torch.from_numpy(words.view(np.int32)).cuda())
    ro, co, vo = oracle.slice_csr(A.rowptr, A.col, A.val, words)
    m = int(nnz_out.item())
    assert m == len(co)
    assert np.array_equal(S.rowptr.cpu().numpy(), ro)
    assert np.array_equal(S.col[:m].cpu().numpy(), co)
    assert np.array_equal(S.val[:m].cpu().numpy().view(np.uint32), vo.view(np.uint32))


@pytest.mark.parametrize("n_rows,launches", [(4096, 2), (4097, 4), (8192, 2), (8193, 4), (300_000, 4)])
def test_slice_of_mostly_empty_rows(n_rows, launches):
    """The two-launch slice marks the rows with its tiles' threads, so more
    rows than 4,096 a tile take the form with a pass of its own for them."""
    n_cols, nnz = 5000, 4096 if n_rows < 5000 else 8192
    lens = np.bincount(np.random.default_rng(n_rows).integers(0, n_rows, nnz), minlength=n_rows)
    A = synth.bucket_csr(lens, n_cols, seed=n_rows % 1000)
    X = rsc.DeviceCsr.from_host(A.rowptr, A.col, A.val, n_cols)
    words = np.random.default_rng(1).integers(0, 1 << 32, (n_cols + 31) // 32, dtype=np.uint64).astype(np.uint32)
    words[-1] &= np.uint32((1 << n_cols % 32) - 1)
    mask = torch.from_numpy(words.view(np.int32)).cuda()
    S, nnz_out = rsc.slice_csr(X, mask)
    ro, co, vo = oracle.slice_csr(A.rowptr, A.col, A.val, words)
    m = int(nnz_out.item())
    assert m == len(co) and np.array_equal(S.rowptr.cpu().numpy(), ro)
    assert np.array_equal(S.col[:m].cpu().numpy(), co)
    assert np.array_equal(S.val[:m].cpu().numpy().view(np.uint32), vo.view(np.uint32))
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        rsc.slice_csr(X, mask)
    n = ctypes.c_size_t()
    assert rsc.lib().hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    assert n.value == launches


@pytest.mark.parametrize("n,d", [(1, 4), (63, 100), (65, 64), (64, 65), (65_536, 96), (65_536, 100), (65_537, 100), (70_001, 64)])
def test_scores_rows_per_block(n, d):
    """Keys and row norms over both block sizes and both load policies, bit
    for bit."""
    ld = (d + 3) // 4 * 4
    B = synth.dense_normal(n, d, seed=n, ld=ld)
    cn2 = np.random.default_rng(n).random(n)
    key, rn2 = rsc.pair_scores(torch.from_numpy(cn2).cuda(), torch.from_numpy(B).cuda(), d=d, with_rn2=True)
    want = oracle.pair_keys(cn2, B, d=d)
    assert np.array_equal(key.cpu().numpy().view(np.uint64), want["key"])
    assert np.array_equal(rn2.cpu().numpy().view(np.uint64), want["rn2"].view(np.uint64))


@pytest.mark.parametrize("n", [1, 255, 257, 8191, 8192, 8193, 16_384, 16_385])
def test_norm_totals(n):
    """The norms' totals over one block of 8,192 terms, which is stored by
    itself, and over several: within (n - 1) u of the exact sum, twice the
    same bits."""
    val = np.random.default_rng(n).standard_normal(n).astype(np.float32)
    X = rsc.DeviceCsr.from_host(np.arange(n + 1), np.arange(n), val, n)
    B = synth.dense_normal(n, 8, seed=n)
    cache = rsc.Cache(X, X)
    Bd = torch.from_numpy(B).cuda()
    cache.score(Bd)
    totals = cache.norms()
    rn2 = oracle.pair_keys(val.astype(np.float64) ** 2, B)["rn2"]
    for got, terms in zip(totals, (val.astype(np.float64) ** 2, rn2)):
        want = math.fsum(terms)
        # (n - 1) roundings of the sum, and one of the exact sum
        assert abs(got - want) <= n * 2.0 ** -53 * want, n
    cache.score(Bd)
    assert cache.norms() == totals
    cache.close()


def test_previous_selection_is_kept():
    """The selection a refresh replaces, for n in the one-block and the tiled
    selection, top-k after randomized and k = 0 after top-k."""
    for n in (3000, 20_000):
        A = synth.erdos_renyi(n, 6.0 / n, seed=n)
        X = rsc.DeviceCsr.from_host(A.rowptr, A.col, A.val, n)
        B = torch.from_numpy(synth.dense_normal(n, 16, seed=n + 1)).cuda()
        cache = rsc.Cache(X, X)
        order = torch.randperm(n, device="cuda").int()

        def mask():
            w = rsc.copy_to_host(cache.buffers()[4], (n + 31) // 32, np.uint32)
            return np.unpackbits(w.view(np.uint8), bitorder="little")[:n].astype(bool)

        masks = []
        for step, how in enumerate(["random", "topk", "none", "topk"]):
            if how == "random":
                cache.refresh_random(B, n // 4, 5, step)
            else:
                cache.refresh(B, 0 if how == "none" else n // 5 + step, step)
            masks.append(mask())
            if step:
                _, both, prev_k = cache.staleness(order)
                assert prev_k == masks[-2].sum() and both == (masks[-2] & masks[-1]).sum(), (n, step)
        cache.close()


@pytest.mark.parametrize("n", [1, 2, 255, 257, 1023, 1024, 1025, 65_537, 1024 * 8192, 1024 * 8192 + 1])
def test_sampler_tile_edges(n):
    """The sampler's CDF around its tiles of 1,024 columns, around the 256
    block maxima, and on both sides of 8,192 tiles, from which on the tile
    sums are scanned by a launch of their own: whole numbers, the oracle's."""
    rng = np.random.default_rng(n)
    key = (rng.random(n) ** 3 + 1e-12).view(np.uint64) + np.uint64(1)
    key[rng.random(n) < 0.2] = 0
    key[n - 1] = np.uint64(0x4010000000000001)  # the largest one last
    k = min(n, 50_000) + 3
    o = oracle.sample_columns(key, k, n)
    count, colw, mask = rsc.sample_columns(torch.from_numpy(key.view(np.int64)).cuda(), k, n)
    assert np.array_equal(count.cpu().numpy(), o["count"])
    assert np.array_equal(colw.cpu().numpy().view(np.uint64), o["colw"].view(np.uint64))
    assert np.array_equal(mask.cpu().numpy().view(np.uint32), o["mask"])
