"""The SpMM's lane layouts with several entries per load instruction, at the
edges of their blocks of steps, register pairs, 64-entry runs and long rows:
against the oracle, with infinities and NaN in B rows that no entry uses, and
the forms with 32-bit and 64-bit addresses (and with the hub hint) against
each other bit for bit."""
import os

import numpy as np
import pytest
import torch

import oracle
import paper_2210_10737_amd as rsc
import synth

pytestmark = pytest.mark.gpu
FLT_MIN = np.float32(np.finfo(np.float32).tiny)
LENS = [0, 1, 2, 3, 4, 5, 7, 8, 9, 12, 13, 15, 16, 17, 24, 25, 31, 32, 33, 40, 47, 48, 49, 56, 57, 63, 64, 65, 96,
        127, 128, 129, 1023, 1024, 1025, 1088, 1089]


@pytest.fixture(scope="module", autouse=True)
def _gpu(gpu):
    yield


def ragged(n_cols, seed):
    lens = np.array(LENS * 3)
    np.random.default_rng(seed).shuffle(lens)
    return synth.bucket_csr(lens, n_cols, seed=seed)


@pytest.mark.parametrize("d", [1, 4, 13, 16, 17, 32, 33, 41, 64, 65, 100, 128])
def test_layout_edges(d):
    n_cols = 1300
    A = ragged(n_cols, seed=d)
    B = synth.dense_normal(n_cols + 2, d, seed=50 + d, ld=(d + 3) // 4 * 4 + 4)
    # the first and last rows of B are no entry's: what stands in for an
    # entry past the end of a run must not reach a sum
    col = A.col + 1
    B[0], B[-1] = np.inf, np.nan
    X = rsc.DeviceCsr.from_host(A.rowptr, col, A.val, n_cols + 2)
    Y = rsc.spmm(X, torch.from_numpy(B).cuda(), d=d).cpu().numpy()
    Yo, S = oracle.spmm(A.rowptr, col, A.val, B, d=d, with_mag=True)
    # a group's fp32 chain has at most 64 / G entries, G = 16 .. 2 for the
    # 16- .. 128-float layouts; then the groups' tree and one rounding
    chain = {16: 4, 32: 8, 64: 16, 128: 32}[next(w for w in (16, 32, 64, 128) if d <= w)]
    err = np.max(np.abs(Y.astype(np.float64) - Yo) / np.maximum(S, FLT_MIN))
    assert err <= (chain + 6) * 2.0 ** -24, (d, err)


@pytest.mark.parametrize("d", [16, 30, 64, 100])
def test_wide_addresses(d):
    """An operand of more than 4 GiB between its first and last row is read
    with 64-bit addresses: the same sums as its compact copy's."""
    n_cols = 1_100_000
    A = synth.bucket_csr(np.array(LENS * 2), n_cols, seed=3)
    Bc = torch.from_numpy(synth.dense_normal(n_cols, (d + 3) // 4 * 4, seed=4)).cuda()
    wide = torch.zeros((n_cols, 1024), dtype=torch.float32, device="cuda")
    wide[:, :Bc.shape[1]] = Bc
    X = rsc.DeviceCsr.from_host(A.rowptr, A.col, A.val, n_cols)
    assert torch.equal(rsc.spmm(X, wide, d=d), rsc.spmm(X, Bc, d=d))


@pytest.mark.parametrize("d", [64, 100, 128])
def test_hinted_layouts(d):
    """A plan whose gathers take the hub hint (B over 512 MiB) adds in the
    order of the unhinted form."""
    n_cols = 2_200_000
    A = synth.bucket_csr(np.array(LENS * 40), n_cols, seed=6)
    B = torch.from_numpy(synth.dense_normal(n_cols, d, seed=8)).cuda()
    assert B.numel() * 4 > 512 << 20
    X = rsc.DeviceCsr.from_host(A.rowptr, A.col, A.val, n_cols)
    os.environ.pop("RSC_SPMM_HINT", None)
    plan = rsc.SpmmPlan(X)
    assert torch.equal(plan.run(B), rsc.spmm(X, B))
    plan.close()


@pytest.mark.parametrize("d", [16, 41, 100, 200, 300])
def test_long_rows_listed_or_found(d):
    """Long rows come from a plan's list or are found by the block that holds
    them, also in the last, partial block: one result, the oracle's."""
    n_cols = 4000
    for tail in range(4):   # 0 to 3 rows in the last block, long ones among them
        lens = np.array([5, 1025, 3, 0, 2, 2000, 1100, 1026] + [1500, 1, 1030][:tail])
        A = synth.bucket_csr(lens, n_cols, seed=60 + tail)
        B = synth.dense_normal(n_cols, d, seed=61, ld=(d + 3) // 4 * 4)
        Bd = torch.from_numpy(B).cuda()
        X = rsc.DeviceCsr.from_host(A.rowptr, A.col, A.val, n_cols)
        Y = rsc.spmm(X, Bd, d=d)
        plan = rsc.SpmmPlan(X)
        assert torch.equal(plan.run(Bd, d=d), Y), (d, tail)
        plan.close()
        Yo, S = oracle.spmm(A.rowptr, A.col, A.val, B, d=d, with_mag=True)
        # a 64-entry fp32 chain at most, then fp64
        assert np.max(np.abs(Y.cpu().numpy().astype(np.float64) - Yo) / np.maximum(S, FLT_MIN)) <= 66 * 2.0 ** -24


def test_wide_blocks():
    """Mean row of 32 entries and 16,384 rows: 8 waves per block, with long
    rows, against one row fewer (4 waves) and the oracle."""
    n = 16384
    lens = np.full(n, 33)
    lens[[0, 7, 8, 5000, n - 1]] = [1025, 2000, 1030, 1500, 1100]
    A = synth.bucket_csr(lens, 3000, seed=71)
    B = synth.dense_normal(3000, 200, seed=72)
    Bd = torch.from_numpy(B).cuda()
    X = rsc.DeviceCsr.from_host(A.rowptr, A.col, A.val, 3000)
    Y = rsc.spmm(X, Bd)
    plan = rsc.SpmmPlan(X)
    assert torch.equal(plan.run(Bd), Y)
    plan.close()
    m = int(A.rowptr[n - 1])
    X1 = rsc.DeviceCsr.from_host(A.rowptr[:n], A.col[:m], A.val[:m], 3000)
    short = torch.from_numpy(np.flatnonzero(lens[:-1] <= 1024)).cuda()
    assert torch.equal(rsc.spmm(X1, Bd)[short], Y[:-1][short])   # a short row is one wave's in both
    Yo, S = oracle.spmm(A.rowptr, A.col, A.val, B, with_mag=True)
    assert np.max(np.abs(Y.cpu().numpy().astype(np.float64) - Yo) / np.maximum(S, FLT_MIN)) <= 66 * 2.0 ** -24


def _side_by_side(n_rows, first, count, n_cols, seed):
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 4, n_rows)
    lens[first:first + count] = rng.integers(1025, 1400, count)
    return synth.bucket_csr(lens, n_cols, seed=seed)


@pytest.mark.parametrize("d", [130, 200, 256, 257, 300, 512, 600])
def test_long_rows_halved(d):
    """Long rows of 129 and more features, halved over two blocks: through a
    descriptor, with 64-bit addresses (an operand of more than 4 GiB) and with
    the hub hint (B over 512 MiB), the same bits; NaN in the B rows and
    features that no entry or output uses."""
    n_cols = 1_100_000
    A = synth.bucket_csr(np.array([1024, 1025, 3, 1088, 5, 0, 2000, 64, 65, 1500, 1026]), n_cols - 2, seed=d)
    col = A.col + 1
    wide = torch.full((n_cols, 1024), float("nan"), device="cuda")
    wide[1:-1, :d] = torch.randn((n_cols - 2, d), generator=torch.Generator("cuda").manual_seed(d), device="cuda")
    B = wide[:, :(d + 3) // 4 * 4].contiguous()
    X = rsc.DeviceCsr.from_host(A.rowptr, col, A.val, n_cols)
    Y = rsc.spmm(X, B, d=d)
    assert torch.equal(rsc.spmm(X, wide, d=d), Y)
    plan = rsc.SpmmPlan(X)
    assert torch.equal(plan.run(B, d=d), Y)
    plan.close()
    used = np.unique(col)
    Bh = np.zeros((n_cols, d), np.float32)
    Bh[used] = B[torch.from_numpy(used.astype(np.int64)).cuda(), :d].cpu().numpy()
    Yo, S = oracle.spmm(A.rowptr, col, A.val, Bh, d=d, with_mag=True)
    err = np.max(np.abs(Y.cpu().numpy().astype(np.float64) - Yo) / np.maximum(S, FLT_MIN))
    assert err <= 66 * 2.0 ** -24   # a 64-entry fp32 chain at most, then fp64


@pytest.mark.parametrize("n_rows,first,count", [
    (5000, 0, 600),              # more blocks look than there are groups of 256 rows
    (4099, 4000, 99),            # up to the last row
    (262_143, 262_043, 100),     # the most rows that are looked at, one a thread
    (262_144, 262_044, 100),     # the fewest that are listed
    (70_000, 0, 8),
])
@pytest.mark.parametrize("d", [30, 100, 200, 300])
def test_long_rows_side_by_side(n_rows, first, count, d):
    """Long rows in one run of rows: found by the blocks that look for them,
    listed, or from a plan, the same bits, and the oracle's values."""
    n_cols = 3000
    A = _side_by_side(n_rows, first, count, n_cols, seed=n_rows % 1000 + d)
    B = synth.dense_normal(n_cols, d, seed=62, ld=(d + 3) // 4 * 4)
    Bd = torch.from_numpy(B).cuda()
    X = rsc.DeviceCsr.from_host(A.rowptr, A.col, A.val, n_cols)
    Y = rsc.spmm(X, Bd, d=d)
    plan = rsc.SpmmPlan(X)
    assert torch.equal(plan.run(Bd, d=d), Y)
    plan.close()
    rows = np.unique(np.r_[np.arange(first, first + count), np.arange(0, n_rows, 211)]).astype(np.int32)
    Yo, S = oracle.spmm(A.rowptr, A.col, A.val, B, rows=rows, d=d, with_mag=True)
    err = np.max(np.abs(Y.cpu().numpy()[rows].astype(np.float64) - Yo) / np.maximum(S, FLT_MIN))
    assert err <= 66 * 2.0 ** -24   # a 64-entry fp32 chain at most, then fp64


@pytest.mark.parametrize("d", [16, 32, 64])
def test_long_pieces_side_by_side(d):
    """Column-blocked: long pieces in a run of rows, over the edges of the
    windows that share them out and in the last, partial one."""
    n_cols = 4000
    lens = np.random.default_rng(5).integers(0, 40, 5001)
    lens[1000:1300] = 3500
    lens[4980:] = 3300
    A = synth.bucket_csr(lens, n_cols, seed=63)
    B = synth.dense_normal(n_cols, d, seed=64)
    X = rsc.DeviceCsr.from_host(A.rowptr, A.col, A.val, n_cols)
    old = os.environ.get("RSC_SPMM_BLOCKED")
    os.environ["RSC_SPMM_BLOCKED"] = "2"
    try:
        Y = rsc.spmm(X, torch.from_numpy(B).cuda()).cpu().numpy()
    finally:
        os.environ.pop("RSC_SPMM_BLOCKED") if old is None else os.environ.update(RSC_SPMM_BLOCKED=old)
    Yo, S = oracle.spmm(A.rowptr, A.col, A.val, B, with_mag=True)
    # as above, and each of the two partial rows rounded once
    assert np.max(np.abs(Y.astype(np.float64) - Yo) / np.maximum(S, FLT_MIN)) <= 67 * 2.0 ** -24


@pytest.mark.parametrize("d", [41, 256])
def test_sorted_hubs_cost_what_scattered_ones_cost(d):
    """Rows sorted by length put the hubs side by side; without a plan they
    must still go to as many blocks as the same rows in any order (in as many
    blocks as four rows fill, they took three and a half times as long)."""
    n = 60_013
    lens = np.minimum(16.0 * ((np.arange(n) + 0.5) / n) ** (-1 / 1.1) / 7, 30_000).astype(np.int64) + 1
    B = torch.from_numpy(synth.dense_normal(n, (d + 3) // 4 * 4, seed=7)).cuda()
    times = []
    for order in (np.arange(n), np.random.default_rng(2).permutation(n)):
        A = synth.bucket_csr(lens[order], n, seed=8)
        X = rsc.DeviceCsr.from_host(A.rowptr, A.col, A.val, n)
        ws = torch.empty(rsc.spmm_workspace_bytes(X), dtype=torch.uint8, device="cuda")
        Y = rsc.spmm(X, B, d=d, ws=ws)
        best = float("inf")
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(4):
                rsc.spmm(X, B, d=d, out=Y, ws=ws)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
    assert times[0] <= 1.6 * times[1], times


def test_one_long_row_costs_its_bytes():
    """A row that outweighs all others is one block's serial chain: with four
    times the features it may take little more than four times as long (nine
    times, with the gathers of four waves in flight)."""
    n_cols = 1_000_000
    lens = np.full(1000, 4)
    lens[500] = 300_000
    A = synth.bucket_csr(lens, n_cols, seed=9)
    X = rsc.DeviceCsr.from_host(A.rowptr, A.col, A.val, n_cols)
    best = {}
    for d in (64, 256):
        B = torch.randn((n_cols, d), device="cuda")
        Y = rsc.spmm(X, B)
        best[d] = float("inf")
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            rsc.spmm(X, B, out=Y)
            b.record()
            b.synchronize()
            best[d] = min(best[d], a.elapsed_time(b))
    assert best[256] <= 5 * best[64], best
