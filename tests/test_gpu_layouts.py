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
