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
