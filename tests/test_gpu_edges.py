"""GPU parity at the edges of the kernels' work splits and of the dispatch
rules, against the oracle: structure bit-exact and, since every c_ij takes its
terms in ascending k with rounded products as the oracle does, values
bit-exact too."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

mls = pytest.importorskip("paper_1804_00695_amd")


def check(A, B):
    C = mls.spgemm(mls.DeviceCsr.from_host(A), mls.DeviceCsr.from_host(B))
    mls.check_errors()
    rp, ci, v = C.numpy()
    R, _ = oracle.spgemm(A, B)
    assert np.array_equal(rp, R.row_ptr) and np.array_equal(ci, R.col_idx)
    assert np.array_equal(v, R.values)
    return R


# 1024 rows per binning block; up to 256 blocks are summed by the scatter
# itself, more by the scan (512 blocks per step of each of its two halves)
@pytest.mark.parametrize("rows", [1, 1023, 1024, 1025, 262143, 262144, 262145, 263168, 1049600, 1050625])
def test_binning_blocks(rows):
    A = synth.poisson_csr(rows, 700, 1.5, seed=rows)
    B = synth.random_csr(700, 90, 0.06, 3)   # rows of C on both sides of the smallest class's 32
    check(A, B)


# rows of B around and past the 64 lanes of a wave (one or several steps per
# row) in every numeric class that gives a row a whole wave; the chunk of 64
# entries of A staged with more than 64 steps
@pytest.mark.parametrize("cls", [1, 2, 3])
@pytest.mark.parametrize("len_b", [33, 63, 64, 65, 81, 128, 129, 200])
def test_long_rows_of_b(cls, len_b):
    g = synth.rng(len_b)
    ncols = {1: 128, 2: 500, 3: 1000}[cls] if len_b <= 128 else max(len_b, {1: 128, 2: 500, 3: 1000}[cls])
    rows = [np.sort(g.choice(ncols, min(len_b, ncols), replace=False)) if k % 5 else np.zeros(0, np.int64)
            for k in range(150)]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    B = synth.Csr(150, ncols, rp, np.concatenate(rows).astype(np.int32), g.standard_normal(int(rp[-1])))
    A = synth.poisson_csr(70, 150, 70.0, seed=len_b)
    mls.set_option(mls._abi.OPT_GROUP_SIZE, 64)
    try:
        check(A, B)
    finally:
        mls.set_option(mls._abi.OPT_GROUP_SIZE, 0)
