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
