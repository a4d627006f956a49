"""The softmax pass over rows that the accumulate wrote (layers whose output the
accumulate does not fuse) divides by the row's sum: one rounding per output.
With k columns at the row's maximum, one column 18 below it and the others 200
below, the exponentials are 1, v = exp(-18) < 2^-24 and 0, and the sum is k to
the bit in every order, so the outputs are 1 / k and v / k rounded once (v is
the output of the row with k = 1)."""
import numpy as np
import pytest
import torch

import paper_2207_05808_amd as mdn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

KS = [1, 3, 5, 7, 9, 11, 13, 17, 23, 37, 43, 49, 59, 61, 83, 97]


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


# columns around the pass's chunk counts (1, 2, 4, 8, 16 of 256 columns) and past them
@pytest.mark.parametrize("C,M", [(48, 100), (64, 128), (16, 256), (48, 260), (96, 512), (48, 516), (112, 1024),
                                 (48, 1028), (32, 2048), (48, 2052), (16, 4096), (48, 4100)])
def test_one_rounding(C, M):
    bits = np.arange(16)[:, None] >> np.arange(3, -1, -1)[None] & 1
    A = (2.0 * bits - 1.0).astype(np.float32)                      # row i takes prototype i of every codebook
    split = np.tile(np.arange(4, dtype=np.int32), (C, 1))
    lut = np.zeros((C, 16, M), np.int8)
    rng = np.random.default_rng(M)
    ones = np.zeros((16, M), bool)
    at = np.empty(16, int)
    for i, k in enumerate(KS):
        cols = rng.permutation(M)
        ones[i, cols[:k]] = True
        at[i] = cols[k]
    lut[0] = np.where(ones, 0, -100)
    lut[0, np.arange(16), at] = -9
    args = (dev(A), dev(split), dev(np.zeros((C, 15), np.float32)), dev(lut), dev(np.full(C, 2.0, np.float32)),
            dev(np.zeros(C, np.float32)))
    y = mdn.matmul_act(*args, act="softmax").cpu().numpy()
    ks = np.array(KS, np.float32)
    v = y[0, at[0]]
    assert 0 < v < 2.0 ** -24
    assert (v / ks != v * (np.float32(1) / ks)).any()              # (the inputs tell a division from a product)
    ref = np.where(ones, (np.float32(1) / ks)[:, None], np.float32(0))
    ref[np.arange(16), at] = v / ks
    assert np.array_equal(y, ref)
