"""The gather-fused kernel's split for few rows: row counts on both sides of
every switch of the rows per wavefront (a workgroup per CU of 8 or 16
wavefronts of 1, 2 or 4 row groups), tables of at most and of more than four
16-byte units per thread, int8 and fp32, the layer outputs, the given indices.
Bit-exact against the oracle (the softmax within its bound, like the other
sigma tests)."""
import numpy as np
import pytest
import torch

import paper_2207_05808_amd as mdn
from paper_2207_05808_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def problem(N, D, C, M, seed):
    rng = np.random.default_rng(seed)
    A = rng.standard_normal((N, D)).astype(np.float32)
    split = rng.integers(0, D, (C, 4)).astype(np.int32)
    thr = rng.standard_normal((C, 15)).astype(np.float32)
    return A, split, thr, rng.standard_normal(M).astype(np.float32)


# rows per workgroup: 8 or 16 wavefronts x 64 / C rows x 1, 2 or 4; 256 workgroups
CASES = [(1, 32, 64), (17, 32, 64), (4096, 32, 64), (4097, 32, 64), (8193, 32, 64), (16385, 32, 64),
         (4096, 64, 64), (4097, 64, 64), (8193, 64, 64), (8192, 16, 128), (8193, 16, 128), (300, 8, 256),
         (32768, 4, 16), (32769, 4, 16), (1000, 1, 48), (70, 2, 512)]


@pytest.mark.parametrize("N,C,M", CASES)
def test_int8(orc, N, C, M):
    A, split, thr, bias = problem(N, 72, C, M, N + C)
    lut, scale, offset = W.random_codes(C, M, seed=N, max_shift=2)
    args = [dev(x) for x in (A, split, thr, lut, scale, offset)]
    ridx, racc, ry = orc.matmul(A, split, thr, lut, scale, offset)
    y, acc, idx = mdn.matmul(*args, want_acc=True, want_idx=True)
    assert np.array_equal(host(idx), ridx) and np.array_equal(host(acc), racc) and np.array_equal(host(y), ry)
    z = ry + bias
    assert np.array_equal(host(mdn.matmul_act(*args, col_bias=dev(bias), act="relu")),
                          np.where(z > 0, z, np.float32(0)))
    s = host(mdn.matmul_act(*args, col_bias=dev(bias), act="softmax"))
    ref = orc.sigma(ry, bias, 3)
    d = np.abs(z - z.max(axis=1, keepdims=True)).astype(np.float64)
    assert (np.abs(s - ref) <= 1.01 * (d + M + 5) * 2.0 ** -24 * ref + 2.0 ** -120).all()
    acc2, y2 = mdn.lut_accumulate(dev(ridx), *args[3:], want_acc=True)
    assert np.array_equal(host(acc2), racc) and np.array_equal(host(y2), ry)


@pytest.mark.parametrize("N,C,M", [(3, 32, 40), (2049, 16, 64), (4097, 16, 64), (500, 8, 100), (700, 64, 36)])
def test_fp32(orc, N, C, M):
    A, split, thr, _ = problem(N, 40, C, M, N + C)
    lut = W.random_fp32_table(C, M, seed=N)
    ridx, ry = orc.matmul_f32(A, split, thr, lut)
    y, idx = mdn.matmul_f32(dev(A), dev(split), dev(thr), dev(lut), want_idx=True)
    assert np.array_equal(host(idx), ridx) and np.array_equal(host(y), ry)
