"""The one-hot product from one row up: every codebook padding (16 to 128 in
steps of 16), both slice widths (32 columns while every wavefront has at most
one 64-row tile, else 64), rows and columns around the tiles, several shift
groups, and the fused calls that take it when they are given an index array and
a single launch when they are not.  Sums, outputs and indices bit-exact."""
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


@pytest.mark.parametrize("N,C,M,max_shift", [(1, 16, 16, 0), (31, 16, 1028, 8), (33, 32, 100, 3), (64, 48, 36, 14),
                                             (65, 64, 132, 2), (577, 64, 96, 6), (130, 80, 64, 7), (1000, 96, 32, 1),
                                             (1025, 112, 4100, 3), (513, 128, 2052, 1), (4097, 32, 516, 5),
                                             (9000, 16, 640, 9), (70000, 64, 20, 1), (33000, 48, 68, 2)])
def test_accumulate(orc, N, C, M, max_shift):
    lut, scale, offset = W.random_codes(C, M, seed=N + C, max_shift=max_shift)
    idx = W.random_indices(N, C, seed=N)
    acc, y = mdn.lut_accumulate(dev(idx), dev(lut), dev(scale), dev(offset), want_acc=True)
    _, y1 = mdn.lut_accumulate(dev(idx), dev(lut), dev(scale), dev(offset))
    racc, ry = orc.lut_accumulate(idx, lut, scale, offset)
    assert np.array_equal(host(acc), racc) and np.array_equal(host(y), ry) and np.array_equal(host(y1), ry)


@pytest.mark.parametrize("N,D,C,M", [(1, 64, 32, 100), (300, 130, 48, 64), (2000, 512, 64, 100), (777, 96, 96, 32),
                                     (5000, 64, 16, 200)])
@pytest.mark.parametrize("act", ["none", "relu"])
def test_fused_with_and_without_indices(orc, N, D, C, M, act):
    """The two routes of one call: through an index array and as one launch."""
    rng = np.random.default_rng(N + C)
    A = rng.standard_normal((N, D)).astype(np.float32)
    split = rng.integers(0, D, (C, 4)).astype(np.int32)
    thr = rng.standard_normal((C, 15)).astype(np.float32)
    lut, scale, offset = W.random_codes(C, M, seed=C, max_shift=2)
    bias = rng.standard_normal(M).astype(np.float32)
    args = [dev(x) for x in (A, split, thr, lut, scale, offset)]
    ridx, _, ry = orc.matmul(A, split, thr, lut, scale, offset)
    assert mdn.matmul_index_bytes(args[0], C, M, act=act) == N * C
    idx = torch.empty((N, C), dtype=torch.uint8, device=DEV)
    if act == "none":
        y, _, _ = mdn.matmul(*args, idx_out=idx)
        one = torch.empty((N, M), dtype=torch.float32, device=DEV)
        mdn.matmul_noalloc(*args, one)
        assert np.array_equal(host(one), ry)
    else:
        y = mdn.matmul_act(*args, col_bias=dev(bias), act=act, idx_out=idx)
        z = ry + bias
        ry = np.where(z > 0, z, np.float32(0))
    assert np.array_equal(host(idx), ridx) and np.array_equal(host(y), ry)


@pytest.mark.parametrize("act", ["none", "relu"])
@pytest.mark.parametrize("C,M", [(32, 100), (64, 72)])
@pytest.mark.parametrize("D", [4096, 4100, 4608, 10300, 10301])
def test_wide_rows(orc, D, C, M, act):
    """Rows of A around and past the widest that the encode can stage, with and
    without an index array."""
    N = 130
    rng = np.random.default_rng(D + C)
    A = rng.standard_normal((N, D), dtype=np.float32)
    split = rng.integers(0, D, (C, 4)).astype(np.int32)
    split[0] = D - 1
    thr = rng.standard_normal((C, 15), dtype=np.float32)
    lut, scale, offset = W.random_codes(C, M, seed=D, max_shift=2)
    ridx, racc, ry = orc.matmul(A, split, thr, lut, scale, offset)
    if act == "relu":
        ry = np.maximum(ry, 0)
    args = [dev(x) for x in (A, split, thr, lut, scale, offset)]
    assert np.array_equal(host(mdn.matmul_act(*args, act=act)), ry)
    idx = torch.empty((N, C), dtype=torch.uint8, device=DEV)
    assert np.array_equal(host(mdn.matmul_act(*args, act=act, idx_out=idx)), ry)
    assert np.array_equal(host(idx), ridx)
    if act == "none":
        y, acc, idx = mdn.matmul(*args, want_acc=True, want_idx=True)
        assert np.array_equal(host(idx), ridx) and np.array_equal(host(acc), racc) and np.array_equal(host(y), ry)
        assert np.array_equal(host(mdn.matmul(*args)[0]), ry)
        y = torch.empty((N, M), device=DEV)
        assert np.array_equal(host(mdn.matmul_noalloc(*args, y_out=y, idx_out=idx)), ry)


def test_wide_rows_of_the_row_streaming_kernel(orc):
    """Its shapes too go in two phases only where the encode has a plan."""
    N, D, C, M = 98304, 4100, 64, 128
    A = torch.randn(N, D, device=DEV)
    rng = np.random.default_rng(9)
    split = rng.integers(0, D, (C, 4)).astype(np.int32)
    thr = rng.standard_normal((C, 15), dtype=np.float32)
    lut, scale, offset = W.random_codes(C, M, seed=9, max_shift=2)
    y, acc, idx = mdn.matmul(A, *(dev(x) for x in (split, thr, lut, scale, offset)), want_acc=True, want_idx=True)
    rows = torch.cat([torch.arange(200), torch.arange(49000, 49200), torch.arange(N - 200, N)]).to(DEV)
    ridx, racc, ry = orc.matmul(host(A[rows]), split, thr, lut, scale, offset)
    assert np.array_equal(host(idx[rows]), ridx) and np.array_equal(host(acc[rows]), racc)
    assert np.array_equal(host(y[rows]), ry)


def test_outputs_past_2_gib(orc):
    """One column of row groups would hold 2^31 bytes of outputs: two groups
    per slice, their seam at row 16512."""
    N, C, M = 33000, 48, 16384
    lut, scale, offset = W.random_codes(C, M, seed=3, max_shift=8)
    idx = W.random_indices(N, C, seed=4)
    didx, args = dev(idx), [dev(x) for x in (lut, scale, offset)]
    acc, y = mdn.lut_accumulate(didx, *args, want_acc=True)
    for r0, r1 in ((0, 16000), (16000, N)):   # one group per slice each
        part, ypart = mdn.lut_accumulate(didx[r0:r1], *args, want_acc=True)
        assert torch.equal(acc[r0:r1], part) and torch.equal(y[r0:r1], ypart)
    rows = np.r_[0:20, 16500:16520, N - 20:N]
    racc, ry = orc.lut_accumulate(idx[rows], lut, scale, offset)
    at = torch.from_numpy(rows).to(DEV)
    assert np.array_equal(host(acc[at]), racc) and np.array_equal(host(y[at]), ry)


@pytest.mark.parametrize("N,C,M", [(131100, 16, 260), (140000, 32, 196), (263000, 48, 132), (131073, 64, 304),
                                   (90000, 64, 452), (60000, 48, 700), (131080, 64, 4096)])
def test_slices_of_128_columns(orc, N, C, M):
    """Many rows: the slices and groups of ragged rows, the last slice of three
    quarters, very wide outputs (and 16 codebooks' gathers), against the same
    rows in small calls, and a few of them against the oracle."""
    lut, scale, offset = W.random_codes(C, M, seed=M, max_shift=8)
    idx = W.random_indices(N, C, seed=C)
    didx, args = dev(idx), [dev(x) for x in (lut, scale, offset)]
    _, y = mdn.lut_accumulate(didx, *args)
    for r0 in range(0, N, 16000):
        assert torch.equal(y[r0:r0 + 16000], mdn.lut_accumulate(didx[r0:r0 + 16000], *args)[1])
    acc, y2 = mdn.lut_accumulate(didx, *args, want_acc=True)
    assert torch.equal(y, y2)
    rows = np.r_[0:9, N // 2:N // 2 + 9, N - 9:N]
    racc, ry = orc.lut_accumulate(idx[rows], lut, scale, offset)
    at = torch.from_numpy(rows).to(DEV)
    assert np.array_equal(host(acc[at]), racc) and np.array_equal(host(y[at]), ry)
