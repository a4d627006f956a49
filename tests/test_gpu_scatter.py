"""The fit's bucket sums and gradient steps where their split can go wrong:
bucket sizes around the stages of rows (56 and 224, in groups of 224 and 448)
and, where a wavefront takes a bucket, its batches (16 and 64 rows),
one bucket with every row and the others empty, column counts around the tiles
(16, 64) and around the residual kernels' forms (64, 128, 256 columns in
registers, more through memory), the sort's batches (64 rows, 8 at a time, 16
wavefronts), infinities, NaN and signed zeros.  Bit-exact against the oracle:
every sum takes its rows in ascending order on both sides.
"""
import numpy as np
import pytest
import torch

import paper_2207_05808_amd as mdn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def indices(rng, N, C, kind):
    idx = rng.integers(0, 16, (N, C)).astype(np.uint8)
    if kind == "one":        # all rows in one bucket, another one per codebook
        idx[:] = np.arange(C) % 16
    elif kind == "skew":     # half of the rows in bucket 3, a few in 15
        idx[rng.random((N, C)) < 0.5] = 3
        idx[idx == 15] = 14
        idx[N // 2] = 15
    return idx


@pytest.mark.parametrize("N,C,M,kind", [(55, 2, 16, "one"), (56, 3, 17, "one"), (57, 1, 64, "one"), (223, 2, 33, "one"),
                                        (224, 5, 65, "one"), (225, 1, 1, "one"), (449, 2, 128, "one"),
                                        (1024, 17, 129, "skew"), (8193, 4, 512, "skew"), (9000, 3, 513, "even"),
                                        (20000, 2, 70, "skew"),
                                        # a wavefront per bucket: batches of 16 and 64 rows
                                        (0, 2, 10, "even"), (1, 1, 1, "one"), (15, 8, 64, "one"), (64, 40, 65, "one"),
                                        (65, 9, 300, "one"), (129, 70, 64, "skew"), (1000, 250, 130, "skew"),
                                        (1024, 256, 128, "one")])
def test_sums(orc, N, C, M, kind):
    rng = np.random.default_rng(N + M)
    idx = indices(rng, N, C, kind)
    Y = (rng.standard_normal((N, M)) * 3).astype(np.float32)
    Y[:1] = -0.0
    assert np.array_equal(host(mdn.encoder_scatter(dev(idx), dev(Y))), orc.encoder_scatter(idx, Y))


def test_sums_not_finite(orc):
    rng = np.random.default_rng(5)
    idx = indices(rng, 700, 3, "skew")
    Y = rng.standard_normal((700, 40)).astype(np.float32)
    Y[3, 5], Y[600, 7], Y[699, 39], Y[10, 39] = np.inf, np.nan, -np.inf, np.inf
    with np.errstate(invalid="ignore"):
        ref = orc.encoder_scatter(idx, Y)
    assert np.array_equal(host(mdn.encoder_scatter(dev(idx), dev(Y))), ref, equal_nan=True)


@pytest.mark.parametrize("N,C,M,kind", [(224, 2, 16, "one"), (449, 3, 17, "skew"), (700, 9, 64, "skew"),
                                        (500, 4, 128, "even"), (600, 3, 129, "skew"), (300, 70, 256, "even"),
                                        (450, 2, 300, "skew"),
                                        # a wavefront per bucket
                                        (17, 5, 16, "one"), (81, 20, 17, "one"), (130, 12, 128, "skew"),
                                        (200, 30, 129, "skew"), (1500, 96, 64, "skew"), (300, 80, 300, "even")])
def test_gradient_steps(orc, N, C, M, kind):
    rng = np.random.default_rng(N + M)
    idx = indices(rng, N, C, kind)
    Y = rng.standard_normal((N, M)).astype(np.float32)
    T0 = (rng.standard_normal((C, 16, M)) / C).astype(np.float32)
    bias = rng.standard_normal(M).astype(np.float32)
    args = (0.5, 1e-4, 3)
    T = host(mdn.fit_lut_gd(dev(idx), dev(Y), dev(T0), "relu", *args, col_bias=dev(bias)))
    assert np.array_equal(T, orc.fit_lut_gd(idx, Y, T0, 2, *args, bias=bias))
