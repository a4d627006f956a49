"""Table build where its shortcuts begin and end: prototype columns that are
all zero are skipped (none of them, most of them, whole codebooks, more columns
than one list holds), weights and prototypes that are not finite, every tile
form (4 columns per thread with 16-byte rows or without, 1 column, narrow tables
spread over the prototypes), weights few enough for every workgroup to look
through, byte offsets of the codes.  Bit-exact against the oracle; where NaN or infinities
occur, against a double sum over every column and the quantizer of that table.
"""
import ctypes

import numpy as np
import pytest
import torch

import paper_2207_05808_amd as mdn
from paper_2207_05808_amd import _lib

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def problem(C, D, M, kind, seed):
    rng = np.random.default_rng(seed)
    P = rng.standard_normal((C, 16, D)).astype(np.float32)
    B = rng.standard_normal((D, M)).astype(np.float32)
    if kind == "blocks":          # contiguous subspaces, the last columns in none
        L = max(1, D // C)
        for c in range(C):
            P[c, :, :c * L] = 0
            P[c, :, (c + 1) * L:] = 0
    elif kind == "scattered":     # a column here and there, one prototype of it only, codebook 0 all zero
        keep = rng.random((C, D)) < 0.1
        P *= keep[:, None, :]
        P *= (np.arange(16)[None, :, None] == rng.integers(0, 16, (C, 1, D))) | (rng.random((C, 1, D)) < 0.5)
        P[0] = np.where(rng.random((16, D)) < 0.5, np.float32(-0.0), np.float32(0.0))
    return P, B


def build(P, B, byte_offset=0, shared=False):
    """maddness_build_lut with the codes `byte_offset` bytes past a 256-byte boundary, guards on both sides."""
    C, _, D = P.shape
    M = B.shape[1]
    n = C * 16 * M
    buf = torch.full((n + 512,), 0x5A, dtype=torch.uint8, device=DEV)
    at = (-buf.data_ptr()) % 256 + byte_offset
    scale = torch.empty(C, device=DEV)
    offset = torch.empty(C, device=DEV)
    p = lambda t, o=0: ctypes.c_void_p(t.data_ptr() + o)
    Pd, Bd = dev(P), dev(B)
    fn = "maddness_build_lut_shared" if shared else "maddness_build_lut"
    _lib.check(fn, getattr(_lib.lib(), fn)(p(Pd), p(Bd), C, D, M, p(buf, at), p(scale), p(offset),
                                           ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    b = host(buf)
    assert (b[:at] == 0x5A).all() and (b[at + n:] == 0x5A).all()
    return b[at:at + n].view(np.int8).reshape(C, 16, M), host(scale), host(offset)


CASES = [  # C, D, M, kind, byte offset of the codes
    (1, 1, 1, "dense", 0), (4, 64, 10, "blocks", 1), (3, 700, 37, "dense", 0), (5, 513, 300, "blocks", 0),
    (70, 560, 4096, "blocks", 0),      # 4 columns per thread, vector rows
    (70, 560, 4096, "blocks", 3),      # codes off 4 bytes: scalar rows
    (90, 270, 3001, "scattered", 0),   # ragged last tile, M % 4 != 0
    (64, 1100, 4100, "scattered", 0),  # more columns than one list, ragged vector tile
    (512, 512, 17, "blocks", 0),
    # narrow tables (16, 64, 128 columns), few weights and more than that
    (3, 256, 16, "dense", 0), (3, 257, 16, "scattered", 2), (7, 64, 17, "dense", 0), (7, 65, 64, "blocks", 0),
    (20, 600, 65, "dense", 1), (5, 32, 128, "dense", 0), (5, 33, 128, "blocks", 0), (2, 16, 129, "dense", 0),
    (2, 17, 256, "dense", 0), (300, 16, 1000, "scattered", 0), (300, 3, 1024, "blocks", 0),
]


@pytest.mark.parametrize("C,D,M,kind,off", CASES)
def test_build_matches_oracle(orc, C, D, M, kind, off):
    P, B = problem(C, D, M, kind, seed=C + D + M)
    for shared in (False, True):
        lut, scale, offset = build(P, B, off, shared)
        rl, rs, ro = (orc.build_shared_lut if shared else orc.build_quantized_lut)(P, B)
        assert np.array_equal(scale, rs) and np.array_equal(offset, ro) and np.array_equal(lut, rl)
    assert np.array_equal(host(mdn.build_lut_f32(dev(P), dev(B))), orc.build_lut_f32(P, B))


@pytest.mark.parametrize("C,D,M", [(4, 64, 10), (66, 530, 4096), (4, 300, 16), (5, 70, 33), (5, 41, 100), (4, 6, 100),
                                   (9, 41, 300), (260, 530, 1025), (3, 1030, 97)])
@pytest.mark.parametrize("where", ["weight in a skipped column", "weight in a used column", "prototype"])
def test_build_not_finite(C, D, M, where):
    P, B = problem(C, D, M, "blocks", seed=C)
    if where == "prototype":
        P[1, 3, D // C], P[2, 5, 2 * (D // C)] = np.inf, np.nan
    else:
        d = C * (D // C) if where == "weight in a skipped column" and D % C else 0
        B[d, M // 2], B[d, M - 1], B[1, 0] = np.inf, np.nan, -np.inf
    T = np.zeros((C, 16, M))
    with np.errstate(invalid="ignore"):
        for d in range(D):
            T += P[:, :, d:d + 1].astype(np.float64) * B[d].astype(np.float64)
        T32 = T.astype(np.float32)
    assert np.array_equal(host(mdn.build_lut_f32(dev(P), dev(B))), T32, equal_nan=True)
    rl, rs, ro = (host(t) for t in mdn.quantize_lut(dev(T)))
    lut, scale, offset = build(P, B)
    assert np.array_equal(scale, rs) and np.array_equal(offset, ro, equal_nan=True) and np.array_equal(lut, rl)
