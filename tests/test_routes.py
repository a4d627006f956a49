"""Which kernels a call is sent to, and with what split, on the CPU: the C ABI's
planning (csrc/api.hip) linked with launchers that only write down what they are
given, for a chip of 256 compute units.  Nothing is launched and no pointer is
read."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2207_05808_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

STUBS = r"""
#include "internal.hpp"
#include <stdio.h>
#include <string>
static std::string g_log;
static hipError_t note(const std::string& s) { g_log += s + "\n"; return hipSuccess; }
extern "C" const char* routes() { static std::string out; out = g_log; g_log.clear(); return out.c_str(); }
namespace mdn {
int device_cus() { return 256; }
int macc_staged(int C) { return C <= 64 ? C : C <= 96 ? 96 : 128; }
hipError_t launch_gfused(int elem, int ng, int uq, const GArgs& g, int nw, int, hipStream_t) {
  return note("gfused " + std::to_string(g.R) + " " + std::to_string(nw) + (g.idx_in ? " idx" : ""));
}
hipError_t launch_softmax_rows(float*, int64_t, int, int, hipStream_t) { return note("softmax"); }
hipError_t launch_tacc(int, int, const TArgs&, int, int, hipStream_t) { return note("tacc"); }
hipError_t launch_trow(int, const TArgs& t, int, hipStream_t) { return note(t.only_wide ? "trow-wide" : "trow"); }
hipError_t launch_rlane_f32(const TArgs&, int, hipStream_t) { return note("rlane-f32"); }
hipError_t launch_rlane_i8(const TArgs&, int, hipStream_t) { return note("rlane-i8"); }
hipError_t launch_fenc(const FArgs&, int, hipStream_t) { return note("fenc"); }
hipError_t launch_macc(const MArgs& m, int blocks, hipStream_t) {
  return note("macc " + std::to_string(m.W) + " " + std::to_string(m.nslices) + " " + std::to_string(m.rows_per_group) +
              " " + std::to_string(blocks) + " " + std::to_string(m.xcd_map));
}
hipError_t launch_tavg(const TArgs&, int, int, hipStream_t) { return note("tavg"); }
hipError_t launch_path(int mode, int, int, int, const KArgs&, dim3, dim3, hipStream_t) {
  return note(mode == kEncode ? "encode" : mode == kAccum ? "accum" : "fused");
}
hipError_t launch_build_lut(const float*, const float*, int, int, int, int8_t*, float*, float*, int, int, hipStream_t) {
  return note("build");
}
hipError_t launch_build_lut_f32(const float*, const float*, int, int, int, float*, int, hipStream_t) { return note("build-f32"); }
hipError_t launch_quantize_lut(const double*, int, int, int8_t*, float*, float*, int, hipStream_t) { return note("quantize"); }
hipError_t launch_gram(const uint8_t*, int64_t, int, int32_t*, int, hipStream_t) { return note("gram"); }
hipError_t launch_scatter(const uint8_t*, int64_t, int, const float*, int, double*, int32_t*, int32_t*, hipStream_t) {
  return note("scatter");
}
hipError_t launch_fit_gd(const uint8_t*, int64_t, int, const float*, int, const float*, int, const float*, double, double,
                         int, double*, double*, double*, int32_t*, int32_t*, hipStream_t) { return note("gd"); }
hipError_t launch_fit_ridge(const uint8_t*, int64_t, int, const float*, int, const float*, double, double*, int32_t*,
                            double*, int32_t*, int32_t*, int, hipStream_t) { return note("ridge"); }
}  // namespace mdn
"""


@pytest.fixture(scope="module")
def api(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not found")
    d = tmp_path_factory.mktemp("routes")
    src = d / "stubs.hip"
    src.write_text(STUBS)
    so = str(d / "libroutes.so")
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(CSRC, "api.hip"), str(src),
                        "-o", so], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    import torch  # noqa: F401  (the process's HIP runtime, as the library takes it)
    L = ctypes.CDLL(so)
    from paper_2207_05808_amd import _lib
    real = _lib.lib()
    for f in ("maddness_matmul", "maddness_matmul_act", "maddness_lut_accumulate", "maddness_matmul_index_bytes"):
        getattr(L, f).argtypes, getattr(L, f).restype = getattr(real, f).argtypes, getattr(real, f).restype
    L.routes.restype = ctypes.c_char_p
    return L


FAKE = ctypes.c_void_p(0x1000)


def fits_gathers(C, M):
    """Tables the gather-fused kernel takes (C divides 64, 16-bit entries in 160 KB of LDS beside its offsets)."""
    return 64 % C == 0 and 2 * (16 * C + 1) * (M + 7 & ~7) < 150_000


def accumulate(L, N, C, M):
    assert L.maddness_lut_accumulate(FAKE, N, C, FAKE, FAKE, FAKE, M, None, FAKE, None) == 0
    return L.routes().decode().split("\n")[:-1]


def check_split(route, N, M):
    """The one-hot product's split covers every row and column, in groups whose outputs stay below 2^31 bytes."""
    name, W, nslices, rows, blocks, xcd = route.split()
    W, nslices, rows, blocks, xcd = int(W), int(nslices), int(rows), int(blocks), int(xcd)
    assert name == "macc" and W in (32, 64, 128) and nslices == -(-M // W)
    groups = blocks // nslices
    assert blocks == groups * nslices and rows % 64 == 0
    assert groups * rows >= N and (rows - 64) * groups < N + 64 * groups
    assert rows * M * 4 < 1 << 31
    assert xcd == (blocks % 8 == 0)
    return W, groups


@pytest.mark.parametrize("N,C,M", [(524287, 64, 4096), (524288, 64, 4096), (600000, 48, 4096), (1048575, 64, 4096),
                                   (32704, 48, 16384), (32768, 48, 16384), (65535, 64, 16384), (1048576, 128, 4096),
                                   (3000000, 128, 4096), (5, 16, 4000000), (1 << 31, 64, 100)])
def test_one_hot_product_at_any_output_size(api, N, C, M):
    """Large outputs keep the one-hot product; they take more row groups."""
    (route,) = accumulate(api, N, C, M)
    W, groups = check_split(route, N, M)
    # whole rounds of (almost) a workgroup per compute unit
    slices = -(-M // W)
    full = min(max(1, 256 // slices), -(-N // 64))
    assert any(groups % g == 0 for g in range(-(-3 * full // 4), full + 1))


def test_one_hot_product_of_ragged_rows(api):
    """Output rows that are no whole 64-byte pieces: a multiple of 8 workgroups
    wherever that costs at most a quarter of them, so that the slices of a row
    group run on one XCD; 128 columns only for up to 64 codebooks and many rows."""
    for C in (32, 48, 64, 96, 128):
        for M in range(132, 3000, 52):
            for N in (40000, 131072, 700000):
                (route,) = accumulate(api, N, C, M)
                W, groups = check_split(route, N, M)
                slices = -(-M // W)
                assert W == 64 or (W == 128 and C <= 64 and N * -(-M // 64) >= 524288)
                full = 256 // slices
                if M % 16 and any(g * slices % 8 == 0 for g in range(-(-3 * full // 4), full + 1)):
                    assert groups * slices % 8 == 0
                assert 4 * groups >= 3 * full


def test_few_codebooks_and_many_ragged_rows_gather(api):
    for C, M, N, gathers in ((16, 196, 163839, False), (16, 196, 163840, True), (16, 128, 1 << 20, True),
                             (16, 100, 1 << 22, False), (16, 208, 4096, True), (16, 1000, 1 << 20, False),
                             (32, 132, (1 << 20) - 1, False), (32, 132, 1 << 20, True), (32, 196, 1 << 20, False),
                             (64, 132, 1 << 20, False)):
        (route,) = accumulate(api, N, C, M)
        assert route.startswith("gfused") == gathers


def test_one_hot_product_split(api):
    rng = random.Random(7)
    for _ in range(400):
        C = 16 * rng.randint(1, 8)
        M = 4 * int(2 ** rng.uniform(2, 13))
        N = int(2 ** rng.uniform(0, 24))
        route = accumulate(api, N, C, M)
        if route[0].startswith("gfused"):
            assert fits_gathers(C, M) and (M % 16 == 0 or (M > 128 and N >= 131072))
            continue
        assert len(route) == 1
        check_split(route[0], N, M)


@pytest.mark.parametrize("act", [0, 2])
@pytest.mark.parametrize("D,two", [(576, True), (4096, True), (4100, False), (4608, False), (10301, False)])
def test_two_phases_where_the_encode_has_a_plan(api, D, two, act):
    for C, M in ((32, 100), (64, 72)):
        n = api.maddness_matmul_index_bytes(FAKE, 1000, D, D, C, M, 0, act)
        assert n == (1000 * C if two else 0)
        assert api.maddness_matmul_act(FAKE, 1000, D, D, FAKE, FAKE, C, FAKE, FAKE, FAKE, M, None, act, FAKE, FAKE,
                                       None) == 0
        route = api.routes().decode().split("\n")[:-1]
        assert [r.split()[0] for r in route] == (["encode", "macc"] if two else ["gfused"])


def route(L, N, D, C, M, act, lda=None):
    n = L.maddness_matmul_index_bytes(FAKE, N, D, lda or D, C, M, 0, act)
    assert L.maddness_matmul_act(FAKE, N, D, lda or D, FAKE, FAKE, C, FAKE, FAKE, FAKE, M, None, act, FAKE,
                                 FAKE if n > 0 else None, None) == 0
    return "+".join(r.split()[0] for r in L.routes().decode().split("\n")[:-1])


@pytest.mark.parametrize("N,D,C,M,act,want", [
    # rows of A in 16-byte units: two phases against the general kernel, and
    # against the gathers while the encode has little to read or for many codebooks
    (64, 576, 32, 100, 0, "encode+macc"), (300000, 576, 32, 100, 0, "encode+macc"), (64, 576, 64, 40, 0, "fused"),
    (32768, 128, 16, 200, 2, "encode+macc"), (131072, 128, 16, 200, 2, "gfused"), (16384, 2304, 16, 200, 2, "gfused"),
    (300000, 1024, 32, 132, 2, "encode+macc"), (131072, 128, 32, 100, 2, "gfused"), (131072, 256, 64, 60, 2, "encode+macc"),
    (16384, 4096, 32, 132, 2, "gfused"), (4096, 4096, 32, 100, 2, "encode+macc"),
    # rows that are not
    (1024, 577, 32, 100, 0, "fused"), (8192, 577, 32, 100, 0, "encode+macc"), (1024, 577, 64, 72, 0, "encode+macc"),
    (1024, 1025, 64, 72, 0, "fused"), (1024, 257, 32, 100, 0, "fused"), (4096, 257, 32, 100, 0, "encode+macc"),
    (1000, 4101, 64, 72, 2, "gfused"), (4096, 129, 16, 200, 0, "encode+macc"), (100000, 1025, 16, 200, 0, "fused"),
    (131072, 577, 32, 100, 2, "gfused"), (131072, 577, 16, 200, 2, "gfused"), (1000, 257, 32, 100, 2, "encode+macc"),
    (131072, 129, 16, 200, 2, "gfused"), (8192, 577, 64, 72, 2, "encode+macc"), (4096, 1025, 64, 72, 2, "gfused"),
    # the row-streaming kernel's shapes
    (131072, 512, 64, 128, 0, "encode+macc"), (131072, 513, 64, 128, 0, "encode+macc"),
    (131072, 512, 64, 112, 2, "fenc+trow-wide"),
    # a row softmax: large outputs of few codebooks in a kernel that fuses it
    (48000, 128, 16, 512, 3, "encode+macc+softmax"), (49152, 128, 16, 512, 3, "encode+trow"),
    (131072, 256, 32, 512, 3, "encode+trow"), (131072, 384, 48, 512, 3, "encode+macc+softmax"),
    (65000, 384, 48, 64, 3, "encode+macc+softmax"), (65536, 384, 48, 64, 3, "encode+tacc"),
    (131072, 640, 80, 32, 3, "encode+tacc"), (131072, 384, 48, 100, 3, "encode+macc+softmax"),
    (131072, 768, 96, 64, 3, "encode+macc+softmax"), (1 << 20, 384, 48, 128, 3, "encode+macc+softmax"),
    # no single launch
    (131072, 577, 64, 100, 2, "encode+macc"), (64, 1025, 48, 64, 2, "encode+macc")])
def test_fused_routes(api, N, D, C, M, act, want):
    assert route(api, N, D, C, M, act) == want


def test_row_stride_counts_as_alignment(api):
    assert route(api, 131072, 576, 32, 100, 2) == "encode+macc"
    assert route(api, 131072, 576, 32, 100, 2, lda=577) == "gfused"
    assert route(api, 1024, 576, 32, 100, 0, lda=578) == "fused"
