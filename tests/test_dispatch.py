"""CPU test of the rules that choose a kernel (csrc/dispatch.h, built here with the host
compiler): where a rule changes its mind, and that the shapes of the GPU tests reach the
kernels they are there for."""
import ctypes
import os
import subprocess

import pytest

from paper_2606_15682_amd import build as libbuild

SOURCE = """
#include "dispatch.h"
using namespace reqat;
extern "C" {
int nv_one_launch_(int64_t elems, int dense) { return nv_one_launch(elems, dense); }
int product_(int fmt, int64_t M, int64_t N, int64_t K, int big_ok) { return pick_product_tile((Fmt)fmt, M, N, K, big_ok); }
int decode_(int fmt, int64_t M, int64_t N, int64_t K) { return pick_decode_tile((Fmt)fmt, M, N, K); }
int w4a16_(int64_t M, int64_t N, int64_t K, int64_t ldx) { return pick_w4a16(M, N, K, ldx); }
int w4a16_splits_(int64_t M, int64_t N, int64_t K) { return gemm_w4a16_splits(M, N, K); }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("dispatch")
    (d / "rules.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", libbuild.CSRC,
                    str(d / "rules.cpp"), "-o", str(d / "rules.so")], check=True)
    lib = ctypes.CDLL(os.path.join(str(d), "rules.so"))
    size = ctypes.c_int64
    lib.nv_one_launch_.argtypes = [size, ctypes.c_int]
    lib.product_.argtypes = [ctypes.c_int, size, size, size, ctypes.c_int]
    lib.decode_.argtypes = [ctypes.c_int, size, size, size]
    lib.w4a16_.argtypes = [size] * 4
    lib.w4a16_splits_.argtypes = [size] * 3
    return lib


@pytest.mark.parametrize("elems,dense,strided", [(16, 1, 1), (1 << 16, 1, 1), ((1 << 16) + 16, 1, 0),
                                                 (96 * 2048, 1, 0), (96 * 2048 + 16, 0, 0)])
def test_computed_nvfp4_scale(rules, elems, dense, strided):
    """One launch up to 3 * 2^16 elements, but only up to 2^16 where rows have a stride: the
    walk over such rows costs twice the two launches at the end of that range."""
    ask = lambda d: rules.nv_one_launch_(elems, d)
    assert (ask(1), ask(0)) == (dense, strided)


NV, MX = 0, 1
SKINNY, T32x32, T32x128, T64x32, T64x64F = -1, 5, 6, 7, 8


@pytest.mark.parametrize("fmt,M,N,K,tile", [
    (MX, 64, 7168, 5120, T64x32), (MX, 64, 27648, 5120, T64x64F), (NV, 32, 7168, 5120, T32x32), (NV, 24, 27648, 5120, T32x128),
    (NV, 16, 27648, 5120, SKINNY), (MX, 16, 27648, 5120, SKINNY),
    # where the first rule, rounds of tiles alone, lost up to 1.65 times to the skinny kernel
    (NV, 39, 22560, 1664, T64x64F), (NV, 45, 17776, 640, SKINNY), (NV, 39, 17920, 1536, SKINNY),
    (MX, 58, 17, 1152, SKINNY), (MX, 50, 304, 896, SKINNY), (MX, 53, 1504, 2432, SKINNY), (NV, 57, 20, 24960, SKINNY),
    (NV, 19, 17024, 1280, T32x128)])
def test_w4a4_decode_tile(rules, fmt, M, N, K, tile):
    assert rules.decode_(fmt, M, N, K) == tile


W16_DECODE, W16_SPLIT = -2, -1


@pytest.mark.parametrize("M,N,K,kernel", [
    (4, 7168, 5120, W16_DECODE), (1, 37888, 3584, W16_DECODE), (4, 55296, 5120, W16_DECODE), (16, 1536, 1536, W16_DECODE),
    (4, 5120, 27648, W16_SPLIT), (16, 27648, 5120, W16_SPLIT), (7, 5120, 13824, W16_SPLIT),
    # many rounds of short rows, where the decode kernel took up to 1.4 times as long
    (5, 40832, 512, W16_SPLIT), (1, 47216, 640, W16_SPLIT), (3, 47888, 768, W16_SPLIT), (7, 28608, 640, W16_SPLIT)])
def test_w4a16_decode_kernel(rules, M, N, K, kernel):
    assert rules.w4a16_(M, N, K, K) == kernel


@pytest.mark.parametrize("N", [1 << 27, 3 << 27, (1 << 31) - 16])
def test_no_launch_of_2_to_the_32_threads(rules, N):
    """Weight matrices with so many rows that a workgroup per tile would need a grid of 2^32
    threads or more stay with the kernels that ran them before the tiles."""
    tiles = lambda M, tm, tn: -(-M // tm) * -(-N // tn)
    limit = (1 << 32) // 512
    for M in (1, 4, 16):
        assert rules.w4a16_(M, N, 128, 128) == W16_SPLIT or -(-N // 16) < limit
    for M in (33, 64, 65, 150, 1000):
        t = rules.w4a16_(M, N, 128, 128)
        assert t == W16_SPLIT or tiles(M, *((64, 64), (64, 128), (128, 128), (128, 128))[t]) < limit
    for fmt in (NV, MX):
        for M in (17, 40, 64):
            t = rules.decode_(fmt, M, N, 128)
            assert t == SKINNY or tiles(M, 64, {T32x32: 32, T32x128: 128, T64x32: 32, T64x64F: 64}[t]) < limit
        for M in (65, 130, 150, 1000):
            for big in (0, 1):
                t = rules.product_(fmt, M, N, 128, big)
                assert t in (-1, 5) or tiles(M, *((64, 64), (64, 128), (128, 128), (64, 128), (128, 128))[t]) < limit
                assert t != 5 or big


PRODUCT = ["64x64", "64x128", "128x128", "64x128 deep", "128x128 deep", "256x256"]
DECODE = {-1: "skinny", 5: "32x32", 6: "32x128", 7: "64x32", 8: "64x64 few"}
W4A16 = ["64x64", "64x128", "128x128", "128x128x8"]


def test_shapes_of_the_gpu_tests_reach_their_kernels(rules):
    """The kernel that each GPU test names for a shape is the one the rules pick for it."""
    from tests import (test_gpu_decode_tiles, test_gpu_gemm_multiround_tiles, test_gpu_gemm_tiles, test_gpu_graph,
                       test_gpu_product_instances, test_gpu_w4a16_decode, test_gpu_w4a16_tiles)

    def w4a4(fmt, M, N, K):
        if M <= 64:
            return DECODE[rules.decode_(fmt, M, N, K)]
        return PRODUCT[rules.product_(fmt, M, N, K, K % (256 if fmt == NV else 128) == 0)]

    def w4a16(M, N, K):
        t = rules.w4a16_(M, N, K, K)
        return W4A16[t] if t >= 0 else "decode" if t == W16_DECODE else "split" if rules.w4a16_splits_(M, N, K) > 1 else "unsplit"

    wrong = [(name, f, M, N, K, w4a4(f, M, N, K))
             for module in (test_gpu_decode_tiles.CASES, test_gpu_gemm_tiles.CASES, test_gpu_gemm_multiround_tiles.CASES,
                            test_gpu_product_instances.W4A4)
             for name, fmts, M, N, K in module for f in fmts if w4a4(f, M, N, K) != name]
    p = test_gpu_product_instances
    wrong += [(name, M, N, K, w4a16(M, N, K))
              for name, M, N, K in p.W4A16 + p.W4A16_STRIDED + p.W4A16_SPECIAL + test_gpu_graph.W4A16 +
              [("64x64", *shape) for shape in test_gpu_w4a16_tiles.SMALL] +
              [case[:4] for case in test_gpu_w4a16_tiles.LARGE] +
              [("decode", M, *shape) for M in test_gpu_w4a16_decode.ROWS for shape in test_gpu_w4a16_decode.SHAPES]
              if w4a16(M, N, K) != name]
    assert not wrong
