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
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("dispatch")
    (d / "rules.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", libbuild.CSRC,
                    str(d / "rules.cpp"), "-o", str(d / "rules.so")], check=True)
    return ctypes.CDLL(os.path.join(str(d), "rules.so"))


@pytest.mark.parametrize("elems,dense,strided", [(16, 1, 1), (1 << 16, 1, 1), ((1 << 16) + 16, 1, 0),
                                                 (96 * 2048, 1, 0), (96 * 2048 + 16, 0, 0)])
def test_computed_nvfp4_scale(rules, elems, dense, strided):
    """One launch up to 3 * 2^16 elements, but only up to 2^16 where rows have a stride: the
    walk over such rows costs twice the two launches at the end of that range."""
    ask = lambda d: rules.nv_one_launch_(ctypes.c_int64(elems), d)
    assert (ask(1), ask(0)) == (dense, strided)
