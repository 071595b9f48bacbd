"""The launch plans' host arithmetic (csrc/plan.h), compiled alone and checked on
the CPU: bounds up to the int32 range's end."""

import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_09590_amd", "csrc")
INT32_MAX = 2**31 - 1

WRAPPERS = """
#include "plan.h"
extern "C" {
int longest(int max_ctx, int width) { return bros::longest_blocks(max_ctx, width); }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("plan")
    src, so = d / "plan.cpp", d / "plan.so"
    src.write_text(WRAPPERS)
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-ftrapv", "-shared", "-fPIC", "-I", CSRC, str(src),
                    "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    I = ctypes.c_int
    lib.longest.argtypes = [I, I]
    return lib


@pytest.mark.parametrize("max_ctx", [1, 15, 16, 17, INT32_MAX - 15, INT32_MAX - 14, INT32_MAX])
def test_longest_blocks(plan, max_ctx):
    assert plan.longest(max_ctx, INT32_MAX) == max(1, -(-max_ctx // 16))
    assert plan.longest(max_ctx, 7) == min(7, max(1, -(-max_ctx // 16)))
    assert plan.longest(0, 7) == 1
