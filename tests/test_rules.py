"""Ranges and rules of dispatch (csrc/rules.h, plain C++) checked on the CPU: the header the library is built from, compiled
into a small shared object of its own."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2210_17323_amd", "csrc")
SOURCE = """
#include "rules.h"
using namespace gptq;
extern "C" {
int64_t outer_block(int64_t group) { return alg1_outer_block(group); }
int64_t block_columns(int64_t o0, int64_t o1, int i) { return strip_block_columns(o0, o1, i); }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, so = d / "rules.cpp", d / "rules.so"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(so)], check=True)
    L = ctypes.CDLL(str(so))
    i64 = ctypes.c_int64
    L.outer_block.restype, L.outer_block.argtypes = i64, [i64]
    L.block_columns.restype, L.block_columns.argtypes = i64, [i64, i64, ctypes.c_int]
    return L


@pytest.mark.parametrize("n,group", [(1, 0), (129, 0), (1025, 0), (4228, 0), (1280, 256), (2048, 1024), (4096, 2048), (1536, 384), (3840, 640), (2304, 1152)])
def test_a_strip_launch_reads_the_columns_it_walks_and_no_others(rules, n, group):
    """Columns past a launch's own are written by the helper stream meanwhile (the deferred update of the launch before)."""
    ob = rules.outer_block(group)
    assert ob in (128, 1024) and (group < 128 or ob % group == 0 or group % ob == 0)
    for o0 in range(0, n, ob):
        o1 = min(o0 + ob, n)
        read = set()
        for i in range(8):
            first = o0 + 128 * i
            read |= set(range(first, first + min(128, rules.block_columns(o0, o1, i))))
        assert read == set(range(o0, o1)), (o0, o1)
