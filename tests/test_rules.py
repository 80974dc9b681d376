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
int row_tiles(int form, int64_t r) { return strip_row_tiles(form, r); }
int product_small(int64_t m, int64_t n) { return product_small_tiles(m, n); }
int triangle_guarded_(int64_t m, int64_t k) { return triangle_guarded(m, k); }
int f32_small_tiles(int64_t n, int64_t t) { return hessian_f32_small_tiles(n, t); }
int tokens_tile_(int64_t n, int64_t t) { return tokens_tile(n, t); }
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
    L.row_tiles.argtypes = [ctypes.c_int, i64]
    L.f32_small_tiles.argtypes = [i64, i64]
    L.product_small.argtypes = L.triangle_guarded_.argtypes = L.tokens_tile_.argtypes = [i64, i64]
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


# float32 Hessians: (channels, tokens, microseconds with the small tiles, with the float32 product), measured on one card
F32_TIMES = [
    (256, 4096, 41, 245), (1000, 16, 12, 23), (1024, 64, 12, 12), (1408, 4096, 135, 250), (1500, 512, 42, 67), (1544, 64, 15, 20),
    (1664, 64, 14, 12), (1664, 512, 42, 38), (1664, 4096, 247, 251), (1920, 4096, 248, 252), (2040, 4096, 338, 393), (2048, 64, 20, 13), (2048, 512, 59, 41), (2048, 4096, 338, 253),
    (2056, 64, 22, 16), (2056, 512, 59, 56), (2056, 4096, 349, 367), (2144, 8, 22, 17), (2200, 64, 22, 19), (2300, 4096, 357, 395), (2500, 64, 28, 26),
    (2500, 512, 78, 70), (2500, 8192, 907, 753), (2560, 4096, 456, 255), (2700, 4096, 476, 372), (2816, 8192, 933, 499), (2824, 512, 96, 90),
    (2950, 4096, 573, 614), (2950, 512, 100, 90), (3000, 64, 34, 32), (3000, 8192, 1152, 1244), (3072, 64, 33, 20), (3072, 8192, 1159, 957),
]


@pytest.mark.parametrize("n,t,small,product", F32_TIMES)
def test_float32_hessians_take_the_faster_kernel(rules, n, t, small, product):
    """No call goes to the slower of the two by more than the runs differ; beyond 3072 channels it is always the product."""
    chosen = small if rules.f32_small_tiles(n, t) else product
    assert chosen <= 1.05 * min(small, product) + 1
    assert not rules.f32_small_tiles(3073, t)


# float32 products, K = 1024: (rows, columns, microseconds with 256 x 128 tiles, with 128 x 128 tiles, with the guarded kernel)
PRODUCT_TIMES = [
    (2048, 4098, 263, 208, 254), (4096, 2050, 254, 194, 244), (8192, 1026, 254, 193, 245), (2304, 4994, 255, 197, 242), (2048, 6018, 256, 198, 242),
    (4096, 2946, 257, 197, 243), (2048, 6530, 257, 257, 325), (12288, 1026, 259, 257, 329), (2048, 8066, 261, 259, 324), (4096, 4098, 381, 320, 390),
    (2304, 9090, 383, 383, 456), (8192, 4098, 635, 572, 680), (12288, 12162, 2361, 2304, 2636),
]


@pytest.mark.parametrize("m,n,tall,small,guarded", PRODUCT_TIMES)
def test_products_of_ragged_columns_are_no_slower_than_through_the_guarded_kernel(rules, m, n, tall, small, guarded):
    assert (small if rules.product_small(m, n) else tall) <= guarded


# triangular float32 products: (channels, tokens, microseconds with 128 x 128 direct-to-LDS tiles, with the guarded kernel)
TRIANGLE_TIMES = [
    (1664, 64, 10.4, 10.7), (2688, 128, 15.8, 17.6), (2944, 64, 16.8, 16.5), (3200, 64, 18.4, 18.2), (3200, 128, 26.0, 26.6), (3968, 64, 19.8, 20.1),
    (4224, 64, 26.5, 25.0), (4224, 128, 37.4, 37.1), (4224, 192, 48.2, 49.0), (4480, 64, 26.7, 25.4),
    (5248, 64, 34.3, 33.3), (5248, 128, 48.7, 48.2), (5504, 64, 34.7, 35.2), (5504, 128, 49.1, 50.2), (6272, 64, 43.5, 41.3), (6272, 128, 59.6, 58.2), (6272, 192, 78.0, 78.7),
    (8320, 64, 70.4, 65.9), (8320, 128, 102.2, 99.5), (8320, 192, 134.1, 135.3), (10368, 64, 106.6, 97.9), (14464, 64, 227, 206), (14464, 128, 310, 302),
    (14464, 192, 405, 404), (14464, 256, 492, 508), (14464, 512, 876, 935),
]


@pytest.mark.parametrize("n,t,small,guarded", TRIANGLE_TIMES)
def test_short_triangular_products_take_the_faster_kernel(rules, n, t, small, guarded):
    """... within 2 %; whole tiles of 256 rows never take the guarded one."""
    assert (guarded if rules.triangle_guarded_(n, t) else small) <= 1.02 * min(small, guarded)
    assert not rules.triangle_guarded_(n // 256 * 256, t)


def test_products_take_large_tiles_once_they_fill_the_chip(rules):
    for m, n, small in ((4096, 2048, 0), (4096, 1920, 1), (3840, 2048, 1), (4224, 4096, 1), (256, 32768, 0), (256, 32640, 1), (128, 65536, 1), (4096, 3201, 0)):
        assert bool(rules.product_small(m, n)) == bool(small), (m, n)


@pytest.mark.parametrize("form", [0, 1, 2])
def test_strip_height_covers_the_rows_in_the_fewest_rounds_that_pay(rules, form):
    """One strip per CU as long as that lasts; a taller strip only where the lower one would need another round."""
    for rt in (1, 2, 3, 4):
        assert rules.row_tiles(form, 16 * rt * 256) == rt
    assert rules.row_tiles(form, 1) == 1 and rules.row_tiles(form, 4097) == 2 and rules.row_tiles(form, 8193) == 3
    assert rules.row_tiles(form, 12289) == 4
    # many rounds: four rounds of 48 rows beat three of 64, which are strips of 32 one behind the other (a call on 2048 columns, driven by
    # U / R / R with groups: 2432 against 2483 us, 2442 against 2538, 2618 against 2618)
    assert rules.row_tiles(form, 49152) == 3 and rules.row_tiles(form, 41216) == 3


def test_token_major_cases_take_the_route_they_name(rules):
    """A call is read in place where its channels come in whole 16 bytes, the channel-major call has no workspace and the rule names a tile."""
    import paper_2210_17323_amd as g
    from test_gpu_hessian_tokens import CASES
    for dtype, n, t, _, tile in CASES:
        in_place = n % 8 == 0 and g.gptq_hessian_accumulate_workspace_bytes(n, t, dtype) == 0
        assert (rules.tokens_tile_(n, t) if in_place else 0) == tile, (n, t)
    # every line of the rule is reached
    assert {c[4] for c in CASES} == {0, 128, 256}
