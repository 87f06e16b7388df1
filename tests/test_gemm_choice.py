"""choose_gemm (host code of the library) against measured times.

Each row is a projection inside a decode step whose weights come from memory:
its rows, K, 32-token tiles, whether the weights are packed, and by how many us
each kernel shape (GemmShape.wide) is slower there than the fastest of them.
The shape that the library takes is within 0.5 us of the fastest (0.8 us with 40
tiles, in layers of 80 us and more)."""

import ctypes

import pytest

from paper_2607_18839_amd import _lib

EPI = dict(qkv=0, o=1, gate_up=2, down=1)   # csrc/gemm.h

MEASURED = [
    ("down", 2048, 6144, 7, True, {0: 0.0, 1: 12.3, 2: 16.6, 4: 31.5}),
    ("down", 2048, 6144, 8, True, {0: 0.0, 1: 10.9, 2: 18.2, 4: 36.5}),
    ("down", 2048, 6144, 5, True, {0: 0.0, 1: 10.3, 2: 15.0, 4: 21.3}),
    ("down", 2048, 6144, 6, True, {0: 0.0, 1: 9.7, 2: 16.7, 4: 25.4}),
    ("down", 1024, 3072, 14, True, {0: 0.0, 1: 5.5, 2: 8.9, 4: 15.1}),
    ("down", 1024, 3072, 10, True, {0: 0.0, 1: 4.7, 2: 8.0, 4: 13.9}),
    ("down", 1024, 3072, 16, True, {0: 0.0, 1: 5.0, 2: 8.1, 4: 17.7}),
    ("down", 1024, 3072, 9, True, {0: 0.0, 1: 4.0, 2: 7.1, 4: 11.8}),
    ("down", 1024, 3072, 12, True, {0: 0.0, 1: 4.2, 2: 7.6, 4: 17.3}),
    ("gate_up", 6144, 1024, 32, False, {0: 19.2, 2: 6.5, 4: 0.0}),
    ("gate_up", 12288, 2048, 32, True, {0: 88.8, 1: 53.5, 2: 11.4, 4: 0.0}),
    ("gate_up", 12288, 2048, 16, False, {0: 36.2, 2: 9.2, 4: 0.0}),
    ("gate_up", 12288, 2048, 40, True, {0: 118.8, 1: 51.3, 2: 13.6, 4: 0.0}),
    ("gate_up", 6144, 1024, 48, False, {0: 24.7, 2: 7.0, 4: 0.0}),
    ("gate_up", 6144, 1024, 28, False, {0: 14.7, 2: 5.0, 4: 0.0}),
    ("gate_up", 12288, 2048, 6, True, {0: 17.2, 1: 8.3, 2: 5.4, 4: 0.0}),
    ("gate_up", 3072, 512, 40, False, {0: 5.4, 2: 2.9, 4: 0.0}),
    ("o", 512, 512, 20, True, {0: 2.1, 1: 0.0, 2: 1.4, 4: 5.1}),
    ("o", 512, 512, 18, True, {0: 2.1, 1: 0.0, 2: 1.6, 4: 5.0}),
    ("gate_up", 3072, 512, 4, True, {0: 1.6, 1: 0.0, 2: 0.5, 4: 2.9}),
    ("gate_up", 3072, 512, 4, False, {0: 1.7, 2: 0.0, 4: 4.6}),
    ("gate_up", 12288, 2048, 14, False, {0: 31.1, 2: 6.2, 4: 0.0}),
    ("gate_up", 3072, 512, 36, False, {0: 5.3, 2: 2.4, 4: 0.0}),
    ("gate_up", 3072, 512, 3, True, {0: 1.4, 1: 0.0, 2: 0.5, 4: 2.3}),
    ("gate_up", 12288, 2048, 28, True, {0: 76.8, 1: 28.1, 2: 7.0, 4: 0.0}),
    ("gate_up", 12288, 2048, 18, True, {0: 42.2, 1: 19.6, 2: 6.0, 4: 0.0}),
    ("gate_up", 6144, 1024, 2, True, {0: 0.4, 1: 0.0, 2: 1.5, 4: 2.2}),
    ("gate_up", 6144, 1024, 40, True, {0: 26.3, 1: 9.2, 2: 0.5, 4: 0.0}),
    ("qkv", 1280, 1024, 2, True, {0: 0.0, 1: 2.9, 2: 4.4, 4: 5.4}),
    ("o", 1024, 1024, 2, True, {0: 0.0, 1: 3.3, 2: 5.4, 4: 6.6}),
    ("down", 1024, 3072, 2, True, {0: 0.0, 1: 9.5, 2: 14.3, 4: 16.4}),
    ("qkv", 1280, 1024, 2, False, {0: 0.0, 2: 2.5, 4: 10.3}),
    ("o", 1024, 1024, 2, False, {0: 0.0, 2: 3.7, 4: 13.8}),
    ("gate_up", 6144, 1024, 2, False, {0: 3.3, 2: 0.0, 4: 9.1}),
    ("down", 1024, 3072, 2, False, {0: 0.0, 2: 8.8, 4: 36.3}),
    ("qkv", 1280, 1024, 5, True, {0: 0.0, 1: 2.1, 2: 3.2, 4: 5.8}),
    ("o", 1024, 1024, 5, True, {0: 0.0, 1: 2.2, 2: 4.1, 4: 7.3}),
    ("gate_up", 6144, 1024, 5, True, {0: 0.6, 1: 0.0, 2: 0.9, 4: 3.1}),
    ("down", 1024, 3072, 5, True, {0: 0.0, 1: 9.0, 2: 12.0, 4: 16.2}),
    ("qkv", 1280, 1024, 5, False, {0: 0.0, 2: 2.2, 4: 10.6}),
    ("o", 1024, 1024, 5, False, {0: 0.0, 2: 3.4, 4: 15.0}),
    ("gate_up", 6144, 1024, 5, False, {0: 0.1, 2: 0.0, 4: 5.8}),
    ("down", 1024, 3072, 5, False, {0: 0.0, 2: 7.0, 4: 37.2}),
    ("qkv", 1280, 1024, 40, True, {0: 4.9, 1: 1.3, 2: 0.0, 4: 3.2}),
    ("o", 1024, 1024, 40, True, {0: 2.8, 1: 0.5, 2: 0.0, 4: 4.1}),
    ("down", 1024, 3072, 40, True, {0: 8.9, 1: 3.4, 2: 0.0, 4: 9.6}),
    ("qkv", 1280, 1024, 40, False, {0: 2.3, 2: 0.0, 4: 6.5}),
    ("o", 1024, 1024, 40, False, {0: 1.0, 2: 0.0, 4: 9.5}),
    ("gate_up", 6144, 1024, 40, False, {0: 28.7, 2: 13.0, 4: 0.0}),
    ("down", 1024, 3072, 40, False, {0: 12.3, 2: 0.0, 4: 25.8}),
    # the draft MLP between passes over a head that stays in cache
    ("gate_up", 2048, 2048, 5, True, {0: 2.9, 1: 0.0, 2: 2.1, 4: 5.5}),
    ("gate_up", 2048, 2048, 7, True, {0: 0.0, 1: 2.6, 2: 5.2, 4: 11.4}),
]


def choose_gemm(use, rows, k, tiles, packed):
    fn = getattr(_lib.load(), "_ZN3hpd11choose_gemmEiiibbi")
    fn.restype, fn.argtypes = ctypes.c_uint64, [ctypes.c_int] * 3 + [ctypes.c_bool] * 2 + [ctypes.c_int]
    v = fn(rows, k, 32 * tiles, packed, use in ("gate_up", "down"), EPI[use])
    return v & 0xffffffff, v >> 32   # GemmShape: rg, wide


@pytest.mark.parametrize("row", MEASURED, ids=lambda r: "-".join(str(v) for v in r[:5]))
def test_the_fastest_shape_is_taken(row):
    use, rows, k, tiles, packed, slower = row
    _, wide = choose_gemm(use, rows, k, tiles, packed)
    assert slower[wide] <= (0.8 if tiles == 40 else 0.5), (wide, slower)
