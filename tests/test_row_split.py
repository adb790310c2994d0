"""The rule that says which attention calls run with two waves per row, against measurements: each point below is a call
whose two forms were timed and differ by 4 % or more, and the rule has to take the faster one (compiled here: the rule is
plain C++ on host values)."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    out = tmp_path_factory.mktemp("row_split")
    src, lib = out / "rule.cpp", out / "librule.so"
    src.write_text('#include "row_split.h"\n'
                   'extern "C" int rule(long rows, long even_rows, int longest, int kv_heads, int group, int dense, int bk32, int int8,\n'
                   '                    int fp8, int by_position) {\n'
                   '  return sale::two_waves_per_row({rows, even_rows, longest, kv_heads, group, dense != 0, bk32 != 0, int8 != 0,\n'
                   '                                  fp8 != 0, by_position != 0});\n}\n'
                   'extern "C" int heads(int bk32, int group, long rows, int words) {\n'
                   '  return sale::select_heads_per_wave(bk32 != 0, group, rows, words);\n}\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2505_24179_amd", "csrc"), str(src),
                    "-o", str(lib)], check=True)
    fn = ctypes.CDLL(str(lib)).rule
    fn.argtypes = [ctypes.c_long] * 2 + [ctypes.c_int] * 8
    fn.heads = ctypes.CDLL(str(lib)).heads
    fn.heads.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_long, ctypes.c_int]
    return fn


# (kind, 64-key blocks of the longest row, rows, KV heads, query heads per KV head): us with one wave per row, with two
MEASURED = [
    # short rows, more of them than places for their halves
    ("dense", 1, 576, 64, 9, 14.1, 16.1), ("dense", 1, 660, 20, 33, 14.3, 16.2), ("sparse", 1, 768, 192, 4, 15.9, 18.9),
    ("sparse", 2, 768, 96, 4, 19.8, 21.8), ("dense", 4, 1280, 80, 4, 29.6, 30.9), ("sparse", 4, 1280, 80, 4, 30.2, 32.6),
    ("sparse32", 4, 1280, 80, 4, 30.1, 32.7), ("sparse", 8, 1280, 160, 1, 41.1, 44.0), ("sparse32", 16, 1536, 24, 4, 45.8, 48.8),
    ("sparse32", 16, 2048, 32, 4, 53.2, 61.0),
    # few rows, or long ones
    ("dense", 1, 512, 128, 4, 14.8, 12.0), ("sparse", 4, 512, 32, 4, 20.9, 17.9), ("dense", 4, 1024, 64, 4, 25.8, 24.6),
    ("sparse", 6, 960, 40, 4, 29.4, 27.1), ("dense", 6, 960, 40, 4, 28.5, 26.8), ("sparse", 8, 1024, 32, 4, 33.3, 28.8),
    ("sparse32", 8, 1024, 32, 4, 32.8, 29.6), ("fp8", 8, 1024, 32, 4, 41.7, 39.6), ("fp8", 8, 1536, 48, 4, 55.0, 52.1),
    ("fp8", 3, 960, 80, 4, 37.9, 36.0), ("sparse", 12, 1008, 21, 4, 39.3, 37.0), ("dense", 16, 512, 8, 4, 41.6, 27.6),
    ("dense", 16, 1024, 16, 4, 45.3, 37.0), ("sparse", 16, 1024, 16, 4, 44.6, 36.5), ("fp8", 16, 1024, 16, 4, 50.4, 44.5),
    ("fp8 dense", 16, 1024, 16, 4, 50.0, 43.0), ("sparse", 24, 1248, 13, 4, 57.1, 54.5), ("dense", 32, 1152, 4, 9, 69.3, 62.0),
    ("sparse32", 32, 1152, 4, 9, 60.0, 53.3), ("fp8", 32, 1152, 4, 9, 65.8, 58.8), ("sparse", 48, 1536, 8, 4, 90.9, 85.7),
    ("sparse32", 64, 1280, 5, 4, 77.6, 73.9), ("sparse", 64, 1024, 4, 4, 102.1, 73.7), ("fp8 dense", 64, 1280, 5, 4, 103.3, 98.2),
    ("sparse", 109, 1308, 4, 3, 127.6, 116.3), ("sparse32", 109, 1308, 4, 3, 100.7, 88.6), ("fp8", 128, 1536, 3, 4, 125.9, 118.0),
    ("fp8 dense", 2, 1536, 192, 4, 48.0, 43.3),
    # more rows than that
    ("sparse", 16, 1536, 24, 4, 47.9, 50.4), ("dense", 16, 1536, 24, 4, 50.0, 52.2), ("dense", 6, 1056, 44, 4, 32.2, 33.7),
    ("sparse", 32, 1792, 14, 4, 71.9, 80.8), ("sparse32", 32, 1792, 14, 4, 66.6, 77.5), ("sparse", 32, 2048, 16, 4, 75.8, 84.7),
    ("dense", 32, 1408, 11, 4, 74.6, 80.8), ("sparse", 64, 2048, 8, 4, 115.4, 130.4), ("sparse32", 64, 2048, 8, 4, 92.4, 104.2),
    ("sparse32", 60, 1920, 8, 4, 85.8, 98.4), ("dense", 64, 1536, 6, 4, 124.4, 131.9), ("fp8", 64, 2048, 8, 4, 108.8, 116.1),
    ("fp8 dense", 128, 1536, 3, 4, 170.2, 181.3), ("int8", 32, 1792, 14, 4, 79.7, 89.3),
    # many KV heads on every XCD
    ("dense", 16, 1008, 63, 1, 50.2, 57.5), ("dense", 16, 1008, 21, 3, 48.7, 41.2), ("dense", 16, 688, 43, 1, 47.4, 40.4),
    ("dense", 16, 992, 62, 1, 49.8, 46.6), ("sparse", 16, 992, 62, 1, 48.6, 44.9), ("dense", 64, 1216, 19, 1, 126.1, 147.1),
    ("sparse", 64, 1216, 19, 1, 114.8, 121.3), ("sparse32", 64, 1216, 19, 1, 91.5, 97.5),
    ("sparse", 64, 1152, 18, 1, 105.9, 93.2), ("sparse32", 64, 1152, 18, 1, 84.5, 77.1),
    ("int8 dense", 64, 1152, 18, 1, 129.8, 114.9), ("int8 dense", 64, 1216, 19, 1, 129.1, 136.1),
    ("int8", 64, 1216, 19, 1, 120.5, 113.9), ("sparse32", 27, 1215, 45, 1, 71.2, 74.7), ("dense", 27, 1215, 45, 1, 69.8, 87.0),
    ("int8 dense", 27, 1215, 45, 1, 83.4, 90.8), ("dense", 1, 580, 580, 1, 29.5, 21.0), ("dense", 64, 960, 15, 1, 118.7, 108.4),
    ("dense", 256, 1280, 5, 1, 416.0, 486.8), ("sparse", 256, 1280, 5, 1, 217.1, 226.1),
    ("sparse32", 256, 1280, 5, 1, 155.6, 169.4), ("sparse", 256, 1280, 1, 5, 199.9, 166.2),
]


@pytest.mark.parametrize("kind,longest,rows,kv_heads,group,one,two", MEASURED)
def test_rule_takes_the_faster_form(rule, kind, longest, rows, kv_heads, group, one, two):
    assert abs(one - two) >= 0.04 * min(one, two)
    got = rule(rows, rows, longest, kv_heads, group, "dense" in kind, "sparse32" in kind, "fp8" in kind or "int8" in kind,
               "fp8" in kind, False)
    assert bool(got) == (two < one)


def test_few_rows_always_and_many_never(rule):
    """Up to 512 rows every half row has a place of its own; beyond the limits the form was measured with it is not used."""
    for dense, bk32, int8, fp8, most in ((0, 0, 0, 0, 1536), (0, 0, 1, 0, 1536), (0, 1, 0, 0, 1536), (0, 1, 1, 0, 1536),
                                         (0, 0, 1, 1, 1536), (1, 0, 0, 0, 1280), (1, 0, 1, 0, 1280), (1, 0, 1, 1, 1536)):
        for kv_heads, group in ((1, 1), (8, 4), (63, 1), (5, 2), (512, 1)):
            for longest in (1, 2, 3, 4, 7, 8, 16, 31, 64, 100, 4096):
                on = [rule(rows, rows, longest, kv_heads, group, dense, bk32, int8, fp8, False) for rows in range(1, 2200)]
                limit = sum(on)
                assert 512 <= limit <= most and all(on[:limit])


# Selection-Pass: (query heads, KV heads, tokens): us with two heads per wave, with four
SELECT = [
    (32, 8, 12288, 178.8, 182.2), (32, 8, 16384, 280.4, 287.2), (32, 8, 20480, 402.7, 412.8), (32, 8, 25024, 586.2, 601.0),
    (64, 8, 16384, 532.8, 539.3), (4, 1, 32768, 145.0, 165.5), (8, 1, 30720, 239.5, 242.9), (8, 2, 32768, 266.5, 270.9),
    (12, 1, 32768, 396.1, 384.7), (32, 8, 30720, 866.9, 829.3), (32, 8, 40960, 1415.4, 1387.8), (32, 8, 49152, 1982.5, 1941.5),
    (4, 1, 65536, 486.3, 478.2), (8, 2, 49152, 562.3, 554.6), (16, 2, 65536, 1765.9, 1726.5), (8, 2, 65536, 914.8, 887.7),
    (32, 8, 65536, 3438.3, 3288.1), (4, 1, 131072, 1822.5, 1744.7), (8, 2, 131072, 3468.2, 3429.3), (32, 8, 131072, 13309.0, 12531.1),
]


@pytest.mark.parametrize("q_heads,kv_heads,tokens,two,four", SELECT)
def test_selection_takes_the_faster_number_of_heads(rule, q_heads, kv_heads, tokens, two, four):
    assert abs(two - four) >= 0.01 * min(two, four)
    rows, words = tokens // 64 * q_heads, -(-tokens // 4096)
    assert rule.heads(0, q_heads // kv_heads, rows, words) == (4 if four < two else 2)
    assert rule.heads(1, q_heads // kv_heads, rows, words) == 2
    assert rule.heads(0, 3, rows, words) == 1 and rule.heads(0, 6, rows, words) == 2
