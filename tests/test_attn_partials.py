"""Partial sums of attention spans: the last workgroup of a group to arrive merges them with ordinary
loads, which is sound only while no 128-byte line holds values of two groups (another group's merge
could have brought the line into the reader's L2 before the values were written).  The layout
functions of the kernels are compiled for the host and every value of a launch is placed."""
import ctypes
import itertools
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LINE = 32  # floats

SRC = """
#include "attn_part.h"
extern "C" {
size_t out_at(size_t row, int H, int h, int nspan, int sp, int hd) { return sd2::part_out(row, H, h, nspan, sp, hd); }
size_t ml_at(size_t rows, int H, int hd, size_t block, int nspan, int sp, int i) {
    return sd2::part_ml(rows, H, hd, block, nspan, sp, i);
}
size_t row_floats(int nsplit, int hd) { return sd2::part_row(nsplit, hd); }
size_t floats(size_t rows, int H, int hd, size_t blocks) { return sd2::part_floats(rows, H, hd, blocks); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("part")
    (d / "p.cpp").write_text(SRC)
    so = d / "p.so"
    subprocess.check_call(["g++", "-shared", "-fPIC", "-O2", "-std=c++17", "-I",
                           os.path.join(ROOT, "paper_2511_09844_amd", "csrc"), str(d / "p.cpp"), "-o", str(so)])
    lib = ctypes.CDLL(str(so))
    sz, i = ctypes.c_size_t, ctypes.c_int
    lib.out_at.restype = lib.ml_at.restype = lib.floats.restype = lib.row_floats.restype = sz
    lib.out_at.argtypes = [sz, i, i, i, i, i]
    lib.ml_at.argtypes = [sz, i, i, sz, i, i, i]
    lib.floats.argtypes = [sz, i, i, sz]
    lib.row_floats.argtypes = [i, i]
    return lib


def _check(values, size):
    """values: (group, first float, floats) of everything a launch writes."""
    seen, owner = set(), {}
    for group, at, n in values:
        for x in range(at, at + n):
            assert x not in seen and x < size
            seen.add(x)
            assert owner.setdefault(x // LINE, group) == group, f"line {x // LINE}: groups {owner[x // LINE]}, {group}"


@pytest.mark.parametrize("hd", [32, 64, 128])
@pytest.mark.parametrize("nseq,rps,Hkv,G", [(1, 1, 12, 1), (1, 6, 12, 1), (2, 4, 3, 5), (3, 15, 2, 4), (2, 9, 1, 8)])
def test_few_row_spans_share_no_line_between_groups(lib, hd, nseq, rps, Hkv, G):
    # groups of k_vattn: (sequence, KV head, 16 query vectors)
    H, rows, ncg = Hkv * G, nseq * rps, (rps * G + 15) // 16
    for nspan in (1, 3, 8):
        values = []
        for b, kvh, v, sp in itertools.product(range(nseq), range(Hkv), range(rps * G), range(nspan)):
            block, row, h = (b * Hkv + kvh) * ncg + v // 16, b * rps + v // G, kvh * G + v % G
            values.append((block, lib.out_at(row, H, h, nspan, sp, hd), hd))
            values.append((block, lib.ml_at(rows, H, hd, block, nspan, sp, v % 16), 2))
        _check(values, nspan * lib.floats(rows, H, hd, nseq * Hkv * ncg))


@pytest.mark.parametrize("hd", [32, 64, 128])
@pytest.mark.parametrize("nseq,rps,Hkv,G", [(1, 16, 12, 1), (1, 37, 3, 4), (3, 17, 1, 5)])
def test_many_row_spans_share_no_line_between_groups(lib, hd, nseq, rps, Hkv, G):
    # groups of k_pattn: (sequence, KV head, 16 rows)
    H, rows, nqb = Hkv * G, nseq * rps, (rps + 15) // 16
    for nspan in (1, 3):
        values = []
        for b, kvh, i, g, sp in itertools.product(range(nseq), range(Hkv), range(rps), range(G), range(nspan)):
            group, row, h = (b * Hkv + kvh) * nqb + i // 16, b * rps + i, kvh * G + g
            values.append((group, lib.out_at(row, H, h, nspan, sp, hd), hd))
            values.append((group, lib.ml_at(rows, H, hd, group * G + g, nspan, sp, i % 16), 2))
        _check(values, nspan * lib.floats(rows, H, hd, nseq * Hkv * nqb * G))


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("nsplit", [2, 3, 9, 13, 24])
def test_persistent_runs_share_no_line_between_groups(lib, hd, nsplit):
    # a group holds whole (row, head) pairs: 2 rows x 3 heads, every run live
    values = [(rh, rh * lib.row_floats(nsplit, hd) + sp * (hd + 4), hd + 2) for rh in range(6) for sp in range(nsplit)]
    _check(values, 6 * lib.row_floats(nsplit, hd))
