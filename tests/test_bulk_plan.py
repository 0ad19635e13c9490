"""The bulk form's plan (csrc/bulk_plan.hpp), compiled for the CPU: which calls have one, and that
every plan fits the hardware and its own arrays."""
import ctypes
import os
import random
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1710_11246_amd", "csrc")
DRIVER = """
#include <math.h>
#include <stddef.h>
#include <stdint.h>
namespace {
#include "bulk_plan.hpp"
}
extern "C" int plan(uint64_t n, uint32_t buckets, uint32_t num_cu, int insert, int keys_only,
                    uint64_t since_reset, uint64_t *out)
{
    BulkPlan P;
    if (!bulk_plan(BulkCall{n, buckets, num_cu, insert != 0, keys_only != 0, since_reset}, &P))
        return 0;
    const uint64_t v[] = {P.rows, P.waves, P.chunk, P.a.span, P.a.parts, P.a.tiles, P.a.tile,
                          P.a.row, P.a.queue, P.split_lds, P.part_lds, P.merge_lds, P.starts, P.key,
                          P.place, P.flag, P.val, P.later, P.total};
    for (unsigned i = 0; i < sizeof(v) / sizeof(v[0]); ++i)
        out[i] = v[i];
    return 1;
}
"""
FIELDS = ("rows waves chunk span parts tiles tile row queue split_lds part_lds merge_lds "
          "starts key place flag val later total").split()
KINDS = ["search", "search of keys", "insert"]
TOP = 1 << 26           # operations of a batch that is not taken in pieces
LARGEST = 6_600_000     # buckets whose slabs fit the compute units' LDS in every kind
LEAST = {"search": 1 << 21, "search of keys": 1 << 21, "insert": 1 << 17}


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = str(d / "plan.cpp"), str(d / "plan.so")
    open(src, "w").write(DRIVER)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                           "-I", CSRC, src, "-o", lib])
    f = ctypes.CDLL(lib).plan
    f.argtypes = [ctypes.c_uint64, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_int, ctypes.c_int,
                  ctypes.c_uint64, ctypes.c_void_p]

    def call(n, buckets, kind, num_cu=256, since_reset=0):
        out = (ctypes.c_uint64 * len(FIELDS))()
        ok = f(n, buckets, num_cu, kind == "insert", kind == "search of keys", since_reset, out)
        return dict(zip(FIELDS, out)) if ok else None
    return call


def check(p, n, buckets, kind):
    lds = 160 * 1024
    assert p["split_lds"] <= lds and p["part_lds"] <= lds and p["merge_lds"] <= lds
    assert p["parts"] <= 15872 and p["tiles"] <= 2048 and p["span"] <= 1000
    assert p["span"] * p["parts"] >= buckets > p["span"] * (p["parts"] - 1)
    assert p["chunk"] == min(n, TOP)
    assert p["tile"] * p["tiles"] >= p["chunk"] > p["tile"] * (p["tiles"] - 1)
    assert p["tile"] == 1024 * p["rows"] and p["rows"] in (4, 8, 16, 32)
    # a part's starts are 16-bit places of a tile; 32 of a thread's operations are bits of a word
    assert p["tile"] <= 1 << 15 and 2 * p["row"] > p["parts"]
    assert 64 <= p["queue"] <= 32 * 64 * p["waves"] and p["queue"] % 4 == 0
    # what the kernels lay out in LDS, and in the workspace
    row = {"search": 33 * 8 + 32 + 1, "search of keys": 33 * 8 + 64 + 1,
           "insert": 33 * 8 + 64 + 12}[kind]
    runs = 8 * p["tiles"] + 4 + 4 * p["waves"]
    need = p["span"] * row + 8 + runs + (4 * p["queue"] if kind == "insert" else 4 + 6 * p["queue"])
    assert p["part_lds"] >= need
    slots = p["tile"] * p["tiles"]
    size = dict(starts=4 * p["row"] * p["tiles"], key=4 * slots, place=2 * slots, flag=slots)
    if kind == "insert":
        size.update(val=4 * slots, later=4 * slots)
    at = sorted((p[f], s) for f, s in size.items())
    end = 256
    for off, s in at:
        assert off >= end and off % 256 == 0
        end = off + s
    assert p["total"] >= end


def per_bucket(kind):
    return [6, 6.3, 7, 8, 9.5, 11, 12.9, 14, 16, 17.3, 19.3, 22, 25.9] + (
        [] if kind == "insert" else [31, 40, 77, 150, 800])


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("num_cu", [256, 304, 32])
def test_no_holes(plan, kind, num_cu):
    """Between its lines every batch has a plan: from the smallest batch on, from six operations
    per bucket, up to the buckets whose slabs fit."""
    least = 3 << 20 if "search" in kind else LEAST[kind]
    n = least
    sizes = []
    while n < TOP:
        sizes += [n, n + 1, n + n // 100]
        n = n * 9 // 8
    sizes += [3 << 24, 1 << 25, (1 << 25) + 1, TOP - 1, TOP, TOP + 1, 3 << 25, (1 << 32) - 1]
    missing = []
    for n in sizes:
        for per in per_bucket(kind):
            b = int(min(n, TOP) / per)
            if kind == "insert" and n > 26 * b:
                continue
            if not 1024 <= b <= LARGEST:
                continue
            p = plan(n, b, kind, num_cu)
            if p is None:
                missing.append((n, b))
            else:
                check(p, n, b, kind)
    assert not missing


@pytest.mark.parametrize("kind", KINDS)
def test_plans_of_drawn_calls(plan, kind):
    rng = random.Random(KINDS.index(kind))
    found = 0
    for _ in range(4000):
        n = int(2 ** rng.uniform(16, 27))
        b = max(1, int(n / 2 ** rng.uniform(1, 12)))
        p = plan(n, b, kind, rng.choice([256, 256, 64, 228, 304]))
        if p is not None:
            found += 1
            check(p, n, b, kind)
    assert found > 500


def test_lines(plan):
    for kind in KINDS:
        b = 40000
        assert plan(LEAST[kind] - 1, 6000 if kind == "insert" else b, kind) is None
        assert plan(LEAST[kind], 6000 if kind == "insert" else b, kind)
        n = 6 * b * 9
        assert plan(n, n // 6, kind) and plan(n, n // 6 + 1, kind) is None
        assert plan(TOP, (TOP // 6) - 1, kind) is None  # slabs that do not fit
        assert plan(1 << 22, 1023, kind) is None
    assert plan((3 << 20) - 1, (1 << 15) - 1, "search") is None and plan(3 << 20, 1024, "search")
    # inserts that the base slabs have no room for
    assert plan(26 * 20000, 20000, "insert") and plan(26 * 20000 + 1, 20000, "insert") is None
    assert plan(20 * 20000, 20000, "insert", since_reset=6 * 20000)
    assert plan(20 * 20000, 20000, "insert", since_reset=6 * 20000 + 1) is None
