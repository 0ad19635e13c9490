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
PAYS = """
extern "C" int pays(uint64_t n, uint32_t buckets, int insert, int keys_only, uint64_t since_reset,
                    int counted)
{
    return bulk_pays(BulkCall{n, buckets, 256, insert != 0, keys_only != 0, since_reset}, counted);
}
"""
KINDS = ["search", "search of keys", "insert"]
TOP = 1 << 26           # operations of a batch that is not taken in pieces
LARGEST = 6_600_000     # buckets whose slabs fit the compute units' LDS in every kind
LEAST = {"search": 1 << 21, "search of keys": 1 << 21, "insert": 1 << 17}


@pytest.fixture(scope="module")
def library(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = str(d / "plan.cpp"), str(d / "plan.so")
    open(src, "w").write(DRIVER + PAYS)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                           "-I", CSRC, src, "-o", lib])
    return ctypes.CDLL(lib)


@pytest.fixture(scope="module")
def pays(library):
    f = library.pays
    f.argtypes = [ctypes.c_uint64, ctypes.c_uint32, ctypes.c_int, ctypes.c_int, ctypes.c_uint64,
                  ctypes.c_int]
    return lambda n, buckets, kind, held=0, counted=True: bool(
        f(n, buckets, kind == "insert", kind == "search of keys", held, counted))


@pytest.fixture(scope="module")
def plan(library):
    f = library.plan
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


@pytest.mark.parametrize("kind", ["search", "search of keys"])
def test_where_searches_pay(pays, kind):
    """Per bucket: 10 of lists of one slab, 16 up to two slabs, 64 beyond and where it is unknown."""
    slab = 62 if kind == "search of keys" else 31
    n = 7 << 19
    assert pays(n, 60000, kind) and not pays(n - 1, 60000, kind)
    for n in (7 << 19, 1 << 23, 1 << 26, 1 << 28):
        m = min(n, TOP)
        for per_slab, per in ((0, 10), (2 / 3 - .01, 10), (2 / 3 + .01, 16), (1.99, 16), (2.01, 64),
                              (50, 64)):
            b = m // per
            assert pays(n, b, kind, int(per_slab * slab * b))
            assert not pays(n, b + 1, kind, int(per_slab * slab * (b + 1)))
        assert pays(n, m // 64, kind, 0, False) and not pays(n, m // 64 + 1, kind, 0, False)


def test_where_inserts_pay(pays):
    """An empty table from 2^17 at 15 per bucket, 2^18 at ten and 3 * 2^17 at six; any other from
    2^20 at twelve."""
    for n, per in ((1 << 17, 15), ((1 << 18) - 1, 15), (1 << 18, 10), ((3 << 17) - 1, 10),
                   (3 << 17, 6), (1 << 26, 6)):
        assert pays(n, n // per, "insert") and not pays(n, n // per + 1, "insert")
    assert not pays((1 << 17) - 1, 2000, "insert")
    for held in (1, 100000):
        assert pays(1 << 20, (1 << 20) // 12, "insert", held)
        assert not pays(1 << 20, (1 << 20) // 12 + 1, "insert", held)
        assert not pays((1 << 20) - 1, 20000, "insert", held)


def test_what_pays_has_a_plan(plan, pays):
    """From 1024 buckets up to those whose slabs fit, and within the base slabs' room."""
    rng = random.Random(9)
    found = 0
    for _ in range(20000):
        kind = rng.choice(KINDS)
        n = int(2 ** rng.uniform(17, 28))
        b = int(n / 2 ** rng.uniform(1, 8))
        held = rng.choice([0, 0, int(b * rng.uniform(0, 30))])
        if not 1024 <= b <= LARGEST or kind == "insert" and n + held > 26 * b:
            continue
        if pays(n, b, kind, held):
            found += 1
            assert plan(n, b, kind, since_reset=held)
    assert found > 500
