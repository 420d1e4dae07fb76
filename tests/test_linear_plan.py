"""How massv_linear cuts a call into workgroups (csrc/linear_plan.h, plain host code, compiled here by itself): a call uses
what massv_linear_workspace asks for and no more."""
import os
import shutil
import subprocess

import pytest

import test_gpu_linear as shapes
from paper_2505_10526_amd import binding

CSRC = os.path.join(os.path.dirname(binding.__file__), "csrc")
DRIVER = r"""
#include "linear_plan.h"
#include <cstdio>
#include <cstring>
#include <initializer_list>
using namespace massv;
static bool same(const LinPlan& a, const LinPlan& b) { return !memcmp(&a, &b, sizeof a); }
// "plan M N K": the plan with the room asked for, and those bytes.  "rooms M0 M1 N K": over these row counts, the first where the plan with the room
// asked for is not the plan with more, or where a smaller room does not hold what is planned into it (or 0), and how many split K.
int main() {
    char what[16];
    int a, b, c, d;
    while (scanf("%15s", what) == 1) {
        if (!strcmp(what, "plan") && scanf("%d %d %d", &a, &b, &c) == 3) {
            const LinPlan p = linear_plan(a, b, c, linear_asked_room(a, b, c));
            printf("%d %d %d %zu\n", p.tile, p.parts, p.big, linear_asked_room(a, b, c));
        } else if (!strcmp(what, "rooms") && scanf("%d %d %d %d", &a, &b, &c, &d) == 4) {
            int bad = 0, split = 0;
            for (int M = a; M <= b; ++M) {
                const size_t asked = linear_asked_room(M, c, d), one = (size_t)M * c * 4;
                const LinPlan all = linear_plan(M, c, d, asked);
                split += all.parts > 1;
                bool ok = linear_plan(M, c, d, 0).parts == 1 && linear_part_bytes(all, M, c) <= asked;
                for (size_t more : {(size_t)0, one, 2 * one, (size_t)64 << 20, (size_t)1 << 33, kLinAnyRoom - asked}) ok = ok && same(linear_plan(M, c, d, asked + more), all);
                for (size_t room = one; room < asked; room += one) ok = ok && linear_part_bytes(linear_plan(M, c, d, room + 255), M, c) <= room + 255;
                if (!ok && !bad) bad = M;
            }
            printf("%d %d\n", bad, split);
        } else return 1;
    }
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(DRIVER)
    subprocess.check_call([cxx, "-O2", "-std=c++17", "-I", CSRC, str(d / "plan.cpp"), "-o", str(d / "plan")])

    def run(lines):
        out = subprocess.run([str(d / "plan")], input="\n".join(lines), text=True, capture_output=True, check=True).stdout
        return [tuple(int(v) for v in line.split()) for line in out.splitlines()]
    return run


# N, K of the maps of the 7B, 12B and 1.5B shapes and their projectors, and a few beside them
WIDTHS = [(3584, 18944), (18944, 3584), (3584, 3584), (4608, 3584), (3840, 15360), (15360, 3840), (8192, 3840), (3840, 4096), (3840, 8192), (1536, 8960),
          (8960, 1536), (2048, 1536), (1536, 1536), (5120, 5120), (3584, 5120), (5120, 1280), (4096, 10752), (4096, 11008), (11008, 4096), (320, 18944),
          (512, 4160), (1024, 1024), (16, 64), (8192, 8192)]


def test_more_room_than_asked_for_changes_nothing(ask):
    got = ask([f"rooms 1 8000 {n} {k}" for n, k in WIDTHS])
    assert [w for w, (bad, _) in zip(WIDTHS, got) if bad] == [], got
    assert sum(split for _, split in got) > 5000                     # (plans that split K are what it is about)


def test_the_library_asks_for_that_room(ask):
    shapes = [(m, n, k) for n, k in WIDTHS for m in (1, 16, 60, 129, 150, 192, 300, 1111, 4097)]
    lib = binding.load()
    for (m, n, k), (_, _, _, nbytes) in zip(shapes, ask([f"plan {m} {n} {k}" for m, n, k in shapes])):
        least = (((m + 15) // 16 * 16 * k * 2) + 255) // 256 * 256
        assert lib.massv_linear_workspace(m, n, k, binding.BF16) == least + nbytes, (m, n, k)


# unsplit squares over a long K were 2 to 18 % slower in these than 256 x 128 with K in two (or three); and neighbours where they are the faster ones
@pytest.mark.parametrize("M,N,K,fj,parts", [(1000, 3840, 15360, 2, 2), (1148, 3584, 18944, 2, 2), (460, 5120, 5120, 2, 3), (900, 4096, 11008, 2, 2), (1800, 2048, 16384, 2, 2),
                                            (600, 5120, 5120, 1, 1), (700, 3584, 5120, 1, 1), (1000, 3584, 3584, 1, 1), (530, 3840, 3840, 1, 1)])
def test_tile_of_long_k(ask, M, N, K, fj, parts):
    assert ask([f"plan {M} {N} {K}"])[0][:3] == (fj, parts, 0)


# the same by how full the last row tile is: squares took 40.0 us for 378 x 4096 -> 6144 and 256 x 128 with K in three 36.6, 31.5 and 32.4 for 262 rows; 76.0 and 70.5
# for 1145 x 8192 -> 3072, 64.7 and 67.0 for 1065; 42.8 and 37.2 for 600 x 4608 -> 3584; two rounds of 192 rows 113 for 2046 x 5120 -> 5120, one of 256 rows 105
@pytest.mark.parametrize("M,N,K,fj,parts", [(378, 6144, 4096, 2, 3), (262, 6144, 4096, 1, 1), (1145, 3072, 8192, 2, 2), (1065, 3072, 8192, 1, 1), (600, 3584, 4608, 2, 3),
                                            (630, 3584, 3584, 2, 3), (128, 18944, 3584, 1, 1), (2046, 5120, 5120, 4, 1), (1136, 4096, 11008, 4, 3)])
def test_tile_of_full_rows(ask, M, N, K, fj, parts):
    assert ask([f"plan {M} {N} {K}"])[0][:3] == (fj, parts, 0)


@pytest.mark.parametrize("name,fj,split", [("TALL", 4, False), ("TALL_SPLIT", 4, True), ("SQUARE", 1, False), ("SQUARE_SPLIT", 1, True), ("LOW192", 3, False),
                                           ("LOW192_SPLIT", 3, True), ("FLAT", 2, False), ("FLAT_SPLIT", 2, True)])
def test_shapes_of_the_tile_tests_take_their_tiles(ask, name, fj, split):
    """The lists of test_gpu_linear.py are there for one tile each; split ones with ranges of K of unequal length among them."""
    listed = getattr(shapes, name)
    got = ask([f"plan {m} {n} {k}" for m, n, k in listed])
    assert all((f, p > 1, big) == (fj, split, 0) for f, p, big, _ in got), list(zip(listed, got))
    assert not split or sum(k // 64 % p != 0 for (_, _, k), (_, p, _, _) in zip(listed, got)) >= 2


def test_shapes_of_both_heights_end_in_halves(ask):
    got = ask([f"plan {m} {n} {k}" for m, n, k in shapes.MIXED])
    assert [s for s, (_, _, big, _) in zip(shapes.MIXED, got) if not big] == [(6145, 4096, 64)]       # (a row of tiles too many)
