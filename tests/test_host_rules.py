"""Rules that the library's host code decides by, on the CPU: a small program
built from its internal headers prints what they answer."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

MAIN = """
#include <cstdio>
#include "lcd_host.h"
using namespace lcd;
int main() {
    long long a[8];
    char what[32];
    while (std::scanf("%31s %lld %lld %lld %lld %lld %lld", what, a, a + 1, a + 2, a + 3, a + 4, a + 5) == 7) {
        const std::string w = what;
        long long r = -1;
        if (w == "first_pool")
            r = first_pool(a[0], a[1], a[2], a[3], a[4], a[5]);
        else if (w == "row_ahead")
            r = row_ahead((int32_t)a[0], (int32_t)a[1], (int32_t)a[2], a[3]);
        else if (w == "lds_fits")
            r = team_lds_fits((int32_t)a[0], a[1]);
        else if (w == "lds_bytes")
            r = block_table_bytes((int32_t)a[0], block_hbits((int32_t)a[0])) + kTeamShBytes;
        else if (w == "holds")
            r = team_table_holds((int32_t)a[0]);
        std::printf("%lld\\n", r);
    }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    src, exe = str(d / "rules.cpp"), str(d / "rules")
    with open(src, "w") as f:
        f.write("#include <string>\n" + MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-D__HIP_PLATFORM_AMD__", "-I", ROCM + "/include", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1301_0955_amd", "csrc"), src, "-o", exe], check=True)

    def ask(rows):
        text = "".join("%s %s\n" % (w, " ".join(str(x) for x in (list(a) + [0] * 6)[:6])) for w, *a in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [int(x) for x in out.split()]
    return ask


def test_first_pool_leaves_the_tables_their_memory(rules):
    """A sweep that fits with the least pool fits with the one that is chosen."""
    G = 1 << 30
    rows, at = [], []
    for free in (G, 2 * G, 5 * G, 14 * G, 280 * G):
        for other in (0, free // 2, free - G // 16, free - G // 256, free, free + G):
            for sets, scales, n in ((1, 1, 1), (20_000, 32, 100_000), (115_000, 2, 1 << 22), (14_184, 64, 10 ** 7),
                                    (2 ** 24, 100, 2 ** 27), (0, 8, 0)):
                least = max(1 << 16, sets * (scales // 4 + 2) * 32)
                rows.append(("first_pool", least, sets, scales, n, free, other))
                at.append((least, free, other))
    for (least, free, other), r in zip(at, rules(rows)):
        assert r >= least
        if r > least:
            assert 4 * r <= (free - other) // 16


def test_first_pool_has_room_for_a_record_every_second_scale(rules):
    assert rules([("first_pool", 1 << 16, 4000, 8, 60_013, 280 << 30, 6 << 30)]) == [4000 * 6 * 512]


def test_reading_ahead_ends_with_the_entries(rules):
    """Offsets of a row that starts close to the largest index a graph can have."""
    M = 2 ** 31 - 1
    rows = [("row_ahead", beg, off, k, nnz) for nnz in (M, M - 600, 1000) for beg in (nnz - 600, nnz - 64, nnz - 9, nnz)
            for off in (0, 8, 9, 63, 64, 511) for k in (0, 9, 2000) if beg >= 0]
    for (_, beg, off, k, nnz), r in zip(rows, rules(rows)):
        assert r == (off < k and beg + off < nnz), (beg, off, k, nnz)


def test_table_sizes_that_hash_slots_cannot_name_are_refused(rules):
    """16-bit index fields keep one bit for claims: no table between 32,768 entries and the wide ones."""
    caps = {1: 1, 16384: 1, 32768: 1, 32769: 0, 49152: 0, 65535: 0, 65536: 1, 131072: 1, 2 ** 30: 1, 2 ** 30 + 1: 0,
            0: 0, -2 ** 31: 0}
    assert rules([("holds", c) for c in caps]) == list(caps.values())


def test_lds_tables_fit_what_is_launched(rules):
    """Every accepted capacity fits with the layout that runs; in 160 KiB the accepted ones end at 4,096."""
    caps = list(range(64, 8256, 64))
    for lds in (64 << 10, 160 << 10):
        ok = rules([("lds_fits", c, lds) for c in caps])
        size = rules([("lds_bytes", c) for c in caps])
        assert all(b <= lds for a, b in zip(ok, size) if a) and any(ok) and not all(ok)
    assert [c for c, a in zip(caps, ok) if a] == list(range(64, 4160, 64))
    assert rules([("lds_fits", 100, 160 << 10), ("lds_fits", 8256, 1 << 30)]) == [0, 0]
