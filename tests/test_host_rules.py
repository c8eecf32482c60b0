"""Host rules of the library that need no device, compiled from their own
headers (csrc/*.hpp, plain C++) and run on the CPU."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1709_08018_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstring>
#include <cstdlib>
#include "walk_layout.hpp"
using namespace kl;
int main(int argc, char** argv) {
    unsigned long long n; unsigned b, s, t;
    while (scanf("%llu %u %u %u", &n, &b, &s, &t) == 4) {
        const WalkBinned L = walk_binned_layout(n, b, s, t);
        printf("%d %u %u %llu %llu %llu %d\n", (int)walk_binned_ok(1024, 1024, s), L.walkers, L.chunks,
               (unsigned long long)L.blocks, (unsigned long long)L.off_starts, (unsigned long long)L.bytes,
               (int)walk_clears(L, (unsigned long long)t * 32768));
    }
}
"""


LEASES = r"""
#include <cstdio>
#include "host_rules.hpp"
int main() {
    unsigned long long held, want;
    int idle;
    while (scanf("%llu %llu %d", &held, &want, &idle) == 3) {
        const kl::TableLease l = kl::table_lease(held, want, idle);
        printf("%d %d %llu %d\n", (int)l.lease, (int)l.release, (unsigned long long)l.allocate, idle);
        fflush(stdout);
    }
}
"""


MERGES = r"""
#include <cstdio>
#include "host_rules.hpp"
int main() {
    unsigned long long bins, units;
    int fp64, letters, tiling;
    while (scanf("%d %d %d %llu %llu", &fp64, &letters, &tiling, &bins, &units) == 5)
        printf("%d\n", (int)kl::batch_merges(fp64, letters, tiling, bins, units));
}
"""


def _compile(tmp_path, text):
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(text)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return str(exe)


@pytest.fixture(scope="module")
def walk_rules(tmp_path_factory):
    exe = _compile(tmp_path_factory.mktemp("walk_rules"), PROGRAM)

    def ask(cases):
        text = "".join("%d %d %d %d\n" % c for c in cases)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]

    return ask


def test_binned_walks_keep_their_staging_bound(walk_rules):
    """Every binned walk, up to the longest of 2^19 drawn points from any
    place in a block of eight, stages at most what 256 walkers of the longest
    walk take, 2^27 slots of 2 bytes and one region more, whatever the number
    of walkers; and at least one workgroup a launch."""
    bound = 2 ** 27 + 2048
    cases = [(n, burn, steps, tiles) for n in (1, 256, 257, 512, 513, 100000, 2 ** 30)
             for burn in (0, 1, 6, 7, 8, 13) for tiles in (1, 256)
             for steps in (1, 2, 8, 64, 1000, 131072, 262136, 262137, 262144, 262145, 400000, 524287, 524288)]
    for (n, burn, steps, tiles), (ok, walkers, chunks, blocks, ids, total, _) in zip(cases, walk_rules(cases)):
        where = (n, burn, steps, tiles)
        assert ok == 1, where
        first, last = (burn + 1) // 8, (burn + steps) // 8
        assert chunks == last - first + 1, where
        assert 1 <= blocks <= -(-n // walkers), where
        assert blocks * walkers * 8 * chunks <= bound, where
        assert ids == 2 * blocks * walkers * 8 * chunks and total == ids + 4 * blocks * chunks * (tiles + 1), where


def test_longer_walks_are_not_binned(walk_rules):
    """Past 2^19 drawn points, up to the most a walk may have, the automatic
    choice is the direct path."""
    cases = [(1, 0, s, 32) for s in (524289, 2 ** 31, 2 ** 32 - 8, 2 ** 32 - 7, 2 ** 32 - 2)]
    assert [r[0] for r in walk_rules(cases)] == [0] * len(cases)


def test_few_walkers_leave_the_clearing_to_a_launch(walk_rules):
    """The walkers clear the image themselves only where there are enough of
    them, 128 bins a thread at most: 3,000 walkers (6 workgroups) do not clear
    2500 x 2500 bins (191 tiles), nor 512 an image of 255 tiles; 2^20 do."""
    cases = [(3000, 0, 100, 191), (512, 0, 512, 255), (512, 0, 64, 2), (512, 0, 64, 3), (513, 0, 64, 4),
             (1 << 20, 0, 64, 32), (1 << 20, 0, 64, 256), (2, 0, 400000, 1), (2, 0, 400000, 2)]
    assert [r[6] for r in walk_rules(cases)] == [0, 0, 1, 0, 1, 1, 1, 1, 0]


MIB = 1 << 20


def test_large_buffer_is_given_back(tmp_path):
    """The buffer of the null stream's calls: it grows with a call, up to 192
    MiB; above 64 MiB it is given back by the 32nd call in a row that 64 MiB
    would have served, or that is above 192 MiB and takes a temporary, and a
    large call in between starts the count again; 64 MiB and less are kept."""
    p = subprocess.Popen([_compile(tmp_path, LEASES)], stdin=subprocess.PIPE, stdout=subprocess.PIPE, text=True)
    state = dict(held=0, idle=0)

    def call(want):
        p.stdin.write("%d %d %d\n" % (state["held"], want, state["idle"]))
        p.stdin.flush()
        lease, release, allocate, state["idle"] = map(int, p.stdout.readline().split())
        assert lease == (want <= 192 * MIB)
        assert release <= (state["held"] > 0) and (not allocate or release or not state["held"])
        state["held"] = allocate or (0 if release else state["held"])
        assert not lease or state["held"] >= want
        return state["held"]

    try:
        assert call(100) == MIB and call(MIB) == MIB and call(MIB + 1) == MIB + 1
        assert call(64 * MIB) == 64 * MIB and [call(5) for _ in range(100)] == [64 * MIB] * 100
        for large in (64 * MIB + 1, 150 * MIB, 192 * MIB):
            for small in (5, 64 * MIB, 192 * MIB + 1, 1 << 40):
                assert call(large) == large
                assert [call(small) for _ in range(31)] == [large] * 31
                assert call(64 * MIB + 1) == large                        # used: the count starts again
                assert [call(small) for _ in range(31)] == [large] * 31
                after = 0 if small > 192 * MIB else max(small, MIB)
                assert call(small) == after
                assert [call(5) for _ in range(40)] == [max(after, MIB)] * 40
                assert call(192 * MIB + 1) == max(after, MIB)             # a temporary; what is small stays
    finally:
        p.stdin.close()
        p.wait()


def test_batches_that_merge_their_runs(tmp_path):
    """Runs are merged up to four letters; with five in FP32, and in FP64 in
    tilings of 2^23 bins up and fewer than 8,192 units alone (forty sets of
    five letters and the tiling to depth 16 took longer merged); never with
    six."""
    cases = [(p, r, t, b, u) for p in (0, 1) for r in range(1, 9) for t in (0, 1)
             for b in (1, 1 << 20, (1 << 23) - 1, 1 << 23) for u in (1, 8191, 8192)]
    exe = _compile(tmp_path, MERGES)
    out = subprocess.run([exe], input="".join("%d %d %d %d %d\n" % c for c in cases), capture_output=True, text=True,
                         check=True).stdout.split()
    for (p, r, t, b, u), got in zip(cases, out):
        want = r <= 4 or (r == 5 and (p == 0 or (t == 1 and b >= 1 << 23 and u < 8192)))
        assert got == str(int(want)), (p, r, t, b, u)
