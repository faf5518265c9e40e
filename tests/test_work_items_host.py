"""The rules that cut units of targets into work items (csrc/worklist.h), compiled
for the host: the items of any set of units stay within the bound that the work
list is sized with (a longer list would lose items), up to the largest pair work
that positions of 2^31 - 2 particles can have, where the step limit no longer
fits an int."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"

PROGRAM = r"""
#include <cstdio>
#include "worklist.h"
using namespace hsr;
// reads sets: number of units, then a count and a window each; writes the items,
// the constant part of their bound and the largest item's targets
int main() {
    long long units;
    while (std::scanf("%lld", &units) == 1) {
        int* c = new int[units];
        int* w = new int[units];
        unsigned long long pairs = 0;
        for (long long k = 0; k < units; ++k) {
            if (std::scanf("%d %d", &c[k], &w[k]) != 2) return 1;
            pairs += (unsigned long long)c[k] * (unsigned long long)w[k];
        }
        const int limit = item_limit(pairs);
        long long items = 0, targets = 0;
        int largest = 0;
        for (long long k = 0; k < units; ++k) {
            const int T = item_size(w[k], limit);
            const Pieces s = pieces_of(c[k], T);
            items += s.items();
            targets += (long long)s.full * s.T + s.p + s.q - c[k];
            if (T > largest) largest = T;
        }
        std::printf("%lld %d %lld %d\n", items, kMaxSplitItems, targets, largest);
        delete[] c;
        delete[] w;
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("items")
    src, exe = d / "items.hip", d / "items"
    src.write_text(PROGRAM)
    subprocess.check_call([HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-w",
                           "-I", os.path.join(ROOT, "paper_1211_4864_amd", "csrc"),
                           "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)])
    return str(exe)


def _sets():
    big = 2 ** 31 - 2
    yield [(1, 1)]
    yield [(big, big)]                                     # one cell holds all
    yield [(big // 27, big)] * 27                          # the smallest periodic box
    yield [(big // 8, 2 ** 29)] * 8
    yield [(300_000_000, 300_000_000), (64, 300_000_064)]
    yield [(2 ** 26, 2 ** 30 + 1)] * 4
    yield [(5, 2 ** 28)] * 1000
    rng = np.random.default_rng(1)
    for _ in range(60):
        units = int(10 ** rng.uniform(0, 3.5))
        top = rng.uniform(0, 9 - np.log10(units) * 0.9)
        c = np.maximum(1, 10 ** rng.uniform(0, max(top, 0.1), units)).astype(np.int64)
        w = np.minimum(c * rng.integers(1, 28, units), big)
        yield list(zip(c.tolist(), w.tolist()))


def test_items_stay_within_the_bound(program):
    sets = list(_sets())
    text = "\n".join(f"{len(s)}\n" + "\n".join(f"{c} {w}" for c, w in s) for s in sets)
    out = subprocess.run([program], input=text, capture_output=True, text=True, check=True)
    lines = out.stdout.split("\n")[:-1]
    assert len(lines) == len(sets)
    for s, line in zip(sets, lines):
        items, split, lost, largest = map(int, line.split())
        n = sum(c for c, _ in s)
        assert lost == 0
        assert items <= min(n, 2 * len(s) + n // 64 + 1 + split), (len(s), n, items)
        assert 1 <= largest <= 64
