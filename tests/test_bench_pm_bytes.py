"""The benchmark's bytes of a particle-mesh solve (bench.py, pm_bytes) follow the
path that the library takes: sets in input order have no sort, 256^3 has two
radix passes of which the first reads no index, 8^3 none."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


@pytest.mark.parametrize("n,ng,path,per", [
    (32768, 128, "input order", 68),
    ((1 << 17) + 8, 8, "input order", 68), ((1 << 17) + 9, 8, "0 radix passes", 132),
    (1 << 18, 32, "1 radix passes", 144), (1 << 18, 64, "1 radix passes", 144),
    (128 ** 3, 128, "2 radix passes", 164), (256 ** 3, 256, "2 radix passes", 164),
    (393216, 512, "input order", 68), (393217, 512, "2 radix passes", 164),
])
def test_bytes_of_a_solve(n, ng, path, per):
    got = bench.pm_bytes(n, ng)
    assert got["path"] == path and got["bytes_per_particle"] == per
    assert got["bytes"] == 144 * ng ** 3 + per * n


def test_the_rules_are_the_library_s():
    src = open(os.path.join(ROOT, "paper_1211_4864_amd", "csrc", "pm.hip")).read()
    assert "return n <= (1 << 17) + std::min<int64_t>((int64_t)ng * ng * ng / 64, 1 << 18);" in src
    assert "const int bits = 3 * (lg - kSideBits);" in src
    assert "*passes = (bits + 8) / 9;" in src and "constexpr int kSideBits = 3;" in src
