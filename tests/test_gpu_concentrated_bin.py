"""Binning of concentrated sets (csrc/bin.hip): the counting sort's heavy buckets,
from 1024 entries on (2048 where a bucket is 64 sort keys, and 4160 in 2^19
particles), whose places come from counts per segment of the input.
cell_start, the permutation and the records bitwise against the reference layout
(oracle/binning.py): buckets at the border's both sides, in buckets of one sort
key, of 8 and of 64; keys met in one segment only and in all; last segments of
one particle; several heavy buckets beside light ones.  And the time: a set on
one point must not take the square of its size."""
import numpy as np
import pytest
import torch

import paper_1211_4864_amd as hsr
from oracle import binning

pytestmark = pytest.mark.gpu


def _check(cuda, pos, box, r_cut):
    n = pos.shape[0]
    mass = np.random.default_rng(n).random(n).astype(np.float32)
    cs, perm, rec = hsr.bin(torch.from_numpy(pos).to(cuda), torch.from_numpy(mass).to(cuda),
                            box, r_cut)
    torch.cuda.synchronize()
    _, perm_r, cs_r, rec_r = binning.chaining_mesh(pos, mass, box, r_cut)
    assert np.array_equal(cs.cpu().numpy(), cs_r)
    assert np.array_equal(perm.cpu().numpy(), perm_r)
    assert np.array_equal(rec.cpu().numpy(), rec_r)


# cells per axis at 20001 particles: buckets of one key, of 8 and of 64
@pytest.mark.parametrize("cells", [3, 15, 40])
@pytest.mark.parametrize("m", [1023, 1024, 1025, 2047, 2048, 2049, 12289])
@pytest.mark.parametrize("where", ["point", "cell", "first", "last"])
def test_border(cuda, cells, m, where):
    """m particles on one point or all over one cell, at random places of the
    input, or a point's all together at its beginning or end."""
    n = 20001
    rng = np.random.default_rng(m + cells)
    pos = rng.random((n, 3))
    inside = rng.random((m, 3)) * 0.98 + 0.01 if where == "cell" else np.full((m, 3), 0.3)
    at = {"first": np.arange(m), "last": np.arange(n - m, n)}.get(
        where, rng.choice(n, m, replace=False))
    pos[at] = (np.floor(0.6 * cells) + inside) / cells
    _check(cuda, pos, 1.0, float(np.float32(0.999 / cells)))


@pytest.mark.parametrize("m", [4159, 4160, 4161, 40000])
def test_border_of_the_largest_sets(cuda, m):
    """Buckets of 64 keys at 2^19 particles: segments of 16 blocks down to one."""
    n, cells = 1 << 19, 100
    rng = np.random.default_rng(m)
    pos = rng.random((n, 3))
    pos[rng.choice(n, m, replace=False)] = (60 + rng.random((m, 3)) * 0.98 + 0.01) / cells
    _check(cuda, pos, 1.0, float(np.float32(0.999 / cells)))


@pytest.mark.parametrize("n", [1023, 1024, 1025, 2047, 2048, 2049, 4097, (1 << 18) + 1, 1 << 19])
@pytest.mark.parametrize("cells", [3, 40, 100])
def test_all_on_one_point(cuda, n, cells):
    _check(cuda, np.tile([[0.437, 0.902, 0.011]], (n, 1)), 1.0, float(np.float32(0.999 / cells)))


@pytest.mark.parametrize("box", [1.0, -1.0])
@pytest.mark.parametrize("n,cells", [(70001, 3), (70001, 25), (70001, 60), (1 << 19, 100)])
def test_several_heavy_buckets(cuda, n, cells, box):
    """Four clumps inside single cells (one of them a point), a background."""
    rng = np.random.default_rng(cells)
    pos = rng.random((n, 3))
    who = rng.integers(0, 6, n)
    corner = np.floor(rng.random((4, 3)) * cells)
    for c in range(4):
        k = int((who == c).sum())
        u = rng.random((k, 3)) * 0.9 + 0.05 if c else np.full((k, 3), 0.5)
        pos[who == c] = (corner[c] + u) / cells
    _check(cuda, pos, box, float(np.float32(0.999 / cells)))


def _time(cuda, pos, box, r_cut):
    """Smallest time of a call over 5 runs of 4."""
    p = torch.from_numpy(pos).to(cuda)
    m = torch.ones(pos.shape[0], dtype=torch.float32, device=cuda)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = float("inf")
    for _ in range(5):
        torch.cuda.synchronize()
        a.record()
        for _ in range(4):
            hsr.bin(p, m, box, r_cut)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / 4)
    return best


@pytest.mark.parametrize("n", [1 << 16, 1 << 19])
@pytest.mark.parametrize("share", [1.0, 0.1])
def test_time_is_linear(cuda, n, share):
    """All particles or a tenth on one point: at most 4 times a uniform set's
    time (radix passes take 1.1 to 1.8 times; a place found by counting every
    entry of the bucket, and an add per particle on one counter, 5 to 290)."""
    rng = np.random.default_rng(11)
    pos = rng.random((n, 3))
    r_cut = float(np.float32(3.0 / 128))
    even = _time(cuda, pos, 1.0, r_cut)
    pos[rng.choice(n, int(share * n), replace=False)] = 0.437
    dense = _time(cuda, pos, 1.0, r_cut)
    print(f"n {n} share {share}: {even * 1e3:.0f} us, on one point {dense * 1e3:.0f} us", flush=True)
    assert dense <= 4.0 * even
