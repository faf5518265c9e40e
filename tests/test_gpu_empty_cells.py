"""cell_start of sets beyond the counting sort's border (csrc/bin.hip) where long
runs of cells are empty: whole runs of 4096 cells are written by waves of their
own, the rest by the entries around them.  Bitwise against the reference layout
(oracle/binning.py) with occupied cells at and beside multiples of 4096, in
meshes that are one or many such runs; and the time: a set in one corner of a
large mesh must not wait for one wave to write the others."""
import numpy as np
import pytest
import torch

import paper_1211_4864_amd as hsr
from oracle import binning

pytestmark = pytest.mark.gpu
N0 = (1 << 19) + 1


def _positions(occupied, cells, rng):
    c = np.asarray(occupied)[rng.integers(0, len(occupied), N0)]
    c[:len(occupied)] = occupied
    corner = np.stack([c // cells ** 2, c // cells % cells, c % cells], axis=1)
    return (corner + 0.02 + 0.96 * rng.random((N0, 3))) / cells


@pytest.mark.parametrize("cells,occupied", [
    (16, [0]), (16, [4095]), (16, [7, 4095]), (17, [0]), (17, [4096]), (17, [4912]),
    (100, [0]), (100, [999999]), (100, [4095]), (100, [4096]), (100, [4097]),
    (100, [8190, 8191]), (100, [4095, 8192]), (100, [4094, 8191]), (100, [4096, 12288]),
    (100, [3, 500000, 500001, 999998]), (100, [999423]), (100, [999424, 999999]),
    (100, list(range(0, 1000000, 4096))), (100, list(range(4095, 1000000, 8192))),
])
def test_runs(cuda, cells, occupied):
    pos = _positions(occupied, cells, np.random.default_rng(len(occupied)))
    mass = np.ones(N0, dtype=np.float32)
    r_cut = float(np.float32(0.9999 / cells))
    assert hsr.grid_dim(-1.0, r_cut) == cells
    cs, perm, rec = hsr.bin(torch.from_numpy(pos).to(cuda), torch.from_numpy(mass).to(cuda),
                            -1.0, r_cut)
    torch.cuda.synchronize()
    _, perm_r, cs_r, rec_r = binning.chaining_mesh(pos, mass, -1.0, r_cut)
    assert np.array_equal(cs.cpu().numpy(), cs_r)
    assert np.array_equal(perm.cpu().numpy(), perm_r)
    assert np.array_equal(rec.cpu().numpy(), rec_r)


@pytest.mark.parametrize("where", ["first", "last", "both"])
def test_time_of_a_corner(cuda, where):
    """In one or two corners of 400^3 cells: at most 4 times the time of a set
    all over it (the cells are read and written once either way; one wave per
    run takes 170 times as long)."""
    rng = np.random.default_rng(12)
    m = torch.ones(N0, dtype=torch.float32, device=cuda)
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def best(pos):
        p, least = torch.from_numpy(pos).to(cuda), float("inf")
        for _ in range(5):
            torch.cuda.synchronize()
            a.record()
            hsr.bin(p, m, -1.0, 0.0025)
            b.record()
            torch.cuda.synchronize()
            least = min(least, a.elapsed_time(b))
        return least
    assert hsr.grid_dim(-1.0, 0.0025) == 400
    pos = rng.random((N0, 3))
    even = best(pos)
    pos *= 0.01
    if where == "last":
        pos += 0.985
    if where == "both":
        pos[::2] += 0.985
    corner = best(pos)
    print(f"{where}: {even * 1e3:.0f} us, in a corner {corner * 1e3:.0f} us", flush=True)
    assert corner <= 4.0 * even
