"""The counting sort of small sets (csrc/bin.hip): cell_start, the permutation
and the records are bitwise those of the reference layout (oracle/binning.py),
as the radix sort of larger sets leaves them: sub-cell code, then input index
inside a cell.  Sizes at the edges of a wave and of a block, and on both sides
of the two sorts' border; buckets of whole cells, of 2^3 and of 4^3 sub-cells;
buckets longer than a wave, coincident particles; positions outside the box and
non-finite ones."""
import numpy as np
import pytest
import torch

import paper_1211_4864_amd as hsr
from oracle import binning

pytestmark = pytest.mark.gpu


def _check(cuda, pos, box, r_cut, seed):
    n = pos.shape[0]
    mass = np.random.default_rng(seed).random(n).astype(np.float32)
    cs, perm, rec = hsr.bin(torch.from_numpy(pos).to(cuda), torch.from_numpy(mass).to(cuda),
                            box, r_cut)
    torch.cuda.synchronize()
    _, perm_r, cs_r, rec_r = binning.chaining_mesh(pos, mass, box, r_cut)
    assert np.array_equal(cs.cpu().numpy(), cs_r)
    assert np.array_equal(perm.cpu().numpy(), perm_r)
    assert np.array_equal(rec.cpu().numpy(), rec_r, equal_nan=True)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 257, 4097, (1 << 19) - 1, 1 << 19,
                               (1 << 19) + 1])
@pytest.mark.parametrize("cells", [3, 9, 60])
def test_uniform_sizes(cuda, n, cells):
    pos = np.random.default_rng(n + cells).random((n, 3))
    _check(cuda, pos, 1.0, float(np.float32(0.999 / cells)), n)


@pytest.mark.parametrize("box", [1.0, -1.0])
def test_long_buckets_and_odd_positions(cuda, box):
    rng = np.random.default_rng(5)
    clump = 0.42 + 1e-3 * rng.random((5000, 3))
    same = np.tile([[0.77, 0.1, 0.3]], (700, 1))
    far = rng.random((300, 3)) * 4.0 - 1.5
    odd = rng.random((5, 3))
    odd[0, 0], odd[1, 1], odd[2, 2] = np.nan, np.nan, np.nan
    pos = np.concatenate([clump, same, far, odd, rng.random((2000, 3))])
    pos = pos[rng.permutation(pos.shape[0])]
    for cells in (3, 8, 40):
        _check(cuda, pos, box, float(np.float32(0.999 / cells)), cells)
