"""The radix path of the binning (sets beyond the counting sort's border,
csrc/bin.hip): cell_start written during the gather, bitwise against the
reference layout (oracle/binning.py), with long runs of empty cells before,
between and after the particles, a single occupied cell, and uniform sets at
digits of 8 and 9 bits."""
import numpy as np
import pytest
import torch

import paper_1211_4864_amd as hsr
from oracle import binning

pytestmark = pytest.mark.gpu
N0 = (1 << 19) + 1


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


@pytest.mark.parametrize("cells", [3, 20, 100])
def test_uniform(cuda, cells):
    _check(cuda, np.random.default_rng(cells).random((N0 + 77, 3)), 1.0,
           float(np.float32(0.999 / cells)))


@pytest.mark.parametrize("where", ["first", "middle", "last", "both ends"])
def test_empty_runs(cuda, where):
    rng = np.random.default_rng(3)
    lo = {"first": 0.0, "middle": 0.51, "last": 0.991, "both ends": 0.0}[where]
    pos = lo + 0.008 * rng.random((N0, 3))
    if where == "both ends":
        pos[::2] += 0.991
    _check(cuda, pos, -1.0, float(np.float32(0.999 / 100)))
