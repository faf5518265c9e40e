"""Binning by the radix passes at the widest digits: 220 cells per axis make keys
of 30 bits and digits of 10, 300 cells 31 and 11, whose scatter is a kernel of its
own (csrc/bin.hip).  Sets beyond the counting sort's border, bitwise against the
reference layout (oracle/binning.py): all over the mesh, and with half of them in
a clump, whose digits are mostly equal."""
import numpy as np
import pytest
import torch

import paper_1211_4864_amd as hsr
from oracle import binning

pytestmark = pytest.mark.gpu
N0 = (1 << 19) + 78


@pytest.mark.parametrize("cells", [220, 300])
@pytest.mark.parametrize("clump", [False, True])
def test_wide_digits(cuda, cells, clump):
    rng = np.random.default_rng(cells)
    pos = rng.random((N0, 3))
    if clump:
        pos[::2] = 0.61 + 0.01 * pos[::2]
    mass = rng.random(N0).astype(np.float32)
    r_cut = float(np.float32(0.9999 / cells))
    assert hsr.grid_dim(1.0, r_cut) == cells
    cs, perm, rec = hsr.bin(torch.from_numpy(pos).to(cuda), torch.from_numpy(mass).to(cuda),
                            1.0, r_cut)
    torch.cuda.synchronize()
    _, perm_r, cs_r, rec_r = binning.chaining_mesh(pos, mass, 1.0, r_cut)
    assert np.array_equal(cs.cpu().numpy(), cs_r)
    assert np.array_equal(perm.cpu().numpy(), perm_r)
    assert np.array_equal(rec.cpu().numpy(), rec_r)
