"""The PM solver's two ways through the particles (csrc/pm.hip): in input order
for small sets, sorted by tiles of 8^3 cells for larger ones.  Sets on both
sides of the border between them, at every number of radix passes (none at 8^3,
one, two), with tiles below and above the LDS thresholds, and a clump inside one
tile; against the float64 oracle with the bound of test_gpu_pm.py."""
import numpy as np
import pytest
import torch

from oracle import pm
import paper_1211_4864_amd as hsr
from workloads import plummer_clustered

pytestmark = pytest.mark.gpu
TOL = 1e-5


def _border(ng):
    return (1 << 17) + min(ng ** 3 // 64, 1 << 18)


def _solve(cuda, pos, mass, ng):
    out = hsr.pm_accel(torch.from_numpy(pos).to(cuda), torch.from_numpy(mass).to(cuda), 1.0, ng)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _check(cuda, pos, mass, ng):
    got = _solve(cuda, pos, mass, ng)
    ref = pm.accel(pos, mass.astype(np.float64), 1.0, ng)
    err = np.linalg.norm(got - ref, axis=1).max()
    rms = np.sqrt((np.linalg.norm(ref, axis=1) ** 2).mean())
    print(f"ng {ng} n {pos.shape[0]}: max |da| / rms|a| = {err / rms:.3e}", flush=True)
    assert err <= TOL * rms


@pytest.mark.parametrize("ng", [8, 16, 64, 128])
@pytest.mark.parametrize("over", [0, 1])
def test_border(cuda, ng, over):
    n = _border(ng) + over
    pos, _ = plummer_clustered(n, 60 + ng, 40, 0.5, 1.0 / max(ng, 32))
    mass = ((np.random.default_rng(61).random(n) + 0.5) / n).astype(np.float32)
    _check(cuda, pos, mass, ng)


@pytest.mark.parametrize("ng", [64, 256])
def test_sparse_and_dense_tiles(cuda, ng):
    """A clump inside one tile (many blocks of one tile), a line of coincident
    particles, positions outside the box, and a background whose tiles hold
    fewer particles than the LDS passes take."""
    rng = np.random.default_rng(62)
    n_back = _border(ng)
    clump = (np.array([8.5, 16.5, 24.5]) + 6.0 * rng.random((9000, 3))) / ng
    same = np.tile([[0.9999, 0.5, 0.25]], (700, 1))
    back = rng.random((n_back, 3)) * 1.5 - 0.25
    pos = np.concatenate([clump, same, back])[rng.permutation(n_back + 9700)]
    mass = np.full(pos.shape[0], np.float32(1.0 / pos.shape[0]))
    _check(cuda, pos, mass, ng)


def test_paths_agree(cuda):
    """Particles of zero mass that carry a set over the border change its way,
    not its density: the others' accelerations agree to the fixed point's and
    float32's rounding."""
    ng, n = 32, 1 << 16
    pos, _ = plummer_clustered(n, 63, 20, 0.6, 1.0 / ng)
    more = np.random.default_rng(64).random(((1 << 18) - n, 3))
    few = _solve(cuda, pos, np.full(n, np.float32(2.0 ** -16)), ng)
    mass = np.concatenate([np.full(n, 2.0 ** -16), np.zeros(len(more))]).astype(np.float32)
    many = _solve(cuda, np.concatenate([pos, more]), mass, ng)
    assert np.abs(many[:n] - few).max() <= 1e-6 * np.abs(few).max()
