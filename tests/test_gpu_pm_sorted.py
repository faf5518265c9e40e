"""The particle-mesh solver on both sides of its size rule (csrc/pm.hip): sets in
input order and sets sorted by tiles of 8^3 cells.  The deposit sums in fixed
point, so that neither the input order nor the run changes a bit: a permuted
input gives the permuted output and a second call the first one's, with unequal
masses, whose order inside a tile the permutation really changes.  At 512^3 the
sort's keys take 27 bits and two passes of 9.  Where the float64 oracle
(oracle/pm.py) is asked, the bound is that of test_gpu_pm.py."""
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


def _set(ng, n, seed):
    pos, _ = plummer_clustered(n, seed, 40, 0.6, 1.0 / max(ng, 32))
    return pos, ((np.random.default_rng(seed).random(n) + 0.5) / n).astype(np.float32)


def _solve(cuda, pos, mass, ng):
    out = hsr.pm_accel(torch.from_numpy(pos).to(cuda), torch.from_numpy(mass).to(cuda), 1.0, ng)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _check(got, pos, mass, ng):
    ref = pm.accel(pos, mass.astype(np.float64), 1.0, ng)
    err = np.linalg.norm(got - ref, axis=1).max()
    rms = np.sqrt((np.linalg.norm(ref, axis=1) ** 2).mean())
    print(f"ng {ng} n {pos.shape[0]}: max |da| / rms|a| = {err / rms:.3e}", flush=True)
    assert err <= TOL * rms


@pytest.mark.parametrize("ng", [8, 16, 32, 64, 128, 256, 512])
@pytest.mark.parametrize("over", [0, 1])
def test_order_and_run_change_no_bit(cuda, ng, over):
    n = _border(ng) + over
    pos, mass = _set(ng, n, 70 + ng)
    perm = np.random.default_rng(71).permutation(n)
    a = _solve(cuda, pos, mass, ng)
    assert np.array_equal(a, _solve(cuda, pos, mass, ng))
    assert np.array_equal(a[perm], _solve(cuda, pos[perm], mass[perm], ng))


def test_shared_cells_sorted(cuda):
    """Runs of particles in one grid cell longer than a block's share, and exactly
    coincident particles, in a set that is sorted."""
    ng = 32
    rng = np.random.default_rng(72)
    lump = np.array([0.3, 0.6, 0.1]) + rng.random((5000, 3)) * 0.9 / ng
    same = np.tile([[0.71, 0.22, 0.93]], (3000, 1))
    pos = np.concatenate([lump, same, rng.random((_border(ng), 3))])
    mass = np.concatenate([np.full(5000, 2e-5), np.full(3000, 1e-5),
                           np.full(_border(ng), 3e-6)]).astype(np.float32)
    perm = rng.permutation(pos.shape[0])
    _check(_solve(cuda, pos[perm], mass[perm], ng), pos[perm], mass[perm], ng)


def test_largest_grid_sorted(cuda):
    ng = 512
    pos, mass = _set(ng, _border(ng) + 1, 73)
    _check(_solve(cuda, pos, mass, ng), pos, mass, ng)
