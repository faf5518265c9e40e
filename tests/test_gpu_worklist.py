"""Work items split below 64 targets: where one unit's window exceeds the step
limit, its targets are cut into items of 32, 16, ... 1 targets with more lanes
per target (csrc/worklist.hip).  Force and VJP against the float64 oracle on
sets whose dense clump takes every item size, with the tolerances of the
force and VJP parity tests (1e-5 and 1e-4 of max(|x*|, 0.1 floor))."""
import numpy as np
import pytest
import torch

import oracle
import paper_1211_4864_amd as hsr
from workloads import cotangent, fit_fgrid

pytestmark = pytest.mark.gpu

FIT = fit_fgrid(1.0 / 24, 3.0, 1e-5 * 128.0 ** 2)


def _clump(n, clump, seed):
    """`clump` of n particles inside a ball of 0.4 cells, the rest uniform."""
    rng = np.random.default_rng(seed)
    d = rng.standard_normal((clump, 3))
    d *= (rng.random(clump) ** (1 / 3) * 0.4 / 24 / np.linalg.norm(d, axis=1))[:, None]
    pos = np.concatenate([0.53 + d, rng.random((n - clump, 3))])
    mass = ((rng.random(n) + 0.5) / n).astype(np.float32)
    p = rng.permutation(n)
    return pos[p], mass[p]


@pytest.mark.parametrize("n,clump", [
    (1, 0), (255, 254), (257, 257),     # at and around the smallest step limit
    (1030, 1030), (4100, 4099),         # items of 16 and of a few targets
    (9000, 6001),                       # odd remainders beside a sparse background
])
@pytest.mark.parametrize("box", [1.0, -1.0])
def test_split_items_match_oracle(cuda, n, clump, box):
    pos, mass = _clump(n, clump, 100 + n)
    g = cotangent(n, 7)
    p, m = torch.from_numpy(pos).to(cuda), torch.from_numpy(mass).to(cuda)
    acc = hsr.force(p, m, box, FIT.r_cut, FIT.eps, FIT.coeffs)
    grad = hsr.force_vjp(p, m, box, FIT.r_cut, FIT.eps, FIT.coeffs, torch.from_numpy(g).to(cuda))
    torch.cuda.synchronize()
    ref, an, _ = oracle.force(pos, mass, box, FIT.r_cut, FIT.eps, FIT.coeffs)
    err = oracle.rel_err_floored(acc.cpu().numpy(), ref, an).max()
    gref, bn, amb = oracle.force_vjp(pos, mass, box, FIT.r_cut, FIT.eps, FIT.coeffs,
                                     g.astype(np.float64), cut_band=1e-6)
    dev = np.linalg.norm(grad.cpu().numpy() - gref, axis=1)
    bound = 1e-4 * np.maximum(np.linalg.norm(gref, axis=1), 0.1 * bn) + amb
    print(f"n {n} clump {clump} box {box}: force {err:.2e}, vjp / bound "
          f"{np.max(dev / np.maximum(bound, 1e-300)):.2e}", flush=True)
    assert err <= 1e-5
    assert np.all(dev <= bound)


def test_list_modes_agree(cuda):
    """2^19 particles take the counting sort and one list of items, one more the
    radix sort and a list per XCD: a particle of zero mass that carries the set
    over the border leaves the others' force and VJP as they are, to the float32
    rounding of other groupings of the sums (the parity tests' tolerances)."""
    n = 1 << 19
    rng = np.random.default_rng(8)
    pos = np.concatenate([rng.random((n - 40000, 3)), 0.3 + 0.02 * rng.random((40000, 3)),
                          [[0.9, 0.9, 0.9]]])
    mass = np.full(n + 1, np.float32(1.0 / n))
    mass[n] = 0.0
    g = cotangent(n + 1, 9)
    g[n] = 0.0
    fit = fit_fgrid(1.0 / 80, 3.0, 1e-5 * 128.0 ** 2)
    p, m, gt = (torch.from_numpy(a).to(cuda) for a in (pos, mass, g))
    sr = (1.0, fit.r_cut, fit.eps, fit.coeffs)
    out = []
    for k in (n, n + 1):
        pk, mk, gk = p[:k].contiguous(), m[:k].contiguous(), gt[:k].contiguous()
        out.append((hsr.force(pk, mk, *sr)[:n].double(), hsr.force_vjp(pk, mk, *sr, gk)[:n]))
    for a, b, tol in zip(out[0], out[1], (1e-5, 1e-4)):
        scale = a.norm(dim=1).clamp(min=float(a.norm(dim=1).mean()) * 0.1)
        assert float(((a - b).norm(dim=1) / scale).max()) <= tol
