"""Workspaces smaller than hacc_sr_workspace_bytes: the counters of the finer
sub-cells may be left out (csrc/api.hip, layout_in), the results stay the same
to the bit; below that the calls are refused before any GPU work.  A buffer of
the size that the library would need without those counters, and with its lists
and the sort's buffers side by side, serves."""
import ctypes

import numpy as np
import pytest
import torch

import paper_1211_4864_amd as hsr
from paper_1211_4864_amd import _lib
from workloads import cotangent, fit_fgrid

pytestmark = pytest.mark.gpu
ENOSPACE = -3


def _align(v):
    return (v + 255) // 256 * 256


def _without_sub_cells(n, cells):
    """Size of the layout whose sort counts cells only: keys, indices and their
    sorted copies, radix histograms, records twice, two item lists and their
    buckets, four tables over the cells, two over the columns."""
    ncell = cells ** 3
    items = 2 * min(n, ncell) + n // 64 + 1
    cb = max(ncell - 1, 0).bit_length()
    bits = cb + (6 if cb + 6 <= 31 else 3 if cb + 3 <= 31 else 0)
    db = min(11, max(8, (bits + 2) // 3))
    hist = (1 << db) * ((n + 4095) // 4096)
    scan = (max(hist, ncell + 1) + 4095) // 4096 + 1
    parts = [4 * n] * 4 + [4 * (ncell + 1), 4 * hist, 4 * scan, 16 * n, 16 * n, 4 * (ncell + 1),
                           16 * items, 16 * items, 4 * items, 4 * (2 * 1024 + 17), 4 * ncell,
                           8 * cells ** 2, 4 * cells ** 2]
    return sum(_align(p) for p in parts) + 256


def _call(lib, dev, fn, size, *args):
    ws = torch.empty(size, dtype=torch.uint8, device=dev) if size else None
    _lib.check(lib.hacc_sr_set_stream(ctypes.c_void_p(torch.cuda.current_stream(dev).cuda_stream)))
    _lib.check(lib.hacc_sr_set_workspace(ctypes.c_void_p(ws.data_ptr() if size else 0), size))
    rc = getattr(lib, fn)(*args)
    torch.cuda.synchronize()
    _lib.check(lib.hacc_sr_set_workspace(None, 0))
    return rc


def _ptr(t):
    return ctypes.c_void_p(t.data_ptr())


@pytest.mark.parametrize("n,cells", [(20000, 8), (65536, 16), (93750, 18), (1 << 19, 32),
                                     (40000, 30), (1000, 4), ((1 << 19) + 1, 40)])
def test_smaller_workspace(cuda, n, cells):
    lib = hsr.load()
    box = -1.0
    r_cut = float(np.float32(0.9999 / cells))
    fit = fit_fgrid(r_cut / 3, 3.0, 0.164)
    rng = np.random.default_rng(n)
    pos = rng.random((n, 3))
    pos[: n // 8] = 0.5 + 0.2 / cells * rng.random((n // 8, 3))
    p = torch.from_numpy(pos).to(cuda)
    m = torch.from_numpy(rng.random(n).astype(np.float32)).to(cuda)
    g = torch.from_numpy(cotangent(n, 3)).to(cuda)
    poly = _lib.poly_array(fit.coeffs)
    sr = (n, box, ctypes.c_float(r_cut), ctypes.c_float(fit.eps), poly)
    usual = hsr.workspace_bytes(n, box, r_cut)
    small = min(usual, _without_sub_cells(n, cells))
    out = []
    for size in (usual, small):
        cs = torch.full((cells ** 3 + 1,), -1, dtype=torch.int32, device=cuda)
        perm = torch.full((n,), -1, dtype=torch.int32, device=cuda)
        rec = torch.full((n, 4), float("nan"), dtype=torch.float32, device=cuda)
        acc = torch.full((n, 3), float("nan"), dtype=torch.float32, device=cuda)
        grad = torch.full((n, 3), float("nan"), dtype=torch.float64, device=cuda)
        assert _call(lib, cuda, "hacc_sr_bin", size, _ptr(p), _ptr(m), n, box,
                     ctypes.c_float(r_cut), _ptr(cs), _ptr(perm), _ptr(rec)) == 0
        assert _call(lib, cuda, "hacc_sr_force", size, _ptr(p), _ptr(m), *sr, _ptr(acc)) == 0
        assert _call(lib, cuda, "hacc_sr_force_vjp", size, _ptr(p), _ptr(m), *sr, _ptr(g),
                     _ptr(grad)) == 0
        out.append((cs, perm, rec, acc, grad))
    for a, b in zip(*out):
        assert torch.equal(a, b)
    assert _call(lib, cuda, "hacc_sr_force", small // 2, _ptr(p), _ptr(m), *sr,
                 _ptr(acc)) == ENOSPACE


@pytest.mark.parametrize("ng,n", [(8, 16), (8, 5000), (16, 140000), (64, 300000)])
def test_pm_workspace(cuda, ng, n):
    """Two grids, tables over an axis, one word for the largest mass, keys and
    indices twice, two records, histograms and their block sums."""
    passes = (3 * (ng.bit_length() - 4) + 8) // 9
    db = max(8, -(-3 * (ng.bit_length() - 4) // passes)) if passes else 8
    hist = (1 << db) * ((n + 4095) // 4096)
    parts = [8 * ng ** 3] * 2 + [8 * ng, 16 * ng, 4] + [4 * n] * 4 + [16 * n] * 2 + [
        4 * hist, 4 * ((hist + 4095) // 4096 + 1)]
    size = sum(_align(p) for p in parts) + 256
    lib = hsr.load()
    rng = np.random.default_rng(ng)
    p = torch.from_numpy(rng.random((n, 3))).to(cuda)
    m = torch.from_numpy(rng.random(n).astype(np.float32)).to(cuda)
    ref = hsr.pm_accel(p, m, 1.0, ng)
    out = torch.full((n, 3), float("nan"), dtype=torch.float32, device=cuda)
    assert _call(lib, cuda, "hacc_sr_pm_accel", size, _ptr(p), _ptr(m), n, 1.0, ng,
                 ctypes.c_float(0.8), 3, _ptr(out)) == 0
    assert torch.equal(ref, out)


def test_kept_binning_in_a_smaller_workspace(cuda):
    """The VJP on the force's own binning, whose work list lies where the sort's
    buffers were, in the usual workspace and in one without the finer counters."""
    lib = hsr.load()
    n, cells, box = 65536, 16, 1.0
    r_cut = float(np.float32(0.9999 / cells))
    fit = fit_fgrid(r_cut / 3, 3.0, 0.164)
    rng = np.random.default_rng(9)
    p = torch.from_numpy(rng.random((n, 3))).to(cuda)
    m = torch.from_numpy(rng.random(n).astype(np.float32)).to(cuda)
    g = torch.from_numpy(cotangent(n, 4)).to(cuda)
    sr = (n, box, ctypes.c_float(r_cut), ctypes.c_float(fit.eps), _lib.poly_array(fit.coeffs))
    ref = hsr.force_vjp(p, m, box, r_cut, fit.eps, fit.coeffs, g)
    for size in (hsr.workspace_bytes(n, box, r_cut), _without_sub_cells(n, cells)):
        ws = torch.empty(size, dtype=torch.uint8, device=cuda)
        stream = torch.cuda.current_stream(cuda).cuda_stream
        _lib.check(lib.hacc_sr_set_stream(ctypes.c_void_p(stream)))
        _lib.check(lib.hacc_sr_set_workspace(_ptr(ws), size))
        acc = torch.empty((n, 3), dtype=torch.float32, device=cuda)
        grad = torch.full((n, 3), float("nan"), dtype=torch.float64, device=cuda)
        assert lib.hacc_sr_force(_ptr(p), _ptr(m), *sr, _ptr(acc)) == 0
        token = ctypes.c_uint64(0)
        assert lib.hacc_sr_binning_token(ctypes.byref(token)) == 0 and token.value
        assert lib.hacc_sr_force_vjp_binned(token, *sr, _ptr(g), _ptr(grad)) == 0
        torch.cuda.synchronize()
        _lib.check(lib.hacc_sr_set_workspace(None, 0))
        assert torch.equal(grad, ref)
