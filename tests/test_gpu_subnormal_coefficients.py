"""Coefficients whose reciprocals overflow: FP64 operators in the subnormal range
and FP32 copies with diagonals below theirs are stored scaled by a power of two.

A power of two commutes with every rounding away from the ends of the range, so
all results are the same bits as those of the same (already rounded) operator
scaled into the normal range, times the ratio of the scales."""
import numpy as np
import pytest
import torch

from paper_1803_02481_amd import hipbmg as HB
from paper_1803_02481_amd import inputs

pytestmark = pytest.mark.gpu
UP = 2.0 ** 515          # applied twice: 2^1030 itself is out of range


def g(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def planes2(nx, ny, medium, seed):
    """Planes around 2^-1030, with their subnormal rounding, and the same times 2^1030."""
    if medium == "blocks":   # normal and subnormal regions side by side
        cells = g(inputs.cells_log10_blocks(nx, ny, 8, -3.0, 3.0, seed=seed))
    else:
        cells = g(inputs.cells_lognormal(nx, ny, 1.0, seed=seed))
    p = HB.fv5_from_cells(cells)
    low = p / UP / UP
    return low, low * UP * UP


@pytest.mark.parametrize("shape", [(3, 3), (33, 33), (65, 257), (129, 97), (513, 385)])
@pytest.mark.parametrize("medium", ["lognormal", "blocks"])
@pytest.mark.parametrize("prm", [{}, {"collapse_level": 0}, {"nu1": 1, "nu2": 2}])
def test_fp64_solve(shape, medium, prm):
    ny, nx = shape
    if prm.get("collapse_level", -1) >= 0 and min(shape) <= 3:
        prm = {}
    low, ref = planes2(nx, ny, medium, 51)
    b = g(inputs.load_uniform(nx, ny, seed=52))
    v, vinfo = HB.Hierarchy(ref, **prm).solve(b, tol=1e-9)
    h = HB.Hierarchy(low, **prm)
    u, info = h.solve(b / UP, tol=1e-9)
    assert torch.equal(u / UP, v) and info.history() == vinfo.history()
    for l in range(h.L):
        assert bool(torch.isfinite(h.stencil(l)).all())
    assert torch.equal(h.stencil(h.L - 1)[:3, 1:-1, 1:-1], low[:, 1:-1, 1:-1])


def test_single_operations():
    nx = ny = 33
    low, ref = planes2(nx, ny, "lognormal", 53)
    b, x = g(inputs.load_uniform(nx, ny, seed=54)), g(np.random.default_rng(55).standard_normal((ny, nx)))
    a, c = HB.Hierarchy(low), HB.Hierarchy(ref)
    l = a.L - 1
    assert torch.equal(a.op_smooth(l, b / UP, x * UP, 2) / UP, c.op_smooth(l, b, x, 2))
    for p, q, s in zip(a.op_smooth_restrict(l, b / UP, x * UP, 2), c.op_smooth_restrict(l, b, x, 2), (UP, UP, 1 / UP)):
        assert torch.equal(p / s, q)


def test_batch_with_one_subnormal_problem():
    low, ref = planes2(65, 65, "lognormal", 56)
    other = HB.fv5_from_cells(g(inputs.cells_lognormal(33, 97, 1.0, seed=57)))
    b0, b1 = g(inputs.load_uniform(65, 65, seed=58)), g(inputs.load_uniform(33, 97, seed=59))
    for precision in (HB.FP64, HB.MIXED):   # the mixed batch runs in FP64
        us, infos = HB.BatchHierarchy([low, other], precision=precision).solve([b0 / UP, b1], tol=1e-9)
        vs, vinfos = HB.BatchHierarchy([ref, other]).solve([b0, b1], tol=1e-9)
        assert torch.equal(us[0] / UP, vs[0]) and torch.equal(us[1], vs[1])
        assert [i.cycles for i in infos] == [i.cycles for i in vinfos]


@pytest.mark.parametrize("shape", [(3, 3, 3), (17, 17, 17), (33, 17, 49), (65, 65, 65)])
@pytest.mark.parametrize("prm", [{}, {"collapse_level": 0}])
def test_3d(shape, prm):
    nz, ny, nx = shape
    p = HB.fv7_from_cells(g(inputs.cells3_lognormal(nx, ny, nz, sigma=1.0, seed=60)))
    low = p / UP / UP
    ref = low * UP * UP
    b = g(inputs.load3_uniform(nx, ny, nz, seed=61))
    x = g(np.random.default_rng(62).standard_normal(shape))
    c, a = HB.Hierarchy3(ref, **prm), HB.Hierarchy3(low, **prm)
    v, vinfo = c.solve(b, tol=1e-9)
    u, info = a.solve(b / UP, tol=1e-9)
    assert torch.equal(u / UP, v) and info.history() == vinfo.history()
    l = a.L - 1
    assert torch.equal(a.smooth(l, b / UP, x * UP, 2) / UP, c.smooth(l, b, x, 2))
    assert torch.equal(a.residual(l, b / UP, x * UP) * UP, c.residual(l, b, x))


@pytest.mark.parametrize("shape", [(33, 33), (65, 129)])
@pytest.mark.parametrize("k", [126, 134, 142])
def test_fp32_operations_on_levels_below_their_normal_range(shape, k):
    ny, nx = shape
    p = HB.fv5_from_cells(g(inputs.cells_lognormal(nx, ny, 1.0, seed=63)))
    s, sb = 2.0 ** -k, 2.0 ** -90          # the operator's and the right-hand side's factor
    b = g(inputs.load_uniform(nx, ny, seed=64)).float()
    x = g(np.random.default_rng(65).standard_normal((ny, nx))).float()
    a, c = HB.Hierarchy(p * s, precision=HB.MIXED), HB.Hierarchy(p, precision=HB.MIXED)
    t = 2.0 ** (k - 90)                    # what the iterates scale by
    l = a.L - 1
    assert torch.equal(a.op32_smooth(l, b * sb, x * t, 2) / t, c.op32_smooth(l, b, x, 2))
    for u, v, f in zip(a.op32_smooth_restrict(l, b * sb, x * t, 2), c.op32_smooth_restrict(l, b, x, 2), (t, t, sb)):
        assert torch.equal(u / f, v)
    n = float(b[1:-1, 1:-1].double().norm())
    e, hist = a.op32_inner(b * sb, 3, n * sb)
    r, rhist = c.op32_inner(b, 3, n)
    assert torch.equal(e / t, r) and list(hist) == list(rhist)
    st, ref = a.level32(l)[0], c.level32(l)[0]
    assert torch.equal(st, ref * s)
