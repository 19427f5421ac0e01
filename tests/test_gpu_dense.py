"""The dense operator of the coarse levels (what a hierarchy with the default
collapse choice applies) against the collapsed workgroup of the same levels.

Both do the V-cycle of levels 0..top from zero, one as a product with a matrix
of n <= 2048 unknowns formed in FP64, one phase by phase.  A dot product of n
terms is off by at most n eps of its absolute sum; with the coarse operators'
absolute sums within about 1e2 of the result, 2048 * 1.1e-16 * 1e2 = 2.3e-11
per cycle bounds the FP64 difference after the three cycles compared, each of
which damps the earlier ones'.  FP32 cycles round the same coarse correction
to float (6e-8) and amplify it over three cycles by at most a few per cycle:
5e-6 relative to the largest value."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1803_02481_amd import hipbmg as HB
from paper_1803_02481_amd import inputs

pytestmark = pytest.mark.gpu


def g(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def dense_top(h):
    top = -1
    for l in range(h.L - 1):
        ny, nx = h.size(l)
        if (nx - 2) * (ny - 2) <= 2048:
            top = l
    return top


# (ny, nx) -> unknowns of the highest dense level: 1; 9; 225; 961; 128 (an
# exact row of the padded matrix); 361 above an even coarsest grid; 3 x 127;
# 1457 and 1833 (more than one row of loads); 1 x 31
@pytest.mark.parametrize("shape", [(5, 5), (9, 9), (33, 33), (129, 129), (19, 35), (41, 41), (9, 257), (65, 97),
                                   (161, 193), (5, 65)])
@pytest.mark.parametrize("prm", [{}, {"residual_correction": 0}, {"nu1": 3, "nu2": 2}])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_dense_operator_is_the_collapse(shape, prm, precision):
    ny, nx = shape
    planes = g(O.fv5(inputs.cells_log10_blocks(nx, ny, 4, seed=17)))
    prec = HB.FP64 if precision == "fp64" else HB.MIXED
    auto = HB.Hierarchy(planes, precision=prec, max_cycles=3, **prm)
    forced = HB.Hierarchy(planes, precision=prec, max_cycles=3, collapse_level=dense_top(auto), **prm)
    for seed in (3, 4):   # the second solve uses the operator the first one formed
        b = inputs.load_uniform(nx, ny, seed=seed)
        if precision == "fp64":
            u, v = (h.solve(g(b), tol=1e-30, check=False)[0] for h in (auto, forced))
            bound = 3e-11
        else:
            r = g(b.astype(np.float32))
            n = float(np.linalg.norm(b[1:-1, 1:-1]))
            u, v = (h.op32_inner(r, 3, n)[0] for h in (auto, forced))
            bound = 5e-6
        assert bool(torch.isfinite(u).all())
        assert float((u - v).abs().max()) <= bound * float(v.abs().max())


# the previous cycle's test rides along with the first coarse launch: the dense
# operator (35^2, 65^2), a tile kernel of four or eight waves (129^2, 513 x 257,
# 1025^2); 2049 x 257 has it in a launch of its own
@pytest.mark.parametrize("shape", [(35, 35), (65, 65), (129, 129), (257, 513), (1025, 1025), (257, 2049)])
@pytest.mark.parametrize("ahead", ["0", "2", "7"])
def test_stopping_cycle_is_the_capped_one(shape, ahead, monkeypatch):
    # a solve that meets its tolerance after k cycles returns the bits of one
    # capped at k, and its history, whatever ran after the test was met
    monkeypatch.setenv("HIPBMG_AHEAD", ahead)
    ny, nx = shape
    planes = HB.fv5_from_cells(g(inputs.cells_lognormal(nx, ny, 1.0, seed=5)))
    b = g(inputs.load_uniform(nx, ny, seed=6))
    h = HB.Hierarchy(planes)
    u, info = h.solve(b, tol=1e-8)
    again, _ = h.solve(b, tol=1e-8)
    assert torch.equal(u, again)
    capped = HB.Hierarchy(planes, max_cycles=info.cycles)
    v, capped_info = capped.solve(b, tol=1e-30, check=False)
    assert torch.equal(u, v)
    assert info.history() == capped_info.history() and info.cycles >= 3
    # a right-hand side of zeros and one that is not finite, between solves
    z, zi = h.solve(torch.zeros_like(b), u=torch.ones_like(b), tol=1e-8)
    assert zi.cycles == 0 and float(z.abs().max()) == 0.0
    bad = b.clone()
    bad[1, 1] = float("nan")
    with pytest.raises(HB.HipBMGError) as e:
        h.solve(bad, tol=1e-8)
    assert e.value.status == HB.ENAN
    after, _ = h.solve(b, tol=1e-8)
    assert torch.equal(u, after)


# the level below the finest: streaming with r/C stored (577 x 609), and with r/C
# formed by the up leg (1025^2)
@pytest.mark.parametrize("shape", [(1153, 1217), (2049, 2049)])
@pytest.mark.parametrize("reaction", [False, True])
def test_check_rides_a_streaming_leg(shape, reaction, monkeypatch):
    ny, nx = shape
    planes = HB.fv5_from_cells(g(inputs.cells_lognormal(nx, ny, 1.0, seed=15)))
    if reaction:   # no zero row sums: the coarse diagonals are loaded
        planes = planes.clone()
        planes[0, 1:-1, 1:-1] *= 1.0 + 1e-6
    b = g(inputs.load_uniform(nx, ny, seed=16))
    h = HB.Hierarchy(planes)
    u, info = h.solve(b, tol=1e-8)
    capped = HB.Hierarchy(planes, max_cycles=info.cycles)
    v, capped_info = capped.solve(b, tol=1e-30, check=False)
    assert torch.equal(u, v)
    assert info.history() == capped_info.history() and info.cycles >= 3
    # mixed precision: every refinement step's inner cycles end by such tests
    got = []
    for ahead in ("0", "2", "7"):
        monkeypatch.setenv("HIPBMG_AHEAD", ahead)
        m = HB.Hierarchy(planes, precision=HB.MIXED)
        w, minfo = m.solve(b, tol=1e-10)
        got.append((w, minfo.cycles, minfo.history(), minfo.relres))
        m.close()
    assert got[0][3] <= 1e-10
    for w, cyc, hist, _ in got[1:]:
        assert torch.equal(w, got[0][0]) and cyc == got[0][1] and hist == got[0][2]


def test_check_rides_a_leg_that_looks_again():
    # a level below the finest beyond 2^21 vertices: its tiles end early once the
    # test they carry is met
    ny, nx = 1025, 8321
    planes = HB.fv5_from_cells(g(inputs.cells_lognormal(nx, ny, 1.0, seed=17)))
    b = g(inputs.load_uniform(nx, ny, seed=18))
    for scale in (1.0, 1.0 + 1e-6):   # formed and loaded diagonals
        p = planes.clone()
        p[0, 1:-1, 1:-1] *= scale
        h = HB.Hierarchy(p)
        u, info = h.solve(b, tol=1e-8)
        again, _ = h.solve(b, tol=1e-8)
        v, capped = HB.Hierarchy(p, max_cycles=info.cycles).solve(b, tol=1e-30, check=False)
        assert torch.equal(u, v) and torch.equal(u, again)
        assert info.history() == capped.history() and info.cycles >= 3
