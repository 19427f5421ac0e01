"""Coefficients below the normal range of FP32: a mixed-precision hierarchy, whose
FP32 kernels divide by reciprocals that would overflow, solves in FP64, with the
FP64 hierarchy's bits."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1803_02481_amd import hipbmg as HB
from paper_1803_02481_amd import inputs

pytestmark = pytest.mark.gpu
SCALE = 2.0 ** -133   # connections around 1e-40


def g(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("shape", [(33, 33), (65, 257), (129, 97)])
def test_mixed_solves_tiny_coefficients(shape):
    ny, nx = shape
    planes, b = g(O.fv5(inputs.cells_lognormal(nx, ny, 1.0, seed=61))), g(inputs.load_uniform(nx, ny, seed=62))
    ref, iref = HB.Hierarchy(planes * SCALE).solve(b * SCALE, tol=1e-10)
    u, info = HB.Hierarchy(planes * SCALE, precision=HB.MIXED).solve(b * SCALE, tol=1e-10)
    assert info.relres <= 1e-10 and info.cycles == iref.cycles
    assert torch.equal(u, ref)
    # a normal FP32 range stays mixed
    v, vinfo = HB.Hierarchy(planes * 2.0 ** -60, precision=HB.MIXED).solve(b * 2.0 ** -60, tol=1e-10)
    assert vinfo.relres <= 1e-10 and vinfo.outer_steps < vinfo.cycles


def test_mixed_batch_with_a_tiny_problem():
    planes, bs = [], []
    for k, (nx, ny) in enumerate([(65, 65), (129, 33), (33, 97)]):
        f = SCALE if k == 1 else 1.0
        planes.append(g(O.fv5(inputs.cells_lognormal(nx, ny, 1.0, seed=63 + k)) * f))
        bs.append(g(inputs.load_uniform(nx, ny, seed=66 + k) * f))
    ref, _ = HB.BatchHierarchy(planes, precision=HB.FP64).solve(bs, tol=1e-10)
    us, infos = HB.BatchHierarchy(planes, precision=HB.MIXED).solve(bs, tol=1e-10)
    for u, r, i in zip(us, ref, infos):
        assert i.relres <= 1e-10 and torch.equal(u, r)
