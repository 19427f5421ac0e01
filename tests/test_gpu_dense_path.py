"""What a default hierarchy runs below its grid-wide kernels is the dense operator,
whatever the machine calibration makes of the alternatives."""
import ctypes
import os

import numpy as np
import pytest
import torch

from paper_1803_02481_amd import hipbmg as HB
from paper_1803_02481_amd import inputs

pytestmark = pytest.mark.gpu
N_BEFORE = 24   # doubles of the model's parameters ahead of its 2 x 8 + 2 x 8 stage terms


def g(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.fixture
def free_stages():
    """Agglomeration stages that cost next to nothing, for the time of a test."""
    HB.calibrate()
    HB.lib()
    f = ctypes.CDLL(os.path.join(os.path.dirname(HB.__file__), "libhipbmg.so"))._ZN4hbmg12model_paramsEv
    f.restype = ctypes.POINTER(ctypes.c_double)
    p = f()
    old = p[N_BEFORE: N_BEFORE + 32]
    for k in range(32):
        p[N_BEFORE + k] = 1e-9
    yield
    for k in range(32):
        p[N_BEFORE + k] = old[k]


@pytest.mark.parametrize("shape", [(257, 257), (513, 1025)])
def test_dense_operator_replaces_searched_stages(shape, free_stages):
    ny, nx = shape
    planes = HB.fv5_from_cells(g(inputs.cells_lognormal(nx, ny, 1.0, seed=41)))
    b = g(inputs.load_uniform(nx, ny, seed=42))
    h = HB.Hierarchy(planes)
    h.profile(True, levels=True)
    u, info = h.solve(b, tol=1e-9)
    lv = h.profile_levels(0)
    assert info.search_us < min(list(info.model_us)[: info.levels])   # the search did find stages cheaper
    assert info.cluster_stages == 0
    top = max(l for l in range(h.L - 1) if (h.size(l)[0] - 2) * (h.size(l)[1] - 2) <= 2048)
    assert [l for l in range(h.L) if lv[l][5]] == [top] and lv[top][5] == info.cycles


# info names what runs: the dense operator's levels, or none where the collapse is
# forced, in a batch and in 3D; and the model's time of it
@pytest.mark.parametrize("shape", [(5, 5), (65, 65), (161, 193), (1025, 1025)])
def test_info_names_the_configuration_in_use(shape):
    HB.calibrate()
    ny, nx = shape
    planes = HB.fv5_from_cells(g(inputs.cells_lognormal(nx, ny, 1.0, seed=43)))
    b = g(inputs.load_uniform(nx, ny, seed=44))
    for precision in (HB.FP64, HB.MIXED):
        h = HB.Hierarchy(planes, precision=precision)
        _, info = h.solve(b, tol=1e-9)
        sizes = [h.size(l) for l in range(h.L)]
        assert info.dense_levels == sum((m - 2) * (n - 2) <= 2048 for m, n in sizes[:-1])
        above = sum(h.model_levels()["grid_us"][info.dense_levels: h.L])
        assert above < info.path_us < above + 60.0   # the levels above, one product, the test
        forced = HB.Hierarchy(planes, precision=precision, collapse_level=info.dense_levels - 1)
        _, finfo = forced.solve(b, tol=1e-9)
        assert finfo.dense_levels == 0 and finfo.collapse_level == info.dense_levels - 1
    _, infos = HB.BatchHierarchy([planes, planes]).solve([b, b], tol=1e-9)
    assert all(i.dense_levels == 0 for i in infos)
