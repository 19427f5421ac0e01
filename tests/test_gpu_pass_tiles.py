"""The pipelined finest pass of a small grid as tiles against the streaming pass
of the same grid (HIPBMG_RB_FUSED3 forces it): every vertex is updated by the
same expressions from the same values, so the iterates are the same bits; the
norm's partial sums are in another order (n eps relative: 1e-12)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_1803_02481_amd import hipbmg as HB
from paper_1803_02481_amd import inputs

pytestmark = pytest.mark.gpu


def g(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


# (ny, nx): one pair of coarse vertices; a strip of exactly 54 column pairs, one
# pair less and one more; row blocks of exactly 4 and 8 steps, one less and one more;
# three strips; a thin grid each way; just within the limits of FP64 and FP32
@pytest.mark.parametrize("shape", [(5, 5), (17, 107), (15, 105), (19, 109), (33, 33), (65, 325), (9, 1025),
                                   (513, 5), (609, 641), (993, 1025)])
@pytest.mark.parametrize("precision,reaction,rescorr", [("fp64", False, 1), ("fp64", True, 1), ("fp64", False, 0),
                                                        ("mixed", False, 1), ("mixed", True, 0)])
def test_tiles_equal_streaming_pass(shape, precision, reaction, rescorr, monkeypatch):
    ny, nx = shape
    planes = np.array(O.fv5(inputs.cells_log10_blocks(nx, ny, 4, seed=51)))
    if reaction:   # the diagonal is not the sum of the connections
        planes[0, 1:-1, 1:-1] *= 1.0 + 1e-3 * np.random.default_rng(5).random((ny - 2, nx - 2))
    planes, b = g(planes), g(inputs.load_uniform(nx, ny, seed=52))
    runs = []
    for env in ({"HIPBMG_RB_FUSED3": "5"}, {}):
        monkeypatch.delenv("HIPBMG_RB_FUSED3", raising=False)
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        h = HB.Hierarchy(planes, precision=HB.FP64 if precision == "fp64" else HB.MIXED, max_cycles=4,
                         residual_correction=rescorr, collapse_level=0)
        u, info = h.solve(b, tol=1e-30, check=False)
        runs.append((u, info.cycles, np.array(info.history()), info.rb_pipelined))
        h.close()
    (u0, c0, h0, r0), (u1, c1, h1, r1) = runs
    assert r0 == 5
    assert r1 in (4, 8) if nx * ny <= (3 << 17 if precision == "fp64" else 1 << 20) else r1 > 0
    assert c1 == c0
    assert torch.equal(u1, u0)
    assert np.all(np.abs(h1 - h0) <= 1e-12 * np.abs(h0))
