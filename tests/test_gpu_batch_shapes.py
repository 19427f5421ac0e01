"""The batch tuner's tile shapes: each launch of a batched cycle keeps its own,
and none of them changes an iterate."""
import pytest
import torch

from paper_1803_02481_amd import hipbmg as HB
from paper_1803_02481_amd import inputs
from oracle import oracle as O

pytestmark = pytest.mark.gpu


def batch_case(sizes, npt):
    planes = [torch.as_tensor(O.fv5(inputs.cells_lognormal(nx, ny, 1.0, seed=300 + k))) for k, (nx, ny) in
              enumerate(sizes)]
    if npt == 9:
        planes = [torch.cat([p, torch.zeros((2,) + tuple(p.shape[1:]), dtype=p.dtype)]) for p in planes]
    bs = [torch.as_tensor(inputs.load_uniform(nx, ny, seed=400 + k)) for k, (nx, ny) in enumerate(sizes)]
    return [p.cuda().contiguous() for p in planes], [b.cuda().contiguous() for b in bs]


@pytest.mark.parametrize("npt,precision,pipelined", [(5, "fp64", True), (5, "mixed", True), (5, "fp64", False),
                                                     (9, "fp64", False), (9, "mixed", False)])
def test_shape_of_each_launch_does_not_change_the_iterate(npt, precision, pipelined, monkeypatch):
    monkeypatch.delenv("HIPBMG_BATCH_WPG", raising=False)
    monkeypatch.delenv("HIPBMG_RB", raising=False)
    if pipelined:
        monkeypatch.delenv("HIPBMG_NO_FUSE3", raising=False)
    else:
        monkeypatch.setenv("HIPBMG_NO_FUSE3", "1")
    # one strip and several, even and odd row-pair counts, a thin grid
    sizes = [(257, 257), (131, 97), (513, 65), (9, 301), (129, 257), (67, 65)]
    planes, bs = batch_case(sizes, npt)
    prec = HB.FP64 if precision == "fp64" else HB.MIXED
    runs = []
    # the third batch takes the shapes that the second one left in the cache
    for tune in ("0", "1", "1"):
        monkeypatch.setenv("HIPBMG_BATCH_TUNE", tune)
        bh = HB.BatchHierarchy(planes, precision=prec, collapse_level=1, max_cycles=5)
        us, infos = bh.solve(bs, tol=1e-30, check=False)
        runs.append((us, [i.cycles for i in infos]))
        if tune == "0":
            assert bh.tile_shape(0, 3)[:2] == (1, 0)
        bh.close()
    for us, cyc in runs[1:]:
        assert cyc == runs[0][1]
        for k in range(len(sizes)):
            assert torch.equal(us[k], runs[0][0][k]), (sizes[k], k)
