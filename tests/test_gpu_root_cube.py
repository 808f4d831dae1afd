"""The launch that starts a build and takes its extremes, at the edges of its grid: the root cube and the
reported inputs, each with the element that decides at the first, a middle and the last place (exact)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bh():
    import paper_1112_4539_amd as bh
    bh.load()
    assert torch.cuda.is_available()
    return bh


# 4097 is the smallest tree of these launches; 1024 workgroups of 256 cover 262,144 particles in one turn
@pytest.mark.parametrize("n", [4097, 4352, 4353, 262143, 262144, 262145, 300001])
def test_root_cube_and_reports(bh, n):
    print(f"[root cube] n={n}", flush=True)
    base = torch.rand((n, 3), dtype=torch.float64, generator=torch.Generator().manual_seed(n))
    mass = torch.ones(n, dtype=torch.float64, device="cuda")
    off = torch.tensor([0, n], device="cuda")
    ws = None
    for i in (0, n // 2, n - 1):
        for axis, x in ((0, -2.5), (1, 3.5), (2, 7.25)):
            pos = base.clone()
            pos[i, axis] = x
            T = bh.Tree(pos.cuda(), mass, ws)
            ws = T.workspace
            T.check()                               # what the workspace held before is not reported again
            ext = pos.max(0).values - pos.min(0).values
            assert T.export()[0]["l"][0] == float(ext.max())
            for bad in (float("nan"), float("-inf")):
                p, m = pos.clone(), mass.clone()
                p[i, axis] = bad
                m[i] = bad
                with pytest.raises(ValueError):
                    bh.Tree(p.cuda(), mass, ws).check()
                with pytest.raises(ValueError):
                    bh.build_forest(pos.cuda(), m, off, None).check()
    bh.build_forest(base.cuda(), mass, off).check()
    with pytest.raises(ValueError):
        bh.build_forest(base.cuda(), mass, torch.tensor([0, n - 1], device="cuda")).check()
