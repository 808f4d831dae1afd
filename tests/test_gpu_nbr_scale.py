"""Neighbour search of FP32 trees over the range of FP32 coordinates: the wave's FP32 filter has to
pass every pair that the FP64 test accepts, also where FP32 squares overflow.  Counts, ordered hashes
and lists bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from tests.util import tree_cases

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bh():
    import paper_1112_4539_amd as bh
    bh.load()
    assert torch.cuda.is_available()
    return bh


# radius 0.4 times 2^k: the filter's bound turns to +inf between k = 51 and 52, squares overflow from
# distances of 2^64 on, differences at k = 128 (coordinates within 2^127 of zero)
@pytest.mark.parametrize("k", [-60, -49, -48, 51, 52, 63, 64, 65, 66, 70, 100, 128])
@pytest.mark.parametrize("name", ["random1000", "duplicates"])
def test_neighbours_fp32_scales(bh, name, k):
    print(f"[nbr scale] {name} times 2^{k}", flush=True)
    radius = 0.4 * 2.0 ** k
    pos = ((tree_cases()[name] - 0.5) * 2.0 ** k).astype(np.float32)
    assert np.all(np.isfinite(pos))
    mass = np.ones(len(pos), np.float32)
    T = bh.Tree(torch.tensor(pos, device="cuda"), torch.tensor(mass, device="cuda"))
    out = T.neighbours(radius, maxlen=len(pos), density=False)
    w = oracle.Tree(pos.astype(np.float64), mass.astype(np.float64)).neighbours(radius, maxlen=len(pos))
    assert 0 < w["count"].sum() < len(pos) * (len(pos) - 1)
    np.testing.assert_array_equal(out["count"].cpu().numpy(), w["count"])
    np.testing.assert_array_equal(out["hash"].cpu().numpy().view(np.uint64), w["hash"])
    np.testing.assert_array_equal(out["lists"].cpu().numpy(), w["lists"])
