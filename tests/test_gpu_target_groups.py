"""Training targets of groups on either side of the entries whose logarithms are kept on chip
(7456), and of a group that takes each run of the fixed sums past one entry, against the oracle."""
import numpy as np
import pytest

from oracle import surrogate as S
from paper_1903_10741_amd import workloads as W
from test_gpu_surrogate import _ffs, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,group", [(7455, 7455), (7456, 7456), (7457, 7457), (15000, 7456),
                                         (15000, 7500), (5000, 5000)])
def test_target_groups(count, group):
    torch, ffsga = _ffs()
    _say("targets of", count, "in groups of", group)
    obj = np.random.default_rng(count).integers(1, 10**6, size=count).astype(np.int64)
    got = ffsga.Surrogate(W.surrogate_init(0)).targets(torch.from_numpy(obj), group)
    want = S.targets(obj, group)
    assert (np.abs(got.cpu().numpy().astype(np.float64) - want) <= S.U32 * np.abs(want) + 1e-9).all()
