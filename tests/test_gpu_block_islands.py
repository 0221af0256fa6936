"""Several islands of the size that a block, not a wave, replaces when they run on one stream, with
migration between them, on either side of that size, against the oracle; the same in island groups."""
import numpy as np
import pytest

import oracle
from paper_1903_10741_amd import workloads as W
from test_gpu_decode import _ffs, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("islands,rows,cols", [(2, 32, 32), (3, 33, 32), (3, 31, 33), (5, 8, 129)])
def test_islands_replaced_by_blocks(islands, rows, cols):
    torch, ffsga = _ffs()
    inst = W.random_instance(3, n_jobs=9, n_stages=2, machines=2, p_max=9, percent=70)
    gp = W.GaParams(islands, rows, cols, mig_interval=2, mig_k=3)
    d = ffsga.DeviceInstance.from_host(inst)
    st = oracle.ga_run(inst, gp, 5, 0, 0, 5, n_threads=8)
    for groups in (1, 0):
        _say(islands, "islands of", rows, "x", cols, "groups", groups)
        ffsga.set_island_groups(groups)
        try:
            ga = ffsga.GA(d, ffsga.GaConfig.of(gp), 5, 0, 0)
            ga.step(5)
            ga.status()
            assert (int(ga.ga.island_groups) == 1) == (groups == 1)
        finally:
            ffsga.set_island_groups(0)
        for k in ("prio", "obj", "elite", "elite_obj"):
            assert (ga.view()[k].cpu().numpy() == np.asarray(st[k])).all(), (groups, k)
