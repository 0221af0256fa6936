"""Islands on either side of the size from which a block, not a wave, replaces them, and the
classical GA's running fitness sums around its rows of 64, against the CPU oracle (exact)."""
import numpy as np
import pytest

import oracle
from paper_1903_10741_amd import workloads as W
from test_gpu_decode import _ffs, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", [0, 1, 2])
@pytest.mark.parametrize("rows,cols", [(1, 1), (5, 13), (11, 93), (32, 32), (5, 205), (3, 700)])
def test_one_large_island(scheme, rows, cols):
    torch, ffsga = _ffs()
    _say("one island of", rows, "x", cols, "scheme", scheme)
    inst = W.random_instance(3, n_jobs=9, n_stages=2, machines=2, p_max=9, percent=70)
    gp = W.GaParams(1, rows, cols, mig_interval=0, mig_k=0)
    ga = ffsga.GA(ffsga.DeviceInstance.from_host(inst), ffsga.GaConfig.of(gp, scheme=scheme), 5, 0, 0)
    ga.step(3)
    ga.status()
    st = (oracle.ga_run(inst, gp, 5, 0, 0, 3, n_threads=8) if scheme == 0 else
          oracle.ga_run_scheme(inst, gp, scheme, 5, 0, 0, 3, n_threads=8))
    for k in ("prio", "obj", "elite", "elite_obj"):
        assert (ga.view()[k].cpu().numpy() == np.asarray(st[k])).all(), k
