"""GAs at the default on-chip slots under each decode rule and with X/Y chromosomes: schedules of
5000 to 8000 slots, in a population that leaves each decode room for them, one that leaves room for
some of them and one that leaves none, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1903_10741_amd import workloads as W
from test_gpu_decode import _ffs, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["job", "fifo", "power", "both", "xy"])
@pytest.mark.parametrize("shape", [(3, 5, 7), (5, 29, 31), (7, 29, 31)])
def test_ga_default_slots(kind, shape):
    torch, ffsga = _ffs()
    _say("GA at the default slots,", kind, shape)
    inst = W.random_instance(29, n_jobs=50, n_stages=3, machines=[2, 2, 1], p_max=150, percent=60)
    inst.decode_rules = {"fifo": 1, "power": 2, "both": 3}.get(kind, 0)
    gp = W.GaParams(*shape, mig_interval=2, mig_k=2, encoding=int(kind == "xy"))
    ga = ffsga.GA(ffsga.DeviceInstance.from_host(inst), ffsga.GaConfig.of(gp), 5, 0, 0)
    if shape == (3, 5, 7):
        assert ga.ga.lds_slots > 8192 and ga.overflows() == 0
    ga.step(2)
    ga.status()
    st = oracle.ga_run(inst, gp, 5, 0, 0, 2, n_threads=8)
    for k in ("prio", "obj", "elite", "elite_obj"):
        assert (ga.view()[k].cpu().numpy() == np.asarray(st[k])).all(), k
