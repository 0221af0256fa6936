"""ffs_ga.narrow_lds reports the decoder of 16-bit ready times: 1 for job-priority vectors under the
default rules on at most 32768 slots, with off-chip redos in the wide layout over the same LDS; 0
for a decode rule, for more slots and for X/Y chromosomes. Whole state against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1903_10741_amd import workloads as W
from test_gpu_decode import _ffs, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,slots,narrow", [("job", 256, 1), ("job", 32768, 1), ("job", 32832, 0),
                                               ("fifo", 256, 0), ("power", 32768, 0), ("xy", 256, 0)])
def test_narrow_layout(kind, slots, narrow):
    torch, ffsga = _ffs()
    _say("narrow layout:", kind, "slots", slots)
    inst = W.random_instance(71, n_jobs=60, n_stages=4, machines=[2, 3, 1, 2], p_max=400, percent=50)
    inst.decode_rules = {"fifo": 1, "power": 2}.get(kind, 0)
    gp = W.GaParams(2, 5, 8, mig_interval=2, mig_k=1, encoding=int(kind == "xy"))
    d = ffsga.DeviceInstance.from_host(inst)
    assert d.horizon > 32832
    ga = ffsga.GA(d, ffsga.GaConfig.of(gp, lds_slots=slots), 5, 0, 0)
    ga.step(3)
    ga.status()
    assert int(ga.ga.lds_slots) == slots and int(ga.ga.narrow_lds) == narrow
    assert kind == "xy" or (ga.overflows() > 0) == (slots == 256)
    st = oracle.ga_run(inst, gp, 5, 0, 0, 3, n_threads=8)
    for k in ("prio", "obj", "elite", "elite_obj"):
        assert (ga.view()[k].cpu().numpy() == np.asarray(st[k])).all(), k
