"""FFS_LDS_AUTO where generation 0 is decoded in two parts or in one: on either side of 16 waves a
compute unit (256 units), with sizing slots that leave a unit fewer than 16 waves and with slots
that leave it all; state, work and a generation against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1903_10741_amd import workloads as W
from test_gpu_decode import _ffs, _say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p_max", [150, 20])  # horizons of 10812 and 1499 slots
@pytest.mark.parametrize("rules", [0, 1])
@pytest.mark.parametrize("pop", [4096, 4097, 4609])
def test_auto_slots_in_one_part_or_two(pop, rules, p_max):
    torch, ffsga = _ffs()
    _say("auto slots, pop", pop, "rules", rules, "p_max", p_max)
    inst = W.random_instance(37, n_jobs=40, n_stages=3, machines=[2, 2, 1], p_max=p_max, percent=60)
    inst.decode_rules = rules
    gp = W.GaParams(1, 1, pop, mig_interval=0, mig_k=0)
    ga = ffsga.GA(ffsga.DeviceInstance.from_host(inst),
                  ffsga.GaConfig.of(gp, lds_slots=ffsga.FFS_LDS_AUTO), 5, 0, 0)
    st = oracle.ga_init(inst, gp, 5, 0, 0, n_threads=8)
    assert (ga.view()["obj"].cpu().numpy() == st["obj"]).all()
    work = oracle.decode_pop(inst, st["prio"], n_threads=8, want_work=True)[1]
    assert int(ga.view()["work"].item()) == int(work.sum())
    ga.step(1)
    ga.status()
    st = oracle.ga_run(inst, gp, 5, 0, 0, 1, n_threads=8)
    for k in ("prio", "obj", "elite", "elite_obj"):
        assert (ga.view()[k].cpu().numpy() == np.asarray(st[k])).all(), k
