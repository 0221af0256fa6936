"""Each kernel holds the decoder of one set of decode rules: plans, work counts and GAs of every
scheme under each rule (and a rule bit that means nothing), on the slots where the default rules
change decoders (32768), far fewer (off-chip redos by the wave and by the overflow kernel) and the
default, at widths of 1 to 16 machines, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1903_10741_amd import workloads as W
from test_gpu_decode import _compare, _ffs, _say

pytestmark = pytest.mark.gpu

MACHINES = {4: [1, 3, 2, 4], 8: [5, 1, 8, 2], 16: [16, 9, 1, 12]}


def _inst(width, rules, n=70, p_max=120):
    inst = W.random_instance(61 + width, n_jobs=n, n_stages=4, machines=MACHINES[width], p_max=p_max,
                             percent=40)
    inst.decode_rules = rules
    return inst


@pytest.mark.parametrize("rules", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("width", [4, 8, 16])
def test_decode_forms(width, rules):
    inst = _inst(width, rules, p_max=400)  # a horizon beyond 32768 slots
    assert oracle.horizon_bound(inst) > 32832
    for slots in (0, 256, 32768, 32832):
        _say("forms: width", width, "rules", rules, "slots", slots)
        _compare(inst, W.random_population(width, 6, inst.n_active), lds_slots=slots)


@pytest.mark.parametrize("rules", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("scheme", [0, 1, 2])
def test_ga_forms(scheme, rules):
    torch, ffsga = _ffs()
    inst = _inst((4, 8, 16)[scheme], rules)
    gp = W.GaParams(1 if scheme else 3, 6, 7, mig_interval=0 if scheme else 2, mig_k=0 if scheme else 2)
    d = ffsga.DeviceInstance.from_host(inst)
    st = (oracle.ga_run(inst, gp, 5, 0, 0, 3, n_threads=8) if scheme == 0 else
          oracle.ga_run_scheme(inst, gp, scheme, 5, 0, 0, 3, n_threads=8))
    for slots in (0, 192) + ((ffsga.FFS_LDS_AUTO,) if scheme == 0 else ()):
        _say("forms: GA scheme", scheme, "rules", rules, "slots", slots)
        ga = ffsga.GA(d, ffsga.GaConfig.of(gp, lds_slots=slots, scheme=scheme), 5, 0, 0)
        ga.step(3)
        ga.status()
        assert slots != 192 or ga.overflows() > 0
        for k in ("prio", "obj", "elite", "elite_obj"):
            assert (ga.view()[k].cpu().numpy() == np.asarray(st[k])).all(), (slots, k)
