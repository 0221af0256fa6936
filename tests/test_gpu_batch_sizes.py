"""A batch whose largest size class lies just past the slots up to which the default rules have
their own decoder (32768), with a shop whose horizon keeps it on those slots and whose schedules
end in the last of them."""
import numpy as np
import pytest

import oracle
from paper_1903_10741_amd import workloads as W
from test_gpu_batch import GA, _ffs, _same, _say, _state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rules", [0, 1])
def test_batch_slot_below_its_class(rules):
    torch, ffsga = _ffs()
    _say("batch slot of 32768 slots in a class of 32832, rules", rules)
    # any two ops together break the peak, and an op takes as long on each of the 16 machines: a
    # schedule is the sum of all ops, one slot short of the horizon
    n = 150
    inst = W.random_instance(41, n_jobs=n, n_stages=2, machines=16, p_max=40)
    p = np.random.default_rng(43).integers(1, 41, size=(n, 2))
    p[:, 0] += (32767 - p.sum()) // n
    p[0, 0] += 32767 - p.sum()
    inst.proc = np.ascontiguousarray(np.broadcast_to(p[:, :, None], (n, 2, 16)), dtype=np.int32)
    inst.power = np.full((n, 2, 16), 6, np.int32)
    inst.q_max = 10
    inst.decode_rules = rules
    d = ffsga.DeviceInstance.from_host(inst)
    assert d.horizon == 32768
    b = ffsga.Batch(ffsga.BatchConfig(n_slots=1, max_jobs=n, max_genes=n, max_stages=2, o_max=16,
                                      max_horizon=40000, ga=ffsga.GaConfig.of(GA, lds_slots=32832),
                                      blocks=7))
    b.set(0, d, 3, 0, 0)
    b.step(2)
    b.status()
    _same(_state(b, 0), oracle.ga_run(inst, GA, 3, 0, 0, 2), f"rules {rules}")
