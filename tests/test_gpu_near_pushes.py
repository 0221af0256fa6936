"""On-chip decodes whose ops are pushed right by one to a few rows of 64 slots: no op fits where its
machine is free, two at most run at once, and windows of up to 64 slots end in the next row, in the
two after it and past those, up to the last slots. Plans, work and objectives against the oracle at
the slots that hold every schedule and 64 fewer."""
import numpy as np
import pytest

import oracle
from paper_1903_10741_amd import workloads as W
from test_gpu_decode import _compare, _say
from test_gpu_decode_slots import _instance

pytestmark = pytest.mark.gpu

CASES = {
    # jobs, machines, times, powers, peak
    "two at once, rows": (44, [3, 5], [20, 40, 60, 64], [3], 7),
    "two at once, one machine between": (60, [4, 1, 4], [33, 48, 63, 64], [4, 5], 10),
    "one at once, four machines": (30, [4, 4], [31, 32, 33], [6], 10),
    "one at once, sixteen machines": (40, [16, 9], [16, 17, 40], [6], 10),
    "uneven powers": (82, [3, 2, 3], list(range(10, 65)), [2, 9, 13], 20),
    "long and short": (60, [3, 2, 3], [5, 50, 64, 65, 100, 128, 129], [4, 11], 18),
    "peak of a byte": (40, [5, 4], [30, 64], [100, 155, 255], 255),
}


@pytest.mark.parametrize("name", CASES)
def test_near_pushes(name):
    _say("near pushes:", name)
    inst = _instance(*CASES[name], 47)
    pop = W.random_population(53, 20, inst.n_active)
    span = 0
    for prio in pop:
        _, s, m, _ = oracle.decode(inst, prio, want_schedule=True)
        j, g = np.indices(s.shape)
        span = max(span, int((s + np.asarray(inst.proc)[j, g, m]).max()))
    full = -(-span // 64) * 64
    for slots in (0, full, max(full - 64, 64), max(full - 192, 64)):
        _compare(inst, pop, lds_slots=slots)
