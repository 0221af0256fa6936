"""Stages of few jobs, on few and on many machines, under a peak that lets two or three ops run at
once: their first ops are pushed past the stage before, by a walk over rows or by the search, on
either side of where the decoder changes from one to the other. Plans, work and objectives against
the oracle at the slots that hold every schedule and 64 fewer."""
import numpy as np
import pytest

import oracle
from paper_1903_10741_amd import workloads as W
from test_gpu_decode import _compare, _say
from test_gpu_decode_slots import _instance

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("machines", [[2, 3, 2], [6, 7, 6], [8, 8], [16, 12, 16]])
@pytest.mark.parametrize("jobs", [1, 7, 16, 17, 24, 25, 28, 29, 32, 33])
def test_short_stages(jobs, machines):
    _say("short stages:", jobs, machines)
    inst = _instance(jobs, machines, [12, 33, 47, 64], [3, 4], 10, 61)
    pop = W.random_population(67, 8, inst.n_active)
    span = 0
    for prio in pop:
        _, s, m, _ = oracle.decode(inst, prio, want_schedule=True)
        j, g = np.indices(s.shape)
        span = max(span, int((s + np.asarray(inst.proc)[j, g, m]).max()))
    full = -(-span // 64) * 64
    for slots in (0, full, max(full - 64, 64)):
        _compare(inst, pop, lds_slots=slots)
