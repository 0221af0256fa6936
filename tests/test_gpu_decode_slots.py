"""The default-rules decoder on its on-chip profile (ffs_decode through the C ABI) where its
64-slot windows, its rows of 64 slots and its chunks of 16 ops end, against the CPU oracle.

Integer path: objectives, start times, machines and work counts are identical (zero tolerance).
"""
import numpy as np
import pytest

import oracle
from paper_1903_10741_amd import workloads as W
from test_gpu_decode import _compare, _ffs, _say

pytestmark = pytest.mark.gpu


def _instance(n, machines, times, powers, q_max, seed, running=(), fixed=()):
    """n jobs whose P and Q are drawn from `times` and `powers`."""
    rng = np.random.default_rng(seed)
    shape = (n, len(machines), max(machines))
    inst = W.initial_instance(rng.choice(times, size=shape), rng.choice(powers, size=shape),
                              np.zeros(n, np.int32), np.full(n, 50, np.int32), machines, q_max, 3)
    inst.running = np.asarray(running, np.int32).reshape(-1, 2)
    if len(fixed):
        inst.fixed = np.asarray(fixed, np.int32).reshape(-1, 3)
    return inst


CASES = {
    # windows of one row, one more, two rows and one more; 4, 8 and 16 lanes a stage
    "p 63-65": (40, [3, 2], [1, 63, 64, 65], [1, 4, 6], 9, [], []),
    "p 127-129": (30, [5, 8], [64, 127, 128, 129, 200], [2, 5], 9, [], []),
    "sixteen machines": (35, [16, 9, 1], [1, 2, 31, 32, 33, 64], [1, 3], 12, [], []),
    # every op draws the whole peak: pushed past all before it, further than the 15 rows
    # searched at once
    "whole peak": (120, [16], [50, 63, 64], [7], 7, [], []),
    "whole peak, long": (60, [4], [65, 128, 129], [7], 7, [], []),
    "byte peak": (33, [4, 4], [3, 40, 64, 65], [1, 100, 255], 255, [], []),
    "unit ops": (129, [4, 4, 4], [1], [1], 2, [], []),
    # ops that run at RS past the peak (a lowered peak): only later slots are free
    "over the peak": (20, [4, 3], [1, 20, 64, 90], [1, 4], 6, [(70, 5), (130, 4), (1, 1)], []),
    "kept ops": (20, [4, 3], [1, 20, 64, 90], [1, 4], 6, [(5, 2)],
                 [(10, 75, 6), (200, 328, 3), (331, 332, 6)]),
    **{f"n {n}": (n, [3, 2, 4, 1], list(range(1, 40)), [1, 3, 5], 8, [], [])
       for n in (1, 15, 16, 17, 64, 65)},
}


@pytest.mark.parametrize("name", CASES)
def test_decode_on_chip_edges(name):
    """At the default slots, and at the last multiple of 64 slots that holds every schedule and
    64 fewer, where the longest is redone off chip."""
    _say("on-chip decode edges:", name)
    inst = _instance(*CASES[name][:5], 41, *CASES[name][5:])
    pop = W.random_population(43, 24, inst.n_active)
    span = 0
    for prio in pop:
        _, s, m, _ = oracle.decode(inst, prio, want_schedule=True)
        j, g = np.indices(s.shape)
        span = max(span, int((s + np.asarray(inst.proc)[j, g, m]).max()))
    full = -(-span // 64) * 64
    for slots in sorted({0, full, max(full - 64, 64)}):
        _compare(inst, pop, lds_slots=slots, schedule=slots != full)


@pytest.mark.parametrize("kind,pop", [("job", 3), ("job", 700), ("job", 4200), ("fifo", 5), ("xy", 5)])
def test_decode_default_slots(kind, pop):
    """Schedules of 5000 to 8000 slots at the default slots, which grow with the LDS that a
    population leaves each decode: one population a compute unit holds alone, one of a few waves
    a unit and one of more than the chip holds at once; the FIFO rules; X/Y chromosomes."""
    torch, ffsga = _ffs()
    _say("default slots,", kind, "pop", pop)
    inst = W.random_instance(29, n_jobs=50, n_stages=3, machines=[2, 2, 1], p_max=150, percent=60)
    inst.decode_rules = 1 if kind == "fifo" else 0
    d = ffsga.DeviceInstance.from_host(inst)
    xy = kind == "xy"
    prio = W.random_xy_population(31, pop, inst) if xy else W.random_population(31, pop, inst.n_active)
    got = ffsga.ffs_decode(d, torch.from_numpy(prio).cuda(), xy=xy).cpu().numpy()
    want = oracle.decode_xy_pop(inst, prio) if xy else oracle.decode_pop(inst, prio, n_threads=8)
    assert (got == want).all()
    if kind == "job":
        gp = W.GaParams(1, 1, pop, mig_interval=0, mig_k=0)
        ga = ffsga.GA(d, ffsga.GaConfig.of(gp), 5, 0, 0)
        assert ga.ga.lds_slots > 4096 and ga.overflows() == 0
        assert (ga.view()["obj"].cpu().numpy() == oracle.ga_init(inst, gp, 5, 0, 0)["obj"]).all()


@pytest.mark.parametrize("pop", [2048, 2049, 2200])
def test_auto_slots_in_two_parts(pop):
    """FFS_LDS_AUTO on either side of the population from which generation 0 is decoded in two
    parts (4 waves on each of 256 compute units, twice): state and a generation equal the oracle's."""
    torch, ffsga = _ffs()
    _say("auto slots, pop", pop)
    inst = W.random_instance(37, n_jobs=40, n_stages=3, machines=[2, 2, 1], p_max=150, percent=60)
    gp = W.GaParams(1, 1, pop, mig_interval=0, mig_k=0)
    ga = ffsga.GA(ffsga.DeviceInstance.from_host(inst),
                  ffsga.GaConfig.of(gp, lds_slots=ffsga.FFS_LDS_AUTO), 5, 0, 0)
    assert (ga.view()["obj"].cpu().numpy() == oracle.ga_init(inst, gp, 5, 0, 0, n_threads=8)["obj"]).all()
    ga.step(1)
    ga.status()
    st = oracle.ga_run(inst, gp, 5, 0, 0, 1, n_threads=8)
    for k in ("prio", "obj", "elite", "elite_obj"):
        assert (ga.view()[k].cpu().numpy() == np.asarray(st[k])).all(), k
