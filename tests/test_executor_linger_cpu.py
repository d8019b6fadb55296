"""A freed tensor whose outgoing copy may still run keeps its range of the slab until an allocation
needs it or the run ends; the compute stream is made to wait for the copy then, and not before."""
import pytest

from paper_1811_12174_amd import planner
from paper_1811_12174_amd.executor import Executor, OutOfBudget
from paper_1811_12174_amd.program import Gap, Program, unet_program


class Log:
    """Backend that records what it is asked for, in order."""
    def __init__(self):
        self.ops, self.live = [], {}

    def slab(self, n):
        self.size = n

    def alloc(self, info, off):
        for t, (o, n) in self.live.items():     # never into a range another block still holds
            assert off + info.nbytes <= o or o + n <= off, (info.name, t)
        self.live[info.name] = (off, info.nbytes)
        return info.name

    def free(self, block):
        del self.live[block]

    def call(self, c, blocks):
        self.ops.append(c.fn)

    def swap_out(self, info, block):
        self.ops.append("out " + info.name)
        return info.name

    def __getattr__(self, name):
        if name not in ("release_after", "prefetch_start", "wait_in", "evict", "release"):
            raise AttributeError(name)
        return lambda h, *a: self.ops.append(name + " " + h)


def program():
    """a is made, read later and freed behind the up-sampling; then three more tensors are made."""
    p = Program(2)
    p.external("x", (1, 2, 2, 2, 256))                                   # 4096 bytes
    p.pool_fwd("x", p.new("a", (1, 1, 1, 1, 256)))                       # 512
    p.upsample_fwd("a", p.new("b", (1, 2, 2, 2, 256)))
    p.upsample_bwd("b", p.new("c", (1, 1, 1, 1, 256)), "a")              # last use of a and b
    p.upsample_fwd("c", p.new("d", (1, 2, 2, 2, 256)))
    p.upsample_bwd("d", p.new("e", (1, 1, 1, 1, 256)), "c")              # c, d and e live: 5120 bytes
    return p.finish()


@pytest.mark.parametrize("budget,early", [(5120, True), (8192, False)])
def test_freed_range_waits_for_need(budget, early):
    be, p = Log(), program()
    gaps = [Gap("a", 0, 0, 2)]
    ex = Executor(be, p, budget=budget)
    ex.run(p.instructions(gaps, 1), {"x": "x"})
    assert not be.live and ex.peak <= budget
    k = be.ops.index("release_after a")
    last = len(be.ops) - 1 - be.ops[::-1].index("upsample_bwd")
    assert be.ops.count("release_after a") == 1 and be.ops.count("release a") == 1
    assert (k < last) == early, be.ops


# U-Nets whose every idle gap fits the byte floor of that selection when freed ranges are free at once;
# when they linger the holes do not line up there
@pytest.mark.parametrize("shape", [(32, 1, 3, 1, 64, 64, 64), (32, 1, 4, 1, 128, 128, 128), (16, 1, 3, 2, 40, 48, 56), (64, 1, 4, 2, 256, 256, 256)])
def test_budgets_reach_what_ranges_freed_at_once_reach(shape):
    p = unet_program(*shape)
    gaps = p.gaps(3)
    ins, ext = p.instructions(gaps, 1), {t: t for t, i in p.tensors.items() if i.external}

    def least(budget, **how):       # the search of planner.swap_all
        while True:
            try:
                Executor(planner.SimBackend(), p, budget=budget, **how).run(ins, ext)
                return budget
            except OutOfBudget:
                budget = int(budget * 1.02)
    floor = planner.simulate(p, gaps, 1, None, True)[0].peak
    plan = planner.swap_all(p)
    assert plan.budget == least(floor, linger=False) < least(floor)
    # a step decides as the simulation did, and the plan runs so
    how = planner.lingers(p, plan, plan.budget, 0)
    Executor(planner.SimBackend(), p, budget=plan.budget, linger=how).run(p.instructions(plan.gaps, plan.lead, plan.at), ext)
    # with room ranges linger, and an equal plan is not worked out again
    assert planner.lingers(p, plan, 2 * plan.budget, 0) and len(p.lingers) == 2
    again = planner.Plan(list(plan.gaps), plan.lead, plan.eager, dict(plan.at))
    assert planner.lingers(p, again, plan.budget, 0) == how and len(p.lingers) == 2
