"""The parallel start of exhaustive searches (every worker takes a share of
its instance's first branchings) and the hand-over of half frames: counts,
node and failure counts equal the CPU oracle's for any number of workers,
with teams that are smaller, equal and larger than a branching, a last
workgroup that is not full, several instances per ring and both branching
schemes."""
import numpy as np
import pytest

import cspgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cb():
    from paper_1909_09213_amd import cubics
    return cubics


@pytest.fixture(scope="module")
def ctx(cb):
    return cb.Context(0)


@pytest.fixture(scope="module")
def small():
    insts = [cspgen.queens(7), cspgen.rb(1, n=14, d=6, dens_pm=400, tight_pm=350, base=701),
             cspgen.rb_sweep(3, base=702, nlo=10, nhi=12, dlo=34, dhi=40, plo=500, phi=600, tlo=680, thi=700),
             cspgen.global_twin(2, n=6, d=6, k_ad=4)]
    return [(x, [oracle.solve(x, oracle.MODE_COUNT, two_way=t) for t in (False, True)]) for x in insts]


@pytest.mark.parametrize("two_way", [False, True])
@pytest.mark.parametrize("layout", [1, 2, 3])
@pytest.mark.parametrize("workers", [2, 3, 7, 13, 333, 0])
def test_any_team_counts_the_same_tree(ctx, cb, small, workers, layout, two_way):
    for inst, refs in small:
        print("team", inst.name, workers, layout, two_way, flush=True)
        r = ctx.solve(ctx.load(inst), cb.MODE_COUNT, workers=workers, layout=layout, two_way=two_way)
        ref = refs[int(two_way)]
        assert (r.count, r.nodes, r.fails) == (ref.count, ref.nodes, ref.fails)


@pytest.mark.parametrize("batch,workers,active", [(3, 2, 0), (3, 7, 0), (5, 64, 0), (9, 40, 1), (24, 70, 3), (40, 0, 8)])
def test_teams_of_a_batch(ctx, cb, batch, workers, active):
    insts = [cspgen.rb_sweep(i, base=703, nlo=8, nhi=11, dlo=4, dhi=6, plo=350, phi=550, tlo=300, thi=450)
             for i in range(batch)]
    print("teams", batch, workers, active, flush=True)
    res = ctx.solve_batch([ctx.load(x) for x in insts], cb.MODE_COUNT, workers=workers, active_per_xcd=active)
    for x, r in zip(insts, res):
        ref = oracle.solve(x, oracle.MODE_COUNT)
        assert (r.count, r.nodes, r.fails) == (ref.count, ref.nodes, ref.fails)


def test_team_solutions_and_roots_without_a_branching(ctx, cb):
    """All solutions are stored once, and instances that end at their root
    (a solution, a failure, no variables) are counted once."""
    inst = cspgen.queens(6)
    r = ctx.solve(ctx.load(inst), cb.MODE_ALL, sol_capacity=16)
    assert r.count == r.n_written == 4 and len({tuple(x) for x in r.solutions}) == 4
    one = cspgen.queens(5).fix({0: 1, 1: 3, 2: 5, 3: 2, 4: 4})
    none = cspgen.queens(5).fix({0: 1, 1: 1})
    for x in (one, none):
        ref = oracle.solve(x, oracle.MODE_COUNT)
        for layout in (1, 2, 3):
            r = ctx.solve(ctx.load(x), cb.MODE_COUNT, layout=layout)
            assert (r.count, r.nodes, r.fails) == (ref.count, ref.nodes, ref.fails)


def test_worker_bound_searches_leave_when_nothing_is_queued(ctx, cb):
    """Without donation an idle worker leaves once every instance is taken;
    each instance is searched by one worker, the same way every time."""
    insts = [cspgen.rb_sweep(i, base=704, nlo=9, nhi=13, dlo=4, dhi=7, plo=350, phi=550, tlo=250, thi=400)
             for i in range(30)]
    probs = [ctx.load(x) for x in insts]
    for workers in (1, 4, 29, 0):
        res = ctx.solve_batch(probs, cb.MODE_FIRST, donate=False, workers=workers, layout=cb.LAYOUT_LANE)
        for x, r in zip(insts, res):
            ref = oracle.solve(x, oracle.MODE_FIRST)
            assert (r.verdict, r.nodes) == ("SAT" if ref.count else "UNSAT", ref.nodes)
            if r.solutions is not None and len(r.solutions):
                assert oracle.verify(x, np.asarray(r.solutions[0]))


@pytest.mark.parametrize("batch", [1, 5, 40])
def test_more_workers_than_fit_on_the_device(ctx, cb, batch):
    """A grid that is not resident as a whole: workgroups that start late (or
    find their share taken) must not be waited for."""
    insts = [cspgen.rb_sweep(i, base=703, nlo=8, nhi=11, dlo=4, dhi=6, plo=350, phi=550, tlo=300, thi=450)
             for i in range(batch)]
    probs = [ctx.load(x) for x in insts]
    for layout, active in ((1, 0), (3, 0), (1, 2)):
        print("late", batch, layout, active, flush=True)
        res = ctx.solve_batch(probs, cb.MODE_COUNT, workers=30001, layout=layout, active_per_xcd=active)
        for x, r in zip(insts, res):
            ref = oracle.solve(x, oracle.MODE_COUNT)
            assert (r.count, r.nodes, r.fails) == (ref.count, ref.nodes, ref.fails)
