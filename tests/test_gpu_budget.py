"""Node budgets.  A worker holds at most 128 nodes that it has not counted
against its instance's budget, and takes up no more of the instance once it
has seen the budget used up: a search whose tree is larger than the budget by
more than 128 nodes for each worker that took part ends as LIMIT within that
slack, and one whose tree is smaller than the budget is complete."""
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


def _free(sizes):
    """Variables without constraints."""
    n, z = len(sizes), np.zeros(0, np.int64)
    return cspgen.Instance(lo=np.full(n, 3, np.int32), dsize=np.array(sizes, np.int32), type=np.zeros(0, np.int32),
                           arity=np.zeros(0, np.int32), var_off=np.zeros(1, np.int64), vars=np.zeros(0, np.int32),
                           par_off=np.zeros(1, np.int64), params=z, tab_off=np.zeros(1, np.int64),
                           tabs=np.zeros(0, np.uint32), name="free")


@pytest.mark.parametrize("two_way", [False, True])
@pytest.mark.parametrize("sizes", [(2, 3, 5, 7, 30), (2, 9, 31), (3, 4, 31, 31), (2, 30, 200)])
@pytest.mark.parametrize("layout", [1, 2, 3])
def test_one_worker_stops_within_128_nodes(ctx, cb, layout, sizes, two_way):
    """Also where the last open variable has more values than a node under a
    budget may close."""
    inst = _free(sizes)
    ref = oracle.solve(inst, oracle.MODE_COUNT, two_way=two_way)
    p = ctx.load(inst)
    for budget in (1, 31, 96, 127, 128, 129, 300, 500, ref.nodes - 129):
        if budget + 128 >= ref.nodes:
            continue
        r = ctx.solve(p, cb.MODE_COUNT, layout=layout, workers=1, max_nodes=budget, two_way=two_way)
        assert r.verdict == "LIMIT" and budget <= r.nodes < budget + 128, budget
        assert r.count < ref.count
    for budget in (ref.nodes + 1, 10 * ref.nodes):
        r = ctx.solve(p, cb.MODE_COUNT, layout=layout, workers=1, max_nodes=budget, two_way=two_way)
        assert (r.verdict, r.count, r.nodes, r.fails) == ("SAT", ref.count, ref.nodes, 0)


@pytest.fixture(scope="module")
def large():
    """A tree of 1.1e6 nodes."""
    inst = cspgen.rb(0, n=30, d=10, dens_pm=250, tight_pm=390)
    ref = oracle.solve(inst, oracle.MODE_COUNT)
    assert ref.nodes > 10 ** 6
    return inst, ref


@pytest.mark.parametrize("workers,budget", [(0, 1000), (0, 100000), (1, 50000), (7, 5000), (64, 20000), (64, 70000)])
@pytest.mark.parametrize("layout", [1, 2, 3])
def test_a_large_tree_is_not_searched_past_its_budget(ctx, cb, large, layout, workers, budget):
    """With every worker of the device, with a few that open the tree as a team
    (64 and 70,000), and with a few that share one worker's."""
    inst, ref = large
    r = ctx.solve(ctx.load(inst), cb.MODE_COUNT, layout=layout, workers=workers, max_nodes=budget)
    took_part = min(r.tasks, workers) if workers else r.tasks
    print("budget", layout, workers, budget, r.nodes, r.tasks, flush=True)
    assert r.verdict == "LIMIT"
    assert budget <= r.nodes < budget + 128 * took_part
    # one worker opens the tree: by 1,000 nodes a few dozen have joined it, not
    # the thousands of the device
    assert r.nodes < (8 * budget if budget == 1000 else ref.nodes // 2)
    r = ctx.solve(ctx.load(inst), cb.MODE_COUNT, layout=layout, workers=workers, max_nodes=ref.nodes + 1)
    assert (r.verdict, r.count, r.nodes, r.fails) == ("SAT", ref.count, ref.nodes, ref.fails)


@pytest.mark.parametrize("layout", [1, 2, 3])
@pytest.mark.parametrize("tree", ["random", "even"])
def test_a_tree_of_fewer_nodes_than_the_workers_slack(ctx, cb, layout, tree):
    """147,718 and 2^18 - 1 nodes, less than 128 for each worker of the device:
    none of them may search its share of the tree unchecked."""
    inst = cspgen.rb(0, n=20, d=10, dens_pm=350, tight_pm=400, base=77) if tree == "random" else _free([2] * 17)
    for budget in (1, 1000, 5000):
        r = ctx.solve(ctx.load(inst), cb.MODE_COUNT, layout=layout, max_nodes=budget)
        print("small tree", layout, budget, r.verdict, r.nodes, r.tasks, flush=True)
        assert r.verdict == "LIMIT" and budget <= r.nodes < budget + 128 * r.tasks


@pytest.mark.parametrize("active", [0, 2])
@pytest.mark.parametrize("mode", ["count", "first"])
def test_budgets_of_a_batch(ctx, cb, active, mode):
    """Each instance has its own budget: the small trees are complete, the
    large ones stop."""
    workers, budget = 48, 3000
    insts = [cspgen.rb(i // 2, n=20, d=10, dens_pm=350, tight_pm=400, base=77) if i % 2 else cspgen.queens(6)
             for i in range(24)]
    m, om = (cb.MODE_COUNT, oracle.MODE_COUNT) if mode == "count" else (cb.MODE_FIRST, oracle.MODE_FIRST)
    res = ctx.solve_batch([ctx.load(x) for x in insts], m, workers=workers, max_nodes=budget, active_per_xcd=active)
    for x, r in zip(insts, res):
        ref = oracle.solve(x, om, max_nodes=200000)
        if mode == "first":
            assert r.verdict == "SAT" and oracle.verify(x, np.asarray(r.solutions[0]))
        elif ref.nodes <= budget:
            assert (r.verdict, r.count, r.nodes, r.fails) == ("SAT", ref.count, ref.nodes, ref.fails)
        else:
            assert ref.nodes > budget + 128 * workers
            assert r.verdict == "LIMIT" and budget <= r.nodes < budget + 128 * min(workers, r.tasks)
