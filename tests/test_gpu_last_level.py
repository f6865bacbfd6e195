"""Nodes whose only open variable is closed in one step: counts and node
counts in closed form, at every domain width and around the node budget, and
against the paths that store or cap solutions (which try every value)."""
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


@pytest.mark.parametrize("k", [1, 2, 3, 31, 32, 33, 64, 65, 200, 256])
@pytest.mark.parametrize("layout", [1, 2, 3])
def test_one_free_variable(ctx, cb, k, layout):
    p = ctx.load(_free([k]))
    for kw, below in (({}, k), ({"two_way": True}, 2 * k - 2), ({"workers": 1}, k), ({"max_nodes": 10 ** 6}, k)):
        r = ctx.solve(p, cb.MODE_COUNT, layout=layout, **kw)
        assert (r.verdict, r.count, r.nodes, r.fails) == ("SAT", k, 1 + (below if k > 1 else 0), 0), kw
    r = ctx.solve(p, cb.MODE_ALL, layout=layout, sol_capacity=k)
    assert r.n_written == r.count == k and sorted(x[0] for x in r.solutions) == list(range(3, 3 + k))


@pytest.mark.parametrize("sizes", [(2, 2), (3, 7, 2), (40, 33), (2, 2, 2, 2, 2, 2, 2), (9, 70, 5)])
def test_free_products(ctx, cb, sizes):
    """First-fail order: the k-th level holds the product of the k smallest
    domains."""
    inst = _free(sizes)
    s = sorted(sizes)
    nodes = 1 + sum(int(np.prod(s[:j + 1])) for j in range(len(s)))
    for layout in (1, 2, 3):
        r = ctx.solve(ctx.load(inst), cb.MODE_COUNT, layout=layout)
        assert (r.count, r.nodes, r.fails) == (int(np.prod(s)), nodes, 0)


@pytest.mark.parametrize("budget", [1, 40, 100, 128, 200, 5000])
def test_a_budget_stays_within_its_slack(ctx, cb, budget):
    """A worker stops within 128 nodes past max_nodes."""
    inst = _free([2, 3, 5, 7, 30])
    total = oracle.solve(inst, oracle.MODE_COUNT).nodes
    for layout in (1, 2, 3):
        r = ctx.solve(ctx.load(inst), cb.MODE_COUNT, layout=layout, workers=1, max_nodes=budget)
        assert r.nodes <= budget + 128 or r.nodes == total
        assert r.verdict == ("LIMIT" if r.nodes < total else r.verdict)
