"""The limits of the parallel start of exhaustive searches: how a team divides
itself over the children of a branching, and the counts of launches whose
workers do not make a team."""
import os
import subprocess

import numpy as np
import pytest

import cspgen

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1909_09213_amd", "csrc")

# Every member of a team takes a child in range that counts the member among
# its own, and the children's members follow on each other from 0 to the size.
DIVIDE = r"""
#include "cubics_internal.h"
#include <cstdio>
#include <cstdlib>
using namespace cubics;
int main(int argc, char **argv) {
    for (int a = 1; a < argc; ++a) {
        const long long size = atoll(argv[a]);
        if (!team_allowed(size)) { printf("%lld refused\n", size); continue; }
        for (int m : {2, 3, 7, 64, 100, 255, 256}) {
            if (m >= size) continue;
            long long next = 0;
            for (int k = 0; k < m; ++k) {
                const long long lo = team_first(k, (int)size, m), hi = team_first(k + 1, (int)size, m);
                if (lo != next || hi <= lo || hi > size) { printf("%lld/%d: child %d\n", size, m, k); return 1; }
                for (long long r : {lo, hi - 1})
                    if (team_child_of((int)r, (int)size, m) != k) { printf("%lld/%d: rank %lld\n", size, m, r); return 1; }
                next = hi;
            }
            if (next != size) { printf("%lld/%d: %lld\n", size, m, next); return 1; }
        }
        printf("%lld ok\n", size);
    }
}
"""


def test_a_team_divides_without_gaps(tmp_path):
    src, exe = tmp_path / "divide.cpp", tmp_path / "divide"
    src.write_text(DIVIDE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)])
    top = 1 << 22
    sizes = [2, 3, 5, 257, 5120, 6144, 30001, 1000003, top - 1, top]
    out = subprocess.run([str(exe)] + [str(s) for s in sizes + [top + 1, 9_000_000, 44_700_000, 1 << 31]],
                         capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert out.stdout.split("\n")[:-1] == [f"{s} ok" for s in sizes] + \
        [f"{s} refused" for s in (top + 1, 9_000_000, 44_700_000, 1 << 31)]


@pytest.mark.gpu
def test_more_workers_than_a_team_holds():
    """Nine million workers on three free variables, one of 256 values: every
    value is searched (the members of so large a team could not be counted in
    the products that divide it)."""
    from paper_1909_09213_amd import cubics as cb
    z = np.zeros(0, np.int64)
    inst = cspgen.Instance(lo=np.zeros(3, np.int32), dsize=np.array([256, 3, 2], np.int32), type=np.zeros(0, np.int32),
                           arity=np.zeros(0, np.int32), var_off=np.zeros(1, np.int64), vars=np.zeros(0, np.int32),
                           par_off=np.zeros(1, np.int64), params=z, tab_off=np.zeros(1, np.int64),
                           tabs=np.zeros(0, np.uint32), name="free")
    ctx = cb.Context(0)
    print("nine million workers", flush=True)
    r = ctx.solve(ctx.load(inst), cb.MODE_COUNT, layout=cb.LAYOUT_LANE, workers=9_000_000)
    assert (r.verdict, r.count, r.nodes, r.fails) == ("SAT", 1536, 1 + 2 + 6 + 1536, 0)


@pytest.mark.gpu
@pytest.mark.parametrize("batch", [1, 4])
def test_learned_branching_with_more_workers_than_fit(batch):
    """The learned kernel, whose workgroups hold the networks in LDS and of which
    the fewest fit at once: late workgroups must not be waited for, and each
    team's members choose the same variable at the same node."""
    import oracle
    from paper_1909_09213_amd import cubics as cb, learn
    insts = learn.instances(cspgen.SEED_EVAL, 12)
    refs = [oracle.solve(x, oracle.MODE_COUNT, max_nodes=300000) for x in insts]
    insts, refs = zip(*[(x, r) for x, r in zip(insts, refs) if r.verdict != "LIMIT"][:batch])
    assert len(insts) == batch
    ctx = cb.Context(0)
    probs, pol = [ctx.load(x) for x in insts], cb.Policy(ctx, learn.init_theta(1))
    for workers in (1, 30001, 0):
        print("learned, late", batch, workers, flush=True)
        res = ctx.solve_batch(probs, cb.MODE_COUNT, branching=cb.BRANCH_LEARNED, policy=pol, workers=workers,
                              layout=cb.LAYOUT_LANE)
        for r, ref in zip(res, refs):
            assert (r.verdict, r.count) == (ref.verdict, ref.count)
