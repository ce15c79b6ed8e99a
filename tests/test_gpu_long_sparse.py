"""What the sparse store of long columns leaves out (MI355X only).

From the second iteration of a call the scan takes only the (column, sub-tile)
pairs that can hold an active entry, and keeps only candidates above a bound
of the column's threshold.  A call of several iterations is compared bit for
bit with the dense store, which leaves out nothing: columns without weight or
with a weight below the rounding of w, more candidates than slots, groups of
64 columns that span measures, last tiles with rows past R, and every cost
layout.
"""
import sys

import numpy as np
import pytest
import torch

from paper_2309_05315_amd import inputs
from paper_2309_05315_amd import mam

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


CASES = [
    # f32 grid, 4096-row tiles, many measures in one group of columns
    (lambda: inputs.free_support(seed=21, K=18, M=6, dtype="f32"), dict(rows_per_tile=4096, grid=True)),
    (lambda: inputs.free_support(seed=22, K=6, M=20, dtype="f64"), dict(rows_per_tile=2048, grid=True)),
    # one row more than two tiles; stored costs, scalar loads
    (lambda: inputs.tiny_problem(41, R=2049, S=[70, 3, 64, 1], dtype="f32", rho=3.0), dict(rows_per_tile=1024)),
    (lambda: inputs.tiny_problem(42, R=4100, S=[65, 130], dtype="f64", rho=0.3), dict(rows_per_tile=1024)),
    # fewer slots than candidates: sub-tiles recomputed, stored as patches or dense
    (lambda: inputs.tiny_problem(43, R=3000, S=[40, 90], dtype="f32", rho=60.0),
     dict(rows_per_tile=1024, candidate_slots=2)),
    (lambda: inputs.tiny_problem(44, R=2600, S=[33, 31], masses=[0.7, 1.3], gamma=0.05), dict(rows_per_tile=1024)),
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("weights", ["as drawn", "tiny and zero"])
def test_pruned_scan_equals_dense(case, weights):
    gen, sched = CASES[case]
    p = gen()
    if weights != "as drawn":
        # a third of the columns at weights below the rounding of w, some 0;
        # the others of a measure make up its mass
        rng = np.random.default_rng(case)
        j0 = 0
        for n in p.S:
            q = p.q[j0:j0 + n]
            mass, pick = q.sum(), rng.random(n) < 0.33
            pick[int(np.argmax(q))] = False
            q[pick] = rng.choice([0.0, 1e-30, 1e-19, 1e-14], size=int(pick.sum()))
            q[~pick] *= mass / q[~pick].sum()
            if p.dtype == "f32":
                q[:] = q.astype(np.float32)
            j0 += n
    say(f"case {case} R={p.R} M={p.M} T={p.T} {p.dtype} weights={weights} {sched}")
    sd = mam.solver_for(p, **sched)
    ss = mam.solver_for(p, sparse_store=True, **sched)
    assert ss.schedule()["rows_per_tile"] > 0
    for s in (sd, ss):
        s.init()
    for step, (iters, graph) in enumerate([(1, 0), (2, 0), (11, 0), (9, 4)]):
        for s in (sd, ss):
            s.graph(graph)
            s.iterate(iters)
        for x, y in zip(sd.plans(), ss.plans()):
            np.testing.assert_array_equal(x, y, err_msg=f"plans after call {step}")
        np.testing.assert_array_equal(sd.marginals().cpu().numpy(), ss.marginals().cpu().numpy())
        np.testing.assert_array_equal(sd.barycenter().cpu().numpy(), ss.barycenter().cpu().numpy())
