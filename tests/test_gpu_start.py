"""The library's own start against the same start given (MI355X only): one
value per column, filled in vectors, and marginals taken from q."""
import sys

import numpy as np
import pytest

from paper_2309_05315_amd import inputs
from paper_2309_05315_amd import mam

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.mark.parametrize("R,S,dtype,sched", [
    (1, [3, 70], "f64", {}), (7, [5, 4, 130], "f32", {}), (64, [257], "f32", {}), (513, [66, 1], "f64", {}),
    (1027, [65, 9], "f32", {}), (2051, [37, 64], "f64", dict(rows_per_tile=1024)),
    (8193, [9, 67], "f32", {}),
])
def test_default_start_equals_given_start(R, S, dtype, sched):
    """init() fills the plans with (T)(q_s/R) and takes their marginals from q;
    init(theta0) reads them: the same plans, and after an iteration (which
    reads both) the same plans and barycenter bit for bit."""
    p = inputs.tiny_problem(51, R=R, S=S, dtype=dtype)
    say(f"case start R={R} S={S} {dtype} {sched}")
    s = mam.solver_for(p, **sched)
    s.init()
    start = s.theta.clone()
    q = s.q.cpu().numpy().astype(np.float64)
    want = (q / R).astype(np.float32 if dtype == "f32" else np.float64)
    got = start.cpu().numpy()
    assert np.array_equal(got[:, :R], np.repeat(want[:, None], R, axis=1))
    m0 = s.marginals().cpu().numpy().copy()
    s.iterate(1)
    a = (s.theta[:, :R].cpu().numpy().copy(), s.barycenter().cpu().numpy().copy())
    s.init(start)
    np.testing.assert_array_equal(m0, s.marginals().cpu().numpy())
    s.iterate(1)
    np.testing.assert_array_equal(a[0], s.theta[:, :R].cpu().numpy())
    np.testing.assert_array_equal(a[1], s.barycenter().cpu().numpy())


def test_graphs_outlive_an_init_and_follow_its_inputs():
    """init() keeps the captured iterations while buffers and schedule stay:
    new costs and weights in the same buffers, a given start and the default
    one are followed as by a solver of their own."""
    a, b = (inputs.tiny_problem(seed, R=130, S=[40, 33, 70], dtype="f64", rho=2.0) for seed in (61, 62))
    say("case graph over init R=130 f64")
    s = mam.solver_for(a)
    s.graph(5)
    got = []
    for k, p in enumerate((a, b, a, b)):
        o = mam.solver_for(p)
        s.cost.copy_(o.cost)
        s.q.copy_(o.q)
        o.init()
        if k == 2:
            start = 0.5 * o.theta
            o.init(start)
            s.init(start)
        else:
            s.init()
        for x in (s, o):
            x.iterate(13)
        np.testing.assert_array_equal(s.theta.cpu().numpy(), o.theta.cpu().numpy())
        np.testing.assert_array_equal(s.barycenter().cpu().numpy(), o.barycenter().cpu().numpy())
        got.append(s.barycenter().cpu().numpy())
        o.close()
    assert not np.array_equal(got[0], got[1])


@pytest.mark.parametrize("bad", ["weight", "cost", "mass"])
def test_batch_refuses_a_bad_problem_by_its_number(bad):
    """The checks of all problems in one launch name the problem at fault."""
    probs = [inputs.tiny_problem(70 + i, R=9 + 60 * i, S=[5, 30 + i], dtype="f32") for i in range(5)]
    p = probs[3]
    if bad == "weight":
        p.q[2] = -1e-3
    elif bad == "cost":
        p.cost.flat[-1] = np.inf
    else:
        p.q[:5] *= 1.5
    say(f"case bad {bad}")
    with pytest.raises(mam.MAMError, match="problem 3"):
        mam.Batch(probs).init()
