"""Calls of several iterations against the same iterations one call at a time
(MI355X only).

A call of one iteration runs the dense column kernels; a longer one may keep
the plans as -b plus their active entries in between (sparse_iterations says
whether it does).  Both store the same values and add the same numbers in the
same order, so plans, marginals and barycenters are compared bit for bit.  The
dense kernels are held to the oracle in the other files; here the sizes are
the edges of the sparse kernels: blocks of 64 rows, partial vectors, columns
with more active entries than a column lists, with entries exactly at their
threshold, without weight or with a weight below the rounding of w, every cost
layout.
"""
import dataclasses
import sys

import numpy as np
import pytest
import torch

from paper_2309_05315_amd import inputs
from paper_2309_05315_amd import mam

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def state(s):
    return (s.barycenter().cpu().numpy(), s.marginals().cpu().numpy(), s.theta.cpu().numpy())


def both(p, iters, graph=0, **kw):
    """(one call per iteration, one call) from the default start."""
    out = []
    for whole in (False, True):
        say(f"case {p.name} R={p.R} M={p.M} T={p.T} {p.dtype} rho={p.rho} gamma={p.gamma} iters={iters} {kw} whole={whole}")
        s = mam.solver_for(p, **kw)
        if whole and graph:
            s.graph(graph)
        s.init()
        if whole:
            s.iterate(iters)
        else:
            for _ in range(iters):
                s.iterate(1)
        out.append(state(s))
        s.close()
    return out


def same(a, b):
    for x, y in zip(a, b):
        assert np.array_equal(x, y), float(np.abs(x - y).max())


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("R,S", [(5, [90001, 1, 180000]), (63, [9000, 12001]), (64, [21000]), (65, [10007, 11000]),
                                 (1023, [700, 619, 7]), (1025, [707, 623]), (4099, [210, 113]), (8192, [84, 83])])
def test_ragged_sizes(R, S, dtype):
    """Random supports: rows at the edges of the blocks, columns without
    weight, waves of 4 (up to 2^13 columns), 16 and 32 columns."""
    p = inputs.tiny_problem(R + len(S), R=R, S=S, dtype=dtype, zero_frac=0.15)
    same(*both(p, 14))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nt", [16, 64, 128, 256])
def test_threshold_sums_keep_the_column_kernels_order(dtype, nt):
    """Active sets of three and more entries in every thread shape (also the
    sub-wave ones, which start a call differently), and more of them than a
    column lists: rho widens the sets."""
    p = inputs.balanced_plain(K=16, M=22, dtype=dtype)
    for rho in (1.0, 3.0):
        same(*both(dataclasses.replace(p, rho=rho), 9, threads_per_column=nt))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("gamma,relaxed", [(0.05, False), (0.2, True), (0.0, False)])
def test_unbalanced_and_relaxed(gamma, relaxed, dtype):
    p = inputs.tiny_problem(23, R=1100, S=[470, 341, 488], masses=[0.7, 1.0, 1.3], gamma=gamma, dtype=dtype)
    if relaxed:
        p = dataclasses.replace(p, cost=(p.cost - 0.002).astype(np.float32).astype(np.float64))
    same(*both(p, 20, relaxed=relaxed))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_small_weights_and_graph_replay(dtype):
    """Gaussian tails (weights far below the rounding of w: columns without
    an active entry), an indexed cost, replayed from a graph."""
    same(*both(inputs.balanced_plain(K=24, M=5, dtype=dtype), 40, graph=8))
    same(*both(inputs.balanced_sparse(K=22, M=40, dtype=dtype), 30, graph=7))


def test_unaligned_plans_and_a_cost_rebuilt_in_place():
    """Column strides off the vector width; the cost changed between two
    calls (its block minima belong to one call); padding rows untouched."""
    p = inputs.tiny_problem(61, R=301, S=[2160, 2229], dtype="f32")
    res = []
    for whole in (False, True):
        s = mam.Solver(301, p.S, dtype=torch.float32, cost_mode=mam.COST_PER_COLUMN, cost_ncols=p.T, ld=303, cost_ld=301)
        cost = torch.from_numpy(p.cost).float().cuda()
        theta = torch.full((p.T, 303), 123.0, device="cuda")
        s.bind(theta, cost, torch.from_numpy(p.q).float().cuda())
        s.init()
        for _ in range(3):
            if whole:
                s.iterate(8)
            else:
                for _ in range(8):
                    s.iterate(1)
            cost.copy_(cost.roll(7, 0))
        assert bool((theta[:, 301:] == 123.0).all())
        res.append(state(s))
        s.close()
    same(*res)


@pytest.mark.parametrize("test", ["dp", "dist", "dtheta"])
def test_stopping_tests(test):
    """A run stopped by its test leaves the iterate of the same plain iterations."""
    p = inputs.balanced_sparse(K=26, M=4, dtype="f64")
    s = mam.solver_for(p)
    s.init()
    s.graph(5)
    probe = s.iterate_until(36, test, -1.0, 9)
    s.init()
    r = s.iterate_until(400, test, probe["value"], 9)
    # (the value need not fall monotonically: an earlier check may meet it too)
    assert r["converged"] and r["iterations"] <= 36 and r["value"] <= probe["value"]
    got = state(s)
    s.init()
    for _ in range(r["iterations"]):
        s.iterate(1)
    same(state(s), got)


def test_recorded_active_sets():
    """Reverse mode over a recorded sparse run against windows of one
    iteration, which the dense kernels record."""
    for p in (inputs.adjoint_problem(K=24, M=3, dtype="f64")[0],
              dataclasses.replace(inputs.unbalanced_dense(K=22, M=7, gamma=0.02, dtype="f32"), rho=3.0)):
        g = torch.linspace(-1, 1, p.R, dtype=torch.float64, device="cuda")
        grads = []
        for ck in (0, 9, 1):
            s = mam.solver_for(p)
            s.init()
            s.record(20, ck)
            grads.append([x.cpu().numpy() for x in s.backward(g)])
            s.close()
        assert np.abs(grads[0][1]).max() > 0.0
        for other in grads[1:]:
            same(grads[0], other)


@pytest.mark.parametrize("dtype,gamma", [("f64", np.inf), ("f32", np.inf), ("f32", 0.05)])
def test_bundles(dtype, gamma):
    """Bundles that are first drawn late in a call, and one that is not drawn
    at all (its plans stay as they were)."""
    p = inputs.balanced_sparse(K=24, M=9, dtype=dtype)
    if np.isfinite(gamma):
        p = dataclasses.replace(p, gamma=gamma)
    seq = [0, 0, 1, 0, 1, 1, 0] * 5 + [2] * 3 + [1, 2, 0, 1] * 4
    res = []
    for whole in (False, True):
        say(f"case bundles {dtype} gamma={gamma} whole={whole}")
        s = mam.solver_for(p)
        s.init()
        s.set_bundles([m % 4 for m in range(p.M)])
        for part in (seq, seq[::-1]):
            if whole:
                s.iterate_bundles(part)
            else:
                for b in part:
                    s.iterate_bundles([b])
        res.append(state(s))
        s.close()
    same(*res)


@pytest.mark.parametrize("dtype,M", [("f32", 16), ("f64", 17), ("f32", 33), ("f32", 95)])
def test_measures_over_several_workgroups(dtype, M):
    """With a finite gamma the second part of the close deals a block's
    measures over workgroups of 16: one workgroup, one measure in the second,
    several, the most that the sparse iterations take."""
    rng = np.random.default_rng(M)
    S = [int(x) for x in rng.integers(1, 3 * 5_400_000 // (130 * 4 * M) + 30, size=M)]
    p = inputs.tiny_problem(80 + M, R=130, S=S, dtype=dtype, rho=1.0, masses=list(rng.uniform(0.5, 1.5, M)), gamma=0.05)
    same(*both(p, 11))


def dyadic_problem(K, M, S, levels, dtype="f64", rho=1024.0):
    """M measures on S pixels each of a K x K grid, integer costs and weights
    of a few binary digits: many entries of w lie exactly at a column's
    threshold, or miss it by the rounding of one quotient."""
    rng = np.random.default_rng(5)
    R = K * K
    pts = inputs.grid_points(K) * K
    cols = np.concatenate([np.sort(rng.permutation(R)[:S]) for _ in range(M)])
    q = np.concatenate([np.bincount(rng.integers(0, S, levels * S), minlength=S) for _ in range(M)]) / (512.0 * levels)
    return inputs.Problem(name=f"dyadic_K{K}_M{M}_S{S}", R=R, S=[S] * M, cost=np.rint(inputs.sq_euclid(pts, pts)), q=q,
                          dtype=dtype, iters=20, rho=rho, col_index=cols.astype(np.int32))


@pytest.mark.parametrize("K,M,S,levels", [(26, 8, 512, 4), (26, 8, 512, 8), (24, 8, 576, 4), (32, 3, 1024, 16)])
def test_entries_at_the_threshold(K, M, S, levels):
    """Which of them a threshold is formed over decides its last bit, and on
    such data the last bits decide where mass goes."""
    for iters in (12, 40):
        same(*both(dyadic_problem(K, M, S, levels), iters))


def test_recorded_sets_at_the_threshold():
    """A recorded set that takes in an entry at the threshold, or leaves it
    out, changes the gradient by a whole part of it."""
    p = dyadic_problem(26, 8, 512, 4)
    g = torch.linspace(-1, 1, p.R, dtype=torch.float64, device="cuda") ** 2
    grads = []
    for ck in (0, 9, 1):
        s = mam.solver_for(p)
        s.init()
        s.record(30, ck)
        grads.append([x.cpu().numpy() for x in s.backward(g)])
        s.close()
    for other in grads[1:]:
        same(grads[0], other)


def test_rises_below_the_rounding_of_their_sum():
    """Two measures of 2048 columns.  In the first iteration 512 columns of
    one put their weight on a row of theta0's choosing and never again: a rise
    of 2^-14, and then only a column of weight 2^-56 in each, which the other
    pulls towards its own row by 2^-68 an iteration, a quarter of what a sum
    of 2^-14 rounds to.  After 2048 iterations their mass starts to move."""
    R, S, tiny = 192, 2048, 2.0 ** -56
    cost = np.ones((2 * S, R))
    cost[:, 140] = 0.0
    q = np.full(2 * S, 2.0 ** -11)
    theta0 = np.repeat(q[:, None] / 256, R, 1)
    theta0[100:612, 141] = 2.0
    for j, (own, other) in ((5, (10, 75)), (S + 5, (75, 10))):
        q[j] = tiny
        theta0[j] = 0.0
        cost[j] = 1.0
        cost[j, own] = 0.0
        cost[j, other] = tiny
    res = []
    for part in (7, 2600):  # calls of seven iterations are dense
        say(f"case rises part={part}")
        s = mam.Solver(R, [S, S], dtype=torch.float64, cost_mode=mam.COST_PER_COLUMN, cost_ncols=2 * S)
        put = lambda x, ld: torch.nn.functional.pad(torch.from_numpy(x), (0, ld - R)).cuda()
        s.bind(torch.zeros(2 * S, s.ld, dtype=torch.float64, device="cuda"), put(cost, s.cost_ld), torch.from_numpy(q).cuda())
        s.init(put(theta0, s.ld))
        for k in range(0, 2600, part):
            s.iterate(min(part, 2600 - k))
        res.append(state(s))
        s.close()
    assert res[0][2][5, 75] > res[0][2][6, 75]  # some of it has: more than the value of an inactive entry
    same(*res)


@pytest.mark.parametrize("seed", range(6))
def test_relaxed_entries_at_the_threshold(seed):
    """Relaxed columns (and no damping step: gamma = 0): an entry that the
    threshold's last round left out stays 0, though it may lie an ulp above
    the threshold."""
    rng = np.random.default_rng([11, seed])
    R, S = 479, [100, 41, 94, 132, 96, 888, 120, 92, 233]
    T = sum(S)
    p = inputs.Problem(name=f"dyadic_relaxed_{seed}", R=R, S=S, cost=rng.integers(0, 400, (T, R)) - 3.0,
                       q=rng.integers(0, 5, T) / 2048.0, dtype="f64", iters=8, rho=4096.0, gamma=0.0,
                       col_index=np.arange(T, dtype=np.int32))
    for iters in (8, 20):
        same(*both(p, iters, relaxed=True))


def long_columns(R, S, dtype, **kw):
    """rho keeps the active sets small: the estimate at the start is 5 to 14 rows."""
    return inputs.tiny_problem(R + len(S), R=R, S=S, dtype=dtype, rho=0.05, **kw)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("gamma", [np.inf, 0.05])
@pytest.mark.parametrize("R,S", [(4096, [310, 313]), (4097, [340, 283]), (4099, [310, 313]), (8192, [184, 183])])
def test_more_than_64_blocks(R, S, gamma, dtype):
    """Block bounds, drifts and d^2 partials of a second 64 blocks; a first
    iteration of 256 to 1024 threads."""
    p = long_columns(R, S, dtype, gamma=gamma, zero_frac=0.1)
    s = mam.solver_for(p)
    s.init()
    assert s.sparse_iterations(30) and not s.sparse_iterations(1)
    s.close()
    same(*both(p, 30))
    same(*both(p, 30, threads_per_column=1024))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_more_than_64_blocks_recorded(dtype):
    p = long_columns(8000, [150, 133], dtype)
    g = torch.linspace(-1, 1, p.R, dtype=torch.float64, device="cuda")
    grads = []
    for ck in (0, 1):
        s = mam.solver_for(p)
        s.init()
        assert s.sparse_iterations(20) and not s.sparse_iterations(1)
        s.record(20, ck)
        grads.append([x.cpu().numpy() for x in s.backward(g)])
        s.close()
    assert np.abs(grads[0][1]).max() > 0.0
    same(*grads)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("R,S,nt", [(70, [9000, 11003], 16), (130, [3001, 2999, 4100], 16), (256, [2600, 2700], 16),
                                    (100, [7001, 7005], 32), (301, [4601, 4600, 4300], 32), (512, [4300, 4301], 32)])
def test_sub_wave_first_iteration(R, S, nt, dtype):
    """Groups of 16 and 32 lanes store patches from a call's first iteration
    on: values per lane from 4 to 16, rows off the vector width, columns
    without weight, lists of up to 16 entries and columns with more."""
    for rho in (0.3, 12.0):
        p = inputs.tiny_problem(R, R=R, S=S, dtype=dtype, rho=rho, zero_frac=0.1)
        s = mam.solver_for(p, threads_per_column=nt)
        s.init()
        assert s.sparse_iterations(20)
        s.close()
        same(*both(p, 20, threads_per_column=nt))


def test_sub_wave_calls_do_not_start_dense():
    """A call of nine iterations on groups of 32 lanes, against one wave per
    column: as long as its first iteration left every column to the whole-wave
    path, the column kernels took 2.3 times as long on a batch."""
    p = inputs.tiny_problem(3, R=250, S=[5003] * 8, dtype="f32")
    ms = {}
    for nt in (32, 64):
        s = mam.solver_for(p, threads_per_column=nt)
        times = []
        for k in range(5):
            s.init()
            s.timing(k > 0)
            s.iterate(9)
            if k:
                times.append(s.timing_read()[0])
        ms[nt] = min(times)
        s.close()
    say(f"column kernels {ms}")
    assert ms[32] <= 1.4 * ms[64]


def test_wide_sets_at_the_start_need_longer_calls():
    """Estimates of 6 to 50 active rows per column at the start: the first
    iterations of a sparse call cost more the wider the sets are, so a call
    has to be longer to make that good, until the run has them behind it."""
    p = inputs.balanced_plain(K=32, M=8, dtype="f32")
    least = {}
    for rho in (1.0, 4.0, 7.0):
        s = mam.solver_for(dataclasses.replace(p, rho=rho))
        s.init()
        least[rho] = next(n for n in range(1, 60) if s.sparse_iterations(n))
        s.iterate(60)
        assert s.sparse_iterations(8) and not s.sparse_iterations(7)
        s.close()
    say(f"least iterations {least}")
    assert least[1.0] == 8 < least[4.0] < least[7.0] <= 30


def test_a_batch_weighs_its_problems_by_their_columns():
    """Bits of a batch with one problem of very wide sets, which it can carry,
    and with all of them like that, when it stays dense."""
    probs = inputs.batched_problems(n=24, k_range=(20, 28), iters=10)
    for wide, sparse in ((0, True), (1, True), (24, False)):
        these = [dataclasses.replace(q, rho=200.0) if i < wide else q for i, q in enumerate(probs)]
        b = mam.Batch(these)
        b.init()
        assert b.sparse_iterations(100) == sparse
        b.iterate(30)
        for i in (0, 1, 23):
            one = mam.solver_for(these[i])
            one.init()
            for _ in range(30):
                one.iterate(1)
            assert np.array_equal(b.barycenter(i).cpu().numpy(), one.barycenter().cpu().numpy())
            one.close()
        b.close()


@pytest.mark.parametrize("R,few", [(1024, 10), (1024, 3), (4000, 25)])
def test_a_measure_of_few_columns(R, few):
    """Its columns hold a part of the barycenter's rows each, more than they
    list.  The same bits, and no more time than dense iterations (calls of
    seven) take."""
    p = inputs.tiny_problem(3, R=R, S=[1024] * 7 + [few], dtype="f32")
    ms, res = {}, []
    for part in (7, 140):
        s = mam.solver_for(p)
        times = []
        for _ in range(3):
            s.init()
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            for _ in range(140 // part):
                s.iterate(part)
            e[1].record()
            torch.cuda.synchronize()
            times.append(e[0].elapsed_time(e[1]))
        assert s.sparse_iterations(part) == (part == 140)
        ms[part] = min(times)
        res.append(state(s))
        s.close()
    say(f"R={R} few={few}: {ms}")
    same(*res)
    assert ms[140] < 1.05 * ms[7]


def test_a_cost_rebuilt_in_place_with_wider_sets():
    """The choice of a route is by the costs at the start.  With the cost cut
    to a 256th in place the sets are 256 times as wide: the next call, sparse
    still, gives the same bits, and the ones after it are dense until the run
    is twice as long."""
    p = inputs.balanced_plain(K=32, M=8, dtype="f32")
    res = []
    for whole in (False, True):
        s = mam.solver_for(p)
        s.init()
        s.iterate(40)
        s.cost.mul_(1.0 / 256)
        for part in (10, 70):
            if whole:
                assert s.sparse_iterations(part) == (part == 10)
                s.iterate(part)
                torch.cuda.synchronize()  # (the note of a call that runs is not waited for)
            else:
                for _ in range(part):
                    s.iterate(1)
        res.append(state(s))
        if whole:
            assert not s.sparse_iterations(100)
            s.iterate(100)
            assert s.sparse_iterations(100)
            s.init()
            assert not s.sparse_iterations(100)  # by the estimate of these costs
            s.cost.mul_(256.0)
            s.init()
            assert s.sparse_iterations(100)
        s.close()
    same(*res)
