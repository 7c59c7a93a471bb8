"""Regularised components where the product over the energy denominators ends:
first order, which has none (every component is the bare weight), alone, in sets
of mixed orders and served; and shifts so large that the product of the shifted
denominators leaves the range of a double (the component goes to zero, the main
weight is untouched)."""
import numpy as np
import pytest

import oracle as O

from test_gpu_parity import TOL, Run, _check_samples, _task
from test_gpu_server import Server

pytestmark = pytest.mark.gpu

K = 4


@pytest.fixture(scope="module")
def M():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_24532_amd as M
    M.lib()
    return M


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("q,x,group", [(2, 0.0, -1), (4, 0.3, -1), (4, 0.3, 0)])
def test_first_order_components(M, q, x, group, precision):
    print(f"case reg order=1 q={q} x={x} group={group} precision={precision}", flush=True)
    count = 3000
    pb = O.problem(1, 0, density=0.16, proton_fraction=x, q=q, seed=1, task_key=7, group=group,
                   reg_k=K, reg_eta=1.5, label_method=0)
    grid = O.uniform_grid(6)
    wo, co = O.sample_values(pb, grid, 0, 0, count)
    wro = O.sample_values_reg(pb, grid, 0, 0, count)
    assert np.count_nonzero(wo) > 0 and np.array_equal(wro, np.repeat(wo[:, None], K, 1))
    task = _task(1, 0, q, 0.16, x, 7)
    run = Run(M, [task if group < 0 else task + (1,)], max_samples=4096, precision=precision)
    try:
        M.mbpt_set_regularization(run.ctx, K, 1.5)
        w = M.mbpt_dump_samples(run.set, 0, 0, 0, count)
        wr = M.mbpt_dump_samples_reg(run.set, 0, 0, 0, count, K)
    finally:
        run.close()
    _check_samples(w, wo, co, (q, x, group, precision))
    for k in range(K):
        _check_samples(wr[:, k], wo, co, (q, x, group, precision, k))


@pytest.mark.parametrize("mode", [0, 1, 2, 3])
@pytest.mark.parametrize("q,x", [(2, 0.0), (4, 0.3)])
def test_mixed_orders(M, q, x, mode):
    """An equation of state over orders 1 to 3 with components, each iteration
    against the oracle's (the tolerances of the full runs of single orders)."""
    print(f"case reg mixed q={q} mode={mode}", flush=True)
    N, iters, eta = 1 << 14, 3, 1.0
    cases = [(1, 0), (2, 0), (3, 1), (3, 2)]
    tasks = [_task(o, d, q, 0.12, x, 3 + i) for i, (o, d) in enumerate(cases)]
    tasks.append(_task(1, 0, q, 0.16, x, 9) + (1,))
    run = Run(M, tasks, max_samples=N, mode=mode)
    try:
        M.mbpt_set_regularization(run.ctx, 3, eta)
        per, _ = M.mbpt_integrate(run.set, N, iters)
        logs = [M.mbpt_iteration_log(run.set, t) for t in range(len(tasks))]
        rlogs = [M.mbpt_regularized_log(run.set, t, 3) for t in range(len(tasks))]
    finally:
        run.close()
    for t, task in enumerate(tasks):
        pb = O.problem(task[0], task[1], density=task[3], proton_fraction=x, q=q, seed=1,
                       task_key=task[5], group=0 if len(task) > 6 else -1, reg_k=3, reg_eta=eta,
                       label_method=0)
        _, Io, Vo, Iro, Vro, _ = O.integrate_reg(pb, N, iters)
        assert np.allclose(logs[t][0], Io, rtol=1e-9, atol=0), (t, logs[t][0], Io)
        assert np.allclose(rlogs[t][0], Iro, rtol=1e-9, atol=0), (t, rlogs[t][0], Iro)
        assert np.allclose(rlogs[t][1], Vro, rtol=1e-7, atol=0), (t, rlogs[t][1], Vro)
        assert np.isfinite(per[t].E_per_A) and per[t].sigma > 0


def test_served_first_order(M):
    """A first-order request of a regularised server: the components and the
    extrapolation are the estimate itself (weights sum to one)."""
    import torch
    s = Server.__new__(Server)
    s.M, s.stream = M, torch.cuda.Stream()
    s.ctx = M.mbpt_context_create(stream=s.stream.cuda_stream)
    M.mbpt_set_regularization(s.ctx, 3, 1.0)
    need = M.mbpt_server_workspace_query(s.ctx, 2, 1 << 14)
    s.buf, ptr = M.device_workspace(need)
    s.srv = M.mbpt_server_create(s.ctx, 2, 1 << 14, 4, ptr, need)
    try:
        t = M.mbpt_server_submit(s.srv, 1, 0, 1, 0.16, 0.3, 0.0, 0.0, 1 << 14, 3 << 14)
        s.run()
        r, done, *_ = M.mbpt_server_poll(s.srv, t)
        E, S, E0, S0 = M.mbpt_server_poll_regularized(s.srv, t, 3)
    finally:
        s.close()
    assert done and r.iters_done == 3 and np.isfinite(r.E_per_A) and r.sigma > 0
    # each estimate: sums of 2^14 weights rounded at 2^-53 of their size, variances
    # of a few per cent: 1e-12 relative is 50 times that
    assert np.allclose(E, r.E_per_A, rtol=1e-12, atol=0), (E, r.E_per_A)
    assert E0 == pytest.approx(r.E_per_A, rel=1e-12)


@pytest.mark.parametrize("eta", [1e30, 1e90, 1e300])
@pytest.mark.parametrize("order,did,q", [(2, 0, 2), (3, 1, 4), (4, 7, 4), (5, 50, 2)])
def test_large_shift(M, order, did, q, eta):
    print(f"case reg order={order} q={q} eta={eta}", flush=True)
    count, x = 1500, 0.3 if q == 4 else 0.0
    pb = O.problem(order, did, density=0.16, proton_fraction=x, q=q, seed=1, task_key=7,
                   reg_k=K, reg_eta=eta, label_method=0 if order < 4 or q == 2 else 1)
    grid = O.uniform_grid(3 * (order + 1))
    wo, co = O.sample_values(pb, grid, 0, 0, count)
    wro = O.sample_values_reg(pb, grid, 0, 0, count)
    run = Run(M, [_task(order, did, q, 0.16, x, 7)], max_samples=4096)
    try:
        M.mbpt_set_regularization(run.ctx, K, eta)
        w = M.mbpt_dump_samples(run.set, 0, 0, 0, count)
        wr = M.mbpt_dump_samples_reg(run.set, 0, 0, 0, count, K)
    finally:
        run.close()
    _check_samples(w, wo, co, (order, q, eta))
    # as accurate as w relative to its own size: the factor between them is a
    # product of denominators, whose condition numbers are in W_cond
    ratio = np.abs(wro) / np.where(wo != 0, np.abs(wo), np.inf)[:, None]
    bound = TOL * co[:, None] * ratio + 1e-300
    assert (np.abs(wr - wro) <= bound).all(), (order, q, eta)
