"""The sample kernels at the sizes where work items, wavefronts and queues
end: the first iteration (uniform grid) of a task set equals the mean and the
variance of the oracle's weights of the same samples.  The bounds are the
per-sample ones, averaged: |I - mean w| <= mean(tol W_cond), and for the
variance twice that of every |w - mean w|."""
import numpy as np
import pytest

import oracle as O

from test_gpu_parity import Run, _task

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_24532_amd as M
    M.lib()
    return M


def _check_first_iteration(M, cases, N, precision, mode, block, spt):
    tasks = [_task(o, d, q, n, x, 11 + k) for k, (o, d, q, n, x) in enumerate(cases)]
    run = Run(M, tasks, max_samples=max(N, 2), mode=mode, block=block, spt=spt,
              precision=M.MBPT_FP32 if precision == "fp32" else M.MBPT_FP64)
    try:
        per, _ = M.mbpt_integrate(run.set, N, 1)
        logs = [M.mbpt_iteration_log(run.set, k) for k in range(len(tasks))]
    finally:
        run.close()
    tol = 1e-5 if precision == "fp32" else 1e-12
    for k, (o, d, q, n, x) in enumerate(cases):
        pb = O.problem(o, d, density=n, proton_fraction=x, q=q, seed=1, task_key=11 + k,
                       label_method=1 if q == 4 and o >= 4 else 0)
        w, cond = O.sample_values(pb, O.uniform_grid(3 * (o + 1)), 0, 0, N)
        I, V = logs[k][0][0], logs[k][1][0]
        slack = 1e-14 * np.abs(w).mean() + 1e-300
        assert per[k].n_evals == N
        assert abs(I - w.mean()) <= tol * cond.mean() + slack, (o, d, q, x, I, w.mean())
        dev = w - w.mean()
        want = (dev * dev).mean() / (N - 1)
        bound = 2 * (np.abs(dev) * (tol * (cond + cond.mean()) + slack)).mean() / (N - 1)
        bound += 1e-12 * ((w * w).mean() / (N - 1)) + (tol * cond).max() ** 2 / (N - 1)
        assert abs(V - want) <= bound, (o, d, q, x, V, want)


ALL4 = [(4, d, 4, 0.16, (0.0, 0.25, 0.5, 0.8)[d % 4]) for d in range(39)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("mode,N,block,spt", [(0, 257, 256, 1), (1, 2, 64, 1), (1, 2049, 256, 16)])
def test_every_fourth_order_diagram(M, precision, mode, N, block, spt):
    """All 39 diagrams through the kernel that holds them, one launch per task
    and one launch for all, at proton fractions 0 to 0.8."""
    print(f"case all o4 {precision} mode={mode} N={N}", flush=True)
    _check_first_iteration(M, ALL4, N, precision, mode, block, spt)


@pytest.mark.parametrize("order,did,nb,alpha", [
    (2, 0, 2, 1.5), (2, 0, 3, 0.7), (2, 0, 63, 1.5), (2, 0, 64, 1.5), (2, 0, 65, 1.5),
    (2, 0, 128, 0.7), (5, 42, 50, 1.5)])
def test_refined_grid(M, order, did, nb, alpha):
    """The grid after one iteration at the edges of the refinement's lanes (64
    bins to a half) and waves (fifth order: 18 dimensions on 16 waves), at the
    default compression exponent and another.  Histogram and edges are sums of
    at most 10^4 rounded terms: 1e-10 absolute on edges in [0, 1]."""
    N = 9001
    print(f"case grid order={order} nb={nb} alpha={alpha}", flush=True)
    ctx = M.mbpt_context_create(n_bins=nb, alpha=alpha)
    try:
        s = M.mbpt_create_task_set(ctx, [_task(order, did, 2, 0.12, 0.0, 5)])
        nbytes = M.mbpt_workspace_query(s, N, 2)
        buf, ptr = M.device_workspace(nbytes)
        M.mbpt_bind_workspace(s, ptr, nbytes, N, 2)
        M.mbpt_integrate(s, N, 1)
        got = M.mbpt_get_grid(s, 0, 3 * (order + 1), nb)
        M.mbpt_task_set_destroy(s)
    finally:
        M.mbpt_context_destroy(ctx)
    pb = O.problem(order, did, density=0.12, seed=1, task_key=5, n_bins=nb, alpha=alpha)
    _, _, _, edges = O.integrate(pb, N, 1)
    assert np.abs(got - np.ravel(edges)).max() < 1e-10


@pytest.mark.parametrize("ntasks", [1, 90, 400, 1300])
def test_staged_copies(M, ntasks):
    """Parameters, tables and results of sets below and above the staging of the
    copies: every task's first iteration (a uniform grid: no histogram, whose
    atomic sums have no fixed order, has entered yet) is the same as alone, the
    same stream of samples summed in the same order, so equal. Parameters uploaded again and again without a
    wait go through the staging several times over."""
    ctx = M.mbpt_context_create(seed=5)

    def integrate(tasks):
        s = M.mbpt_create_task_set(ctx, tasks)
        M.mbpt_set_blocking(s, 256, 4)
        nbytes = M.mbpt_workspace_query(s, 2048, 3)
        buf, ptr = M.device_workspace(nbytes)
        M.mbpt_bind_workspace(s, ptr, nbytes, 2048, 3)
        for k in range(40):
            M.mbpt_set_training(s, k % 2)
        M.mbpt_set_density(s, 0.12)
        per, _ = M.mbpt_integrate(s, 2048, 3)
        out = []
        for k, r in enumerate(per):
            assert r.iters_done == 3 and r.n_evals == 3 * 2048
            log = M.mbpt_iteration_log(s, k)
            out.append((log[0][0], log[1][0]))
        M.mbpt_task_set_destroy(s)
        del buf
        return out

    tasks = [(2, 0, M.MBPT_NEUTRON, 0.16, 0.0, k, 0) for k in range(ntasks)]
    out = integrate(tasks)
    assert len(set(out)) == ntasks
    for k in sorted({0, ntasks // 2, ntasks - 1}):
        assert integrate(tasks[k:k + 1])[0] == out[k]
    M.mbpt_context_destroy(ctx)
