"""The automatic work-item size against the memory it needs: what a workspace
or the static scratch held with items of two blocks per CU, it holds still, and
a bound set can be given those items."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_24532_amd as M
    M.lib()
    return M


def _spread(samples):
    """Samples per thread that leave one task two blocks per CU, at most 16."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return max(1, min(16, samples // (2 * 256 * cus)))


def _set(M, tasks, spt=0, mode=0):
    ctx = M.mbpt_context_create(stream=M.current_stream())
    s = M.mbpt_create_task_set(ctx, tasks)
    M.mbpt_set_launch_mode(s, mode)
    if spt:
        M.mbpt_set_blocking(s, 256, spt)
    return ctx, s


def _bind(M, s, nbytes, samples, iters):
    buf, ptr = M.device_workspace(nbytes)
    M.mbpt_bind_workspace(s, ptr, nbytes, samples, iters)
    return buf


@pytest.mark.parametrize("samples", [20001, (1 << 20) - 1, 1 << 20, 1500007, 1 << 21, 1 << 23])
def test_workspace_of_two_blocks_per_cu(M, samples):
    """A workspace sized for items of two blocks per CU binds without a blocking
    set, and gives the run with those items or larger ones."""
    print(f"case samples={samples}", flush=True)
    tasks = [(2, 0, 1, 0.16, 0.3, 3), (2, 0, 1, 0.12, 0.5, 4)]
    spread = _spread(samples)
    ctx, s = _set(M, tasks, spt=spread)
    try:
        nbytes = M.mbpt_workspace_query(s, samples, 2)
        buf = _bind(M, s, nbytes, samples, 2)
        want, _ = M.mbpt_integrate(s, samples, 1)
    finally:
        M.mbpt_task_set_destroy(s)
        M.mbpt_context_destroy(ctx)
    ctx, s = _set(M, tasks)
    try:
        buf = _bind(M, s, nbytes, samples, 2)
        assert M.mbpt_get_blocking(s)[1] >= spread
        got, _ = M.mbpt_integrate(s, samples, 1)
        for a, b in zip(got, want):
            assert a.E_per_A == pytest.approx(b.E_per_A, rel=1e-13)
            assert a.n_evals == samples
        del buf
        # with the queried size those items can be asked for, none smaller
        # than both sizes
        need = M.mbpt_workspace_query(s, samples, 2)
        buf = _bind(M, s, need, samples, 2)
        auto = M.mbpt_get_blocking(s)[1]
        M.mbpt_set_blocking(s, 256, spread)
        got, _ = M.mbpt_integrate(s, samples, 1)
        for a, b in zip(got, want):
            assert a.E_per_A == b.E_per_A and a.sigma == b.sigma
        if min(auto, spread) > 1:
            with pytest.raises(M.MbptError):
                M.mbpt_set_blocking(s, 256, min(auto, spread) - 1)
    finally:
        M.mbpt_task_set_destroy(s)
        M.mbpt_context_destroy(ctx)


def test_static_scratch_holds_250_tasks(M):
    """250 fourth-order tasks of 2^21 samples fit the static scratch."""
    tasks = [(4, k % 39, 1, 0.16, 0.3, k) for k in range(250)]
    samples = 1 << 21
    ctx, s = _set(M, tasks, mode=1)
    try:
        got, _ = M.mbpt_integrate_noalloc(s, samples, 1)
    finally:
        M.mbpt_task_set_destroy(s)
        M.mbpt_context_destroy(ctx)
    ctx, s = _set(M, tasks, spt=_spread(samples))
    try:
        got_task, _ = M.mbpt_integrate_noalloc(s, samples, 1)
    finally:
        M.mbpt_task_set_destroy(s)
        M.mbpt_context_destroy(ctx)
    ctx, s = _set(M, tasks)
    try:
        auto, _ = M.mbpt_integrate_noalloc(s, samples, 1)
        for a, b, c in zip(got, got_task, auto):
            assert a.n_evals == b.n_evals == c.n_evals == samples
            scale = 1e-13 * (abs(b.E_per_A) + b.sigma)
            assert np.isfinite(a.E_per_A) and abs(a.E_per_A - b.E_per_A) <= scale
            assert abs(c.E_per_A - b.E_per_A) <= scale
    finally:
        M.mbpt_task_set_destroy(s)
        M.mbpt_context_destroy(ctx)


def test_larger_sets_than_the_scratch_stay_refused(M):
    ctx, s = _set(M, [(4, k % 39, 1, 0.16, 0.3, k) for k in range(400)])
    try:
        with pytest.raises(M.MbptError):
            M.mbpt_integrate_noalloc(s, 1 << 21, 1)
    finally:
        M.mbpt_task_set_destroy(s)
        M.mbpt_context_destroy(ctx)


@pytest.mark.parametrize("points,blocks,most", [(1, 1, 1), (1, 4, 2), (3, 1, 2), (15, 1, 4),
                                                (3, 4, 4), (1, 16, 4)])
def test_groups_take_small_items(M, points, blocks, most):
    """Sets of the four fourth-order groups (3, 22, 13 and 1 members): a launch
    waits for the items of the largest, so its items are at most a quarter of
    the launch in units of the largest group's samples (two samples per thread
    below twelve)."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    samples = 256 * cus * blocks
    sizes = [len(M.mbpt_group_members(4, p)) for p in range(4)]
    assert sizes == [3, 22, 13, 1]
    tasks = [(4, p, 1, 0.16, 0.3, 4 * k + p, 1) for k in range(points) for p in range(4)]
    ctx, s = _set(M, tasks, mode=1)
    try:
        buf = _bind(M, s, M.mbpt_workspace_query(s, samples, 1), samples, 1)
        assert M.mbpt_get_blocking(s) == (256, most)
        del buf
    finally:
        M.mbpt_task_set_destroy(s)
        M.mbpt_context_destroy(ctx)


@pytest.mark.parametrize("order,did,label_mode,hf", [(3, 1, 1, 0), (4, 20, 1, 0), (4, 20, 0, 1),
                                                     (5, 300, 0, 1)])
def test_costly_samples_take_two_blocks_per_cu(M, order, did, label_mode, hf):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    samples = 256 * cus * 4
    ctx = M.mbpt_context_create(stream=M.current_stream(), label_mode=label_mode, spectrum=hf)
    s = M.mbpt_create_task_set(ctx, [(order, did, 1, 0.16, 0.3, 1)])
    try:
        buf = _bind(M, s, M.mbpt_workspace_query(s, samples, 1), samples, 1)
        assert M.mbpt_get_blocking(s) == (256, 2)
        del buf
    finally:
        M.mbpt_task_set_destroy(s)
        M.mbpt_context_destroy(ctx)
