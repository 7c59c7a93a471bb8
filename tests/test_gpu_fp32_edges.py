"""FP32 integrand at cutoffs where the regulator's exponent leaves the range of
a float on both sides (p^n overflows, Lambda^-n underflows): the samples go to
fp64, each within the fp32 tolerance of the oracle."""
import numpy as np
import pytest

import oracle as O

from test_gpu_fp32 import TOL32
from test_gpu_parity import _task

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_24532_amd as M
    M.lib()
    return M


@pytest.mark.parametrize("order,did,q", [(2, 0, 2), (2, 0, 4), (3, 0, 2), (4, 7, 4)])
@pytest.mark.parametrize("reg_exp,Lambda", [(16, 400.0), (16, 2000.0), (14, 1500.0)])
def test_large_cutoff(M, order, did, q, reg_exp, Lambda):
    print(f"case order={order} q={q} reg_exp={reg_exp} Lambda={Lambda}", flush=True)
    count, x = 3000, 0.3 if q == 4 else 0.0
    pb = O.problem(order, did, density=0.16, proton_fraction=x, q=q, seed=1, task_key=5,
                   label_method=0 if order < 4 else 1, reg_exp=reg_exp, Lambda=Lambda)
    wo, co = O.sample_values(pb, O.uniform_grid(3 * (order + 1)), 0, 0, count)
    assert np.count_nonzero(wo) > 0
    ctx = M.mbpt_context_create(precision=M.MBPT_FP32, seed=1)
    try:
        M.mbpt_set_interaction(ctx, reg_exp=reg_exp, Lambda=Lambda)
        s = M.mbpt_create_task_set(ctx, [_task(order, did, q, 0.16, x, 5)])
        nbytes = M.mbpt_workspace_query(s, 4096, 2)
        buf, ptr = M.device_workspace(nbytes)
        M.mbpt_bind_workspace(s, ptr, nbytes, 4096, 2)
        w = M.mbpt_dump_samples(s, 0, 0, 0, count)
        M.mbpt_task_set_destroy(s)
    finally:
        M.mbpt_context_destroy(ctx)
    assert np.all(np.abs(w - wo) <= TOL32 * co + 1e-300), (order, q, reg_exp, Lambda)
