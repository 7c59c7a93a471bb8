"""FP32 integrand at cutoffs where the regulator's exponent leaves the range of
a float on both sides (p^n overflows, Lambda^-n underflows): the samples go to
fp64, each within the fp32 tolerance of the oracle."""
import numpy as np
import pytest

import oracle as O

from test_gpu_fp32 import TOL32
from test_gpu_parity import TOL, _task

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


def _denominators(order, did, pb, count):
    """Products of the Yukawa and energy denominators [MeV^(n-1) fm^-4n] of the
    uniform grid's first samples, from the map and the diagram's lines."""
    d = O.diagram_dict(order, did)
    x, _, _ = O.map_samples(O.uniform_grid(3 * (order + 1)), 3 * (order + 1), 50, 1, 5, 0, 0, count)
    kFn, kFp, Rp = O.fermi_momenta(pb)
    k = []
    for j, l in enumerate(d["loop_line"]):
        R = Rp if d["is_particle"][l] else max(kFn, kFp)
        r, c, az = R * x[:, 3 * j], 2 * x[:, 3 * j + 1] - 1, 2 * np.pi * x[:, 3 * j + 2]
        s = np.sqrt(1 - c * c)
        k.append(r[:, None] * np.stack([s * np.cos(az), s * np.sin(az), c], 1))
    line = [sum(c * kj for c, kj in zip(row, k)) for row in d["coef"]]
    prod = np.ones(count)
    for v in range(order):
        o, i = d["vout"][v], d["vin"][v]
        p, q = (line[o[0]] - line[o[1]]) / 2, (line[i[0]] - line[i[1]]) / 2
        prod *= (((p - q) ** 2).sum(1) + pb.mpi ** 2) * (((p + q) ** 2).sum(1) + pb.mpi ** 2)
    for cut in d["cut"]:
        prod *= pb.hbar2_m / 2 * sum(c * (kl * kl).sum(1) for c, kl in zip(cut, line))
    return np.abs(prod)


@pytest.mark.parametrize("order,did,q,Lambda", [(3, 0, 2, 100.0), (3, 1, 4, 100.0),
                                                (4, 20, 4, 30.0)])
def test_large_denominators_in_fp64(M, order, did, q, Lambda):
    """A sample whose denominators multiply to 1e30 or more is evaluated in fp64:
    its weight is the oracle's to the fp64 tolerance."""
    print(f"case order={order} id={did} q={q} Lambda={Lambda}", flush=True)
    count, x = 20000 if order < 4 else 6000, 0.3 if q == 4 else 0.0
    pb = O.problem(order, did, density=0.16, proton_fraction=x, q=q, seed=1, task_key=5,
                   label_method=0 if order < 4 else 1, Lambda=Lambda)
    wo, co = O.sample_values(pb, O.uniform_grid(3 * (order + 1)), 0, 0, count)
    prod = _denominators(order, did, pb, count)
    # (1e30 and the product as the kernel rounds them in fp32: within 1e-5)
    large = (prod > 1.0001e30) & (wo != 0)
    assert np.count_nonzero(large & (prod < 4e32)) > 50
    ctx = M.mbpt_context_create(precision=M.MBPT_FP32, seed=1)
    try:
        M.mbpt_set_interaction(ctx, Lambda=Lambda)
        s = M.mbpt_create_task_set(ctx, [_task(order, did, q, 0.16, x, 5)])
        nbytes = M.mbpt_workspace_query(s, 4096, 2)
        buf, ptr = M.device_workspace(nbytes)
        M.mbpt_bind_workspace(s, ptr, nbytes, 4096, 2)
        w = M.mbpt_dump_samples(s, 0, 0, 0, count)
        M.mbpt_task_set_destroy(s)
    finally:
        M.mbpt_context_destroy(ctx)
    bad = large & (np.abs(w - wo) > TOL * co + 1e-300)
    assert not bad.any(), (order, did, int(bad.sum()), int(large.sum()))
