"""A served request's sums are grouped by the request alone: one iteration of it
(the histogram atomics reorder later ones) gives the same bits alone and in a
server full of requests of its order."""
import pytest

from test_gpu_server import M, Server  # noqa: F401 (M: the fixture)

pytestmark = pytest.mark.gpu

SLOTS = 48


def _first_iteration(M, requests, max_samples):
    s = Server(M, slots=SLOTS, max_samples=max_samples)
    try:
        tickets = [M.mbpt_server_submit(s.srv, *r) for r in requests]
        s.run()
        r, done, *_ = M.mbpt_server_poll(s.srv, tickets[0])
        assert done and r.iters_done == 1 and r.n_evals == requests[0][7]
        return r.E_per_A, r.sigma
    finally:
        s.close()


@pytest.mark.parametrize("order,did,group", [(1, 0, 0), (2, 0, 0), (3, 1, 0), (4, 20, 0),
                                             (5, 300, 0), (3, 1, 1), (4, 2, 1)])
@pytest.mark.parametrize("samples", [1 << 14, 100003, 1 << 18])
def test_same_bits_alone_and_in_company(M, order, did, group, samples):  # noqa: F811
    print(f"case order={order} id={did} group={group} samples={samples}", flush=True)
    differing = []
    for x in (0.05, 0.2, 0.35, 0.5):
        first = (order, did, 1, 0.16, x, 1e-9, 0.0, samples, samples, group)
        other = (order, did, 1, 0.12, x, 1e-9, 0.0, samples, samples, group)
        alone = _first_iteration(M, [first], 1 << 18)
        assert alone[1] > 0.0
        if _first_iteration(M, [first] + [other] * (SLOTS - 1), 1 << 18) != alone:
            differing.append(x)
    assert not differing
