"""1D Euler lines by who does what: batches with fewer tiles than workgroups and more, and the
resident solver's rounds of four segments, the last one full or of one segment.  Bit for bit
the same line alone on the streaming sweeps, which test_gpu_line.py checks against the oracle."""
import numpy as np
import pytest

from paper_2108_12742_amd import workloads as W
from tests import parity as PT

pytestmark = pytest.mark.gpu

STEPS, CFL = 4, 0.3


def _problem(E, n, order):
    return E.make_problem("euler1d", n, 1, order, x_lo=0.0, x_hi=1.0, bc_x="transmissive")


def _alone(torch, E, n, order, resident=False):
    E.enoao_set_resident(resident)
    E.enoao_set_coop(False)
    try:
        u = PT.to_dev(torch, W.riemann_1d(n, n).u0)
        E.enoao_solve(E.enoao_plan_create(_problem(E, n, order)), u, 1e300, cfl=CFL, max_steps=STEPS)
        return u.cpu().numpy()
    finally:
        E.enoao_set_resident(True)
        E.enoao_set_coop(True)


@pytest.mark.parametrize("order", [5, 7])
@pytest.mark.parametrize("resident", [False, True])
@pytest.mark.parametrize("count,least,most", [(3, 1, 130), (20, 130, 1500), (60, 253, 600), (200, 300, 1800)])
def test_batch_of_lines(count, least, most, resident, order):
    torch = PT.torch_cuda()
    from paper_2108_12742_amd import enoao as E
    print(f"[shares] {count} lines of {least} to {most} resident {resident} order {order}", flush=True)
    sizes = [int(n) for n in np.linspace(least, most, count)]
    E.enoao_set_resident(resident)
    try:
        batch = E.enoao_batch_create([_problem(E, n, order) for n in sizes])
        us = [PT.to_dev(torch, W.riemann_1d(n, n).u0) for n in sizes]
        E.enoao_batch_step(batch, us, STEPS, CFL)
        E.enoao_batch_query(batch, raise_on_failure=True)
    finally:
        E.enoao_set_resident(True)
    for i in sorted({0, count // 3, count // 2, count - 1}):
        assert np.array_equal(us[i].cpu().numpy(), _alone(torch, E, sizes[i], order)), sizes[i]


@pytest.mark.parametrize("order", [5, 7])
@pytest.mark.parametrize("n", [1, 63, 64, 252, 253, 315, 316, 504, 505, 567])
def test_rounds_of_a_line(n, order):
    torch = PT.torch_cuda()
    from paper_2108_12742_amd import enoao as E
    print(f"[shares] line of {n} order {order}", flush=True)
    assert np.array_equal(_alone(torch, E, n, order, resident=True), _alone(torch, E, n, order))
