"""Strong pressure jumps (ratios of 1e3 to 1e8).  A selected flux is formed from the chosen
candidates and the face's own two nodes: were it formed as a distance from the candidate
that was rejected because its window crosses the jump, the rounding of the large side would
reach the small one, magnified by the small side's eigenvectors.  Evaluations and steps
against the oracle (parity.RTOL, as for every other case), every solver, and in conserved
components L exactly zero where a cell and the cells beside it hold one state.  (A
characteristic field whose speed is alpha on both sides has a jump of rounding size alone,
and takes the top candidate across it.)"""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2108_12742_amd import workloads as W
from tests import parity as PT

pytestmark = pytest.mark.gpu

RATIOS = [1e3, 1e5, 1e8]
METHODS = [(5, "characteristic"), (7, "characteristic"), (5, "component"), (7, "component")]


def _evaluate(torch, E, ep_rec, u0):
    """L (checked against the oracle) of a recording plan."""
    plan = E.enoao_plan_create(ep_rec)
    L = torch.full(u0.shape, float("nan"), dtype=torch.float64, device="cuda")
    E.enoao_rhs(plan, PT.to_dev(torch, u0), L)
    L = L.cpu().numpy()
    PT.check_rhs(PT.oracle_problem(ep_rec), u0, L, E.enoao_get_selection(plan))
    return plan, L


def _quiet(u0):
    """cells that hold the same state as the cells beside them"""
    same = np.ones(u0.shape[1:], bool)
    for axis in (1, 2):
        d = (np.diff(u0, axis=axis) == 0.0).all(0)
        pad = [(0, 0), (0, 0)]
        pad[axis - 1] = (1, 0)
        same &= np.pad(d, pad, constant_values=True)
        pad[axis - 1] = (0, 1)
        same &= np.pad(d, pad, constant_values=True)
    return same


@pytest.mark.parametrize("order,recon", METHODS)
@pytest.mark.parametrize("ratio", RATIOS)
@pytest.mark.parametrize("at", [62, 251])  # across a segment's end, across a workgroup's
def test_line_jump(at, ratio, order, recon):
    torch = PT.torch_cuda()
    from paper_2108_12742_amd import enoao as E
    print(f"[jump] line at {at} ratio {ratio:.0e} order {order} {recon}", flush=True)
    n = 300
    one = np.ones(n)
    kw = dict(x_lo=0.0, x_hi=1.0, bc_x="transmissive", recon_vars=recon)
    ep, ep_rec = (E.make_problem("euler1d", n, 1, order, record_selection=r, **kw) for r in (False, True))
    op = PT.oracle_problem(ep)
    for p in (np.where(np.arange(n) <= at, ratio, 1.0), np.where(np.arange(n) <= at, 1.0, ratio)):
        u0 = W.conserved_1d(one, 0.1 * one, p)[:, None, :]
        plan, L = _evaluate(torch, E, ep_rec, u0)
        assert recon == "characteristic" or (L[:, _quiet(u0)] == 0.0).all()
        dt = O.cfl_dt(op, u0, 0.3)
        got, recs = PT.gpu_step_recorded(torch, E, plan, u0, dt)
        PT.check_step(op, u0, dt, got, recs)
        ends = []
        for resident, coop in ((False, False), (True, False), (False, True)):
            E.enoao_set_resident(resident)
            E.enoao_set_coop(coop)
            try:
                v = PT.to_dev(torch, u0)
                E.enoao_solve(E.enoao_plan_create(ep), v, 1e300, dt_fixed=dt, max_steps=1)
                ends.append(v.cpu().numpy())
            finally:
                E.enoao_set_resident(True)
                E.enoao_set_coop(True)
        for v in ends:
            assert np.array_equal(v, got)


@pytest.mark.parametrize("order,recon", METHODS)
@pytest.mark.parametrize("ratio", RATIOS)
@pytest.mark.parametrize("shape", ["x", "y", "corner"])
def test_grid_jump(shape, ratio, order, recon):
    torch = PT.torch_cuda()
    from paper_2108_12742_amd import enoao as E
    print(f"[jump] grid {shape} ratio {ratio:.0e} order {order} {recon}", flush=True)
    nx, ny = 130, 40
    x, y = np.meshgrid(np.arange(nx), np.arange(ny))
    one = np.ones((ny, nx))
    kw = dict(bc_x="transmissive", bc_y="transmissive", recon_vars=recon)
    ep, ep_rec = (E.make_problem("euler2d", nx, ny, order, record_selection=r, **kw) for r in (False, True))
    op = PT.oracle_problem(ep)
    inside = {"x": x <= 55, "y": y <= 17, "corner": (x <= 55) & (y <= 17)}[shape]
    for p in (np.where(inside, ratio, 1.0), np.where(inside, 1.0, ratio)):
        u0 = W.conserved_2d(one, 0.1 * one, -0.2 * one, p)
        plan, L = _evaluate(torch, E, ep_rec, u0)
        assert recon == "characteristic" or (L[:, _quiet(u0)] == 0.0).all()
        dt = O.cfl_dt(op, u0, 0.3)
        got, recs = PT.gpu_step_recorded(torch, E, plan, u0, dt)
        PT.check_step(op, u0, dt, got, recs)
        for tiles in (0, 4):  # without a record; then with half the rows a wave walks
            plan = E.enoao_plan_create(ep)
            if tiles:
                E.enoao_plan_set_tiles(plan, tiles)
            u = PT.to_dev(torch, u0)
            E.enoao_step(plan, u, dt)
            torch.cuda.synchronize()
            E.enoao_plan_check(plan)
            assert np.array_equal(u.cpu().numpy(), got)
