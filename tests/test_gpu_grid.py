"""The 2D stage kernels (enoao_grid.hip) at the edges of their split of the plane: widths
around a strip's columns (56 at order 5, 54 at order 7) and around the pieces of a listed
row (14 columns), one row and few rows, rough data (nearly every face goes to the
selection, in pieces) and smooth (none does), lists long enough that each wave takes an
entry of its own.  Tolerances: parity.RTOL, as for every other 2D case."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2108_12742_amd import workloads as W
from tests import parity as PT

pytestmark = pytest.mark.gpu

# nx, ny, rough data, boundary
SHAPES = [(1, 1, True, "periodic"), (13, 2, True, "transmissive"), (14, 3, False, "transmissive"),
          (15, 1, True, "periodic"), (42, 6, True, "periodic"), (53, 5, True, "transmissive"),
          (54, 4, True, "periodic"), (55, 7, True, "periodic"), (56, 9, True, "transmissive"),
          (57, 2, True, "transmissive"), (112, 3, True, "periodic"), (113, 8, False, "periodic"),
          (225, 150, True, "transmissive")]


def _state(nx, ny, rough):
    rng = np.random.default_rng(97 * nx + ny)
    x, y = np.meshgrid(np.linspace(0, 2 * np.pi, nx, endpoint=False), np.linspace(0, 2 * np.pi, ny, endpoint=False))
    amp = 0.2 if rough else 0.0
    noise = lambda: amp * rng.uniform(-1.0, 1.0, (ny, nx))
    eps = 0.0 if rough else 1e-7
    return W.conserved_2d(1.0 + eps * np.sin(x) * np.cos(y) + noise(), 0.3 + noise(), -0.2 + noise(),
                          1.0 + eps * np.cos(x + y) + noise())


@pytest.mark.parametrize("order,recon", [(5, "characteristic"), (7, "characteristic"), (5, "component"), (7, "component")])
@pytest.mark.parametrize("nx,ny,rough,bc", SHAPES)
def test_stage_at_strip_edges(nx, ny, rough, bc, order, recon):
    torch = PT.torch_cuda()
    from paper_2108_12742_amd import enoao as E
    print(f"[grid] {nx}x{ny} rough={rough} {bc} order {order} {recon}", flush=True)
    ep = E.make_problem("euler2d", nx, ny, order, bc_x=bc, bc_y=bc, recon_vars=recon)
    ep_rec = E.make_problem("euler2d", nx, ny, order, bc_x=bc, bc_y=bc, recon_vars=recon, record_selection=True)
    op = PT.oracle_problem(ep)
    u0 = _state(nx, ny, rough)
    plan_rec = E.enoao_plan_create(ep_rec)
    L = torch.full((4, ny, nx), float("nan"), dtype=torch.float64, device="cuda")
    E.enoao_rhs(plan_rec, PT.to_dev(torch, u0), L)
    sel = E.enoao_get_selection(plan_rec)
    if rough:
        PT.check_rhs(op, u0, L.cpu().numpy(), sel)
    else:  # L, 1e-7, is a difference of fluxes of 1: rounding alone is 1e-8 of it
        assert O.rhs_replay(op, u0, sel)[3] == 0
    dt = 0.25 * O.cfl_dt(op, u0, 0.3)
    got, recs = PT.gpu_step_recorded(torch, E, plan_rec, u0, dt)
    PT.check_step(op, u0, dt, got, recs)
    # without a record; then with half the rows a wave walks
    for tiles in (0, 4):
        plan = E.enoao_plan_create(ep)
        if tiles:
            E.enoao_plan_set_tiles(plan, tiles)
        u = PT.to_dev(torch, u0)
        E.enoao_step(plan, u, dt)
        torch.cuda.synchronize()
        E.enoao_plan_check(plan)
        assert np.array_equal(u.cpu().numpy(), got)
