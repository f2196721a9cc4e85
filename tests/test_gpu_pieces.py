"""The lists of rows with faces to select (enoao_grid.hip): rows with any number of listed
faces, from one to all of a strip's, cut into pieces of at most 32 (ten columns of a narrow
grid), and lists of several members dealt to the waves, short and long.  Against the oracle
(parity.RTOL), and bit for bit between a lone problem and the same one in a batch or a pool."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2108_12742_amd import workloads as W
from tests import parity as PT

pytestmark = pytest.mark.gpu

METHODS = [(5, "characteristic"), (7, "component")]


def _patches(nx, ny):
    """constant but for rough patches, a little wider from row to row and wrapping around: from
    a few listed faces a row to nearly all"""
    rng = np.random.default_rng(1009 * nx + ny)
    x, y = np.meshgrid(np.arange(nx), np.arange(ny))
    rough = ((x - 3 * y) % nx) <= (y * max(nx, 1)) // max(ny, 1)
    noise = lambda: np.where(rough, 0.2 * rng.uniform(-1.0, 1.0, (ny, nx)), 0.0)
    return W.conserved_2d(1.0 + noise(), 0.3 + noise(), -0.2 + noise(), 1.0 + noise())


def _rough(nx, ny):
    rng = np.random.default_rng(1013 * nx + ny)
    noise = lambda: 0.2 * rng.uniform(-1.0, 1.0, (ny, nx))
    return W.conserved_2d(1.0 + noise(), 0.3 + noise(), -0.2 + noise(), 1.0 + noise())


@pytest.mark.parametrize("order,recon", METHODS)
@pytest.mark.parametrize("nx,ny", [(10, 9), (11, 12), (20, 14), (21, 30), (50, 40), (51, 40), (56, 64), (57, 64), (167, 80)])
def test_rows_of_any_length(nx, ny, order, recon):
    torch = PT.torch_cuda()
    from paper_2108_12742_amd import enoao as E
    print(f"[pieces] {nx}x{ny} order {order} {recon}", flush=True)
    u0 = _patches(nx, ny)
    for bc in ("periodic", "transmissive"):
        ep, ep_rec = (E.make_problem("euler2d", nx, ny, order, bc_x=bc, bc_y=bc, recon_vars=recon, record_selection=r)
                      for r in (False, True))
        op = PT.oracle_problem(ep)
        plan = E.enoao_plan_create(ep_rec)
        L = torch.full((4, ny, nx), float("nan"), dtype=torch.float64, device="cuda")
        E.enoao_rhs(plan, PT.to_dev(torch, u0), L)
        PT.check_rhs(op, u0, L.cpu().numpy(), E.enoao_get_selection(plan))
        dt = 0.25 * O.cfl_dt(op, u0, 0.3)
        got, recs = PT.gpu_step_recorded(torch, E, plan, u0, dt)
        PT.check_step(op, u0, dt, got, recs)
        u = PT.to_dev(torch, u0)
        E.enoao_step(E.enoao_plan_create(ep), u, dt)
        assert np.array_equal(u.cpu().numpy(), got)


@pytest.mark.parametrize("order,recon", METHODS)
@pytest.mark.parametrize("sizes", [[(1, 40), (11, 7), (56, 1)], [(1, 90), (57, 3), (300, 200), (12, 1), (56, 300), (40, 40), (700, 400)]],
                         ids=["short", "long"])
def test_lists_of_several_members(sizes, order, recon):
    torch = PT.torch_cuda()
    from paper_2108_12742_amd import enoao as E
    print(f"[pieces] members {sizes} order {order} {recon}", flush=True)
    steps, cfl = 2, 0.05
    probs = [E.make_problem("euler2d", nx, ny, order, recon_vars=recon) for nx, ny in sizes]
    states = [(_rough if i % 3 else _patches)(nx, ny) for i, (nx, ny) in enumerate(sizes)]
    alone = []
    for p, u0 in zip(probs, states):
        u = PT.to_dev(torch, u0)
        E.enoao_solve(E.enoao_plan_create(p), u, 1e300, cfl=cfl, max_steps=steps)
        alone.append(u.cpu().numpy())
    us = [PT.to_dev(torch, u0) for u0 in states]
    batch = E.enoao_batch_create(probs)
    E.enoao_batch_step(batch, us, steps, cfl)
    E.enoao_batch_query(batch, raise_on_failure=True)
    pool = E.enoao_pool_create(probs[0], len(probs), sum(E.enoao_pool_member_bytes(p) for p in probs) + (1 << 16))
    slots = [E.enoao_pool_admit(pool, p, PT.to_dev(torch, u0), max_steps=steps, cfl=cfl) for p, u0 in zip(probs, states)]
    E.enoao_pool_step(pool, steps)
    served = [E.enoao_pool_retire(pool, k, p.shape) for k, p in zip(slots, probs)]
    for a, b, c in zip(alone, us, served):
        assert np.isfinite(a).all()
        assert np.array_equal(a, b.cpu().numpy())
        assert np.array_equal(a, np.asarray(c.cpu() if hasattr(c, "cpu") else c).reshape(a.shape))
