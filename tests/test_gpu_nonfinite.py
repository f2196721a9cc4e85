"""A NaN in one node stays where the selection leaves it: a face that does not touch the
node chooses candidates whose stencils avoid it, so on a constant state L is zero to
rounding except in the cells that share a face with the node.  The bound that spares most
faces the selection must not overlook a NaN in its window."""
import numpy as np
import pytest

from paper_2108_12742_amd import workloads as W
from tests import parity as PT

pytestmark = pytest.mark.gpu

METHODS = [(5, "characteristic"), (7, "characteristic"), (5, "component"), (7, "component")]


@pytest.mark.parametrize("order,recon", METHODS)
@pytest.mark.parametrize("ny", [1, 30])
@pytest.mark.parametrize("components", [slice(0, None), slice(-1, None), slice(0, 1)], ids=["all", "energy", "density"])
def test_nan_in_one_node(components, ny, order, recon):
    torch = PT.torch_cuda()
    from paper_2108_12742_amd import enoao as E
    print(f"[nan] ny {ny} {components} order {order} {recon}", flush=True)
    nx, x, y = 130, 60, ny // 2
    one = np.ones((ny, nx))
    u = W.conserved_1d(one[0], 0.3 * one[0], one[0])[:, None, :] if ny == 1 else \
        W.conserved_2d(one, 0.3 * one, -0.2 * one, one)
    u = np.array(u)
    u[components, y, x] = np.nan
    kw = dict(x_lo=0.0, x_hi=1.0, y_lo=0.0, y_hi=1.0, recon_vars=recon)
    plan = E.enoao_plan_create(E.make_problem("euler1d" if ny == 1 else "euler2d", nx, ny, order, **kw))
    L = torch.zeros(u.shape, dtype=torch.float64, device="cuda")
    E.enoao_rhs(plan, PT.to_dev(torch, u), L)
    L = L.cpu().numpy()
    with pytest.raises(RuntimeError):
        E.enoao_plan_check(plan)
    far = np.ones((ny, nx), bool)
    for dx, dy in ((0, 0), (1, 0), (-1, 0), (0, 1), (0, -1)):
        if 0 <= y + dy < ny:
            far[y + dy, x + dx] = False
    # fluxes of size 4 at most, over dx = 1 / 130 (dy = 1 / 30): their rounding
    assert np.isnan(L[:, ~far]).any()
    assert (np.abs(L[:, far]) <= PT.RTOL * 4 * nx).all(), np.argwhere(~(np.abs(L).max(0) <= PT.RTOL * 4 * nx) & far)


@pytest.mark.parametrize("eq", ["euler1d", "advection"])
def test_cooperative_solver_takes_any_nan(eq):
    """The cooperative solver's workgroups tell an empty word by the bits of a signalling NaN.
    A caller's state may hold those bits, at a workgroup's end, where they are sent to its
    neighbour: a non-physical state like any other."""
    torch = PT.torch_cuda()
    from paper_2108_12742_amd import enoao as E
    n = 1000
    ep = E.make_problem(eq, n, 1, 5, x_lo=0.0, x_hi=1.0)
    u = np.ones((1, 1, n)) if eq == "advection" else W.conserved_1d(*(np.full(n, x) for x in (1.0, 0.3, 1.0)))[:, None, :]
    u = np.ascontiguousarray(u)
    u.view(np.uint64)[-1, 0, 251:253] = 0xFFF7FFFFFFFFFFFF
    for coop in (False, True):
        E.enoao_set_resident(False)
        E.enoao_set_coop(coop)
        try:
            print(f"[nan] cooperative {coop} {eq}", flush=True)
            plan, v = E.enoao_plan_create(ep), PT.to_dev(torch, u)
            with pytest.raises(E.EnoaoError, match="non-physical"):
                E.enoao_solve(plan, v, 1e300, cfl=0.3, max_steps=5)
            assert np.array_equal(v.cpu().numpy().view(np.uint64), u.view(np.uint64))
        finally:
            E.enoao_set_resident(True)
            E.enoao_set_coop(True)
