"""Device memory: a plan takes what enoao_workspace_bytes says, and a pool no more than its
arena (beside its control data)."""
import pytest

from tests import parity as PT

pytestmark = pytest.mark.gpu

SLACK = 4 << 20  # the allocator's granularity, twice


def _taken(torch, make):
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    kept = make()
    torch.cuda.synchronize()
    return before - torch.cuda.mem_get_info()[0], kept


@pytest.mark.parametrize("record", [False, True])
@pytest.mark.parametrize("eq,nx,ny", [("advection", 5000000, 1), ("euler1d", 3000000, 1), ("euler2d", 2048, 2048),
                                      ("euler2d", 1, 1 << 21), ("euler2d", 57, 50000)])
def test_workspace_bytes(eq, nx, ny, record):
    torch = PT.torch_cuda()
    from paper_2108_12742_amd import enoao as E
    print(f"[memory] {eq} {nx} x {ny} record {record}", flush=True)
    ep = E.make_problem(eq, nx, ny, record_selection=record)
    E.enoao_plan_create(ep)  # (what the runtime keeps from the first on)
    taken, plan = _taken(torch, lambda: E.enoao_plan_create(ep))
    assert abs(taken - E.enoao_workspace_bytes(ep)) <= SLACK


@pytest.mark.parametrize("eq,n", [("euler1d", 1000), ("euler2d", 128)])
def test_pool_stays_within_its_arena(eq, n):
    torch = PT.torch_cuda()
    from paper_2108_12742_amd import enoao as E
    like, arena = E.make_problem(eq, n, n if eq == "euler2d" else 1), 4 << 30
    print(f"[memory] pool {eq}", flush=True)
    E.enoao_pool_create(like, 16, 1 << 20)
    taken, pool = _taken(torch, lambda: E.enoao_pool_create(like, 16, arena))
    assert taken <= arena + SLACK
    assert E.enoao_pool_usage(pool)[1] == arena
