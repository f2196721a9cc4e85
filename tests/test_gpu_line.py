"""The 1D Euler fluxes at the edges of their split: lines around a segment's 63 cells and a
workgroup's four segments, rough data (nearly every face goes to the selection: three
passes of a wave, or the workgroup's shared lists) and data with a single jump (a list in
one wave).  The evaluation against the oracle (parity.RTOL, as for every other case), and
the streaming, LDS-resident (waves sharing and not) and cooperative solvers against each
other, which agree bit for bit."""
import numpy as np
import pytest

from paper_2108_12742_amd import workloads as W
from tests import parity as PT

pytestmark = pytest.mark.gpu


def _state(n, rough):
    rng = np.random.default_rng(31 * n + rough)
    x = np.arange(n) / n
    if rough:
        return W.conserved_1d(*(1.0 + 0.2 * rng.uniform(-1.0, 1.0, n) for _ in range(3)))[:, None, :]
    jump = np.where(x < 0.4, 0.0, 0.3)
    return W.conserved_1d(1.0 + jump, 0.2 + 0.0 * x, 1.0 + jump)[:, None, :]


@pytest.mark.parametrize("order,recon", [(5, "characteristic"), (7, "characteristic"), (5, "component"), (7, "component")])
@pytest.mark.parametrize("n,rough", [(1, True), (62, True), (63, False), (64, True), (65, True), (252, True),
                                     (253, False), (505, True), (4000, True)])
def test_line_fluxes_at_segment_edges(n, rough, order, recon):
    torch = PT.torch_cuda()
    from paper_2108_12742_amd import enoao as E
    print(f"[line] {n} rough={rough} order {order} {recon}", flush=True)
    kw = dict(x_lo=0.0, x_hi=1.0, bc_x="transmissive", recon_vars=recon)
    u0 = _state(n, rough)
    ep_rec = E.make_problem("euler1d", n, 1, order, record_selection=True, **kw)
    plan = E.enoao_plan_create(ep_rec)
    u = PT.to_dev(torch, u0)
    L = torch.full_like(u, float("nan"))
    E.enoao_rhs(plan, u, L)
    PT.check_rhs(PT.oracle_problem(ep_rec), u0, L.cpu().numpy(), E.enoao_get_selection(plan))

    ep = E.make_problem("euler1d", n, 1, order, **kw)
    steps, got = 3, {}
    for name in ("streaming", "alone", "batch"):
        E.enoao_set_resident(name != "streaming")
        E.enoao_set_coop(name != "streaming")
        try:
            if name == "batch":  # more members than compute units; a few of this size
                if n > 600:
                    continue
                members = [ep] * 2 + [E.make_problem("euler1d", 8, 1, order, **kw)] * 300
                states = [PT.to_dev(torch, u0) for _ in range(2)] + [PT.to_dev(torch, _state(8, True)) for _ in range(300)]
                E.enoao_batch_step(E.enoao_batch_create(members), states, steps, 0.2)
                assert torch.equal(states[0], states[1])
                v = states[0]
            else:
                v = PT.to_dev(torch, u0)
                E.enoao_solve(E.enoao_plan_create(ep), v, 1e300, cfl=0.2, max_steps=steps)
            torch.cuda.synchronize()
            got[name] = v.cpu().numpy()
        finally:
            E.enoao_set_resident(True)
            E.enoao_set_coop(True)
    for name, v in got.items():
        assert np.array_equal(v, got["streaming"]), name


@pytest.mark.parametrize("eq,bc", [("euler1d", "periodic"), ("euler1d", "transmissive"), ("advection", "periodic")])
@pytest.mark.parametrize("order", [5, 7])
@pytest.mark.parametrize("n", [252, 253, 757, 1263, 2020, 20163])
def test_cooperative_halos(n, order, eq, bc):
    """Workgroups of 252 cells whose last one holds fewer than a halo (1, 3, 4 or 3 cells: a
    halo then spans two workgroups, or wraps), one workgroup alone, and more than a wave of
    them: bit for bit the streaming kernels' result."""
    torch = PT.torch_cuda()
    from paper_2108_12742_amd import enoao as E
    print(f"[coop] {eq} {n} order {order} {bc}", flush=True)
    u0 = _state(n, True) if eq == "euler1d" else 1.0 + np.random.default_rng(n).uniform(-0.5, 0.5, (1, 1, n))
    ep = E.make_problem(eq, n, 1, order, x_lo=0.0, x_hi=1.0, bc_x=bc)
    got = []
    for coop in (False, True):
        E.enoao_set_resident(False)
        E.enoao_set_coop(coop)
        try:
            v = PT.to_dev(torch, u0)
            plan = E.enoao_plan_create(ep)
            E.enoao_profile(plan, True)
            t, steps = E.enoao_solve(plan, v, 1e300, cfl=0.2, max_steps=7)
            torch.cuda.synchronize()
            assert ("coop" in {k for k, (_, c) in E.enoao_profile_read(plan).items() if c}) == coop
            got.append((v.cpu().numpy(), t, steps))
        finally:
            E.enoao_set_resident(True)
            E.enoao_set_coop(True)
    assert np.array_equal(got[0][0], got[1][0]) and got[0][1:] == got[1][1:]


@pytest.mark.parametrize("members", [2, 63, 65, 200])
def test_streaming_batch_chunks(members):
    """Chunks of a streaming batch of uneven members (counts around a wave's width): every
    member as on its own, bit for bit."""
    torch = PT.torch_cuda()
    from paper_2108_12742_amd import enoao as E
    print(f"[batch] {members}", flush=True)
    rng = np.random.default_rng(members)
    sizes = [int(n) for n in np.exp(rng.uniform(np.log(1), np.log(3000), members))]
    kw = dict(x_lo=0.0, x_hi=1.0, bc_x="transmissive")
    probs = [E.make_problem("euler1d", n, 1, 5, **kw) for n in sizes]
    u0 = [_state(n, k % 2 == 0) for k, n in enumerate(sizes)]
    E.enoao_set_resident(False)
    E.enoao_set_coop(False)
    try:
        states = [PT.to_dev(torch, u) for u in u0]
        E.enoao_batch_step(E.enoao_batch_create(probs), states, 3, 0.2)
        for k in {0, members // 2, members - 1, int(np.argmax(sizes)), int(np.argmin(sizes))}:
            v = PT.to_dev(torch, u0[k])
            E.enoao_solve(E.enoao_plan_create(probs[k]), v, 1e300, cfl=0.2, max_steps=3)
            torch.cuda.synchronize()
            assert torch.equal(v, states[k]), (k, sizes[k])
    finally:
        E.enoao_set_resident(True)
        E.enoao_set_coop(True)
