"""A batch's states are checked together (enoao._dev_ptrs); what is refused, and how, is what
the check of a single state refuses."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")


def _refusals(device):
    good = torch.zeros((3, 1, 8), dtype=torch.float64, device=device)
    yield np.zeros((3, 1, 8)), TypeError
    yield good.float(), TypeError
    yield torch.zeros((3, 1, 16), dtype=torch.float64, device=device)[:, :, ::2], TypeError
    yield torch.zeros((3, 8), dtype=torch.float64, device=device), ValueError
    yield torch.zeros((3, 1, 9), dtype=torch.float64, device=device), ValueError


def test_host_states_are_refused():
    from paper_2108_12742_amd import enoao as E
    for bad in [torch.zeros((3, 1, 8), dtype=torch.float64)] + [b for b, _ in _refusals("cpu")]:
        with pytest.raises(TypeError):
            E._dev_ptrs([bad], [(3, 1, 8)])


def test_fewer_states_than_members_are_refused():
    from paper_2108_12742_amd import enoao as E
    with pytest.raises(ValueError):
        E._dev_ptrs([], [(3, 1, 8)])
    with pytest.raises(ValueError):
        E._dev_ptrs([torch.zeros((3, 1, 8), dtype=torch.float64)], [(3, 1, 8)] * 2)


@pytest.mark.gpu
def test_more_states_than_members():
    from paper_2108_12742_amd import enoao as E
    states = [torch.zeros((3, 1, 8), dtype=torch.float64, device="cuda") for _ in range(3)]
    assert list(E._dev_ptrs(states, [(3, 1, 8)] * 2))[:2] == [u.data_ptr() for u in states[:2]]


@pytest.mark.gpu
def test_refused_states_and_addresses():
    from paper_2108_12742_amd import enoao as E
    good = [torch.zeros((3, 1, n), dtype=torch.float64, device="cuda") for n in (8, 8, 20)]
    shapes = [tuple(u.shape) for u in good]
    assert list(E._dev_ptrs(good, shapes)) == [u.data_ptr() for u in good]
    for bad, error in _refusals("cuda"):
        with pytest.raises(error):
            E._dev_ptrs([good[0], bad, good[2]], shapes)
