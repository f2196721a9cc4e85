"""How a pool's or batch's list entries are dealt to waves (fix_2d in enoao_grid.hip), written
out again here: every entry once, and no wave with two passes more than another."""
import pytest


def _deal(n, n_two, n_one):
    """entries of each of n waves: those of two passes are 0 .. n_two - 1"""
    each, more = divmod(n_two, n)
    fewer = n - more
    few = n_one <= 2 * fewer
    d, rest = (fewer, n_one) if few else (n, n_one - 2 * fewer)
    each1, more1 = divmod(rest, d)
    waves = []
    for w in range(n):
        k = w - more if few else n - 1 - w
        twos = each + (w < more)
        ones = 0 if few and w < more else each1 + (k < more1) + (0 if few or w < more else 2)
        jump = w * each + min(w, more) + twos
        to = n_two + k * each1 + min(k, more1) + (0 if few else 2 * min(k, fewer))
        waves.append(list(range(jump - twos, jump)) + list(range(to, to + ones)))
    return waves


@pytest.mark.parametrize("n", [1, 2, 3, 7, 16, 60])
def test_every_entry_once_and_evenly(n):
    for n_two in (0, 1, n - 1, n, n + 1, 3 * n + 2, 10 * n):
        for n_one in (0, 1, 2, n, 2 * n - 1, 2 * n, 2 * n + 1, 5 * n + 3):
            waves = _deal(n, n_two, n_one)
            assert sorted(sum(waves, [])) == list(range(n_two + n_one))
            passes = [sum(2 if e < n_two else 1 for e in w) for w in waves]
            assert max(passes) - min(passes) <= 2, (n_two, n_one, passes)
