"""The workspace holds what a solve's sweeps use: no volume integral where one
sweep per stage does without."""
import pytest

import workloads as W
from paper_2404_12703_amd import binding as B


def _bytes(E, N, **kw):
    return B.workspace_bytes(W.params(N, node_type=1, **kw), E)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("N", [2, 5, 7])
def test_volume_integral(N, precision):
    E, vol = 1000, 5 * 1000 * (N + 1) ** 3 * (4 if precision else 8)
    euler = _bytes(E, N, viscous=0, mu=0.0, precision=precision)
    one = _bytes(E, N, viscous=0, mu=0.0, shock=1, precision=precision)
    smooth = _bytes(E, N, viscous=0, mu=0.0, shock=1, alpha_smooth=1, precision=precision)
    assert 0 < one - euler <= 4 * (E + 2) + 255  # the list of the blend pass
    assert 0 <= smooth - one - vol <= 255
    assert 0 <= _bytes(E, N, viscous=0, mu=0.0, volume_flux=1, precision=precision) - euler - vol <= 255
