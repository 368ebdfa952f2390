"""Where the set-up stops to take a mesh for one of parallelepipeds, on the
CPU: curving above the rounding of the coordinates is never flattened, however
thin the elements or far the origin, and a recognised mesh keeps the discrete
metric identity at round-off."""
import numpy as np
import pytest

import workloads as W
from test_affine_setup import SHEAR, _run, driver  # noqa: F401


def _layers(h, wave, N):
    """four layers of thickness h over the unit square, displaced by a share of their thickness"""
    m = W.box_mesh((4, 4, 4), 0.0, 1.0, N)
    x = m.x_geo
    x[:, 2] = 4 * h * x[:, 2] + wave * h * np.sin(2 * np.pi * x[:, 0]) * np.cos(2 * np.pi * x[:, 1])
    return m


# amplitudes of 15 to 1e4 roundings of the coordinates
@pytest.mark.parametrize("K,N,amp", [(8, 7, 1e-12), (8, 9, 1e-12), (12, 9, 1e-11), (16, 7, 1e-12), (3, 3, 1e-11)])
def test_slight_curving_is_kept(driver, tmp_path, K, N, amp):  # noqa: F811
    m = W.box_mesh((K, K, K), 0.0, 2 * np.pi, N, amp=amp)
    affine, spread, closure = _run(driver, tmp_path, m, N, 0)
    assert affine == 0 and spread > 0.0
    assert closure <= 1e-11  # the curl form's own residual at these sizes: up to 5e-12


@pytest.mark.parametrize("h", [1e-4, 1e-5])
@pytest.mark.parametrize("N", [3, 5, 7])
def test_thin_layers(driver, tmp_path, N, h):  # noqa: F811
    affine, spread, closure = _run(driver, tmp_path, _layers(h, 0.0, N), N, 0)
    assert affine == 1 and spread == 0.0 and closure <= 1e-12
    affine, spread, closure = _run(driver, tmp_path, _layers(h, 1e-4, N), N, 0)
    assert affine == 0 and spread > 0.0


@pytest.mark.parametrize("amp", [1e-6, 1e-12])
def test_waves_within_an_element(driver, tmp_path, amp):  # noqa: F811
    """every element curved alike: its mean metrics are the flat element's"""
    m = W.box_mesh((4, 4, 4), 0.0, 1.0, 7)
    m.x_geo[:, 2] += amp * np.sin(8 * np.pi * m.x_geo[:, 0])
    affine, spread, _ = _run(driver, tmp_path, m, 7, 0)
    assert affine == 0 and spread > 0.0


@pytest.mark.parametrize("origin", [0.0, 100.0, 1e5])
def test_far_from_the_origin(driver, tmp_path, origin):  # noqa: F811
    m = W.box_mesh((3, 3, 3), 0.0, 1.0, 7)
    x = m.x_geo
    m.x_geo = x + 1e-9 * np.prod(np.sin(2 * np.pi * x), axis=1, keepdims=True) + origin
    affine, _, closure = _run(driver, tmp_path, m, 7, 0)
    assert affine == 0
    assert closure <= max(1e-12, 2.2e-16 * origin * 343)  # eps x/h n_geo^3, without the factor lost between means


@pytest.mark.parametrize("shear", [False, True])
@pytest.mark.parametrize("K", [(3, 2, 4), (2, 2, 40), (12, 12, 12)])
@pytest.mark.parametrize("N,ngeo", [(1, 1), (3, 3), (5, 1), (7, 7), (9, 9)])
def test_identity_of_recognised_meshes(driver, tmp_path, N, ngeo, K, shear):  # noqa: F811
    m = W.box_mesh(K, 0.0, 2 * np.pi, ngeo)
    if shear:
        m.x_geo = np.einsum("dc,ecg->edg", SHEAR, m.x_geo)
    affine, spread, closure = _run(driver, tmp_path, m, N, 0)
    assert affine == 1 and spread == 0.0
    assert closure <= 1e-12


@pytest.mark.parametrize("N,ngeo", [(1, 1), (4, 4), (7, 1), (9, 9)])
def test_oblique_lattice(driver, tmp_path, N, ngeo):  # noqa: F811
    """all nine metrics nonzero; the box stays its period"""
    m = W.box_mesh((3, 2, 3), 0.0, 2 * np.pi, ngeo, rotate=True)
    m.x_geo = np.einsum("dc,ecg->edg", np.array([[-1.0, -1, 0], [-1, 0, 1], [0, 2, 1]]), m.x_geo)
    affine, spread, closure = _run(driver, tmp_path, m, N, 0)
    assert affine == 1 and spread == 0.0 and closure <= 1e-12
