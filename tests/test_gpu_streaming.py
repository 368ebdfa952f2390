"""The instances of the sweeps that stream their working set (384 MB and more)
against the others, which the oracle's small meshes reach: many copies of one
small periodic mesh in one solve have to give the bits of the one, stage after
stage, and its dissipation rates.  Euler recomputes its own traces there, the
surface sweep at N = 6 has a form without a loop, and boxes and the dissipation
sweep have instances of their own."""
import copy
import math

import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

STREAM = 384 << 20


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


def _copies(m, R):
    """R copies of the mesh at the same place, each periodic in itself"""
    c, E = copy.copy(m), m.n_elems
    c.K = (m.K[0], m.K[1], m.K[2] * R)
    c.x_geo = np.tile(m.x_geo, (R, 1, 1))
    c.nbr_elem = (m.nbr_elem[None] + E * np.arange(R)[:, None, None]).reshape(R * E, 6)
    c.nbr_face, c.nbr_orient = np.tile(m.nbr_face, (R, 1)), np.tile(m.nbr_orient, (R, 1))
    return c


def _check(N, nodes, curved, **kw):
    import paper_2404_12703_amd as P
    m = W.box_mesh((3, 3, 2), 0.0, 2 * np.pi, N if curved else 1, amp=0.05 if curved and N > 1 else 0.0, rotate=True)
    p = W.params(N, node_type=nodes, **kw)
    U = W.random_smooth_state(m.points(W.gl_points(N) if nodes == 0 else W.lgl_points(N)), 5, 1.4, m.period)
    if p["shock_capturing"]:
        U[4, ::5, : U.shape[2] // 2] *= 1.5  # jumps that the indicator sees
    one = P.Solver(p, m)
    R = math.ceil(STREAM / (P.workspace_bytes(p, 400 * m.n_elems) / 400)) + 1
    while P.workspace_bytes(p, R * m.n_elems) < STREAM:
        R += R // 50 + 1
    many = P.Solver(p, _copies(m, R))
    one.set_state(U)
    many.set_state(np.tile(U, (1, R, 1)))
    if not p["precision"]:
        assert rel(one.rhs(0.0), O.Oracle(p, m).rhs(U, 0.0)) <= (1e-10 if p["shock_capturing"] else 1e-12)
    dt = 0.5 * one.stable_dt(0.9, 0.9)
    one.advance(2, dt)
    many.advance(2, dt)
    V = many.state().reshape(5, R, m.n_elems, -1)
    A = one.state()
    assert all(np.array_equal(V[:, r], A) for r in range(R))
    if p["viscous"]:
        # the copies' equal sums, added in another order
        d, D = np.array(one.dissipation()), np.array(many.dissipation())
        assert np.all(np.abs(d - D) <= 1e-13 * np.abs(d))


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nodes", [0, 1])
@pytest.mark.parametrize("N", range(1, 10))
def test_euler(N, nodes, precision):
    _check(N, nodes, True, riemann=nodes, viscous=0, mu=0.0, precision=precision)


@pytest.mark.parametrize("nodes", [0, 1])
@pytest.mark.parametrize("N", range(1, 10))
def test_viscous_boxes(N, nodes):
    _check(N, nodes, False, riemann=nodes, mu=1e-2, viscosity=nodes, T_ref=0.9)


@pytest.mark.parametrize("riemann", [0, 1])
@pytest.mark.parametrize("nodes", [0, 1])
@pytest.mark.parametrize("N", [5, 6, 7])
def test_viscous_curved(N, nodes, riemann):
    _check(N, nodes, True, riemann=riemann, mu=1e-2)


@pytest.mark.parametrize("N", [3, 6])
@pytest.mark.parametrize("kw", [dict(viscous=0, mu=0.0, shock=1), dict(mu=1e-2, shock=1), dict(mu=1e-2, volume_flux=1)])
def test_shock_and_split(N, kw):
    _check(N, 1, True, riemann=0, **kw)
