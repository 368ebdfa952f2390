"""GPU parity of the kernels' parallelepiped path with the oracle: box and
stretched box meshes, relabelled, at every degree, both node families,
Sutherland's law, workgroups that the last elements do not fill, and the other
operators (Euler, split form, blend), which read one node's metrics.  (The mixed
form has no such path: its case holds it to its bound on the same meshes.)"""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


def _mesh(N, ngeo, shear):
    m = W.box_mesh((3, 2, 3), 0.0, 2 * np.pi, ngeo, rotate=True)
    if shear:
        # x' = S x keeps the box periodic along the columns of S; the oracle
        # matches faces modulo a box, so only box-preserving stretches here
        m.x_geo = m.x_geo * np.array([1.0, 0.7, 1.6])[None, :, None]
        m.period = m.period * np.array([1.0, 0.7, 1.6])
    return m


def _both(p, m, U):
    import paper_2404_12703_amd as P
    o, s = O.Oracle(p, m), P.Solver(p, m)
    s.set_state(U)
    return o, s


def _state(m, N, nodes):
    X = m.points(W.gl_points(N) if nodes == 0 else W.lgl_points(N))
    return W.random_smooth_state(X, 4, 1.4, 2 * np.pi * np.ones(3))


@pytest.mark.parametrize("nodes", [0, 1])
@pytest.mark.parametrize("N", range(1, 10))
def test_viscous_steps(N, nodes):
    """the affine volume sweep; ngeo = N as well as 1, a stretched box, Sutherland's law on Lobatto nodes"""
    m = _mesh(N, N if nodes else 1, nodes)
    p = W.params(N, node_type=nodes, riemann=1 - nodes, mu=1e-2, viscosity=nodes, T_ref=0.9)
    U = _state(m, N, nodes)
    o, s = _both(p, m, U)
    assert rel(s.rhs(0.0), o.rhs(U, 0.0)) <= 1e-12
    d, do = s.dissipation(), o.dissipation(U)
    assert np.all(np.abs(d - do) <= 1e-12 * np.abs(do))
    assert np.all(np.abs(s.integrals() - o.integrals(U)) <= 1e-13 * np.abs(o.integrals(np.abs(U))))
    dt = o.stable_dt(U, 0.9, 0.9)
    assert abs(s.stable_dt(0.9, 0.9) - dt) <= 1e-13 * dt
    s.advance(3, dt)
    assert rel(s.state(), o.advance(U, dt, 3)) <= 1e-12


@pytest.mark.parametrize("N", [1, 3, 5, 7, 9])
def test_viscous_mixed(N):
    m = _mesh(N, 1, 0)
    p = W.params(N, node_type=0, riemann=1, mu=1e-2, precision=1)
    U = _state(m, N, 0)
    o, s = _both(p, m, U)
    # the mixed form's bound on O(1) states at every degree
    assert rel(s.rhs(0.0), o.rhs(U, 0.0)) <= 2e-5


@pytest.mark.parametrize("N", [2, 4, 5, 7])
@pytest.mark.parametrize("form", ["euler", "euler shock", "split", "split shock", "viscous shock"])
def test_other_operators(N, form):
    m = _mesh(N, 1, 1)
    split, shock, visc = int("split" in form), int("shock" in form), int("euler" not in form)
    p = W.params(N, node_type=1, riemann=0, viscous=visc, mu=1e-2, shock=shock, volume_flux=split)
    U = _state(m, N, 1)
    o, s = _both(p, m, U)
    if shock:
        alpha = np.zeros(m.n_elems)
        alpha[::3] = np.random.default_rng(1).uniform(0.1, 1.0, len(alpha[::3]))
        o.set_alpha(alpha)
        s.set_alpha(alpha)
    assert rel(s.rhs(0.0), o.rhs(U, 0.0)) <= 1e-12
