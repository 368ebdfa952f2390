"""GPU parity of the one-sweep Euler kernel with the oracle at every degree:
both node families, curved relabelled meshes, workgroups that the last
elements do not fill; with shock capturing, workgroups that mix blended and
plain elements and the indicator's own factors."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


def _case(N, nodes, K, shock=0, riemann=0, alpha_smooth=0):
    m = W.box_mesh(K, 0.0, 2 * np.pi, N, amp=0.05, rotate=True)
    p = W.params(N, node_type=nodes, riemann=riemann, viscous=0, shock=shock, mu=0.0, alpha_smooth=alpha_smooth)
    X = m.points(W.gl_points(N) if nodes == 0 else W.lgl_points(N))
    return m, p, W.random_smooth_state(X, 5, 1.4, m.period)


def _solver(p, m):
    import paper_2404_12703_amd as P
    return P.Solver(p, m)


# K (3, 2, 3): 18 elements, which no workgroup of several elements divides
@pytest.mark.parametrize("nodes", [0, 1])
@pytest.mark.parametrize("N", range(1, 10))
def test_euler_steps(N, nodes):
    m, p, U = _case(N, nodes, (3, 2, 3), riemann=nodes)
    o, s = O.Oracle(p, m), _solver(p, m)
    s.set_state(U)
    assert rel(s.rhs(0.0), o.rhs(U, 0.0)) <= 1e-12
    dt = o.stable_dt(U, 0.9, 0.9)
    s.advance(3, dt)
    assert rel(s.state(), o.advance(U, dt, 3)) <= 1e-12


@pytest.mark.parametrize("smooth", [0, 1])
@pytest.mark.parametrize("N", range(2, 8))
def test_euler_shock(N, smooth):
    """frozen factors, some zero; then the indicator's (smoothed: two sweeps)"""
    m, p, U = _case(N, 1, (3, 2, 3), shock=1, alpha_smooth=smooth)
    U = U.copy()
    U[4, ::5, : U.shape[2] // 2] *= 1.5  # jumps that the indicator sees
    o, s = O.Oracle(p, m), _solver(p, m)
    alpha = np.zeros(m.n_elems)
    alpha[::4] = np.random.default_rng(2).uniform(0.2, 1.0, len(alpha[::4]))
    o.set_alpha(alpha)
    s.set_alpha(alpha)
    s.set_state(U)
    assert rel(s.rhs(0.0), o.rhs(U, 0.0)) <= 1e-12
    assert np.array_equal(s.alpha(), alpha)
    o.set_alpha(None)
    s.set_alpha(None)
    Rg, Ro = s.rhs(0.0), o.rhs(U, 0.0)
    ag, ao = s.alpha(), o.alpha()
    assert (ao > 0).any() and np.array_equal(ag > 0, ao > 0)
    assert np.abs(ag - ao).max() <= 1e-10
    assert rel(Rg, Ro) <= 1e-10  # the factors' own difference enters
    dt = 0.5 * o.stable_dt(U, 0.9, 0.9)
    s.advance(2, dt)
    assert rel(s.state(), o.advance(U, dt, 2)) <= 1e-11
