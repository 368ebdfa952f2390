"""GPU parity of the Euler sweep's two orders of loads with the oracle: meshes
from one workgroup per CU on, where Lobatto nodes at N <= 2 recompute their
traces; last workgroups that the elements do not fill; FP64 and mixed."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


def rel(a, b):
    return float(np.linalg.norm((a - b).ravel()) / np.linalg.norm(b.ravel()))


# 32 elements per workgroup at N = 1, 9 at N = 2: below, at and above 256 workgroups
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nodes", [0, 1])
@pytest.mark.parametrize("N,K", [(1, (20, 20, 20)), (1, (32, 16, 16)), (1, (21, 20, 20)), (2, (13, 13, 13)),
                                 (2, (16, 16, 9)), (2, (17, 13, 11))])
def test_euler_steps(N, K, nodes, precision):
    import paper_2404_12703_amd as P
    m = W.box_mesh(K, 0.0, 2 * np.pi, N, amp=0.05 if N > 1 else 0.0, rotate=True)
    p = W.params(N, node_type=nodes, riemann=nodes, viscous=0, mu=0.0, precision=precision)
    X = m.points(W.gl_points(N) if nodes == 0 else W.lgl_points(N))
    U = W.random_smooth_state(X, 8, 1.4, m.period)
    o, s = O.Oracle(p, m), P.Solver(p, m)
    s.set_state(U)
    # FP64: round-off; mixed: the form's bounds on O(1) states
    assert rel(s.rhs(0.0), o.rhs(U, 0.0)) <= (1e-12 if precision == 0 else 2e-5)
    dt = 0.5 * o.stable_dt(U, 0.9, 0.9)
    s.advance(3, dt)
    assert rel(s.state(), o.advance(U, dt, 3)) <= (1e-12 if precision == 0 else 1e-5)
