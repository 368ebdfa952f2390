"""The dissipation sweep at every degree, both node families, curved meshes:
workgroups of several elements, odd node counts, more elements than one
thread of the final sum takes; FP64 and the mixed form."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("nodes", [0, 1])
@pytest.mark.parametrize("N,K", [(1, (13, 11, 9)), (2, (5, 4, 3)), (3, (3, 2, 3)), (4, (3, 2, 3)), (5, (2, 3, 2)),
                                 (6, (2, 2, 3)), (7, (2, 3, 2)), (8, (2, 2, 2)), (9, (2, 2, 2))])
def test_dissipation(N, K, nodes, precision):
    import paper_2404_12703_amd as P
    m = W.box_mesh(K, 0.0, 2 * np.pi, N, amp=0.05 if N > 1 else 0.0, rotate=True)
    law = 1 - nodes
    p = W.params(N, node_type=nodes, mu=1e-2, viscosity=law, T_ref=0.9, precision=precision)
    X = m.points(W.gl_points(N) if nodes == 0 else W.lgl_points(N))
    U = W.random_smooth_state(X, 6, 1.4, m.period)
    s = P.Solver(p, m)
    s.set_state(U)
    ref = O.Oracle(p, m).dissipation(U)
    d = s.dissipation()
    # FP64: round-off of sums of squares; mixed: squares of FP32 gradients, whose bound is 1e-5
    assert np.all(np.abs(d - ref) <= (1e-12 if precision == 0 else 4e-5) * np.abs(ref))
    assert np.array_equal(d, s.dissipation()) and np.array_equal(d, s.dissipation_noalloc())
    assert np.array_equal(s.state(), U)
