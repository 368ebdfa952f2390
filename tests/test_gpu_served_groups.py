"""Streams of requests that share a group and differ in what chooses an
instance of its kernels: both Riemann solvers, both viscosity laws, curved
meshes and boxes, in every form of the operator.  Each request has the bits of
the same solve alone, in whatever company and order it arrives."""
import itertools

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

FORMS = {
    "gauss": dict(node_type=0, mu=1e-2),
    "lobatto": dict(node_type=1, mu=1e-2),
    "euler gauss": dict(node_type=0, viscous=0, mu=1e-2),
    "euler lobatto": dict(node_type=1, viscous=0, mu=1e-2),
    "split": dict(node_type=1, mu=1e-2, volume_flux=1),
    "shock": dict(node_type=1, mu=1e-2, shock=1),
    "euler shock": dict(node_type=1, viscous=0, mu=1e-2, shock=1),
}


def _serve(cases, N, seed):
    """cases: (mesh size, curved, parameters); every request against its own solve"""
    import paper_2404_12703_amd as P
    jobs = []
    for i, (K, curved, p) in enumerate(cases):
        m = W.box_mesh(K, 0.0, 2 * np.pi, N if curved else 1, amp=0.05 if curved else 0.0, rotate=True, seed=i)
        X = m.points(W.gl_points(N) if p["nodes"] == 0 else W.lgl_points(N))
        U = W.random_smooth_state(X, i, 1.4, m.period)
        if p["shock_capturing"]:
            U[4, ::5, : U.shape[2] // 2] *= 1.3
        s = P.Solver(p, m)
        s.set_state(U)
        dt = 0.3 * s.stable_dt(0.9, 0.9)
        s.advance(3, dt)
        jobs.append((p, m, U, dt, s.state()))
    server = P.Server(256 << 20, 256 << 20, max_active=len(jobs))
    ids = {}
    for i in np.random.default_rng(seed).permutation(len(jobs)):
        p, m, U, dt, _ = jobs[i]
        ids[int(i)] = server.submit(p, m, U, 3, dt)
    server.run()
    for i, (p, m, U, dt, alone) in enumerate(jobs):
        assert np.isfinite(alone).all()
        assert np.array_equal(server.fetch(ids[i])[0], alone), (i, m.amp, p["riemann"], p["viscosity"], p["precision"])


@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("N", [3, 5, 6, 7])
def test_mixed_stream(N, form):
    cases = [((2 + i % 2, 2, 2), curved, W.params(N, riemann=rs, viscosity=law, T_ref=0.9, precision=precision, **FORMS[form]))
             for i, (curved, rs, law, precision) in enumerate(itertools.product((False, True), (0, 1), (0, 1), (0, 1)))]
    _serve(cases, N, 3)


@pytest.mark.parametrize("N,K", [(1, (12, 12, 12)), (2, (9, 8, 8))])
def test_euler_group_above_one_workgroup_per_cu(N, K):
    """Lobatto nodes: each request below, the group above the size from which the traces are recomputed"""
    cases = [(K, N > 1, W.params(N, riemann=i % 2, precision=i // 6, **FORMS["euler lobatto"])) for i in range(12)]
    _serve(cases, N, 4)
