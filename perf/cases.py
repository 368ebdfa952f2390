"""Performance cases of the DGSEM Navier-Stokes library: what a program does with it.

Three kinds of pass:

* ``solve``: a solver at hand, a new initial state on the device, ``steps`` Runge-Kutta
  steps, the state read into a device tensor.  From the small solves, where the latency
  of a stage counts, to 16.8 million degrees of freedom; FP64 and mixed precision; Gauss
  and Lobatto nodes, Euler and Navier-Stokes, weak and split form, shock capturing,
  curved and Cartesian boxes, cubic and uneven ones;
* ``analysis``: what a run samples between its steps: the quadrature integrals, the
  dissipation rates and the stable time step of a state;
* ``served``: a batch of independent small solves from host memory through the server.

Everything is made from the seed: the curving of the mesh, the initial state (the
Taylor-Green vortex, the manufactured solution, or a blast, each with a smooth
disturbance of a few per cent in all variables) and the requests.
"""
import math

import numpy as np
import torch
from numpy.polynomial import legendre

import paper_2404_12703_amd as dg

GAMMA, R_GAS = 1.4, 1.0


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _solve(name, K, N, **options):
    case = {"kind": "solve", "Kx": K[0], "Ky": K[1], "Kz": K[2], "N": N, "flow": "tgv", "Ma": 0.1, "Re": 1600.0,
            "curved": False, "nodes": 0, "riemann": 1, "viscous": 1, "precision": 0, "shock": 0, "split": 0,
            "sutherland": 0, "scheme": 0, "steps": 4}
    case.update(options)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # a convergence study's solve: 4096 DOF, 10 steps; all latency
        _solve("mms_4_n3", (4, 4, 4), 3, flow="mms", riemann=0, steps=10),
        # the low-load end of a strong-scaling (PID) curve, one small Taylor-Green solve
        _solve("tgv_4_n7_cartesian", (4, 4, 4), 7, steps=10),
        # one served-size solve alone: about as many workgroups as the GPU holds at once
        _solve("tgv_10_n5_cartesian", (10, 10, 10), 5, Ma=0.2, Re=800.0, steps=5),
        # the middle of the PID curve: a Cartesian box of 2.1 million DOF
        _solve("tgv_16_n7_cartesian", (16, 16, 16), 7),
        # the benchmark workload: the curved 24^3 vortex at N = 7
        _solve("tgv_24_n7_curved", (24, 24, 24), 7, curved=True),
        # the largest: the mixed-precision form on the curved 32^3 mesh
        _solve("tgv_32_n7_mixed", (32, 32, 32), 7, curved=True, precision=1, steps=2),
        # an uneven box at a degree whose element fills a compute unit
        _solve("tgv_13x11x9_n9_curved", (13, 11, 9), 9, curved=True),
        # inviscid flow without shock capturing, odd number of nodes per line
        _solve("euler_27x24x25_n4_curved", (27, 24, 25), 4, curved=True, viscous=0, Ma=0.3),
        # the blast: Euler, Lobatto nodes, indicator and subcell blend
        _solve("blast_28_n5_shock", (28, 28, 28), 5, flow="blast", nodes=1, riemann=0, viscous=0, shock=1),
        # the production scheme: supersonic, split form, Sutherland's law, blend, fourteen stages
        _solve("supersonic_18_n7_split", (18, 18, 18), 7, flow="jump", curved=True, Ma=1.25, nodes=1, riemann=0, shock=1,
               split=1, sutherland=1, scheme=1, steps=1),
        # the samples of a run's log: kinetic energy, dissipation rates, time step
        {"name": "analysis_24_n7", "kind": "analysis", "Kx": 24, "Ky": 24, "Kz": 24, "N": 7, "curved": True, "nodes": 0,
         "precision": 0, "Ma": 0.1, "Re": 1600.0},
        # a burst of requests through the serving loop, host memory to host memory
        {"name": "served_12", "kind": "served", "count": 12, "Kmin": 4, "Kmax": 9, "steps_min": 20, "steps_max": 60,
         "mix": 0, "precision": 0},
    ]


def draw(rng):
    kind = rng.choices(["solve", "analysis", "served"], [8, 1, 1])[0]
    N = rng.choice([1, 2, 3, 3, 4, 5, 5, 6, 7, 7, 7, 8, 9])
    if kind == "served":
        first = rng.randint(20, 40)
        return {"kind": "served", "count": rng.randint(4, 14), "Kmin": 3 + rng.randint(0, 2), "Kmax": rng.randint(6, 9),
                "steps_min": first, "steps_max": first + rng.randint(5, 25), "mix": rng.randint(1, 10 ** 6),
                "precision": rng.choice([0, 0, 1])}
    # sizes over their logarithm, from a few elements to 7 million DOF
    dof = math.exp(rng.uniform(math.log(4000.0), math.log(7.0e6)))
    K = (dof / (N + 1) ** 3) ** (1.0 / 3.0)
    Ks = [max(2, min(40, round(K * rng.uniform(0.8, 1.25)))) for _ in range(3)]
    curved = rng.random() < 0.5 and N > 1
    nodes = rng.choice([0, 0, 1])
    precision = rng.choice([0, 0, 0, 1])
    Ma, Re = round(rng.uniform(0.08, 0.3), 3), round(rng.uniform(400.0, 1600.0), 1)
    if kind == "analysis":
        return {"kind": "analysis", "Kx": Ks[0], "Ky": Ks[1], "Kz": Ks[2], "N": N, "curved": curved, "nodes": nodes,
                "precision": precision, "Ma": Ma, "Re": Re}
    options = {"curved": curved, "nodes": nodes, "precision": precision, "Ma": Ma, "Re": Re,
               "riemann": rng.choice([0, 1, 1]), "steps": rng.randint(1, 4)}
    form = rng.choice(["standard", "standard", "standard", "euler", "mms", "split", "shock", "supersonic"])
    if form == "euler":
        options.update(viscous=0)
    elif form == "mms":
        options.update(flow="mms", riemann=0, curved=False)
    elif form == "split":
        options.update(nodes=1, split=1, precision=0, sutherland=rng.choice([0, 1]))
    elif form in ("shock", "supersonic") and 2 <= N <= 7:
        if form == "shock":
            options.update(flow="blast", nodes=1, riemann=0, viscous=0, shock=1, precision=0, curved=False)
        else:
            options.update(flow="jump", Ma=1.25, nodes=1, riemann=0, shock=1, split=1, sutherland=1, scheme=1, steps=1,
                           precision=0)
    return _solve(None, Ks, N, **options)


# ---------------------------------------------------------------------------
# points and meshes (host) and initial states (device)
# ---------------------------------------------------------------------------
def _gauss(N):
    return legendre.leggauss(N + 1)


def _lobatto(N):
    x = np.array([-1.0, 1.0])
    if N > 1:
        P = legendre.Legendre.basis(N)
        r = np.sort(P.deriv().roots().real)
        for _ in range(3):
            r = r - P.deriv()(r) / P.deriv(2)(r)
        x = np.concatenate([[-1.0], r, [1.0]])
    x = 0.5 * (x - x[::-1])
    return x, 2.0 / (N * (N + 1) * legendre.Legendre.basis(N)(x) ** 2)


def _box(case):
    """corner, side length and number of elements of the periodic box"""
    lo, length = (-1.0, 2.0) if case.get("flow") in ("mms", "blast") else (0.0, 2.0 * math.pi)
    return lo, length, (case["Kx"], case["Ky"], case["Kz"])


def _phases(seed):
    return np.random.default_rng([int(seed), 1]).uniform(0.0, 2.0 * np.pi, (3, 3))


def _points(case, seed, r):
    """node positions [3, E, n, n, n] (xi fastest) of the tensor points of r in every element, on the host"""
    lo, length, K = _box(case)
    n = len(r)
    axes = []
    for d in range(3):
        h = length / K[d]
        axes.append(lo + h * (np.arange(K[d])[:, None] + 0.5 * (np.asarray(r)[None, :] + 1.0)))
    X = np.empty((3, K[2], K[1], K[0], n, n, n))
    X[0] = axes[0][None, None, :, None, None, :]
    X[1] = axes[1][None, :, None, None, :, None]
    X[2] = axes[2][:, None, None, :, None, None]
    if case.get("curved"):
        ph = _phases(seed)
        k = 2.0 * np.pi / length
        s = [[np.sin(k * (axes[d] - lo) + ph[m, d]) for d in range(3)] for m in range(3)]
        for m in range(3):
            X[m] += 0.05 * (s[m][0][None, None, :, None, None, :] * s[m][1][None, :, None, None, :, None]
                            * s[m][2][:, None, None, :, None, None])
    return X.reshape(3, -1, n, n, n)


class _Mesh:
    """what dg.Solver and dg.Server take: geometry nodes and connectivity"""

    def __init__(self, case, seed):
        self.ngeo = case["N"] if case.get("curved") else 1
        r, _ = _lobatto(self.ngeo)
        X = _points(case, seed, r)
        self.n_elems = X.shape[1]
        self.x_geo = np.ascontiguousarray(np.moveaxis(X, 0, 1).reshape(self.n_elems, 3, -1))
        _, _, (Kx, Ky, Kz) = _box(case)
        e = np.arange(self.n_elems).reshape(Kz, Ky, Kx)
        sides = [np.roll(e, -s, axis=2 - d) for d in range(3) for s in (-1, 1)]
        self.nbr_elem = np.ascontiguousarray(np.stack([s.ravel() for s in sides], axis=1))
        self.nbr_face = np.tile(np.array([1, 0, 3, 2, 5, 4], dtype=np.int8), (self.n_elems, 1))
        self.nbr_orient = np.zeros((self.n_elems, 6), dtype=np.int8)


def _initial(case, seed, X):
    """conservative state [5, E, n3] at the positions X [3, E, n, n, n] (a float64 tensor)"""
    lo, length, _ = _box(case)
    rng = np.random.default_rng([int(seed), 2])
    Ma = case.get("Ma", 0.1)
    x, y, z = X[0], X[1], X[2]
    zero = torch.zeros_like(x)
    flow = case.get("flow", "tgv")
    if flow == "mms":
        rho = 2.0 + 0.1 * torch.sin(math.pi * (x + y + z))
        u, v, w, p = 1.0 + zero, 1.0 + zero, 1.0 + zero, rho.clone()
    elif flow == "blast":
        # a pressure ratio of 30 in a ball of radius 0.3: a share of the elements is blended at once
        rho, u, v, w = 1.0 + zero, zero, zero, zero
        p = torch.where(_ball(X, rng, length, 0.15 * length), 30.0 + zero, 1.0 + zero)
    else:
        p0 = 1.0 / (GAMMA * Ma * Ma)
        u = torch.sin(x) * torch.cos(y) * torch.cos(z)
        v = -torch.cos(x) * torch.sin(y) * torch.cos(z)
        w = zero
        p = p0 + (torch.cos(2.0 * x) + torch.cos(2.0 * y)) * (2.0 + torch.cos(2.0 * z)) / 16.0
        rho = p / p0
        if flow == "jump":
            # a supersonic flow's fronts: a ball of doubled pressure blends about 7% of the 18^3 elements
            p = torch.where(_ball(X, rng, length, 0.25 * length), 2.0 * p, p)
    # a smooth periodic disturbance of every variable; the pressure's scales with the flow's, not with p0
    k = 2.0 * math.pi / length
    amp = 0.02
    scale = [rho, 1.0, 1.0, 1.0, p if flow in ("mms", "blast") else 1.0 / GAMMA]
    out = []
    for q, s in zip((rho, u, v, w, p), scale):
        f = zero
        for _ in range(2):
            m = rng.integers(1, 3, 3) * k
            ph = rng.uniform(0.0, 2.0 * np.pi, 3)
            f = f + torch.sin(m[0] * x + ph[0]) * torch.sin(m[1] * y + ph[1]) * torch.sin(m[2] * z + ph[2])
        out.append(q + amp * s * f)
    rho, u, v, w, p = out
    U = torch.stack([rho, rho * u, rho * v, rho * w, p / (GAMMA - 1.0) + 0.5 * rho * (u * u + v * v + w * w)])
    return U.reshape(5, X.shape[1], -1).contiguous()


def _ball(X, rng, length, radius):
    c = rng.uniform(0.0, length, 3)
    d2 = 0.0
    for d in range(3):
        t = X[d] - float(c[d])
        t = t - length * torch.round(t / length)
        d2 = d2 + t * t
    return d2 < radius * radius


def _viscosity(case):
    if case.get("flow") in ("mms", "blast"):
        return 1e-3 if case.get("viscous", 1) else 0.0
    return 1.0 / case["Re"] if case.get("viscous", 1) else 0.0


def _params(case):
    Ma = case.get("Ma", 0.1)
    p0 = 1.0 / (GAMMA * Ma * Ma)
    low_mach = case.get("flow", "tgv") == "tgv"
    return {"N": case["N"], "nodes": case.get("nodes", 0), "riemann": case.get("riemann", 1),
            "precision": case.get("precision", 0), "viscous": case.get("viscous", 1),
            "source": 1 if case.get("flow") == "mms" else 0, "shock_capturing": case.get("shock", 0),
            "gamma": GAMMA, "R": R_GAS, "Pr": 0.71 if case.get("sutherland") else 0.72, "mu": _viscosity(case),
            "ind_a": 0.05 if case.get("flow") == "blast" else 0.5,
            "volume_flux": case.get("split", 0), "viscosity": case.get("sutherland", 0),
            "time_scheme": case.get("scheme", 0), "T_ref": p0 / R_GAS if case.get("sutherland") else 1.0,
            "p_ref": p0 if case.get("precision") and low_mach else 0.0}


def _step(case):
    """a step below the stability limit, from the case alone"""
    lo, length, K = _box(case)
    flow, Ma = case.get("flow", "tgv"), case.get("Ma", 0.1)
    speed = {"mms": 3.0, "blast": 8.0}.get(flow, 1.0 + 1.5 / Ma)
    return 0.5 * length / max(K) / ((2 * case["N"] + 1) * speed * 3.0)


# ---------------------------------------------------------------------------
# prepare and run
# ---------------------------------------------------------------------------
def _requests(case, seed):
    """the requests of a served case: small Cartesian Taylor-Green solves of mixed degree and size (the case's
    mix), each with a flow of its own (the seed's)"""
    mix, rng = np.random.default_rng(case["mix"]), np.random.default_rng([int(seed), 3])
    out = []
    for i in range(case["count"]):
        K = int(mix.integers(case["Kmin"], case["Kmax"] + 1))
        one = _solve(None, (K, K, K), int((3, 5, 7)[i % 3]), Ma=float(rng.uniform(0.05, 0.3)),
                     Re=float(rng.uniform(400.0, 1600.0)), precision=case["precision"],
                     steps=int(mix.integers(case["steps_min"], case["steps_max"] + 1)))
        out.append((one, int(seed) * 100 + i))
    return out


def _nodes(case):
    return _gauss(case["N"]) if case.get("nodes", 0) == 0 else _lobatto(case["N"])


def prepare(case, seed):
    if case["kind"] == "served":
        jobs = []
        for one, s in _requests(case, seed):
            X = torch.from_numpy(_points(one, s, _nodes(one)[0]))
            jobs.append({"params": _params(one), "mesh": _Mesh(one, s), "U0": _initial(one, s, X).numpy(),
                         "steps": one["steps"], "dt": _step(one)})
        return {"kind": "served", "server": dg.Server(1 << 30, 1 << 30, max_active=64), "jobs": jobs}
    solver = dg.Solver(_params(case), _Mesh(case, seed))
    X = torch.from_numpy(_points(case, seed, _nodes(case)[0])).cuda()
    U0 = _initial(case, seed, X)
    state = {"kind": case["kind"], "solver": solver, "U0": U0, "out": torch.empty_like(U0)}
    if case["kind"] == "solve":
        state.update(steps=case["steps"], dt=_step(case))
    return state


def run(state):
    if state["kind"] == "served":
        server = state["server"]
        ids = [server.submit(j["params"], j["mesh"], j["U0"], j["steps"], j["dt"]) for j in state["jobs"]]
        server.run()
        return [server.fetch(i)[0] for i in ids]
    solver = state["solver"]
    solver.set_state(state["U0"], 0.0)
    if state["kind"] == "analysis":
        return {"integrals": solver.integrals(), "dissipation": solver.dissipation(), "dt": solver.stable_dt(0.9, 0.9)}
    solver.advance(state["steps"], state["dt"])
    solver.state_into(state["out"])
    return state["out"]


def work(case):
    """Bytes: per stage the state and the register read and written, the metrics, 1/J and the face
    normals read (the Cartesian boxes' metrics too: a general mesh is what the entry point takes).
    Flops: the contractions of the operator and its pointwise fluxes, about 250 per node and 350 per
    face node."""
    if case["kind"] == "served":
        # each request's mean size and step count
        K = 0.5 * (case["Kmin"] + case["Kmax"])
        parts = [_solve(None, (K, K, K), N, precision=case["precision"],
                        steps=0.5 * (case["steps_min"] + case["steps_max"])) for N in (3, 5, 7)]
        per = [work(p) for p in parts]
        return {k: case["count"] / 3.0 * sum(p[k] for p in per) for k in ("bytes", "flops")}
    n = case["N"] + 1
    dof = case["Kx"] * case["Ky"] * case["Kz"] * n ** 3
    rs = 4 if case.get("precision") else 8
    f = 6.0 / n
    geometry = rs * (10.0 + 3.0 * f)
    if case["kind"] == "analysis":
        # one read of the state and the metrics serves all three samples
        return {"bytes": dof * (40.0 + geometry), "flops": dof * (3 * n * 24 + 150.0)}
    stages = (14 if case["scheme"] else 5) * case["steps"]
    flops = 3 * n * (10.0 + (24.0 if case["viscous"] else 0.0) + (40.0 if case["split"] else 0.0)) + 250.0 + 350.0 * f
    return {"bytes": stages * dof * (160.0 + geometry), "flops": stages * dof * flops}


# ---------------------------------------------------------------------------
# the same in 64 bits, from the method's equations: plain torch
# ---------------------------------------------------------------------------
CK_A = (0.0, -567301805773.0 / 1357537059087.0, -2404267990393.0 / 2016746695238.0,
        -3550918686646.0 / 2091501179385.0, -1275806237668.0 / 842570457699.0)
CK_B = (1432997174477.0 / 9575080441755.0, 5161836677717.0 / 13612068292357.0, 1720146321549.0 / 2090206949498.0,
        3134564353537.0 / 4481467310338.0, 2277821191437.0 / 14882151754819.0)
CK_C = (0.0, 1432997174477.0 / 9575080441755.0, 2526269341429.0 / 6820363962896.0, 2006345519317.0 / 3224310063776.0,
        2802321613138.0 / 2924317926251.0)
ND_A = (0.0, -0.7188012108672410, -0.7785331173421570, -0.0053282796654044, -0.8552979934029281, -3.9564138245774565,
        -1.5780575380587385, -2.0837094552574054, -0.7483334182761610, -0.7032861106563359, 0.0013917096117681,
        -0.0932075369637460, -0.9514200470875948, -7.1151571693922548)
ND_B = (0.0367762454319673, 0.3136296607553959, 0.1531848691869027, 0.0030097086818182, 0.3326293790646110,
        0.2440251405350864, 0.3718879239592277, 0.6204126221582444, 0.1524043173028741, 0.0760894927419266,
        0.0077604214040978, 0.0024647284755382, 0.0780348340049386, 5.5059777270269628)
ND_C = (0.0, 0.0367762454319673, 0.1249685262725025, 0.2446177702277698, 0.2476149531070420, 0.2969311120382472,
        0.3978149645802642, 0.5270854589440328, 0.6981269994175695, 0.8190890835352128, 0.8527059887098624,
        0.8604711817462826, 0.8627060376969976, 0.8734213127600976)


def _lagrange(x, t):
    """M[b, a] = l_a(t_b)"""
    x, t = np.asarray(x, np.longdouble), np.asarray(t, np.longdouble)
    M = np.ones((len(t), len(x)), np.longdouble)
    for a in range(len(x)):
        for c in range(len(x)):
            if c != a:
                M[:, a] *= (t - x[c]) / (x[a] - x[c])
    return M


def _derivative(x):
    x = np.asarray(x, np.longdouble)
    lam = np.array([1.0 / np.prod(x[j] - np.delete(x, j)) for j in range(len(x))])
    D = np.array([[lam[j] / lam[i] / (x[i] - x[j]) if i != j else 0.0 for j in range(len(x))] for i in range(len(x))])
    return D - np.diag(D.sum(axis=1))


def _along(M, f, d):
    """the matrix M along reference direction d of f [..., k, j, i]"""
    if d == 0:
        return f @ M.T
    if d == 1:
        return M @ f
    return (M @ f.reshape(*f.shape[:-2], -1)).reshape(*f.shape[:-3], M.shape[0], *f.shape[-2:])


class _Operator:
    def __init__(self, case, seed, device):
        self.case, N = case, case["N"]
        self.N, self.n = N, N + 1
        self.p = _params(case)
        self.grid = _box(case)[2][::-1]
        t = lambda a: torch.from_numpy(np.asarray(a, np.float64)).to(device)  # noqa: E731
        x, w = _nodes(case)
        self.x, self.w = x, w
        D = _derivative(x)
        lm, lp = _lagrange(x, [-1.0])[0], _lagrange(x, [1.0])[0]
        self.wt = t(w)
        self.D, self.Dhat = t(D), t(-(w[None, :] / w[:, None]) * D.T)
        self.l = (t(lm), t(lp))
        self.lhat = (t(lm / w), t(lp / w))
        # geometry: to the Lobatto points of degree N, the curl form, to the solution points
        mesh = _Mesh(case, seed)
        self.E = mesh.n_elems
        ng = mesh.ngeo + 1
        X = t(mesh.x_geo).reshape(self.E, 3, ng, ng, ng).transpose(0, 1)
        xl, _ = _lobatto(N)
        up, down, DL = t(_lagrange(_lobatto(mesh.ngeo)[0], xl)), t(_lagrange(xl, x)), t(_derivative(xl))
        tensor = lambda M, f: _along(M, _along(M, _along(M, f, 0), 1), 2)  # noqa: E731
        X = X - X.mean(dim=(2, 3, 4), keepdim=True)
        X = tensor(up, X)
        dX = [_along(DL, X, d) for d in range(3)]
        JaL = [[None] * 3 for _ in range(3)]
        for c in range(3):
            m, q = (c + 1) % 3, (c + 2) % 3
            for i in range(3):
                b, e = (i + 1) % 3, (i + 2) % 3
                JaL[i][c] = _along(DL, X[q] * dX[b][m], e) - _along(DL, X[q] * dX[e][m], b)
        self.Ja = [torch.stack([tensor(down, JaL[i][c]) for c in range(3)]) for i in range(3)]
        A = [torch.stack([tensor(down, dX[j][c]) for c in range(3)]) for j in range(3)]
        self.J = (A[0] * torch.linalg.cross(A[1], A[2], dim=0)).sum(0)
        # outward face vectors at the plus faces; the neighbour's minus face has their negative
        self.ns = []
        for d in range(3):
            face = torch.stack([JaL[d][c].select(3 - d, N) for c in range(3)])
            self.ns.append(down @ face @ down.T)

    # ---- neighbours: element e's plus face in direction d is its neighbour's minus face
    def _shift(self, f, d, s):
        g = f.reshape(f.shape[0], *self.grid, *f.shape[2:])
        return torch.roll(g, s, dims=1 + (2 - d)).reshape(f.shape)

    def _trace(self, f, d, side):
        return _along(self.l[side][None, :], f, d).squeeze(4 - d)

    def _lift(self, face, d, side):
        """the face values through l-hat, spread along direction d"""
        shape = [1, 1, 1, 1, 1]
        shape[4 - d] = self.n
        return face.unsqueeze(4 - d) * self.lhat[side].reshape(shape)

    # ---- pointwise physics
    def _prim(self, U):
        rho = U[0]
        u = U[1:4] / rho
        p = (GAMMA - 1.0) * (U[4] - 0.5 * rho * (u * u).sum(0))
        return rho, u, p, p / (rho * R_GAS)

    def _mu(self, T):
        if not self.p["viscosity"]:
            return self.p["mu"]
        th = T / self.p["T_ref"]
        return self.p["mu"] * 1.4042 * th ** 1.5 / (th + 0.4042)

    def _advective(self, U, m):
        """flux along the vector field m"""
        rho, u, p, _ = self._prim(U)
        un = (u * m).sum(0)
        F = U * un
        F[1:4] += p * m
        F[4] += p * un
        return F

    def _viscous(self, u, mu, g, m):
        """viscous flux along m: g[d] the gradients of (u, v, w, T)"""
        G = torch.stack([g[d][:3] for d in range(3)])
        div = G[0, 0] + G[1, 1] + G[2, 2]
        lam = mu * GAMMA * R_GAS / ((GAMMA - 1.0) * self.p["Pr"])
        tau = [sum(mu * (G[d, c] + G[c, d]) * m[d] for d in range(3)) - 2.0 / 3.0 * mu * div * m[c] for c in range(3)]
        heat = lam * sum(g[d][3] * m[d] for d in range(3))
        return torch.stack([torch.zeros_like(div), tau[0], tau[1], tau[2],
                            tau[0] * u[0] + tau[1] * u[1] + tau[2] * u[2] + heat])

    def _llf(self, UL, UR, nv):
        rL, uL, pL, _ = self._prim(UL)
        rR, uR, pR, _ = self._prim(UR)
        lam = torch.maximum((uL * nv).sum(0).abs() + (GAMMA * pL / rL).sqrt(),
                            (uR * nv).sum(0).abs() + (GAMMA * pR / rR).sqrt())
        return 0.5 * (self._advective(UL, nv) + self._advective(UR, nv)) - 0.5 * lam * (UR - UL)

    def _roe(self, UL, UR, nv):
        rL, uL, pL, _ = self._prim(UL)
        rR, uR, pR, _ = self._prim(UR)
        a, b = rL.sqrt(), rR.sqrt()
        u = (a * uL + b * uR) / (a + b)
        H = (a * (UL[4] + pL) / rL + b * (UR[4] + pR) / rR) / (a + b)
        q2 = (u * u).sum(0)
        c = ((GAMMA - 1.0) * (H - 0.5 * q2)).sqrt()
        r, un = a * b, (u * nv).sum(0)
        du, dr, dp = uR - uL, rR - rL, pR - pL
        dun = (du * nv).sum(0)
        one = torch.ones_like(un)
        waves = [((un - c).abs() * (dp - r * c * dun) / (2 * c * c), torch.cat([one[None], u - c * nv, (H - un * c)[None]])),
                 (un.abs() * (dr - dp / (c * c)), torch.cat([one[None], u, (0.5 * q2)[None]])),
                 ((un + c).abs() * (dp + r * c * dun) / (2 * c * c), torch.cat([one[None], u + c * nv, (H + un * c)[None]]))]
        s = du - dun * nv
        waves.append((un.abs() * r, torch.cat([0 * one[None], s, (u * s).sum(0)[None]])))
        return 0.5 * (self._advective(UL, nv) + self._advective(UR, nv)) - 0.5 * sum(f * v for f, v in waves)

    # ---- shock capturing
    def _alpha(self, U):
        rho, _, p, _ = self._prim(U)
        n, N = self.n, self.N
        V = np.stack([math.sqrt(a + 0.5) * legendre.Legendre.basis(a)(self.x) for a in range(n)], axis=1)
        Vi = torch.from_numpy(np.linalg.inv(V)).to(U.device)
        m = _along(Vi, _along(Vi, _along(Vi, rho * p, 0), 1), 2) ** 2
        r = torch.arange(n, device=U.device)
        top = torch.maximum(torch.maximum(r[:, None, None], r[None, :, None]), r[None, None, :])
        total = m.sum((1, 2, 3))
        one, two = (m * (top == N)).sum((1, 2, 3)), (m * (top == N - 1)).sum((1, 2, 3))
        c1 = (m * (top < N)).sum((1, 2, 3))
        E = torch.maximum(one / total, torch.where(c1 > 0, two / c1, 0 * c1))
        T = self.p["ind_a"] * 10.0 ** (-1.8 * n ** 0.25)
        al = 1.0 / (1.0 + torch.exp(-(math.log(9999.0) / T) * (E - T)))
        al = torch.where(al < 1e-3, 0 * al, al)
        return torch.where(al > 1.0 - 1e-3, torch.ones_like(al), al)

    def _subcells(self, U, Ja):
        """the finite-volume subcell operator of the elements given"""
        rho, u, p, _ = self._prim(U)
        q = torch.cat([rho[None], u, p[None]])
        xh = np.concatenate([[-1.0], -1.0 + np.cumsum(self.w)])
        V = torch.zeros_like(U)
        for d in range(3):
            ax = 4 - d
            at = lambda f, i: f.select(ax, i)  # noqa: E731
            dJ = _along(self.D, Ja[d], d)
            acc = at(Ja[d], 0).clone()
            slope = [torch.zeros_like(at(q, 0))] * self.n
            for i in range(1, self.N):
                a = (at(q, i) - at(q, i - 1)) / (self.x[i] - self.x[i - 1])
                b = (at(q, i + 1) - at(q, i)) / (self.x[i + 1] - self.x[i])
                slope[i] = torch.where(a * b > 0, a.sign() * torch.minimum(a.abs(), b.abs()), 0 * a)
            for i in range(self.N):
                acc = acc + self.w[i] * at(dJ, i)
                s = (acc * acc).sum(0).sqrt()
                sides = []
                for k in (i, i + 1):
                    v = at(q, k) + slope[k] * (xh[i + 1] - self.x[k])
                    sides.append(torch.stack([v[0], v[0] * v[1], v[0] * v[2], v[0] * v[3],
                                              v[4] / (GAMMA - 1) + 0.5 * v[0] * (v[1:4] ** 2).sum(0)]))
                F = self._llf(sides[0], sides[1], acc / s) * s
                at(V, i).add_(F / self.w[i])
                at(V, i + 1).sub_(F / self.w[i + 1])
        return V

    # ---- the volume integrals
    def _weak(self, U, Ja):
        return sum(_along(self.Dhat, self._advective(U, Ja[d]), d) for d in range(3))

    def _split(self, U, Ja):
        rho, u, p, T = self._prim(U)
        H = (U[4] + p) / rho
        q = torch.cat([rho[None], u, p[None], H[None]])
        S = self.D + self.Dhat
        V = torch.zeros_like(U)
        for d in range(3):
            ax = 4 - d
            for a in range(self.n):
                m = 0.5 * (Ja[d] + Ja[d].narrow(ax, a, 1))
                h = 0.5 * (q + q.narrow(ax, a, 1))
                f = h[0] * (h[1:4] * m).sum(0)
                F = torch.cat([f[None], f * h[1:4] + h[4] * m, (f * h[5])[None]])
                shape = [1] * 5
                shape[ax] = self.n
                V += S[:, a].reshape(shape) * F
        return V

    # ---- the lifted gradients and the time derivative
    def gradients(self, U):
        _, u, _, T = self._prim(U)
        v = torch.cat([u, T[None]])
        G = [sum(_along(self.Dhat, self.Ja[i][d] * v, i) for i in range(3)) for d in range(3)]
        self.tr = [(self._trace(U, d, 0), self._trace(U, d, 1)) for d in range(3)]
        for d in range(3):
            own, nbr = self.tr[d][1], self._shift(self.tr[d][0], d, -1)
            po, pn = self._prim(own), self._prim(nbr)
            avg = 0.5 * (torch.cat([po[1], po[3][None]]) + torch.cat([pn[1], pn[3][None]]))
            for c in range(3):
                face = avg * self.ns[d][c]
                G[c] = G[c] + self._lift(face, d, 1) - self._lift(self._shift(face, d, 1), d, 0)
        return [g / self.J for g in G]

    def rhs(self, U, t):
        U = U.reshape(5, self.E, self.n, self.n, self.n)
        visc = self.p["viscous"]
        if visc:
            g = self.gradients(U)
        else:
            self.tr = [(self._trace(U, d, 0), self._trace(U, d, 1)) for d in range(3)]
        _, u, _, T = self._prim(U)
        volume = self._split if self.p["volume_flux"] else self._weak
        V = volume(U, self.Ja)
        if self.p["shock_capturing"]:
            al = self._alpha(U)
            at = torch.nonzero(al > 0).flatten()
            if len(at):
                Ub, Jb = U[:, at], [m[:, at] for m in self.Ja]
                V[:, at] += al[at].reshape(1, -1, 1, 1, 1) * (self._subcells(Ub, Jb) - volume(Ub, Jb))
        if visc:
            mu = self._mu(T)
            for d in range(3):
                V = V - _along(self.Dhat, self._viscous(u, mu, g, self.Ja[d]), d)
        for d in range(3):
            UL, UR = self.tr[d][1], self._shift(self.tr[d][0], d, -1)
            s = (self.ns[d] ** 2).sum(0).sqrt()
            nv = self.ns[d] / s
            F = (self._roe if self.p["riemann"] else self._llf)(UL, UR, nv)
            if visc:
                for side, W in ((1, UL), (0, UR)):
                    gt = [self._trace(g[c], d, side) for c in range(3)]
                    if side == 0:
                        gt = [self._shift(h, d, -1) for h in gt]
                    _, uf, _, Tf = self._prim(W)
                    F = F - 0.5 * self._viscous(uf, self._mu(Tf), gt, nv)
            F = F * s
            V = V + self._lift(F, d, 1) - self._lift(self._shift(F, d, 1), d, 0)
        R = -V / self.J
        if self.p["source"]:
            c = 0.1 * math.pi * torch.cos(math.pi * (self.X.sum(0) - t))
            for k, f in enumerate((2.0, 3.0, 3.0, 3.0, 2.0 * (3.0 * GAMMA - 2.0) / (GAMMA - 1.0))):
                R[k] += f * c
        return R.reshape(5, self.E, -1)


def _exact_solve(case, seed, device):
    op = _Operator(case, seed, device)
    op.X = torch.from_numpy(_points(case, seed, _nodes(case)[0])).to(device)
    U = _initial(case, seed, op.X)
    A, B, C = (ND_A, ND_B, ND_C) if case["scheme"] else (CK_A, CK_B, CK_C)
    dt, du = _step(case), torch.zeros_like(U)
    for s in range(case["steps"]):
        for a, b, c in zip(A, B, C):
            du = a * du + dt * op.rhs(U, (s + c) * dt)
            U = U + b * du
    return U


def _exact_analysis(case, seed, device):
    op = _Operator(case, seed, device)
    X = torch.from_numpy(_points(case, seed, _nodes(case)[0])).to(device)
    U = _initial(case, seed, X).reshape(5, op.E, op.n, op.n, op.n)
    w = op.wt
    wJ = w[:, None, None] * w[None, :, None] * w[None, None, :] * op.J
    rho, u, p, T = op._prim(U)
    volume = wJ.sum()
    kinetic = (wJ * 0.5 * rho * (u * u).sum(0)).sum() / volume
    g = op.gradients(U)
    curl = (g[1][2] - g[2][1]) ** 2 + (g[2][0] - g[0][2]) ** 2 + (g[0][1] - g[1][0]) ** 2
    div = g[0][0] + g[1][1] + g[2][2]
    mu = op.p["mu"]
    eps = [(wJ * mu * curl).sum() / volume, 4.0 / 3.0 * (wJ * mu * div * div).sum() / volume]
    c, lam, vis = (GAMMA * p / rho).sqrt(), 0.0, 0.0
    for d in range(3):
        size = (op.Ja[d] ** 2).sum(0).sqrt()
        lam = lam + ((u * op.Ja[d]).sum(0).abs() + c * size) / op.J
        vis = vis + (size / op.J) ** 2
    nu = max(4.0 / 3.0, GAMMA / op.p["Pr"]) * mu / rho
    dt = min(float((0.9 * 2.0 / ((2 * op.N + 1) * lam)).min()), float((0.9 * 4.0 / (op.n ** 4 * nu * vis)).min()))
    return {"integrals": torch.stack([(wJ * U[k]).sum() for k in range(5)] + [kinetic, volume]).cpu().numpy(),
            "dissipation": torch.stack(eps).cpu().numpy(), "dt": dt}


def exact(case, seed):
    device = "cuda" if torch.cuda.is_available() else "cpu"
    if case["kind"] == "served":
        return [_exact_solve(one, s, device).cpu().numpy() for one, s in _requests(case, seed)]
    if case["kind"] == "analysis":
        return _exact_analysis(case, seed, device)
    return _exact_solve(case, seed, device)
