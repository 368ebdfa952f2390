"""The set-up's recognition of meshes of parallelepipeds, on the CPU: box
meshes of every degree, size, place and relabelling are recognised, sheared
ones too, any real curving is not; a recognised mesh holds the same metrics at
every node of an element and keeps the discrete metric identity."""
import os
import struct
import subprocess

import numpy as np
import pytest

import workloads as W
from paper_2404_12703_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2404_12703_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
SHEAR = np.array([[1.0, 0.3, -0.2], [0.1, 0.9, 0.4], [-0.3, 0.2, 1.2]])


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("affine") / "driver")
    cmd = [HIPCC, "-x", "hip", "--offload-host-only", "-std=c++17", "-O2", "-I" + os.path.join(ROOT, "include"),
           "-I" + CSRC, os.path.join(ROOT, "tests", "sanitize", "affine_driver.cpp"), os.path.join(CSRC, "setup.cpp"),
           os.path.join(CSRC, "solver.cpp"), "-Wl,--unresolved-symbols=ignore-in-object-files", "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return out


def _run(driver, tmp_path, m, N, nodes):
    path = str(tmp_path / "case.bin")
    with open(path, "wb") as f:
        f.write(struct.pack("<i", 1) + bytes(B.make_params(W.params(N, node_type=nodes))))
        f.write(struct.pack("<qi", m.x_geo.shape[0], int(m.ngeo)))
        for a, dt in ((m.x_geo, np.float64), (m.nbr_elem, np.int64), (m.nbr_face, np.int8), (m.nbr_orient, np.int8)):
            f.write(np.ascontiguousarray(a, dtype=dt).tobytes())
    r = subprocess.run([driver, path], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    t = r.stdout.split()
    return int(t[1]), float(t[3]), float(t[5])


# D-hat's rows hold entries up to about n^2/2: a metric off by eps = 2.2e-16
# leaves a residual of a few n^2 eps; neighbours that differ by the rounding of
# the coordinates (eps x/h n_geo^3, x/h <= 2 max(K) below) add l-hat (<= n^2/2) times that
def _bound(N, ngeo, xh):
    n = N + 1
    return 2.2e-16 * n * n * (8.0 + xh * ngeo ** 3)


@pytest.mark.parametrize("shear", [False, True])
@pytest.mark.parametrize("K,lo,hi", [((3, 2, 4), 0.0, 2 * np.pi), ((9, 3, 2), -1.0, 1.0), ((2, 2, 40), 0.0, 2 * np.pi)])
@pytest.mark.parametrize("N,ngeo,nodes", [(1, 1, 0), (3, 1, 0), (3, 3, 0), (5, 1, 1), (5, 5, 1), (7, 1, 0), (7, 7, 1),
                                          (9, 9, 0)])
def test_boxes_are_recognised(driver, tmp_path, N, ngeo, nodes, K, lo, hi, shear):
    m = W.box_mesh(K, lo, hi, ngeo, rotate=True)
    if shear:
        m.x_geo = np.einsum("dc,ecg->edg", SHEAR, m.x_geo)
    affine, spread, closure = _run(driver, tmp_path, m, N, nodes)
    assert affine == 1 and spread == 0.0
    assert closure <= _bound(N, ngeo, 2 * max(K))


@pytest.mark.parametrize("amp", [1e-10, 0.05])
@pytest.mark.parametrize("N", [2, 3, 7])
def test_curved_meshes_are_not(driver, tmp_path, N, amp):
    m = W.box_mesh((3, 2, 4), 0.0, 2 * np.pi, N, amp=amp, rotate=True)
    affine, spread, closure = _run(driver, tmp_path, m, N, 0)
    assert affine == 0 and spread > 0.0
    assert closure <= 1e-12
