"""The obstacles' far field at the edges of what it accepts, against the oracle
to the parity tests' own tolerances: a barrier cap h_eps that binds for
obstacles far beyond a cell, radii that only the device holds, no memory for
the field, poses that have no cell, and their sums far from every obstacle."""
import os
import re
import subprocess
import sys

import numpy as np
import pytest

import oracle
from conftest import f32_params
from parity_checks import check
from test_gpu_field import TRACTOR, _step
from paper_2504_06437_amd import _lib as A
from paper_2504_06437_amd import workloads as W

pytestmark = pytest.mark.gpu

TESTS = os.path.dirname(os.path.abspath(__file__))
FIELD_HPP = os.path.join(os.path.dirname(TESTS), "paper_2504_06437_amd", "csrc", "mppi_field.hpp")


def _world(body):
    if body == "quadrotor":
        return W.quad_large(K=4096, T=100, J=400, with_map=False)
    if body == "quadrotor, costmap":
        return W.quad_large(K=5700, T=61, J=400, cells=64)
    if body == "pitch-rate quadrotor":
        wl = W.quad_large(K=4096, T=100, J=400, with_map=False)
        wl["params"] = dict(W.base_params("quad5", 4096, 100, 2))
        wl["x0"], wl["x_ref"] = wl["x0"][:5], np.ascontiguousarray(wl["x_ref"][:, :5])
        return wl
    if body == "vehicle":
        return W.car(K=6000, T=60, J=470)
    wl = W.car(K=1501, T=70, J=350)
    wl["params"]["shape"] = TRACTOR
    return wl


@pytest.mark.parametrize("body,h_eps", [("quadrotor", 0.5), ("quadrotor", 20.0), ("quadrotor, costmap", 2.0),
                                        ("vehicle", 10.0), ("tractor", 5.0), ("quadrotor", 1e6)])
def test_cap_binds_beyond_the_cell(body, h_eps):
    """B = 1/max(h, h_eps) holds for every obstacle, near and far; h_eps =
    1e6 caps them all (every list is full: the poses walk)."""
    g, ref, p = _step(_world(body), h_eps=h_eps)
    check(g, ref, p, what=f"{body} h_eps {h_eps}")


@pytest.mark.parametrize("body", ["quadrotor", "vehicle"])
def test_radii_on_the_device_count_by_their_magnitude(body):
    """h = |p - c|^2 - r^2 does not see the sign of r, and device memory is not
    checked: the same costs with some radii negated, bit for bit."""
    from paper_2504_06437_amd.controller import Controller
    from paper_2504_06437_amd.hip import DeviceArray
    wl = _world(body)
    c = Controller(dict(wl["params"], tile_samples=32))
    c.load_workload(wl)
    costs = []
    for sign in (1.0, -1.0):
        obs = wl["obstacles"].copy()
        obs[::3, 2] *= np.float32(sign)
        d = DeviceArray.from_numpy(obs)
        assert c.L.mppi_set_obstacles(c.h, len(obs), d.ptr, A.MEM_DEVICE) == A.OK
        c.set_state({"counter": 0, "S_e": 1.0, "U": wl["U0"]})
        c.step(wl["x0"])
        costs.append(c.costs())
    c.close()
    np.testing.assert_array_equal(costs[1], costs[0])


@pytest.mark.parametrize("body,place", [("vehicle", "outside"), ("vehicle", "full"), ("vehicle, costmap", "full"),
                                        ("tractor", "outside"), ("quadrotor, costmap", "full"),
                                        ("pitch-rate quadrotor", "outside")])
def test_poses_without_a_cell_walk(body, place):
    """Outside the grids, and where a cell's list is full (200 obstacles within
    half a metre, six metres off the start), a wave's poses walk the obstacles:
    the layout forms of the paper's bodies by their own."""
    wl = _world(body.split(",")[0] if body.startswith("vehicle") else body)
    if body == "vehicle, costmap":
        wl["map"] = W.quad_large(K=1, T=1, J=1, cells=64)["map"]
    obs = wl["obstacles"].copy()
    if place == "outside":
        obs[:, 0] += 300.0
    else:
        rng = np.random.default_rng(1)
        obs[:200, :2] = np.float32([8.0, 4.0]) + rng.uniform(-0.5, 0.5, (200, 2)).astype(np.float32)
        obs[:200, 2] = 0.1
    g, ref, p = _step(dict(wl, obstacles=obs))
    check(g, ref, p, what=f"{body} {place}")


def test_barrier_far_from_every_obstacle():
    """350 obstacles a kilometre off, ten points: beta_0 is 3.5e-3, and nothing
    but its terms enters it.  Bound: 90 groups' sums in turn, each addition half
    an ulp of FP32, 5e-6, and as much for the poses' rounding (1e-4 m in 1e3)."""
    wl = _world("tractor")
    obs = wl["obstacles"].copy()
    obs[:, 0] += 1000.0
    from paper_2504_06437_amd.controller import Controller
    c = Controller(wl["params"])
    c.load_workload(dict(wl, obstacles=obs))
    c.step(wl["x0"])
    got = c.info()["beta0"]
    c.close()
    x, y, th = (float(v) for v in wl["x0"][:3])
    body = np.float32(wl["params"]["shape"]).astype(np.float64)
    px = x + body[:, 0] * np.cos(th) - body[:, 1] * np.sin(th)
    py = y + body[:, 0] * np.sin(th) + body[:, 1] * np.cos(th)
    o = obs.astype(np.float64)
    h = (px[:, None] - o[:, 0]) ** 2 + (py[:, None] - o[:, 1]) ** 2 - o[:, 2] ** 2
    want = np.sum(1.0 / h)
    assert abs(got - want) <= 1e-5 * want, (got, want)


@pytest.mark.parametrize("model", ["quad6", "car"])
@pytest.mark.parametrize("K", [4300, 70])
def test_barriers_of_the_end_poses(model, K):
    """beta_0 and beta_d with a field (K = 4300) and without, in a world so dense
    that the goal lies inside obstacles: 8e-7 relative, from the clamped form's
    eight roundings and its reciprocal's ulp (6e-7 with the obstacle's own) and
    the five additions in which 32 lanes meet."""
    from paper_2504_06437_amd.controller import Controller
    wl = W.quad_large(K=K, T=60, J=2048, with_map=False) if model == "quad6" else W.car(K=K, T=60, J=800)
    p = dict(wl["params"], tile_samples=32)
    c = Controller(p)
    c.load_workload(wl)
    c.step(wl["x0"])
    i = c.info()
    c.close()
    ref = oracle.step(f32_params(dict(p, K=1)), oracle.World.from_workload(wl), wl["x0"], wl["U0"], wl["x_ref"], 1.0, 0)
    for key in ("beta0", "beta_d"):
        assert abs(i[key] - ref[key]) <= 8e-7 * ref[key], (key, i[key], ref[key])


CHILD = """
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path[:0] = sys.argv[2:4]
from parity_checks import check
from test_gpu_field import _step
from paper_2504_06437_amd import workloads as W
g, ref, p = _step(W.quad_large(K=4096, T=100, J=400, with_map=False))
check(g, ref, p, what="no memory for the field")
assert ctypes.c_int.in_dll(stub, "refused").value == 1
print("walked")
"""


def test_without_memory_for_the_field_the_poses_walk(tmp_path):
    """The allocation of the field alone is refused (a process whose hipMalloc
    fails for that one size): the obstacles are set, and the step is right."""
    macros = re.findall(r"kFieldMacros\d = (\d+)", open(FIELD_HPP).read())        # 16 cells of 64 words each
    size = 256 + sum(int(n) for n in macros) * 16 * 64 * 4
    stub = str(tmp_path / "fail_malloc.so")
    subprocess.check_call(["gcc", "-shared", "-fPIC", f"-DFAIL_BYTES={size}", os.path.join(TESTS, "native", "fail_malloc.c"),
                           "-o", stub, "-ldl"])
    r = subprocess.run([sys.executable, "-c", CHILD, stub, TESTS, os.path.dirname(TESTS)], capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0 and "walked" in r.stdout, r.stderr[-2000:]
