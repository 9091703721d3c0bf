"""The obstacles' far field: an iteration whose barriers come from it matches
the oracle to the parity tests' own tolerances (parity_checks: costs within
1e-4 relative plus the barrier's conditioning over the FP32 position budget,
weights and U* to 1e-4) wherever the field's parts change over -- on both sides
of the size rule, with several lanes per pose and one, cells whose near list is
full, grids stretched by a far obstacle, starts outside every grid, bodies that
are not the paper's, and the costmap beside it; the indicator's decisions agree
with its margins."""
import numpy as np
import pytest

import oracle
from conftest import f32_params
from parity_checks import check, gpu_outputs
from test_gpu_variants import _iteration
from paper_2504_06437_amd import workloads as W

pytestmark = pytest.mark.gpu

TRACTOR = [[2.4, 0.9], [2.4, -0.9], [1.2, 1.3], [1.2, -1.3], [0.0, 1.3], [0.0, -1.3],
           [-1.2, 1.3], [-1.2, -1.3], [-2.0, 0.8], [-2.0, -0.8]]
AXIS = [[0.25, 0.0], [-0.2, 0.0], [0.15, 0.0], [0.0, 0.0], [-0.1, 0.0], [0.05, 0.0], [-0.25, 0.0]]


def _step(wl, **over):
    from paper_2504_06437_amd.controller import Controller
    p = dict(wl["params"], **over)
    c = Controller(p)
    c.load_workload(wl)
    u0 = c.step(wl["x0"])
    g = gpu_outputs(c, u0, with_noise=False)
    assert c.info()["status"] == 0
    c.close()
    ref = oracle.step(f32_params(p), oracle.World.from_workload(wl), wl["x0"], wl["U0"], wl["x_ref"], 1.0, 0)
    assert ref["status"] == 0
    return g, ref, p


def _world(name):
    # (the size rule: a step has to save what building the field costs, about
    # 5.8e-7 K T (J - 50) us of the quadrotors', 8.3e-7 K T (J - 115) of the
    # vehicle's against 26 + J / 10)
    if name == "quad at the rule":              # the first J with a field at this K, T
        return W.quad_large(K=4096, T=100, J=276, with_map=False)
    if name == "quad below the rule":           # ... the last without
        return W.quad_large(K=4096, T=100, J=275, with_map=False)
    if name == "quad, one lane a pose":
        wl = W.quad_large(K=3400, T=100, J=400, with_map=False)
        wl["params"]["tile_samples"] = 128
        return wl
    if name == "quad, four lanes a pose":
        wl = W.quad_large(K=20000, T=17, J=400, with_map=False)
        wl["params"]["tile_samples"] = 16
        return wl
    if name == "quad with a costmap":
        return W.quad_large(K=5700, T=61, J=400, cells=64)
    if name == "quad, body on an axis only":
        wl = W.quad_large(K=4871, T=70, J=400, with_map=False)
        wl["params"]["shape"] = AXIS
        return wl
    if name == "vehicle at the rule":
        return W.car(K=4301, T=60, J=470)
    if name == "vehicle, tractor body":
        wl = W.car(K=1501, T=70, J=350)
        wl["params"]["shape"] = TRACTOR
        return wl
    wl = W.quad_large(K=3401, T=100, J=400, with_map=False)
    obs = wl["obstacles"].copy()
    if name == "near lists full":               # 200 obstacles within half a metre, 6 m off the start
        rng = np.random.default_rng(1)
        obs[:200, :2] = np.float32([8.0, 4.0]) + rng.uniform(-0.5, 0.5, (200, 2)).astype(np.float32)
        obs[:200, 2] = 0.1
    elif name == "one obstacle 30 km off":
        obs[0] = [30000.0, -20000.0, 1.0]
    elif name == "start outside the grids":
        obs[:, 0] += 300.0
    elif name == "all obstacles on one spot":
        obs[:] = [9.0, 9.0, 0.5]
    else:
        raise ValueError(name)
    return dict(wl, obstacles=obs)


@pytest.mark.parametrize("name", [
    "quad at the rule", "quad below the rule", "quad, one lane a pose", "quad, four lanes a pose",
    "quad with a costmap", "quad, body on an axis only", "vehicle at the rule", "vehicle, tractor body",
    "near lists full", "one obstacle 30 km off", "start outside the grids", "all obstacles on one spot"])
def test_iteration_by_the_far_field_matches_oracle(name):
    g, ref, p = _step(_world(name))
    check(g, ref, p, what=name)


@pytest.mark.parametrize("controller", ["vanilla", "log"])
def test_indicator_by_near_lists_decides_as_the_oracle(controller):
    """Far obstacles never decide, and every near one is listed: the variants'
    own check (samples whose every step keeps |h| >= 1e-3 m^2 have the
    oracle's cost to 1e-4, the others up to whole collision weights)."""
    _iteration(W.car(K=4400, T=60, J=300), controller)
