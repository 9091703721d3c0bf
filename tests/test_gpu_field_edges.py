"""The obstacles' far field at the edges of what it accepts, against the oracle
to the parity tests' own tolerances: a barrier cap h_eps that binds for
obstacles far beyond a cell."""
import pytest

from parity_checks import check
from test_gpu_field import TRACTOR, _step
from paper_2504_06437_amd import workloads as W

pytestmark = pytest.mark.gpu


def _world(body):
    if body == "quadrotor":
        return W.quad_large(K=4096, T=100, J=400, with_map=False)
    if body == "quadrotor, costmap":
        return W.quad_large(K=5700, T=61, J=400, cells=64)
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
