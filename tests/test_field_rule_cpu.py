"""Which of the GPU tests' worlds run by the obstacles' far field: the rule is
asked on the host for every one of them, so that a changed constant cannot turn
a test of the field into one of the walk unseen."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import test_gpu_field as TF
import test_gpu_field_edges as TE
import test_gpu_field_paths as TP
from paper_2504_06437_amd import _lib as A
from paper_2504_06437_amd import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_06437_amd", "csrc")


@pytest.fixture(scope="module")
def wanted(tmp_path_factory):
    hipcc = shutil.which("hipcc")
    if hipcc is None:
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("field") / "field_rule_check")
    subprocess.check_call([hipcc, "-O1", "-std=c++17", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                           os.path.join(ROOT, "tests", "native", "field_rule_check.cpp"), "-o", exe])

    def ask(wl, **over):
        p = dict(wl["params"], **over)
        shape = np.float32(p["shape"])
        # the layout forms of the tests' bodies: the paper's, and points on the axis only
        kind = 0
        if len(shape) == 8 and p["model"] == "car":
            kind = 1
        elif len(shape) == 7 and not shape[:, 1].any():
            kind = 2 if np.array_equal(shape[:, 0], -shape[::-1, 0]) else 1
        row = (A.MODELS[p["model"]], p["K"], p["T"], len(wl["obstacles"]), len(shape), kind,
               A.COST_MODE[p.get("cost_mode", "dbas")])
        out = subprocess.run([exe], input=" ".join(str(v) for v in row) + "\n", capture_output=True, text=True, check=True)
        return out.stdout.strip() == "1"

    return ask


def test_worlds_of_the_field_tests(wanted):
    for name in ("quad at the rule", "quad, one lane a pose", "quad, four lanes a pose", "quad with a costmap",
                 "quad, body on an axis only", "vehicle at the rule", "vehicle, tractor body", "near lists full",
                 "one obstacle 30 km off", "start outside the grids", "all obstacles on one spot"):
        assert wanted(TF._world(name)), name
    assert not wanted(TF._world("quad below the rule"))
    assert wanted(W.car(K=4400, T=60, J=300), **W.CONTROLLERS["vanilla"])


@pytest.mark.parametrize("body", ["quadrotor", "quadrotor, costmap", "pitch-rate quadrotor", "vehicle", "tractor"])
def test_worlds_at_the_edges(wanted, body):
    assert wanted(TE._world(body))


def test_worlds_of_the_paths(wanted):
    assert wanted(TP.vehicle(True)) and not wanted(TP.vehicle(False))
    for name in TP.MANY:
        assert wanted(TP.many(name)), name
    assert [wanted(wl) for wl in TP.fleet()] == TP.FLEET_FIELDS
