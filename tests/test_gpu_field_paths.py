"""The obstacles' far field on every path that takes it: the vehicle on both
sides of its size rule and obstacle counts past one pass of the build against
the oracle; the call without a handle (eager and replayed from a graph), the
batch and the server bit for bit what a controller alone computes."""
import ctypes

import numpy as np
import pytest

from parity_checks import check
from test_gpu_field import _step
from test_gpu_graph import Capture
from test_zz_no_alloc import _controller_step, _noalloc_step
from paper_2504_06437_amd import workloads as W

pytestmark = pytest.mark.gpu

MANY = ["513", "2048", "300 around one spot"]
FLEET_FIELDS = [True, False, True, True, False]


def vehicle(field):
    """The first obstacle count with a field at K = 4301, T = 60, and the last without."""
    return W.car(K=4301, T=60, J=444 if field else 443)


def many(name):
    """513: one obstacle past the build's 512 threads.  2048: the most, whose
    build needs more than 64 KiB of LDS.  300 within a metre, others around: more
    than 256 near a macro cell, where the cells take the widest threshold."""
    if name == "300 around one spot":
        wl = W.quad_large(K=5200, T=60, J=600, with_map=False)
        obs = wl["obstacles"].copy()
        rng = np.random.default_rng(5)
        obs[:300, :2] = np.float32([12.0, 9.0]) + rng.uniform(-0.5, 0.5, (300, 2)).astype(np.float32)
        obs[:300, 2] = 0.1
        return dict(wl, obstacles=obs)
    J = int(name)
    return W.quad_large(K=5200 if J < 1000 else 4300, T=60, J=J, with_map=False)


def fleet():
    """Five controllers, three of them with a field, of tile shapes of their own."""
    wls = [W.quad_large(K=8192, T=64, J=230, with_map=False), W.car(K=700, T=20, J=90),
           W.car(K=4301, T=60, J=460), W.quad_large(K=6000, T=90, J=300, with_map=False),
           W.quad_small(K=300, T=20, J=10)]
    for i, wl in enumerate(wls):
        wl["params"].update(tile_samples=(32, 16, 32, 64, 16)[i], seed=40 + i)
        wl["U0"] = np.zeros_like(wl["U0"])
    return wls


@pytest.mark.parametrize("field", [True, False])
def test_vehicle_at_its_rule_matches_oracle(field):
    g, ref, p = _step(vehicle(field))
    check(g, ref, p, what=f"vehicle, field {field}")


@pytest.mark.parametrize("name", MANY)
def test_many_obstacles_match_oracle(name):
    g, ref, p = _step(many(name))
    check(g, ref, p, what=name)


@pytest.mark.parametrize("member", [0, 2])
def test_noalloc_by_the_field_equals_the_controller(member):
    wl = fleet()[member]
    p, st, want = _controller_step(wl, wl["params"]["tile_samples"])
    got = _noalloc_step(p, wl, st)
    assert want["status"] == 0 and got["status"] == 0
    for key in ("Ustar", "Unext", "u0"):
        np.testing.assert_array_equal(got[key], want[key], err_msg=key)


def test_noalloc_by_the_field_replays():
    """The build and the step in a graph: every replay is the eager call on the
    obstacles that are in place then, with another world's eager call between."""
    from paper_2504_06437_amd import _lib as A
    from paper_2504_06437_amd.controller import Controller, make_config
    from paper_2504_06437_amd.hip import DeviceArray, synchronize
    L = A.load()
    rng = np.random.default_rng(11)
    wl, between = fleet()[0], fleet()[3]
    own = Controller(wl["params"])          # its stream is used

    class Call:
        def __init__(self, w):
            T = w["params"]["T"]
            self.cfg, self.prob = make_config(w["params"]), A.Problem()
            self.obs = DeviceArray.from_numpy(w["obstacles"])
            self.ref, self.x0 = DeviceArray.from_numpy(w["x_ref"]), DeviceArray.from_numpy(w["x0"])
            self.U = DeviceArray.from_numpy(w["U0"])
            self.Ustar, self.Unext = DeviceArray((T, 2)), DeviceArray((T, 2))
            self.prob.J, self.prob.obs, self.prob.x_ref = len(w["obstacles"]), self.obs.ptr, self.ref.ptr

        def run(self, stream):
            assert L.mppi_step_noalloc(ctypes.byref(self.cfg), ctypes.byref(self.prob), 0, ctypes.c_void_p(stream),
                                       self.x0.ptr, self.U.ptr, 5, ctypes.c_float(1.0), self.Ustar.ptr,
                                       self.Unext.ptr, None, None) == A.OK

    call, other = Call(wl), Call(between)
    g = Capture(own.stream)
    with g:
        call.run(own.stream)
    for _ in range(3):
        moved = wl["obstacles"] + np.float32([1, 1, 0]) * rng.uniform(-0.2, 0.2, wl["obstacles"].shape).astype(np.float32)
        call.obs.upload(moved)
        call.run(own.stream)
        synchronize()
        want = call.Ustar.numpy()
        other.run(own.stream)
        call.Ustar.upload(np.zeros_like(want))
        g.replay()
        np.testing.assert_array_equal(call.Ustar.numpy(), want)
    g.close()
    own.close()


def test_batch_and_server_by_the_field_equal_alone():
    from paper_2504_06437_amd.controller import Batch, Controller, Server
    wls = fleet()
    alone, mixed = [], []
    for wl in wls:
        for kind in (alone, mixed):
            c = Controller(wl["params"])
            c.load_workload(wl)
            kind.append(c)
    batch, srv = Batch(mixed), Server()
    ids = [srv.add_robot(wl["params"], wl["obstacles"]) for wl in wls]
    for step in range(3):
        if step == 2:                       # a world that moves: the batch's field is built anew
            wls[0]["obstacles"] = wls[0]["obstacles"] + np.float32([0.1, -0.1, 0.0])
            for c in (alone[0], mixed[0]):
                c.set_obstacles(wls[0]["obstacles"])
        tickets = [srv.submit(i, wl["x0"], wl["x_ref"]) for i, wl in zip(ids, wls)]
        served = [srv.wait(t)[0] for t in tickets]
        u_b, sts = batch.step([wl["x0"] for wl in wls])
        assert np.all(sts == 0)
        for i, (a, m, wl) in enumerate(zip(alone, mixed, wls)):
            u_a = a.step(wl["x0"])
            np.testing.assert_array_equal(u_b[i], u_a)
            np.testing.assert_array_equal(m.controls(), a.controls())
            np.testing.assert_array_equal(m.costs(), a.costs())
            if step < 2 or i > 0:
                np.testing.assert_array_equal(served[i], u_a)
                if step < 2:
                    np.testing.assert_array_equal(srv.robot_state(ids[i])[0], a.controls())
    srv.close()
    batch.close()
    for c in alone + mixed:
        c.close()
