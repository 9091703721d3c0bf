"""Iterations a caller captures into a graph of its own: what the handle reports
after a replay, which the host does not see, is what ran last."""
import ctypes

import numpy as np
import pytest

import oracle
from conftest import f32_params
from parity_checks import check, gpu_outputs
from paper_2504_06437_amd import workloads as W

pytestmark = pytest.mark.gpu


class Capture:
    """A graph of what is issued on `stream` inside the with block."""

    def __init__(self, stream):
        from paper_2504_06437_amd import hip
        self.hip, self.stream = hip.runtime(), ctypes.c_void_p(stream)
        self.graph, self.exec = ctypes.c_void_p(), ctypes.c_void_p()

    def __enter__(self):
        assert self.hip.hipStreamBeginCapture(self.stream, 1) == 0      # thread-local
        return self

    def __exit__(self, kind, *_):
        assert self.hip.hipStreamEndCapture(self.stream, ctypes.byref(self.graph)) == 0
        if kind is None:
            assert self.hip.hipGraphInstantiate(ctypes.byref(self.exec), self.graph, None, None,
                                                ctypes.c_size_t(0)) == 0

    def replay(self, stream=None):
        s = ctypes.c_void_p(stream) if stream else self.stream
        assert self.hip.hipGraphLaunch(self.exec, s) == 0
        assert self.hip.hipStreamSynchronize(s) == 0

    def close(self):
        self.hip.hipGraphExecDestroy(self.exec)
        self.hip.hipGraphDestroy(self.graph)


def test_plan_after_a_replay_is_the_replays():
    """Two iterations in a graph (the warm start's halves return to their
    places), replayed between pairs of synchronous steps: U* is the eager
    controller's every time."""
    from paper_2504_06437_amd.controller import Controller
    from paper_2504_06437_amd.hip import DeviceArray
    wl = W.quad_small(K=512, T=20, J=10)
    p = dict(wl["params"], tile_samples=16)
    c, eager = Controller(p), Controller(p)
    for h in (c, eager):
        h.load_workload(wl)
        h.step(wl["x0"])
    x0 = DeviceArray.from_numpy(wl["x0"])
    g = Capture(c.stream)
    with g:
        c.step_async(x0.at(0))
        c.step_async(x0.at(0))
    for _ in range(3):
        for h in (c, eager):
            h.step(wl["x0"])
            h.step(wl["x0"])
        np.testing.assert_array_equal(c.last_optimal(), eager.last_optimal())
        g.replay()
        eager.step_async(x0.at(0))
        eager.step_async(x0.at(0))
        np.testing.assert_array_equal(c.last_optimal(), eager.last_optimal())
    g.close()
    c.close()
    eager.close()


@pytest.mark.parametrize("K,T,J", [(512, 20, 40), (8192, 64, 400)])
def test_inputs_are_in_place_for_a_replay_on_another_stream(K, T, J):
    """Obstacles (with and without a far field) and the reference, set between
    replays on a stream that nothing orders behind the controller's own."""
    from paper_2504_06437_amd.controller import Controller
    from paper_2504_06437_amd.hip import DeviceArray, runtime
    rng = np.random.default_rng(J)
    wl = W.quad_large(K=K, T=T, J=J, with_map=False)
    p = dict(wl["params"], tile_samples=32)
    c, eager, other = Controller(p), Controller(p), Controller(p)     # other: its stream alone is used
    x0 = DeviceArray.from_numpy(wl["x0"])
    for h in (c, eager):
        h.load_workload(wl)
    g = Capture(c.stream)
    with g:
        c.step_async(x0.at(0))
        c.step_async(x0.at(0))
    for _ in range(3):
        obs = wl["obstacles"] + np.float32([1, 1, 0]) * rng.uniform(-0.2, 0.2, (J, 3)).astype(np.float32)
        ref = wl["x_ref"] + rng.uniform(-0.1, 0.1, wl["x_ref"].shape).astype(np.float32)
        for h in (c, eager):
            h.set_reference(ref)
            h.set_obstacles(obs)
        g.replay(other.stream)
        eager.step_async(x0.at(0))
        eager.step_async(x0.at(0))
        np.testing.assert_array_equal(c.last_optimal(), eager.last_optimal())
        np.testing.assert_array_equal(c.costs(), eager.costs())
    runtime().hipDeviceSynchronize()
    g.close()
    for h in (c, eager, other):
        h.close()


@pytest.mark.parametrize("J", [420, 40])
def test_replay_after_another_obstacle_count(J):
    """A graph holds its obstacle count: after 420 or 40 obstacles are set it
    runs the first 400 of the buffer, and takes no barrier from a field that was
    built for others.  The parity tests' own check against the oracle."""
    from paper_2504_06437_amd.controller import Controller
    from paper_2504_06437_amd.hip import DeviceArray
    wl = W.quad_large(K=8192, T=64, J=450, with_map=False)
    p = dict(wl["params"], tile_samples=32)
    c = Controller(p)
    x0 = DeviceArray.from_numpy(wl["x0"])
    first = wl["obstacles"][:400]
    c.load_workload(wl)                     # (the buffer holds 450)
    c.set_obstacles(first)
    g = Capture(c.stream)
    with g:
        c.step_async(x0.at(0))
    new = W.quad_large(K=1, T=1, J=450, with_map=False, seed=9)["obstacles"][:J]
    c.set_obstacles(new)
    held = dict(wl, obstacles=np.concatenate([new[:400], first[J:]]))
    g.replay()
    got = gpu_outputs(c, c.last_optimal()[0], with_noise=False)
    ref = oracle.step(f32_params(p), oracle.World.from_workload(held), wl["x0"], wl["U0"], wl["x_ref"], 1.0, 0)
    check(got, ref, p, what=f"400 held, {J} set")
    g.close()
    c.close()
