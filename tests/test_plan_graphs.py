"""Graphs of one plan recorded apart from each other: an apply recorded before the
plan's build is, and builds of batches of several sizes.  A graph keeps the device
addresses it was recorded with, so a replay must find the maps and the tiles of the
batch staged last there, whatever was recorded in between.  Maps set inside a
capture likewise, where the first batch of a plan is accepted and any later one
refused; and batches staged while earlier ones are in flight, with no event between
a build and its apply.  The maps differ in
their group sizes (at equal tile counts, as a graph's launches need).  On the CPU
build of the runtime and kernels, whose shim records and replays launches
(tests/cpu_kernels/capture.cpp), and on the GPU; each replay is compared with the
eager result of the same maps, bit for bit (integer inputs)."""
import ctypes as C

import numpy as np
import pytest

from tests import cpu_build
from tests.gpu_harness import Run, hipmod, to_dev
from tests.test_gpu_tiles import _workload
from tests.test_plan_capture import _graph_api

SKEWS = ((0, 0, 0, 0), (-1, 2, -2, 1), (3, -1, 0, -2))


@pytest.mark.skipif(not cpu_build.available(), reason="needs the ROCm host clang")
@pytest.mark.parametrize("sequence,T", [("apply_then_build", 16), ("apply_then_build", 200), ("two_sizes", 100),
                                        ("two_sizes", 5000), ("maps_in_capture", 16), ("maps_in_capture", 200),
                                        ("maps_in_capture", 5000), ("maps_in_capture_built_outside", 16),
                                        ("maps_in_capture_built_outside", 200),
                                        ("maps_in_capture_built_outside", 5000), ("batches_in_flight", 16),
                                        ("batches_in_flight", 200), ("batches_in_flight", 5000)])
def test_on_the_cpu(sequence, T):
    r = cpu_build.program("capture", sequence, str(T))
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr


class Graphs:
    """One context and plan, its y in one buffer, and what was recorded."""

    def __init__(self, T):
        self.hip = hipmod()
        self.lib = _graph_api(self.hip)
        self.T = T
        self.w = _workload(1700 + T, [("a", 264, 136)], 4, 16, T, 12, (1, 2), exact=True)
        self.run = Run(self.w)
        self.x, self.y, self.y0 = to_dev(self.w.x(0)), to_dev(self.w.y0(0)), to_dev(self.w.y0(0))
        self.execs = []

    def maps(self, T):
        """T tokens in four groups, per skew; every map holds a user of the largest rank."""
        out = []
        for k, skew in enumerate(SKEWS):
            rng = np.random.default_rng([2608, 3579, T, k])
            order = rng.permutation(T)
            tok_c = np.repeat(np.arange(4), [T // 4 + s for s in skew]).astype(np.int32)
            slots = self.w.referenced_slots()
            tok_u = rng.choice(slots, size=T).astype(np.int32)
            tok_u[0] = slots[np.argmax(self.w.slot_rank[slots])]
            tok_u[5] = -1
            out.append((tok_c[order], tok_u))
        return out

    def reset(self):
        self.hip.check(self.lib.hipMemcpyAsync(self.y.ptr, self.y0.ptr, self.w.y0(0).nbytes, 3, self.run.stream), "copy")

    def set(self, m):
        self.run.plan.set_maps(*m, None, self.run.stream)

    def build(self):
        self.run.plan.build(self.run.stream)

    def apply(self):
        self.run.ctx.apply(0, self.run.plan, self.x.ptr, self.y.ptr, self.run.stream)

    def result(self):
        self.run._stream.synchronize()
        return self.y.to_host()

    def expected(self, maps):
        plan, self.run.plan = self.run.plan, self.run.ctx.plan()
        out = []
        for m in maps:
            self.reset(); self.set(m); self.build(); self.apply()
            out.append(self.result())
        self.run.plan.close()
        self.run.plan = plan
        return out

    def record(self, *steps):
        self.run._stream.synchronize()
        graph, ex = C.c_void_p(), C.c_void_p()
        self.hip.check(self.lib.hipStreamBeginCapture(self.run.stream, 0), "begin capture")
        for s in steps:
            s()
        self.hip.check(self.lib.hipStreamEndCapture(self.run.stream, C.byref(graph)), "end capture")
        self.hip.check(self.lib.hipGraphInstantiate(C.byref(ex), graph, None, None, 0), "instantiate")
        self.hip.check(self.lib.hipGraphDestroy(graph), "destroy")
        self.execs.append(ex)
        return ex

    def replay(self, ex):
        self.hip.check(self.lib.hipGraphLaunch(ex, self.run.stream), "launch")

    def close(self):
        self.run._stream.synchronize()
        for ex in self.execs:
            self.hip.check(self.lib.hipGraphExecDestroy(ex), "destroy")
        for d in (self.x, self.y, self.y0):
            d.free()
        self.run.close()


@pytest.mark.gpu
@pytest.mark.parametrize("T", [16, 200])
def test_an_apply_recorded_before_a_build(T):
    print(f"\n[gpu case] apply graph, then build graph, {T} tokens", flush=True)
    g = Graphs(T)
    try:
        maps = g.maps(T)
        want = g.expected(maps)
        g.set(maps[0]); g.build()
        apply = g.record(g.apply)
        g.set(maps[1])
        build = g.record(g.build)
        for k in (1, 2, 0, 1):
            g.set(maps[k]); g.reset()
            g.replay(build); g.replay(apply)
            assert np.array_equal(g.result(), want[k]), k
        for k in (2, 0):
            g.set(maps[k]); g.build(); g.reset()
            g.replay(apply)
            assert np.array_equal(g.result(), want[k]), ("eager build", k)
        assert g.run.plan.errors(g.run.stream) == 0
    finally:
        g.close()


@pytest.mark.gpu
def test_builds_of_two_sizes():
    print("\n[gpu case] graphs of 5000 and of 200 tokens on one plan", flush=True)
    g = Graphs(5000)
    try:
        sizes = (5000, 200)
        maps = [g.maps(T) for T in sizes]
        want = [g.expected(m) for m in maps]
        execs = []
        for m in maps:
            g.set(m[0])
            execs.append(g.record(g.build, g.apply))
        for k in (0, 1, 2, 0):
            for m, w, ex in zip(maps, want, execs):
                g.set(m[k]); g.reset()
                g.replay(ex)
                assert np.array_equal(g.result(), w[k]), (len(m[0][0]), k)
    finally:
        g.close()


@pytest.mark.gpu
@pytest.mark.parametrize("T", [16, 200, 5000])
def test_maps_set_inside_a_capture(T):
    print(f"\n[gpu case] maps set inside a capture, {T} tokens", flush=True)
    from paper_2608_03579_amd import salt
    g = Graphs(T)
    try:
        maps = g.maps(T)
        want = g.expected(maps)

        def second():
            with pytest.raises(salt.SaltError) as e:
                g.set(maps[1])
            assert e.value.status == salt.ERR_BAD_STATE

        ex = g.record(lambda: g.set(maps[0]), g.build, g.apply, second)
        last = 0
        for k in (None, None, 1, 2, None, 0, 1):
            if k is not None:
                g.set(maps[k])
                last = k
            g.reset()
            g.replay(ex)
            assert np.array_equal(g.result(), want[last]), (k, last)
        g.record(second)
        g.set(maps[2]); g.build(); g.reset(); g.apply()
        assert np.array_equal(g.result(), want[2])
        assert g.run.plan.errors(g.run.stream) == 0
    finally:
        g.close()
