"""A plan build and an apply recorded into a HIP graph and replayed: every replay must
serve the maps staged last (set_maps outside the graph, same batch size), for batches
whose eager builds carry the maps in the kernel's arguments and for those that read
them in place.  Each replay is compared with the eager result of the same maps."""
import ctypes as C

import numpy as np
import pytest

from tests.gpu_harness import Run, hipmod, to_dev
from tests.test_gpu_tiles import _workload

pytestmark = pytest.mark.gpu


def _graph_api(hip):
    lib = hip._hip
    for name, args in {"hipStreamBeginCapture": [C.c_void_p, C.c_int],
                       "hipStreamEndCapture": [C.c_void_p, C.POINTER(C.c_void_p)],
                       "hipGraphInstantiate": [C.POINTER(C.c_void_p), C.c_void_p, C.c_void_p, C.c_void_p, C.c_size_t],
                       "hipGraphLaunch": [C.c_void_p, C.c_void_p], "hipGraphExecDestroy": [C.c_void_p],
                       "hipGraphDestroy": [C.c_void_p]}.items():
        getattr(lib, name).restype = C.c_int
        getattr(lib, name).argtypes = args
    return lib


@pytest.mark.parametrize("T", [16, 200])
def test_replays_serve_the_maps_staged_last(T):
    print(f"\n[gpu case] captured plan build, {T} tokens", flush=True)
    hip = hipmod()
    lib = _graph_api(hip)
    w = _workload(700 + T, [("a", 264, 136)], 4, 16, T, 12, (1, 2))
    run = Run(w)
    xd, yd = to_dev(w.x(0)), to_dev(w.y0(0))
    y0 = to_dev(w.y0(0))
    maps = [(np.roll(w.tok_c, k), np.roll(w.tok_u, k)) for k in (0, 3, 7)]

    def reset():
        hip.check(lib.hipMemcpyAsync(yd.ptr, y0.ptr, w.y0(0).nbytes, 3, run.stream), "copy")

    def apply():
        run.ctx.apply(0, run.plan, xd.ptr, yd.ptr, run.stream)

    try:
        want = []
        for c, u in maps:
            reset()
            run.plan.set_maps(c, u, None, run.stream)
            run.plan.build(run.stream)
            apply()
            run._stream.synchronize()
            want.append(yd.to_host())
        run.plan.set_maps(*maps[0], None, run.stream)
        run._stream.synchronize()
        graph, ex = C.c_void_p(), C.c_void_p()
        hip.check(lib.hipStreamBeginCapture(run.stream, 0), "begin capture")
        run.plan.build(run.stream)
        apply()
        hip.check(lib.hipStreamEndCapture(run.stream, C.byref(graph)), "end capture")
        hip.check(lib.hipGraphInstantiate(C.byref(ex), graph, None, None, 0), "instantiate")
        for k in (0, 1, 2, 1, 0):
            reset()
            run.plan.set_maps(*maps[k], None, run.stream)
            hip.check(lib.hipGraphLaunch(ex, run.stream), "launch")
            run._stream.synchronize()
            assert np.array_equal(yd.to_host(), want[k]), k
        assert run.plan.errors(run.stream) == 0
        hip.check(lib.hipGraphExecDestroy(ex), "destroy")
        hip.check(lib.hipGraphDestroy(graph), "destroy")
    finally:
        for d in (xd, yd, y0):
            d.free()
        run.close()
