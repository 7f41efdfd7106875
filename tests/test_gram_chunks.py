"""salt_adapter_gram at the edges of its K chunks (1024 elements up to rank 32, each
chunk's Grams stored by one block and added up in float64; 2048 and atomics above):
a chunk exactly, a chunk and eight elements, less than one step, and ranks on both
sides of 16 and 32.  Integer factors, bit-exact against the oracle."""
import pytest

from tests.gpu_harness import to_dev
from tests.test_gpu_gram import _check, _ctx, _related, _workload

pytestmark = pytest.mark.gpu

TABLES = [("a", 1024, 8), ("b", 1032, 2048), ("c", 8, 3080), ("d", 504, 1016)]


@pytest.mark.parametrize("r1,r_extra,dtype", [(15, 1, "bf16"), (16, 1, "bf16"), (30, 2, "bf16"), (31, 2, "bf16"),
                                              (16, 1, "f32")])
def test_gram_chunk_edges(r1, r_extra, dtype):
    print(f"\n[gpu case] gram chunks r1={r1} extra={r_extra} {dtype}", flush=True)
    w = _workload(TABLES, [r1, r_extra], dtype, exact=True)
    b1, r1_, b2, r2 = _related(w, r1, r_extra)
    ctx = _ctx(w)
    d1, d2 = to_dev(b1), to_dev(b2)
    try:
        _check(w, b1, r1_, b2, r2, ctx.adapter_gram(d1.ptr, r1_, d2.ptr, r2))
    finally:
        d1.free(); d2.free()
        ctx.close()
