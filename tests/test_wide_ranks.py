"""The apply of residual ranks above 2 and of 128-token tiles (in the lane layouts)
at the sizes where it can go wrong: ranks at the edges of the 16-rank chunks, the
8-rank passes and the row groups, tiles that hold narrow and wide ranks side by
side, tokens with and without a centroid, every tile size, centroid ranks that
fill their fragments or not, rows shorter than a step or a chunk and past one by
eight elements.  Integer inputs, which must come out bit-exact (every partial sum
is an integer below 2^24), on the CPU build of the kernel sources under
AddressSanitizer and on the GPU."""
import numpy as np
import pytest

from paper_2608_03579_amd import synth
from tests import cpu_build
from tests.test_gpu_tiles import _run_all
from tests.test_host_kernels import _check

SHAPES = [("a", 8, 136), ("b", 136, 8), ("c", 648, 264)]

CASES = [
    # name, dtype, C, r_c, T, n_slots, ranks, tile tokens
    ("m16 ranks 0-18", "bf16", 3, 40, 40, 14, (0, 1, 3, 8, 9, 15, 16, 17, 18), 16),
    ("m32 ranks 1/2/66/72", "bf16", 2, 64, 100, 12, (1, 2, 66, 72), 32),
    ("m64 ranks 2/3", "bf16", 1, 24, 130, 9, (2, 3), 64),
    ("m64 no centroid ranks 4/33", "bf16", 0, 0, 150, 10, (4, 33), 64),
    ("m128 rank 1", "bf16", 1, 8, 420, 20, (1,), 128),
    ("m128 rank 1 r_c 72", "bf16", 1, 72, 410, 20, (1,), 128),
    ("m128 ranks 0/2", "bf16", 1, 56, 390, 20, (0, 2), 128),
    ("m128 ranks 1/17", "bf16", 1, 72, 400, 20, (1, 17), 128),
    ("fp32 ranks 1/5/20", "f32", 2, 24, 36, 10, (1, 5, 20), 16),
]


def _workload(name, dtype, C, r_c, T, n_slots, ranks):
    """Every rank of `ranks` occurs; about a sixth of the users carry no centroid (but for 128-token tiles)."""
    rng = np.random.default_rng([2608, 3579, 91, len(name), T])
    slot_rank = np.resize(np.asarray(ranks, np.int32), n_slots)
    rng.shuffle(slot_rank)
    tok_u = np.concatenate([np.arange(n_slots), rng.integers(0, n_slots, size=T - n_slots)]).astype(np.int32)
    rng.shuffle(tok_u)
    user_c = rng.integers(0, max(C, 1), size=n_slots).astype(np.int32)
    if C == 0 or T < 300:
        user_c[rng.random(n_slots) < (1.0 if C == 0 else 0.17)] = -1
    return synth.Workload(cfg=9, seed=len(name) + T, name="wide ranks", dtype=dtype, tables=SHAPES, n_centroids=C,
                          r_c=r_c, n_slots=n_slots, r_u_max=int(slot_rank.max()), slot_rank=slot_rank,
                          tok_c=user_c[tok_u], tok_u=tok_u, gamma=None, y0_kind="int", exact=True)


@pytest.mark.skipif(not cpu_build.available(), reason="needs the ROCm host clang")
@pytest.mark.parametrize("name,dtype,C,r_c,T,n_slots,ranks,m", CASES)
def test_on_the_cpu(name, dtype, C, r_c, T, n_slots, ranks, m, tmp_path):
    _check(_workload(name, dtype, C, r_c, T, n_slots, ranks), tmp_path, m, exact=True)


@pytest.mark.gpu
@pytest.mark.parametrize("name,dtype,C,r_c,T,n_slots,ranks,m", CASES)
def test_on_the_gpu(name, dtype, C, r_c, T, n_slots, ranks, m):
    print(f"\n[gpu case] wide ranks: {name}", flush=True)
    _run_all(_workload(name, dtype, C, r_c, T, n_slots, ranks), want_m=m, exact=True)
