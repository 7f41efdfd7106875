"""Plan builds at the edges of their kernels' ranges: batches carried in the kernel's
arguments (up to 64 tokens), sorted by one block of each size (up to 256, 512, 2048
and 4096, read from the staging buffer in place), sorted in chunks (above); runs of 64 keys and their merges filled to the last key and one past it.
Plan and outputs against the oracle (integer inputs, bit-exact)."""
import numpy as np
import pytest

from tests import cpu_build
from tests.test_gpu_tiles import _run_all, _workload
from tests.test_host_kernels import _check

SIZES = [1, 2, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1531, 2048, 2049, 4096, 4097, 8192, 8193]


def _batch(T):
    w = _workload(900 + T, [("a", 8, 16)], 5, 8, T, min(60, T), (1, 2), exact=True)
    if T > 2:                                     # some tokens without a centroid, some without a slot
        w.tok_c[::7] = -1
        w.tok_u[::11] = -1
    return w


@pytest.mark.skipif(not cpu_build.available(), reason="needs the ROCm host clang")
@pytest.mark.parametrize("T", [1, 65, 300, 1531, 2049])
def test_on_the_cpu(T, tmp_path):
    w = _batch(T)
    mean = T / len(np.unique(w.tok_c))
    _check(w, tmp_path, 16 if mean <= 24 else (32 if mean <= 96 else (64 if mean <= 384 else 128)), exact=True)


@pytest.mark.gpu
@pytest.mark.parametrize("T", SIZES)
def test_on_the_gpu(T):
    print(f"\n[gpu case] plan of {T} tokens", flush=True)
    _run_all(_batch(T), exact=True)
