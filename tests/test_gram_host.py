"""salt_adapter_gram's host side on the CPU build of the library
(tests/cpu_kernels/gram.cpp): what a context's first call allocates, how large the
scratch is where one table is much wider than the others, and the answer where the
device has no room for every K chunk's Grams."""
import pytest

from tests import cpu_build

pytestmark = pytest.mark.skipif(not cpu_build.available(), reason="needs the ROCm host clang")


@pytest.mark.parametrize("check,r1,r2", [("first_call", 3, 2), ("scratch", 16, 9), ("scratch", 17, 32),
                                         ("scratch", 33, 2), ("no_memory", 16, 9), ("no_memory", 17, 32),
                                         ("no_memory", 33, 2)])
def test_gram(check, r1, r2):
    r = cpu_build.program("gram", check, str(r1), str(r2))
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
