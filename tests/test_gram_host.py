"""salt_adapter_gram's host side on the CPU build of the library
(tests/cpu_kernels/gram.cpp): what a context's first call allocates."""
import pytest

from tests import cpu_build

pytestmark = pytest.mark.skipif(not cpu_build.available(), reason="needs the ROCm host clang")


@pytest.mark.parametrize("check,r1,r2", [("first_call", 3, 2)])
def test_gram(check, r1, r2):
    r = cpu_build.program("gram", check, str(r1), str(r2))
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
