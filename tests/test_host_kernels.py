"""Single kernels on the CPU build."""
import pytest

from host_library import host_library, host_run  # noqa: F401


@pytest.mark.parametrize("v,slot", [(2, 0), (17, 3), (2, 2 ** 27 - 1), (2, 2 ** 27), (9, 2 ** 22)])
def test_build_product_at_slot(host_library, v, slot):  # noqa: F811
    """Blocks whose elements lie below and above 2^32 in the window (a window of
    fewer than six times the occupied orbitals' blocks is not cut any smaller)."""
    host_run(host_library, "seg_slot", v, slot)
