"""The engine on the CPU build."""
import pytest

from host_library import host_library, host_run  # noqa: F401


@pytest.mark.parametrize("of_gradient", [0, 1])
def test_derivatives_after_a_dropped_queue(host_library, of_gradient):  # noqa: F811
    """An error drops the operations that are queued, the clearing of a
    derivative among them: the next evaluation clears it again."""
    host_run(host_library, "dropped_queue", of_gradient)
