"""The engine on the CPU build."""
import pytest

from host_library import host_run


@pytest.mark.parametrize("of_gradient", [0, 1])
def test_derivatives_after_a_dropped_queue(host_library, of_gradient):
    """An error drops the operations that are queued, the clearing of a
    derivative among them: the next evaluation clears it again."""
    host_run(host_library, "dropped_queue", of_gradient)


@pytest.mark.parametrize("M,N,K", [(16, 16, 128), (5, 33, 150)])
@pytest.mark.parametrize("ms,apart", [(0, 0), (0.004, 0), (0.1, 1)])
def test_tuned_split_of_products_in_one_level(host_library, M, N, K, ms, apart):
    """Products that share a level with others into the same output run with the
    split that the tuner found for them by themselves, if it saves more than a
    launch."""
    host_run(host_library, "tuned_level", M, N, K, ms, apart)


@pytest.mark.parametrize("o,v", [(2, 3), (3, 9), (1, 4)])
def test_sum_over_three_runs_takes_no_memory(host_library, o, v):
    host_run(host_library, "three_runs", o, v)


@pytest.mark.parametrize("extents,code", [((2, 31, 17), 0), ((4, 1024, 1024), -1), ((128, 256, 256), -1)])
def test_extent_of_a_sum_over_three_runs(host_library, extents, code):
    """The limit of 2^22 terms holds for the whole sum: more than 161 virtual
    orbitals are refused when a context is created."""
    host_run(host_library, "three_runs_extent", *extents, code)
