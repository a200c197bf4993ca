"""Whole evaluations on the CPU build, where every access is checked against its
allocation and every buffer load against its resource: the smallest blocks,
whose rows are fewer than the steps the gathered products load ahead (up to 12
virtual orbitals), and one above, in one window and in several."""
import pytest

from host_library import host_run


@pytest.mark.parametrize("o,v,blocks", [(1, 1, 0), (1, 4, 0), (2, 5, 0), (3, 3, 0), (3, 3, 7), (2, 8, 0), (2, 12, 0),
                                        (2, 13, 0)])
def test_fp64(host_library, o, v, blocks):
    # FP64 rounding of up to 1e4 terms per element stays near 1e-14
    host_run(host_library, "evaluate", o, v, 0, blocks, 1e-12)


@pytest.mark.parametrize("o,v", [(2, 3), (2, 9)])
@pytest.mark.parametrize("precision", [1, 2, 3])
def test_reduced_precisions(host_library, o, v, precision):
    # FP32 keeps 24 bits, three bf16 slices as many, two 16; sums of up to 1e4
    # terms of either sign lose a few more
    host_run(host_library, "evaluate", o, v, precision, 0, 2e-3 if precision == 3 else 1e-4)


@pytest.mark.parametrize("o,v", [(1, 1), (1, 3), (3, 1), (2, 4)])
@pytest.mark.parametrize("first,then", [(2, 0), (1, 0), (0, 2), (0, 1)])
def test_precision_switch(host_library, o, v, first, then):
    host_run(host_library, "precision_switch", o, v, first, then)


@pytest.mark.parametrize("o,v,precision,steps,tangent", [
    (3, 3, 0, 0, 0), (3, 3, 0, 1, 0), (3, 3, 1, 0, 0), (3, 3, 2, 0, 0), (3, 2, 0, 0, 1), (3, 2, 2, 0, 1)])
def test_launches_counted(host_library, o, v, precision, steps, tangent):
    """The dipole's pass alone, steps, each kind of precision and derivatives."""
    host_run(host_library, "launch_count", o, v, precision, steps, tangent)
