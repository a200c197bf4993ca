"""Intermediates are stored over what the last evaluation left, not cleared and
added to.  An evaluation after one of a much larger state gives what it gave
before it, in each precision (the products that store and those that add, at
sizes below and above one tile and with k split or not)."""
import numpy as np
import pytest
import torch

from paper_2407_18947_amd import _lib
from paper_2407_18947_amd.inputs import make_system, random_state

pytestmark = pytest.mark.gpu
FIELD = np.array([0.01, -0.02, 0.03])


@pytest.mark.parametrize("o,v", [(1, 1), (2, 5), (3, 21), (6, 24)])
@pytest.mark.parametrize("prec,tol", [(_lib.RTCC3_FP64, 1e-12), (_lib.RTCC3_FP32, 1e-5), (_lib.RTCC3_BF16X3, 1e-5)])
def test_nothing_is_left_of_the_last_evaluation(o, v, prec, tol):
    print(f"repeated evaluations o={o} v={v} precision={prec}", flush=True)
    s = make_system(o, v, seed=61)
    ctx = _lib.Context(s, prec)

    def run(y):
        yd = torch.tensor(y, dtype=torch.complex128, device="cuda")
        td = torch.full((ctx.terms_size(),), 3.0, dtype=torch.complex128, device="cuda")
        dy = torch.full_like(yd, 5.0)
        torch.cuda.synchronize()
        _lib.rtcc3_rhs_terms(ctx.ctx, FIELD, yd, td, 1)
        _lib.rtcc3_rhs(ctx.ctx, FIELD, yd, dy)
        return dict(ctx.split_terms(td.cpu().numpy()), dy=dy.cpu().numpy())

    y = random_state(o, v, 5)
    first = run(y)
    run(1e3 * random_state(o, v, 6))
    again = run(y)
    ctx.close()
    for name in first:
        # sums in another order: rounding of the precision, relative to the term
        assert np.abs(again[name] - first[name]).max() <= tol * np.abs(first[name]).max() + 1e-15, name
