"""The dipole by itself, which leaves out the triples' amplitude terms, against
the one that comes with them, with one window and with pair windows, each after
an evaluation of another state."""
import numpy as np
import pytest
import torch

from paper_2407_18947_amd import _lib
from paper_2407_18947_amd.inputs import make_system, random_state

pytestmark = pytest.mark.gpu
FIELD = np.array([0.01, -0.02, 0.03])


@pytest.mark.parametrize("o,v,wb", [(1, 2, 0), (3, 9, 0), (5, 17, 0), (4, 18, 11), (17, 2, 0)])
@pytest.mark.parametrize("prec", [_lib.RTCC3_FP64, _lib.RTCC3_BF16X3])
def test_dipole_alone(o, v, wb, prec):
    print(f"dipole alone o={o} v={v} window_blocks={wb} precision={prec}", flush=True)
    ctx = _lib.Context(make_system(o, v, seed=81), prec)
    if wb:
        ctx.set_option(_lib.RTCC3_OPT_WINDOW_BLOCKS, wb)
    y, other = (torch.tensor(random_state(o, v, k), dtype=torch.complex128, device="cuda") for k in (3, 4))
    ctx.set_state(random_state(o, v, 3))
    td = torch.zeros(ctx.terms_size(), dtype=torch.complex128, device="cuda")
    torch.cuda.synchronize()
    _lib.rtcc3_rhs_terms(ctx.ctx, FIELD, y, td, 1)
    with_terms = ctx.split_terms(td.cpu().numpy())["mu"]
    _lib.rtcc3_rhs_terms(ctx.ctx, FIELD, other, td, 1)
    alone = np.asarray(_lib.rtcc3_dipole(ctx.ctx, FIELD))
    ctx.close()
    # the same sums in another order; a reduced precision forms them alike
    assert np.abs(alone - with_terms).max() <= 1e-12 * max(1.0, np.abs(with_terms).max())
