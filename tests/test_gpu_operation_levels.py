"""Queued operations against one evaluation at a time: the terms and the
right-hand side of sizes whose products are all small (one launch for several),
all large, and mixed, with sums of several products into one output, on one and
on several streams."""
import numpy as np
import pytest
import torch

from oracle import rtcc3 as orc
from paper_2407_18947_amd import _lib
from paper_2407_18947_amd.inputs import make_system, random_state

pytestmark = pytest.mark.gpu
FIELD = np.array([0.01, -0.02, 0.03])


@pytest.mark.parametrize("o,v", [(1, 2), (2, 3), (3, 16), (2, 40), (6, 17)])
@pytest.mark.parametrize("single", [0, 1])
def test_terms_of_queued_operations(o, v, single):
    print(f"operation levels o={o} v={v} single_stream={single}", flush=True)
    s = make_system(o, v, seed=71)
    y = random_state(o, v, 8)
    ctx = _lib.Context(s)
    ctx.set_option(_lib.RTCC3_OPT_SINGLE_STREAM, single)
    yd = torch.tensor(y, dtype=torch.complex128, device="cuda")
    td = torch.zeros(ctx.terms_size(), dtype=torch.complex128, device="cuda")
    torch.cuda.synchronize()
    for _ in range(2):
        _lib.rtcc3_rhs_terms(ctx.ctx, FIELD, yd, td, 1)
    got = ctx.split_terms(td.cpu().numpy())
    ctx.close()
    ref = orc.rhs_terms(orc.Model.from_system(s), y, FIELD, triples="explicit" if o * v < 60 else "loop")
    for k in ["R1", "R2", "G1", "G2", "Y1", "D", "mu"]:
        b = ref[k].numpy()
        # FP64 rounding of up to 1e5 terms per element stays near 1e-13
        assert np.abs(got[k] - b).max() <= 1e-11 * np.abs(b).max() + 1e-15, k
