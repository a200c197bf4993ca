"""The FP64 triples products whose fragments come straight from memory, at the
sizes where their tiles end: rows and columns one below, at and one above a
block of 16 and a tile of 64, contraction lengths of every remainder by four,
runs of one entry (o = 1) and windows that cut the runs short.  Against the
oracle's terms, element by element, 1e-11 of the term's largest element (FP64
rounding of up to 1e5 terms per element stays near 1e-13)."""
import numpy as np
import pytest
import torch

from oracle import rtcc3 as orc
from paper_2407_18947_amd import _lib
from paper_2407_18947_amd.inputs import make_system, random_state

pytestmark = pytest.mark.gpu
FIELD = np.array([0.01, -0.02, 0.03])


@pytest.mark.parametrize("o,v,wb", [(1, 1, 0), (1, 17, 0), (2, 15, 0), (2, 16, 0), (3, 8, 0), (4, 16, 0), (2, 33, 0),
                                    (17, 3, 0), (5, 13, 7), (4, 18, 11), (6, 11, 40)])
def test_fragment_products(o, v, wb):
    print(f"fragment products o={o} v={v} window_blocks={wb}", flush=True)
    s = make_system(o, v, seed=51)
    m = orc.Model.from_system(s)
    y = random_state(o, v, 9)
    ctx = _lib.Context(s)
    if wb:
        ctx.set_option(_lib.RTCC3_OPT_WINDOW_BLOCKS, wb)
    yd = torch.tensor(y, dtype=torch.complex128, device="cuda")
    td = torch.zeros(ctx.terms_size(), dtype=torch.complex128, device="cuda")
    torch.cuda.synchronize()
    _lib.rtcc3_rhs_terms(ctx.ctx, FIELD, yd, td, 1)
    got = ctx.split_terms(td.cpu().numpy())
    dy = torch.zeros_like(yd)
    _lib.rtcc3_rhs(ctx.ctx, FIELD, yd, dy)  # the windows of the pass without the density
    dy = dy.cpu().numpy()
    ctx.close()
    ref = orc.rhs_terms(m, y, FIELD, triples="explicit" if o * v < 60 else "loop")
    for k in ["X1", "X2", "Y1", "Y2", "D", "mu"]:
        b = ref[k].numpy()
        assert np.abs(got[k] - b).max() <= 1e-11 * np.abs(b).max() + 1e-15, k
    full = np.concatenate([x.ravel() for x in (-1j * (got["R1"] + got["X1"]), -1j * (got["R2"] + got["X2"]),
                                               1j * (got["G1"] + got["Y1"]), 1j * (got["G2"] + got["Y2"]))])
    assert np.abs(dy - full).max() <= 1e-12 * np.abs(full).max() + 1e-15
