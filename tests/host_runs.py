"""What the tests of the library's CPU build run, each in its own process:
python host_runs.py LIBRARY FUNCTION ARGUMENTS."""
import ctypes
import os
import sys

import numpy as np

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
from paper_2407_18947_amd import _lib  # noqa: E402
from paper_2407_18947_amd.inputs import make_system, random_state  # noqa: E402

FIELD = np.array([0.01, -0.02, 0.03])


def device(a):
    """A copy of an array in an allocation of its own."""
    a = np.ascontiguousarray(a, dtype=np.complex128)
    L = _lib.load()
    L.emu_alloc.restype, L.emu_alloc.argtypes = ctypes.c_void_p, [ctypes.c_size_t]
    b = np.frombuffer((ctypes.c_char * a.nbytes).from_address(L.emu_alloc(a.nbytes)), dtype=np.complex128)
    b = b.reshape(a.shape)
    b[...] = a
    return b


def evaluate(o, v, precision, blocks, tol):
    """Terms and right-hand side against the oracle, to tol of a term's largest element."""
    from oracle import rtcc3 as orc
    o, v, precision, blocks, tol = int(o), int(v), int(precision), int(blocks), float(tol)
    s = make_system(o, v, seed=51)
    y = random_state(o, v, 9)
    ctx = _lib.Context(s, precision)
    if blocks:
        ctx.set_option(_lib.RTCC3_OPT_WINDOW_BLOCKS, blocks)
    yd, td, dy = device(y), device(np.zeros(ctx.terms_size())), device(np.zeros(y.size))
    _lib.rtcc3_rhs_terms(ctx.ctx, FIELD, yd, td, 1)
    got = ctx.split_terms(td)
    _lib.rtcc3_rhs(ctx.ctx, FIELD, yd, dy)
    ctx.close()
    ref = orc.rhs_terms(orc.Model.from_system(s), y, FIELD, triples="explicit")
    for k in ["R1", "R2", "G1", "G2", "X1", "X2", "Y1", "Y2", "D", "mu"]:
        b = ref[k].numpy()
        assert np.abs(got[k] - b).max() <= tol * np.abs(b).max() + 1e-15, (k, np.abs(got[k] - b).max())
    full = np.concatenate([x.ravel() for x in (-1j * (got["R1"] + got["X1"]), -1j * (got["R2"] + got["X2"]),
                                               1j * (got["G1"] + got["Y1"]), 1j * (got["G2"] + got["Y2"]))])
    assert np.abs(dy - full).max() <= tol * np.abs(full).max() + 1e-15


def seg_slot(v, slot):
    """A block of a segmented product far up in the window."""
    f = _lib.load().drive_seg_slot
    f.restype = ctypes.c_double
    err = f(int(v), int(slot))
    # five terms of order one per element
    assert err <= 1e-13, err


def dropped_queue(of_gradient):
    """Derivatives after an evaluation that ended in an error."""
    f = _lib.load().drive_dropped_queue
    f.restype = ctypes.c_double
    err = f(int(of_gradient))
    assert err == 0.0, err


def tuned_level(M, N, K, ms, apart):
    """Two products into one output: launches of their own where their split saves enough."""
    f = _lib.load().drive_tuned_level
    f.restype = ctypes.c_double
    n = (ctypes.c_long * 2)()
    f.argtypes = [ctypes.c_int] * 3 + [ctypes.c_double, ctypes.c_void_p]
    err = f(int(M), int(N), int(K), float(ms), n)
    # 2K products of order one each in both parts
    assert err <= 1e-13 * int(K), err
    assert list(n) == ([2, 0] if int(apart) else [0, 1]), list(n)


def three_runs(o, v):
    """A sum over three runs of indices needs no copy, and reserves none."""
    f = _lib.load().drive_three_runs
    f.restype = ctypes.c_double
    extra = ctypes.c_size_t()
    err = f(int(o), int(v), ctypes.byref(extra))
    # v^3 products of order one
    assert err <= 1e-14 * int(v) ** 3, err
    assert extra.value == 0, extra.value


def three_runs_extent(b, d, e, code):
    """Sums longer than a product takes are refused, also where a run becomes a batch."""
    got = _lib.load().drive_three_runs_extent(int(b), int(d), int(e))
    assert got == int(code), got


def precision_switch(o, v, first, then):
    """A context switched to another precision evaluates, with what it allocated
    when it was created, like one created with it."""
    o, v = int(o), int(v)
    s, y = make_system(o, v, seed=41), device(random_state(o, v, 5))
    terms = []
    for precision in (int(first), int(then)):
        ctx = _lib.Context(s, precision)
        if precision != int(then):
            ctx.set_option(_lib.RTCC3_OPT_PRECISION, int(then))
        td = device(np.zeros(ctx.terms_size()))
        _lib.rtcc3_rhs_terms(ctx.ctx, FIELD, y, td, 1)
        terms.append(ctx.split_terms(td))
        ctx.close()
    for name in terms[0]:
        a, b = terms[0][name], terms[1][name]
        # the same arithmetic; FP64 sums in another order
        assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max() + 1e-15, name


def launch_count(o, v, precision, steps, tangent):
    """rtcc3_last_timing()[2] against the launches themselves: two numbers of
    windows of one system differ by the kernels of the windows alone."""
    o, v, precision, steps, tangent = int(o), int(v), int(precision), int(steps), int(tangent)
    L = _lib.load()
    ctx = _lib.Context(make_system(o, v, seed=3), precision)
    if tangent:
        ctx.set_option(_lib.RTCC3_OPT_TANGENT, 1)
    ctx.set_state(random_state(o, v, 2))
    field = np.zeros((2 * steps + 1, 3))
    seen = []
    for blocks in (0, 6):
        ctx.set_option(_lib.RTCC3_OPT_WINDOW_BLOCKS, blocks)
        L.emu_reset_launches()
        if tangent:
            ctx.propagate_tangent(steps, 0.05, field, np.ones_like(field))
        else:
            ctx.propagate(steps, 0.05, field)
        seen.append((L.emu_launches(b""), _lib.rtcc3_last_timing(ctx.ctx)[2]))
    ctx.close()
    assert seen[1][0] > seen[0][0], seen
    assert seen[1][0] - seen[0][0] == seen[1][1] - seen[0][1], seen


def products(seed, count):
    """Plain products of random forms; errors in units of their bound."""
    f = _lib.load().drive_products
    f.restype = ctypes.c_double
    err = f(int(seed), int(count))
    assert err <= 1.0, err


def product(*args):
    """One plain product: its six extents, batch, form and split of k."""
    a = [int(x) for x in args]
    f = _lib.load().drive_product
    f.restype = ctypes.c_double
    err = f((ctypes.c_int * 6)(*a[:6]), *a[6:])
    assert err <= 1.0, err


def block(o, v, one_by_one):
    """Block products with all groups in a launch, or one group at a time."""
    f = _lib.load().drive_block
    f.restype = ctypes.c_double
    n = ctypes.c_long()
    err = f(int(o), int(v), int(one_by_one), ctypes.byref(n))
    # o^2 v^2 products of order one
    assert err <= 1e-14 * int(o) ** 2 * int(v) ** 2, err
    assert n.value == (8 if int(one_by_one) else 2), n.value


if __name__ == "__main__":
    _lib.LIBPATH = sys.argv[1]
    globals()[sys.argv[2]](*sys.argv[3:])
