"""FP16 stencils with the halves read inside the FMA and strided neighbours:
the smallest extents (every neighbour a wrap), both time boundaries, both
daggers, full and reconstructed links, column counts around a thread's share,
and columns whose site norms are near both ends of FP32 or zero.

Tolerance per column, relative L2: every stored number (input, link, output)
is within 2^-11 of its size or its site's largest, and three of them enter a
product, 3 * 2^-11 = 1.5e-3; twice that where the hop and the site term cancel.
"""
import numpy as np
import pytest

import synth
from oracle import staggered as S
from oracle import wilson as W
from paper_2201_09004_amd import lq as L

pytestmark = pytest.mark.gpu
TOL = 2 * 3 * 2.0 ** -11
SCALE = np.array([1.0, 1e30, 0.0, 1e-30, 3.0, 1e-3, 7e4])


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = L.lq_init(0)
    yield c
    L.lq_finalize(c)


def check(out, want):
    for o, w in zip(out, want):
        assert np.isfinite(o).all()
        assert np.linalg.norm(o - w) <= TOL * np.linalg.norm(w)


@pytest.mark.parametrize("Lx,ap", [((2, 2, 2, 2), True), ((4, 2, 6, 2), False), ((6, 4, 2, 10), True)])
@pytest.mark.parametrize("n", [1, 3, 7])
def test_wilson(ctx, Lx, ap, n):
    U = synth.su3_field(Lx, 0.4, 31)
    f = L.lq_gauge_load(ctx, Lx, U, antiperiodic=ap)
    psi = synth.gaussian_spinor(Lx, n, 32) * SCALE[:n].reshape((n,) + (1,) * 6)
    act = L.action(L.LQ_WILSON, m=0.1)
    try:
        for prec in (16, 16 | L.LQ_PREC_RECON12):
            check(L.lq_apply(ctx, act, f, L.LQ_OP_D, prec, psi), [W.wilson(U, p, 0.1, ap) for p in psi])
            check(L.lq_apply(ctx, act, f, L.LQ_OP_DDAG, prec, psi),
                  [W.gamma5(W.wilson(U, W.gamma5(p), 0.1, ap)) for p in psi])
            check(L.lq_apply(ctx, act, f, L.LQ_OP_HOP, prec, psi), [-0.5 * W.hop(U, p, ap) for p in psi])
    finally:
        L.lq_field_free(f)


@pytest.mark.parametrize("Lx,ap", [((4, 4, 4, 4), True), ((4, 6, 4, 10), False)])
@pytest.mark.parametrize("n", [1, 5, 7])
def test_staggered(ctx, Lx, ap, n):
    V, Wl = synth.hisq_fields(Lx, 51)
    f = L.lq_hisq_load(ctx, Lx, V, Wl, antiperiodic=ap)
    chi = synth.gaussian_colour(Lx, n, 52) * SCALE[:n].reshape((n,) + (1,) * 5)
    act = L.action(L.LQ_HISQ, m=0.05)
    try:
        check(L.lq_apply(ctx, act, f, L.LQ_OP_D, 16, chi), [S.hisq(V, Wl, c, 0.05, ap) for c in chi])
        check(L.lq_apply(ctx, act, f, L.LQ_OP_HOP, 16, chi), [S.hop(V, Wl, c, ap) for c in chi])
    finally:
        L.lq_field_free(f)
