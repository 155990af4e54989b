"""CG whose scalar steps run inside its vector kernels (few partials) or as
kernels of their own: Wilson normal equations and single-mass HISQ on lattices
at, below and above the limit between the two (1024 tiles of 64 sites), in
every sloppy storage.  The FP64 true residual with the oracle operator meets
the target."""
import pytest

import synth
from oracle import solve as OS
from oracle import staggered as S
from oracle import wilson as W
from paper_2201_09004_amd import lq as L

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = L.lq_init(0)
    yield c
    L.lq_finalize(c)


@pytest.mark.parametrize("Lx,cols", [((4, 4, 4, 2), 3), ((16, 16, 16, 16), 1), ((16, 16, 16, 18), 2)])
@pytest.mark.parametrize("sloppy", [64, 32, 16])
def test_cgne(ctx, Lx, cols, sloppy):
    U = synth.su3_field(Lx, 0.3, 61)
    b = synth.gaussian_spinor(Lx, cols, 62)
    f = L.lq_gauge_load(ctx, Lx, U)
    try:
        x, st = L.lq_solve(ctx, L.action(L.LQ_WILSON, m=0.2), f, L.params(tol=1e-9, sloppy_bits=sloppy), b)
    finally:
        L.lq_field_free(f)
    assert st["status"] == 0
    assert max(OS.rel_residual(lambda v: W.wilson(U, v, 0.2), xi, bi) for xi, bi in zip(x, b)) <= 1e-9


@pytest.mark.parametrize("Lx,cols", [((4, 4, 4, 6), 5), ((16, 16, 16, 32), 1), ((16, 16, 16, 36), 2)])
@pytest.mark.parametrize("sloppy", [64, 32, 16])
def test_hisq_cg(ctx, Lx, cols, sloppy):
    V, Wl = synth.hisq_fields(Lx, 63)
    b = synth.gaussian_colour(Lx, cols, 64)
    f = L.lq_hisq_load(ctx, Lx, V, Wl)
    try:
        x, st = L.lq_solve(ctx, L.action(L.LQ_HISQ, m=0.2), f, L.params(tol=1e-9, sloppy_bits=sloppy), b)
    finally:
        L.lq_field_free(f)
    assert st["status"] == 0
    ev = S.even_mask(Lx)
    for xi, bi in zip(x, b):
        assert OS.rel_residual(lambda v: S.even_normal(V, Wl, v, 0.2), xi, bi * ev) <= 1e-9
