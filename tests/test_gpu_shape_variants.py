"""Every number of columns per thread, forced, in every storage that has it:
bitwise the results of one column per thread (1, 2, 3, 4, 6, and one hop per
wave as -8; a number that a kernel does not have falls to 1)."""
import numpy as np
import pytest
import torch

import synth
from paper_2201_09004_amd import lq as L

pytestmark = pytest.mark.gpu
SHAPES = ("2,0", "3,0", "4,0", "6,0", "-8,0")


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = L.lq_init(0)
    yield c
    L.lq_finalize(c)


@pytest.mark.parametrize("kind,prec", [(L.LQ_WILSON, 64), (L.LQ_WILSON, 32), (L.LQ_WILSON, 16),
                                       (L.LQ_TM_CLOVER, 64), (L.LQ_TM_CLOVER, 32)])
def test_daggered_operator(ctx, monkeypatch, kind, prec):
    Lx = (6, 4, 4, 10)
    f = L.lq_gauge_load(ctx, Lx, synth.su3_field(Lx, 0.3, 71))
    v = synth.gaussian_spinor(Lx, 7, 72)
    act = L.action(kind, m=0.1, mu=0.2, c_sw=1.1) if kind == L.LQ_TM_CLOVER else L.action(kind, m=0.1)
    try:
        monkeypatch.setenv("LQ_TUNE_FORCE", "1,0")
        want = L.lq_apply(ctx, act, f, L.LQ_OP_DDAG, prec, v)
        for shape in SHAPES:
            monkeypatch.setenv("LQ_TUNE_FORCE", shape)
            assert np.array_equal(L.lq_apply(ctx, act, f, L.LQ_OP_DDAG, prec, v), want), shape
    finally:
        L.lq_field_free(f)


@pytest.mark.parametrize("sloppy", [64, 32, 16])
@pytest.mark.parametrize("cols", [5, 7])
def test_cgne(ctx, monkeypatch, sloppy, cols):
    """D p with |D p|^2 per column (the fused reduction over ragged column groups): a whole solve."""
    Lx = (6, 6, 4, 10)
    f = L.lq_gauge_load(ctx, Lx, synth.su3_field(Lx, 0.3, 73))
    b = synth.gaussian_spinor(Lx, cols, 74)
    prm = L.params(tol=1e-9, sloppy_bits=sloppy)
    act = L.action(L.LQ_WILSON, m=0.2)
    try:
        monkeypatch.setenv("LQ_TUNE_FORCE", "1,0")
        want, st = L.lq_solve(ctx, act, f, prm, b)
        assert st["status"] == 0
        for shape in SHAPES:
            monkeypatch.setenv("LQ_TUNE_FORCE", shape)
            assert np.array_equal(L.lq_solve(ctx, act, f, prm, b)[0], want), shape
    finally:
        L.lq_field_free(f)


@pytest.mark.parametrize("cols", [5, 7])
@pytest.mark.parametrize("nu_pre", [0, 1])
def test_multigrid_cycle(ctx, monkeypatch, cols, nu_pre):
    """The cycle's residual, its odd sites added onto the correction, source and Schur stencils."""
    Lx = (8, 8, 8, 8)
    f = L.lq_gauge_load(ctx, Lx, synth.su3_field(Lx, 0.2, 81))
    act = L.action(L.LQ_TM_CLOVER, m=-0.0695, mu=0.01, c_sw=1.0509)
    b = synth.point_sources(Lx)[:cols]
    prm = L.params(tol=1e-8, solver=3)
    try:
        monkeypatch.setenv("LQ_TUNE_FORCE", "1,0")
        L.lq_mg_setup(ctx, act, f, L.mg_params(n_vec=6, seed=3, nu_pre=nu_pre, nu_post=2))
        want, st = L.lq_solve(ctx, act, f, prm, b)
        assert st["status"] == 0
        for shape in SHAPES:
            monkeypatch.setenv("LQ_TUNE_FORCE", shape)
            assert np.array_equal(L.lq_solve(ctx, act, f, prm, b)[0], want), shape
    finally:
        L.lq_field_free(f)
