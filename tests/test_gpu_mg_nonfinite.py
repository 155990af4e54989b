"""Multigrid on a batch in which a source is not finite (or overflows the
cycle's FP32, or is zero): the other columns are solved as ever."""
import numpy as np
import pytest
import torch

import synth
from oracle import solve as OS
from oracle import wilson as W
from paper_2201_09004_amd import lq as L

pytestmark = pytest.mark.gpu
M, MU, CSW = -0.0695, 0.01, 1.0509


@pytest.mark.parametrize("factor", [np.nan, np.inf, 1e100, 0.0])
def test_other_columns_are_solved(factor):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    Lx = (8, 8, 8, 8)
    U = synth.su3_field(Lx, 0.2, 81)
    b = synth.gaussian_spinor(Lx, 5, 82)
    bad = b.copy()
    bad[1] *= factor
    bad[3] *= factor
    act = L.action(L.LQ_TM_CLOVER, m=M, mu=MU, c_sw=CSW)
    ctx = L.lq_init(0)
    f = L.lq_gauge_load(ctx, Lx, U)
    try:
        L.lq_mg_setup(ctx, act, f, L.mg_params(n_vec=6, seed=3, gcr_kmax=8, nu_post=2))
        x, st = L.lq_solve(ctx, act, f, L.params(tol=1e-9, solver=3), bad)
    finally:
        L.lq_field_free(f)
        L.lq_finalize(ctx)
    assert st["status"] == 0
    F = W.field_strength(U)
    for k in (0, 2, 4):
        assert OS.rel_residual(lambda v: W.tm_clover(U, v, M, CSW, MU, F=F), x[k], b[k]) <= 1e-9
    assert factor != 0.0 or not (x[1].any() or x[3].any())
