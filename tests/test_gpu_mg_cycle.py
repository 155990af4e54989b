"""The multigrid cycle with its fused passes: column counts that no column
block divides, pre-smoothing, cycles shorter and longer than one pass of eight
directions.  A wrong residual, smoothing step or correction would still converge
through the FP64 updates, but in more steps: the counts are held to those of the
unfused cycle (65, 101, 45, 62, 43) plus two, and the residual with the oracle
operator to the target."""
import pytest

import synth
from oracle import solve as OS
from oracle import wilson as W
from paper_2201_09004_amd import lq as L

pytestmark = pytest.mark.gpu
M, MU, CSW = -0.0695, 0.01, 1.0509


@pytest.mark.parametrize("nu_pre,kmax,cols,steps", [(0, 8, 12, 65), (0, 3, 5, 101), (1, 8, 1, 45), (0, 10, 3, 62),
                                                    (1, 17, 4, 43)])
def test_cycle_steps(nu_pre, kmax, cols, steps):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    Lx = (8, 8, 8, 8)
    U = synth.su3_field(Lx, 0.2, 81)
    b = synth.point_sources(Lx)[:cols]
    ctx = L.lq_init(0)
    f = L.lq_gauge_load(ctx, Lx, U)
    act = L.action(L.LQ_TM_CLOVER, m=M, mu=MU, c_sw=CSW)
    try:
        L.lq_mg_setup(ctx, act, f, L.mg_params(n_vec=6, seed=3, nu_pre=nu_pre, gcr_kmax=kmax, nu_post=2))
        x, st = L.lq_solve(ctx, act, f, L.params(tol=1e-10, solver=3), b)
    finally:
        L.lq_field_free(f)
        L.lq_finalize(ctx)
    assert st["status"] == 0 and st["iters"] <= steps + 2
    F = W.field_strength(U)
    for xi, bi in zip(x[:2], b[:2]):
        assert OS.rel_residual(lambda v: W.tm_clover(U, v, M, CSW, MU, F=F), xi, bi) <= 1e-10
