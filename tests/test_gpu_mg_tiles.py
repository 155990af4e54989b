"""Multigrid transfers and coarse stencil on the matrix cores at the edges of
their tiles: aggregates of 81 and 24 sites (no multiple of the four and sixteen
sites of a group), 6, 18 and 30 vectors (one and two row tiles, both partly
filled), 5, 12 and 13 columns (a partly filled and a second column block).

Tolerance per column, relative L2, for FP32: n products of numbers rounded to
2^-24 each, summed in some order, are within (n + 2) 2^-24 of the result in the
worst case and sqrt(n + 2) 2^-24 as errors add up; n = 6 * 81 at the most for the
transfers, and their inputs' norms exceed the restriction's by at most
sqrt(12 V / (2 nv Vc)) <= 13, so 13 * 23 * 6e-8 = 1.8e-5; the coarse operator's
nine blocks of 60: 9 * 60 -> 23 * 6e-8 times its entries' spread, the same bound.
"""
import numpy as np
import pytest

import synth
from oracle import multigrid as MG
from paper_2201_09004_amd import lq as L

pytestmark = pytest.mark.gpu
CASES = [((6, 6, 6, 6), (3, 3, 3, 3), 30, 13), ((6, 6, 6, 6), (3, 3, 3, 3), 18, 5), ((4, 4, 4, 6), (2, 2, 2, 3), 18, 12),
         ((4, 4, 6, 4), (2, 2, 3, 2), 6, 13)]


@pytest.mark.parametrize("Lx,block,nv,cols", CASES)
def test_tiles(Lx, block, nv, cols):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    U = synth.su3_field(Lx, 0.3, 611)
    m, csw, mu = -0.2, 1.0, 0.1
    vecs = synth.gaussian_spinor(Lx, nv, 612)
    Q = MG.block_orthonormalize(vecs, block)
    ctx = L.lq_init(0)
    f = L.lq_gauge_load(ctx, Lx, U)
    act = L.action(L.LQ_TM_CLOVER, m=m, mu=mu, c_sw=csw)
    try:
        L.lq_mg_setup(ctx, act, f, L.mg_params(block=block, n_vec=nv, null_vecs=vecs))
        cshape = (cols, Q.shape[0], 2, nv)
        fine = synth.gaussian_spinor(Lx, cols, 613)
        rng = np.random.default_rng(614)
        vc = rng.standard_normal(cshape) + 1j * rng.standard_normal(cshape)
        got = (L.lq_mg_apply(ctx, act, f, L.LQ_MG_RESTRICT, 32, fine, cshape),
               L.lq_mg_apply(ctx, act, f, L.LQ_MG_PROLONG, 32, vc, fine.shape),
               L.lq_mg_apply(ctx, act, f, L.LQ_MG_COARSE, 32, vc, cshape))
        for k in range(cols):
            want = (MG.restrict(Q, fine[k], Lx, block), MG.prolong(Q, vc[k], Lx, block),
                    MG.coarse_apply(U, Q, block, vc[k], m, csw, mu))
            for g, w in zip(got, want):
                assert np.linalg.norm(g[k] - w) <= 1.8e-5 * np.linalg.norm(w)
        got64 = L.lq_mg_apply(ctx, act, f, L.LQ_MG_COARSE, 64, vc, cshape)
        want = MG.coarse_apply(U, Q, block, vc[-1], m, csw, mu)
        assert np.linalg.norm(got64[-1] - want) <= 1.8e-5 * 2.0 ** -29 * np.linalg.norm(want) + 1e-13 * np.linalg.norm(want)
    finally:
        L.lq_field_free(f)
        L.lq_finalize(ctx)
