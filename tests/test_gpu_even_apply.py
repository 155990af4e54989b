"""Even-site operators through lq_apply at the edges of the pack kernels' tiles
(32 checkerboard indices per workgroup for Wilson-type columns, 128 for
staggered ones): one partial workgroup, one exact, one index past it.  The odd
sites of the output are zero whatever it held before, and odd sites of the
input do not enter.

Tolerances (relative L2) as in test_gpu_parity.py: FP64 1e-12 for operators of
two stencils, FP32 1e-6, FP16 3e-3.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import lattice as lat
from oracle import staggered as S
from oracle import wilson as W
from paper_2201_09004_amd import lq as L

pytestmark = pytest.mark.gpu
TOL = {64: 1e-12, 32: 1e-6, 16: 3e-3}


@pytest.fixture(scope="module")
def ctx():
    c = L.lq_init(0)
    yield c
    L.lq_finalize(c)


def _apply(ctx, act, f, op, prec, v):
    inp = torch.from_numpy(v).cuda()
    out = torch.full_like(inp, complex(float("nan"), float("nan")))
    return L.lq_apply(ctx, act, f, op, prec, inp, out).cpu().numpy()


@pytest.mark.parametrize("Lx", [(2, 2, 2, 2), (4, 4, 2, 2), (4, 2, 2, 6)])  # Vh = 8, 32, 48
@pytest.mark.parametrize("prec,cols", [(64, 1), (32, 5)])
def test_schur_edges(ctx, Lx, prec, cols):
    U = synth.su3_field(Lx, 0.2, 41)
    v = synth.gaussian_spinor(Lx, cols, 42)
    f = L.lq_gauge_load(ctx, Lx, U)
    try:
        out = _apply(ctx, L.action(L.LQ_TM_CLOVER, m=0.1, mu=0.05, c_sw=1.0), f, L.LQ_OP_SCHUR, prec, v)
    finally:
        L.lq_field_free(f)
    eo = W.EvenOdd(U, 0.1, 1.0, 0.05)
    want = np.array([eo.mhat(c) for c in v])
    assert np.all(out[:, lat.parity(Lx) == 1] == 0)
    assert np.linalg.norm(out - want) < TOL[prec] * np.linalg.norm(want)


@pytest.mark.parametrize("Lx", [(4, 4, 4, 4), (4, 4, 4, 6), (4, 4, 4, 10)])  # Vh = 128, 192, 320
@pytest.mark.parametrize("prec,cols", [(64, 3), (32, 1), (16, 4)])
def test_normal_even_edges(ctx, Lx, prec, cols):
    V, Wl = synth.hisq_fields(Lx, 43)
    v = synth.gaussian_colour(Lx, cols, 44)
    f = L.lq_hisq_load(ctx, Lx, V, Wl)
    try:
        out = _apply(ctx, L.action(L.LQ_HISQ, m=0.1), f, L.LQ_OP_NORMAL_EVEN, prec, v)
    finally:
        L.lq_field_free(f)
    want = np.array([S.even_normal(V, Wl, c, 0.1) for c in v])
    assert np.all(out[:, lat.parity(Lx) == 1] == 0)
    assert np.linalg.norm(out - want) < TOL[prec] * np.linalg.norm(want)
