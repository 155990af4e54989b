"""Launch shapes of the Wilson-type stencils, forced: one hop per wave, and
the register-blocked daggered operators, give bitwise the columns of one thread
per site, which is compared with the oracle (FP64 1e-13, FP32 1e-6)."""
import numpy as np
import pytest

import synth
from oracle import overlap as OV
from oracle import wilson as W
from paper_2201_09004_amd import lq as L

pytestmark = pytest.mark.gpu
TOL = {64: 1e-13, 32: 1e-6}
# 2 Vh = 16, 640, 1440 sites: less than a tile, exact tiles, a ragged tail across the parities
LATS = [(2, 2, 2, 2), (4, 4, 4, 10), (6, 6, 4, 10)]


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = L.lq_init(0)
    yield c
    L.lq_finalize(c)


def _oracle(kind, op, U, v):
    if kind == "wilson":
        f = {L.LQ_OP_D: lambda p: W.wilson(U, p, 0.1), L.LQ_OP_HOP: lambda p: -0.5 * W.hop(U, p),
             L.LQ_OP_DDAG: lambda p: W.gamma5(W.wilson(U, W.gamma5(p), 0.1))}[op]
    elif kind == "tm":
        f = {L.LQ_OP_D: lambda p: W.tm_clover(U, p, 0.1, 1.1, 0.2),
             L.LQ_OP_DDAG: lambda p: W.tm_clover_dag(U, p, 0.1, 1.1, 0.2)}[op]
    else:
        f = lambda p: OV.hw(U, p, 1.5)  # noqa: E731
    return np.array([f(p) for p in v])


@pytest.mark.parametrize("Lx", LATS)
@pytest.mark.parametrize("prec", [64, 32, 32 | L.LQ_PREC_RECON12])
@pytest.mark.parametrize("kind,op", [("wilson", L.LQ_OP_D), ("wilson", L.LQ_OP_DDAG), ("wilson", L.LQ_OP_HOP),
                                     ("tm", L.LQ_OP_D), ("tm", L.LQ_OP_DDAG), ("hw", L.LQ_OP_HW)])
def test_shapes_bitwise(ctx, monkeypatch, Lx, prec, kind, op):
    U = synth.su3_field(Lx, 0.3, 71)
    v = synth.gaussian_spinor(Lx, 5, 72)
    act = {"wilson": lambda: L.action(L.LQ_WILSON, m=0.1),
           "tm": lambda: L.action(L.LQ_TM_CLOVER, m=0.1, mu=0.2, c_sw=1.1),
           "hw": lambda: L.action(L.LQ_OVERLAP, m=0.0, rho=1.5, cheb_N=1)}[kind]()
    f = L.lq_gauge_load(ctx, Lx, U)
    try:
        out = {}
        for shape in ("1,0", "-8,0", "2,0", "3,0", "4,0"):
            monkeypatch.setenv("LQ_TUNE_FORCE", shape)
            out[shape] = L.lq_apply(ctx, act, f, op, prec, v)
    finally:
        L.lq_field_free(f)
    want = _oracle(kind, op, U, v)
    assert np.linalg.norm(out["1,0"] - want) < TOL[prec & ~L.LQ_PREC_RECON12] * np.linalg.norm(want)
    for shape, o in out.items():
        assert np.array_equal(o, out["1,0"]), shape


def test_cgne_same_under_every_shape(ctx, monkeypatch):
    """|D p|^2 of the epilogue is summed alike too: the whole solve is bitwise the same."""
    Lx = (6, 6, 4, 10)
    U = synth.su3_field(Lx, 0.3, 73)
    b = synth.gaussian_spinor(Lx, 2, 74)
    f = L.lq_gauge_load(ctx, Lx, U)
    try:
        x = []
        for shape in ("1,0", "-8,0"):
            monkeypatch.setenv("LQ_TUNE_FORCE", shape)
            x.append(L.lq_solve(ctx, L.action(L.LQ_WILSON, m=0.2), f, L.params(tol=1e-9, sloppy_bits=32), b)[0])
    finally:
        L.lq_field_free(f)
    assert np.array_equal(x[0], x[1])
