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


@pytest.mark.parametrize("prec,tol", [(64, 1e-13), (32, 1e-6)])
@pytest.mark.parametrize("op", [L.LQ_OP_SITE, L.LQ_OP_SITE_INV])
def test_site_term(ctx, prec, tol, op):
    """Column counts around the columns per thread: each column as in a call of its own, A A^-1 = 1."""
    Lx = (6, 4, 4, 10)
    f = L.lq_gauge_load(ctx, Lx, synth.su3_field(Lx, 0.3, 71))
    act = L.action(L.LQ_TM_CLOVER, m=0.1, mu=0.2, c_sw=1.1)
    v = synth.gaussian_spinor(Lx, 13, 72)
    try:
        one = np.concatenate([L.lq_apply(ctx, act, f, op, prec, v[k:k + 1]) for k in range(13)])
        for n in (2, 3, 4, 5, 7, 8, 9, 13):
            assert np.array_equal(L.lq_apply(ctx, act, f, op, prec, v[:n]), one[:n]), n
        other = L.LQ_OP_SITE_INV if op == L.LQ_OP_SITE else L.LQ_OP_SITE
        back = L.lq_apply(ctx, act, f, other, prec, one)
    finally:
        L.lq_field_free(f)
    # |A| |A^-1| < 4 here: a few roundings of each storage
    assert np.linalg.norm(back - v) < 10 * tol * np.linalg.norm(v)


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9])
def test_site_term_beyond_the_cache(ctx, n):
    """FP64 A with more than 128 MiB of matrices: two and four columns per thread, as on a lattice with fewer."""
    small, big = (4, 4, 4, 4), (16, 16, 32, 32)
    act = L.action(L.LQ_TM_CLOVER, m=0.1, mu=0.2, c_sw=1.1)
    U = torch.from_numpy(synth.su3_field(small, 0.3, 71)).reshape(4, 4, 4, 4, 4, 3, 3)  # t, z, y, x
    v = torch.from_numpy(synth.gaussian_spinor(small, n, 72)).reshape(n, 4, 4, 4, 4, 12)
    reps = [big[3 - k] // 4 for k in range(4)]
    Ub = U.repeat(*reps, 1, 1, 1).reshape(-1, 4, 3, 3).contiguous().cuda()
    vb = v.repeat(1, *reps, 1).reshape(n, -1, 4, 3).contiguous().cuda()
    fs = L.lq_gauge_load(ctx, small, U.reshape(-1, 4, 3, 3).contiguous().numpy(), antiperiodic=False)
    fb = L.lq_gauge_load(ctx, big, Ub, antiperiodic=False)
    try:
        want = torch.from_numpy(L.lq_apply(ctx, act, fs, L.LQ_OP_SITE, 64, v.reshape(n, -1, 4, 3).numpy()))
        got = L.lq_apply(ctx, act, fb, L.LQ_OP_SITE, 64, vb)
    finally:
        L.lq_field_free(fs)
        L.lq_field_free(fb)
    want = want.reshape(n, 4, 4, 4, 4, 12).repeat(1, *reps, 1).reshape(got.shape)
    assert torch.equal(got.cpu(), want)
