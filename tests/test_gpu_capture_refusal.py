"""A call that the library refuses for its arguments leaves the caller's stream
alone: a capture that is under way on it ends and replays as if the call had not
been made."""
import ctypes as C
import gc

import pytest
import torch

from paper_2201_09004_amd import lq as L

pytestmark = pytest.mark.gpu
LX = (4, 4, 4, 4)
V = 256


@pytest.mark.parametrize("kind,ops", [
    (L.LQ_WILSON, [L.LQ_OP_SITE, L.LQ_OP_SITE_INV, L.LQ_OP_SCHUR, L.LQ_OP_SIGN, L.LQ_OP_NORMAL_EVEN, 9, -1]),
    (L.LQ_TM_CLOVER, [L.LQ_OP_SIGN, L.LQ_OP_NORMAL_EVEN, 9]),
    (L.LQ_OVERLAP, [L.LQ_OP_SITE, L.LQ_OP_SCHUR, L.LQ_OP_NORMAL_EVEN, 9]),
    (L.LQ_HISQ, [L.LQ_OP_SITE, L.LQ_OP_SITE_INV, L.LQ_OP_SCHUR, L.LQ_OP_HW, L.LQ_OP_SIGN, 9]),
])
def test_refused_operator_in_a_capture(kind, ops):
    torch.zeros(1, device="cuda")
    ctx = L.lq_init(0)
    U = torch.eye(3, dtype=torch.complex128, device="cuda").expand(V, 4, 3, 3).contiguous()
    f = L.lq_hisq_load(ctx, LX, U, U) if kind == L.LQ_HISQ else L.lq_gauge_load(ctx, LX, U)
    act = L.action(kind, m=0.1, rho=1.5, cheb_N=4) if kind == L.LQ_OVERLAP else L.action(kind, m=0.1)
    b = torch.ones((1, V, 3) if kind == L.LQ_HISQ else (1, V, 4, 3), dtype=torch.complex128, device="cuda")
    out = torch.empty_like(b)
    x = torch.zeros(4, device="cuda")
    torch.cuda.synchronize()
    stream_arg = lambda: C.c_void_p(torch.cuda.current_stream().cuda_stream)  # noqa: E731
    codes = []
    gc.collect()
    gc.disable()  # a graph of another test may be garbage; its destructor must not run inside the capture
    try:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            x += 1
            for op in ops:
                for prec in (64, 32, 16):
                    codes.append(L.load().lq_apply_dev(ctx, C.byref(act), f, op, prec, 1, L._ptr(b), L._ptr(out),
                                                       stream_arg()))
            x += 1
        for n in range(1, 4):
            g.replay()
            torch.cuda.synchronize()
            assert x.tolist() == [2.0 * n] * 4
    finally:
        gc.enable()
        L.lq_field_free(f)
        L.lq_finalize(ctx)
    assert set(codes) == {L.LQ_EINVAL}
