"""Working memory kept between calls: threads on streams of their own, calls
of many sizes in turn, and a context finalized while another works, give
bitwise what one thread alone gets (every kernel's result is independent of
timing)."""
import threading

import pytest
import torch

from paper_2201_09004_amd import lq as L

pytestmark = pytest.mark.gpu


def _unitary(n, seed):
    g = torch.Generator().manual_seed(seed)
    z = torch.randn(n, 3, 3, dtype=torch.complex128, generator=g)
    return torch.linalg.qr(z)[0].contiguous()


def test_streams_and_threads_share_no_block():
    shapes = [((4, 4, 4, 8), 1), ((8, 8, 4, 6), 3), ((4, 4, 4, 8), 5), ((8, 8, 8, 8), 2)]
    ctx = L.lq_init(0)
    fields, inputs, want = {}, [], []
    act = L.action(L.LQ_WILSON, m=0.2)
    for k, (Lx, n) in enumerate(shapes):
        V = Lx[0] * Lx[1] * Lx[2] * Lx[3]
        if Lx not in fields:
            fields[Lx] = L.lq_gauge_load(ctx, Lx, _unitary(4 * V, k).reshape(V, 4, 3, 3).cuda())
        g = torch.Generator(device="cuda").manual_seed(k)
        inputs.append(torch.randn(n, V, 4, 3, dtype=torch.complex128, device="cuda", generator=g))
    prm = L.params(tol=1e-8, sloppy_bits=32)

    def work():
        out = [L.lq_apply(ctx, act, fields[Lx], L.LQ_OP_D, 32, v) for (Lx, _), v in zip(shapes, inputs)]
        return out + [L.lq_solve(ctx, act, fields[shapes[0][0]], prm, inputs[0])[0]]

    try:
        want = work()
        torch.cuda.synchronize()
        got, errors = {}, []

        def thread(i):
            try:
                with torch.cuda.stream(torch.cuda.Stream()):
                    other = L.lq_init(0)  # a second context comes and goes
                    got[i] = [work() for _ in range(4)]
                    L.lq_finalize(other)
                    torch.cuda.current_stream().synchronize()
            except Exception as e:  # reported by the main thread
                errors.append(e)

        ts = [threading.Thread(target=thread, args=(i,)) for i in range(3)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        assert not errors, errors
        for runs in got.values():
            for run in runs:
                for a, b in zip(run, want):
                    assert torch.equal(a, b)
    finally:
        for f in fields.values():
            L.lq_field_free(f)
        L.lq_finalize(ctx)
