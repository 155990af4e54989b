"""Working memory of calls on many streams: a stream of its own for every call
takes no more memory than one stream, also for calls that are refused on the
way, and the results do not change."""
import ctypes as C
import threading

import pytest
import torch

from paper_2201_09004_amd import lq as L

pytestmark = pytest.mark.gpu
LX, N = (8, 8, 16, 16), 12  # an FP64 column set of 38 MiB
SLACK = 8 << 20


@pytest.fixture(scope="module")
def problem():
    g = torch.Generator(device="cuda").manual_seed(5)
    V = LX[0] * LX[1] * LX[2] * LX[3]
    U = torch.linalg.qr(torch.randn(4 * V, 3, 3, dtype=torch.complex128, generator=torch.Generator().manual_seed(4)))[0]
    ctx = L.lq_init(0)
    f = L.lq_gauge_load(ctx, LX, U.reshape(V, 4, 3, 3).contiguous().cuda())
    v = torch.randn(N, V, 4, 3, dtype=torch.complex128, device="cuda", generator=g)
    yield ctx, f, v
    L.lq_field_free(f)
    L.lq_finalize(ctx)


def free_bytes():
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def streams(n):
    """Streams that have run something (a queue's own memory is there)."""
    s = [torch.cuda.Stream() for _ in range(n)]
    for t in s:
        with torch.cuda.stream(t):
            torch.zeros(8, device="cuda")
    return s


def test_a_stream_for_every_call(problem):
    ctx, f, v = problem
    act = L.action(L.LQ_WILSON, m=0.2)
    want = L.lq_apply(ctx, act, f, L.LQ_OP_D, 64, v)
    out = torch.empty_like(v)
    own = streams(12)
    before = free_bytes()
    for s in own:
        with torch.cuda.stream(s):
            L.lq_apply(ctx, act, f, L.LQ_OP_D, 64, v, out)
    # 12 calls' own blocks would be 900 MiB
    assert before - free_bytes() <= SLACK
    assert torch.equal(out, want)


def test_refused_calls_keep_nothing_apart(problem):
    ctx, f, v = problem
    tm = L.action(L.LQ_TM_CLOVER, m=0.1, mu=0.1, c_sw=1.0)
    out = torch.empty_like(v)

    def refused(s):
        with torch.cuda.stream(s):
            with pytest.raises(L.LqError):
                L.lq_apply(ctx, tm, f, L.LQ_OP_D, 16, v, out)  # no FP16 site matrices

    own = streams(12)
    refused(own[0])
    before = free_bytes()
    for s in own:
        refused(s)
    assert before - free_bytes() <= SLACK


def test_host_and_device_calls_share_blocks(problem):
    ctx, f, v = problem
    act = L.action(L.LQ_WILSON, m=0.2)
    want = L.lq_apply(ctx, act, f, L.LQ_OP_D, 64, v)
    h = v.cpu().numpy()
    got = L.lq_apply(ctx, act, f, L.LQ_OP_D, 64, h)
    assert torch.equal(torch.from_numpy(got), want.cpu())
    before = free_bytes()
    for _ in range(3):
        L.lq_apply(ctx, act, f, L.LQ_OP_D, 64, v, want)
        L.lq_apply(ctx, act, f, L.LQ_OP_D, 64, h)
    assert before - free_bytes() <= SLACK


def test_per_thread_stream(problem):
    """hipStreamPerThread (handle 2): its blocks are those of every other stream, and each thread's calls are its own."""
    ctx, f, v = problem
    act = L.action(L.LQ_WILSON, m=0.2)
    want = [L.lq_apply(ctx, act, f, L.LQ_OP_D, p, v) for p in (64, 32)]
    outs = [torch.empty_like(v) for _ in range(4)]

    def apply_on(stream, prec, out):
        r = L.load().lq_apply_dev(ctx, C.byref(act), f, L.LQ_OP_D, prec, N, L._ptr(v), L._ptr(out), C.c_void_p(stream))
        assert r == L.LQ_OK, L.last_error()

    apply_on(2, 64, outs[0])
    before = free_bytes()
    apply_on(0, 64, outs[0])
    apply_on(2, 64, outs[0])
    assert before - free_bytes() <= SLACK and torch.equal(outs[0], want[0])
    errors = []

    def thread(k):
        try:
            for i in range(6):
                apply_on(2, (64, 32)[(i + k) % 2], outs[k])
                assert torch.equal(outs[k], want[(i + k) % 2])
        except Exception as e:  # reported by the main thread
            errors.append(e)

    ts = [threading.Thread(target=thread, args=(k,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors
