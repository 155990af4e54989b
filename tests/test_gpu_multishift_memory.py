"""HISQ with two masses where memory is short: the multi-shift stage takes the
residuals of its deferred updates only after what it cannot do without, so that
it does not fail where one residual fits, and the context works on afterwards."""
import pytest
import torch

from paper_2201_09004_amd import lq as L

pytestmark = pytest.mark.gpu
LX, N, MASSES = (16, 16, 16, 32), 24, [0.1, 0.3]
UNIT = N * (LX[0] * LX[1] * LX[2] * LX[3] // 2) * 24  # one FP32 column set of the even sites, 36 MiB


def test_room_for_one_residual():
    V = LX[0] * LX[1] * LX[2] * LX[3]
    g = torch.Generator().manual_seed(3)
    few = torch.linalg.qr(torch.randn(4096, 3, 3, dtype=torch.complex128, generator=g))[0].contiguous()
    links = [few[torch.randint(4096, (V * 4,), generator=g)].reshape(V, 4, 3, 3).cuda() for _ in range(2)]
    b = torch.randn(N, V, 3, dtype=torch.complex128, generator=g).cuda()
    x = torch.zeros((2,) + tuple(b.shape), dtype=b.dtype, device="cuda")
    act = L.action(L.LQ_HISQ, m=MASSES[0])
    prm = L.params(tol=1e-9, sloppy_bits=32, masses=MASSES)
    ctx = L.lq_init(0)
    f = L.lq_hisq_load(ctx, LX, *links)
    try:
        L.lq_solve(ctx, act, f, prm, b[:1].contiguous())  # the links at both precisions, the first shapes
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        with pytest.raises(L.LqError) as e:  # more than there is: every block that waits goes back to the device
            L.lq_copy_bandwidth(ctx, 2 * torch.cuda.mem_get_info()[1])
        assert e.value.code == L.LQ_ENOMEM
        # right-hand sides, their copies and solutions in FP64 take 10 units, the
        # multi-shift stage 7 with one residual and 16 with nine; the refinement
        # takes 22 of its own
        left = 10 * UNIT + 10 * UNIT
        fill = []
        for _ in range(8):  # the device reports some of its free memory late
            more = torch.cuda.mem_get_info()[0] - left
            if more < (16 << 20):
                break
            try:
                fill.append(torch.empty(more, dtype=torch.uint8, device="cuda"))
            except torch.OutOfMemoryError:
                break
        try:
            _, st = L.lq_solve(ctx, act, f, prm, b, x)  # where the device had more than it said
            assert st["status"] == 0 and st["true_rel_res"] <= 1e-9
        except L.LqError as e:
            assert e.code == L.LQ_ENOMEM and "multi-shift" not in str(e)
        del fill
        torch.cuda.empty_cache()
        x.zero_()
        _, st = L.lq_solve(ctx, act, f, prm, b, x)
        assert st["status"] == 0 and st["true_rel_res"] <= 1e-9
    finally:
        L.lq_field_free(f)
        L.lq_finalize(ctx)
