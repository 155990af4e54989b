"""Launch shapes kept per lattice: two lattices of one volume, of which only the
first is divided by the kept traversal order, and shapes in a cache file that
the lattice or the kernel does not have, give what an untuned launch gives."""
import numpy as np
import pytest
import torch

import synth
from paper_2201_09004_amd import lq as L

pytestmark = pytest.mark.gpu
LATS = [(8, 8, 12, 8), (16, 8, 6, 8)]  # z slabs of 4 planes divide the first alone


def apply_one(ctx, kind, Lx, prec, op):
    if kind == L.LQ_HISQ:
        f = L.lq_hisq_load(ctx, Lx, *synth.hisq_fields(Lx, 51))
        v = synth.gaussian_colour(Lx, 3, 52)
    else:
        f = L.lq_gauge_load(ctx, Lx, synth.su3_field(Lx, 0.3, 53))
        v = synth.gaussian_spinor(Lx, 3, 54)
    try:
        return L.lq_apply(ctx, L.action(kind, m=0.1), f, op, prec, v)
    finally:
        L.lq_field_free(f)


def run(kind, prec, op):
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ctx = L.lq_init(0)
    try:
        return [apply_one(ctx, kind, Lx, prec, op) for Lx in LATS]
    finally:
        L.lq_finalize(ctx)


@pytest.mark.parametrize("kind", [L.LQ_WILSON, L.LQ_HISQ])
@pytest.mark.parametrize("prec", [64, 16])
@pytest.mark.parametrize("shape", ["3 4 0 1", "5 0 0 1", "1 0 7 1", "-8 0 0 1"])
def test_kept_shape_of_another_lattice(tmp_path, monkeypatch, kind, prec, shape):
    monkeypatch.setenv("LQ_TUNE", "0")
    want = run(kind, prec, L.LQ_OP_D)
    monkeypatch.delenv("LQ_TUNE")
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("LQ_TUNE_CACHE", str(path))
    run(kind, prec, L.LQ_OP_D)
    keys = [line.split()[0] for line in path.read_text().splitlines()]
    assert len(keys) == len(set(keys)) == 2
    path.write_text("".join(f"{k} {shape}\n" for k in keys))
    for got in (run(kind, prec, L.LQ_OP_D), run(kind, prec, L.LQ_OP_D)):
        for a, b in zip(got, want):
            assert np.array_equal(a, b)
