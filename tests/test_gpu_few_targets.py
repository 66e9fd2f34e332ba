"""Calls of few targets (four lanes per target) against calls of many (one):
the same targets give the same bits on both sides of the line, which lies at
49,152 targets."""
import numpy as np
import pytest
import torch

from gpu_helpers import DEV, dev, say
from paper_2510_18838_amd import pcms, synth

pytestmark = pytest.mark.gpu

LINE = 49152


def _same(a, b):
    return torch.equal(a.nan_to_num(7.0), b.nan_to_num(7.0))


@pytest.mark.parametrize("dim,degree,nf,mode", [(2, 2, 1, synth.FIXED), (3, 1, 3, synth.GROW),
                                                (3, 2, 9, synth.KNN), (5, 1, 4, synth.GROW)])
def test_same_bits_on_both_sides_of_the_line(dim, degree, nf, mode):
    n = 30000
    r = (30.0 / (n * synth.unit_ball_volume(dim))) ** (1.0 / dim)
    p = synth.uniform_problem(81, n, LINE + 1, dim, degree, mode, n_fields=nf, radius=r, k=30,
                              n_min=12, k_cap=48)
    src, vals, tgt = dev(p.src), dev(p.vals), dev(p.tgt)
    rad = pcms.radius_of(p)
    for prec in (pcms.FP64, pcms.MIXED_REFINE):
        o = pcms.opts(precision=prec)
        say(f"{dim}-D degree {degree} mode {mode} precision {prec}")
        out, st, _ = pcms.pcms_mls_transfer(src, vals, tgt, degree, rad, p.k_cap, o=o)
        for m in (LINE, 1000, 63, 1):
            few, fst, _ = pcms.pcms_mls_transfer(src, vals, tgt[:m].contiguous(), degree, rad,
                                                 p.k_cap, o=o)
            assert torch.equal(fst, st[:m]) and _same(few, out[:, :m]), (prec, m)
        op = pcms.Operator(src, tgt[:1000].contiguous(), degree, rad, p.k_cap, o=o)
        if prec == pcms.FP64:
            assert _same(op.apply(vals), out[:, :1000])
        op.free()
    g = pcms.pcms_grid_build(src, cell_width=r)
    many = pcms.pcms_neighbors(g, tgt, rad, p.k_cap)
    few = pcms.pcms_neighbors(g, tgt[:1000].contiguous(), rad, p.k_cap)
    torch.cuda.synchronize()
    for key in ("n_kept", "n_found", "r2", "status"):
        assert torch.equal(many[key][:1000], few[key]), key
    kept = torch.arange(p.k_cap, device=DEV) < few["n_kept"][:, None]
    assert torch.equal(many["nbr"][:1000][kept], few["nbr"][kept])
    assert np.isfinite(few["r2"].cpu().numpy()).all()
    g.free()
