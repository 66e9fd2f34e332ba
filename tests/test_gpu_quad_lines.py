"""Quadratic bases in 4-D and 5-D take four lanes per target up to 4,096 targets
(FP64) or 32,768: the same targets give the same bits on both sides."""
import pytest
import torch

from gpu_helpers import dev, say
from paper_2510_18838_amd import pcms, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,precision,line", [(4, pcms.FP64, 4096), (5, pcms.FP64, 4096),
                                                (4, pcms.MIXED, 32768), (5, pcms.MIXED_REFINE, 32768)])
@pytest.mark.parametrize("mode", [synth.KNN, synth.GROW])
def test_same_bits(dim, precision, line, mode):
    n = 20000
    r = (60.0 / (n * synth.unit_ball_volume(dim))) ** (1.0 / dim)
    p = synth.uniform_problem(90 + dim, n, line + 1, dim, 2, mode, n_fields=2, radius=r, k=60,
                              n_min=40, k_cap=96)
    src, vals, tgt = dev(p.src), dev(p.vals), dev(p.tgt)
    rad, o = pcms.radius_of(p), pcms.opts(precision=precision)
    say(f"{dim}-D precision {precision} mode {mode}")
    many, mst, _ = pcms.pcms_mls_transfer(src, vals, tgt, 2, rad, p.k_cap, o=o)
    for m in (line, 300):
        few, st, _ = pcms.pcms_mls_transfer(src, vals, tgt[:m].contiguous(), 2, rad, p.k_cap, o=o)
        assert torch.equal(st, mst[:m])
        assert torch.equal(few.nan_to_num(7.0), many[:, :m].nan_to_num(7.0))
