"""An operator is not built inside a stream capture: its arrays outlive the
graph, so the build refuses before it enqueues anything."""
import pytest
import torch

from gpu_helpers import dev, say
from paper_2510_18838_amd import pcms, synth

pytestmark = pytest.mark.gpu


def test_build_is_refused_in_a_capture():
    p = synth.uniform_problem(3, 500, 400, 2, 1, synth.FIXED, n_fields=1, radius=0.2, k_cap=32)
    src, tgt, vals = dev(p.src), dev(p.tgt), dev(p.vals)
    rad = pcms.radius_of(p)
    summary = torch.zeros(4, dtype=torch.int32, device=src.device)
    o = pcms.opts(flags=pcms.ASYNC, summary=summary)
    before = pcms.Operator(src, tgt, p.degree, rad, p.k_cap)   # its block is pooled
    want = before.apply(vals).clone()
    before.free()
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    marker = torch.zeros(1, device=src.device)
    torch.cuda.synchronize()
    say("build in a capture")
    with torch.cuda.graph(g, stream=s):
        with pytest.raises(pcms.PcmsError):
            pcms.Operator(src, tgt, p.degree, rad, p.k_cap, o=o)
        marker += 1
    g.replay()
    torch.cuda.synchronize()
    assert marker.item() == 1
    op = pcms.Operator(src, tgt, p.degree, rad, p.k_cap)
    assert torch.equal(op.apply(vals), want)
    op.free()
