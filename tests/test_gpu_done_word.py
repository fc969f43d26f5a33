"""The epoch's end at every way its workgroups are counted: one alone, up to
16 (one level), more (two).  Several epochs each, so that a count left over
from one would end the next too early: every tile once, results bitwise."""
import pytest
import torch

from _gpu import DEV, as_u32, new_request, say
from paper_2604_22228_amd import pcoll as pc
from paper_2604_22228_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("groups", [1, 2, 15, 16, 17, 31, 32, 33, 256])
def test_done_word_group_counts(groups, graph):
    say(f"case groups={groups} graph={graph}")
    P, n, parts = 3, 1024 * 512 + 77, 16
    stream = torch.cuda.current_stream(DEV)
    xs = synth.normal_f32(P, n, groups, device=DEV)
    y = torch.empty(n, device=DEV)
    req = new_request([n], pc.FLOAT32, pc.SUM, parts, P, tile_elems=1024,
                      groups=groups, debug=1, graph=graph)
    req.bind([xs], [y], stream=stream)
    for k in range(5):
        y.fill_(float("nan"))
        xs[k % P].add_(1.0)
        want = (xs[0] + xs[1]) + xs[2]
        torch.cuda.synchronize()
        req.start()
        req.pready_range(0, parts // 2)
        req.pready_range(parts // 2 + 1, parts - 1)
        req.wait()
        got = y.clone()  # on the request's stream
        hits, tiles = req.tile_hits()
        torch.cuda.synchronize()
        assert req.stats().groups == groups
        assert list(hits) == list(tiles)
        assert (as_u32(got.cpu().numpy()) == as_u32(want.cpu().numpy())).all()
    req.free()
