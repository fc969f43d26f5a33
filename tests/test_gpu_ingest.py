"""The work queue around the sizes its ingest works in (64 and 256 ready
entries): readiness from the host one by one and as a list, from the device,
and from both with the same partitions signalled twice.  Every tile is
reduced exactly once, and the output is the rank-order sum bit for bit."""
import numpy as np
import pytest
import torch

from _gpu import DEV, new_request, say
from paper_2604_22228_amd import pcoll as pc
from paper_2604_22228_amd import synth
from paper_2604_22228_amd.streams import independent_streams

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("buckets", [1, 3])
@pytest.mark.parametrize("nparts", [1, 63, 65, 256, 257, 700])
def test_every_tile_once(nparts, buckets):
    P = 3
    counts = [nparts * 256 + 37 * (b + 1) for b in range(buckets)]
    xs = [synth.normal_f32(P, c, 50 + b, device=DEV)
          for b, c in enumerate(counts)]
    outs = [torch.empty(c, device=DEV) for c in counts]
    want = [(x[0] + x[1]) + x[2] for x in xs]
    stream = torch.cuda.Stream(DEV)
    side = independent_streams(stream, 1)[0]
    torch.cuda.synchronize()
    req = new_request(counts, pc.FLOAT32, pc.SUM, nparts, P, debug=1,
                      tile_elems=1024, publish_batch=3)
    req.bind(xs, outs, stream=stream)
    n = req.nparts_total
    for epoch, mode in enumerate(["each", "list", "device", "both", "each"]):
        say(f"case parts={nparts} buckets={buckets} {mode}")
        order = synth.permutation(n, epoch).astype(np.int32)
        dev = torch.from_numpy(order).to(DEV)
        for o in outs:
            o.fill_(float("nan"))
        torch.cuda.synchronize()
        req.start()
        if mode == "each":
            for p in order:
                req.pready(int(p))
        elif mode == "list":
            req.pready_list(order)
        else:
            # the device signals all; the host some of them, before and after
            k = n // 3
            if mode == "both":
                req.pready_list(order[:k])
            req.pready_on_stream(dev, n, side)
            if mode == "both":
                for p in order[k:2 * k]:
                    req.pready(int(p))
        req.wait()
        torch.cuda.synchronize()
        hits, tiles = req.tile_hits()
        assert all(h == t and t >= 1 for h, t in zip(hits, tiles))
        for o, w in zip(outs, want):
            assert torch.equal(o.view(torch.int32), w.view(torch.int32))
    req.free()
