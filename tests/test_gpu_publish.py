"""Published tiles are counted once per partition and group: partitions of one
tile, of a few and of more than a batch, batches that end inside a partition,
and all of them complete while another partition is still awaited."""
import time

import pytest
import torch

from _gpu import DEV, new_request, say
from paper_2604_22228_amd import pcoll as pc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("groups", [1, 3])
@pytest.mark.parametrize("batch", [1, 3, 64])
@pytest.mark.parametrize("tiles", [1, 2, 5, 64, 131])
def test_partitions_arrive_while_one_is_awaited(tiles, batch, groups):
    P, nparts, tile = 2, 4, 1024
    n = nparts * tiles * tile - 7
    say(f"case publish tiles={tiles} batch={batch} groups={groups}")
    bufs = [torch.randint(-1000, 1000, (n,), dtype=torch.int32, device=DEV)
            for _ in range(P)]
    out = torch.zeros_like(bufs[0])
    want = bufs[0] + bufs[1]
    req = new_request([n], pc.INT32, pc.SUM, nparts, P)
    req.bind([bufs], [out], stream=torch.cuda.Stream(DEV))
    req.set_config(tile_elems=tile, min_tile_elems=tile, groups=groups,
                   publish_batch=batch, guide=0, debug=1)
    torch.cuda.synchronize()
    for last in (0, nparts - 1):
        out.zero_()
        torch.cuda.synchronize()
        early = [p for p in range(nparts) if p != last]
        req.start()
        req.pready_list(early)
        t0 = time.perf_counter()
        while (not all(req.parrived(p) for p in early)
               and time.perf_counter() - t0 < 3):
            pass
        arrived = [req.parrived(p) for p in range(nparts)]
        req.pready(last)
        req.wait()
        assert arrived == [p != last for p in range(nparts)]
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        hits, per_part = req.tile_hits()
        assert per_part == [tiles] * nparts
        assert hits == per_part
    req.free()
