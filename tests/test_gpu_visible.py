"""A partition that has arrived can be read at once by kernels on other
streams while the request's kernel still runs (it waits for the partitions
not yet readied): the results are in memory, not in some cache, whole rows,
ragged ends and block scales alike."""
import time

import numpy as np
import pytest
import torch

from _gpu import DEV, new_request, say
from paper_2604_22228_amd import pcoll as pc
from paper_2604_22228_amd import synth
from paper_2604_22228_amd.streams import independent_streams

pytestmark = pytest.mark.gpu


def _inputs(dtype, P, n):
    if dtype == pc.FLOAT32:
        return synth.normal_f32(P, n, 5, device=DEV), None, None
    if dtype == pc.BFLOAT16:
        return synth.bf16_codes(P, n, 5, device=DEV), None, None
    rng = np.random.default_rng(5)
    q = [torch.from_numpy(rng.integers(0, 0x7F, n).astype(np.uint8)).to(DEV)
         for _ in range(P)]
    if dtype == pc.MXFP8_E4M3:
        s = [torch.from_numpy(rng.integers(120, 130, (n + 31) // 32)
                              .astype(np.uint8)).to(DEV) for _ in range(P)]
    else:
        s = [torch.from_numpy(rng.uniform(.5, 2, (n + 255) // 256)
                              .astype(np.float32)).to(DEV) for _ in range(P)]
    return q, s, torch.zeros_like(s[0])


@pytest.mark.parametrize("dtype", [pc.FLOAT32, pc.BFLOAT16, pc.FP8_E4M3,
                                   pc.MXFP8_E4M3])
def test_arrived_partition_is_visible_to_other_kernels(dtype):
    P, n, nparts = 4, 3_000_000 // 32 * 32 + (3 if dtype in (
        pc.FLOAT32, pc.BFLOAT16) else 0), 3
    say(f"case visible dtype={dtype} n={n}")
    bufs, scales, osc = _inputs(dtype, P, n)
    out = torch.zeros_like(bufs[0])
    stream = torch.cuda.Stream(DEV)
    side = independent_streams(stream, 1)[0]
    want, wsc = torch.zeros_like(out), None if osc is None else \
        torch.zeros_like(osc)
    pc.pcoll_reduce_noalloc(n, dtype, pc.SUM, nparts, bufs, want, scales, wsc,
                            torch.cuda.current_stream(DEV))
    torch.cuda.synchronize()
    req = new_request([n], dtype, pc.SUM, nparts, P)
    req.bind([bufs], [out], scales and [scales], osc is not None and [osc] or
             None, stream=stream)
    for part in (2, 0, 1, 2):  # the ragged end first and last
        out.fill_(1)
        if osc is not None:
            osc.fill_(1)
        # caches of every die hold the old contents
        stale = out.view(torch.uint8).sum(dtype=torch.int64)
        torch.cuda.synchronize()
        _, off, ln = req.part_info(part)
        req.start()
        req.pready(part)
        t0 = time.perf_counter()
        while not req.parrived(part) and time.perf_counter() - t0 < 3:
            pass
        with torch.cuda.stream(side):
            got = out[off:off + ln].clone()
            gsc = None
            if osc is not None:
                blk = 32 if dtype == pc.MXFP8_E4M3 else 256
                cut = slice(off // blk, (off + ln + blk - 1) // blk)
                gsc = osc[cut].clone()
        side.synchronize()
        assert not req.test()  # the kernel still waits for the others
        for p in range(nparts):
            if p != part:
                req.pready(p)
        req.wait()
        torch.cuda.synchronize()
        assert stale is not None
        assert torch.equal(got.view(torch.uint8),
                           want[off:off + ln].view(torch.uint8)), part
        if gsc is not None:
            assert torch.equal(gsc.view(torch.uint8),
                               wsc[cut].view(torch.uint8)), part
        assert torch.equal(out.view(torch.uint8), want.view(torch.uint8))
    req.free()
