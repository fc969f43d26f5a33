"""The direct kernel behind pcoll_reduce_noalloc: sizes at the edges of its
rows, tiles and tile-size rule, a message beyond 2^31 elements, two calls
that overlap on two streams, and replays of a captured call."""
import numpy as np
import pytest
import torch

from _gpu import DEV, new_request, say
from paper_2604_22228_amd import pcoll as pc
from paper_2604_22228_amd import synth

pytestmark = pytest.mark.gpu
ROW = {pc.FLOAT32: 256, pc.BFLOAT16: 512, pc.FP8_E4M3: 1024}


def _inputs(dtype, P, n, seed):
    if dtype == pc.FLOAT32:
        return synth.normal_f32(P, n, seed, device=DEV), None
    if dtype == pc.BFLOAT16:
        return synth.bf16_codes(P, n, seed, device=DEV), None
    gen = np.random.default_rng(seed)
    q = [torch.from_numpy(gen.integers(0, 0x7F, n).astype(np.uint8)).to(DEV)
         for _ in range(P)]
    s = [torch.from_numpy(gen.uniform(0.5, 2, (n + 255) // 256)
                          .astype(np.float32)).to(DEV) for _ in range(P)]
    return q, s


@pytest.mark.parametrize("rows", [0, 1, 4, 5, 4095, 4096, 4097])
@pytest.mark.parametrize("dtype", [pc.FLOAT32, pc.BFLOAT16, pc.FP8_E4M3])
def test_direct_edges(dtype, rows):
    P, stream = 5, torch.cuda.current_stream(DEV)
    for n in {max(1, rows * ROW[dtype] + k) for k in (-1, 0, 1, 131)}:
        say(f"case direct dtype={dtype} n={n}")
        bufs, scales = _inputs(dtype, P, n, rows + 7)
        outs = []
        for direct in (False, True):
            y = torch.full_like(bufs[0], 3)
            s = None if scales is None else torch.zeros_like(scales[0])
            if direct:
                pc.pcoll_reduce_noalloc(n, dtype, pc.SUM, 3, bufs, y, scales,
                                        s, stream)
            else:
                req = new_request([n], dtype, pc.SUM, 3, P)
                req.bind([bufs], [y], scales and [scales], s is not None and
                         [s] or None, stream=stream)
                req.start()
                req.pready_range(0, 2)
                req.wait()
                req.free()
            torch.cuda.synchronize()
            outs.append((y, s))
        assert torch.equal(outs[0][0].view(torch.uint8),
                           outs[1][0].view(torch.uint8))
        if scales is not None:
            assert torch.equal(outs[0][1], outs[1][1])


@pytest.mark.parametrize("dtype,P", [(pc.FLOAT32, 4), (pc.FLOAT32, 8),
                                     (pc.FLOAT32, 3), (pc.BFLOAT16, 16)])
@pytest.mark.parametrize("past", [-1, 0, 131])
def test_direct_large_shape(dtype, P, past):
    # 128 MiB of inputs, where the launch shape changes
    stream = torch.cuda.current_stream(DEV)
    n = (1 << 27) // (P * (2 if dtype == pc.BFLOAT16 else 4)) + past
    say(f"case direct large dtype={dtype} P={P} n={n}")
    bufs, _ = _inputs(dtype, P, n, P)
    outs = [torch.full_like(bufs[0], 3) for _ in range(2)]
    pc.pcoll_reduce_noalloc(n, dtype, pc.SUM, 5, bufs, outs[0], None, None,
                            stream)
    req = new_request([n], dtype, pc.SUM, 5, P)
    req.bind([bufs], [outs[1]], stream=stream)
    req.start()
    req.pready_range(0, 4)
    req.wait()
    req.free()
    torch.cuda.synchronize()
    assert torch.equal(outs[0].view(torch.uint8), outs[1].view(torch.uint8))


def test_direct_beyond_2_31_elements():
    n = (1 << 31) + 4096 * 3 + 5
    say(f"case direct n={n}")
    x = torch.randint(-30000, 30000, (n,), dtype=torch.int16, device=DEV)
    x &= 0x3FFF  # finite, positive bf16: max over one rank is the identity
    y = torch.zeros_like(x)
    pc.pcoll_reduce_noalloc(n, pc.BFLOAT16, pc.MAX, 3, [x], y, None, None,
                            torch.cuda.current_stream(DEV))
    torch.cuda.synchronize()
    assert torch.equal(x, y)


def test_direct_beyond_2_32_threads():
    # 2^24 tiles of the usual 2048 elements would be a grid of 2^32 threads
    n, step = (1 << 35) + 4096 * 3 + 5, 1 << 27
    if torch.cuda.mem_get_info(DEV)[0] < 4 * n + (8 << 30):
        pytest.skip("needs 136 GiB of device memory")
    say(f"case direct n={n}")
    base = torch.randint(0, 0x4000, (step,), dtype=torch.int16, device=DEV)
    x = torch.empty(n, dtype=torch.int16, device=DEV)
    y = torch.zeros_like(x)
    for k, at in enumerate(range(0, n, step)):
        torch.bitwise_xor(base[:min(step, n - at)], k, out=x[at:at + step])
    pc.pcoll_reduce_noalloc(n, pc.BFLOAT16, pc.MAX, 33, [x], y, None, None,
                            torch.cuda.current_stream(DEV))
    torch.cuda.synchronize()
    for at in range(0, n, step):
        assert torch.equal(x[at:at + step], y[at:at + step]), at
    del x, y
    torch.cuda.empty_cache()


def test_direct_calls_overlap_and_replay():
    P, n = 4, 3_000_001
    streams = [torch.cuda.Stream(DEV) for _ in range(2)]
    xs = [synth.normal_f32(P, n, 70 + i, device=DEV) for i in range(2)]
    want = [((x[0] + x[1]) + x[2]) + x[3] for x in xs]
    ys = [torch.empty(n, device=DEV) for _ in range(2)]

    def call(i, stream):
        pc.pcoll_reduce_noalloc(n, pc.FLOAT32, pc.SUM, 9, xs[i], ys[i], None,
                                None, stream)

    torch.cuda.synchronize()
    for _ in range(20):
        for i in range(2):
            call(i, streams[i])
    torch.cuda.synchronize()
    for y, w in zip(ys, want):
        assert torch.equal(y.view(torch.int32), w.view(torch.int32))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=streams[0]):
        call(0, streams[0])
    for k in range(4):
        ys[0].fill_(float("nan"))
        xs[0][0].add_(1.0)  # new values in the same buffers
        w = ((xs[0][0] + xs[0][1]) + xs[0][2]) + xs[0][3]
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(ys[0].view(torch.int32), w.view(torch.int32)), k
