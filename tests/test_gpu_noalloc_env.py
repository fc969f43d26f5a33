"""The environment's launch shape on the allocation-free epoch: whatever tile,
workgroup count, layout and wavefronts it asks for, sensible or not, the same
bits as with none."""
import pytest
import torch

from _gpu import DEV, say
from paper_2604_22228_amd import pcoll as pc
from paper_2604_22228_amd import synth

pytestmark = pytest.mark.gpu
SHAPES = [{"TILE": "1024"}, {"TILE": "65536", "GROUP_WAVES": "8"},
          {"GROUPS": "1"}, {"GROUPS": "300", "INTERLEAVE": "1"},
          {"GROUPS_PER_CU": "1"}, {"GROUP_WAVES": "1", "INTERLEAVE": "0"},
          {"GROUP_WAVES": "3", "TILE": "3000", "INTERLEAVE": "5"},
          {"GROUP_WAVES": "99", "TILE": "-4", "INTERLEAVE": "-2",
           "GROUPS": "x"}]


@pytest.mark.parametrize("dtype,P", [(pc.FLOAT32, 8), (pc.BFLOAT16, 3),
                                     (pc.FP8_E4M3, 4)])
@pytest.mark.parametrize("n", [5, 256 * 1024 + 131, (1 << 22) + 4097])
def test_environment_shapes(monkeypatch, dtype, P, n):
    stream = torch.cuda.current_stream(DEV)
    scales = None
    if dtype == pc.FLOAT32:
        xs = synth.normal_f32(P, n, 5, device=DEV)
    elif dtype == pc.BFLOAT16:
        xs = synth.bf16_codes(P, n, 5, device=DEV)
    else:
        gen = torch.Generator(DEV).manual_seed(5)
        xs = [torch.randint(0, 0x7E, (n,), generator=gen, device=DEV,
                            dtype=torch.uint8) for _ in range(P)]
        scales = [torch.rand((n + 255) // 256, generator=gen, device=DEV) + .5
                  for _ in range(P)]

    def run():
        y = torch.full_like(xs[0], 3)
        s = None if scales is None else torch.zeros_like(scales[0])
        pc.pcoll_reduce_noalloc(n, dtype, pc.SUM, 3, xs, y, scales, s, stream)
        torch.cuda.synchronize()
        return y.view(torch.uint8), s

    want = run()
    for env in SHAPES:
        say(f"case noalloc env dtype={dtype} n={n} {env}")
        with monkeypatch.context() as m:
            for k, v in env.items():
                m.setenv("PCOLL_" + k, v)
            got = run()
        assert torch.equal(got[0], want[0]), env
        assert scales is None or torch.equal(got[1], want[1]), env
