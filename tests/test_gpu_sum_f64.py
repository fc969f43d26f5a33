"""The compensated sums of the 8-bit payloads where the kernels' binary64
route has to decide how Sum2 rounds: terms that cancel, terms missing or
below the exactness bound, equal power-of-two scales (ties), scales far
apart, at binary32's lower and upper end.  Codes and scales bitwise against
the oracle's binary32 Sum2."""
import numpy as np
import pytest
import torch

from _gpu import DEV, as_u32, new_request, run_epoch, say
from oracle import get as get_oracle
from paper_2604_22228_amd import pcoll as pc

pytestmark = pytest.mark.gpu
N = 256 * 96 + 32  # a partial row at the end
KMAX = {"e4m3": 448.0, "e5m2": 57344.0}


@pytest.fixture(scope="module")
def orc():
    return get_oracle()


def _codes(rng, dtype, ranks, mode):
    """Finite codes; per mode dense, gradient-like, with zeros, cancelling
    pairs of ranks."""
    inf = 0x7C if dtype == "e5m2" else 0x7F
    finite = np.array([c for c in range(256) if (c & 0x7F) < inf], np.uint8)
    q = rng.choice(finite, size=(ranks, N))
    if mode == "gradients":
        x = rng.standard_normal((ranks, N)).astype(np.float32)
        top = 448.0 if dtype != "e5m2" else 57344.0
        t = torch.from_numpy(x * np.float32(top / 60)).clamp(-top, top)
        q = t.to(torch.float8_e5m2 if dtype == "e5m2"
                 else torch.float8_e4m3fn).view(torch.uint8).numpy().copy()
    elif mode == "zeros":
        q[rng.random((ranks, N)) < 0.5] = 0x80
        q[:, 5000:9000] = 0  # whole blocks of zeros
    elif mode == "cancel":
        half = ranks // 2
        q[half:2 * half] = q[:half] ^ 0x80
    elif mode == "top":  # small codes for scales near the top
        q = (q & 0x80) | (q % 32)
    return q


def _scales(rng, dtype, ranks, mode, spread):
    if dtype == "mx":
        nb = N // 32
        base = 241 if mode == "top" else 100
        b = base + rng.integers(0, spread + 1, size=(ranks, nb))
        b[:, 7] = 0  # the smallest scale, nonzero codes
        b[0, 9] = 0  # one rank far below the others
        return np.minimum(b, 243).astype(np.uint8)
    nb = (N + 255) // 256
    s = np.exp2(rng.uniform(0, spread, size=(ranks, nb)) - 12)
    if mode in ("cancel", "zeros"):
        s = np.exp2(np.round(np.log2(s)))  # powers of two: ties
        if mode == "cancel":
            s[:] = s[:1]
    s = s * (2.0 ** 136 / KMAX[dtype] if mode == "top" else 1.0)
    s[:, 3] *= 2.0 ** -120 if mode != "top" else 1.0
    s[:, 11] = 0.0 if mode == "zeros" else s[:, 11]
    return s.astype(np.float32)


@pytest.mark.parametrize("ranks", [3, 8, 16])
@pytest.mark.parametrize("mode,spread", [
    ("dense", 0), ("dense", 25), ("gradients", 2), ("gradients", 12),
    ("zeros", 6), ("cancel", 8), ("top", 2)])
@pytest.mark.parametrize("dtype", ["e4m3", "e5m2", "mx"])
def test_sum2_through_binary64(orc, dtype, mode, spread, ranks):
    say(f"case {dtype} {mode} spread={spread} P={ranks}")
    rng = np.random.default_rng(ranks * 1000 + spread)
    q = _codes(rng, dtype, ranks, mode)
    s = _scales(rng, dtype, ranks, mode, spread)
    stream = torch.cuda.current_stream(DEV)
    dq = [torch.from_numpy(x).to(DEV) for x in q]
    ds = [torch.from_numpy(x).to(DEV) for x in s]
    out = torch.full((N,), 0x7F, dtype=torch.uint8, device=DEV)
    osc = torch.zeros_like(ds[0])
    code, ref = {"e4m3": (pc.FP8_E4M3, orc.sum_e4m3_f32),
                 "e5m2": (pc.FP8_E5M2, orc.sum_e5m2_f32),
                 "mx": (pc.MXFP8_E4M3, orc.sum_mx_f32)}[dtype]
    req = new_request([N], code, pc.SUM, 3, ranks, comp=1)
    req.bind([dq], [out], rank_scales=[ds], out_scales=[osc], stream=stream)
    run_epoch(req, [1, 0, 2], stream)
    gq, gs = out.cpu().numpy(), osc.cpu().numpy()
    req.free()
    wq, ws = ref(list(q), list(s), comp=True)[:2]
    if dtype == "mx":
        assert np.array_equal(gs, ws)
    else:
        assert np.array_equal(as_u32(gs), as_u32(ws))
    assert np.array_equal(gq, wq)
