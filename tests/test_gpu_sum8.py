"""The compensated sums of the 8-bit payloads, which the kernels take from
plain binary32 sums (e4m3, e5m2) and integers (MX blocks) wherever that gives
Sum2's codes and scales.  Finite inputs that leave few or many values open
(sums halfway between two codes, near ties for a block's largest value, one
rank far below the others) against the oracle's Sum2; infinities and NaN, in
codes and scales, against the kernels' own Sum2, which a whole row takes when
it holds an infinite scale (e4m3, e5m2) or scales far apart (MX)."""
import numpy as np
import pytest
import torch

from _gpu import DEV, as_u32, new_request, say
from oracle import get as get_oracle
from paper_2604_22228_amd import pcoll as pc

pytestmark = pytest.mark.gpu
DTYPE = {"e4m3": pc.FP8_E4M3, "e5m2": pc.FP8_E5M2, "mx": pc.MXFP8_E4M3}
BLOCK = {"e4m3": 256, "e5m2": 256, "mx": 32}
N = 1024 * 24 + 512  # whole rows and half a one


@pytest.fixture(scope="module")
def orc():
    return get_oracle()


def _reduce(dtype, q, s, size=None):
    """Codes and scales of the sum; in buckets of `size` elements each."""
    n, blk = q.shape[1], BLOCK[dtype]
    size = size or n
    nb = n // size
    dq = [torch.from_numpy(x.copy()).to(DEV) for x in q]
    ds = [torch.from_numpy(x.copy()).to(DEV) for x in s]
    out = torch.full((n,), 0x55, dtype=torch.uint8, device=DEV)
    osc = torch.zeros_like(ds[0])
    cut = [slice(i * size, (i + 1) * size) for i in range(nb)]
    cuts = [slice(i * size // blk, -(-(i + 1) * size // blk))
            for i in range(nb)]
    req = new_request([size] * nb, DTYPE[dtype], pc.SUM, 1, q.shape[0], comp=1)
    req.bind([[x[c] for x in dq] for c in cut], [out[c] for c in cut],
             rank_scales=[[x[c] for x in ds] for c in cuts],
             out_scales=[osc[c] for c in cuts],
             stream=torch.cuda.current_stream(DEV))
    req.start()
    req.pready_range(0, nb - 1)
    req.wait()
    req.free()
    torch.cuda.synchronize()
    return out.cpu().numpy(), osc.cpu().numpy()


def _finite(dtype):
    top = 0x7C if dtype == "e5m2" else 0x7F
    return np.array([c for c in range(256) if (c & 0x7F) < top], np.uint8)


def _inputs(dtype, mode, ranks, rng):
    q = rng.choice(_finite(dtype), size=(ranks, N))
    nb = N // BLOCK[dtype]
    if dtype == "mx":
        b = 120 + rng.integers(0, 3, size=(ranks, nb))
        if mode == "spread":  # around the integers' limits, 9 to 11
            b = 120 + rng.integers(0, 13, size=(ranks, nb))
            b[:, ::2] = 120 + rng.integers(0, 10, size=b[:, ::2].shape)
        elif mode == "far":
            b[0] = rng.integers(0, 120, size=nb)
        elif mode == "ends":
            b = np.where(rng.random((1, nb)) < 0.5, rng.integers(0, 12, nb),
                         rng.integers(236, 245, nb)) + 0 * b
            q = (q & 0x80) | (q % 64)
        return q, b.astype(np.uint8)
    s = np.float32(1.2345678) * np.exp2(rng.integers(-3, 4, (ranks, nb)))
    if mode == "equal":  # sums are multiples of one odd number
        s[:] = np.float32(0.7654321)
    elif mode == "ones":
        s[:] = 1.0
    elif mode == "powers":
        s = np.exp2(rng.integers(0, 8, (ranks, nb)).astype(np.float64))
    elif mode == "spread":
        s = np.exp2(rng.uniform(0, 40, (ranks, nb)))
    elif mode == "far":
        s[0] *= 2.0 ** -25
    elif mode == "flat":  # every value of a block ties for the largest
        q[:] = q[:, :1]
    elif mode == "near":  # the same, but for one rank far below
        q[1:] = q[1:, :1]
        s[0] *= 2.0 ** -18
    elif mode == "cancel":
        q[1] = q[0] ^ 0x80
        s[1] = s[0]
        s[2:] *= 2.0 ** -22
    elif mode == "ends":  # scales at binary32's lower end
        s = s * 2.0 ** -126
        s[:, ::3] *= 2.0 ** -15
    return q, s.astype(np.float32)


MODES = {"e4m3": ["odd", "equal", "ones", "powers", "spread", "far", "flat",
                  "near", "cancel", "ends"],
         "mx": ["odd", "spread", "far", "ends"]}
MODES["e5m2"] = MODES["e4m3"]


@pytest.mark.parametrize("n", [1, 15, 16, 17, 255, 257, 700, 1023, 1025])
@pytest.mark.parametrize("ranks", [2, 3, 8, 16])
@pytest.mark.parametrize("dtype", ["e4m3", "e5m2"])
def test_last_row(orc, dtype, ranks, n):
    say(f"case last row {dtype} P={ranks} n={n}")
    rng = np.random.default_rng(n)
    q, s = _inputs(dtype, "odd", ranks, rng)
    q, s = q[:, :n], s[:, :(n + 255) // 256]
    gq, gs = _reduce(dtype, q, s)
    ref = {"e4m3": orc.sum_e4m3_f32, "e5m2": orc.sum_e5m2_f32}[dtype]
    wq, ws = ref(list(q.copy()), list(s.copy()), comp=True)[:2]
    assert np.array_equal(as_u32(gs), as_u32(ws))
    assert np.array_equal(gq, wq)


@pytest.mark.parametrize("ranks", [3, 5, 8, 9, 16])
@pytest.mark.parametrize("dtype,mode",
                         [(d, m) for d in DTYPE for m in MODES[d]])
def test_sum2_bits(orc, dtype, mode, ranks):
    say(f"case {dtype} {mode} P={ranks}")
    rng = np.random.default_rng(ranks * 31 + len(mode))
    q, s = _inputs(dtype, mode, ranks, rng)
    gq, gs = _reduce(dtype, q, s)
    ref = {"e4m3": orc.sum_e4m3_f32, "e5m2": orc.sum_e5m2_f32,
           "mx": orc.sum_mx_f32}[dtype]
    wq, ws = ref(list(q), list(s), comp=True)[:2]
    if dtype == "mx":
        assert np.array_equal(gs, ws)
    else:
        assert np.array_equal(as_u32(gs), as_u32(ws))
    assert np.array_equal(gq, wq)


@pytest.mark.parametrize("ranks", [3, 8, 16])
@pytest.mark.parametrize("what", ["none", "inf codes", "mixed inf codes",
                                  "nan codes", "inf scale", "nan scale"])
@pytest.mark.parametrize("dtype", ["e4m3", "e5m2"])
def test_special_values_as_sum2(dtype, what, ranks):
    if dtype == "e4m3" and "inf codes" in what:
        pytest.skip("e4m3 has no infinities")
    say(f"case {dtype} {what} P={ranks}")
    rng = np.random.default_rng(ranks)
    n = 1024 * 12
    q = rng.choice(_finite(dtype), size=(ranks, n))
    s = rng.uniform(0.5, 2.0, (ranks, n // 256)).astype(np.float32)
    at = rng.random((ranks, n)) < 1 / 4096
    at[:, ::1800] = True
    if what == "inf codes":
        q[at] = 0x7C
    elif what == "mixed inf codes":
        q[at] = rng.choice(np.array([0x7C, 0xFC], np.uint8), size=at.sum())
    elif what == "nan codes":
        q[at] = rng.choice(np.array([0x7F, 0xFF], np.uint8), size=at.sum())
    elif what == "inf scale":
        s[ranks - 1, 5::9] = np.inf
    elif what == "nan scale":
        s[1, 5::9] = np.nan
    gq, gs = _reduce(dtype, q, s)
    # each block beside one of an infinite scale, whose row takes Sum2 itself
    nb = n // 256
    q2, s2 = np.zeros((ranks, nb, 512), np.uint8), np.ones((ranks, nb, 2), "f")
    q2[:, :, :256], s2[:, :, 0] = q.reshape(ranks, nb, 256), s
    q2[0, :, 256:], s2[0, :, 1] = 0x38, np.inf
    wq, ws = _reduce(dtype, q2.reshape(ranks, -1), s2.reshape(ranks, -1),
                     size=512)
    wq, ws = wq.reshape(nb, 512)[:, :256].reshape(-1), ws.reshape(nb, 2)[:, 0]
    assert np.array_equal(as_u32(gs), as_u32(ws))
    assert np.array_equal(gq, wq)


@pytest.mark.parametrize("ranks", [3, 8, 16])
@pytest.mark.parametrize("what", ["none", "nan codes", "byte 255",
                                  "byte 255 of zeros"])
def test_mx_special_values_as_sum2(what, ranks):
    say(f"case mx {what} P={ranks}")
    rng = np.random.default_rng(ranks)
    n = 1024 * 12
    q = rng.choice(_finite("mx"), size=(ranks, n))
    b = (120 + rng.integers(0, 6, (ranks, n // 32))).astype(np.uint8)
    if what == "nan codes":
        q[rng.random((ranks, n)) < 1 / 2048] = 0x7F
        q[1, ::1500] = 0xFF
    elif "255" in what:
        b[1, 5::67] = 255
        b[ranks - 1, 9::71] = 255
        if what.endswith("zeros"):
            for r, k in ((1, slice(5, None, 67)), (ranks - 1,
                                                   slice(9, None, 71))):
                q.reshape(ranks, -1, 32)[r, k] = 0
    gq, gs = _reduce("mx", q, b)
    # a block in every row whose scales are too far apart for anything else
    wide = b.copy()
    wide[0, 31::32], wide[1, 31::32] = 100, 160
    wq, ws = _reduce("mx", q, wide)
    keep = np.arange(n // 32) % 32 != 31
    assert np.array_equal(gs[keep], ws[keep])
    assert np.array_equal(gq.reshape(-1, 32)[keep], wq.reshape(-1, 32)[keep])
    if what == "nan codes":  # and they are NaN where a term is
        isnan = ((q & 0x7F) == 0x7F).any(axis=0)
        assert np.array_equal((gq & 0x7F) == 0x7F, isnan)
