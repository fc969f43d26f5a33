"""The workloads that the library's speed is measured on.

A case is a dict of plain values: `kind` says which public entry points it
goes through, the rest its sizes and options.

  reduce   a persistent request (init, bind kept; start, ready calls, wait
           timed): one message, or several buckets laid out in one arena per
           rank as a gradient buffer is, readied from the host
  device   the same request readied from the device: each rank's gradients
           are packed to bf16 on a producer stream and marked there, while
           the request's kernel waits
  noalloc  the allocation-free epoch
  pack     a producer-side packer

Inputs come from torch generators on the GPU.  exact() gives the same
results in binary64 with torch alone.
"""
import math

import numpy as np
import torch

from paper_2604_22228_amd import pcoll as pc
from paper_2604_22228_amd import streams, synth

DTYPES = {"i32": pc.INT32, "f32": pc.FLOAT32, "bf16": pc.BFLOAT16,
          "bf16pair": pc.BF16_PAIR, "e4m3": pc.FP8_E4M3, "e5m2": pc.FP8_E5M2,
          "mx": pc.MXFP8_E4M3}
OPS = {"sum": pc.SUM, "max": pc.MAX}
EIGHT_BIT = ("e4m3", "e5m2", "mx")
FLOAT8 = {"e4m3": torch.float8_e4m3fn, "e5m2": torch.float8_e5m2,
          "mx": torch.float8_e4m3fn}
FMT_MAX = {"e4m3": 448.0, "e5m2": 57344.0}
BLOCK = {"e4m3": 256, "e5m2": 256, "mx": 32}
ALIGN = 256  # elements between the starts of two buckets in an arena


def listed():
    return [
        # the smallest message of the size sweep: a few bias or norm
        # gradients, where only the calls and the launch count
        {"name": "f32_sum_r8_4KiB", "kind": "reduce", "dtype": "f32",
         "op": "sum", "ranks": 8, "count": 1024, "parts": 1,
         "ready": "each"},
        # the plain workload: one 1 MiB message, 8 partitions in order
        {"name": "f32_sum_r4_1MiB", "kind": "reduce", "dtype": "f32",
         "op": "sum", "ranks": 4, "count": 262144, "parts": 8,
         "ready": "each"},
        # a layer's gradient of no round size over an odd number of ranks
        {"name": "f32_sum_r3_ragged", "kind": "reduce", "dtype": "f32",
         "op": "sum", "ranks": 3, "count": 3000017, "parts": 13,
         "ready": "list"},
        # the headline: a large message whose 64 partitions become ready one
        # by one
        {"name": "f32_sum_r8_256MiB", "kind": "reduce", "dtype": "f32",
         "op": "sum", "ranks": 8, "count": 1 << 26, "parts": 64,
         "ready": "each"},
        # exact integer reduction over the most ranks
        {"name": "i32_sum_r16_64MiB", "kind": "reduce", "dtype": "i32",
         "op": "sum", "ranks": 16, "count": 1 << 24, "parts": 256,
         "ready": "list"},
        # a model's gradients in 64 bf16 buckets of 64 KiB .. 64 MiB
        {"name": "bf16_sum_r8_batch64", "kind": "reduce", "dtype": "bf16",
         "op": "sum", "ranks": 8, "buckets": 64, "lo": 1 << 15,
         "hi": 1 << 25, "sizes_seed": 22231, "parts": 32, "ready": "list"},
        # bf16 gradients whose sum is wanted to 16 significant bits
        {"name": "bf16pair_sum_r8_batch8", "kind": "reduce",
         "dtype": "bf16pair", "op": "sum", "ranks": 8, "buckets": 8,
         "lo": 1 << 16, "hi": 1 << 24, "sizes_seed": 5, "parts": 16,
         "ready": "list"},
        # 8-bit gradients with block scales, 128 buckets, about 2^30 elements
        {"name": "e4m3_sum_r8_batch128", "kind": "reduce", "dtype": "e4m3",
         "op": "sum", "ranks": 8, "buckets": 128, "lo": 1 << 19,
         "hi": 1 << 25, "sizes_seed": 22233, "parts": 32, "ready": "list"},
        # the same values' OCP MX form, a quarter of the model
        {"name": "mx_sum_r8_batch32", "kind": "reduce", "dtype": "mx",
         "op": "sum", "ranks": 8, "buckets": 32, "lo": 1 << 19,
         "hi": 1 << 25, "sizes_seed": 22234, "parts": 32, "ready": "list"},
        # the encode direction: a rank packs its gradients, ragged end
        {"name": "pack_e4m3_2p26", "kind": "pack", "dtype": "e4m3",
         "count": (1 << 26) + 77},
        # a serving loop that may not allocate: one small bf16 message
        {"name": "noalloc_bf16_r8_2MiB", "kind": "noalloc", "dtype": "bf16",
         "op": "sum", "ranks": 8, "count": 1048583, "parts": 16},
        # gradients packed and marked on the device while the kernel waits
        {"name": "device_bf16_r8_8MiB", "kind": "device", "dtype": "bf16",
         "op": "sum", "ranks": 8, "count": 1 << 22, "parts": 8},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: every dtype, op and rank count the library takes, sizes
    over the listed cases' range, odd ones mostly."""
    kind = rng.choice(["reduce", "reduce", "reduce", "batch", "batch", "pack",
                       "noalloc", "device"])
    if kind == "pack":
        return {"kind": "pack", "dtype": rng.choice(["bf16", "e4m3", "e5m2",
                                                     "mx"]),
                "count": _log_int(rng, 1 << 10, 1 << 27)}
    ranks = rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 8, 8, 12, 16])
    if kind == "device":
        return {"kind": "device", "dtype": "bf16", "op": "sum",
                "ranks": rng.choice([2, 3, 4, 6, 8]),
                "count": _log_int(rng, 1 << 12, 1 << 24),
                "parts": rng.choice([1, 4, 8, 16, 32])}
    dtype = rng.choice(list(DTYPES))
    op = rng.choice(["sum", "sum", "max"]) if dtype in ("i32", "f32", "bf16") \
        else "sum"
    if kind == "batch":
        hi = _log_int(rng, 1 << 16, 1 << 23)
        return {"kind": "reduce", "dtype": dtype, "op": op, "ranks": ranks,
                "buckets": rng.randint(2, 48), "lo": 1 << 12, "hi": hi,
                "sizes_seed": rng.randrange(1 << 20),
                "parts": rng.choice([1, 4, 8, 16, 32]), "ready": "list"}
    count = _log_int(rng, 256, 1 << 26)
    if dtype == "mx":  # whole scale blocks
        count = max(32, count // 32 * 32)
    parts = rng.choice([1, 2, 4, 7, 16, 64, 256])
    case = {"kind": kind, "dtype": dtype, "op": op, "ranks": ranks,
            "count": count, "parts": parts}
    if kind == "reduce":
        case["ready"] = rng.choice(["each", "list", "range"])
    return case


# ------------------------------------------------------------------- inputs
def _counts(case):
    if "buckets" not in case:
        return [case["count"]]
    rng = np.random.default_rng(case["sizes_seed"])
    u = rng.uniform(math.log(case["lo"]), math.log(case["hi"]),
                    size=case["buckets"])
    step = 32 if case["dtype"] == "mx" else 1
    return [max(32, int(math.exp(v)) // step * step) for v in u]


def _offsets(counts):
    offs, at = [], 0
    for c in counts:
        offs.append(at)
        at += (c + ALIGN - 1) // ALIGN * ALIGN
    return offs, at


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _values(case, n, gen):
    """One rank's values: integer counters, or gradients (8-bit payloads:
    with 1 % outliers of 50 times the size)."""
    if case["dtype"] == "i32":
        return torch.randint(-(1 << 20), (1 << 20) + 1, (n,), generator=gen,
                             device="cuda", dtype=torch.int32)
    x = torch.randn(n, generator=gen, device="cuda")
    if case["dtype"] in EIGHT_BIT:
        x *= 1e-2
        m = torch.rand(n, generator=gen, device="cuda") < 0.01
        x = torch.where(m, x * 50.0, x)
    elif case["dtype"] != "f32":
        x *= 1e-3
    return x


def _blocks(x, size):
    """x as rows of `size` elements, the last row filled up with zeros."""
    pad = -x.numel() % size
    if pad:
        x = torch.cat([x, x.new_zeros(pad)])
    return x.view(-1, size)


def _mx_exponent(amax):
    """Smallest e >= -127 with amax <= 448 * 2^e."""
    m, k = torch.frexp(amax)
    e = k - 9 + (m > 0.875).to(k.dtype)
    return torch.where(amax == 0, torch.full_like(e, -127),
                       e.clamp_min(-127))


def _quantize(x, dtype):
    """(codes, scales) of binary32 values, with torch alone."""
    b = _blocks(x, BLOCK[dtype])
    amax = b.abs().amax(1)
    if dtype == "mx":
        e = _mx_exponent(amax)
        q = torch.ldexp(b, -e[:, None])
        scale = (e + 127).to(torch.uint8)
    else:
        scale = amax / FMT_MAX[dtype]
        scale = torch.where(scale >= 2.0 ** -126, scale,
                            torch.ones_like(scale))
        q = (b * (1.0 / scale)[:, None]).clamp_(-FMT_MAX[dtype],
                                                FMT_MAX[dtype])
    return q.to(FLOAT8[dtype]).reshape(-1)[:x.numel()], scale


def _dequantize(codes, scale, dtype):
    b = _blocks(codes.to(torch.float64), BLOCK[dtype])
    s = torch.ldexp(torch.ones_like(scale, dtype=torch.float64),
                    scale.to(torch.int32) - 127) if dtype == "mx" \
        else scale.double()
    return (b * s[:, None]).reshape(-1)[:codes.numel()]


def _ranks(case, seed):
    """Yields each rank's arena: (values or codes, scales or None).  Padding
    between buckets is zero."""
    counts = _counts(case)
    offs, total = _offsets(counts)
    gen = _gen(seed)
    whole = all(c % ALIGN == 0 for c in counts)
    for _ in range(case["ranks"]):
        x = _values(case, total, gen)
        if not whole:
            for o, c in zip(offs, counts):
                x[o + c:(o + c + ALIGN - 1) // ALIGN * ALIGN] = 0
        if case["dtype"] in EIGHT_BIT:
            yield _quantize(x, case["dtype"])
        elif case["dtype"] in ("bf16", "bf16pair"):
            yield x.to(torch.bfloat16), None
        else:
            yield x, None


def _slices(arena, offs, counts, block=1):
    return [arena[o // block:(o + c + block - 1) // block]
            for o, c in zip(offs, counts)]


# ------------------------------------------------------------------ prepare
def prepare(case, seed):
    st = {"case": dict(case)}
    if case["kind"] == "pack":
        n = case["count"]
        x = _values(case, n, _gen(seed))
        st["x"] = x
        if case["dtype"] == "bf16":
            st["out"] = torch.zeros(n, dtype=torch.bfloat16, device="cuda")
        else:
            b = BLOCK[case["dtype"]]
            st["out"] = torch.zeros(n, dtype=torch.uint8, device="cuda")
            st["scale"] = torch.zeros(
                (n + b - 1) // b, device="cuda",
                dtype=torch.uint8 if case["dtype"] == "mx" else torch.float32)
        st["stream"] = torch.cuda.current_stream()
        return st

    counts = _counts(case)
    offs, total = _offsets(counts)
    dt = case["dtype"]
    if case["kind"] == "device":
        gen = _gen(seed)
        st["x"] = [_values(case, case["count"], gen)
                   for _ in range(case["ranks"])]
        arenas = [(torch.zeros(total, dtype=torch.bfloat16, device="cuda"),
                   None) for _ in range(case["ranks"])]
    else:
        arenas = list(_ranks(case, seed))
    eight = dt in EIGHT_BIT
    block = BLOCK.get(dt, 1)
    out = torch.zeros(total, device="cuda",
                      dtype=torch.uint8 if eight else arenas[0][0].dtype)
    second = None
    if eight:
        second = torch.zeros(total // block, dtype=arenas[0][1].dtype,
                             device="cuda")
    elif dt == "bf16pair":
        second = torch.zeros_like(out)
    st["out"], st["second"], st["arenas"] = out, second, arenas
    ins = [list(b) for b in zip(*[_slices(a, offs, counts)
                                  for a, _ in arenas])]
    scales = [list(b) for b in zip(*[_slices(s, offs, counts, block)
                                     for _, s in arenas])] if eight else None
    outs = _slices(out, offs, counts)
    seconds = _slices(second, offs, counts, block) if second is not None \
        else None

    if case["kind"] == "noalloc":
        st["ins"], st["scales"] = ins[0], scales[0] if scales else None
        st["stream"] = torch.cuda.current_stream()
        return st

    req = pc.Request(counts, DTYPES[dt], OPS[case["op"]], case["parts"],
                     case["ranks"])
    if case["kind"] == "device":
        bound, producer = _comm_and_producer()
        st["producer"] = producer
        st["ids"] = torch.arange(case["parts"], dtype=torch.int32,
                                 device="cuda")
    else:
        bound = torch.cuda.Stream()
    # the buffers were written on the current stream
    bound.wait_stream(torch.cuda.current_stream())
    req.bind(ins, outs, scales, seconds, stream=bound)
    order = synth.permutation(req.nparts_total, seed).astype(np.int32)
    st["req"], st["stream"] = req, bound
    st["order"] = order if case.get("ready") == "list" else order.tolist()
    return st


_streams = []


def _comm_and_producer():
    """The program's communication stream, and a producer stream that runs
    beside it; both are kept for the whole program."""
    if not _streams:
        bound = torch.cuda.Stream()
        _streams.append((bound, streams.independent_streams(bound, 1)[0]))
    return _streams[0]


# ---------------------------------------------------------------------- run
_PACK8 = {"e4m3": pc.pcoll_pack_fp8, "e5m2": pc.pcoll_pack_e5m2,
          "mx": pc.pcoll_pack_mxfp8}


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "pack":
        if case["dtype"] == "bf16":
            pc.pcoll_pack_bf16(st["x"], st["out"], case["count"],
                               st["stream"])
            return {"out": st["out"]}
        _PACK8[case["dtype"]](st["x"], st["out"], st["scale"], case["count"],
                              st["stream"])
        return {"out": st["out"].view(FLOAT8[case["dtype"]]),
                "scale": st["scale"]}
    if kind == "noalloc":
        pc.pcoll_reduce_noalloc(case["count"], DTYPES[case["dtype"]],
                                OPS[case["op"]], case["parts"], st["ins"],
                                st["out"], st["scales"], st["second"],
                                st["stream"])
        return _outputs(st)
    req = st["req"]
    req.start()
    if kind == "device":
        prod = st["producer"]
        for r, x in enumerate(st["x"]):
            pc.pcoll_pack_bf16(x, st["arenas"][r][0], case["count"], prod)
            req.pready_rank_on_stream(r, st["ids"], case["parts"], prod)
    elif case["ready"] == "each":
        for p in st["order"]:
            req.pready(p)
    elif case["ready"] == "list":
        req.pready_list(st["order"])
    else:
        req.pready_range(0, req.nparts_total - 1)
    req.wait()
    return _outputs(st)


def _outputs(st):
    dt = st["case"]["dtype"]
    if dt in EIGHT_BIT:
        return {"out": st["out"].view(FLOAT8[dt]), "scale": st["second"]}
    if dt == "bf16pair":
        return {"out": st["out"], "low": st["second"]}
    return {"out": st["out"]}


# --------------------------------------------------------------------- work
def work(case):
    if case["kind"] == "pack":
        n = case["count"]
        if case["dtype"] == "bf16":
            return {"bytes": 6 * n, "flops": n}
        b = BLOCK[case["dtype"]]
        return {"bytes": 5 * n + (1 if case["dtype"] == "mx" else 4) *
                ((n + b - 1) // b), "flops": 2 * n}
    ranks, dt = case["ranks"], case["dtype"]
    size = pc.ELEM_BYTES[DTYPES[dt]]
    total = 0
    for n in _counts(case):
        total += (ranks + 1) * size * n
        if dt in EIGHT_BIT:
            total += (ranks + 1) * (1 if dt == "mx" else 4) * (
                (n + BLOCK[dt] - 1) // BLOCK[dt])
        elif dt == "bf16pair":
            total += size * n
        if case["kind"] == "device":  # packing: binary32 in, bf16 out
            total += ranks * 6 * n
    return {"bytes": total, "flops": max(1, ranks - 1) * sum(_counts(case))}


# -------------------------------------------------------------------- exact
def exact(case, seed):
    dt = case["dtype"]
    if case["kind"] == "pack":
        x = _values(case, case["count"], _gen(seed)).double()
        return {"out": x} if dt == "bf16" else _exact_blocks(x, dt)
    if case["kind"] == "device":
        gen = _gen(seed)
        parts = ((_values(case, case["count"], gen).to(torch.bfloat16), None)
                 for _ in range(case["ranks"]))
    else:
        parts = _ranks(case, seed)
    acc = None
    for v, s in parts:
        v = _dequantize(v, s, dt) if s is not None else (
            v if dt == "i32" else v.double())
        if acc is None:
            acc = v
        elif case["op"] == "max":
            acc = torch.maximum(acc, v)
        else:
            acc = acc + v
    if dt in EIGHT_BIT:
        return _exact_blocks(acc, dt)
    if case["kind"] == "device":  # the arena's padding stays zero
        acc = torch.cat([acc, acc.new_zeros(-case["count"] % ALIGN)])
    if dt == "bf16pair":  # the two halves carry the sum together
        return {"out": acc, "low": None}
    return {"out": acc}


def _exact_blocks(x, dt):
    """The 8-bit results before their rounding: each value over its block's
    scale, and the scale."""
    b = _blocks(x, BLOCK[dt])
    amax = b.abs().amax(1)
    if dt == "mx":
        e = _mx_exponent(amax)
        return {"out": torch.ldexp(b, -e[:, None]).reshape(-1)[:x.numel()],
                "scale": None}
    scale = amax / FMT_MAX[dt]
    scale = torch.where(scale >= 2.0 ** -126, scale, torch.ones_like(scale))
    return {"out": (b / scale[:, None]).reshape(-1)[:x.numel()],
            "scale": scale}
