"""The work that programs have this library do, as cases that can be timed.

Every case goes through the Python binding of the C ABI: single calls
(szx.compress, szx.decompress), as a simulation dumping or loading one field
makes them, and planned batches (szx.compress_batch, szx.decompress_batch), as
a dump of many fields makes them. Buffers and the workspace are kept by the
caller and handed in, which is how the ABI is meant to be used. Fields come
from paper_2201_13020_amd.synth and have the shapes, bounds and block sizes of
the benchmark and the tests:

  sines   1-D sums of sines with noise: time series, transects
  grid    2-D and 3-D random fields with a k^(-5/3) spectrum, with or without
          regions of exact zeros: climate slices, turbulence volumes
  state   1-D interleaved complex amplitudes that decay: state vectors
  mixed   a batch of sines and grids of uneven sizes and both element types
"""
import math

import torch

from paper_2201_13020_amd import synth, szx

DEV = "cuda"

# Uncompressed over compressed bytes of these fields at each bound, measured
# once; they only price the bytes of a pass. (float64 keeps more mantissa
# bytes in the same number of kept bits, so its ratios are about twice.)
RATIO = {
    "sines": {1e-2: 7.0, 1e-3: 3.5, 1e-4: 2.8, 1e-5: 2.1},
    "grid": {1e-2: 4.0, 1e-3: 2.8, 1e-4: 2.1, 1e-5: 1.7},
    "state": {1e-2: 19.0, 1e-3: 11.2, 1e-4: 7.7, 1e-5: 5.6},
    "mixed": {0.0: 3.5},
}


def _case(name, do, field, dims, dtype, eb, mode="rel", block=128, zeros=False):
    d = [int(v) for v in dims] + [0] * (3 - len(dims))
    c = dict(do=do, field=field, d0=d[0], d1=d[1], d2=d[2], dtype=dtype, eb=eb, mode=mode, block=block, zeros=zeros)
    return dict(c, name=name) if name else c


def _batch(name, do, count, median, block=128, stream=6):
    c = dict(do=do, field="mixed", count=count, median=median, block=block, stream=stream)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one short record, compressed where it was produced and read back
        # alone: launches and latency count, no bandwidth does
        _case("compress_record_f32", "compress", "sines", (4099,), "float32", 1e-3),
        _case("decompress_record_f32", "decompress", "sines", (4099,), "float32", 1e-3),
        # a two-dimensional slice in double precision at an absolute bound, as
        # a solver writes it at every output step
        _case("compress_slice_f64", "compress", "grid", (365, 731), "float64", 1e-3, mode="abs"),
        # the 1-D benchmark field: 4 MiB, a few waves per compute unit
        _case("compress_series_f32", "compress", "sines", (1 << 20,), "float32", 1e-3),
        # a latitude-longitude field read back, in blocks of 64
        _case("decompress_latlon_f32", "decompress", "grid", (1800, 3600), "float32", 1e-3, block=64),
        # the headline benchmark's volume, dumped and loaded
        _case("compress_volume_f32", "compress", "grid", (100, 500, 500), "float32", 1e-3, zeros=True),
        _case("decompress_volume_f32", "decompress", "grid", (100, 500, 500), "float32", 1e-3, zeros=True),
        # a volume of odd extents in double precision at a tight bound: long
        # strings of stored bytes, no constant blocks, a ragged last block
        _case("compress_volume_f64", "compress", "grid", (157, 211, 389), "float64", 1e-5),
        # the largest single call: a state vector of 2 GiB
        _case("compress_state_f64", "compress", "state", (1 << 28,), "float64", 1e-3),
        _case("decompress_state_f64", "decompress", "state", (1 << 28,), "float64", 1e-5),
        # a dump of many variables at once, 4 KiB to 64 MiB each, both types,
        # planned once and run every time step
        _batch("batch_compress", "compress", 256, 1 << 20),
        _batch("batch_decompress", "decompress", 256, 1 << 20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["compress", "decompress"])
    block = rng.choice([128, 128, 128, 128, 64, 32, 256])
    kind = rng.choice(["sines", "grid", "grid", "state", "mixed"])
    if kind == "mixed":
        return _batch(None, do, _log_int(rng, 8, 256), _log_int(rng, 32 << 10, 1 << 20), block, rng.randrange(20, 1 << 20))
    eb = rng.choice([1e-2, 1e-3, 1e-4, 1e-5])
    mode = rng.choice(["rel", "rel", "abs"])
    dtype = "float64" if kind == "state" else rng.choice(["float32", "float32", "float64"])
    if kind == "state":
        n = 2 * _log_int(rng, 1 << 11, 1 << 26)
        return _case(None, do, kind, (n,), dtype, eb, "rel", block)
    n = _log_int(rng, 1 << 12, 1 << 25)
    if kind == "sines":
        return _case(None, do, kind, (n,), dtype, eb, mode, block)
    nd = rng.choice([2, 3])
    a = [rng.uniform(math.log(1 / 4), math.log(4)) for _ in range(nd)]
    dims = [max(3, int(math.exp(math.log(n) / nd + v - sum(a) / nd))) for v in a]
    return _case(None, do, kind, dims, dtype, eb, mode, block, zeros=rng.random() < 0.5)


# ------------------------------------------------------------------ fields --

def _dims(case):
    return tuple(int(case[k]) for k in ("d0", "d1", "d2") if case[k])


def _state_vector(n, seed):
    """n/2 complex amplitudes |a_k| = exp(-20 k / (n/2)) / norm with uniform
    phases, real and imaginary parts interleaved."""
    half = n // 2
    q = math.exp(-40.0 / half)
    norm = math.sqrt((1.0 - q ** half) / (1.0 - q))
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    out = torch.empty(half, 2, device=DEV, dtype=torch.float64)
    step = 1 << 24
    for s in range(0, half, step):
        e = min(half, s + step)
        mag = torch.exp(torch.arange(s, e, device=DEV, dtype=torch.float64) * (-20.0 / half)) / norm
        ph = torch.rand(e - s, device=DEV, dtype=torch.float64, generator=g) * (2 * math.pi)
        out[s:e, 0] = mag * torch.cos(ph)
        out[s:e, 1] = mag * torch.sin(ph)
    return out.reshape(-1)


def _field(case, seed):
    dims = _dims(case)
    if case["field"] == "state":
        return _state_vector(dims[0], seed)
    return synth.batch_field(dict(dims=dims, dtype=case["dtype"], seed=seed, zero_regions=bool(case["zeros"])), DEV)


def _specs(case):
    return synth.batch_specs(case["count"], median=case["median"], seed_stream=case["stream"])


def _batch_fields(case, seed):
    specs = _specs(case)
    return [synth.batch_field(dict(s, seed=seed * 4096 + s["index"]), DEV) for s in specs], [s["eb"] for s in specs]


def _flat(sizes, dtype):
    """One zeroed buffer and its pieces of the given sizes, each piece at a
    multiple of 256 bytes."""
    w = torch.empty(0, dtype=dtype).element_size()
    per = 256 // w
    at, pos = [], 0
    for n in sizes:
        at.append(pos)
        pos += -(-max(n, 1) // per) * per
    buf = torch.zeros(max(pos, 1), dtype=dtype, device=DEV)
    return buf, [buf[a:a + max(n, 1)] for a, n in zip(at, sizes)]


def _sizes_on_host(sizes):
    return [int(v) for v in sizes.cpu().view(torch.int64)]


# ----------------------------------------------------------------- prepare --

def _prepare_single(case, seed):
    x = _field(case, seed)
    dims, eb, mode, block = _dims(case), case["eb"], case["mode"], case["block"]
    out = torch.zeros(szx.compress_bound(x.dtype, dims, eb, mode, block), dtype=torch.uint8, device=DEV)
    size = torch.zeros(1, dtype=torch.uint64, device=DEV)
    ws = torch.empty(szx.workspace_size(x.dtype, dims, eb, mode, block), dtype=torch.uint8, device=DEV)
    if case["do"] == "compress":
        return dict(do="compress", x=x, eb=eb, mode=mode, block=block, out=out, size=size, ws=ws)
    # the stream as a program that loads it has it: its bytes alone, and the
    # parameters from its header
    szx.compress(x, eb, mode, block, out=out, out_size=size, ws=ws)
    n = _sizes_on_host(size)[0]
    stream = out[:n].clone()
    info = szx.inspect(stream[:96].cpu())
    return dict(do="decompress", stream=stream, nbytes=n, info=info, ws=ws,
                out=torch.zeros(x.numel(), dtype=x.dtype, device=DEV),
                status=torch.zeros(1, dtype=torch.uint32, device=DEV))


def _by_type(xs):
    """Zeroed outputs for fields like xs: one buffer per element type and each
    field's piece of it."""
    bufs, pieces = {}, [None] * len(xs)
    for key, dt in (("f32", torch.float32), ("f64", torch.float64)):
        idx = [i for i, x in enumerate(xs) if x.dtype == dt]
        bufs[key], got = _flat([xs[i].numel() for i in idx], dt)
        for i, p in zip(idx, got):
            pieces[i] = p
    return bufs, pieces


def _prepare_batch(case, seed):
    xs, ebs = _batch_fields(case, seed)
    block = case["block"]
    caps = [szx.compress_bound(x.dtype, x.shape, eb, "rel", block) for x, eb in zip(xs, ebs)]
    buf, outs = _flat(caps, torch.uint8)
    sizes = torch.zeros(len(xs), dtype=torch.uint64, device=DEV)
    comp = szx.compress_batch(xs, ebs, "rel", block, outs=outs, sizes=[sizes[i:i + 1] for i in range(len(xs))])
    if case["do"] == "compress":
        return dict(do="batch", batch=comp, result=dict(streams=buf, sizes=sizes))
    comp.run()
    n = _sizes_on_host(sizes)
    comp.close()
    sbuf, streams = _flat(n, torch.uint8)
    for s, o, k in zip(streams, outs, n):
        s.copy_(o[:k])
    expected = [dict(dtype=x.dtype, dims=tuple(x.shape), block=block) for x in xs]
    bufs, pieces = _by_type(xs)
    status = torch.zeros(len(xs), dtype=torch.uint32, device=DEV)
    dec = szx.decompress_batch(streams, n, expected, outs=pieces, statuses=[status[i:i + 1] for i in range(len(xs))])
    return dict(do="batch", batch=dec, result=dict(bufs, status=status))


def prepare(case, seed):
    return (_prepare_batch if case["field"] == "mixed" else _prepare_single)(case, seed)


# --------------------------------------------------------------------- run --

def run(state):
    if state["do"] == "compress":
        out, size = szx.compress(state["x"], state["eb"], state["mode"], state["block"], out=state["out"],
                                 out_size=state["size"], ws=state["ws"])
        return dict(stream=out, size=size)
    if state["do"] == "decompress":
        out, status = szx.decompress(state["stream"], state["nbytes"], state["info"], out=state["out"],
                                     status=state["status"], ws=state["ws"])
        return dict(values=out, status=status)
    state["batch"].run()
    return state["result"]


# -------------------------------------------------------------- references --

def exact(case, seed):
    """A decompression returns the field that was compressed, within its
    bound: the field itself is what its values are held against. A stream's
    bytes and sizes are whole numbers and have no such value."""
    if case["do"] == "compress":
        return None
    if case["field"] != "mixed":
        return dict(values=_field(case, seed).reshape(-1).double(), status=None)
    xs, _ = _batch_fields(case, seed)
    bufs, pieces = _by_type(xs)
    for p, x in zip(pieces, xs):
        p[:x.numel()] = x.reshape(-1)
    return dict({k: b.double() for k, b in bufs.items()}, status=None)


def work(case):
    """Bytes of one pass: the field and its stream, each once."""
    if case["field"] == "mixed":
        raw = sum(synth.spec_elems(s) * (8 if s["dtype"] == "float64" else 4) for s in _specs(case))
        return dict(bytes=raw * (1 + 1 / RATIO["mixed"][0.0]), flops=0)
    raw = math.prod(_dims(case)) * (8 if case["dtype"] == "float64" else 4)
    ratio = RATIO[case["field"]][case["eb"]] * (2 if case["dtype"] == "float64" and case["field"] != "state" else 1)
    return dict(bytes=raw * (1 + 1 / ratio), flops=0)
