"""The encoder's packing and tile order at the edges of its rows, rings and
tickets, byte for byte against the oracle: strings of every length (kept bytes
0 to the whole word), rows of constant, coded and raw blocks side by side,
tiles that fill a wave's LDS ring, a short last block, and few persistent
workgroups, so that each takes many tiles and its ring wraps again and again."""
import numpy as np
import pytest
import torch

from gpu_util import gpu_compress
from oracle import szref
from paper_2201_13020_amd import szx

pytestmark = pytest.mark.gpu


def field(kind, n, dtype, block):
    """Values whose blocks keep few bytes, many, all of them, or none."""
    r = np.random.default_rng(len(kind) * 1000 + n + block)
    x = r.standard_normal(n)
    if kind == "smooth":  # few mid bytes a value: several strings a dword
        x = np.cumsum(x) * 1e-3
    elif kind == "noise":  # every mantissa byte: the ring fills
        x = x * np.exp2(r.integers(-30, 30, n))
    elif kind == "mixed":  # blocks of every sort next to each other
        nblk = -(-n // block)
        sort = r.integers(0, 5, nblk)
        amp = np.choose(sort, [0.0, 1e-6, 1e-3, 1.0, 1.0])
        x = x * np.repeat(amp, block)[:n] + np.repeat(r.standard_normal(nblk), block)[:n]
        raw = np.repeat(sort == 4, block)[:n] & (r.random(n) < 0.02)
        x[raw] = np.nan
    return x.astype(dtype)


CASES = [  # values, wgs: one tile, ragged tiles, tens of tiles on eight workgroups
    (1, 0), (4097, 0), (8191, 0), (40_000, 0), (600_007, 8), (300_000, 9)]
# (With blocks of 128, 512 and 1024 values the last two take the two-launch path, which has
# a workgroup a tile: test_few_workgroups_above_the_small_calls and
# test_full_rings_follow_partly_filled_ones have the tickets and rings there.)


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("block", [8, 16, 64, 128, 512, 1024])
@pytest.mark.parametrize("kind", ["smooth", "noise", "mixed"])
def test_streams_equal_the_oracle(kind, block, dtype):
    dt = torch.float32 if dtype == "float32" else torch.float64
    for n, wgs in CASES:
        x = field(kind, n, dtype, block)
        cls = szx.size_class(x.nbytes)
        for eb, mode in ((1e-3, "rel"), (0.0, "abs")):
            ref = szref.compress(x, eb, mode, block)
            try:
                szx.set_geometry(dt, cls, wgs)
                out, size = gpu_compress(x, eb, mode, block)
            finally:
                szx.set_geometry(dt, cls, 0)
            assert size == ref.size and np.array_equal(out[:size].cpu().numpy(), ref), (n, wgs, eb)


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("block", [8, 32, 128, 1024])
def test_one_two_and_three_launches_meet(block, dtype):
    """Sizes on both sides of where a single call goes from one workgroup to two
    launches (64 KiB of float32, 96 of float64) and on to three (8192 blocks or
    256 tiles), a size of the smaller workgroup, and of ragged tiles: with
    non-finite values, blocks whose half range is the bound itself, and a
    workspace that first holds anything and then what a call left."""
    w = 4 if dtype == "float32" else 8
    small, most = (16384 if w == 4 else 12288), min(8192 * block, 256 * max(8 * block, 32768 // w))
    for line in (32768 // w, small, 100_003, most):
        for n in (line - 1, line, line + 1):
            for kind in ("mixed", "noise", "steps") if n < 1 << 18 else ("mixed",):
                if kind == "steps":
                    x = (np.random.default_rng(n).integers(0, 4, n) * 0.5).astype(dtype)
                    x[: n // 2] = np.minimum(x[: n // 2], 1)
                else:
                    x = field(kind, n, dtype, block)
                x[n // 3] = np.inf
                for eb, mode in ((1e-2, "rel"), (0.5, "abs"), (0.0, "rel")):
                    ref = szref.compress(x, eb, mode, block)
                    ws = torch.full((szx.workspace_size(dtype, (n,), eb, mode, block),), 0x5A, dtype=torch.uint8,
                                    device="cuda")
                    for use in range(2):
                        out, size = szx.compress(torch.from_numpy(x).cuda(), eb, mode, block, ws=ws)
                        torch.cuda.synchronize()
                        m = int(size.cpu().view(torch.int64))
                        assert m == ref.size and np.array_equal(out[:m].cpu().numpy(), ref), (n, kind, eb, mode, use)


@pytest.mark.parametrize("block", [8, 32, 128, 512, 1024])
@pytest.mark.parametrize("types", ["both", "float32", "float64", "few float32", "few float64"])
def test_batches_of_one_and_both_types(types, block):
    """Batches whose two types share their launches, and batches of one type:
    fields without values, of one tile and of many, all workgroups or eight,
    and (b = 8) an index that is chained; streams and decoded values against
    the oracle, twice over the same workspace."""
    sizes = [0, 1, 70_001, 30_000, 0, 250_003, block, 9]
    fields = []
    for i, n in enumerate(sizes):
        for dt in ("float32", "float64"):
            if types in ("both", dt) or (types[:3] == "few" and (types[4:] != dt or i == 3)):
                x = field("mixed" if i % 2 else "smooth", max(n, 1), dt, block)[:n]
                fields.append((x, (1e-3, 0.0, 1e-2)[i % 3], "rel" if i % 2 else "abs"))
    if block == 8 and types == "both":
        fields.append((field("smooth", 2_100_001, "float32", block), 1e-2, "rel"))
    refs = [szref.compress(x, eb, mode, block) for x, eb, mode in fields]
    b = szx.compress_batch([torch.from_numpy(x).cuda() for x, _, _ in fields], [f[1] for f in fields],
                           [f[2] for f in fields], block)
    for use in range(2):
        if use:
            b.set_geometry(8)
        for o, size in zip(b.outs, b.sizes):
            o.fill_(0xAB)
            size.fill_(0xAB)
        b.run()
        torch.cuda.synchronize()
        for i, ref in enumerate(refs):
            m = int(b.sizes[i].cpu().view(torch.int64))
            assert m == ref.size and np.array_equal(b.outs[i][:m].cpu().numpy(), ref), (i, use)
    d = szx.decompress_batch(b.outs, [r.size for r in refs], [szx.inspect(r[:96].tobytes()) for r in refs])
    for use in range(2):
        for s in d.statuses:
            s.fill_(0xAB)
        d.run()
        torch.cuda.synchronize()
        for i, ref in enumerate(refs):
            assert int(d.statuses[i].cpu().view(torch.int32)) == 0, (i, use)
            y = szref.decompress(ref).ravel()
            assert np.array_equal(d.outs[i][: y.size].cpu().numpy().view(np.uint8), y.view(np.uint8)), (i, use)


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("block", [128, 512, 1024])
def test_few_workgroups_above_the_small_calls(block, dtype):
    """Single calls beyond the one- and two-launch sizes on eight workgroups,
    whose rings wrap many times, and on the default number."""
    dt = torch.float32 if dtype == "float32" else torch.float64
    n = 2_200_003
    for kind in ("mixed", "noise"):
        x = field(kind, n, dtype, block)
        cls = szx.size_class(x.nbytes)
        ref = szref.compress(x, 1e-3, "rel", block)
        for wgs in (8, 0):
            try:
                szx.set_geometry(dt, cls, wgs)
                out, size = gpu_compress(x, 1e-3, "rel", block)
            finally:
                szx.set_geometry(dt, cls, 0)
            assert size == ref.size and np.array_equal(out[:size].cpu().numpy(), ref), (kind, wgs)


@pytest.mark.parametrize("wgs", [0, 2048])
@pytest.mark.parametrize("n32,n64", [(32, 32), (33, 31), (31, 33), (48, 4)])
def test_both_types_with_a_workgroup_beyond_the_resident_ones(n32, n64, wgs):
    """A batch of both types whose float32 tiles number as many as the launch's
    workgroups or a few more or less (32 fields of 1 MiB are 1024 tiles, four a
    compute unit), so that workgroups with a tile of their own start only when
    others have ended; with more workgroups asked for, many of them. Twice over
    one workspace, and on two streams side by side."""
    xs = []
    for i in range(n32 + n64):
        dt = np.float32 if i < n32 else np.float64
        xs.append((np.sin(np.arange(1 << 18 if i < n32 else 1 << 17) * 1e-3 * (i + 1)) + 1e-2 * i).astype(dt))
    refs = [szref.compress(x, 1e-3, "rel", 128) for x in xs]
    dev = [torch.from_numpy(x).cuda() for x in xs]
    batches = [szx.compress_batch(dev, 1e-3, "rel", 128) for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for use in range(2):
        for b, s in zip(batches, streams):
            if wgs:
                b.set_geometry(wgs)
            b.run(s)
        torch.cuda.synchronize()
        for b in batches:
            for i, ref in enumerate(refs):
                m = int(b.sizes[i].cpu().view(torch.int64))
                assert m == ref.size and np.array_equal(b.outs[i][:m].cpu().numpy(), ref), (i, use)


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("block", [128, 256, 512, 1024])
def test_full_rings_follow_partly_filled_ones(block, dtype):
    """Rings of the persistent encoder that fill up behind a pending tile of few
    bytes, and the other way round: runs of smooth blocks between runs that are
    stored whole (a NaN in every block, or no bound), the runs some fractions of a
    tile and some tiles long, on eight and nine workgroups and on the default
    number."""
    dt = torch.float32 if dtype == "float32" else torch.float64
    n = 2_200_003
    r = np.random.default_rng(block)
    nblk = -(-n // block)
    tile = max(8, 32768 // (block * (4 if dtype == "float32" else 8)))
    raw = np.zeros(nblk, bool)
    at = 0
    while at < nblk:
        smooth, full = (int(r.integers(1, 4 * tile)) for _ in range(2))
        raw[at + smooth: at + smooth + full] = True
        at += smooth + full
    x = field("smooth", n, dtype, block)
    first = np.flatnonzero(raw) * block
    x[np.minimum(first + r.integers(0, block, first.size), n - 1)] = np.nan
    for eb in (1e-3, 0.0):
        ref = szref.compress(x, eb, "rel", block)
        cls = szx.size_class(x.nbytes)
        for wgs in (8, 9, 0):
            try:
                szx.set_geometry(dt, cls, wgs)
                out, size = gpu_compress(x, eb, "rel", block)
            finally:
                szx.set_geometry(dt, cls, 0)
            assert size == ref.size and np.array_equal(out[:size].cpu().numpy(), ref), (eb, wgs)
