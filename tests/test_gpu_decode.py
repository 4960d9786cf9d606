"""The decoder's waves at the edges of their rows and stages, bit for bit
against the oracle: strings of every length, codes that carry leading bytes
across lanes, rows of constant, coded and raw blocks side by side, stages filled
to their end, a short last block, every block size."""
import numpy as np
import pytest
import torch

from gpu_util import gpu_decompress, same_bits
from oracle import szref
from paper_2201_13020_amd import szx
from test_gpu_encode import field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("block", [8, 16, 32, 64, 128, 256, 512, 1024])
@pytest.mark.parametrize("kind", ["smooth", "noise", "mixed"])
def test_values_equal_the_oracle(kind, block, dtype):
    for n in (1, 15, 4097, 8191, 100_003):
        x = field(kind, n, dtype, block)
        for eb, mode in ((1e-1, "rel"), (1e-4, "rel"), (0.0, "abs")):
            ref = szref.compress(x, eb, mode, block)
            y, status = gpu_decompress(ref)
            assert status == 0 and same_bits(y, szref.decompress(ref)), (n, eb)


@pytest.mark.parametrize("tiles", [255, 256, 257])
@pytest.mark.parametrize("dtype", ["float32", "float64"])
def test_index_direct_and_chained(dtype, tiles):
    """The index at the line between its two forms (256 tiles of 1024 blocks),
    from workspaces of arbitrary bytes that a call of the other form used last;
    then a stream whose mid-byte total or state bits disagree."""
    ref = {}
    for n in (tiles * 8192 - 3, 30_001 if tiles > 256 else 260 * 8192 + 1):
        s = szref.compress(field("mixed", n, dtype, 8), 1e-2, "rel", 8)
        ref[n] = (s, szref.decompress(s), szx.inspect(s[:96].tobytes()))
    ws = torch.full((max(szx.workspace_size(i["dtype"], i["dims"], 0.0, "rel", 8) for _, _, i in ref.values()),), 0xA5,
                    dtype=torch.uint8, device="cuda")
    for n in list(ref) * 2:
        s, want, info = ref[n]
        y, st = szx.decompress(torch.from_numpy(s).cuda(), s.size, info, ws=ws)
        torch.cuda.synchronize()
        assert int(st.cpu().view(torch.int32)) == 0 and same_bits(y.cpu().numpy(), want), n
    s, _, info = ref[tiles * 8192 - 3]
    for at in (88, 96 + 5):  # the header's mid-byte total, a state byte
        bad = s.copy()
        bad[at] ^= 1
        _, st = szx.decompress(torch.from_numpy(bad).cuda(), s.size, info, ws=ws)
        torch.cuda.synchronize()
        assert int(st.cpu().view(torch.int32)) == 3, at


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("block", [8, 64, 128, 1024])
def test_one_launch_and_two_meet(block, dtype):
    """Sizes on both sides of where a single call goes from one launch to two
    (1024 blocks, 131072 values), and what a flipped byte of every section does
    to the status there."""
    line = min(1024 * block, 131072)
    for n in (line - 1, line, line + 1):
        s = szref.compress(field("mixed", n, dtype, block), 1e-2, "rel", block)
        y, st = gpu_decompress(s)
        assert st == 0 and same_bits(y, szref.decompress(s)), n
        for at in (0, 80, 88, 97):  # magic, block count, mid-byte total, a state byte
            bad = s.copy()
            bad[at] ^= 1
            assert gpu_decompress(bad, szx.inspect(s[:96].tobytes()))[1] == 3, (n, at)


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("block", [8, 16, 32, 64, 128, 256, 512, 1024])
def test_rows_of_raw_blocks(block, dtype):
    """Rows that hold raw blocks alone, which are copied as they lie: all of a
    field's, runs of them between coded and constant blocks (their stored bytes
    start at every alignment), and a short last row or block."""
    r = np.random.default_rng(block)
    for n in (1, 7, 4096, 8191, 40_003, 140_001):
        nblk = -(-n // block)
        for runs in (1, 3, 40):  # blocks a run
            sort = np.repeat(r.integers(0, 4, nblk // runs + 1), runs)[:nblk]
            x = np.cumsum(r.standard_normal(n)) * 1e-2
            x = np.where(np.repeat(sort == 0, block)[:n], 1.0, x).astype(dtype)
            first = np.flatnonzero(sort >= 2) * block
            x[np.minimum(first + r.integers(0, block, first.size), n - 1)] = np.nan
            if runs == 3:
                x[::block] = np.inf
            ref = szref.compress(x, 1e-3, "abs", block)
            y, status = gpu_decompress(ref)
            assert status == 0 and same_bits(y, szref.decompress(ref)), (n, runs)


@pytest.mark.parametrize("dtype,block", [("float32", 128), ("float64", 128), ("float64", 1024)])
def test_raw_blocks_decode_at_half_the_copy_rate(dtype, block):
    """A field of raw blocks, whose decompression only moves bytes, takes at most
    twice the time of a device copy of as many bytes (160 MB each way; lane by
    lane it took three to five times that)."""
    dt = getattr(torch, dtype)
    x = torch.randn((160 << 20) // torch.finfo(dt).bits * 8, device="cuda").to(dt)
    x[::block] = float("nan")
    out, size = szx.compress(x, 1e-3, "abs", block)
    n = int(size.cpu().view(torch.int64))
    ws = torch.zeros(szx.workspace_size(dt, x.shape, 1e-3, "abs", block), dtype=torch.uint8, device="cuda")
    y, st = torch.empty_like(x), torch.zeros(1, dtype=torch.uint32, device="cuda")
    info = dict(dtype=dt, dims=tuple(x.shape), block=block)
    src, dst = torch.empty_like(x), torch.empty_like(x)

    def median(fn):
        ts = []
        for _ in range(15):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            fn()
            b.record()
            b.synchronize()
            ts.append(a.elapsed_time(b))
        return sorted(ts)[7]
    copy = median(lambda: dst.copy_(src))
    took = median(lambda: szx.decompress(out, n, info, out=y, status=st, ws=ws))
    assert int(st.cpu().view(torch.int32)) == 0 and torch.equal(y.view(torch.uint8), x.view(torch.uint8))
    assert took <= 2.0 * copy, (took, copy)


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("block", [8, 128, 512, 1024])
def test_waves_of_constant_blocks(block, dtype):
    """Runs of 256 constant blocks, which the index pass's waves skip, before,
    between and after others, in one index tile and in several."""
    for nblk, const in ((300, [0]), (700, [1]), (1030, [0, 2, 3]), (2600, [0, 1, 2, 3, 5, 8]), (1024, [0, 1, 2, 3])):
        n = nblk * block - 3
        x = np.random.default_rng(nblk).standard_normal(n)
        for k in const:
            x[k * 256 * block: (k + 1) * 256 * block] = 0.25
        x = x.astype(dtype)
        ref = szref.compress(x, 1e-3, "abs", block)
        y, status = gpu_decompress(ref)
        assert status == 0 and same_bits(y, szref.decompress(ref)), (nblk, const)


def test_direct_index_at_its_largest_sum():
    """262144 raw blocks of 1024 doubles, the most that the direct index takes:
    its totals add up to 2^31 mid bytes. Then a header that states one less."""
    n, block = 1 << 28, 1024
    x = torch.randn(n, device="cuda", dtype=torch.float64)
    x[::block] = float("nan")
    out, size = szx.compress(x, 1e-3, "abs", block)
    m = int(size.cpu().view(torch.int64))
    info = szx.inspect(out[:96].cpu().numpy().tobytes())
    assert int(out[88:96].cpu().view(torch.int64)) == 1 << 31
    y, st = szx.decompress(out, m, info)
    torch.cuda.synchronize()
    assert int(st.cpu().view(torch.int32)) == 0 and torch.equal(y.view(torch.int64), x.view(torch.int64))
    out[88:96] = torch.tensor([(1 << 31) - 1], dtype=torch.int64).view(torch.uint8).cuda()
    _, st = szx.decompress(out, m, info)
    torch.cuda.synchronize()
    assert int(st.cpu().view(torch.int32)) == 3
