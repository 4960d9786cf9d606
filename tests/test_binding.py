"""The binding's refusals do not depend on which buffers the caller hands in."""
import pytest
import torch

from paper_2201_13020_amd import szx

HEAD = dict(dtype=torch.float32, dims=(100,), block=128)


@pytest.mark.parametrize("given", [False, True])
def test_host_streams_are_refused(given):
    data = torch.zeros(600, dtype=torch.uint8)
    kw = dict(out=torch.zeros(100), status=torch.zeros(1, dtype=torch.uint32), ws=torch.zeros(1 << 16, dtype=torch.uint8))
    with pytest.raises(ValueError):
        szx.decompress(data, 600, HEAD, **(kw if given else {}))


@pytest.mark.gpu
@pytest.mark.parametrize("given", [False, True])
def test_errors_are_the_same_with_and_without_buffers(given):
    x = torch.zeros(100, device="cuda")
    ws = torch.zeros(1 << 16, dtype=torch.uint8, device="cuda")
    out = torch.zeros(4096, dtype=torch.uint8, device="cuda")
    kw = dict(out=out, out_size=torch.zeros(1, dtype=torch.uint64, device="cuda"), ws=ws) if given else {}
    with pytest.raises(szx.SzError) as e:
        szx.compress(x, -1.0, "abs", 128, **kw)
    assert e.value.code == 1 and "invalid parameters" in str(e.value)
    if given:
        with pytest.raises(szx.SzError) as e:
            szx.compress(x, 1e-3, "rel", 128, out=out[:64], out_size=kw["out_size"], ws=ws)
        assert e.value.code == 2
