"""The decoder's waves at the edges of their rows and stages, bit for bit
against the oracle: strings of every length, codes that carry leading bytes
across lanes, rows of constant, coded and raw blocks side by side, stages filled
to their end, a short last block, every block size."""
import numpy as np
import pytest

from gpu_util import gpu_decompress, same_bits
from oracle import szref
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
