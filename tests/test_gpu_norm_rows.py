"""The fp32 chunk sums load 16 consecutive bytes per lane and exchange them between
neighbouring lanes: sizes around the 16-byte words, granules, half rows, rows and chunks,
bitwise against the oracle, with values whose sum depends on every addition's order."""
import numpy as np
import pytest

import oracle
from golden_io import f32_to_bf16_bits
from gpu_helpers import gpu_norm_and_coef, to_dev, to_host

pytestmark = pytest.mark.gpu

SIZES = [1, 3, 4, 5, 7, 8, 9, 255, 256, 257, 259, 260, 261, 511, 512, 513, 515, 516, 2047, 2048,
         2049, 2303, 2304, 2308, 8187, 8191, 8192, 8193, 8196, 16383, 16384, 16385, 3 * 8192 + 300]


@pytest.mark.parametrize("as_bf16", [False, True])
def test_sizes_at_the_edges_of_words_rows_and_chunks(as_bf16):
    rng = np.random.default_rng(11)
    host = [(rng.standard_t(2, size=n) * 10.0 ** rng.uniform(-4, 2, size=n)).astype(np.float32)
            for n in SIZES]
    if as_bf16:
        host = [f32_to_bf16_bits(x) for x in host]
    sk, S, status, _, _ = gpu_norm_and_coef([to_dev(x) for x in host], 1.0)
    want_k, want, want_status = oracle.grad_sqnorm(host)
    for n, a, b in zip(SIZES, to_host(sk), want_k):
        assert float(a).hex() == float(b).hex(), n
    assert to_host(S)[0].hex() == float(want).hex() and int(to_host(status)[0]) == want_status
