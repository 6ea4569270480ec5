"""The fp32-state step works in words of four elements, rows of 256 and spans of 1024 per
wave: sizes around each, with a bf16 copy, against the oracle, bitwise."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_11919_amd as lt
from golden_io import f32_to_bf16_bits
from gpu_helpers import DEV, HYPER, gpu_norm_and_coef, to_dev, to_host

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 3, 4, 5, 7, 8, 9, 253, 255, 256, 257, 260, 767, 769, 1020, 1021, 1023, 1024, 1025,
         1027, 1280, 2047, 2048, 2050, 70003]


@pytest.mark.parametrize("as_bf16", [False, True])
def test_sizes_at_the_edges_of_words_rows_and_spans(as_bf16):
    rng = np.random.default_rng(3 + as_bf16)
    w = [(rng.standard_normal(n) * 0.02).astype(np.float32) for n in SIZES]
    m = [(rng.standard_normal(n) * 3e-4).astype(np.float32) for n in SIZES]
    v = [(rng.standard_normal(n) ** 2 * 1e-6).astype(np.float32) for n in SIZES]
    for x in v:
        x[rng.random(x.size) < 0.01] = 1e-38  # takes the scaled square root
    g = [(rng.standard_t(3, size=n) * 1e-3).astype(np.float32) for n in SIZES]
    if as_bf16:
        g = [f32_to_bf16_bits(x) for x in g]
    dw, dm, dv, dg = [[to_dev(x) for x in lst] for lst in (w, m, v, g)]
    out = [torch.zeros(n, dtype=torch.bfloat16, device=DEV) for n in SIZES]
    _, _, status, _, coef = gpu_norm_and_coef(dg, 0.05)
    lt.lt_adamw_fp32_step(dw, dg, dm, dv, step=3, coef=coef, status=status, params_bf16=out,
                          **HYPER)
    _, S, _ = oracle.grad_sqnorm(g)
    _, c = oracle.clip_coef(S, 0.05)
    for k, n in enumerate(SIZES):
        oracle.adamw_fp32_step(w[k], g[k], m[k], v[k], step=3, coef=float(c), **HYPER)
        for a, b in ((dw[k], w[k]), (dm[k], m[k]), (dv[k], v[k])):
            assert to_host(a).tobytes() == b.tobytes(), n
        assert np.array_equal(to_host(out[k]), oracle.round_bf16(w[k])), n
