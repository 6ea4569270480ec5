"""Block sizes at the edges of the geometries of k_adamw8_any (waves per block, granules
per lane, blocks per unit) and of the kernel above it: one clipped step of ragged tensors
(shorter than a block, units with a partial last block, row and granule) against the
oracle, bitwise, with scales of every kind."""
import numpy as np
import pytest

import oracle
import paper_2608_11919_amd as lt
from golden_io import f32_to_bf16_bits
from gpu_helpers import HYPER, State, assert_state_equal, gpu_norm_and_coef, to_dev

pytestmark = pytest.mark.gpu

BLOCKS = [192, 320, 448, 576, 704, 832, 960, 1088, 1984, 2112, 4032, 4160, 6144, 6208, 8128, 8256,
          16384, 16448]


@pytest.mark.parametrize("B", BLOCKS)
@pytest.mark.parametrize("code_map", [lt.LT_MAP_LINEAR, lt.LT_MAP_DYNAMIC])
def test_block_sizes_at_the_edges_of_each_geometry(B, code_map):
    rng = np.random.default_rng(B + code_map)
    per = max(1, 1024 // B)
    sizes = [1, B - 9, B, B + 1, per * B, per * B + 8, 2 * per * B - 3, 7 * B + 515, 40 * B + 77]
    ref = State.zero_host([(rng.standard_normal(n) * 0.02).astype(np.float32) for n in sizes], B)
    odd = np.array([0.0, np.inf, -1e-3, np.nan, 1e-42, 3e38, 1e-30], np.float32)
    for k, n in enumerate(sizes):
        ref.mq[k][:] = rng.integers(-128, 128, size=n)
        ref.vq[k][:] = rng.integers(0, 256, size=n)
        for a, scale in ((ref.ma[k], 1e-3), (ref.va[k], 1e-6)):
            a[:] = rng.uniform(0.1, 5.0, size=a.size) * scale
            bad = rng.random(a.size) < 0.15
            a[bad] = rng.choice(odd, size=int(bad.sum()))
    g = [f32_to_bf16_bits((rng.standard_t(3, size=n) * 1e-3).astype(np.float32)) for n in sizes]
    dev = ref.to_dev()
    gd = [to_dev(x) for x in g]
    _, S, status, _, coef = gpu_norm_and_coef(gd, 0.05)
    lt.lt_hybrid8bit_adamw_step(dev.w, gd, dev.mq, dev.ma, dev.vq, dev.va, B, step=3, coef=coef,
                                status=status, code_map=code_map, **HYPER)
    _, rS, _ = oracle.grad_sqnorm(g)
    _, rc = oracle.clip_coef(rS, 0.05)
    omap = oracle.MAP_DYNAMIC if code_map == lt.LT_MAP_DYNAMIC else oracle.MAP_LINEAR
    oracle.hybrid8bit_adamw_step(ref.w, g, ref.mq, ref.ma, ref.vq, ref.va, B, step=3,
                                 coef=float(rc), code_map=omap, n_threads=8, **HYPER)
    assert_state_equal(dev.to_host(), ref, f"B={B}")
