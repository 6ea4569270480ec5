"""A skipped step's bf16 copies are refreshed by the step kernel itself: one block size per
kernel and geometry, both maps, and the fp32-state step.  Weights and states stay as they
were, copies hold the rounded weights, and a tensor without a copy is left alone."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_11919_amd as lt
from gpu_helpers import DEV, HYPER, State, assert_state_equal, gpu_norm_and_coef, to_dev, to_host

pytestmark = pytest.mark.gpu

SIZES = [1, 7, 8, 513, 2048, 70001, 12345, 0, 131072 + 5]


def _inputs(rng):
    w = [(rng.standard_normal(n) * 0.02).astype(np.float32) for n in SIZES]
    g = [(rng.standard_normal(n) * 1e-3).astype(np.float32) for n in SIZES]
    g[4][5] = np.nan
    out = [torch.full((n,), 3.0, dtype=torch.bfloat16, device=DEV) if k != 5 else None
           for k, n in enumerate(SIZES)]
    return w, [to_dev(x) for x in g], out


def _check_copies(out, w):
    for k, o in enumerate(out):
        if o is not None:
            assert np.array_equal(to_host(o), oracle.round_bf16(w[k])), k


@pytest.mark.parametrize("code_map", [lt.LT_MAP_LINEAR, lt.LT_MAP_DYNAMIC])
@pytest.mark.parametrize("B", [64, 512, 1024, 2048, 4096, 8192, 192, 768, 1536, 3072, 7168, 12288,
                               65536])
def test_8bit_step(B, code_map):
    w, g, out = _inputs(np.random.default_rng(B))
    base = State.zero_host(w, B)
    dev = base.to_dev()
    _, _, status, _, coef = gpu_norm_and_coef(g, 1.0)
    lt.lt_hybrid8bit_adamw_step(dev.w, g, dev.mq, dev.ma, dev.vq, dev.va, B, step=2, coef=coef,
                                status=status, params_bf16=out, code_map=code_map, **HYPER)
    assert_state_equal(dev.to_host(), base, f"B={B}")
    _check_copies(out, w)


def test_fp32_state_step():
    w, g, out = _inputs(np.random.default_rng(1))
    dw = [to_dev(x) for x in w]
    m, v = [torch.zeros_like(x) for x in dw], [torch.zeros_like(x) for x in dw]
    _, _, status, _, coef = gpu_norm_and_coef(g, 1.0)
    lt.lt_adamw_fp32_step(dw, g, m, v, step=2, coef=coef, status=status, params_bf16=out, **HYPER)
    for k in range(len(SIZES)):
        assert np.array_equal(to_host(dw[k]), w[k]) and not to_host(m[k]).any()
    _check_copies(out, w)
