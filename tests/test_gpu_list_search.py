"""Lists around the sizes where finding a work unit's tensor takes another round of
64 entries (64, 4096), empty tensors among them, with fewer workers than units so that
a worker's next unit lies many tensors on: both step kernels against the oracle, bitwise."""
import numpy as np
import pytest

import oracle
import paper_2608_11919_amd as lt
from gpu_helpers import HYPER, State, assert_state_equal, gpu_step, oracle_step, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("workgroups", [0, 3])
@pytest.mark.parametrize("K", [1, 2, 63, 64, 65, 129, 4095, 4096, 4097])
def test_tensor_lists_of_every_search_depth(K, workgroups):
    rng = np.random.default_rng(K)
    sizes = [int(n) for n in rng.choice([0, 1, 65, 200, 2049, 4100], size=K)]
    sizes[rng.integers(K)] = 9000
    B = 64
    w = [(rng.standard_normal(n) * 0.02).astype(np.float32) for n in sizes]
    g = [(rng.standard_normal(n) * 1e-3).astype(np.float32) for n in sizes]
    ref = State.zero_host(w, B)
    dev = ref.to_dev()
    w32, m32, v32 = [x.copy() for x in w], [np.zeros_like(x) for x in w], [np.zeros_like(x) for x in w]
    d32 = [[to_dev(x) for x in xs] for xs in (w32, m32, v32)]
    gd = [to_dev(x) for x in g]
    lt.lt_set_max_workgroups(workgroups)
    try:
        gpu_step(dev, gd, B, 1)
        lt.lt_adamw_fp32_step(d32[0], gd, d32[1], d32[2], step=1, **HYPER)
    finally:
        lt.lt_set_max_workgroups(0)
    oracle_step(ref, g, B, 1)
    assert_state_equal(dev.to_host(), ref, f"K={K}")
    for k in range(K):
        oracle.adamw_fp32_step(w32[k], g[k], m32[k], v32[k], step=1, **HYPER)
        for a, b in zip(d32, (w32, m32, v32)):
            assert to_host(a[k]).tobytes() == b[k].tobytes(), k
