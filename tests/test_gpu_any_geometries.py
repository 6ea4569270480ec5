"""Every kernel that takes block sizes that are no power of two, on lists that
rules::any_geom (csrc/rules.h, asked by test_rules.py) gives it: both gradient types, both
code maps, bf16 copies for some of the tensors; ragged tensors with partial last units,
blocks, rows and granules, scales of every kind.  One clipped step against the oracle,
bitwise."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_11919_amd as lt
from golden_io import f32_to_bf16_bits
from gpu_helpers import DEV, HYPER, State, assert_state_equal, gpu_norm_and_coef, to_dev, to_host

pytestmark = pytest.mark.gpu

M = 1 << 20
LINEAR, DYNAMIC = lt.LT_MAP_LINEAR, lt.LT_MAP_DYNAMIC


def _ragged(B, more=()):
    return [1, B - 9, B, B + 1, 2 * B + 8, 7 * B + 515, 12 * B + 77, *more]


# block size, sizes, code maps; the geometry they stand for
CASES = [
    (192, _ragged(192), "ld"),                      # {4, 1, 1}: few blocks
    (1024 - 64, _ragged(960), "ld"),                # {4, 1, 1}
    (192, _ragged(192, [800 * 192 + 13]), "ld"),    # {1, 2, 5}
    (320, _ragged(320, [800 * 320 + 13]), "ld"),    # {1, 2, 3}
    (384, _ragged(384, [800 * 384 + 13]), "ld"),    # {1, 2, 2}
    (640, _ragged(640, [800 * 640 + 13]), "ld"),    # {1, 2, 1}, 640 of 1024 busy
    (704, _ragged(704, [800 * 704 + 13]), "ld"),    # {1, 2, 1}
    (960, _ragged(960, [800 * 960 + 13]), "ld"),    # {1, 2, 1}
    (576, _ragged(576, [12 * M + 13]), "ld"),       # {1, 4, 3}
    (384, _ragged(384, [32 * M + 13]), "l"),        # {1, 4, 5}
    (768, _ragged(768, [32 * M + 13]), "l"),        # {1, 4, 2}
    (1088, _ragged(1088), "ld"), (1984, _ragged(1984), "ld"),    # {4, 1, 1}
    (2112, _ragged(2112), "ld"), (4032, _ragged(4032), "ld"),    # {4, 2, 1}
    (4160, _ragged(4160), "ld"), (6144, _ragged(6144), "ld"),    # {4, 3, 1}
    (6208, _ragged(6208), "ld"), (8128, _ragged(8128), "ld"),    # {8, 2, 1}
    (8256, _ragged(8256), "ld"), (12288, _ragged(12288), "ld"),  # {16, 2, 1}: up to 256 blocks
    (14336, _ragged(14336), "ld"), (16384, _ragged(16384), "ld"),
    (16384, [11000] * 260, "ld"),                   # {16, 2, 1}, more blocks than CUs
    (2112, [1, 700, 2048, 1537] * 3, "ld"),         # generic: no block longer than 2048
    (8128, [1, 700, 2048, 1537] * 3, "ld"),
    (12288, [4096, 33, 2049, 1] * 3, "ld"),         # generic: two goes
    (16384, [8192, 4097, 5, 7001] * 65, "ld"),      # generic: four goes, more blocks than CUs
    (8256, [8256 * 270 + 100], "ld"),               # generic: idle lanes
    (12288, [12288 * 520 + 100], "ld"),             # generic: idle lanes, more blocks
    (16448, _ragged(16448), "ld"),                  # generic: larger blocks
]
PARAMS = [pytest.param(B, s, LINEAR if m == "l" else DYNAMIC, id=f"{B}-{i}-{m}")
          for i, (B, s, maps) in enumerate(CASES) for m in maps]


@pytest.mark.parametrize("as_bf16", [False, True])
@pytest.mark.parametrize("B,sizes,code_map", PARAMS)
def test_geometry(B, sizes, code_map, as_bf16):
    rng = np.random.default_rng(B + 7 * len(sizes) + code_map)
    base = min(max(sizes), M + 1)  # longer tensors repeat their values
    w0 = (rng.standard_normal(base) * 0.02).astype(np.float32)
    g0 = (rng.standard_t(3, size=base) * 1e-3).astype(np.float32)
    m0 = rng.integers(-128 if code_map == DYNAMIC else -127, 128, size=base).astype(np.int8)
    v0 = rng.integers(0, 256, size=base).astype(np.uint8)
    odd = np.array([0.0, np.inf, -1e-3, np.nan, 1e-42, 3e38, 1e-30], np.float32)
    ref = State.zero_host([np.resize(np.roll(w0, k), n) for k, n in enumerate(sizes)], B)
    for k, n in enumerate(sizes):
        ref.mq[k][:] = np.resize(np.roll(m0, 3 * k), n)
        ref.vq[k][:] = np.resize(np.roll(v0, 5 * k), n)
        for a, scale in ((ref.ma[k], 1e-3), (ref.va[k], 1e-6)):
            a[:] = rng.uniform(0.1, 5.0, size=a.size) * scale
            bad = rng.random(a.size) < 0.15
            a[bad] = rng.choice(odd, size=int(bad.sum()))
    g = [np.resize(np.roll(g0, 11 * k), n) for k, n in enumerate(sizes)]
    if as_bf16:
        g = [f32_to_bf16_bits(x) for x in g]
    dev = ref.to_dev()
    gd = [to_dev(x) for x in g]
    copies = [None if k % 3 == 1 else torch.full((n,), 7.0, dtype=torch.bfloat16, device=DEV)
              for k, n in enumerate(sizes)]
    _, S, status, _, coef = gpu_norm_and_coef(gd, 0.05)
    lt.lt_hybrid8bit_adamw_step(dev.w, gd, dev.mq, dev.ma, dev.vq, dev.va, B, step=3, coef=coef,
                                status=status, code_map=code_map, params_bf16=copies, **HYPER)
    _, rS, _ = oracle.grad_sqnorm(g)
    _, rc = oracle.clip_coef(rS, 0.05)
    oracle.hybrid8bit_adamw_step(ref.w, g, ref.mq, ref.ma, ref.vq, ref.va, B, step=3,
                                 coef=float(rc), code_map=oracle.MAP_DYNAMIC
                                 if code_map == DYNAMIC else oracle.MAP_LINEAR, n_threads=8, **HYPER)
    assert_state_equal(dev.to_host(), ref, f"B={B}")
    for k, c in enumerate(copies):
        if c is not None:
            assert np.array_equal(to_host(c), oracle.round_bf16(ref.w[k])), f"copy of tensor {k}"
    # without copies: the kernels that write none
    if max(sizes) <= M:
        again = State(*[[x.copy() for x in ts] for ts in (ref.w, ref.mq, ref.ma, ref.vq, ref.va)])
        lt.lt_hybrid8bit_adamw_step(dev.w, gd, dev.mq, dev.ma, dev.vq, dev.va, B, step=4,
                                    coef=coef, status=status, code_map=code_map, **HYPER)
        oracle.hybrid8bit_adamw_step(again.w, g, again.mq, again.ma, again.vq, again.va, B, step=4,
                                     coef=float(rc), code_map=oracle.MAP_DYNAMIC
                                     if code_map == DYNAMIC else oracle.MAP_LINEAR, n_threads=8,
                                     **HYPER)
        assert_state_equal(dev.to_host(), again, f"B={B}, second step")
