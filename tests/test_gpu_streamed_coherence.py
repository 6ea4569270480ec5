"""The streamed step over pinned memory of each kind: the default and the coherent kind,
which the copy kernel takes, and non-coherent memory, which takes copy commands
(test_rules.py holds the rule).  Bitwise the resident step either way, over two steps (the
second reads what the first wrote back)."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2608_11919_amd as lt
from gpu_helpers import DEV, HYPER

pytestmark = pytest.mark.gpu

B = 256
SIZES = [70000, 4096, 33, 5000]
NON_COHERENT, COHERENT, DEFAULT = 0x80000000, 0x40000000, 0


class Pinned:
    """CPU tensors over one hipHostMalloc allocation made with the given flags."""

    def __init__(self, hip, nbytes, flags):
        self.hip, self.p, self.used = hip, ctypes.c_void_p(), 0
        assert hip.hipHostMalloc(ctypes.byref(self.p), ctypes.c_size_t(nbytes),
                                 ctypes.c_uint(flags)) == 0
        self.raw = np.frombuffer((ctypes.c_uint8 * nbytes).from_address(self.p.value), np.uint8)

    def copy(self, t):
        n = t.numel() * t.element_size()
        out = torch.from_numpy(self.raw[self.used:self.used + n]).view(t.dtype)
        self.used += -(-n // 256) * 256
        out.copy_(t)
        return out

    def free(self):
        assert self.hip.hipHostFree(self.p) == 0


@pytest.mark.parametrize("flags", [DEFAULT, COHERENT, NON_COHERENT])
def test_streamed_step_over_pinned_memory_of_each_kind(flags):
    hip = ctypes.CDLL("libamdhip64.so")
    gen = torch.Generator().manual_seed(9)
    nb = [-(-n // B) for n in SIZES]
    lists = ([torch.randn(n, generator=gen) * 0.02 for n in SIZES],
             [(torch.randn(n, generator=gen) * 1e-3).bfloat16() for n in SIZES],
             [torch.randint(-127, 128, (n,), generator=gen).to(torch.int8) for n in SIZES],
             [torch.rand(n, generator=gen) * 1e-3 for n in nb],
             [torch.randint(0, 256, (n,), generator=gen).to(torch.uint8) for n in SIZES],
             [torch.rand(n, generator=gen) * 1e-6 for n in nb])
    w, g, mq, ma, vq, va = 0, 1, 2, 3, 4, 5
    order = (w, g, mq, ma, vq, va)
    pinned = Pinned(hip, 4 << 20, flags)
    host = [[pinned.copy(t) for t in lists[i]] for i in order]
    dev = [[t.to(DEV) for t in lists[i]] for i in order]
    scalars = lambda: [torch.zeros(1, dtype=dt, device=DEV) for dt in
                       (torch.float64, torch.float32, torch.int32)]
    S, coef, status = scalars()
    S2, coef2, status2 = scalars()
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    for step in (3, 4):
        lt.lt_streamed_hybrid8bit_adamw_step(
            *host, [0, 2, 4], B, step=step, max_norm=1.0, ring_slots=2, sq_total=S2, coef=coef2,
            status=status2, compute_stream=streams[0], h2d_stream=streams[1],
            d2h_stream=streams[2], **HYPER)
        assert lt.lt_read_status(status2, streams[0]) == lt.LT_STATUS_OK
    for step in (3, 4):
        lt.lt_grad_sqnorm(dev[g], S, status)
        lt.lt_clip_coef(S, 1.0, coef)
        lt.lt_hybrid8bit_adamw_step(*dev, B, step=step, coef=coef, status=status, **HYPER)
    assert S2.item() == S.item() and coef2.item() == coef.item()
    for i in order:
        for k, (x, y) in enumerate(zip(host[i], dev[i])):
            assert np.array_equal(x.view(torch.uint8).numpy(),
                                  y.cpu().view(torch.uint8).numpy()), (i, k)
    host = None
    pinned.free()
