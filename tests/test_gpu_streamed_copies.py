"""The streamed step's copies: pinned arrays small enough for the copy kernel (tails of
every length, unit edges, more arrays in a layer than one launch takes), arrays at and
above the size that takes a copy command, pinned arrays off 16-byte alignment, pageable
arrays, and a pinned array that ends with its allocation: bitwise the resident step."""
import numpy as np
import pytest
import torch

import paper_2608_11919_amd as lt
from gpu_helpers import DEV, HYPER

pytestmark = pytest.mark.gpu

B = 256
SIZES = [[1, 2, 3, 5, 15, 16, 17, 255, 4095, 4096, 4097, 8191, 16384, 16385, 0],
         [(1 << 20) - 4, 1 << 20, (1 << 20) + 3, (1 << 22) + 1, 7]]


def _host(t, how):
    if how == "pageable":
        return t.clone()
    skip = 0 if how == "pinned" else 3
    out = torch.zeros(t.numel() + skip, dtype=t.dtype, pin_memory=True)[skip:]
    out.copy_(t)
    return out


@pytest.mark.parametrize("how", ["pinned", "offset", "pageable"])
@pytest.mark.parametrize("keep", [False, True])
def test_streamed_copies_match_the_resident_step(how, keep):
    gen = torch.Generator().manual_seed(5)
    sizes = [n for layer in SIZES for n in layer]
    first = [0, len(SIZES[0]), len(sizes)]
    nb = [-(-n // B) for n in sizes]
    w = [torch.randn(n, generator=gen) * 0.02 for n in sizes]
    g = [(torch.randn(n, generator=gen) * 1e-3).bfloat16() for n in sizes]
    mq = [torch.randint(-127, 128, (n,), generator=gen).to(torch.int8) for n in sizes]
    vq = [torch.randint(0, 256, (n,), generator=gen).to(torch.uint8) for n in sizes]
    ma = [torch.rand(n, generator=gen) * 1e-3 for n in nb]
    va = [torch.rand(n, generator=gen) * 1e-6 for n in nb]
    lists = (w, g, mq, ma, vq, va)
    host = [[_host(t, how) for t in ts] for ts in lists]
    dev = [[t.to(DEV) for t in ts] for ts in lists]
    scalars = lambda: [torch.zeros(1, dtype=dt, device=DEV) for dt in
                       (torch.float64, torch.float32, torch.int32)]
    S, coef, status = scalars()
    lt.lt_grad_sqnorm(dev[1], S, status)
    lt.lt_clip_coef(S, 1.0, coef)
    lt.lt_hybrid8bit_adamw_step(*dev, B, step=3, coef=coef, status=status, **HYPER)
    S2, coef2, status2 = scalars()
    streams = [torch.cuda.Stream() for _ in range(3)]
    torch.cuda.synchronize()
    lt.lt_streamed_hybrid8bit_adamw_step(
        *host, first, B, step=3, max_norm=1.0, ring_slots=2, sq_total=S2, coef=coef2,
        status=status2, compute_stream=streams[0], h2d_stream=streams[1], d2h_stream=streams[2],
        keep_grads=keep, **HYPER)
    assert lt.lt_read_status(status2, streams[0]) == lt.LT_STATUS_OK
    assert S2.item() == S.item() and coef2.item() == coef.item()
    for a, b, before in zip(host, dev, lists):
        for k, (x, y) in enumerate(zip(a, b)):
            assert np.array_equal(x.view(torch.uint8).numpy(), y.cpu().view(torch.uint8).numpy()), k
