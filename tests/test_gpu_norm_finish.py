"""The norm's finish: the last workgroup of the per-tensor combine adds the S_k up in list
order.  Lists around its batch (1024 sums) and run (16 sums) sizes, bitwise against the
oracle, with the workspace used again by the next call (its count has to be back at zero)
and without a workspace, whose descriptors travel in kernel arguments (440 words a launch:
lists of up to 143 tensors need one launch, longer ones two)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_11919_amd as lt
from gpu_helpers import DEV, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [0, 1, 2, 15, 16, 17, 143, 144, 145, 146, 147, 1023, 1024, 1025,
                                   2049])
def test_list_order_total(count):
    rng = np.random.default_rng(count)
    host = [(rng.standard_normal(n) * 10.0 ** rng.integers(-6, 3)).astype(np.float32)
            for n in rng.integers(1, 200, size=count)]
    if count:
        host[count // 2] = (rng.standard_normal(3 * 8192 + 1) * 1e-2).astype(np.float32)
    want_k, want, status = oracle.grad_sqnorm(host) if count else (np.zeros(0), 0.0, 0)
    grads = [to_dev(g) for g in host]
    ws = torch.empty(max(lt.lt_grad_sqnorm_workspace_bytes([g.numel() for g in grads]), 256),
                     dtype=torch.uint8, device=DEV)
    for call in range(4):  # twice on one workspace, twice without
        sk = torch.full((max(count, 1),), -1.0, dtype=torch.float64, device=DEV)
        S = torch.full((1,), -1.0, dtype=torch.float64, device=DEV)
        st = torch.full((1,), -7, dtype=torch.int32, device=DEV)
        if call < 2:
            lt.lt_grad_sqnorm(grads, S, st, sq_per_tensor=sk, workspace=ws)
        else:
            lt.lt_grad_sqnorm_noalloc(grads, S, st, sq_per_tensor=sk)
        assert to_host(S)[0].hex() == float(want).hex(), call
        assert int(to_host(st)[0]) == status
        assert to_host(sk)[:count].tobytes() == np.asarray(want_k).tobytes(), call


def test_nonfinite_sum_in_the_padding_run():
    host = [np.full(5, 1e-3, np.float32) for _ in range(18)]
    host[17][4] = np.nan
    S = torch.zeros(1, dtype=torch.float64, device=DEV)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    lt.lt_grad_sqnorm([to_dev(g) for g in host], S, st)
    assert np.isnan(to_host(S)[0]) and int(to_host(st)[0]) == lt.LT_STATUS_NONFINITE


def fixed_order(partials):
    """One tensor's chunk sums in the stated order: accumulator c mod 256 in ascending c,
    then halving from 128."""
    acc = np.zeros(256)
    for at in range(0, partials.size, 256):
        part = partials[at:at + 256]
        acc[:part.size] += part
    while acc.size > 1:
        acc = acc[:acc.size // 2] + acc[acc.size // 2:]
    return acc[0]


# Both sides of every line between the finish's geometries, with a last workgroup that is
# not full, empty tensors and rounds of loads that end in mid-tensor.
@pytest.mark.parametrize("count", [1, 7, 64, 65, 67])
@pytest.mark.parametrize("longest", [3, 512, 513, 1024, 1025, 2049, 4096, 4097, 9000])
def test_finish_geometries(count, longest):
    rng = np.random.default_rng(count * 10007 + longest)
    chunks = rng.integers(0, min(longest, 700) + 1, size=count)
    chunks[rng.integers(0, count)] = longest
    part = rng.standard_normal(int(chunks.sum())) ** 2 * 10.0 ** rng.integers(-6, 3)
    ends = np.cumsum(chunks)
    want_k = np.array([fixed_order(part[e - c:e]) for c, e in zip(chunks, ends)])
    want = 0.0
    for x in want_k:
        want += x
    numels = [max(int(c) * 8192 - 5, 0) for c in chunks]
    dev = to_dev(part)
    for _ in range(2):
        sk = torch.full((count,), -1.0, dtype=torch.float64, device=DEV)
        S = torch.full((1,), -1.0, dtype=torch.float64, device=DEV)
        st = torch.full((1,), -7, dtype=torch.int32, device=DEV)
        lt.lt_grad_sqnorm_finish(numels, dev, S, st, sk)
        assert to_host(sk).tobytes() == want_k.tobytes()
        assert to_host(S)[0].hex() == float(want).hex() and int(to_host(st)[0]) == 0
