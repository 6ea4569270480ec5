"""The norm's finish counts its workgroups in a workspace word, and the last one writes S and
the status.  With the word overwritten (by more than there are workgroups) the call still
gives this call's S and status, never those an earlier call left, and so do the next ones."""
import pytest
import torch

import paper_2608_11919_amd as lt
from gpu_helpers import DEV

pytestmark = pytest.mark.gpu

COUNT_AT = 8  # bytes: the word behind the workspace's tag


# One workgroup and several of the wave finish, and the workgroup finish (a tensor of more
# than 4096 chunks).
@pytest.mark.parametrize("sizes", [[5000], [5000] * 4, [3000] * 37,
                                   [(4096 + 1) * 8192] + [64] * 9])
@pytest.mark.parametrize("count", [1000, 0xFFFFFFFF])
def test_overwritten_count(sizes, count):
    gen = torch.Generator(device=DEV).manual_seed(2)
    g = [(torch.randn(n, device=DEV, generator=gen) * 1e-3).bfloat16() for n in sizes]
    S = torch.zeros(1, dtype=torch.float64, device=DEV)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    ws = torch.empty(lt.lt_grad_sqnorm_workspace_bytes(sizes), dtype=torch.uint8, device=DEV)
    lt.lt_grad_sqnorm(g, S, status, workspace=ws)
    want = S.item()
    assert want > 0 and status.item() == lt.LT_STATUS_OK
    word = ws[COUNT_AT:COUNT_AT + 4].view(torch.int32)
    assert word.item() == 0  # every launch leaves it ready for the next
    for k in range(3):
        if k == 0:
            word.fill_(count - (1 << 32) if count >> 31 else count)
        for t in g:
            t.neg_()
        S.fill_(-1.0)
        status.fill_(7)
        lt.lt_grad_sqnorm(g, S, status, workspace=ws)
        assert status.item() == lt.LT_STATUS_OK and S.item() == want and word.item() == 0
    g[-1].fill_(float("inf"))
    word.fill_(1000)
    lt.lt_grad_sqnorm(g, S, status, workspace=ws)
    assert status.item() == lt.LT_STATUS_NONFINITE and word.item() == 0
    lt.lt_workspace_release(ws)
