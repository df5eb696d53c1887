"""The median's passes after pass 0: their workgroups agree on whether to run,
whichever of them ends first."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# above 1448 particles (2^20 pairs) the passes run in 64 to 256 workgroups
@pytest.mark.parametrize("N,d", [(1449, 30), (4100, 40), (16384, 30)])
def test_the_last_pass_leaves_the_word_its_workgroups_branch_on(ctx, N, d):
    import paper_2310_01775_amd as S
    print("case", N, d, flush=True)
    th = S.soa(np.random.default_rng(N + d).standard_normal((N, d)))
    ws = torch.zeros(S.Context.svgd_workspace_bytes(N, d), dtype=torch.uint8, device="cuda")
    h = torch.zeros(1, device="cuda")
    first = None
    for _ in range(20):  # one workspace: each select finds the state the one before left
        ctx.svgd_bandwidth(th, h_out=h, workspace=ws)
        torch.cuda.synchronize()
        first = h.clone() if first is None else first
        assert torch.equal(h, first)
    # the select state holds lo, hi, the median's rank among all pairs, mode: no
    # distance, histogram count or candidate of these sizes equals that rank
    words = ws[: ws.numel() // 4 * 4].view(torch.int32)
    at = (words == (N * (N - 1) // 2 + 1) // 2).nonzero().flatten()
    assert at.numel() == 1
    assert words[at + 1].item() == 1  # the passes were wanted, and nothing in them took that back
