"""The median's passes after pass 0: their workgroups agree on whether to run,
whichever of them ends first; the widest particles; and where the select's
state may lie."""
import math

import numpy as np
import pytest
import torch

import workloads as W

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


# FP32 products of 14 and 16 steps, in blocks of 64 and of 256 rows
@pytest.mark.parametrize("N,d", [(1449, 49), (1500, 56), (2003, 57), (4097, 55), (4200, 64)])
def test_bandwidth_of_wide_particles_is_the_order_statistic(ctx, N, d):
    import paper_2310_01775_amd as S
    print("case", N, d, flush=True)
    th = np.random.default_rng(N + d).standard_normal((N, d)).astype(np.float32).astype(np.float64)
    h = torch.zeros(1, device="cuda")
    ctx.svgd_bandwidth(S.soa(th), h_out=h)
    torch.cuda.synchronize()
    m2 = float(h.item()) * math.log(N)
    q = (th * th).sum(1)
    D = (q[:, None] + q[None, :] - 2.0 * (th @ th.T))[np.triu_indices(N, 1)]
    k = (D.size + 1) // 2
    # 64 FP32 products and sums over terms of up to |xi|^2 + |xj|^2 <= 4 D or so
    tol = 256 * 2.0 ** -24
    assert (D < m2 * (1 - tol)).sum() < k <= (D <= m2 * (1 + tol)).sum()


# the finishing workgroup, the passes over the matrix cores' distances and over
# direct ones (structured); every array argument is 4-byte aligned, no more
@pytest.mark.parametrize("N", [700, 1500])
def test_a_workspace_may_start_at_any_four_bytes(ctx, N):
    import paper_2310_01775_amd as S
    d = 18
    rng = np.random.default_rng(N)
    th, g = S.soa(rng.standard_normal((N, d))), S.soa(rng.standard_normal((N, d)))
    need = S.Context.svgd_workspace_bytes(N, d)
    kern = S.struct_kernel(S.KERNEL_PUSH, 3)

    def steps(ws):
        h, h2 = torch.zeros(1, device="cuda"), torch.zeros(2, device="cuda")
        out = [ctx.svgd_step(th, g, h_out=h, workspace=ws), h,
               ctx.svgd_step_structured(th, g, kern, h_out=h2, workspace=ws), h2,
               ctx.svgd_step_bf16(th, g, workspace=ws)]
        torch.cuda.synchronize()
        return out

    ref = steps(torch.zeros(need, dtype=torch.uint8, device="cuda"))
    for shift in (4, 8, 12):
        print("case", N, shift, flush=True)
        buf = torch.zeros(need + 16, dtype=torch.uint8, device="cuda")
        buf[need + shift:] = 77
        for a, b in zip(steps(buf[shift:shift + need]), ref):
            assert torch.equal(a, b)
        assert (buf[:shift] == 0).all() and (buf[need + shift:] == 77).all()


def test_a_solve_workspace_may_start_at_any_four_bytes(ctx):
    import paper_2310_01775_amd as S
    probs = [(W.make_scene(8, p, 2, 3, 40, 0.005), W.cost_weights(), W.make_particles(8, p, N, 3))
             for p, N in enumerate([200, 1500])]
    scenes, w, Ns = ([S.make_scene(s) for s, _, _ in probs], [S.make_cost(c) for _, c, _ in probs], [200, 1500])
    cfg = S.make_cfg(3, lr=1e-3)
    need = S.Context.solve_workspace_bytes(scenes, Ns, cfg)
    outs = []
    for shift in (0, 4):
        print("case", shift, flush=True)
        flat = torch.cat([S.soa(th).reshape(-1) for _, _, th in probs]).contiguous()
        m, v, us = torch.zeros_like(flat), torch.zeros_like(flat), torch.zeros(2, device="cuda")
        buf = torch.zeros(need + 16, dtype=torch.uint8, device="cuda")
        cost = ctx.solve(scenes, w, Ns, cfg, flat, m, v, solve_time_us=us, workspace=buf[shift:shift + need])
        torch.cuda.synchronize()
        assert (us > 0).all()
        outs.append((flat, m, v, cost))
    for a, b in zip(*outs):
        assert torch.equal(a, b)


# two tight clusters: half of all distances within a thousandth of each other,
# far more than the candidate buffer takes from a bracket one histogram wide
@pytest.mark.parametrize("jitter", [1e-4, 1e-3])
@pytest.mark.parametrize("N,d", [(200, 6), (1000, 18), (1500, 30), (4097, 40)])
def test_bandwidth_of_tight_clusters_is_the_order_statistic(ctx, N, d, jitter):
    import paper_2310_01775_amd as S
    print("case", N, d, jitter, flush=True)
    th = jitter * np.random.default_rng(N + d).standard_normal((N, d))
    th[:, 0] += np.where(np.arange(N) % 2, 1.0, -1.0)
    th = th.astype(np.float32).astype(np.float64)
    h = torch.zeros(1, device="cuda")
    ctx.svgd_bandwidth(S.soa(th), h_out=h)
    torch.cuda.synchronize()
    m2 = float(h.item()) * math.log(N)
    D = np.concatenate([((th[i] - th[i + 1:]) ** 2).sum(1) for i in range(N - 1)])
    k = (D.size + 1) // 2
    # 64 FP32 products and sums over terms of up to |xi|^2 + |xj|^2 = D / 2
    tol = 64 * 2.0 ** -24
    assert (D < m2 * (1 - tol)).sum() < k <= (D <= m2 * (1 + tol)).sum()
