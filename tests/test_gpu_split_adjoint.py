"""The reverse sweep split over a workgroup's waves (small particle sets)
against the sweeps that do whole steps in one wave: bit for bit.

For more than one block the packed layout is the whole-step reference; for one
block, where both layouts are the same lanes, a tape with checkpoints too far
apart for the split kernels' LDS is."""
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _setup(N, H, B, T, seed=3):
    import paper_2310_01775_amd as S
    sc = W.make_scene(2, seed, B, H, T, 0.005)
    th = S.soa(W.make_particles(2, seed, N, H))
    return S, S.make_scene(sc), S.make_cost(W.cost_weights(rot=3.0)), th


def _grad(ctx, S, sc, w, th, ckpt, layout, per_phase=False):
    ctx.set_rollout_layout(layout)
    try:
        N = th.shape[1]
        tape = torch.empty(ctx.tape_floats(sc, N, ckpt), device="cuda")
        ctx.rollout_fwd(sc, w, th, tape=tape, ckpt_every=ckpt)
        bar = torch.linspace(-1.5, 0.5, N, device="cuda")
        g = ctx.rollout_adj(sc, w, th, tape, ckpt_every=ckpt, cost_bar=bar, per_phase=per_phase)
        torch.cuda.synchronize()
        return g
    finally:
        ctx.set_rollout_layout(S.LAYOUT_AUTO)


# N, H, B, T: ragged last waves; phases of one step, of fewer and of odd steps
# than a chunk; more workgroups than chunks of four steps leave room for
@pytest.mark.parametrize("N,H,B,T", [(1, 1, 2, 1), (5, 3, 3, 3), (37, 4, 2, 9), (130, 5, 4, 131), (333, 2, 3, 67),
                                     (2101, 8, 4, 24), (3001, 5, 3, 17)])
@pytest.mark.parametrize("per_phase", [False, True])
def test_split_sweep_equals_the_packed_sweep(ctx, N, H, B, T, per_phase):
    S, sc, w, th = _setup(N, H, B, T)
    print("case", N, H, B, T, per_phase, flush=True)
    a = _grad(ctx, S, sc, w, th, 0, S.LAYOUT_BLOCKS, per_phase)
    b = _grad(ctx, S, sc, w, th, 0, S.LAYOUT_PACKED, per_phase)
    assert torch.isfinite(a).all() and torch.equal(a, b)


# K: one step; segments shorter than a chunk; a short segment at each phase's
# end; the longest the split kernel's LDS holds; the two-wave kernel's range;
# beyond both
@pytest.mark.parametrize("N,H,B,T", [(1, 1, 1, 1), (70, 3, 1, 140), (129, 2, 2, 131), (50, 4, 3, 210), (17, 2, 4, 90)])
@pytest.mark.parametrize("K", [1, 3, 16, 31, 36, 50, 64])
def test_checkpointed_split_sweep_equals_the_full_tape(ctx, N, H, B, T, K):
    S, sc, w, th = _setup(N, H, B, T)
    print("case", N, H, B, T, K, flush=True)
    ref = _grad(ctx, S, sc, w, th, 1000, S.LAYOUT_BLOCKS)  # whole-step sweep: 1000 steps exceed the LDS
    assert torch.isfinite(ref).all()
    assert torch.equal(_grad(ctx, S, sc, w, th, K, S.LAYOUT_BLOCKS), ref)
    assert torch.equal(_grad(ctx, S, sc, w, th, 0, S.LAYOUT_BLOCKS), ref)
