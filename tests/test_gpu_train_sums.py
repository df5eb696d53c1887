"""A training step's sums at the edges of their stages: weight-gradient sample
ranges of one MFMA step, of a remainder and of several load groups; the
workgroups' partial sums within one stage of 512, filling it and past it."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import mlp
from test_gpu_mlp import N_IN, _dev, _inputs, _nrm, _params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [64, 192, 8192, 8256])
def test_gradients_and_copies(ctx, M):
    import paper_2310_01775_amd as S
    print("case", M, flush=True)
    x, _ = _inputs(M)
    p = _params(2, x=x)
    c_np = W.f32(np.expm1(np.random.default_rng(M).normal(1.0, 1.0, M)))
    P = _dev(S.pack_mlp(p))
    Wb, fresh = ctx.mlp_weights(), ctx.mlp_weights()
    ctx.mlp_prepare(P, Wb)
    m, v = (torch.zeros(S.MLP_PARAMS, device="cuda") for _ in range(2))
    loss = torch.zeros(1, device="cuda")
    ctx.mlp_train_step(P, Wb, m, v, _dev(x), _dev(c_np), 1, lr=1e-3, loss=loss)
    ctx.mlp_prepare(P, fresh)
    torch.cuda.synchronize()
    L_ref, g_ref = mlp.training_loss_and_grads(p, x, c_np)
    g = S.unpack_mlp(m.cpu().double().numpy() / 0.1, N_IN)
    # BF16 operands (2^-9 each) through three layers and back
    assert abs(float(loss.item()) - L_ref) < 1e-2 * L_ref
    for k in ("W1", "b1", "W2", "b2", "w3", "b3"):
        e = _nrm(g[k], g_ref[k])
        print("grad", k, e, flush=True)
        assert e < 3e-2, k
    assert torch.equal(Wb.view(torch.int16), fresh.view(torch.int16))
