"""The exact median when the sample's bracket misses it: the select then goes
over every pair again, below or above the bracket.

Two clusters of points, split so that the fixed sample's pairs cross between
them much less often (or more often) than all pairs do: by more than half of
all pairs against well under half of the sample, the median is the distance
between the clusters, above the sample's bracket; the other way round it is a
distance inside a cluster, below it."""
import math

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

SAMPLE = 8192


def _mix(x):  # MurmurHash3's 32-bit finaliser
    x = np.asarray(x, dtype=np.uint64) & 0xffffffff
    x = (x ^ (x >> np.uint64(16))) * 0x85ebca6b & 0xffffffff
    x = (x ^ (x >> np.uint64(13))) * 0xc2b2ae35 & 0xffffffff
    return x ^ (x >> np.uint64(16))


def _sample(N):
    t = np.arange(SAMPLE, dtype=np.uint64)
    i = (_mix(2 * t + 1) % np.uint64(N)).astype(int)
    j = (_mix((2 * t + 2) ^ 0x9e3779b9) % np.uint64(N - 1)).astype(int)
    return i, j + (j >= i)


def _clusters(N, kind):
    """Labels +-1: equal halves few sampled pairs cross between ("above"), or
    halves sqrt(N) off equal that many cross between ("below")."""
    i, j = _sample(N)
    n1 = N // 2 if kind == "above" else N // 2 + int(math.sqrt(N))
    s = np.ones(N)
    s[np.random.default_rng(N).permutation(N)[n1:]] = -1.0
    sign = 1.0 if kind == "above" else -1.0
    for _ in range(N):  # exchange the pair of points that gains most, while one gains
        f = sign * s * (np.bincount(i, s[j], N) + np.bincount(j, s[i], N))
        a, b = np.argmin(np.where(s > 0, f, np.inf)), np.argmin(np.where(s < 0, f, np.inf))
        if f[a] + f[b] >= -2.0:  # the two may be sampled together
            break
        s[a], s[b] = -1.0, 1.0
    return s


def _particles(N, d, kind):
    """Every push's side 0, offset and depth hold the cluster, with jitter."""
    rng = np.random.default_rng(N + d)
    th = 0.1 * rng.standard_normal((N, d))
    s = _clusters(N, kind)
    for c in (0, 4, 5):
        th[:, c] += s
    return th.astype(np.float32).astype(np.float64)


def _distances(x):
    q = (x * x).sum(1)
    return np.maximum(q[:, None] + q[None, :] - 2.0 * (x @ x.T), 0.0)


def _assert_missed(D, kind):
    N = D.shape[0]
    k = (N * (N - 1) // 2 + 1) // 2
    m2 = np.sort(D[np.triu_indices(N, 1)])[k - 1]
    s = np.sort(D[_sample(N)].astype(np.float32))
    bits = s.view(np.uint32).astype(np.int64)
    half = 2.0 / math.sqrt(SAMPLE)  # the bracket's ranks; its ends move out by less than a bin
    span = (bits[-1] - bits[0]) // 1024 + 1
    at = np.float32(m2).view(np.uint32).astype(np.int64)
    if kind == "above":
        assert at > bits[math.ceil(SAMPLE * (0.5 + half)) - 1] + span
    else:
        assert at < bits[math.floor(SAMPLE * (0.5 - half)) - 1] - span


def _assert_median(D, m2):
    """m2 is the lower median of the distances as FP32 computes them: in the Gram
    form at most 64 products and sums over terms of up to |x_i|^2 + |x_j|^2, here
    <= 16 D (direct differences lose less)."""
    N = D.shape[0]
    D = D[np.triu_indices(N, 1)]
    k = (D.size + 1) // 2
    tol = 1024 * 2.0 ** -24
    assert (D < m2 * (1 - tol)).sum() < k <= (D <= m2 * (1 + tol)).sum()


# the finishing workgroup; the passes of the split form and of FP32 products
# (8 to 16 steps of 4 coordinates), in blocks of 64 and of 256 rows
@pytest.mark.parametrize("kind", ["above", "below"])
@pytest.mark.parametrize("N,d", [(129, 6), (1000, 12), (1448, 48), (1449, 30), (1500, 32), (1500, 54), (2001, 64),
                                 (4097, 31), (4111, 40), (4200, 64)])
def test_median_outside_the_bracket(ctx, N, d, kind):
    import paper_2310_01775_amd as S
    print("case", N, d, kind, flush=True)
    th = _particles(N, d, kind)
    D = _distances(th)
    _assert_missed(D, kind)
    h = torch.zeros(1, device="cuda")
    theta = S.soa(th)
    ws = ctx.svgd_bandwidth(theta, h_out=h)
    first = h.clone()
    for _ in range(2):
        ctx.svgd_bandwidth(theta, h_out=h, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(h, first)
    _assert_median(D, float(h.item()) * math.log(N))


# direct differences in the passes too, for both kernels' features
@pytest.mark.parametrize("kind", ["above", "below"])
@pytest.mark.parametrize("N,K", [(700, 2), (1500, 3), (1500, 8), (4200, 5)])
def test_structured_medians_outside_the_bracket(ctx, N, K, kind):
    import paper_2310_01775_amd as S
    print("case", N, K, kind, flush=True)
    th = _particles(N, 6 * K, kind)
    t3 = th.reshape(N, K, 6)
    e = np.exp(t3[:, :, :4] - t3[:, :, :4].max(-1, keepdims=True))
    feats = [t3[:, :, 4:].reshape(N, -1), (e / e.sum(-1, keepdims=True)).reshape(N, -1)]
    Ds = [_distances(f) for f in feats]
    for D in Ds:
        _assert_missed(D, kind)
    h = torch.zeros(2, device="cuda")
    ctx.svgd_step_structured(S.soa(th), S.soa(np.ones_like(th)), S.struct_kernel(S.KERNEL_PUSH, K), h_out=h)
    torch.cuda.synchronize()
    for c in range(2):
        _assert_median(Ds[c], float(h[c].item()) * K * math.log(N))


@pytest.mark.parametrize("kind", ["above", "below"])
def test_a_batch_outside_the_bracket_equals_its_loop(ctx, kind):
    import paper_2310_01775_amd as S
    probs = [(W.make_scene(8, p, 2, H, 30, 0.005), W.cost_weights(), _particles(N, 6 * H, kind), N)
             for p, (N, H) in enumerate([(1000, 2), (1500, 5), (1500, 6), (4097, 3)])]
    flat = torch.cat([S.soa(th).reshape(-1) for _, _, th, _ in probs]).contiguous()
    m, v = torch.zeros_like(flat), torch.zeros_like(flat)
    ctx.solve([S.make_scene(s) for s, _, _, _ in probs], [S.make_cost(w) for _, w, _, _ in probs],
              [N for _, _, _, N in probs], S.make_cfg(1, lr=1e-3), flat, m, v)
    torch.cuda.synchronize()
    off = 0
    for s, w, th, N in probs:
        print("case", N, kind, flush=True)
        sc, cw, theta = S.make_scene(s), S.make_cost(w), S.soa(th)
        tape = torch.empty(ctx.tape_floats(sc, N), device="cuda")
        ctx.rollout_fwd(sc, cw, theta, tape=tape)
        g = ctx.rollout_adj(sc, cw, theta, tape, cost_bar=torch.full((N,), -1.0, device="cuda"))
        phi = ctx.svgd_step(theta, g)
        ctx.adam_step(theta, phi, torch.zeros_like(theta), torch.zeros_like(theta), 1, lr=1e-3)
        torch.cuda.synchronize()
        assert torch.equal(flat[off:off + theta.numel()].view_as(theta), theta)
        off += theta.numel()


# a lost particle's distances rank last; with half of the particles lost the
# sample's median (or a small problem's, of all its pairs) is no number's
@pytest.mark.parametrize("N,lost", [(300, 0), (300, 50), (300, 160), (100, 10), (100, 60), (300, 300)])
def test_sampled_median_with_lost_particles(ctx, N, lost):
    import paper_2310_01775_amd as S
    print("case", N, lost, flush=True)
    th = np.random.default_rng(N + lost).standard_normal((N, 6)).astype(np.float32).astype(np.float64)
    th[np.random.default_rng(1).permutation(N)[:lost], 2] = np.nan
    h = torch.zeros(1, device="cuda")
    ctx.svgd_step_bf16(S.soa(th), S.soa(np.ones_like(th)), h_out=h)
    torch.cuda.synchronize()
    i, j = _sample(N) if N > 128 else np.triu_indices(N, 1)
    D = ((th[i] - th[j]) ** 2).sum(1)
    m2 = np.sort(np.where(np.isnan(D), np.inf, D))[(D.size + 1) // 2 - 1]
    if np.isinf(m2):
        assert math.isinf(h.item())
    else:
        assert abs(h.item() * math.log(N) / m2 - 1.0) < 16 * 2.0 ** -24
