"""GPU tests of the layer kernels (fp32 networks as three bf16 planes, larger bf16
networks on few envs): batches at the edges of their tiles and of the rules
that choose them, odd widths, networks of unlike depth, and values that are
not finite.

The fp32 bound is derived, not measured: a layer of K inputs whose operands
are off by dx gives sums off by at most (K + 8) 2^-24 (|W| |x| + |b|) (one
rounding per product and addition, the products left out of the planes, the
bias) + |W| dx, and one rounding of the result; the ReLU passes it on.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_09821_amd import binding, synth

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def _world(actor, critic, bf16, seed=7):
    d = synth.make_world(3 if bf16 else 2, n_envs=64)
    d["policy"] = synth.make_policy(np.random.default_rng(seed), actor, bf16)
    d["critic"] = synth.make_policy(np.random.default_rng(seed + 1), critic, bf16)
    return d


def _obs(N, ld, seed=3):
    rng = np.random.default_rng(seed)
    return rng.standard_normal((226, ld)).astype(np.float32), rng.integers(0, 1 << 20, ld).astype(np.int32)


def _run(ctx, obs, env_n, N, A, value=True):
    f = dict(device="cuda", dtype=torch.float32)
    g = [torch.from_numpy(obs).cuda(), torch.from_numpy(env_n).cuda()]
    out = [torch.full((N, A), 7.0, **f), torch.full((N, A), 7.0, **f), torch.full((N,), 7.0, **f),
           torch.full((N,), 7.0, **f)]
    if value:
        ctx.policy_act_value(g[0], g[1], N, *out)
    else:
        ctx.policy_act(g[0], g[1], N, *out[:3])
        ctx.value(g[0], N, out[3])
    torch.cuda.synchronize()
    return [o.cpu().numpy() for o in out]


def _bounded(net, x):
    """float64 outputs [n][out] of an fp32 MLP and the bound above."""
    x, dx = x.astype(np.float64), np.zeros(x.shape)
    for l, (W, b) in enumerate(zip(net["W"], net["b"])):
        W, b = W.astype(np.float64), b.astype(np.float64)
        z = x @ W.T + b
        dx = (W.shape[1] + 8) * U * (np.abs(x) @ np.abs(W).T + np.abs(b)) + dx @ np.abs(W).T + U * np.abs(z)
        x = np.maximum(z, 0.0) if l < len(net["W"]) - 1 else z
    return x, dx


# 64 x 64 tiles on few and many envs, 128 x 128 tiles (4100 envs: 33 columns of
# them), the 8-wave small kernel; odd widths; one action tile to four; a critic
# deeper and one shallower than the policy
@pytest.mark.parametrize("actor,critic,N,pad", [
    ([226, 1024, 512, 28], [226, 1024, 512, 1], 1, 0),
    ([226, 1024, 512, 28], [226, 1024, 512, 1], 33, 5),
    ([226, 1024, 512, 28], [226, 1024, 512, 1], 1000, 0),
    ([226, 1024, 512, 28], [226, 1024, 512, 1], 4100, 3),
    ([226, 300, 130, 33], [226, 70, 1], 127, 0),
    ([226, 300, 128], [226, 257, 300, 90, 1], 129, 1),
    ([226, 500, 65], [226, 1024, 1024, 1], 2049, 0)])
def test_fp32_layers(actor, critic, N, pad):
    print("fp32 layers %s %s N %d" % (actor, critic, N), flush=True)
    d = _world(actor, critic, False)
    ctx = binding.Context(d, max_envs=N)
    obs, env_n = _obs(N, N + pad)
    A = actor[-1]
    mean, action, logp, value = _run(ctx, obs, env_n, N, A)
    for net, got in ((d["policy"], mean), (d["critic"], value[:, None])):
        ref, bound = _bounded(net, obs[:, :N].T)
        assert (np.abs(got - ref) <= bound).all(), float((np.abs(got - ref) / bound).max())
        # that bound holds for any signs of the errors; over a batch they cancel:
        # fp32 sums in order are 5e-7 to 7e-7 off by norm, planes that lose
        # their third (or a product above 2^-16 of the leading one) 6e-6; by the
        # outputs' size over other observations, one env's may be near zero
        typical = _bounded(net, _obs(500, 500, 9)[0].T)[0]
        err = np.sqrt(np.mean((got - ref) ** 2) / np.mean(typical ** 2))
        print("relative error by norm %.2e" % err, flush=True)
        assert err <= 1e-6
    _, oa, olp = oracle.policy(d["policy"], d["config"]["seed"], obs[:, :N], env_n[:N].view(np.uint32))
    err = np.linalg.norm(action - oa, axis=1) / np.linalg.norm(oa, axis=1)
    assert (err <= 1e-4).all(), float(err.max())
    assert (np.abs(logp - olp) <= 1e-5 * np.abs(olp) + 1e-4).all()
    ctx.close()


# Rows of one weight: an output is one product, which fp32 rounds once (2^-24);
# the plane product left out is below 2^-32 of it (2^-30 where an operand is
# subnormal: its leading plane then has fewer bits) and the joining of the sums
# rounds at 2^-8 of its size, 2^-29 allowed for both.  Weights, observations and
# hidden activations through the whole range of fp32, subnormals with it.
@pytest.mark.parametrize("sw,sx,s2", [(1, 1, 1), (1e-36, 1, 1), (1, 1e-36, 1), (1e-36, 1, 1e30), (1e-39, 1e10, 1),
                                      (1e10, 1e-39, 1), (1.7e38, 0.25, 1), (1e-30, 1.7e38, 1)])
@pytest.mark.parametrize("N,H", [(64, 256), (1000, 1024), (4100, 1024)])
def test_fp32_single_products(N, H, sw, sx, s2):
    print("fp32 single products N %d H %d: %g %g %g" % (N, H, sw, sx, s2), flush=True)
    rng = np.random.default_rng(N + H)
    d = _world([226, H, 512, 128], [226, H, 1], False)

    def rows(n, k, v):
        W = np.zeros((n, k), np.float32)
        W[np.arange(n), np.arange(n) % k] = v
        return W

    w = ((1.0 + rng.random(H)) * sw).astype(np.float32)
    one = rows(1, H, 1.0)
    one[0, 0], one[0, 41] = 0.0, 1.0
    d["policy"]["W"] = [rows(H, 226, w), rows(512, H, 1.0), rows(128, 512, np.float32(s2))]
    d["critic"]["W"] = [rows(H, 226, w), one]
    for net in (d["policy"], d["critic"]):
        net["b"] = [np.zeros_like(b) for b in net["b"]]
    obs = ((1.0 + rng.random((226, N))) * sx).astype(np.float32)
    ctx = binding.Context(d, max_envs=N)
    mean, _, _, value = _run(ctx, obs, np.zeros(N, np.int32), N, 128)
    h = obs.T[:, :128].astype(np.float64) * w[:128].astype(np.float64)
    u = U * (1.0 + 2.0 ** -5)
    assert (np.abs(value - h[:, 41]) <= u * h[:, 41]).all()
    ref, rel = h * float(np.float32(s2)), u if s2 == 1 else 2 * u
    worst = float((np.abs(mean - ref) / ref).max())
    print("worst relative error %.3e" % worst, flush=True)
    assert worst <= rel
    ctx.close()


@pytest.mark.parametrize("N", [262144, 262145, 540001])
def test_fp32_calls_in_parts(N):
    """More than 262144 envs run in equal parts: the same bits as the rows of a
    call in one part, noise by the env's index in the call, nothing written past
    the end."""
    print("fp32 in parts N %d" % N, flush=True)
    A, M = 5, 20000
    d = _world([226, 40, 30, A], [226, 20, 30, 1], False)
    ctx = binding.Context(d, max_envs=N)
    obs, env_n = _obs(N, N + 3)
    got = _run(ctx, obs, env_n, N, A, value=False)
    f = dict(device="cuda", dtype=torch.float32)
    for n0 in (0, N - M):
        g = torch.from_numpy(np.ascontiguousarray(obs[:, n0:n0 + M])).cuda()
        n = torch.from_numpy(env_n[n0:n0 + M].copy()).cuda()
        out = [torch.full((M + 1, A), 7.0, **f), torch.full((M + 1, A), 7.0, **f), torch.full((M + 1,), 7.0, **f),
               torch.full((M + 1,), 7.0, **f)]
        ctx.policy_act(g, n, M, *out[:3])
        ctx.value(g, M, out[3])
        torch.cuda.synchronize()
        assert all(bool((o[M] == 7.0).all()) for o in out)
        rows = [o[:M].cpu().numpy() for o in out]
        assert np.array_equal(rows[0], got[0][n0:n0 + M]) and np.array_equal(rows[3], got[3][n0:n0 + M])
    _, oa, olp = oracle.policy(d["policy"], d["config"]["seed"], obs[:, :N], env_n[:N].view(np.uint32))
    assert (np.linalg.norm(got[1] - oa, axis=1) <= 1e-4 * np.linalg.norm(oa, axis=1)).all()
    assert (np.abs(got[2] - olp) <= 1e-5 * np.abs(olp) + 1e-4).all()
    ctx.close()


def test_fp32_workspace_of_many_envs():
    """The planes take no more memory than the activations of all the envs would
    as fp32 values (1024 wide, two buffers)."""
    envs = 1 << 20
    ctx = binding.Context(_world([226, 1024, 512, 28], [226, 1024, 512, 1], False), max_envs=envs)
    held = binding.im_get_info(ctx.ptr).device_bytes
    ctx.close()
    print("device bytes %d" % held, flush=True)
    assert held <= 2 * envs * 1024 * 4


# both sides of the batch sizes where a network changes kernels, and where the
# two networks stop sharing launches
@pytest.mark.parametrize("bf16,N", [(True, 1), (True, 512), (True, 513), (True, 1024), (True, 1025), (False, 500), (False, 8192),
                                    (False, 8193)])
def test_act_value_equals_the_two_calls(bf16, N):
    print("act_value bf16 %s N %d" % (bf16, N), flush=True)
    d = _world([226, 1024, 512, 28], [226, 512, 256, 1], bf16)
    ctx = binding.Context(d, max_envs=N)
    obs, env_n = _obs(N, N)
    a, b = _run(ctx, obs, env_n, N, 28), _run(ctx, obs, env_n, N, 28, value=False)
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
    if bf16:
        om, oa, olp = oracle.policy(d["policy"], d["config"]["seed"], obs[:, :N], env_n[:N].view(np.uint32))
        err = np.linalg.norm(a[0] - om, axis=1) / np.linalg.norm(om, axis=1)
        assert (err <= 2e-2).all(), float(err.max())
        ov = oracle.value(d["critic"], obs[:, :N])
        rms = np.sqrt(np.mean(ov.astype(np.float64) ** 2))
        assert (np.abs(a[3] - ov) <= 2e-2 * np.maximum(np.abs(ov), rms)).all()
    ctx.close()


# one to four action tiles, one to four MFMA tiles per wave of the one-launch
# kernel, unlike depths (the small critics run in it alone, on the layer kernels
# beside their policy); batches at the edges of the layer kernels' env tiles
@pytest.mark.parametrize("actor,critic", [
    ([226, 1024, 512, 28], [226, 1024, 1024, 512, 1]),
    ([226, 1024, 40], [226, 256, 1]),
    ([226, 512, 1024, 70], [226, 512, 1]),
    ([226, 1024, 700, 600, 128], [226, 768, 900, 1])])
def test_bf16_rows_do_not_depend_on_the_batch(actor, critic):
    """A bf16 row's outputs are the same bits on the layer kernels (up to 1024
    envs) as in the one-launch kernel (more)."""
    A = actor[-1]
    ctx = binding.Context(_world(actor, critic, True), max_envs=1100)
    obs, env_n = _obs(1100, 1100)
    ref = _run(ctx, obs, env_n, 1100, A)
    for N in (1, 32, 33, 130, 1024):
        print("bf16 rows %s %s N %d" % (actor, critic, N), flush=True)
        for value in (True, False):
            got = _run(ctx, obs, env_n, N, A, value)
            for name, x, y in zip(("mean", "action", "logp", "value"), got, ref):
                assert np.array_equal(x, y[:N]), name
    ctx.close()


# (4100 envs: 64 x 64 tiles for 256 features, 128 x 128 for 1024)
@pytest.mark.parametrize("N,H", [(40, 256), (200, 256), (4100, 256), (4100, 1024), (70, 1024)])
def test_fp32_values_that_are_not_finite(N, H):
    """Infinities, NaNs and values above bf16's range in the observation and an
    infinite weight: what fp32 arithmetic gives (a NaN is cleared by the ReLU)."""
    print("fp32 not finite N %d H %d" % (N, H), flush=True)
    d = _world([226, H, 512, 28], [226, H, 1], False)
    d["policy"]["W"][1][5, 7] = np.inf
    obs, env_n = _obs(N, N)
    obs[3, 1], obs[200, 2], obs[17, 5], obs[225, 9], obs[0, N - 1] = np.inf, -np.inf, np.nan, 3.4e38, -3.4e38
    obs[100, 11], obs[101, 11] = np.inf, -np.inf
    ctx = binding.Context(d, max_envs=N)
    mean, _, _, value = _run(ctx, obs, env_n, N, 28)
    for net, got in ((d["policy"], mean), (d["critic"], value[:, None])):
        x = obs.T.astype(np.float64)
        with np.errstate(invalid="ignore", over="ignore"):
            for l, (W, b) in enumerate(zip(net["W"], net["b"])):
                # column by column: a BLAS product does not promise inf and NaN
                W = W.astype(np.float64)
                z = np.stack([(x * w).sum(axis=1) for w in W], axis=1) + b
                x = np.fmax(z, 0.0) if l < len(net["W"]) - 1 else z
        assert np.array_equal(np.isnan(got), np.isnan(x)) and np.array_equal(np.isinf(got), np.isinf(x))
        inf = np.isinf(x)
        assert np.array_equal(np.sign(got[inf]), np.sign(x[inf]))
        fin = np.isfinite(x)
        scale = np.abs(np.where(fin, x, 0.0)).max(axis=1, keepdims=True) + np.zeros_like(x)
        assert (np.abs(got[fin] - x[fin]) <= 1e-4 * np.maximum(scale[fin], 1.0)).all()
    ctx.close()


@pytest.mark.parametrize("N,every", [(64, False), (64, True), (1000, False), (4096, False), (4096, True)])
def test_fp32_values_that_are_not_finite_cost_little(N, every):
    """One pass of fp32 products over the affected tiles, not a walk through each
    sum: at most three times the call's time (measured 1.3 to 2.1), also where
    every env holds an infinity."""
    print("fp32 not finite, cost, N %d every env %s" % (N, every), flush=True)
    d = _world([226, 1024, 512, 28], [226, 256, 1], False)
    ctx = binding.Context(d, max_envs=N)
    obs, env_n = _obs(N, N)
    bad = obs.copy()
    bad[7, :: 1 if every else N] = np.inf
    f = dict(device="cuda", dtype=torch.float32)
    out = [torch.empty((N, 28), **f), torch.empty((N, 28), **f), torch.empty((N,), **f)]
    n = torch.from_numpy(env_n).cuda()
    us = []
    for x in (obs, bad):
        g = torch.from_numpy(x).cuda()
        best = np.inf
        for _ in range(6):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            for _ in range(10):
                ctx.policy_act(g, n, N, *out)
            ev[1].record()
            torch.cuda.synchronize()
            best = min(best, ev[0].elapsed_time(ev[1]) * 100.0)
        us.append(best)
    print("us per call: finite %.1f, not %.1f" % tuple(us), flush=True)
    assert us[1] <= 3.0 * us[0]
    ctx.close()


def _captured(ctx, obs, env_n, N, A):
    """A graph of policy_act on these inputs, and its outputs."""
    f = dict(device="cuda", dtype=torch.float32)
    g = [torch.from_numpy(obs).cuda(), torch.from_numpy(env_n).cuda()]
    out = [torch.zeros((N, A), **f), torch.zeros((N, A), **f), torch.zeros((N,), **f)]
    ctx.policy_act(g[0], g[1], N, *out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.policy_act(g[0], g[1], N, *out)
    return graph, g, out


@pytest.mark.parametrize("bf16", [True, False])
def test_policy_graph_outlives_a_wider_critic(bf16):
    """im_set_critic leaves the policy's buffers where they are: a graph of the
    policy captured before it replays to the same bits, and writes nothing that
    has been handed out since."""
    N, A = 64, 28
    print("policy graph, then a wider critic, bf16 %s" % bf16, flush=True)
    d = _world([226, 1024, 256, A], [226, 256, 1], bf16)
    ctx = binding.Context(d, max_envs=N)
    obs, env_n = _obs(N, N)
    graph, g, out = _captured(ctx, obs, env_n, N, A)
    eager = [o.clone() for o in out]
    wide = binding.Description(_world([226, 1024, 256, A], [226, 2048, 2048, 1], bf16))
    binding.im_set_critic(ctx.ptr, wide.critic)
    filled = [torch.full((n,), 3.0, device="cuda") for n in [1 << 14] * 64 + [1 << 20] * 32]
    for _ in range(3):
        for o in out:
            o.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, eager))
        assert all(bool((x == 3.0).all()) for x in filled)
    ctx.policy_act(g[0], g[1], N, *out)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(out, eager))
    del graph
    ctx.close()


def test_policy_survives_a_critic_that_does_not_fit():
    """A critic whose workspace cannot be allocated (2^24 envs x 16384 wide: 512
    GiB) is refused; the policy's calls go on as before."""
    N, A = 64, 28
    print("critic that does not fit", flush=True)
    d = _world([226, 1024, A], [226, 16384, 1], True)
    ctx = binding.Context(d, max_envs=1 << 24, critic=False)
    obs, env_n = _obs(N, N)
    graph, g, out = _captured(ctx, obs, env_n, N, A)
    eager = [o.clone() for o in out]
    with pytest.raises(binding.ImError) as ei:
        binding.im_set_critic(ctx.ptr, ctx.desc.critic)
    assert ei.value.status == binding.IM_ERR_OOM
    for call in (lambda: ctx.policy_act(g[0], g[1], N, *out), graph.replay):
        for o in out:
            o.zero_()
        call()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, eager))
    with pytest.raises(binding.ImError, match="no critic"):
        ctx.value(g[0], N, out[2])
    del graph
    ctx.close()
