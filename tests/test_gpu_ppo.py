"""The PPO update on the GPU against the oracle (torch float64 autograd and a
plain Adam) on a rollout the oracle generated.

One minibatch's gradient is compared stage by stage, each stage element by
element on the GPU's own inputs to it (read back with im_ppo_read), so that
a rounding decision one side takes differently cannot spread into later
stages:

* gather: the minibatch's observation rounded to bf16, bit for bit;
* forward, every layer of both networks: the oracle's float64 pre-activation
  z of the GPU's (bf16) layer input.  A bf16 output must lie between the
  roundings of relu(z - d) and relu(z + d), with d = (K + 2) 2^-24 (|x| |W|^T
  + |b|) the worst-case error of a float32 sum of the K products and the bias
  in any order; outputs of the last layers (float32): |g - z| <= d + 2^-24 |z|;
* loss gradients at the GPU's mean and value: d loss / d mean as stored in
  bf16 within half a bf16 spacing of the float64 value plus the float32 error
  of the sample's ratio (its log-likelihood sums A terms: (A + 8) 2^-24 sum
  |term|); samples whose ratio lies within twice that error of a clip bound
  may take either branch and are excluded (counted); d loss / d value to
  8 2^-24 relative; the log_std gradient within the per-sample error bounds
  summed (tie samples: either branch);
* backward from the GPU's stored output gradients through its own forward
  activations: the float64 chain rule.  The GPU stores each hidden layer's
  pre-activation gradient in bf16 (a rounding error of at most half a bf16
  spacing, plus the float32 error of the product that formed it), and errors
  of upper layers propagate through W^T and the ReLU masks.  With c the
  per-element bound of those errors, the Hoeffding proxy of a weight
  gradient's error is S^2 = sum_s P[s, i] x[s, k]^2, P[s, i] = c[s, i]^2 +
  mask (P_above W^2)[s, i]; tolerance 7 S (probability of a larger deviation
  below 5e-11 per element), plus 7 2^-24 sqrt(n) (|o| + 3 A) for the
  float32 sums over the n samples (each addition errs by at most 2^-24 times
  a partial sum, bounded by |o| + 3 A with A the root sum of squares of the
  terms; those errors summed like a random walk).

The parameter change of a whole update is compared with the oracle's (cosine
and norm per tensor: Adam's first steps move parameters by about lr times the
sign of their gradient, so components with a gradient near zero may move
either way), one Adam step element by element on the GPU's own gradient,
and the KL-adaptive learning rate; plus self-consistency: determinism, graph
replay, and the rollout copies (policy, critic) refreshed from the masters.
"""
import numpy as np
import pytest
import torch

import oracle
from oracle import ppo
from paper_2609_09821_amd import binding, synth

pytestmark = pytest.mark.gpu

G32, L32 = float(np.float32(synth.GAMMA)), float(np.float32(synth.LAMBDA))


def _rollout(cfg, N, T, perturb=0.03, actor=None, critic=None):
    """A T-step rollout generated by the oracle (policy, critic, env step,
    GAE) with a policy whose weights are the workload's perturbed by a
    relative `perturb` (the update then starts at a KL well above zero, as
    after earlier updates); returns (world description, data dict, summary)."""
    d = synth.make_world(cfg, n_envs=N)
    if actor is not None:
        d["policy"] = synth.make_policy(np.random.default_rng(cfg + 5), actor, True)
        d["critic"] = synth.make_policy(np.random.default_rng(cfg + 6), critic, True)
    w = oracle.World(d)
    pol, crit = d["policy"], d["critic"]
    rng = np.random.default_rng(cfg + 77)
    pol = dict(pol, W=[synth.bf16_round((W * (1 + perturb * rng.standard_normal(W.shape)))
                                        .astype(np.float32)) for W in pol["W"]])
    seed = d["config"]["seed"]
    prev = bool(d["config"]["obs_prev_action"])
    A = pol["dims"][-1]
    st = w.state(N)
    w.reset_envs(st)
    obs = np.zeros((T + 1, w.D, N), np.float32)
    act = np.zeros((T, N, A), np.float32)
    mean = np.zeros((T, N, A), np.float32)
    logp = np.zeros((T, N), np.float32)
    value = np.zeros((T + 1, N), np.float32)
    rew = np.zeros((T, N), np.float32)
    term = np.zeros((T, N), np.uint8)
    trunc = np.zeros((T, N), np.uint8)
    for t in range(T):
        obs[t] = st.obs
        m, a, lp = oracle.policy(pol, seed, st.obs, st.n)
        mean[t], act[t], logp[t] = m, a, lp
        value[t] = oracle.value(crit, st.obs)
        w.standin(st, d["sigma_joint"], d["sigma_vel"])
        w.env_step(st, prev_action=a if prev else None)
        rew[t], term[t], trunc[t] = st.reward, st.terminated, st.truncated
    obs[T] = st.obs
    value[T] = oracle.value(crit, st.obs)
    adv, ret = oracle.gae(rew, term, trunc, value, G32, L32)
    summary, _, _ = oracle.rollout_summary(rew, term, trunc, value, adv, ret,
                                           np.zeros(N, np.float32), np.zeros(N, np.int32))
    data = dict(obs=obs, action=act, mean=mean, logp=logp, value=value, adv=adv, ret=ret)
    return d, data, summary


def _upload(ctx, data, summary, N, T):
    ro = binding.RolloutStorage(ctx, N, T)
    ro.obs.copy_(torch.from_numpy(data["obs"]))
    ro.action.copy_(torch.from_numpy(data["action"]))
    ro.mean.copy_(torch.from_numpy(data["mean"]))
    ro.logp.copy_(torch.from_numpy(data["logp"]))
    ro.value.copy_(torch.from_numpy(data["value"]))
    ro.advantage.copy_(torch.from_numpy(data["adv"]))
    ro.ret.copy_(torch.from_numpy(data["ret"]))
    ro.summary.copy_(torch.from_numpy(summary))
    return ro


def _perm(epochs, n_chunks, seed):
    rng = np.random.default_rng(seed)
    return np.stack([rng.permutation(n_chunks) for _ in range(epochs)]).astype(np.int32)


def _segments(actor, critic):
    out, o = [], 0
    for l, (W, b) in enumerate(zip(actor["W"], actor["b"])):
        out.append(("actor W%d" % l, slice(o, o + W.size))); o += W.size
        out.append(("actor b%d" % l, slice(o, o + b.size))); o += b.size
    out.append(("log_std", slice(o, o + actor["log_std"].size))); o += actor["log_std"].size
    for l, (W, b) in enumerate(zip(critic["W"], critic["b"])):
        out.append(("critic W%d" % l, slice(o, o + W.size))); o += W.size
        out.append(("critic b%d" % l, slice(o, o + b.size))); o += b.size
    return out


U32 = 2.0 ** -24


def _bf16(a):
    """float64 -> float32 -> bf16 (nearest even) -> float64."""
    t = torch.from_numpy(np.ascontiguousarray(a, np.float64)).to(torch.float32)
    return t.to(torch.bfloat16).to(torch.float64).numpy()


def _half_ulp16(a):
    """Half the bf16 spacing at |a| (8 significant bits); 0 at 0."""
    a = np.abs(np.asarray(a, np.float64))
    e = np.floor(np.log2(np.where(a > 0, a, 1.0)))
    return np.where(a > 0, np.exp2(e - 8), 0.0)


def _read(ctx, name, layer=0):
    return ctx.ppo_read(name, layer).float().cpu().numpy().astype(np.float64)


def _forward_stage(bufs, net, which, x, cols):
    """Layer-by-layer forward check of one network on the GPU's own layer
    inputs (bufs: its hidden-layer outputs); returns [(W_l, x_l)], the GPU's
    last-layer input and the number of bf16 roundings taken the other way."""
    layers, flips = [], 0
    L = len(net["W"])
    for l in range(L - 1):
        W = np.asarray(net["W"][l], np.float64)
        b = np.asarray(net["b"][l], np.float64)
        z = ppo.layer_forward(W, b, x)
        d = (W.shape[1] + 2) * U32 * (np.abs(x) @ np.abs(W).T + np.abs(b))
        lo, hi = _bf16(np.maximum(z - d, 0.0)), _bf16(np.maximum(z + d, 0.0))
        H = bufs[l]
        assert H.shape[1] == cols
        out = W.shape[0]
        assert (H[out:] == 0).all(), "%s layer %d: padding rows" % (which, l)
        h = H[:out].T
        bad = (h < lo) | (h > hi)
        assert not bad.any(), "%s layer %d: %d outputs outside the rounding bounds, e.g. %s" % (
            which, l, int(bad.sum()), np.argwhere(bad)[:3].tolist())
        flips += int((h != _bf16(np.maximum(z, 0.0))).sum())
        layers.append((W, x))
        x = h
        del z, d, lo, hi
    return layers, x, flips


def _out_check(name, g, W, b, x):
    z = ppo.layer_forward(W, b, x)
    d = (W.shape[1] + 2) * U32 * (np.abs(x) @ np.abs(W).T + np.abs(b)) + U32 * np.abs(z)
    bad = np.abs(g - z) > d
    assert not bad.any(), "%s: %d outside the float32 bound" % (name, int(bad.sum()))


def _backward_bounds(layers, out, n):
    """Per element tolerance of the weight and bias gradients of one network
    whose top-layer gradient is given exactly (see the module docstring)."""
    L = len(layers)
    tol = [None] * L
    P = None
    for l in range(L - 1, -1, -1):
        W, x = layers[l]
        g = out[l][2]
        if l == L - 1:
            P = np.zeros_like(g)
        else:
            W1, x1 = layers[l + 1]
            g1 = out[l + 1][2]
            mask = x1 > 0
            c = (1.01 * _half_ulp16(g) + (W1.shape[0] + 2) * U32 * (np.abs(g1) @ np.abs(W1))) * mask
            P = c * c + mask * (P @ (W1 * W1))
        x2 = x * x
        A_w = np.sqrt((g * g).T @ x2)
        A_b = np.sqrt((g * g).sum(axis=0))
        acc = 7.0 * U32 * np.sqrt(n)
        tw = 7.0 * np.sqrt(P.T @ x2) + acc * (np.abs(out[l][0]) + 3.0 * A_w)
        tb = 7.0 * np.sqrt(P.sum(axis=0)) + acc * (np.abs(out[l][1]) + 3.0 * A_b)
        tol[l] = (tw + 1e-30, tb + 1e-30)
    return tol


def _gpu_minibatch(ctx, d, p, ep, mb, batch):
    """im_ppo_grad of one minibatch and every stage buffer, on the host."""
    P_ = ctx.ppo_params()
    g = torch.zeros(P_, device="cuda")
    stats = torch.zeros(len(binding.PPO_STATS), dtype=torch.float64, device="cuda")
    ctx.ppo_grad(batch, binding.ppo_params(**p), ep, mb, g, stats)
    torch.cuda.synchronize()
    res = dict(grad=g.cpu().numpy().astype(np.float64), stats=stats.cpu().numpy())
    for name in ("input", "mean", "value", "dmean", "dvalue"):
        res[name] = _read(ctx, name)
    for net, which in ((d["policy"], "actor_hidden"), (d["critic"], "critic_hidden")):
        res[which] = [_read(ctx, which, l) for l in range(len(net["W"]) - 1)]
    return res


def _minibatch_of(perm, ep, mb, mbs):
    n_chunks = perm.shape[1]
    q, r = n_chunks // mbs, n_chunks % mbs
    first = mb * q + min(mb, r)
    return perm[ep][first:first + q + (1 if mb < r else 0)]


def _check_stages(res, d, data, grp, p, am, asd):
    """Stage-by-stage comparison of one minibatch (res: the GPU's gradient,
    statistics and stage buffers) with the oracle; see the module docstring."""
    pol, crit = d["policy"], d["critic"]
    A = pol["dims"][-1]
    M = 64 * len(grp)
    mbd = ppo.gather(data, grp, pol["log_std"])
    gg = res["grad"]
    seg = dict(_segments(pol, crit))

    # gather
    X0 = res["input"]
    cols = X0.shape[1]
    Dm = pol["dims"][0]
    assert cols == (M + 255) // 256 * 256
    assert np.array_equal(X0[:Dm, :M].T, _bf16(mbd["obs"])), "gathered observation"
    assert (X0[Dm:] == 0).all() and (X0[:, M:] == 0).all(), "gather padding"
    x0 = X0[:Dm].T

    # forward
    al, xa, fa = _forward_stage(res["actor_hidden"], pol, "actor_hidden", x0, cols)
    cl, xc, fc = _forward_stage(res["critic_hidden"], crit, "critic_hidden", x0, cols)
    Wa, ba = np.asarray(pol["W"][-1], np.float64), np.asarray(pol["b"][-1], np.float64)
    Wc, bc = np.asarray(crit["W"][-1], np.float64), np.asarray(crit["b"][-1], np.float64)
    MU = res["mean"]
    VV = res["value"]
    _out_check("mean", MU.T, Wa, ba, xa)
    _out_check("value", VV.T, Wc, bc, xc)
    al.append((Wa, xa))
    cl.append((Wc, xc))

    # loss gradients at the GPU's mean and value
    mu, V = MU.T[:M], VV[0, :M]
    o = ppo.output_grads(mu, V, pol["log_std"], mbd, p, am, asd)
    sig = np.exp(np.asarray(pol["log_std"], np.float64))
    act = mbd["action"].astype(np.float64)
    terms = (act - mu) ** 2 / (2 * sig ** 2) + np.abs(np.log(sig)) + 0.5 * ppo.LOG_2PI
    e_lp = (A + 8) * U32 * terms.sum(axis=1) + 8 * U32 * np.abs(mbd["logp_old"])
    rho = 1.01 * e_lp + 8 * U32
    ratio, eps = o["ratio"], p["clip"]
    tie = (np.abs(ratio - (1 + eps)) <= 2 * rho * ratio) | (np.abs(ratio - (1 - eps)) <= 2 * rho * ratio)
    DM = res["dmean"]
    assert (DM[A:] == 0).all() and (DM[:, M:] == 0).all(), "dmean padding"
    dm = DM[:A, :M].T
    em = (rho + 16 * U32)[:, None] * np.abs(o["dmu"])
    tol = 1.01 * _half_ulp16(np.abs(o["dmu"]) * (1 + rho[:, None])) + em + 1e-38
    bad = (np.abs(dm - o["dmu"]) > tol) & ~tie[:, None]
    assert not bad.any(), "d loss / d mean: %d elements, e.g. %s" % (int(bad.sum()), np.argwhere(bad)[:3].tolist())
    Vo, R = mbd["value_old"].astype(np.float64), mbd["ret"].astype(np.float64)
    DV = res["dvalue"][0]
    assert (DV[M:] == 0).all()
    vtie = np.zeros(M, bool)
    if p["clipped_value_loss"]:
        Vc_ = Vo + np.clip(V - Vo, -eps, eps)
        # either side of the clamp, or (clamped) either branch of the max: the
        # two choices then give different gradients (inside the clamp both
        # branches give 2 (V - R) up to the rounding of V_old + (V - V_old))
        vtie = (np.abs(np.abs(V - Vo) - eps) <= 1e-5 * (1 + np.abs(V) + np.abs(Vo))) | \
            ((np.abs((V - R) ** 2 - (Vc_ - R) ** 2) <= 1e-5 * ((V - R) ** 2 + (Vc_ - R) ** 2))
             & (np.abs(V - Vo) > eps))
    vt = 8 * U32 * np.abs(o["dV"]) + 2 * p["value_coef"] / M * 4 * U32 * (np.abs(V) + np.abs(Vo) + np.abs(R))
    bad = (np.abs(DV[:M] - o["dV"]) > vt) & ~vtie
    assert not bad.any(), "d loss / d value: %d samples" % int(bad.sum())
    # log_std: each sample adds dlogp_s ((a - mu)^2 / sigma^2 - 1); a tie sample
    # may add that (active) or nothing (clipped) on either side
    fac = np.abs((act - mu) ** 2 / sig ** 2 - 1.0)
    alt = np.abs((mbd["adv"].astype(np.float64) - am) / (asd + 1e-8)) * ratio / M
    contrib = np.abs(o["dlogp"])[:, None] * fac
    ltol = ((rho + 16 * U32)[:, None] * contrib)[~tie].sum(axis=0) + \
        (np.maximum(contrib, alt[:, None] * fac))[tie].sum(axis=0) + 1e-12
    gl = gg[seg["log_std"]]
    assert (np.abs(gl - o["dlog_std"]) <= ltol).all(), "log_std gradient"
    st = res["stats"]
    for k, key in ((0, "l_pi"), (1, "l_v"), (2, "kl")):
        assert abs(st[k] - o[key]) <= 1e-3 * (abs(o[key]) + 1e-3), (key, st[k], o[key])

    # backward from the GPU's stored output gradients
    worst = {}
    for name, layers, gout in (("actor", al, DM[:A].T), ("critic", cl, DV[:, None])):
        out = ppo.backward(layers, gout)
        tols = _backward_bounds(layers, out, cols)
        for l, ((dW, db, _), (tw, tb)) in enumerate(zip(out, tols)):
            for kind, ref, t in (("W", dW, tw), ("b", db, tb)):
                key = "%s %s%d" % (name, kind, l)
                got = gg[seg[key]].reshape(ref.shape)
                err = np.abs(got - ref)
                bad = err > t
                assert not bad.any(), "%s: %d of %d elements out of tolerance, worst %.3g of its " \
                    "tolerance at %s" % (key, int(bad.sum()), bad.size, float((err / t).max()),
                                         np.unravel_index(np.argmax(err / t), err.shape))
                worst[key] = float((err / t).max())
        del out, tols
    print("stages: %d samples, forward flips actor %d critic %d, ratio ties %d, value ties %d; "
          "worst gradient error / tolerance %s" % (M, fa, fc, int(tie.sum()), int(vtie.sum()),
                                                   {k: round(v, 3) for k, v in worst.items()}))
    return gg, o


# (6, 192, 3, 3): 192-sample minibatches padded to 256 columns, the
# previous-action observation; (3, 1024, 2, 1): a 2048-sample minibatch, 8
# column tiles per masked-gradient GEMM; (4, 16384, 4, 1): the update's
# production shape (S24 361-1024-1024-512-69 networks, a 65536-sample
# minibatch on 256x256 tiles, 32 parts of the critic head's sums)
@pytest.mark.parametrize("cfg,N,T,mbs", [(3, 256, 2, 2), (6, 192, 3, 3), (3, 1024, 2, 1),
                                         (4, 16384, 4, 1)])
def test_minibatch_gradient_stages(cfg, N, T, mbs):
    print("stage parity cfg %d: %d envs x %d steps, %d minibatches" % (cfg, N, T, mbs), flush=True)
    d, data, summary = _rollout(cfg, N, T)
    ctx = binding.Context(d, max_envs=N)
    n_chunks = T * N // 64
    ctx.ppo_setup((n_chunks + mbs - 1) // mbs * 64)
    ro = _upload(ctx, data, summary, N, T)
    perm = _perm(2, n_chunks, cfg)
    gperm = torch.from_numpy(perm).cuda()
    lr = torch.full((1,), 1e-3, device="cuda")
    p = dict(binding.PPO_DEFAULTS, epochs=2, minibatches=mbs, entropy_coef=2.5e-4)
    batch = binding.ppo_batch(ro, gperm, lr)
    x = torch.empty(ctx.ppo_params(), device="cuda")
    ctx.ppo_params(x)
    pol, crit = d["policy"], d["critic"]
    torch.cuda.synchronize()
    assert np.array_equal(x.cpu().numpy(), ppo.flat_params(pol, crit)), "masters start from the networks"
    am, asd = ppo.adv_stats(data["adv"])
    # the production shape checks one minibatch (its float64 checks take ~1 min)
    pairs = ((0, 0),) if T * N >= 65536 else ((0, 0), (1, mbs - 1))
    for ep, mb in pairs:
        res = _gpu_minibatch(ctx, d, p, ep, mb, batch)
        _check_stages(res, d, data, _minibatch_of(perm, ep, mb, mbs), p, am, asd)
    ctx.close()


# networks of different depths and widths: levels that only one of the two has,
# and levels whose tile shapes differ (two launches instead of one)
@pytest.mark.parametrize("actor,critic", [
    ([226, 384, 256, 28], [226, 256, 512, 384, 1]),
    ([226, 512, 128, 256, 28], [226, 512, 1]),
    ([226, 28], [226, 256, 256, 1])])
def test_minibatch_gradient_of_unlike_networks(actor, critic):
    N, T = 192, 2
    d, data, summary = _rollout(3, N, T, actor=actor, critic=critic)
    p = dict(binding.PPO_DEFAULTS, epochs=1, minibatches=1)
    ctx = binding.Context(d, max_envs=N)
    ctx.ppo_setup(N * T)
    ro = _upload(ctx, data, summary, N, T)
    perm = _perm(1, T * N // 64, 3)
    gperm, lr = torch.from_numpy(perm).cuda(), torch.full((1,), 1e-3, device="cuda")
    batch = binding.ppo_batch(ro, gperm, lr)
    res = _gpu_minibatch(ctx, d, p, 0, 0, batch)
    am, asd = ppo.adv_stats(data["adv"])
    _check_stages(res, d, data, _minibatch_of(perm, 0, 0, 1), p, am, asd)
    ctx.close()


# both sides of the sample count where the critic's output layer takes more
# samples per thread; 300 rows, a remainder of either's chunks
@pytest.mark.parametrize("N", [130816, 131392])
def test_critic_output_by_sample_count(N):
    print("critic output of %d samples" % N, flush=True)
    d = synth.make_world(3, n_envs=64)
    d["policy"] = synth.make_policy(np.random.default_rng(1), [226, 64, 28], True)
    d["critic"] = synth.make_policy(np.random.default_rng(2), [226, 300, 1], True)
    ctx = binding.Context(d, max_envs=N)
    ctx.ppo_setup(N)
    ro = binding.RolloutStorage(ctx, N, 1)
    gen = torch.Generator("cuda").manual_seed(N)
    for x in (ro.obs, ro.action, ro.mean, ro.logp, ro.value, ro.advantage, ro.ret):
        x.copy_(torch.randn(x.shape, generator=gen, device="cuda"))
    ro.summary.zero_()
    perm = torch.arange(N // 64, dtype=torch.int32, device="cuda")[None]
    batch = binding.ppo_batch(ro, perm, torch.full((1,), 1e-3, device="cuda"))
    g = torch.empty(ctx.ppo_params(), device="cuda")
    ctx.ppo_grad(batch, binding.ppo_params(**dict(binding.PPO_DEFAULTS, epochs=1, minibatches=1)), 0, 0, g)
    h = ctx.ppo_read("critic_hidden", 0)[:300].double()
    v = ctx.ppo_read("value")[0].double()
    torch.cuda.synchronize()
    w = torch.from_numpy(np.asarray(d["critic"]["W"][1][0], np.float64)).cuda()
    b = float(d["critic"]["b"][1][0])
    ref = (w[:, None] * h).sum(0) + b
    bound = 302 * U32 * ((w.abs()[:, None] * h.abs()).sum(0) + abs(b)) + U32 * ref.abs()
    assert v.shape[0] == (N + 255) // 256 * 256
    assert bool(((v - ref).abs() <= bound).all()), float(((v - ref).abs() / bound).max())
    assert float(ref.std()) > 0.01
    ctx.close()


def test_adam_step_on_the_gpu_gradient():
    # one epoch of one minibatch: the update is one norm clip + Adam step on the
    # minibatch gradient; the oracle's step on the GPU's own gradient, element
    # by element (float32 masters: a few float32 spacings of the result)
    cfg, N, T = 3, 256, 2
    d, data, summary = _rollout(cfg, N, T)
    ctx = binding.Context(d, max_envs=N)
    n_chunks = T * N // 64
    ctx.ppo_setup(n_chunks * 64)
    ro = _upload(ctx, data, summary, N, T)
    perm = _perm(1, n_chunks, 9)
    lr = torch.full((1,), 1e-3, device="cuda")
    p = dict(binding.PPO_DEFAULTS, epochs=1, minibatches=1, desired_kl=0.0, max_grad_norm=0.5)
    batch = binding.ppo_batch(ro, torch.from_numpy(perm).cuda(), lr)
    P_ = ctx.ppo_params()
    g = torch.zeros(P_, device="cuda")
    ctx.ppo_grad(batch, binding.ppo_params(**p), 0, 0, g)
    ctx.ppo_update(batch, binding.ppo_params(**p))
    x1 = torch.empty(P_, device="cuda")
    ctx.ppo_params(x1)
    torch.cuda.synchronize()
    x0 = ppo.flat_params(d["policy"], d["critic"]).astype(np.float64)
    gg = g.cpu().numpy().astype(np.float64)
    xo, _, _ = ppo.adam_step(x0, gg, np.zeros_like(x0), np.zeros_like(x0), 1, 1e-3, p)
    xg = x1.cpu().numpy().astype(np.float64)
    tol = 4 * np.spacing(np.abs(xo).astype(np.float32)).astype(np.float64) + 1e-6 * 1e-3
    bad = np.abs(xg - xo) > tol
    assert not bad.any(), "%d parameters, e.g. %s" % (int(bad.sum()), np.flatnonzero(bad)[:5])
    ctx.close()


def _cos(a, b):
    return float(np.dot(a, b) / max(np.linalg.norm(a) * np.linalg.norm(b), 1e-30))


def test_update_matches_oracle():
    cfg, N, T = 3, 256, 2
    d, data, summary = _rollout(cfg, N, T)
    ctx = binding.Context(d, max_envs=N)
    n_chunks = T * N // 64
    p = dict(binding.PPO_DEFAULTS, epochs=2, minibatches=2, desired_kl=0.0)
    ctx.ppo_setup(n_chunks // 2 * 64)
    ro = _upload(ctx, data, summary, N, T)
    perm = _perm(2, n_chunks, 5)
    lr = torch.full((1,), 1e-3, device="cuda")
    stats = torch.zeros(len(binding.PPO_STATS), dtype=torch.float64, device="cuda")
    batch = binding.ppo_batch(ro, torch.from_numpy(perm).cuda(), lr, stats)
    ctx.ppo_update(batch, binding.ppo_params(**p))
    x = torch.empty(ctx.ppo_params(), device="cuda")
    ctx.ppo_params(x)
    torch.cuda.synchronize()
    pol, crit = d["policy"], d["critic"]
    a, c, olr, recs = ppo.update(pol, crit, data, perm, p, 1e-3)
    x0 = ppo.flat_params(pol, crit).astype(np.float64)
    dg = x.cpu().numpy().astype(np.float64) - x0
    do = ppo.flat_params(a, c).astype(np.float64) - x0
    for name, sl in _segments(pol, crit):
        cs = _cos(dg[sl], do[sl])
        ratio = np.linalg.norm(dg[sl]) / np.linalg.norm(do[sl])
        print("%-10s cos %.4f norm ratio %.4f" % (name, cs, ratio))
        # a tensor of a few elements (the critic's output bias) moves by lr times
        # m / sqrt(v) of gradients that are cancelling sums: its step length is
        # sensitive to the forward's rounding and only its direction is compared
        # (the Adam arithmetic itself is checked element by element on the GPU's
        # own gradient in test_adam_step_on_the_gpu_gradient)
        assert cs >= 0.97, name
        if dg[sl].size >= 16:
            assert abs(ratio - 1.0) <= 0.05, name
    s = stats.cpu().numpy()
    assert s[5] == 4 and s[6] == pytest.approx(1e-3, rel=1e-6)
    for k, key in ((0, "l_pi"), (1, "l_v"), (2, "kl"), (3, "clipfrac")):
        o = sum(r[key] for r in recs)
        assert abs(s[k] - o) <= 5e-2 * abs(o) + 1e-3, (key, s[k], o)
    ctx.close()


@pytest.mark.parametrize("desired_kl,expect", [(1e-9, 2e-4), (1e7, 3e-3)])
def test_kl_adaptive_learning_rate(desired_kl, expect):
    # a KL threshold far below (above) every minibatch's KL: the rate falls
    # (rises) by 1.5 at each of the 4 steps, down to lr_min (up to lr_max)
    cfg, N, T = 3, 256, 2
    d, data, summary = _rollout(cfg, N, T)
    ctx = binding.Context(d, max_envs=N)
    n_chunks = T * N // 64
    p = dict(binding.PPO_DEFAULTS, epochs=2, minibatches=2, desired_kl=desired_kl, lr_min=2e-4,
             lr_max=3e-3)
    ctx.ppo_setup(n_chunks // 2 * 64)
    ro = _upload(ctx, data, summary, N, T)
    perm = _perm(2, n_chunks, 6)
    lr = torch.full((1,), 1e-3, device="cuda")
    ctx.ppo_update(binding.ppo_batch(ro, torch.from_numpy(perm).cuda(), lr), binding.ppo_params(**p))
    _, _, olr, recs = ppo.update(d["policy"], d["critic"], data, perm, p, 1e-3)
    torch.cuda.synchronize()
    assert olr == pytest.approx(expect)
    assert lr.item() == pytest.approx(olr, rel=1e-6)
    ctx.close()


def test_update_is_deterministic_refreshes_the_rollout_copies_and_replays_as_a_graph():
    cfg, N, T = 6, 192, 2
    d, data, summary = _rollout(cfg, N, T)
    n_chunks = T * N // 64
    p = binding.ppo_params(epochs=1, minibatches=2)
    perm = torch.from_numpy(_perm(1, n_chunks, 7)).cuda()

    def run(graph=False):
        ctx = binding.Context(d, max_envs=N)
        ctx.ppo_setup(n_chunks // 2 * 64 + 64)
        ro = _upload(ctx, data, summary, N, T)
        lr = torch.full((1,), 1e-3, device="cuda")
        batch = binding.ppo_batch(ro, perm, lr)
        if graph:
            g = torch.cuda.CUDAGraph()
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                with torch.cuda.graph(g, stream=side):
                    ctx.ppo_update(batch, p)
            torch.cuda.current_stream().wait_stream(side)
            torch.cuda.synchronize()
            g.replay()
        else:
            ctx.ppo_update(batch, p)
        x = torch.empty(ctx.ppo_params(), device="cuda")
        ctx.ppo_params(x)
        # the rollout calls use the trained weights
        obs = ro.obs[0]
        mean = torch.empty((N, d["policy"]["dims"][-1]), device="cuda")
        act = torch.empty_like(mean)
        v = torch.empty(N, device="cuda")
        env_n = torch.zeros(N, dtype=torch.int32, device="cuda")
        ctx.policy_act(obs, env_n, N, mean, act, None)
        ctx.value(obs, N, v)
        torch.cuda.synchronize()
        out = (x.cpu().numpy(), mean.cpu().numpy(), v.cpu().numpy())
        ctx.close()
        return out

    x1, m1, v1 = run()
    x2, m2, v2 = run()
    x3, m3, v3 = run(graph=True)
    assert np.array_equal(x1, x2) and np.array_equal(m1, m2) and np.array_equal(v1, v2)
    assert np.array_equal(x1, x3) and np.array_equal(m1, m3) and np.array_equal(v1, v3)
    x0 = ppo.flat_params(d["policy"], d["critic"])
    assert not np.array_equal(x1, x0)
    # a context built from the trained masters gives the same rollout outputs
    a, c = ppo.unflat(x1, d["policy"], d["critic"])
    a = dict(a, W=[synth.bf16_round(w) for w in a["W"]])
    c = dict(c, W=[synth.bf16_round(w) for w in c["W"]])
    ctx = binding.Context(dict(d, policy=a, critic=c), max_envs=N)
    ro = _upload(ctx, data, summary, N, T)
    mean = torch.empty((N, d["policy"]["dims"][-1]), device="cuda")
    act = torch.empty_like(mean)
    v = torch.empty(N, device="cuda")
    ctx.policy_act(ro.obs[0], torch.zeros(N, dtype=torch.int32, device="cuda"), N, mean, act, None)
    ctx.value(ro.obs[0], N, v)
    torch.cuda.synchronize()
    assert np.array_equal(mean.cpu().numpy(), m1) and np.array_equal(v.cpu().numpy(), v1)
    ctx.close()


def test_ppo_validation():
    d = synth.make_world(2, n_envs=128)
    ctx = binding.Context(d, max_envs=128)
    with pytest.raises(binding.ImError, match="bf16"):
        ctx.ppo_setup(128)
    ctx.close()
    d = synth.make_world(3, n_envs=128)
    ctx = binding.Context(d, max_envs=128)
    ro = binding.RolloutStorage(ctx, 128, 2)
    perm = torch.zeros((1, 4), dtype=torch.int32, device="cuda")
    lr = torch.full((1,), 1e-3, device="cuda")
    with pytest.raises(binding.ImError, match="im_ppo_setup"):
        ctx.ppo_update(binding.ppo_batch(ro, perm, lr), binding.ppo_params(epochs=1))
    ro = binding.RolloutStorage(ctx, 128, 4)          # 8 chunks of 64 envs
    perm = torch.zeros((1, 8), dtype=torch.int32, device="cuda")
    ctx.ppo_setup(128)                                  # minibatches of up to 256 samples
    for over, words in ((dict(epochs=1, minibatches=1), "exceeds"),
                        (dict(epochs=1, minibatches=9), "more minibatches"),
                        (dict(epochs=1, minibatches=2, clip=0.0), "clip"),
                        (dict(epochs=1, minibatches=2, beta1=1.0), "betas"),
                        (dict(epochs=1, minibatches=2, lr_min=1.0, lr_max=0.1), "lr_min")):
        with pytest.raises(binding.ImError, match=words):
            ctx.ppo_update(binding.ppo_batch(ro, perm, lr), binding.ppo_params(**over))
    ro96 = binding.RolloutStorage(ctx, 96, 2)
    with pytest.raises(binding.ImError, match="multiple of 64"):
        ctx.ppo_update(binding.ppo_batch(ro96, perm, lr), binding.ppo_params(epochs=1, minibatches=2))
    ctx.close()


def test_ppo_setup_rejects_operands_of_4_gib():
    # the training GEMMs address [rows][minibatch] bf16 operands with 32-bit
    # extents: 1024-wide layers reach 4 GiB at 2^21 samples; the setup refuses
    # that size before touching the training state (an existing one survives)
    d = synth.make_world(4, n_envs=128)
    ctx = binding.Context(d, max_envs=128)
    ctx.ppo_setup(128)
    with pytest.raises(binding.ImError, match="4 GiB") as ei:
        ctx.ppo_setup(1 << 21)
    assert ei.value.status == binding.IM_ERR_UNSUPPORTED
    ro = binding.RolloutStorage(ctx, 128, 1)
    perm = torch.arange(2, dtype=torch.int32, device="cuda")[None]
    lr = torch.full((1,), 1e-3, device="cuda")
    ctx.ppo_update(binding.ppo_batch(ro, perm, lr), binding.ppo_params(epochs=1, minibatches=1))
    torch.cuda.synchronize()
    ctx.close()


def test_ppo_setup_memory():
    """im_get_info counts the training state, and it is what the header says:
    the hidden units and their masks, two gradient buffers per network, the
    split sums (at most 1024 tiles and one round more), and per sample the
    observation, the rollout's columns and the outputs."""
    Mb, hidden = 131072, 1024 + 1024 + 512
    d = synth.make_world(4, n_envs=128)
    dims = [d["policy"]["W"][0].shape[1], 1024, 1024, 512]
    A = d["policy"]["W"][-1].shape[0]
    d["policy"] = synth.make_policy(np.random.default_rng(1), dims + [A], True)
    d["critic"] = synth.make_policy(np.random.default_rng(2), dims + [1], True)
    ctx = binding.Context(d, max_envs=128)
    before = binding.im_get_info(ctx.ptr).device_bytes
    ctx.ppo_setup(Mb)
    grown = binding.im_get_info(ctx.ptr).device_bytes - before
    ctx.close()
    state = 2 * hidden * Mb * 17 // 8 + 4 * 1024 * Mb * 2
    print("training state %d bytes, activations and gradients %d" % (grown, state), flush=True)
    inputs = Mb * (2 * 384 + 2 * 128 + 4 * (3 * A + 8)) + 2 * 1024 * 8 * (Mb // 128 + 1) + 1024 * 8 * (Mb // 2048 + 1)
    # per weight, padded: master, two moments, gradient (fp32), two bf16 copies
    weights = (2 * (384 * 1024 + 1024 * 1024 + 1024 * 512) + 512 * 128) * 20
    assert state + inputs <= grown <= state + inputs + 2 * (1024 + 64) * 65536 + weights + (4 << 20)
