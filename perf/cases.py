"""The work that a training program has this framework do, as measured cases.

One rollout step of a tracking policy is a policy call (`policy_act`, or
`policy_act_value` while a rollout is collected), the physics, and one fused
env step; a rollout ends with GAE and its summaries, and a PPO update follows.
The cases are those calls, each through the binding, at the sizes of the
benchmark workloads (S15 and S24 humanoids, 64 to 262144 envs):

  act      policy_act / policy_act_value on an observation batch
  step     env_step_fused on a batch whose physics has just run: most envs
           track their clip, a share has fallen and is reset
  gae      GAE and rollout summaries over a T-step storage
  update   ppo_update: all epochs and minibatches over a rollout, and the
           weights it leaves
  grad     ppo_grad: one minibatch's gradient (drawn cases only)

`exact` is the same arithmetic in float64 torch, written from the C header's
description of each call.
"""
import math

import numpy as np
import torch

from paper_2609_09821_amd import binding, synth

DEV = "cuda"

# observation width, hidden widths and action width of the benchmark workloads
NETS = {
    "s15": [226, 1024, 512, 28],
    "s24": [361, 1024, 1024, 512, 69],
    "s24t": [538, 1024, 1024, 512, 69],   # training terms: 2 future frames, previous action
}
TRAIN = dict(reward_form=1, h_term=0.8, grace=4, r_min=synth.R_MIN_6, obs_future=2,
             obs_prev_action=1)
SIGMA = 0.05          # action standard deviation
LR = 1e-5             # the adaptive schedule's floor, where a tracking run spends its time


def listed():
    return [
        # a player or an evaluation: a handful of envs, one step at a time; launch latency
        dict(name="act_f32_s15_64", kind="act", net="s15", bf16=False, value=False, n=64, ld=64),
        # the small training batch in full precision
        dict(name="act_f32_s15_4096", kind="act", net="s15", bf16=False, value=False, n=4096,
             ld=4096),
        # rollout step of an ordinary training batch: action, logp and value
        dict(name="actv_bf16_s24_4096", kind="act", net="s24", bf16=True, value=True, n=4096,
             ld=4096),
        # an odd batch in a padded buffer (envs taken out of a batch of 16384)
        dict(name="actv_bf16_s15_16381", kind="act", net="s15", bf16=True, value=True, n=16381,
             ld=16384),
        # the large batch: policy of the headline workload
        dict(name="act_bf16_s24_65536", kind="act", net="s24", bf16=True, value=False, n=65536,
             ld=65536),
        # env step of the small training batch
        dict(name="step_s15_4096", kind="step", skel="s15", train=False, clips=1, n=4096, ld=4096),
        # env step with the training reward, future frames and previous action, odd batch
        dict(name="step_s24_train_16381", kind="step", skel="s24", train=True, clips=1, n=16381,
             ld=16384),
        # env step of the headline workload
        dict(name="step_s24_65536", kind="step", skel="s24", train=False, clips=1, n=65536,
             ld=65536),
        # the largest batch, 16 clips
        dict(name="step_s15_262144", kind="step", skel="s15", train=False, clips=16, n=262144,
             ld=262144),
        # end of a rollout of the headline workload
        dict(name="gae_65536x32", kind="gae", T=32, n=65536, ld=65536),
        # PPO update of a small training batch: minibatches of 32768 samples
        dict(name="update_s15_4096x32", kind="update", net="s15", n=4096, T=32, epochs=5,
             minibatches=4),
        # PPO update of the headline workload: minibatches of 524288 samples
        dict(name="update_s24_65536x32", kind="update", net="s24", n=65536, T=32, epochs=5,
             minibatches=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["act", "act", "act", "step", "step", "gae", "update", "grad"])
    if kind == "act":
        bf16 = rng.random() < 0.7
        net = rng.choice(["s15", "s24", "s24t"]) if bf16 else "s15"
        n = _log_int(rng, 64, 65536 if bf16 else 16384)
        return dict(kind=kind, net=net, bf16=bf16, value=rng.random() < 0.5, n=n,
                    ld=n + rng.choice([0, 0, 3, 64]))
    if kind == "step":
        skel = rng.choice(["s15", "s24"])
        n = _log_int(rng, 64, 262144 if skel == "s15" else 131072)
        return dict(kind=kind, skel=skel, train=skel == "s24" and rng.random() < 0.5,
                    clips=rng.choice([1, 3, 16]), n=n, ld=n + rng.choice([0, 0, 3, 64]))
    if kind == "gae":
        n = _log_int(rng, 64, 262144)
        return dict(kind=kind, T=rng.randint(8, 48), n=n, ld=n + rng.choice([0, 0, 3, 64]))
    net = rng.choice(["s15", "s24", "s24t"])
    n = 64 * _log_int(rng, 4, 256)
    T = rng.randint(8, 32)
    if kind == "update":
        return dict(kind=kind, net=net, n=n, T=T, epochs=rng.randint(1, 5),
                    minibatches=rng.randint(2, 8))
    return dict(kind=kind, net=net, n=n, T=T, minibatches=rng.randint(2, 8))


# ------------------------------------------------------------------ inputs
def _rng(seed, *more):
    return np.random.default_rng(np.random.SeedSequence([2609, int(seed)] + list(more)))


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) + 1)


def _skeleton(name, rng):
    return synth.skeleton_s15(rng) if name == "s15" else synth.skeleton_s24(rng)


def _net(case, seed):
    dims = NETS[case["net"]]
    bf16 = case.get("bf16", True)
    actor = synth.make_policy(_rng(seed, 1), dims, bf16, SIGMA)
    critic = synth.make_policy(_rng(seed, 2), dims[:-1] + [1], bf16)
    return actor, critic


def _world(skel_name, train, n_clips, seed, actor, critic):
    """Description of a world: skeleton, clips, config and networks."""
    rng = _rng(seed, 3)
    skel = _skeleton(skel_name, rng)
    frames = [300] if n_clips == 1 else [int(f) for f in rng.integers(60, 301, size=n_clips)]
    clips = [synth.make_clip(rng, skel, f) for f in frames]
    cfg = synth.step_config(0, seed=synth.SEED_BASE + int(seed), **(TRAIN if train else {}))
    return dict(skeleton=skel, clips=clips, policy=actor, critic=critic, config=cfg)


def _tiny_nets(dims, seed):
    """Networks of a world whose policy is not called (narrow hidden layer)."""
    d = [dims[0], 32, dims[-1]]
    return synth.make_policy(_rng(seed, 1), d, True, SIGMA), None


def _act_inputs(case, seed):
    g = _gen(seed)
    D = NETS[case["net"]][0]
    # unit-scale features, as heading-frame positions, rotation columns and velocities are
    obs = torch.randn((D, case["ld"]), generator=g, device=DEV)
    env_n = torch.randint(0, 1 << 20, (case["ld"],), generator=g, device=DEV, dtype=torch.int32)
    return obs, env_n


def _step_inputs(case, seed):
    """The env state and the sim state after the physics, from the seed: the
    reference at the next phase with tracking noise; three envs in ten have
    fallen (below the termination height), some clips end."""
    g = _gen(seed)
    n, ld = case["n"], case["ld"]
    dims = NETS["s24t" if case["train"] else case["skel"]]
    actor, critic = _tiny_nets(dims, seed)
    desc = _world(case["skel"], case["train"], case["clips"], seed, actor, critic)
    ref = _Reference(desc)
    A = dims[-1]
    st = dict(
        clip=torch.randint(0, len(desc["clips"]), (n,), generator=g, device=DEV, dtype=torch.int32),
        phase=torch.rand(n, generator=g, device=DEV),
        t=torch.randint(0, 100, (n,), generator=g, device=DEV, dtype=torch.int32),
        n=torch.randint(0, 1 << 20, (n,), generator=g, device=DEV, dtype=torch.int32),
        prev=0.3 * torch.randn((n, A), generator=g, device=DEV) if case["train"] else None)
    ph = torch.clamp(st["phase"] + ref.dphi[st["clip"].long()], max=1.0)
    P, Q, V, W = ref.state(st["clip"], ph)[:4]
    rot, vel = (0.01, 0.05) if case["train"] else (0.05, 0.1)

    def noise(x, s):
        return s * torch.randn(x.shape, generator=g, device=DEV).double()
    fallen = (torch.rand(n, generator=g, device=DEV) < 0.3).double()
    st["pos"] = P + noise(P, 0.005)
    st["pos"][..., 2] -= 0.8 * fallen[:, None]
    st["quat"] = _qmul(Q, _qexp(noise(P, rot)))
    st["linvel"] = V + noise(V, vel)
    st["angvel"] = W + noise(W, vel)
    for k in ("pos", "quat", "linvel", "angvel"):        # [n][B][c] -> [B][c][n]
        st[k] = st[k].permute(1, 2, 0).float().contiguous()
    return desc, ref, st


def _gae_inputs(case, seed):
    g = _gen(seed)
    T, ld = case["T"], case["ld"]
    r = lambda *s: torch.rand(s, generator=g, device=DEV)  # noqa: E731
    return dict(reward=r(T, ld), term=(r(T, ld) < 0.04).to(torch.uint8),
                trunc=(r(T, ld) < 0.02).to(torch.uint8),
                value=2.0 * torch.randn((T + 1, ld), generator=g, device=DEV),
                ep_return=5.0 * r(ld),
                ep_length=torch.randint(0, 50, (ld,), generator=g, device=DEV, dtype=torch.int32))


def _forward(net, x, dt):
    """A bf16 network's output in dtype `dt` from x [m][D]: input and hidden
    activations rounded to bf16 where dt is float64."""
    r = (lambda t: t.float().bfloat16().double()) if dt == torch.float64 else (lambda t: t)
    h = r(x)
    for l, (w, b) in enumerate(zip(net["W"], net["b"])):
        h = torch.addmm(b, h, w.t())
        if l < len(net["W"]) - 1:
            h = r(torch.relu(h))
    return h


def _on_gpu(net, dt):
    return dict(W=[torch.from_numpy(np.asarray(w)).to(DEV, dt) for w in net["W"]],
                b=[torch.from_numpy(np.asarray(b)).to(DEV, dt) for b in net["b"]])


def _rollout_inputs(case, seed, actor, critic):
    """A collected rollout: the actions of the policy (its means up to the
    rounding of its layers), advantages and returns around the critic's values."""
    g = _gen(seed)
    T, n = case["T"], case["n"]
    D, A = NETS[case["net"]][0], NETS[case["net"]][-1]
    a, c = _on_gpu(actor, torch.float32), _on_gpu(critic, torch.float32)
    d = dict(obs=torch.randn((T + 1, D, n), generator=g, device=DEV))
    f = dict(device=DEV, dtype=torch.float32)
    d["mean"], d["value"] = torch.empty((T, n, A), **f), torch.empty((T + 1, n), **f)
    for t in range(T + 1):
        x = d["obs"][t].t()
        if t < T:
            d["mean"][t] = _forward(a, x, torch.float32)
        d["value"][t] = _forward(c, x, torch.float32)[:, 0]
    z = torch.randn((T, n, A), generator=g, device=DEV)
    d["action"] = d["mean"] + SIGMA * z
    ls = float(np.float32(math.log(SIGMA)))
    d["logp"] = (-(0.5 * z.double() ** 2 + ls + 0.5 * math.log(2 * math.pi)).sum(-1)).float()
    d["adv"] = torch.randn((T, n), generator=g, device=DEV)
    d["ret"] = d["value"][:T] + d["adv"]
    chunks = T * n // 64
    d["perm"] = torch.stack([torch.randperm(chunks, generator=g, device=DEV)
                             for _ in range(case.get("epochs", 1))]).to(torch.int32)
    return d


# ----------------------------------------------------------------- program
def prepare(case, seed):
    return {"act": _prepare_act, "step": _prepare_step, "gae": _prepare_gae,
            "update": _prepare_ppo, "grad": _prepare_ppo}[case["kind"]](case, seed)


def _context(case, seed, max_envs):
    actor, critic = _net(case, seed)
    skel = case["net"][:3]
    desc = _world(skel, case["net"] == "s24t", 1, seed, actor, critic)
    return binding.Context(desc, max_envs), actor, critic


def _prepare_act(case, seed):
    ctx = _context(case, seed, case["n"])[0]
    obs, env_n = _act_inputs(case, seed)
    n, A = case["n"], NETS[case["net"]][-1]
    f = dict(device=DEV, dtype=torch.float32)
    return dict(case=case, ctx=ctx, obs=obs, env_n=env_n, mean=torch.zeros((n, A), **f),
                action=torch.zeros((n, A), **f), logp=torch.zeros(n, **f),
                value=torch.zeros(n, **f))


def _prepare_step(case, seed):
    desc, _, st = _step_inputs(case, seed)
    ctx = binding.Context(desc, case["n"], critic=False)
    b = ctx.buffers(case["n"], case["ld"])
    n = case["n"]
    for k in ("pos", "quat", "linvel", "angvel"):
        getattr(b, "body_" + k)[:, :, :n] = st[k]
    for k in ("clip", "phase", "t", "n"):
        getattr(b, "env_" + k)[:n] = st[k]
    if st["prev"] is not None:
        b.prev_action.copy_(st["prev"])
    return dict(case=case, ctx=ctx, bufs=b)


def _prepare_gae(case, seed):
    actor, critic = _tiny_nets(NETS["s15"], seed)
    ctx = binding.Context(_world("s15", False, 1, seed, actor, critic), case["n"], critic=False)
    ro = binding.RolloutStorage(ctx, case["n"], case["T"], case["ld"])
    ro.obs = ro.mean = ro.action = None      # GAE reads the per-step scalars only
    d = _gae_inputs(case, seed)
    for k, v in (("reward", "reward"), ("terminated", "term"), ("truncated", "trunc"),
                 ("value", "value"), ("ep_return", "ep_return"), ("ep_length", "ep_length")):
        getattr(ro, k).copy_(d[v])
    return dict(case=case, ctx=ctx, ro=ro)


def _minibatch_samples(case):
    chunks = case["T"] * case["n"] // 64
    return 64 * -(-chunks // case["minibatches"])


def _prepare_ppo(case, seed):
    ctx, actor, critic = _context(case, seed, case["n"])
    ro = binding.RolloutStorage(ctx, case["n"], case["T"])
    d = _rollout_inputs(case, seed, actor, critic)
    for k in ("obs", "mean", "action", "logp", "value", "ret"):
        setattr(ro, k, d[k])
    ro.advantage = d["adv"]
    ro.summary[binding.SUMMARY_FIELDS.index("advantage_sum")] = d["adv"].double().sum()
    ro.summary[binding.SUMMARY_FIELDS.index("advantage_sq_sum")] = d["adv"].double().square().sum()
    ctx.ppo_setup(_minibatch_samples(case))
    lr = torch.full((1,), LR, device=DEV)
    stats = torch.zeros(len(binding.PPO_STATS), device=DEV, dtype=torch.float64)
    out = torch.zeros(ctx.ppo_params(), device=DEV)
    params = binding.ppo_params(epochs=case.get("epochs", 1), minibatches=case["minibatches"],
                                desired_kl=0.0)
    return dict(case=case, ctx=ctx, ro=ro, perm=d["perm"], lr=lr, stats=stats, out=out,
                params=params, batch=binding.ppo_batch(ro, d["perm"], lr, stats))


def run(s):
    c, ctx = s["case"], s["ctx"]
    kind = c["kind"]
    if kind == "act":
        if c["value"]:
            ctx.policy_act_value(s["obs"], s["env_n"], c["n"], s["mean"], s["action"], s["logp"],
                                 s["value"])
            return s["mean"], s["action"], s["logp"], s["value"]
        ctx.policy_act(s["obs"], s["env_n"], c["n"], s["mean"], s["action"], s["logp"])
        return s["mean"], s["action"], s["logp"]
    if kind == "step":
        b, n = s["bufs"], c["n"]
        ctx.env_step_fused(b)
        return dict(reward=b.reward[:n], terminated=b.terminated[:n], truncated=b.truncated[:n],
                    ref_frame=b.ref_frame[:n], clip=b.env_clip[:n], phase=b.env_phase[:n],
                    t=b.env_t[:n], n=b.env_n[:n], obs=b.obs[:, :n], pos=b.body_pos[:, :, :n],
                    quat=b.body_quat[:, :, :n], linvel=b.body_linvel[:, :, :n],
                    angvel=b.body_angvel[:, :, :n])
    if kind == "gae":
        ro, n = s["ro"], c["n"]
        ctx.gae(ro, synth.GAMMA, synth.LAMBDA)
        return dict(adv=ro.advantage[:, :n], ret=ro.ret[:, :n], ep_return=ro.ep_return[:n],
                    ep_length=ro.ep_length[:n], summary=ro.summary)
    if kind == "update":
        ctx.ppo_update(s["batch"], s["params"])
        ctx.ppo_params(s["out"])
        return dict(weights=s["out"], stats=s["stats"], lr=s["lr"])
    ctx.ppo_grad(s["batch"], s["params"], 0, c["minibatches"] - 1, s["out"], s["stats"])
    return dict(grad=s["out"], stats=s["stats"])


# -------------------------------------------------------------------- work
def work(case):
    kind, n = case["kind"], case["n"]
    if kind == "step":
        B = 15 if case["skel"] == "s15" else 24
        D = NETS["s24t" if case["train"] else case["skel"]][0]
        A = NETS["s24"][-1] if case["train"] else 0
        # sim state in, env state in and out, reward, flags, frame, observation out,
        # and the state of the envs reset (a tenth of the batch)
        per_env = 52 * B + 32 + 4 + 2 + 4 + 4 * D + 4 * A + 0.1 * 52 * B
        return dict(bytes=n * per_env, flops=n * B * 400)
    if kind == "gae":
        # reward, flags, value in; advantage, return out; accumulators in and out
        return dict(bytes=case["T"] * n * 18 + n * 20, flops=case["T"] * n * 12)
    dims = NETS[case["net"]]
    D, A = dims[0], dims[-1]
    mac = sum(i * o for i, o in zip(dims[:-1], dims[1:]))
    vmac = mac - dims[-2] * A + dims[-2]
    if kind == "act":
        eb = 2 if case["bf16"] else 4
        v = case["value"]
        return dict(bytes=n * 4 * (D + 1 + 2 * A + 1 + v) + eb * (mac + (vmac if v else 0)),
                    flops=2.0 * n * (mac + (vmac if v else 0)))
    if kind == "update":
        samples, steps = case["epochs"] * case["T"] * n, case["epochs"] * case["minibatches"]
    else:
        samples, steps = case["T"] * n // case["minibatches"], 1
    # forward, input gradient (not of the first layer) and weight gradient of both networks;
    # observation, action, mean and four scalars per sample; weights and Adam moments per step
    flops = 2.0 * samples * (3 * (mac + vmac) - 2 * D * dims[1])
    return dict(bytes=samples * 4.0 * (D + 2 * A + 4) + steps * 24.0 * (mac + vmac), flops=flops)


def tolerance(case):
    """About four times the distance of the calls from float64 (`exact`), measured."""
    kind = case["kind"]
    if kind == "act":
        # bf16 (1.7e-4 for the mean, 3.2e-4 for the value): a different order of the fp32
        # sums moves hidden activations across bf16 ties; fp32: 5.3e-7
        return {"rel": 1.5e-3, "max": 3e-2} if case["bf16"] else {"rel": 2.5e-6, "max": 1e-4}
    if kind == "step":       # 1.4e-7 (the reward)
        return {"rel": 1e-6, "max": 1e-4}
    if kind == "gae":        # 8e-8 (the fp32 running return)
        return {"rel": 5e-7, "max": 1e-5}
    if kind == "update":     # weights 7e-5, statistics 3.5e-3 (the gradient norm's bf16 backward)
        return {"rel": 4e-3, "max": 1e-1}
    return {"rel": 1e-2, "max": 3e-1}     # gradient 2.5e-3


# ------------------------------------------------------------ float64 truth
def exact(case, seed):
    kind = case["kind"]
    if kind == "update" and case["T"] * case["n"] * case["epochs"] > 1 << 20:
        return None
    with torch.no_grad():
        return {"act": _exact_act, "step": _exact_step, "gae": _exact_gae, "update": _exact_ppo,
                "grad": _exact_ppo}[kind](case, seed)


def _mulhi(a, b):
    a0, a1, b0, b1 = a & 0xFFFF, a >> 16, b & 0xFFFF, b >> 16
    mid = a1 * b0 + ((a0 * b0) >> 16)
    mid2 = a0 * b1 + (mid & 0xFFFF)
    return a1 * b1 + (mid >> 16) + (mid2 >> 16)


def _philox(c, seed):
    """Philox4x32-10 (Salmon et al., SC'11) on int64 tensors of 32-bit words."""
    c = [torch.as_tensor(x, device=DEV, dtype=torch.int64) & 0xFFFFFFFF for x in c]
    c = list(torch.broadcast_tensors(*c))
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    m0, m1 = 0xD2511F53, 0xCD9E8D57
    for _ in range(10):
        h0, l0 = _mulhi(c[0], m0), (c[0] * m0) & 0xFFFFFFFF
        h1, l1 = _mulhi(c[2], m1), (c[2] * m1) & 0xFFFFFFFF
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _normals(n, env_n, A, seed):
    """z [n][A] of the policy's action noise: counter (env, env_n, j, 0)."""
    nb = -(-A // 4)
    e = torch.arange(n, device=DEV)[:, None]
    x = _philox([e, env_n[:n].long()[:, None], torch.arange(nb, device=DEV)[None, :], 0], seed)
    u = [(2.0 * (w >> 9).double() + 1.0) * 2.0 ** -24 for w in x]
    z = []
    for h in (0, 2):
        r = torch.sqrt(-2.0 * torch.log(u[h]))
        z += [r * torch.cos(2 * math.pi * u[h + 1]), r * torch.sin(2 * math.pi * u[h + 1])]
    return torch.stack(z, -1).reshape(n, 4 * nb)[:, :A]


def _exact_act(case, seed):
    actor, critic = _net(case, seed)
    obs, env_n = _act_inputs(case, seed)
    n, A = case["n"], NETS[case["net"]][-1]
    x = obs[:, :n].t().double()
    cfg_seed = synth.SEED_BASE + int(seed)

    def mlp(net):
        net = _on_gpu(net, torch.float64)
        if case["bf16"]:
            return _forward(net, x, torch.float64)
        h = x
        for l, (w, b) in enumerate(zip(net["W"], net["b"])):
            h = torch.addmm(b, h, w.t())
            h = torch.relu(h) if l < len(net["W"]) - 1 else h
        return h
    mean = mlp(actor)
    ls = torch.from_numpy(actor["log_std"]).to(DEV, torch.float64)
    z = _normals(n, env_n, A, cfg_seed)
    out = [mean, mean + torch.exp(ls) * z,
           -(0.5 * z * z + ls + 0.5 * math.log(2 * math.pi)).sum(1)]
    return tuple(out + [mlp(critic)[:, 0]] if case["value"] else out)


def _cross(a, b):
    return torch.linalg.cross(a, b)


def _qmul(a, b):
    aw, ax, ay, az = a.unbind(-1)
    bw, bx, by, bz = b.unbind(-1)
    return torch.stack([aw * bw - ax * bx - ay * by - az * bz,
                        aw * bx + ax * bw + ay * bz - az * by,
                        aw * by - ax * bz + ay * bw + az * bx,
                        aw * bz + ax * by - ay * bx + az * bw], -1)


def _qconj(a):
    return a * torch.tensor([1.0, -1, -1, -1], device=DEV, dtype=a.dtype)


def _qrot(q, v):
    q = q / q.norm(dim=-1, keepdim=True)
    u, w = q[..., 1:], q[..., :1]
    u, v = torch.broadcast_tensors(u, v)
    t = 2.0 * _cross(u, v)
    return v + w * t + _cross(u, t)


def _qexp(r):
    th = r.norm(dim=-1, keepdim=True)
    k = torch.where(th > 0, torch.sin(0.5 * th) / th.clamp(min=1e-300), torch.full_like(th, 0.5))
    return torch.cat([torch.cos(0.5 * th), r * k], -1)


def _qlog(q):
    q = torch.where(q[..., :1] < 0, -q, q)
    s = q[..., 1:].norm(dim=-1, keepdim=True)
    th = 2.0 * torch.atan2(s, q[..., :1])
    return torch.where(s > 0, q[..., 1:] * (th / s.clamp(min=1e-300)), torch.zeros_like(q[..., 1:]))


def _qangle(q):
    return 2.0 * torch.atan2(q[..., 1:].norm(dim=-1), q[..., 0].abs())


def _slerp(a, b, t):
    a, b = a / a.norm(dim=-1, keepdim=True), b / b.norm(dim=-1, keepdim=True)
    b = torch.where((a * b).sum(-1, keepdim=True) < 0, -b, b)
    om = 2.0 * torch.atan2((a - b).norm(dim=-1, keepdim=True), (a + b).norm(dim=-1, keepdim=True))
    so = torch.sin(om)
    lin = so < 1e-12
    so = torch.where(lin, torch.ones_like(so), so)
    q = torch.where(lin, (1 - t) * a + t * b,
                    (torch.sin((1 - t) * om) * a + torch.sin(t * om) * b) / so)
    return q / q.norm(dim=-1, keepdim=True)


class _Reference:
    """The clips' reference motion in float64: poses and velocities of every body."""

    def __init__(self, desc):
        sk, clips = desc["skeleton"], desc["clips"]
        self.B = sk["n_bodies"]
        self.parent = [int(p) for p in sk["parent"]]
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)  # noqa: E731
        self.offset = t(sk["offset"]).double()
        self.mass = t(sk["mass"]).double()
        self.leaf = torch.tensor([b not in self.parent for b in range(self.B)], device=DEV)
        self.movable = t(np.asarray(sk["jtype"]) != synth.JT_FIXED)
        self.F = t(np.array([c["n_frames"] for c in clips], np.int64))
        self.base = torch.cumsum(self.F, 0) - self.F
        self.fps = t(np.array([c["fps"] for c in clips], np.float64))
        dt = float(desc["config"]["dt"])
        self.dphi = t(np.array([np.float32(dt * c["fps"] / (c["n_frames"] - 1)) for c in clips],
                               np.float32))
        self.root_pos = t(np.concatenate([c["root_pos"] for c in clips])).double()
        self.root_quat = t(np.concatenate([c["root_quat"] for c in clips])).double()
        self.local = t(np.concatenate([c["local_quat"] for c in clips])).double()

    def index(self, clip, phase):
        """Frame index and blend at a float32 phase in [0, 1], in float32."""
        s = phase * (self.F[clip.long()] - 1).float()
        i0 = torch.minimum(s.to(torch.int64), self.F[clip.long()] - 2)
        return i0, s - i0.float()

    def state(self, clip, phase):
        """World P, Q, V, W [n][B][.], local rotations and angular velocities."""
        k = clip.long()
        i0, al = self.index(clip, phase)
        j, al, fps = self.base[k] + i0, al.double()[:, None], self.fps[k][:, None]
        p0, p1 = self.root_pos[j], self.root_pos[j + 1]
        q0, q1 = self.root_quat[j], self.root_quat[j + 1]
        P, V = [(1 - al) * p0 + al * p1], [(p1 - p0) * fps]
        Q, W = [_slerp(q0, q1, al)], [_qlog(_qmul(q1, _qconj(q0))) * fps]
        a, b = self.local[j], self.local[j + 1]
        m = self.movable[1:, None]
        one = torch.tensor([1.0, 0, 0, 0], device=DEV, dtype=torch.float64)
        ql = torch.where(m, _slerp(a, b, al[:, None]), one)
        wl = torch.where(m, _qlog(_qmul(b, _qconj(a))) * fps[:, None], torch.zeros_like(one[:3]))
        for c in range(1, self.B):
            p = self.parent[c]
            d = _qrot(Q[p], self.offset[c])
            Q.append(_qmul(Q[p], ql[:, c - 1]))
            P.append(P[p] + d)
            W.append(W[p] + _qrot(Q[p], wl[:, c - 1]))
            V.append(V[p] + _cross(W[p], d))
        S = [torch.stack(x, 1) for x in (P, Q, V, W)]
        return S + [torch.cat([S[1][:, :1], ql], 1), torch.cat([S[3][:, :1], wl], 1)]


def _heading(Q0):
    f = _qrot(Q0, torch.tensor([1.0, 0, 0], device=DEV, dtype=torch.float64))[..., :2]
    h2 = (f * f).sum(-1, keepdim=True)
    return torch.where(h2 < 1e-12, torch.tensor([1.0, 0], device=DEV, dtype=torch.float64),
                       f / h2.clamp(min=1e-300).sqrt())


def _to_heading(cs, v):
    c, s = cs[:, None, 0], cs[:, None, 1]
    return torch.stack([c * v[..., 0] + s * v[..., 1], c * v[..., 1] - s * v[..., 0], v[..., 2]], -1)


def _frame9(cs, org, P, Q):
    e = torch.eye(3, device=DEV, dtype=torch.float64)
    return torch.cat([_to_heading(cs, P - org), _to_heading(cs, _qrot(Q, e[0])),
                      _to_heading(cs, _qrot(Q, e[1]))], -1)


def _exact_step(case, seed):
    desc, ref, st = _step_inputs(case, seed)
    cfg = desc["config"]
    n = case["n"]
    P, Q, V, W = (st[k].double().permute(2, 0, 1) for k in ("pos", "quat", "linvel", "angvel"))
    k = st["clip"].long()
    ph1 = st["phase"] + ref.dphi[k]
    trunc = ph1 >= 1.0
    ev = torch.clamp(ph1, max=1.0)
    i0 = ref.index(st["clip"], ev)[0]
    Pr, Qr, Vr, Wr, ql, wl = ref.state(st["clip"], ev)
    sq = lambda x: (x * x).sum(-1)  # noqa: E731
    m = ref.mass / ref.mass.sum()
    e_com = sq(((P - Pr) * m[:, None]).sum(1))
    ep = sq(P - Pr)
    e_ee = (ep * ref.leaf).sum(1)
    c = {x: float(np.float32(cfg[x])) for x in cfg if isinstance(cfg[x], float)}
    if case["train"]:
        par = torch.tensor([0] + ref.parent[1:], device=DEV)
        Qp = Q[:, par].clone()
        Qp[:, 0] = torch.tensor([1.0, 0, 0, 0], device=DEV, dtype=torch.float64)
        Wp = W[:, par].clone()
        Wp[:, 0] = 0
        th = _qangle(_qmul(_qconj(ql), _qmul(_qconj(Qp), Q)))
        e_jv = sq(_qrot(_qconj(Qp), W - Wp) - wl).sum(1)
        te = _qangle(_qmul(_qconj(Qr), Q))
        r = torch.exp(-c["m_jrot"] * (th * th).sum(1) - c["m_jvel"] * e_jv - c["m_com"] * e_com
                      - c["m_eepos"] * e_ee - c["m_eerot"] * (te * te * ref.leaf).sum(1))
    else:
        r = (c["c_pose"] * torch.exp(-(c["w_pos"] * ep.sum(1) + c["w_ee"] * e_ee))
             + c["c_vel"] * torch.exp(-c["w_vel"] * sq(V - Vr).sum(1))
             + c["c_com"] * torch.exp(-c["w_com"] * e_com))
    t1, n1 = st["t"] + 1, st["n"] + 1
    low = st["pos"][0, 2] < np.float32(cfg["h_term"])
    term = (t1 > int(cfg["grace"])) & (low | ~(r.float() >= np.float32(cfg["r_min"])))
    done = term | trunc
    x = _philox([torch.arange(n, device=DEV), n1.long(), 0, 1], int(cfg["seed"]))
    k_new = _mulhi(x[0], torch.full_like(x[0], len(desc["clips"]))).to(torch.int32)
    ph_new = (x[1] >> 8).float() * 2.0 ** -24
    clip = torch.where(done, k_new, st["clip"])
    phase = torch.where(done, ph_new, ph1)
    S = ref.state(clip, torch.clamp(phase, max=1.0))[:4]
    # the observation reads the sim state as stored (float32)
    P, Q, V, W = (torch.where(done[:, None, None], s.float().double(), o)
                  for s, o in zip(S, (P, Q, V, W)))
    cs = _heading(Q[:, 0])
    org = P[:, :1] * torch.tensor([1.0, 1, 0], device=DEV, dtype=torch.float64)
    obs = [torch.cat([_frame9(cs, org, P, Q), _to_heading(cs, V), _to_heading(cs, W)],
                     -1).reshape(n, -1), phase.double()[:, None]]
    if case["train"]:
        ee = [0] + [b for b in range(ref.B) if bool(ref.leaf[b])]
        phj = phase
        for _ in range(int(cfg["obs_future"])):
            phj = phj + ref.dphi[clip.long()]
            F = ref.state(clip, torch.clamp(phj, max=1.0))
            obs.append(_frame9(cs, org, F[0][:, ee], F[1][:, ee]).reshape(n, -1))
        obs.append(torch.where(done[:, None], torch.zeros_like(st["prev"]), st["prev"]).double())
    sim = [s.permute(1, 2, 0) for s in (P, Q, V, W)]
    return dict(reward=r, terminated=term.to(torch.uint8), truncated=trunc.to(torch.uint8),
                ref_frame=i0.to(torch.int32), clip=clip, phase=phase.double(),
                t=torch.where(done, torch.zeros_like(t1), t1), n=n1, obs=torch.cat(obs, 1).t(),
                pos=sim[0], quat=sim[1], linvel=sim[2], angvel=sim[3])


def _exact_gae(case, seed):
    d = _gae_inputs(case, seed)
    n, T = case["n"], case["T"]
    gam, lam = float(np.float32(synth.GAMMA)), float(np.float32(synth.LAMBDA))
    r, v = d["reward"][:, :n].double(), d["value"][:, :n].double()
    te, tr = d["term"][:, :n].bool(), d["trunc"][:, :n].bool()
    adv = torch.zeros_like(r)
    a = torch.zeros(n, device=DEV, dtype=torch.float64)
    for t in range(T - 1, -1, -1):
        nxt = torch.where(te[t], torch.zeros_like(a), torch.where(tr[t], v[t], v[t + 1]))
        a = r[t] + gam * nxt - v[t] + torch.where(te[t] | tr[t], torch.zeros_like(a), gam * lam * a)
        adv[t] = a
    epr, epl = d["ep_return"][:n].double(), d["ep_length"][:n].double()
    er, el = 0.0, 0.0
    for t in range(T):
        epr, epl, done = epr + r[t], epl + 1, (te[t] | tr[t]).double()
        er, el = er + (done * epr).sum(), el + (done * epl).sum()
        epr, epl = epr * (1 - done), epl * (1 - done)
    ret = adv + v[:T]
    s = torch.stack([r.sum(), te.double().sum(), tr.double().sum(), (te | tr).double().sum(), er,
                     el, adv.sum(), (adv * adv).sum(), v[:T].sum(), ret.sum()])
    return dict(adv=adv, ret=ret, ep_return=epr, ep_length=epl.to(torch.int32), summary=s)


def _mlp_grad(net, g_out, xs):
    """Gradients [dW, db, ...] of a ReLU MLP from the gradient at its output."""
    out, g = [], g_out
    for l in range(len(net["W"]) - 1, -1, -1):
        out = [g.t() @ xs[l], g.sum(0)] + out
        if l:
            g = (g @ net["W16"][l]) * (xs[l] > 0)
    return out


def _layers(net, x):
    r = lambda t: t.float().bfloat16().double()  # noqa: E731
    net["W16"] = [r(w) for w in net["W"]]
    xs, h = [], r(x)
    for l, b in enumerate(net["b"]):
        xs.append(h)
        h = torch.addmm(b, h, net["W16"][l].t())
        h = r(torch.relu(h)) if l < len(net["b"]) - 1 else h
    return h, xs


def _exact_ppo(case, seed):
    """The update (or one minibatch's gradient) in float64: bf16 rounding of the
    input, the weights and the hidden activations in the forward, an exact
    backward through them, Adam on float32 master weights."""
    actor, critic = _net(case, seed)
    d = _rollout_inputs(case, seed, actor, critic)
    p = binding.PPO_DEFAULTS
    n = case["n"]
    nets = [_on_gpu(actor, torch.float64), _on_gpu(critic, torch.float64)]
    ls = torch.from_numpy(actor["log_std"]).to(DEV, torch.float64)
    ls0 = ls.clone()
    adv = d["adv"].double()
    am, asd = adv.mean(), adv.std()
    cpt = n // 64
    eps, f32 = float(np.float32(p["clip"])), torch.float32
    order = [(e, k) for e in range(case["epochs"]) for k in range(case["minibatches"])] \
        if case["kind"] == "update" else [(0, case["minibatches"] - 1)]
    mom = None
    stats = torch.zeros(len(binding.PPO_STATS), device=DEV, dtype=torch.float64)
    for step, (e, k) in enumerate(order, 1):
        q = np.array_split(d["perm"][e].cpu().numpy(), case["minibatches"])[k]
        q = torch.from_numpy(q).to(DEV).long()
        t = (q // cpt)[:, None].expand(-1, 64).reshape(-1)
        en = ((q % cpt) * 64)[:, None].add(torch.arange(64, device=DEV)).reshape(-1)
        x = d["obs"][t, :, en].double()
        act, mo, lo = (d[z][t, en].double() for z in ("action", "mean", "logp"))
        A, R, vo = ((d["adv"][t, en].double() - am) / (asd + 1e-8), d["ret"][t, en].double(),
                    d["value"][t, en].double())
        M = x.shape[0]
        mu, xa = _layers(nets[0], x)
        v, xc = _layers(nets[1], x)
        v = v[:, 0]
        sig = torch.exp(ls)
        z = (act - mu) / sig
        logp = -(0.5 * z * z + ls + 0.5 * math.log(2 * math.pi)).sum(1)
        ratio = torch.exp(logp - lo)
        s1, s2 = -A * ratio, -A * torch.clamp(ratio, 1 - eps, 1 + eps)
        dlogp = torch.where(s1 >= s2, s1, torch.where((ratio - 1).abs() <= eps, s2,
                                                       torch.zeros_like(s2))) / M
        vc = vo + torch.clamp(v - vo, -eps, eps)
        l1, l2 = (v - R) ** 2, (vc - R) ** 2
        dv = torch.where(l1 >= l2, 2 * (v - R),
                         torch.where((v - vo).abs() <= eps, 2 * (vc - R), torch.zeros_like(v)))
        dv = dv * p["value_coef"] / M
        dls = (dlogp[:, None] * (z * z - 1)).sum(0) - p["entropy_coef"]
        g = _mlp_grad(nets[0], dlogp[:, None] * z / sig, xa) + [dls] \
            + _mlp_grad(nets[1], dv[:, None], xc)
        flat = torch.cat([y.reshape(-1) for y in g])
        norm = flat.norm()
        so = torch.exp(ls0)
        kl = (ls - ls0 + (so ** 2 + (mo - mu) ** 2) / (2 * sig ** 2) - 0.5).sum(1).mean()
        terms = [torch.maximum(s1, s2).mean(), torch.maximum(l1, l2).mean(), kl,
                 ((ratio - 1).abs() > eps).double().mean()]
        if case["kind"] == "grad":
            stats[:4] = torch.stack(terms)
            return dict(grad=flat, stats=None)
        stats[:4] += torch.stack(terms)
        stats[4] += norm
        stats[5] += 1
        stats[6] = float(np.float32(LR))
        flat = flat * torch.clamp(p["max_grad_norm"] / (norm + 1e-6), max=1.0)
        mom = mom or (torch.zeros_like(flat), torch.zeros_like(flat))
        b1, b2 = float(np.float32(p["beta1"])), float(np.float32(p["beta2"]))
        mom = (b1 * mom[0] + (1 - b1) * flat, b2 * mom[1] + (1 - b2) * flat * flat)
        upd = LR * (mom[0] / (1 - b1 ** step)) / (torch.sqrt(mom[1] / (1 - b2 ** step)) + p["eps"])
        vec = torch.cat([y.reshape(-1) for y in _flat(nets, ls)])
        vec = (vec - upd).to(f32).double()
        o = 0
        for y in _flat(nets, ls):
            y.copy_(vec[o:o + y.numel()].view(y.shape))
            o += y.numel()
    return dict(weights=torch.cat([y.reshape(-1) for y in _flat(nets, ls)]), stats=stats,
                lr=torch.full((1,), LR, device=DEV, dtype=torch.float64))


def _flat(nets, ls):
    wb = [[y for pair in zip(net["W"], net["b"]) for y in pair] for net in nets]
    return wb[0] + [ls] + wb[1]
