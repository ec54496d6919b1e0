"""What a program built on this package has it do, as cases with sizes, inputs, least work and tolerances.

Five kinds of calls, each through the public entry points (`UpdateStep`, `EvalSweep`, `binding.Context`):

  act    one time step of the rollout: every environment's action, log-density and value from the target networks a
         program materialised at the start of the iteration (`policy_fwd` of both networks on a one-step row selection)
  step   one whole rollout-and-update step (`UpdateStep.run`), with gradients only or with Adam after every minibatch
  gae    vector GAE with scalarisation on a finished rollout, with or without time limits told apart from failures
  loss   clipped-PPO and value loss with their gradients on one minibatch
  eval   evaluation sweep: actions of the actor family on a grid of trade-offs, return vectors, front, hypervolume

Sizes are those of `configs.CONFIGS`, of the benchmark's stress shape and of the ragged test shapes, and `draw` mixes them.
"""
from __future__ import annotations

import math

import torch

from paper_2603_09237_amd import binding, inputs
from paper_2603_09237_amd.configs import ACT_SILU, ACT_TANH, CONFIGS, NET_ACTOR, NET_CRITIC, Config
from paper_2603_09237_amd.evaluate import EvalSweep
from paper_2603_09237_amd.step import UpdateStep

_SIZES = ("K", "P", "N", "T", "obs_dim", "act_dim", "n_hidden", "width", "act", "rank", "hyper_width", "wdtype",
          "mean_tanh", "minibatches", "epochs", "p_done", "sigma_state", "dirichlet_alpha")
_ADAM = dict(lr_actor=3e-4, lr_critic=1e-3, beta1=0.9, beta2=0.999, eps=1e-8)
_DEV = "cuda:0"


def _case(kind, base=None, name=None, adam=False, adv_norm="scalar", trunc=False, **over):
    c = {k: getattr(base if base is not None else CONFIGS[1], k) for k in _SIZES}
    c.update(over)
    c.update(kind=kind, adam=adam, adv_norm=adv_norm, trunc=trunc)
    if name is not None:
        c["name"] = name
    return c


def _config(c):
    return Config(name=str(c.get("name", c["kind"])), **{k: c[k] for k in _SIZES})


def listed():
    c = CONFIGS
    return [
        # a simulator loop asks for actions once per time step: small policies, latency of one call counts
        _case("act", c[3], "act-hopper-bf16"),
        # the same loop with the largest policies
        _case("act", c[5], "act-largest-bf16"),
        # the smallest update step: debugging runs, toy problems; launches count
        _case("step", c[1], "step-tiny-fp32"),
        # ordinary locomotion training, single precision
        _case("step", c[2], "step-quadruped-fp32"),
        # ordinary locomotion training, bf16
        _case("step", c[3], "step-hopper-bf16"),
        # wide policies with many objectives, one minibatch
        _case("step", c[4], "step-humanoid-bf16"),
        # the largest single-GPU training step, minibatches and epochs: the headline workload
        _case("step", c[5], "step-largest-bf16"),
        # PPO as it is trained, optimiser included: state-dependent sigma, odd sizes, several minibatches and epochs
        _case("step", c[3], "step-adam-ragged-bf16", adam=True, K=3, P=24, N=24 * 150, T=25, obs_dim=45, act_dim=6,
              sigma_state=1, minibatches=3, epochs=2),
        # strictly affine hypernetwork, objectives normalised one by one, tanh networks of an odd width
        _case("step", c[2], "step-affine-ragged-fp32", adv_norm="per_objective", K=5, P=10, N=10 * 74, T=50, obs_dim=100,
              act_dim=7, n_hidden=2, width=160, act=ACT_TANH, rank=-1, minibatches=2),
        # a long rollout of very many environments: advantage estimation with time limits, beyond every cache
        _case("gae", c[5], "gae-trunc-long", T=256, N=65536, obs_dim=16, trunc=True),
        # the loss on one minibatch of the same rollout
        _case("loss", c[5], "loss-long", T=256, N=65536, obs_dim=16),
        # judging a trained hypernetwork on a grid of trade-offs
        _case("eval", c[4], "eval-humanoid-bf16"),
    ]


# ---------------------------------------------------------------------------------------------- drawn cases
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _one(rng):
    kind = rng.choice(("step", "step", "step", "step", "act", "gae", "loss", "eval"))
    bf16 = rng.random() < 0.65
    K, P = rng.randint(2, 6), _log(rng, 4, 128)
    sigma = rng.random() < 0.2
    d = dict(K=K, P=P, obs_dim=_log(rng, 8, 128), act_dim=rng.randint(2, 8 if sigma else 10), sigma_state=int(sigma),
             n_hidden=rng.randint(2, 4), width=rng.choice((32, 64, 128, 256, 256, 256, 512, 512, 512, 48, 144, 160, 384)),
             act=rng.choice((ACT_SILU, ACT_SILU, ACT_TANH)), rank=rng.choice((4, 8, 16, 16, -1)), hyper_width=32,
             wdtype=int(bf16), mean_tanh=1, minibatches=1, epochs=1, p_done=rng.choice((0.005, 0.01, 0.02)),
             dirichlet_alpha=rng.choice((0.5, 1.0)))
    adam, norm, trunc = False, "scalar", False
    if kind == "step":
        adam = rng.random() < 0.4
        norm = "per_objective" if rng.random() < 0.15 else "scalar"
        d["minibatches"], d["epochs"] = rng.choice((1, 1, 2, 3, 4)), rng.choice((1, 1, 2))
        d["T"], n_g = _log(rng, 16, 64), d["minibatches"] * max(1, _log(rng, 12, 256) // d["minibatches"])
    elif kind == "act":
        d["T"], n_g = 16, _log(rng, 12, 256)
    elif kind == "eval":
        d["P"] = min(d["P"], 64)
        d["T"], n_g = _log(rng, 16, 64), _log(rng, 12, 256)
    else:
        trunc, d["obs_dim"] = kind == "gae" and rng.random() < 0.5, 16   # observations play no part in these two
        d["minibatches"] = rng.choice((1, 2, 4)) if kind == "loss" else 1
        d["T"], n_g = _log(rng, 16, 256), d["minibatches"] * max(1, _log(rng, 16, 512) // d["minibatches"])
    return _case(kind, None, None, adam, norm, trunc, N=d["P"] * n_g, **d)


def _cost(c):
    """Seconds, roughly: what bounds a draw to the largest listed case."""
    w = work(c)
    flops = w["flops"] * (16 if c["wdtype"] == 0 else 1)
    return w["bytes"] / 2e12 + flops / 500e12


def draw(rng):
    most = 0.8 * _cost(_case("step", CONFIGS[5]))
    while True:
        c = _one(rng)
        if _cost(c) <= most:
            return c


# ---------------------------------------------------------------------------------------------- inputs
def _preferences(cfg, g):
    if cfg.dirichlet_alpha == 0.5:   # Gamma(1/2) variables are half squared normals
        x = torch.randn(cfg.P, cfg.K, device=_DEV, generator=g).square() + 1e-12
    else:
        x = -torch.log(torch.rand(cfg.P, cfg.K, device=_DEV, generator=g) * 0.999 + 5e-4)
    return x / x.sum(1, keepdim=True)


def _hparams(cfg, net, g):
    """Initial parameters of a hypernetwork, block by block at the scales of `inputs.hparam_blocks`."""
    parts = []
    for _, shape, kind, scale in inputs.hparam_blocks(cfg, net):
        n = math.prod(shape)
        parts.append(torch.full((n,), float(scale), device=_DEV) if kind == "const" else
                     torch.randn(n, device=_DEV, generator=g) * float(scale))
    return torch.cat(parts)


def _moved(cfg, net, hp, g, rel=0.05):
    """Parameters some updates later: every block moved by `rel` of its root mean square."""
    out, off = hp.clone(), 0
    for _, shape, _, _ in inputs.hparam_blocks(cfg, net):
        n = math.prod(shape)
        blk = out[off:off + n]
        blk += rel * blk.square().mean().sqrt() * torch.randn(n, device=_DEV, generator=g)
        off += n
    return out


def _rewards(cfg, g):
    r = torch.randn(cfg.T, cfg.N, cfg.K, device=_DEV, generator=g)
    if cfg.K > 2:
        r *= torch.from_numpy(inputs.reward_scales(cfg)).to(_DEV)
    return r


def _flags(cfg, p, g):
    return (torch.rand(cfg.T, cfg.N, device=_DEV, generator=g) < p).to(torch.uint8)


def prepare(case, seed):
    cfg = _config(case)
    g = torch.Generator(device=_DEV).manual_seed(int(seed) * 7919 + 17)
    normal = lambda *shape: torch.randn(*shape, device=_DEV, generator=g)
    T, N, P, K, A = cfg.T, cfg.N, cfg.P, cfg.K, cfg.act_dim
    AO = 2 * A if cfg.sigma_state else A
    s = {"kind": case["kind"], "cfg": cfg}

    if case["kind"] == "step":
        st = UpdateStep(cfg, device=_DEV, optimizer=dict(_ADAM) if case["adam"] else None, adv_norm=case["adv_norm"])
        st.w.copy_(_preferences(cfg, g))
        st.obs.normal_(generator=g)
        st.eps.normal_(generator=g)
        st.rewards.copy_(_rewards(cfg, g))
        st.dones.copy_(_flags(cfg, cfg.p_done, g))
        for net in (NET_ACTOR, NET_CRITIC):
            hp = _hparams(cfg, net, g)
            st.hp_old[net].copy_(hp)
            # bf16: an update in mid-iteration, 3-10 % of the cells outside the clip range.  fp32: the first one of an
            # iteration, where the ratio is one; a cell within rounding of the clip edge would otherwise move a
            # gradient by far more than fp32 arithmetic does
            st.hp[net].copy_(_moved(cfg, net, hp, g) if cfg.wdtype == 1 else hp)
        s["st"] = st
        return s

    ctx = s["ctx"] = binding.Context.from_config(cfg)
    if case["kind"] == "act":
        wdt = torch.bfloat16 if cfg.wdtype == 1 else torch.float32
        s["rows"] = rows = (T // 2, 1, 0, cfg.n_g)
        w = _preferences(cfg, g)
        s["obs"], s["eps"] = normal(T + 1, N, cfg.obs_dim), normal(T, N, A)
        s["mu"], s["a"], s["logp"] = torch.zeros(T, N, AO, device=_DEV), torch.zeros(T, N, A, device=_DEV), torch.zeros(T, N, device=_DEV)
        s["v"] = torch.zeros(T + 1, N, K, device=_DEV)
        s["ws"] = torch.empty(ctx.workspace_bytes(rows), dtype=torch.uint8, device=_DEV)
        s["theta"] = {}
        for net in (NET_ACTOR, NET_CRITIC):   # the iteration's policies, materialised once before the loop over time
            tm = torch.empty(P, ctx.theta_mat_len(net), dtype=wdt, device=_DEV)
            tv = torch.empty(P, ctx.theta_vec_len(net), device=_DEV)
            ctx.hypernet_fwd(net, _hparams(cfg, net, g), w, tm, tv, s["ws"])
            s["theta"][net] = (tm, tv)
    elif case["kind"] == "gae":
        s["r"], s["v"], s["w"] = _rewards(cfg, g), normal(T + 1, N, K), _preferences(cfg, g)
        s["done"] = _flags(cfg, cfg.p_done, g)
        s["trunc"] = _flags(cfg, 0.01, g) if case["trunc"] else None
        s["vtarg"], s["adv_s"] = torch.empty(T, N, K, device=_DEV), torch.empty(T, N, device=_DEV)
    elif case["kind"] == "loss":
        s["rows"] = (0, T, 0, cfg.n_g // cfg.minibatches)
        s["mu"], s["v"], s["vtarg"] = normal(T, N, AO), normal(T, N, K), normal(T, N, K)
        s["mu"][..., :A].tanh_()
        if cfg.sigma_state:
            s["mu"][..., A:].mul_(0.1).sub_(0.5)
            s["logsig"], ls = None, s["mu"][..., A:]
        else:
            s["logsig"] = 0.1 * normal(P, A) - 0.5
            ls = s["logsig"].repeat_interleave(cfg.n_g, 0)
        noise = normal(T, N, A)
        s["a"] = s["mu"][..., :A] + ls.exp() * noise
        logp = -0.5 * noise.square().sum(-1) - ls.sum(-1) - 0.5 * A * math.log(2 * math.pi)
        # log-ratios of a policy in mid-update; none within rounding of an edge of the clip range, where the gradient jumps
        q = 0.12 * normal(T, N)
        for edge in (math.log1p(-cfg.clip_eps), math.log1p(cfg.clip_eps)):
            q = torch.where((q - edge).abs() < 2e-4, q + 4e-4, q)
        s["logp_old"] = logp - q
        s["adv_s"] = normal(T, N) * 2.0 + 0.3
        s["dmu"], s["dv"] = torch.zeros(T, N, AO, device=_DEV), torch.zeros(T, N, K, device=_DEV)
        s["dlogsig"] = None if cfg.sigma_state else torch.zeros(P, A, device=_DEV)
        s["stats"] = torch.zeros(8, device=_DEV)
        s["ws"] = torch.empty(ctx.workspace_bytes(s["rows"]), dtype=torch.uint8, device=_DEV)
    else:
        s["sweep"] = EvalSweep(cfg, device=_DEV)
        s["hp"], s["w"] = _hparams(cfg, NET_ACTOR, g), _preferences(cfg, g)
        s["obs"], s["r"], s["done"] = normal(T + 1, N, cfg.obs_dim), _rewards(cfg, g), _flags(cfg, cfg.p_done, g)
        s["out"] = torch.empty(T + 1, N, AO, device=_DEV)
        # a reference point below the return vectors of this reward distribution
        s["ref"] = torch.full((K,), -10.0, device=_DEV) * (torch.from_numpy(inputs.reward_scales(cfg)).to(_DEV) if K > 2 else 1.0)
    return s


# ---------------------------------------------------------------------------------------------- one pass
def run(s):
    cfg, kind = s["cfg"], s["kind"]
    if kind == "step":
        st = s["st"]
        st.run()
        out = {"mu": st.mu_old, "act": st.act, "logp": st.logp_old, "v": st.v_roll, "vtarg": st.vtarg, "adv": st.adv_s,
               "d_actor": st.dhp[NET_ACTOR], "d_critic": st.dhp[NET_CRITIC], "stats": st.stats}
        if st.optimizer is not None:
            for net, n in ((NET_ACTOR, "actor"), (NET_CRITIC, "critic")):
                out["hp_" + n], out["m_" + n], out["v_" + n] = st.hp[net], st.adam_m[net], st.adam_v[net]
        return out
    ctx = s["ctx"]
    if kind == "act":
        (tm, tv), (cm, cv) = s["theta"][NET_ACTOR], s["theta"][NET_CRITIC]
        ctx.policy_fwd(NET_ACTOR, tm, tv, s["obs"], s["rows"], s["mu"], eps=s["eps"], act=s["a"], logp=s["logp"], ws=s["ws"])
        ctx.policy_fwd(NET_CRITIC, cm, cv, s["obs"], s["rows"], s["v"], ws=s["ws"])
        return s["mu"], s["a"], s["logp"], s["v"]
    if kind == "gae":
        if s["trunc"] is None:
            ctx.vec_gae(s["r"], s["v"], s["done"], s["w"], cfg.gamma, cfg.lam, None, s["vtarg"], s["adv_s"])
        else:
            ctx.vec_gae_trunc(s["r"], s["v"], s["done"], s["trunc"], s["w"], cfg.gamma, cfg.lam, None, s["vtarg"], s["adv_s"])
        return s["vtarg"], s["adv_s"]
    if kind == "loss":
        ctx.ppo_loss_grad(s["rows"], s["mu"], s["logsig"], cfg.act_dim, s["a"], s["logp_old"], s["adv_s"], s["v"], s["vtarg"],
                          cfg.clip_eps, 1, s["dmu"], s["dlogsig"], s["dv"], s["stats"], s["ws"])
        return [t for t in (s["dmu"], s["dlogsig"], s["dv"], s["stats"]) if t is not None]
    ev = s["sweep"]
    ev.actions(s["hp"], s["w"], s["obs"], s["out"])
    J, front, hv = ev.score(s["r"], s["done"], cfg.gamma, s["ref"])
    return s["out"], J, front, hv[:1]


# ---------------------------------------------------------------------------------------------- least work, tolerance
def _net(cfg, net):
    """(weights, biases and sigmas, hypernet parameters) of a network family."""
    sh = inputs.layer_shapes(cfg, net)
    vec = sum(do for do, _ in sh) + (cfg.act_dim if net == NET_ACTOR and not cfg.sigma_state else 0)
    return sum(do * di for do, di in sh), vec, inputs.hparam_count(cfg, net)


def work(case):
    cfg = _config(case)
    T, N, P, K, A, O = cfg.T, cfg.N, cfg.P, cfg.K, cfg.act_dim, cfg.obs_dim
    AO = 2 * A if cfg.sigma_state else A
    cells = T * N
    nets = {net: _net(cfg, net) for net in (NET_ACTOR, NET_CRITIC)}
    # a weight of one preference's network: rank-r product of its factors, or its own row of the affine map
    per_weight = 2.0 * (cfg.rank if cfg.rank >= 0 else cfg.hyper_width)
    if case["kind"] == "gae":
        return {"bytes": 4.0 * (2 * K * cells + K * (cells + N) + cells) + cells * (2 if case["trunc"] else 1), "flops": 8.0 * K * cells}
    if case["kind"] == "loss":
        b = cells // cfg.minibatches
        return {"bytes": 4.0 * b * (2 * AO + A + 2 + 3 * K), "flops": b * (20.0 * A + 4.0 * K)}
    if case["kind"] == "act":
        wsz = 2 if cfg.wdtype == 1 else 4
        return {"bytes": P * sum(m * wsz + 4.0 * v for m, v, _ in nets.values()) + 4.0 * N * (O + 2 * A + AO + 1 + K),
                "flops": 2.0 * N * sum(m for m, _, _ in nets.values())}
    if case["kind"] == "eval":
        m, v, h = nets[NET_ACTOR]
        return {"bytes": 4.0 * (h + (cells + N) * (O + AO) + cells * K + P * K) + cells,
                "flops": 2.0 * (cells + N) * m + P * m * per_weight + 2.0 * P ** max(K - 2, 1)}
    flops, first = 0.0, O * cfg.width
    updates = cfg.minibatches * cfg.epochs
    for net, (m, v, h) in nets.items():
        flops += 2.0 * m * (cells + (N if net == NET_CRITIC else 0))              # rollout
        flops += cfg.epochs * cells * (4.0 * m + 2.0 * (m - first))               # forward, weight and input gradients
        flops += P * m * per_weight * (1 + updates) + P * m * 2 * per_weight * updates   # hypernetwork forward, backward
    hp = sum(h for _, _, h in nets.values())
    data = (cells + N) * (O + K) + cells * (K + A) + cells * (AO + A + 1 + K + 1) + P * K
    state = hp * (2 + (7 if case["adam"] else 1))   # both parameter sets in, gradients out; Adam: m, v and parameters too
    return {"bytes": 4.0 * (data + state) + cells, "flops": flops}


def tolerance(case):
    if case["kind"] in ("gae", "loss"):
        return {"rel": 2e-5, "max": 2e-3}       # fp32 sums over a horizon or over one cell's components
    if case["kind"] in ("act", "eval"):
        return {"rel": 1e-2} if case["wdtype"] == 1 else {"rel": 2e-5, "max": 1e-3}
    if case["adam"]:
        # every minibatch starts from the last one's parameters: its rounding, and the sign of gradients near zero, go on
        # through Adam's normalised step into the next gradient
        return {"rel": 2e-2, "max": 0.9}
    # gradients are cancelling sums over the whole minibatch, taken through the networks and the hypernetwork
    return {"rel": 1e-2, "max": 0.6} if case["wdtype"] == 1 else {"rel": 1e-4, "max": 1e-2}
