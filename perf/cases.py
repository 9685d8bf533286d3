"""The calls of this library that are timed: what a learner has it do with its
batches, from the paper's own learner batch of 32 trajectories to the stress
batch of 16384 lanes.

A case names an entry point (``call``), a batch shape and the options of the
call.  Inputs are drawn on the GPU with the distributions of ``synth/``: unit
normal target logits with a behaviour policy some noise away from them, actions
sampled from the behaviour policy, sparse or ternary rewards, episode ends at
the discounts.  Workspace and output tensors are made once, as a learner that
steps again and again on batches of one shape keeps them.
"""

import math

import torch

import paper_1802_01561_amd as vt

BASELINE_COST, ENTROPY_COST = 0.5, 0.01
TANH_SQ_MEAN = 0.394  # E[tanh(N(0, 1))^2]
MOST_LOGITS = 1000 * 16384 * 18  # of a drawn case: the stress batch's
MOST_HEAD_STEPS = 1000 * 2048


def _case(name, call, T, B, A, **options):
    c = dict(call=call, T=T, B=B, A=A, H=0, logits="f32", grad="f32", behaviour="logits", rewards="raw",
             c_bar=1.0, lam=1.0)
    c.update(options)
    return dict(c, name=name) if name else c


def listed():
    return [
        # Atari learner batch (unroll 20, 32 trajectories, the full action set);
        # the actors send log mu(a|x), rewards are clipped.
        _case("atari_loss", "loss", 20, 32, 18, behaviour="log_probs", rewards="clip"),
        # DeepMind Lab learner batch (unroll 100, 32 trajectories, 9 actions).
        _case("dmlab_loss", "loss", 100, 32, 9),
        # 30 tasks in one batch of DeepMind Lab unrolls, float32 and mixed precision.
        _case("multitask_loss", "loss", 100, 4096, 9),
        _case("multitask_loss_bf16", "loss", 100, 4096, 9, logits="bf16", grad="bf16", rewards="asymmetric"),
        # Whatever trajectories are ready: odd unroll and lane count, a game's
        # minimal action set.
        _case("ragged_loss", "loss", 83, 1021, 6, rewards="clip"),
        # Long unrolls of a modest number of environments, lambda < 1.
        _case("long_unroll_loss", "loss", 1000, 512, 18, c_bar=0.5, lam=0.95),
        # The stress batch: loss and gradients in float32, targets alone from bf16 logits.
        _case("stress_loss", "loss", 1000, 16384, 18),
        _case("stress_targets_bf16", "targets", 1000, 16384, 18, logits="bf16"),
        # A larger discretised action set.
        _case("many_actions_loss", "loss", 100, 512, 48),
        # The output layer in the same call: the DeepMind Lab batch, the 30-task
        # batch in mixed precision, and a large one.
        _case("dmlab_head", "head", 100, 32, 9, H=256),
        _case("multitask_head_bf16", "head", 100, 4096, 18, H=256, logits="bf16", grad="bf16", rewards="clip"),
        _case("large_head", "head", 1000, 2048, 18, H=256),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    call = rng.choice(["loss", "loss", "loss", "targets", "head", "head"])
    T = _log_int(rng, 5, 1000)
    if call == "head":
        A = rng.choice([9, 18, rng.randint(2, 31)])
        H = rng.choice([64, 128, 256, 256])
        B = _log_int(rng, 4, max(4, min(4096, MOST_HEAD_STEPS // T)))
    else:
        A = rng.choice([9, 18, rng.randint(2, 20), rng.randint(2, 64)])
        H = 0
        B = _log_int(rng, 4, max(4, min(16384, MOST_LOGITS // (T * A))))
    c_bar, lam = rng.choice([(1.0, 1.0), (1.0, 1.0), (0.5, 0.95)])
    return _case(None, call, T, B, A, H=H, logits=rng.choice(["f32", "f32", "bf16"]),
                 grad=rng.choice(["f32", "f32", "bf16"]) if call != "targets" else "f32",
                 behaviour=rng.choice(["logits", "logits", "log_probs"]),
                 rewards=rng.choice(["raw", "clip", "asymmetric"]), c_bar=c_bar, lam=lam)


DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}


def _inputs(case, seed):
    """The batch, as device tensors."""
    T, B, A = case["T"], case["B"], case["A"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    kw = dict(generator=g, device="cuda", dtype=torch.float32)
    logits = DTYPE[case["logits"]]
    x = {}
    if case["call"] == "head":
        H = case["H"]
        x["hidden"] = torch.randn((T, B, H), **kw).tanh_().to(torch.bfloat16)
        x["head_weight"] = (torch.randn((H, A + 1), **kw) / math.sqrt(TANH_SQ_MEAN * H)).to(torch.bfloat16)
        x["head_bias"] = torch.randn(A + 1, **kw) * 0.1
        y = torch.randn((T, B, A), **kw)
    else:
        z = torch.randn((T, B, A), **kw)
        y = torch.randn((T, B, A), **kw).mul_(0.5).add_(z)
        x["target_logits"] = z.to(logits)
        x["values"] = torch.randn((T, B), **kw)
    y = y.to(logits)
    # Gumbel-max: argmax of y - log E with E ~ Exp(1) samples from softmax(y).
    noise = torch.empty((T, B, A), device="cuda", dtype=torch.float32).exponential_(generator=g).clamp_(min=1e-30)
    x["actions"] = (y.float() - noise.log_()).argmax(dim=-1).to(torch.int32)
    if case["behaviour"] == "log_probs":
        lp = torch.log_softmax(y.double(), dim=-1)
        x["behaviour_logits"] = lp.gather(-1, x["actions"].long().unsqueeze(-1)).squeeze(-1).float()
    else:
        x["behaviour_logits"] = y
    u = torch.rand((T, B), **kw)
    mag = torch.rand((T, B), **kw) * 10.0 - 5.0
    x["rewards"] = torch.where(u < 0.1, mag, torch.zeros_like(mag))
    if case["rewards"] == "raw":
        x["rewards"] = x["rewards"].clamp(-1.0, 1.0)
    ends = torch.rand((T, B), **kw) < 0.01
    x["discounts"] = torch.where(ends, 0.0, 0.99).to(torch.float32)
    x["bootstrap_value"] = torch.randn(B, **kw)
    return {k: v.contiguous() for k, v in x.items()}


def prepare(case, seed):
    x = _inputs(case, seed)
    T, B, A, H = case["T"], case["B"], case["A"], case["H"]
    f32 = dict(dtype=torch.float32, device="cuda")
    grad = dict(dtype=DTYPE[case["grad"]], device="cuda")
    options = dict(rho_bar=1.0, c_bar=case["c_bar"], lam=case["lam"], behaviour=case["behaviour"],
                   reward_transform=None if case["rewards"] == "raw" else case["rewards"])
    if case["call"] == "targets":
        return vt.vtrace_targets, x, dict(options, vs=torch.empty((T, B), **f32),
                                          pg_advantages=torch.empty((T, B), **f32))
    options.update(baseline_cost=BASELINE_COST, entropy_cost=ENTROPY_COST, grad_dtype=DTYPE[case["grad"]])
    if case["call"] == "head":
        out = vt.HeadLossGrad(torch.empty(4, **f32), torch.empty((T, B, H), **grad),
                              torch.empty((H, A + 1), **f32), torch.empty(A + 1, **f32), None, None, None, None)
        return vt.vtrace_head_loss_grad, x, dict(options, out=out, workspace=vt.Workspace(T, B, A, H=H))
    out = vt.LossGrad(torch.empty(4, **f32), torch.empty((T, B, A), **grad), torch.empty((T, B), **f32),
                      None, None, None)
    return vt.vtrace_loss_grad, x, dict(options, out=out, workspace=vt.Workspace(T, B, A))


def run(state):
    call, x, options = state
    return tuple(call(**x, **options))


def work(case):
    """Each input read once and each output written once.  Operations: per
    logit an exponential and its sums (about 20, as an exp2 polynomial), per
    gradient element 3, per step 60 for the recursion and the losses; for the
    output layer its three products."""
    T, B, A, H = case["T"], case["B"], case["A"], case["H"]
    n = T * B
    wide, grad = 4 if case["logits"] == "f32" else 2, 4 if case["grad"] == "f32" else 2
    scalars = 12  # action, reward, discount
    behaviour = 4 if case["behaviour"] == "log_probs" else A * wide
    rows = 1 if case["behaviour"] == "log_probs" else 2
    flops = n * (rows * A * 20 + 60)
    if case["call"] == "targets":
        return {"bytes": n * (A * wide + behaviour + scalars + 4 + 8) + 4 * B, "flops": flops}
    if case["call"] == "loss":
        return {"bytes": n * (A * wide + behaviour + scalars + 4 + A * grad + 4) + 4 * B, "flops": flops + 3 * A * n}
    layer = (A + 1) * (2 * H + 4 + 4 * H + 4)  # weight, bias and their gradients
    return {"bytes": n * (2 * H + behaviour + scalars + H * grad) + 4 * B + layer,
            "flops": flops + 3 * A * n + 6 * n * H * (A + 1)}


def tolerance(case):
    if case["grad"] == "bf16":  # two bfloat16 roundings of one value: 2^-9 each
        return {"rel": 5e-3, "max": 2e-2}
    if case["call"] == "head":  # d_hidden's operands are bfloat16 pairs, 2^-17
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 1e-6, "max": 1e-4}


def _targets64(z, y_or_lp, values, bootstrap, x, case):
    """log pi, advantages and value targets of Remark 1 in float64."""
    logp = torch.log_softmax(z, dim=-1)
    act = x["actions"].long().unsqueeze(-1)
    log_pa = logp.gather(-1, act).squeeze(-1)
    if case["behaviour"] == "log_probs":
        log_mu = y_or_lp
    else:
        log_mu = torch.log_softmax(y_or_lp, dim=-1).gather(-1, act).squeeze(-1)
    ratio = torch.exp(log_pa - log_mu)
    del log_mu
    f32 = lambda v: float(torch.tensor(v, dtype=torch.float32))  # noqa: E731 (the call's scalars are float32)
    rho = ratio.clamp(max=1.0)
    c = f32(case["lam"]) * ratio.clamp(max=f32(case["c_bar"]))
    r = x["rewards"].double()
    if case["rewards"] == "clip":
        r = r.clamp(-1.0, 1.0)
    elif case["rewards"] == "asymmetric":
        t = torch.tanh(r)
        r = 0.3 * t.clamp(max=0.0) + 5.0 * t.clamp(min=0.0)
    gamma = x["discounts"].double()
    v_next = torch.cat([values[1:], bootstrap.unsqueeze(0)])
    delta = rho * (r + gamma * v_next - values)
    gc = gamma * c
    diff = torch.empty_like(values)
    acc = torch.zeros_like(bootstrap)
    for t in range(values.shape[0] - 1, -1, -1):
        acc = torch.addcmul(delta[t], gc[t], acc)
        diff[t] = acc
    vs = values + diff
    vs_next = torch.cat([vs[1:], bootstrap.unsqueeze(0)])
    adv = rho * (r + gamma * vs_next - values)
    return logp, log_pa, vs, adv


def _loss64(z, y_or_lp, values, bootstrap, x, case):
    """losses, d_logits and d_values in float64."""
    logp, log_pa, vs, adv = _targets64(z, y_or_lp, values, bootstrap, x, case)
    pi = logp.exp()
    ent = -(pi * logp).sum(-1)
    d_logits = adv.unsqueeze(-1) * pi
    d_logits.scatter_add_(-1, x["actions"].long().unsqueeze(-1), -adv.unsqueeze(-1))
    ce = float(torch.tensor(ENTROPY_COST, dtype=torch.float32))
    d_logits += ce * pi * (logp + ent.unsqueeze(-1))
    parts = torch.stack([-(adv * log_pa).sum(), BASELINE_COST * 0.5 * (vs - values).square().sum(),
                         -ce * ent.sum()])
    losses = torch.cat([parts.sum().unsqueeze(0), parts])
    return losses, d_logits, BASELINE_COST * (values - vs)


def exact(case, seed):
    x = _inputs(case, seed)
    T, B, A = case["T"], case["B"], case["A"]
    boot = x["bootstrap_value"].double()
    y = x["behaviour_logits"].double()
    if case["call"] == "targets":
        _, _, vs, adv = _targets64(x["target_logits"].double(), y, x["values"].double(), boot, x, case)
        return vs, adv
    if case["call"] == "loss":
        losses, dz, dv = _loss64(x["target_logits"].double(), y, x["values"].double(), boot, x, case)
        return losses, dz, dv, None, None, None
    hidden = x["hidden"].double().view(T * B, -1)
    w = x["head_weight"].double()
    o = (hidden @ w + x["head_bias"].double()).view(T, B, A + 1)
    losses, dz, dv = _loss64(o[..., :A].contiguous(), y, o[..., A].contiguous(), boot, x, case)
    g = torch.cat([dz, dv.unsqueeze(-1)], dim=-1).view(T * B, A + 1)
    d_hidden = (g @ w.t().contiguous()).view(T, B, -1)
    return losses, d_hidden, hidden.t().contiguous() @ g, g.sum(0), None, None, None, None
