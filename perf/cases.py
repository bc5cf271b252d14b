"""What the time of this library is measured on: passes of the population step as a training loop makes them.

A training loop calls `pbt_step` for every mini-batch (or once for a whole ready interval of a small fp32
population) and, when a member is ready, `pbt_eval` followed by `pbt_exploit_explore`.  Those are the two kinds of
pass here: "step" and "ready".  The listed cases are the workloads of `paper_1711_09846_amd/workloads.py` at their own
sizes, plus sizes that fit no tile; `draw` gives further populations of the same families, from a few small members up
to the sizes of the workload descriptions.
"""
import math

import torch

from paper_1711_09846_amd import binding, workloads as W

FAMILIES = {"mlp_fp32": W.MLP_SMALL, "mlp_bf16": W.MLP_WIDE, "gan": W.GAN_MLP, "transformer": W.TRANSFORMER, "a2c": W.A2C_MLP}
ACTS = {"relu": W.ACT_RELU, "gelu": W.ACT_GELU, "leaky_relu": W.ACT_LEAKY_RELU, "tanh": W.ACT_TANH}
OPTIMIZERS = {"sgd": (W.OPT_SGD_MOMENTUM, dict(momentum=0.9)), "adam": (W.OPT_ADAM, dict(beta1=0.9, beta2=0.999, eps=1e-8)),
              "rmsprop": (W.OPT_RMSPROP, dict(rho=0.99, eps=1e-5))}


def listed():
    mlp, wide, gan, tf, a2c = W.MLP_SMALL, W.MLP_WIDE, W.GAN_MLP, W.TRANSFORMER, W.A2C_MLP
    text = lambda dims: "-".join(str(d) for d in dims)  # noqa: E731
    wide_case = dict(family="mlp_bf16", P=wide.P, dims=text(wide.dims), act="gelu", optimizer="adam", fused=True, batch=wide.batch,
                     n_train=wide.n_train, n_eval=wide.n_eval, n_trunc=wide.n_trunc)
    gan_case = dict(family="gan", P=gan.P, dims=text(gan.dims), dims2=text(gan.dims2), batch=gan.batch, objective="logistic",
                    n_train=gan.n_train, n_eval=gan.n_eval, n_trunc=gan.n_trunc)
    tf_case = dict(family="transformer", P=tf.P, vocab=tf.vocab, d_model=tf.d_model, heads=tf.heads, d_ff=tf.d_ff, blocks=tf.n_blocks,
                   seq=tf.seq, batch=tf.batch, n_train=tf.n_train, n_eval=tf.n_eval, n_trunc=tf.n_trunc)
    small_case = dict(family="mlp_fp32", P=mlp.P, dims=text(mlp.dims), act="relu", optimizer="sgd", batch=mlp.batch, n_train=mlp.n_train,
                      n_eval=mlp.n_eval, n_trunc=mlp.n_trunc)
    return [
        # the small fp32 population: one call runs a whole ready interval of 50 steps
        dict(small_case, name="small_interval", op="step", n_steps=mlp.ready_interval),
        # its ready point, the smallest work a loop asks for: latency of the calls
        dict(small_case, name="small_ready", op="ready"),
        # wide MLPs, Adam inside the weight-gradient pass (the benchmark's setting): bound by the optimiser state's traffic
        dict(wide_case, name="wide_step", op="step"),
        # their ready point: 8192 held-out rows through every member, a fifth of the population copied
        dict(wide_case, name="wide_ready", op="ready"),
        # fewer members with widths and a batch that fill no tile, RMSProp as a pass of its own
        dict(wide_case, name="ragged_step", op="step", P=21, dims="200-712-360-7", act="tanh", optimizer="rmsprop", fused=False, batch=75,
             n_train=5000, n_eval=1000, n_trunc=4),
        # GAN pairs, one discriminator and one generator update
        dict(gan_case, name="gan_step", op="step"),
        # the same pairs with five critic updates on the WGAN-GP objective per generator update
        dict(gan_case, name="wgan_step", op="step", objective="wgan_gp"),
        # the GAN population's ready point: MMD between 2048 generated and held-out rows
        dict(gan_case, name="gan_ready", op="ready"),
        # the largest workload: 16 transformers, 4096 positions each
        dict(tf_case, name="transformer_step", op="step"),
        # its ready point: perplexity over 256 held-out sequences
        dict(tf_case, name="transformer_ready", op="ready"),
        # a small language-model population: 32-wide heads, sizes that are multiples of 8 and of nothing larger
        dict(tf_case, name="transformer_small_step", op="step", P=6, vocab=1000, d_model=192, heads=6, d_ff=776, blocks=2, seq=72, batch=10,
             n_train=500, n_eval=20, n_trunc=1),
        # agents acting with their current policy, then one update on the unroll
        dict(family="a2c", name="a2c_step", op="step", P=a2c.P, dims=text(a2c.dims), batch=a2c.batch, unroll=a2c.unroll, on_policy=True,
             latent=a2c.latent, n_train=a2c.n_train, n_trunc=a2c.n_trunc),
    ]


def draw(rng):
    """One more population of a random family, sizes log-uniform in the ranges up to the listed ones."""
    log = lambda lo, hi, by=1: max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / by)) * by)  # noqa: E731
    family = rng.choice(["mlp_fp32", "mlp_bf16", "mlp_bf16", "gan", "transformer", "a2c"])
    op = "step" if rng.random() < 0.7 else "ready"
    if family == "mlp_fp32":
        P = log(2, 32)
        hidden = [log(12, 96)] if rng.random() < 0.6 else [log(12, 64), log(12, 64)]
        widths = [log(8, 64)] + hidden + [rng.randint(2, 10)]
        optimizer = rng.choice(sorted(OPTIMIZERS))
        batch = log(16, 96)
        # members of this family live in one compute unit's LDS: parameters, optimiser state and a batch of activations
        params = sum(a * b + b for a, b in zip(widths[:-1], widths[1:]))
        while 3 * params + 4 * batch * (sum(widths) + len(widths)) > 36000:
            batch -= 4
        c = dict(family=family, op=op, P=P, dims="-".join(map(str, widths)), act=rng.choice(sorted(ACTS)), optimizer=optimizer, batch=batch,
                 n_train=log(256, 4096), n_eval=log(100, 1024), n_trunc=max(1, P // 4))
        return dict(c, n_steps=rng.randint(10, 50)) if op == "step" else c
    if family == "mlp_bf16":
        P = log(4, 64)
        widths = [log(64, 512, 8)] + [log(64, 1024, 8) for _ in range(rng.choice([1, 2, 2]))] + [rng.randint(2, 32)]
        return dict(family=family, op=op, P=P, dims="-".join(map(str, widths)), act=rng.choice(sorted(ACTS)), optimizer=rng.choice(sorted(OPTIMIZERS)),
                    fused=rng.random() < 0.5, batch=log(16, 128), n_train=log(1000, 65536), n_eval=log(500, 8192), n_trunc=max(1, P // 5))
    if family == "gan":
        P = log(4, 32)
        data = log(64, 784, 8)
        g = [log(32, 128, 8), log(128, 512, 8), log(128, 512, 8), data]
        d = [data, log(128, 512, 8), log(128, 512, 8), 1]
        return dict(family=family, op=op, P=P, dims="-".join(map(str, g)), dims2="-".join(map(str, d)), batch=log(16, 64),
                    objective=rng.choice(["logistic", "wgan_gp"]), n_train=log(1000, 65536), n_eval=log(200, 2048), n_trunc=max(1, P // 5))
    if family == "transformer":
        P = log(2, 16)
        width = rng.choice([32, 64, 64])
        heads = rng.randint(2, 512 // width)
        d = width * heads
        batch = log(4, 32)
        return dict(family=family, op=op, P=P, vocab=log(256, 8192, 8), d_model=d, heads=heads, d_ff=min(2048, d * rng.choice([2, 3, 4])),
                    blocks=rng.randint(1, 4), seq=log(32, 128, 8), batch=batch, n_train=log(100, 8192), n_eval=batch * rng.randint(1, 8),
                    n_trunc=max(1, P // 5))
    P = log(8, 128)
    hidden = [rng.choice([64, 128, 256, log(64, 256, 8)]) for _ in range(2)]
    return dict(family="a2c", op=op, P=P, dims="-".join(map(str, [64 * rng.randint(1, 8)] + hidden + [rng.randint(3, 24)])), batch=rng.randint(8, 32),
                unroll=rng.randint(5, 20), on_policy=rng.random() < 0.7, latent=rng.randint(4, 16), n_train=log(256, 4096), n_trunc=max(1, P // 5))


def _dims(text):
    return [int(d) for d in text.split("-")]


def _workload(case):
    """The workload description of a case: the family's own with the case's sizes and options."""
    base, family = FAMILIES[case["family"]], case["family"]
    kw = dict(P=case["P"], batch=case["batch"], n_train=case["n_train"], n_eval=case.get("n_eval", 1), n_trunc=case["n_trunc"])
    if family == "transformer":
        kw.update(vocab=case["vocab"], d_model=case["d_model"], heads=case["heads"], d_ff=case["d_ff"], n_blocks=case["blocks"], seq=case["seq"])
        return base.replace(**kw)
    kw["dims"] = _dims(case["dims"])
    if family in ("mlp_fp32", "mlp_bf16"):
        kw["optimizer"], kw["opt_const"] = OPTIMIZERS[case["optimizer"]]
        kw["act"], kw["n_classes"] = ACTS[case["act"]], kw["dims"][-1]
        if case["optimizer"] != "adam":     # beta1 and weight decay belong to Adam: the learning rate alone is adapted
            kw.update(roles=[W.ROLE_LR], priors=[("log", 1e-4, 1e-2)], h_max=[math.inf])
        elif family == "mlp_fp32":
            kw.update(priors=[("log", 1e-4, 1e-2)])
    elif family == "gan":
        kw["dims2"] = _dims(case["dims2"])
        if case["objective"] == "wgan_gp":
            kw.update(objective="wgan_gp", n_critic=W.GAN_MLP_WGAN_GP.n_critic, gp_weight=W.GAN_MLP_WGAN_GP.gp_weight, perturb=(0.5, 2.0))
    else:
        kw.update(unroll=case["unroll"], latent=case["latent"], n_actions=kw["dims"][-1] - 1, on_policy=1 if case["on_policy"] else 0)
    return base.replace(**kw)


def _inputs(wl, family, gen):
    """(training inputs, held-out inputs) on the GPU, with the distributions of workloads.py's generators."""
    normal = lambda *shape, **kw: torch.randn(*shape, generator=gen, device="cuda", **kw)  # noqa: E731
    ints = lambda hi, *shape: torch.randint(hi, shape, generator=gen, device="cuda")       # noqa: E731
    if family in ("mlp_fp32", "mlp_bf16"):
        means = normal(wl.n_classes, wl.dims[0])
        out = []
        for n in (wl.n_train, wl.n_eval):
            y = ints(wl.n_classes, n)
            out.append([means[y] + normal(n, wl.dims[0]), y.int()])
        return out[0], out[1]
    if family == "gan":
        d = wl.dims2[0]
        mu, A = normal(wl.n_modes, d) * 0.25, normal(wl.n_modes, wl.rank, d) * (0.25 / math.sqrt(wl.rank))
        out = []
        for n in (wl.n_train, wl.n_eval):
            k = torch.sort(ints(wl.n_modes, n)).values     # rows are filled mode by mode, then shuffled
            x = torch.cat([mu[m] + normal(int(c), wl.rank) @ A[m] for m, c in enumerate(torch.bincount(k, minlength=wl.n_modes).tolist())])
            out.append([x[torch.randperm(n, generator=gen, device="cuda")].contiguous()])
        return out[0], out[1]
    if family == "transformer":
        V, T = wl.vocab, wl.seq + 1
        cdf = torch.cumsum(1.0 / torch.arange(1, V + 1, device="cuda", dtype=torch.float64) ** wl.zipf_s, 0)
        cdf, pi = cdf / cdf[-1], torch.randperm(V, generator=gen, device="cuda")
        out = []
        for n in (wl.n_train, wl.n_eval):
            z = torch.searchsorted(cdf, torch.rand(n, T, generator=gen, device="cuda", dtype=torch.float64)).clamp_(max=V - 1)
            x = [z[:, 0]]
            for t in range(1, T):
                x.append((pi[x[-1]] + z[:, t]) % V)
            out.append([torch.stack(x, 1).int().contiguous()])
        return out[0], out[1]
    nz, d, T, n = wl.latent, wl.dims[0], wl.unroll, wl.n_train
    f64 = dict(dtype=torch.float64)
    A = 0.9 * torch.linalg.qr(torch.randn(nz, nz, generator=gen, device="cuda", **f64).cpu())[0].cuda()
    B, C, w = normal(nz, wl.n_actions, **f64) * 0.3, normal(d, nz, **f64) / 4.0, normal(nz, **f64)
    if wl.on_policy:
        return [A.contiguous(), B.contiguous(), C.contiguous(), w.contiguous(), torch.tensor([1.0, 0.1, 0.1], device="cuda", **f64)], []
    z, act = normal(n, nz, **f64), ints(wl.n_actions, n, T)
    obs, rew = torch.empty(n, T + 1, d, device="cuda"), torch.empty(n, T, device="cuda")
    for t in range(T + 1):
        obs[:, t] = (z @ C.T).float() + normal(n, d)
        if t < T:
            rew[:, t] = (z @ w).float() + 0.1 * normal(n)
            z = z @ A.T + B[:, act[:, t]].T + 0.1 * normal(n, nz, **f64)
    return [obs, act.int(), rew], []


UPDATES = 100


def _grad_rms(wl, family):
    """Size of a gradient element in a run of the workload: the scale of the optimiser state prepared below."""
    if family == "gan":
        return 0.1 if getattr(wl, "objective", "") == "wgan_gp" else 4e-4
    if family == "transformer":
        return 0.06 / math.sqrt(wl.batch * wl.seq)
    return {"mlp_fp32": 1e-2, "mlp_bf16": 1e-3, "a2c": 2e-2}[family]


def _part_way(pop, wl, family, gen):
    """Optimiser state of a population part-way through training (padding stays zero): mean squares spread around the
    square of _grad_rms, first moments a third of their root.  (From all-zero state Adam's first update is +-lr whatever
    the size of the gradient, so two correct implementations would part there by the sign of every near-zero element.)"""
    lay, rms = pop.layout, _grad_rms(wl, family)
    used = torch.zeros(lay.stride, device="cuda")
    for k in range(lay.n_seg):
        used[lay.seg_off[k]:lay.seg_off[k] + lay.seg_len[k]] = 1
    square = torch.randn(wl.P, lay.stride, generator=gen, device="cuda").mul_(0.5).exp_().mul_(used * rms ** 2)
    opt0 = pop.device_view(binding.ARR_OPT0)
    if wl.optimizer == W.OPT_RMSPROP:
        opt0.copy_(square)
    else:
        opt0.normal_(generator=gen).mul_(square.sqrt()).mul_(0.3 if wl.optimizer == W.OPT_ADAM else 2.0)
    if wl.optimizer == W.OPT_ADAM:
        pop.device_view(binding.ARR_OPT1).copy_(square)
    pop.device_view(binding.ARR_T).fill_(UPDATES)
    if family == "a2c":
        hist = pop.device_view(binding.ARR_HIST)
        hist[:, :10].normal_(generator=gen)
        hist.view(torch.int32)[:, 10] = UPDATES


def prepare(case, seed):
    """A population drawn from its priors, with the optimiser state of a run part-way through, and its data sets in
    device memory, as a program holds them inside its loop."""
    family = case["family"]
    wl = _workload(case)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    pop = binding.Population(binding.make_config(wl, seed, fuse_optimizer=1 if case.get("fused") else 0))
    pop.init_population(wl.priors)
    _part_way(pop, wl, family, gen)
    train, held_out = _inputs(wl, family, gen)
    arrays = dict(theta=binding.ARR_W32, opt0=binding.ARR_OPT0, t=binding.ARR_T)
    if wl.optimizer == W.OPT_ADAM:
        arrays["opt1"] = binding.ARR_OPT1
    if case["op"] == "ready":
        arrays.update(hyper=binding.ARR_HYPER, order=binding.ARR_ORDER, donor=binding.ARR_DONOR, parent=binding.ARR_PARENT)
    else:
        arrays["loss"] = binding.ARR_LOSS
        # (the transformer's gradient is judged through the state it goes into: reordered sums put one ReLU gate in a
        # thousand on the other side, which by itself moves the gradient by the root of that, 3 %)
        if not case.get("fused") and family != "transformer":
            arrays["grad"] = binding.ARR_GRAD
        # (an action whose draw lies within rounding of a step of its distribution may differ, and with it the rest of
        # that trajectory: observations and rewards are judged through what is learnt from them)
        if family == "a2c":
            arrays.update(history=binding.ARR_HIST, actions=binding.ARR_TRAJ_ACT)
    state = dict(pop=pop, op=case["op"], n_steps=case.get("n_steps", 1), train=train, held_out=held_out, at=UPDATES,
                 out={k: pop.device_view(a) for k, a in arrays.items()})
    if family == "a2c" and case["op"] == "step":
        state["out"]["history"] = state["out"]["history"][:, :10]      # (the rest of a row is the count)
    if case["op"] == "ready":
        state["score"] = pop.device_view(binding.ARR_SCORE)
        # the selection goes by a score of the program's own (pbt_exploit_explore takes one from the caller), no two alike
        state["fitness"] = torch.randperm(wl.P, generator=gen, device="cuda").float()
    return state


def run(state):
    pop = state["pop"]
    if state["op"] == "step":
        pop.step(state["train"], state["at"], n_steps=state["n_steps"])
        state["at"] += state["n_steps"]
        return state["out"]
    pop.eval(state["held_out"])
    score = state["score"].clone()          # what the program logs; the exploit pass overwrites the array
    pop.exploit_explore(state["at"], state["fitness"])
    state["at"] += 1
    return dict(state["out"], score=score)


def _mats(dims):
    return sum(a * b for a, b in zip(dims[:-1], dims[1:]))


def work(case):
    """Bytes: parameters, optimiser state and the bf16 copy read and written once, the rows drawn, the copied members.
    Flops: the products of the passes over the network (an input gradient is not formed below the first layer)."""
    wl, family, P, B = _workload(case), case["family"], case["P"], case["batch"]
    adam = wl.optimizer == W.OPT_ADAM
    state = 4 * (3 if adam else 2) + (2 if wl.dtype == W.DTYPE_BF16 else 0)       # bytes held per parameter
    update = 2 * state - (2 if wl.dtype == W.DTYPE_BF16 else 0)                   # theta and state read and written, the copy written
    if family == "transformer":
        d, f, V, S, L = wl.d_model, wl.d_ff, wl.vocab, wl.seq, wl.n_blocks
        n = V * d + S * d + L * (4 * d * d + 2 * d * f + 9 * d + f) + 2 * d + d * V + V
        dense, att = L * (4 * d * d + 2 * d * f) + d * V, L * S * d      # per position: multiply-adds of the layers; of one (causal) attention product pair
        if case["op"] == "step":
            return dict(bytes=P * (update * n + 8 * B * S), flops=2 * P * B * S * (3 * dense + 3 * att))
        return dict(bytes=P * 2 * n + 4 * wl.n_eval * (S + 1) + 2 * state * n * wl.n_trunc, flops=2 * P * wl.n_eval * S * (dense + att))
    m = _mats(wl.dims)
    n = m + sum(wl.dims[1:])
    if family == "gan":
        md, first = _mats(wl.dims2), wl.dims2[0] * wl.dims2[1]
        n += md + sum(wl.dims2[1:])
        K = getattr(wl, "n_critic", 1)
        if case["op"] == "ready":
            E, D = wl.n_eval, wl.dims2[0]
            return dict(bytes=P * 2 * n + 4 * E * D + 2 * state * n * wl.n_trunc, flops=P * E * (2 * m + 3 * E * D))   # (one Gram matrix is symmetric)
        gen = 2 * P * B * (3 * m - wl.dims[0] * wl.dims[1] + 2 * md)
        if K == 1:
            dis = 2 * P * B * (m + 2 * (3 * md - first))
        else:
            dis = 2 * P * B * K * (m + 3 * (3 * md - first) + first + md)
        return dict(bytes=P * (update * n + 4 * K * B * wl.dims2[0]), flops=gen + dis)
    if family == "a2c":
        R = B * (wl.unroll + 1)
        if case["op"] == "ready":
            return dict(bytes=2 * state * n * wl.n_trunc, flops=P)
        rows = R * wl.dims[0]
        return dict(bytes=P * (update * n + (2 if wl.on_policy else 6) * rows),
                    flops=2 * P * R * (3 * m - wl.dims[0] * wl.dims[1] + (m if wl.on_policy else 0)))
    if case["op"] == "ready":
        return dict(bytes=P * (2 if wl.dtype else 4) * n + 4 * wl.n_eval * (wl.dims[0] + 1) + 2 * state * n * wl.n_trunc, flops=2 * P * wl.n_eval * m)
    steps = case.get("n_steps", 1)
    drawn = min(steps * P * B, wl.n_train) if steps > 1 else P * B
    return dict(bytes=P * update * n + 4 * drawn * (wl.dims[0] + 1), flops=2 * steps * P * B * (3 * m - wl.dims[0] * wl.dims[1]))


def tolerance(case):
    """About four times what the outputs move when every contraction adds up its products in reverse order (listed cases
    and draws), over two passes: fp32 2e-7 to 2e-6; bf16 networks 1e-5 to 2e-3, most of it activations' gates and bf16
    roundings that fall on the other side; WGAN-GP and transformers, whose gradients add up such differences over five
    updates or eight branches, 8e-3."""
    family = case["family"]
    if family == "mlp_fp32":
        return {"rel": 1e-5}
    if family == "transformer" or case.get("objective") == "wgan_gp":
        return {"rel": 0.03, "max": 0.9}
    if family == "a2c":
        return {"rel": 0.015, "max": 0.9, "differ": 1e-3}
    return {"rel": 0.01, "max": 0.7}
