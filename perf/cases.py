"""Workloads that the library's speed is measured on, through its public entry points.

Three families, each over the range of sizes a program meets:

  programs  batches of program trees, the library's step as a server runs it: the batch's programs are new every time,
            so a pass plans, uploads and executes; with "head" the classifier turns the root maps into answers
  train     the same with the backward pass: gradients of the feature maps and of every module parameter
  moe       one sparsely gated mixture-of-experts layer

Inputs follow the recipes of the benchmark configurations: programs of 10 to 30 tokens, mostly chains, 30 one-argument and
10 two-argument functions (or full binary trees over 8 two-argument functions), N(0,1) feature maps, He-normal weights
with the residual branch damped to a fifth at its last convolution, as networks of this kind are initialised and end
up (an undamped branch doubles the maps' variance at every one of up to 30 modules, and no such network answers anything);
training steps with non-negative maps and weights, every unit active (see _prepare_programs);
tokens with a shared component and gate columns shifted along it until the experts' load follows Zipf's law.
"""
from __future__ import annotations

import math
from collections import deque

import numpy as np
import torch

import paper_1707_02402_amd as dyn

SCHEDULES = {"balanced": dyn.DYNB_SCHED_IMPROVED | dyn.DYNB_PLAN_BALANCE, "improved": dyn.DYNB_SCHED_IMPROVED,
             "standard": dyn.DYNB_SCHED_STANDARD, "depth": dyn.DYNB_SCHED_DEPTH,
             "one_launch": dyn.DYNB_SCHED_IMPROVED | dyn.DYNB_PLAN_PERSISTENT}
HEAD = (32, 256, 28)        # channels after the 1x1 convolution, hidden units, answers


# ------------------------------------------------------------------------------------------ the cases
def _programs(name, B, dtype="bf16", C=128, side=14, trees="chains", schedule="balanced", head=False, kind="programs"):
    return dict(name=name, kind=kind, B=B, dtype=dtype, C=C, side=side, trees=trees, schedule=schedule, head=head)


def _moe(name, T, d, h, E, k, zipf, empty=0.0, noisy=True):
    return dict(name=name, kind="moe", T=T, d=d, h=h, E=E, k=k, zipf=zipf, empty=empty, noisy=noisy)


def listed():
    return [
        # one question about one picture: the latency of a single program, down to the answer
        _programs("answer_1", 1, head=True),
        # a few questions gathered by a server that will not wait for more
        _programs("answer_23", 23, head=True),
        # the smallest engine configuration: fp32, few channels, programs of at most 12 nodes (a test or teaching size)
        _programs("tiny_8_f32", 8, dtype="f32", C=16, side=8, trees="small"),
        # predetermined balanced trees, every internal node a two-argument function
        _programs("balanced_64", 64, trees="balanced"),
        # the headline minibatch
        _programs("programs_256", 256),
        # the batch up to which the method is expected to scale, with the classifier: offline evaluation of a test set
        _programs("programs_1000", 1000, head=True),
        # maps of a smaller backbone stage: the shape the general kernels serve in bf16
        _programs("programs_64_7x7", 64, side=7),
        # a training step of the headline minibatch (weights change every step: nothing is prepared)
        _programs("train_256", 256, kind="train"),
        # a training step in the full precision such networks are usually trained in, small batch
        _programs("train_21_f32", 21, dtype="f32", kind="train"),
        # generation: a handful of tokens, no gate noise, most experts idle
        _moe("moe_decode_37", 37, 512, 1024, 256, 2, 1.1, noisy=False),
        # a training or prefill batch of the small layer, noisy gate
        _moe("moe_4096", 4096, 512, 1024, 256, 2, 1.1),
        # the large layer: 1024 experts, crowded and empty ones
        _moe("moe_16384", 16384, 1024, 2048, 1024, 4, 1.2, empty=0.05),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    family = rng.choice(["programs", "programs", "programs", "train", "moe", "moe", "moe"])
    if family == "moe":
        while True:
            d, h = 8 * _log_int(rng, 8, 128), 8 * _log_int(rng, 8, 256)
            if rng.random() < 0.7:                       # widths are usually round
                d, h = (d + 63) // 64 * 64, (h + 63) // 64 * 64
            E = _log_int(rng, 8, 1024)
            k = min(E, rng.choice([1, 2, 2, 4, 4, 6, 8]))
            T = _log_int(rng, 1, 16384)
            if rng.random() < 0.5:
                T = max(1, T // 64 * 64)
            if T * k * d * h <= 16384 * 4 * 1024 * 2048:
                return dict(kind="moe", T=T, d=d, h=h, E=E, k=k, zipf=round(rng.uniform(0.6, 1.2), 2),
                            empty=rng.choice([0.0, 0.0, 0.05]) if E >= 64 else 0.0, noisy=rng.random() < 0.6)
    schedule = rng.choice(["balanced"] * 6 + ["improved", "standard", "depth", "one_launch"])
    shape = rng.choice(["fused", "fused", "fused", "f32", "other"])
    if shape == "fused":
        dtype, C, side, top = "bf16", 128, 14, (1000 if family == "programs" else 256)
    elif shape == "f32":
        dtype, C, side, top = "f32", rng.choice([16, 32, 64, 128]), rng.choice([7, 8, 14]), 21
    else:                                                # channel counts and sides of other backbones, odd ones among them
        dtype, C, side, top = rng.choice(["f32", "bf16"]), 2 * rng.randint(8, 64), rng.randint(5, 14), 21
    trees = rng.choice(["chains", "chains", "chains", "balanced", "small"])
    if trees == "balanced" and shape == "fused":
        top = min(top, 512)
    return dict(kind=family, B=_log_int(rng, 1, top), dtype=dtype, C=C, side=side, trees=trees, schedule=schedule,
                head=family == "programs" and rng.random() < 0.5)


# ------------------------------------------------------------------------------------------ program trees
def _arity(case):
    unary, binary = {"chains": (30, 10), "balanced": (0, 8), "small": (2, 2)}[case["trees"]]
    return np.array([0] + [1] * unary + [2] * binary, np.uint8)


def _draw_programs(case, seed):
    """Prefix sequences of function ids (0 = SCENE): (concatenated int32, offsets int32)."""
    g = np.random.Generator(np.random.Philox(key=[seed, 17]))
    ar = _arity(case)
    unary, binary = np.flatnonzero(ar == 1), np.flatnonzero(ar == 2)

    def chain():                                         # 10 to 30 tokens, a second argument now and then
        rem, open_, seq = int(g.integers(10, 31)), 1, []
        while rem > 0:
            if rem == open_ or (open_ >= 2 and g.random() < 0.10):
                seq.append(0)
                open_ -= 1
            elif rem >= open_ + 2 and g.random() < 0.15:
                seq.append(int(g.choice(binary)))
                open_ += 1
            else:
                seq.append(int(g.choice(unary)))
            rem -= 1
        return seq

    def full(levels):                                    # full binary tree
        return [0] if levels == 1 else [int(g.choice(binary))] + full(levels - 1) + full(levels - 1)

    def small(depth=0):                                  # at most 4 levels
        if depth == 3 or (depth > 0 and g.random() < 0.2):
            return [0]
        if g.random() < 0.5:
            return [int(g.choice(unary))] + small(depth + 1)
        return [int(g.choice(binary))] + small(depth + 1) + small(depth + 1)

    def small_tree():                                    # ... and at most 12 nodes
        while True:
            seq = small()
            if len(seq) <= 12:
                return seq

    make = {"chains": chain, "balanced": lambda: full(5), "small": small_tree}[case["trees"]]
    progs = [make() for _ in range(case["B"])]
    off = np.zeros(len(progs) + 1, np.int32)
    off[1:] = np.cumsum([len(p) for p in progs])
    return np.concatenate([np.asarray(p, np.int32) for p in progs]), off


class _Live:
    """Plans whose upload may still be running: a plan must outlive the copy that its upload enqueued."""

    def __init__(self):
        self.young, self.old = [], deque()

    def add(self, plan):
        self.young.append(plan)
        if len(self.young) == 32:
            done = torch.cuda.Event()
            done.record()
            self.old.append((done, self.young))
            self.young = []
            while len(self.old) > 1 and self.old[0][0].query():
                self.old.popleft()


def _prepare_programs(case, seed):
    train = case["kind"] == "train"
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    code = dyn.DYNB_BF16 if case["dtype"] == "bf16" else dyn.DYNB_F32
    B, C, S = case["B"], case["C"], case["side"]
    ar = _arity(case)
    n = len(ar)
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, std=1.0, dtype=dt, positive=False):
        v = torch.randn(*shape, generator=g, device="cuda") * std
        return (v.abs() if positive else v).to(dtype)

    # Gradients of a deep ReLU network are not continuous: where a stored activation next to zero rounds the other way, a unit
    # passes its gradient or does not, and with random signs two correct bf16 implementations differ by 8 % in every gradient.
    # Training steps therefore take the signs away: every unit is active, and the gradients can be compared.  The work is
    # the same.  (The mean of |N(0,1)| is 0.8; the scales below keep the maps near it: a convolution passes 0.8 * 0.3 of
    # its input's mean, a join averages.)
    if train:
        def pos(*shape, fan, gain):
            return normal(*shape, std=gain / (0.8 * fan), positive=True)

        weights = dict(w1=pos(n, C, 2 * C, fan=2 * C, gain=1.0), b1=normal(n, C, std=0.01, dtype=torch.float32, positive=True),
                       w3a=pos(n, C, 3, 3, C, fan=9 * C, gain=0.3), b3a=normal(n, C, std=0.01, dtype=torch.float32, positive=True),
                       w3b=pos(n, C, 3, 3, C, fan=9 * C, gain=0.3), b3b=normal(n, C, std=0.01, dtype=torch.float32, positive=True))
    else:
        weights = dict(w1=normal(n, C, 2 * C, std=math.sqrt(2 / (2 * C))), b1=normal(n, C, std=0.01, dtype=torch.float32),
                       w3a=normal(n, C, 3, 3, C, std=math.sqrt(2 / (9 * C))), b3a=normal(n, C, std=0.01, dtype=torch.float32),
                       w3b=normal(n, C, 3, 3, C, std=0.2 * math.sqrt(2 / (9 * C))), b3b=normal(n, C, std=0.01, dtype=torch.float32))
    feats = normal(B, S, S, C, positive=train)
    prog, off = _draw_programs(case, seed)
    flags = SCHEDULES[case["schedule"]] | (dyn.DYNB_PLAN_KEEP if train else 0)
    # buffers a program keeps from batch to batch, sized with this batch
    plan = dyn.dynbatch_plan(prog, off, ar, flags)
    st = dict(case=case, prog=prog, off=off, arity=ar, flags=flags, weights=weights, feats=feats, out=torch.empty_like(feats),
              dev_buf=torch.empty(dyn.dynbatch_plan_device_bytes(plan), dtype=torch.uint8, device="cuda"),
              ws=torch.empty(dyn.dynbatch_workspace_bytes(plan, C, S, S, code), dtype=torch.uint8, device="cuda"), live=_Live())
    if train:
        st["dout"] = normal(B, S, S, C, std=1.0 / B, dtype=torch.float32)
        st["bws"] = torch.empty(dyn.dynbatch_backward_workspace_bytes(plan, C, S, S, code), dtype=torch.uint8, device="cuda")
        f32 = lambda t: torch.empty(t.shape, dtype=torch.float32, device="cuda")
        st["grads"] = dict(dfeats=f32(feats), **{"d" + k: f32(weights[k]) for k in ("w1", "b1", "w3a", "b3a", "w3b", "b3b")})
    elif dyn.dynbatch_packed_weights_bytes(C, S, S, code, n) > 0:
        weights["packed"] = dyn.dynbatch_pack_weights(weights, C, S, S, code)     # constant weights, prepared once
    if case["head"]:
        Cc, F, A = HEAD
        st["head"] = dict(wc=normal(Cc, C, std=math.sqrt(2 / C)), bc=normal(Cc, std=0.01, dtype=torch.float32),
                          wf1=normal(F, S * S * Cc, std=math.sqrt(2 / (S * S * Cc))), bf1=normal(F, std=0.01, dtype=torch.float32),
                          wf2=normal(A, F, std=math.sqrt(2 / F)), bf2=normal(A, std=0.01, dtype=torch.float32))
        st["head_ws"] = torch.empty(dyn.dynbatch_classify_workspace_bytes(C, S, S, code, Cc, F, A, B), dtype=torch.uint8, device="cuda")
        st["probs"] = torch.empty(B, A, dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()                             # (the plan is dropped here: it was never uploaded)
    return st


def _run_programs(st):
    plan = dyn.dynbatch_plan(st["prog"], st["off"], st["arity"], st["flags"])
    dyn.dynbatch_plan_upload(plan, st["dev_buf"])
    out = dyn.dynbatch_execute(plan, st["weights"], st["feats"], out=st["out"], workspace=st["ws"])
    result = [out]
    if "grads" in st:
        grads = dyn.dynbatch_backward(plan, st["weights"], st["feats"], out, st["ws"], st["dout"], workspace=st["bws"], grads=st["grads"])
        result += [grads[k] for k in ("dfeats", "dw1", "db1", "dw3a", "db3a", "dw3b", "db3b")]
    if "head" in st:
        result.append(dyn.dynbatch_classify(out, st["head"], probs=st["probs"], workspace=st["head_ws"]))
    st["live"].add(plan)
    return result


def _work_programs(case):
    train = case["kind"] == "train"
    B, C, P = case["B"], case["C"], case["side"] ** 2
    elt = 2 if case["dtype"] == "bf16" else 4
    ar = _arity(case)
    prog, _ = _draw_programs(case, 1)                    # programs of the recipe: their mix varies little with the seed
    n1, n2 = int((ar[prog] == 1).sum()), int((ar[prog] == 2).sum())
    flops = (n1 + n2) * 2 * 2 * P * C * 9 * C + n2 * 2 * P * C * 2 * C
    used = np.unique(prog)
    params = sum(18 * C * C + (2 * C * C if ar[t] == 2 else 0) for t in used if ar[t] > 0)
    data = 2 * B * P * C * elt + params * elt
    if train:                                            # two transposed convolutions and two contractions per convolution pair
        flops *= 3
        data += B * P * C * 8 + len(ar) * (20 * C * C + 3 * C) * 4           # dout, dfeats, every parameter's gradient
    if case["head"]:
        Cc, F, A = HEAD
        flops += 2 * B * (P * C * Cc + P * Cc * F + F * A)
        data += (Cc * C + F * P * Cc + A * F) * elt + B * A * 4
    return {"bytes": data, "flops": flops}


# ------------------------------------------------------------------------------------------ mixture of experts
def _zipf_target(case):
    """Expected uses per active expert, most used first."""
    n = case["E"] - int(case["empty"] * case["E"])
    w = np.arange(1, n + 1, dtype=np.float64) ** -case["zipf"]
    return np.minimum(w / w.sum() * case["T"] * case["k"], 0.98 * case["T"])


def _prepare_moe(case, seed):
    T, d, h, E, k = (case[x] for x in ("T", "d", "h", "E", "k"))
    g = torch.Generator(device="cuda").manual_seed(seed)
    randn = lambda *s: torch.randn(*s, generator=g, device="cuda")
    # x = sqrt(3/4) z + sqrt(1/4) c with a direction c that all tokens share: a bias-free linear gate can then prefer an
    # expert for most tokens.  The gate columns' shifts along c are fitted on at least 2048 tokens until the load follows
    # the target; experts that are to stay empty get zero columns and a strongly negative noise (or, without noise, a
    # strongly negative shift).
    n_fit = max(T, 2048)
    c = randn(d)
    x_fit = (math.sqrt(0.75) * randn(n_fit, d) + 0.5 * c).to(torch.bfloat16)
    G, Wn = randn(E, d) / math.sqrt(d), (0.1 * randn(E, d) / math.sqrt(d)).to(torch.bfloat16)
    noise = randn(n_fit, E)
    order = torch.randperm(E, generator=g, device="cuda")
    t = torch.from_numpy(_zipf_target(case)).to("cuda", torch.float32) * (n_fit / T)
    active, idle = order[:len(t)], order[len(t):]
    target = torch.zeros(E, device="cuda")
    target[active] = t
    Wn[idle] = 0
    noise[:, idle] = -64.0
    u = c / (c @ c)
    xf = x_fit.float()
    shift = xf @ u
    G[idle] = 0 if case["noisy"] else (-64.0 * u).expand(len(idle), d)
    fixed = xf @ G.T
    if case["noisy"]:
        fixed += noise * torch.nn.functional.softplus(xf @ Wn.float().T)
    beta = torch.zeros(E, device="cuda")
    for _ in range(30):
        load = torch.bincount(torch.topk(fixed + shift[:, None] * beta, k, dim=1).indices.flatten(), minlength=E)
        step = 0.7 * torch.log((target + 1) / (load + 1))
        step[idle] = 0
        beta += step
    Wg = (G + beta[:, None] * u).to(torch.bfloat16)
    st = dict(case=case, x=x_fit[:T].contiguous(), Wg=Wg, Wn=Wn if case["noisy"] else None,
              noise=noise[:T].contiguous() if case["noisy"] else None, out=torch.empty(T, d, dtype=torch.bfloat16, device="cuda"),
              ws=torch.empty(dyn.moe_workspace_bytes(T, d, h, E, k), dtype=torch.uint8, device="cuda"))
    for name, rows, cols in (("W1", h, d), ("W2", d, h)):
        w = torch.empty(E, rows, cols, dtype=torch.bfloat16, device="cuda")
        part = max(1, (1 << 27) // (rows * cols))        # experts per piece: half a gigabyte of fp32
        for e in range(0, E, part):
            m = min(part, E - e)
            w[e:e + m] = randn(m, rows, cols) * math.sqrt(2 / cols)
        st[name] = w
    torch.cuda.synchronize()
    return st


def _run_moe(st):
    return dyn.moe_forward(st["x"], st["Wg"], st["Wn"], st["noise"], st["W1"], st["W2"], st["case"]["k"], out=st["out"], workspace=st["ws"])


def _work_moe(case):
    T, d, h, E, k = (case[x] for x in ("T", "d", "h", "E", "k"))
    gates = 2 if case["noisy"] else 1
    used = float((1 - np.exp(-_zipf_target(case))).sum())                     # experts with at least one use
    return {"bytes": 2 * T * d * 2 + gates * E * d * 2 + (T * E * 4 if case["noisy"] else 0) + used * 2 * d * h * 2,
            "flops": gates * 2 * T * d * E + T * k * 4 * d * h}


# ------------------------------------------------------------------------------------------ the interface
def prepare(case, seed):
    return _prepare_moe(case, seed) if case["kind"] == "moe" else _prepare_programs(case, seed)


def run(state):
    return _run_moe(state) if state["case"]["kind"] == "moe" else _run_programs(state)


def work(case):
    return _work_moe(case) if case["kind"] == "moe" else _work_programs(case)


def tolerance(case):
    """Measured by taking the channels (model and hidden widths) in another order: the same results with every sum in another
    order; about four times the largest relative difference of any output over seeds and sizes of a kind."""
    if case["kind"] == "moe":
        # 2e-4 from hidden rows and outputs that round to the neighbouring bfloat16; in a large batch a token or two may have
        # two gate logits within 1e-6 of each other and take another last expert
        return {"rel": 1e-3 if case["T"] <= 512 else 1e-3 + 0.7 / math.sqrt(case["T"])}
    if case["kind"] == "train":                          # 1.5e-4 in bf16, 6e-7 in fp32: no ReLU decision depends on a rounding
        return {"rel": 1e-3 if case["dtype"] == "bf16" else 3e-6}
    if case["dtype"] == "f32":                           # 1e-6
        return {"rel": 5e-6}
    # stored activations that round to the neighbouring bfloat16, module after module (5.5e-3, 2.9e-3, 1.1e-3 by depth; 9e-3,
    # 6e-3, 5e-3 in the probabilities)
    depth = {"chains": 0, "balanced": 1, "small": 2}[case["trees"]]
    return {"rel": ((3e-2, 2.4e-2, 2e-2) if case["head"] else (2.2e-2, 1.2e-2, 5e-3))[depth]}
