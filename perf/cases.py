"""The work a user of this framework has it do, as cases that can be timed and checked.

A training program steps one pipeline stage of n parameters in R replicas (`Stage.step`, with clipping
`Stage.grad_sqnorm` + `Stage.step_scaled`), or steps its weights itself and asks for the averaging alone
(`Stage.sparse_average`); around that it extrapolates weights (`lookahead`), lists a round's subset
(`Stage.subset_indices_static`) and watches the replicas drift (`Stage.diagnostics`).  Every case names
one of these calls with its sizes and options:

  n, R, tau, K, p          parameters, replicas, delay in rounds, averaging interval, subset fraction
  opt                      "sgd" (momentum 0.9), "adamw" (0.9, 0.999), "nadamw" (0.99, 0.999)
  lookahead, corr, bf16    look-ahead on; "ema" or "none"; bf16 gradients and forward weights
  interleaved              layout of the EMA vectors (default of the framework: one array per replica)
  clip                     every replica clips its gradient to norm 1 first
"""
import math

import numpy as np
import torch

import paper_2601_22442_amd as am

LR, SGD_LR, LAMBDA, GAMMA = 3e-4, 0.1, 0.5, 0.9
W_STD, G_STD = 0.02, 1e-3                # GPT-2 style initial weights, gradients of the evaluated runs
OPT = {"sgd": (am.OPT_SGD, 0.9, 0.0), "adamw": (am.OPT_ADAMW, 0.9, 0.999), "nadamw": (am.OPT_NADAMW, 0.99, 0.999)}
EPS, WEIGHT_DECAY, MOMENTUM_DECAY = 1e-8, 0.01, 0.004
STAGE = 125_829_120                      # 2.5 transformer layers at d = 2048
LARGEST = 16 * STAGE                     # parameters x replicas of the largest step


def _step(name, n, R, tau, p, K=1, opt="adamw", lookahead=False, corr="ema", bf16=False, interleaved=False, clip=False):
    return dict(name=name, call="step", n=n, R=R, tau=tau, K=K, p=p, opt=opt, lookahead=lookahead, corr=corr, bf16=bf16,
                interleaved=interleaved, clip=clip)


def listed():
    return [
        # The 1M configuration with the framework's defaults: every call is short, so launches and the
        # host's part of a call count.
        _step("step_tiny", 1_048_576, 4, 1, 0.05),
        # Two transformer layers at d = 768 with the optimizer of the asynchronous pipelines.
        _step("step_small", 7_077_888, 4, 2, 0.10, opt="nadamw", lookahead=True, interleaved=True),
        # The headline: one stage of a 1B-class model, eight replicas.
        _step("step_stage125m", STAGE, 8, 4, 0.05, lookahead=True, interleaved=True),
        # The same stage in bf16 with sixteen replicas and the plain delayed average at 1 %: the largest.
        _step("step_bf16_r16", STAGE, 16, 8, 0.01, corr="none", bf16=True),
        # Clipping by each replica's own norm, an odd size, and one EMA array per replica, as a replica
        # that keeps its arrays flat has them.
        _step("step_clipped", 31_457_281, 8, 4, 0.05, lookahead=True, clip=True),
        # One round at an averaging interval of five: four local steps and one that averages (SGD with
        # momentum, two replicas, odd size).
        _step("round_k5_sgd", 3_000_017, 2, 2, 0.10, K=5, opt="sgd"),
        # Synchronous sparse averaging (no delay, nothing to correct) over a ragged second block of replicas.
        _step("step_sync_r12", 7_077_891, 12, 0, 0.05, corr="none"),
        # The averaging alone on the headline stage, for a program with an optimizer of its own, ...
        dict(name="average_stage125m", call="average", n=STAGE, R=8, tau=4, p=0.05, corr="ema", interleaved=True),
        # ... and on a small stage with the default layout.
        dict(name="average_tiny", call="average", n=1_048_576, R=4, tau=1, p=0.01, corr="ema", interleaved=False),
        # Consensus error and EMA variance of a stage, looked at while training.
        dict(name="diagnostics", call="diagnostics", n=31_457_281, R=8, corr="ema", interleaved=True),
        # The index list of one round's subset, as a program exchanges or logs it.
        dict(name="indices_stage125m", call="indices", n=STAGE, p=0.05),
        # The stateless look-ahead of one replica's weights to bf16 (two layers at d = 1024, odd).
        dict(name="lookahead_bf16", call="lookahead", n=25_165_823, bf16=True),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["step"] * 6 + ["average"] * 2 + ["diagnostics", "indices", "lookahead"])
    p = round(math.exp(rng.uniform(math.log(0.005), math.log(0.2))), 4)
    if call == "lookahead":
        return dict(call=call, n=_size(rng, 100_003, 2 * STAGE), bf16=rng.random() < 0.5)
    if call == "indices":
        return dict(call=call, n=_size(rng, 100_003, STAGE), p=p)
    R = rng.choice([1, 2, 3, 4, 4, 6, 8, 8, 8, 12])
    n = _size(rng, 100_003, min(STAGE, LARGEST // (2 * R)))
    corr, interleaved = rng.choice(["ema", "ema", "ema", "none"]), rng.random() < 0.5
    if call == "diagnostics":
        return dict(call=call, n=n, R=R, corr=corr, interleaved=interleaved)
    tau = rng.choice([0, 1, 2, 4, 8])
    if call == "average":
        return dict(call=call, n=n, R=R, tau=tau, p=p, corr=corr, interleaved=interleaved)
    bf16 = rng.random() < 0.3
    case = _step("", n, R, tau, p, K=rng.choice([1, 1, 1, 1, 2, 4]), opt=rng.choice(["adamw", "adamw", "nadamw", "sgd"]),
                 lookahead=rng.random() < 0.5, corr=corr, bf16=bf16, interleaved=interleaved, clip=rng.random() < 0.25)
    if case["K"] > 1:
        case["n"] = max(100_003, n // 8)
    del case["name"]
    return case


# ---------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------
def _generator(seed, *key):
    g = torch.Generator(device="cuda")
    g.manual_seed(hash((int(seed),) + key) & 0x7FFFFFFFFFFF)
    return g


def _normal(n, std, seed, *key, dtype=torch.float32):
    x = torch.randn(n, generator=_generator(seed, *key), device="cuda")
    return x.mul_(std).to(dtype)


def _grads(case, seed, k):
    dtype = torch.bfloat16 if case["bf16"] else torch.float32
    return [_normal(case["n"], G_STD, seed, 1, k, i, dtype=dtype) for i in range(case["R"])]


def _config(case, seed):
    opt, beta1, beta2 = OPT[case.get("opt", "adamw")]
    bf16 = case.get("bf16", False)
    return am.make_config(
        case["n"], case["R"], delay=case.get("tau", 1), avg_interval=case.get("K", 1), fraction=case.get("p", 0.05), seed=seed,
        optimizer=opt, beta1=beta1, beta2=beta2, eps=EPS, weight_decay=WEIGHT_DECAY, momentum_decay=MOMENTUM_DECAY,
        lookahead=case.get("lookahead", False), gamma=GAMMA, correction=am.CORR_EMA if case.get("corr", "ema") == "ema" else am.CORR_NONE,
        fwd_dtype=am.BF16 if bf16 else am.F32, grad_dtype=am.BF16 if bf16 else am.F32,
        d_layout=am.D_INTERLEAVED if case.get("interleaved", False) else am.D_PER_REPLICA)


def _warm_steps(case):
    return (case.get("tau", 1) + 1) * case.get("K", 1)     # from here on every round receives


def _lr(case):
    return SGD_LR if case.get("opt") == "sgd" else LR


def _one_step(s):
    """What a training loop does with one replica set of gradients."""
    s["t"] += 1
    st, t, grads = s["stage"], s["t"], s["grads"][s["t"] % 2]
    if not s["clip"]:
        st.step(t, grads, s["lr"], LAMBDA)
        return None
    norms = st.grad_sqnorm(grads)
    st.step_scaled(t, grads, s["lr"], LAMBDA, 1.0, norms.rsqrt().clamp_(max=1.0).float())
    return norms


def prepare(case, seed):
    call = case["call"]
    if call == "lookahead":
        w_prev = _normal(case["n"], W_STD, seed, 0)
        w = w_prev + _normal(case["n"], LR, seed, 2)
        return {"call": call, "w": w, "w_prev": w_prev, "dtype": am.BF16 if case["bf16"] else am.F32}
    if call == "indices":
        # the smallest stage of that many coordinates: the list depends on n, p and the seed alone
        cfg = am.make_config(case["n"], 1, fraction=case["p"], seed=seed, optimizer=am.OPT_SGD, beta1=0.0, correction=am.CORR_NONE)
        st = am.init_state(cfg, torch.zeros(case["n"], device="cuda"))
        room = int(case["n"] * case["p"] + 12 * math.sqrt(case["n"] * case["p"])) + 64
        return {"call": call, "stage": st, "t": 0, "out": torch.zeros(room, dtype=torch.int64, device="cuda"),
                "count": torch.zeros(1, dtype=torch.int64, device="cuda")}
    st = am.init_state(_config(case, seed))
    st.set_w(_normal(case["n"], W_STD, seed, 0))
    s = {"call": call, "stage": st, "t": 0, "K": case.get("K", 1), "clip": case.get("clip", False), "lr": _lr(case)}
    if call == "average":
        # the program's own optimizer moves every replica between two rounds
        moves = [_normal(case["n"], LR, seed, 2, i) for i in range(case["R"])]
        for _ in range(_warm_steps(case)):
            for w, move in zip(st.w, moves):
                w.add_(move)
            s["t"] += 1
            st.sparse_average(s["t"], LAMBDA)
        for w, move in zip(st.w, moves):
            w.add_(move)
        return s
    if call == "diagnostics":
        case = dict(case, bf16=False)
    s["grads"] = [_grads(case, seed, k) for k in range(2)]
    for _ in range(_warm_steps(case)):
        _one_step(s)
    if call == "diagnostics":
        s["grads"] = None
    return s


def _state(st):
    return {k: v for k, v in (("w", st.w), ("m", st.m), ("v", st.v), ("d", st.d_storage), ("fwd", st.fwd)) if v is not None}


def run(s):
    call = s["call"]
    if call == "lookahead":
        return am.lookahead(s["w"], s["w_prev"], GAMMA, s["dtype"])
    if call == "diagnostics":
        return s["stage"].diagnostics()
    if call == "indices":
        s["t"] += 1
        s["stage"].subset_indices_static(s["t"], s["out"], s["count"])
        return {"indices": s["out"], "count": s["count"]}
    if call == "average":
        s["t"] += 1
        s["stage"].sparse_average(s["t"], LAMBDA)
        return {"w": s["stage"].w, **({"d": s["stage"].d_storage} if s["stage"].d_storage is not None else {})}
    for _ in range(s["K"]):
        norms = _one_step(s)
    out = _state(s["stage"])
    if norms is not None:
        out["norms"] = norms
    return out


# ---------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------
def work(case):
    n, call = case["n"], case["call"]
    if call == "lookahead":
        return {"bytes": n * (8 + (2 if case["bf16"] else 4)), "flops": 3 * n}
    if call == "indices":
        return {"bytes": 8 * n * case["p"], "flops": 5 * n}              # twenty products per four coordinates
    R = case["R"]
    d = case["corr"] == "ema"
    if call == "diagnostics":
        return {"bytes": n * R * (8 if d else 4), "flops": n * R * (8 if d else 4)}
    # per selected coordinate and replica: sent 4, received 4, EMA entry read and written 8 (no delay: only the latter)
    sparse = (8 if d else 0) + (8 if case["tau"] else 0)
    if call == "average":
        return {"bytes": n * R * case["p"] * (sparse + 8), "flops": n * R * case["p"] * 6}      # and the weight read and written
    g = 2 if case["bf16"] else 4
    moments = 1 if case["opt"] == "sgd" else 2
    fwd = 2 if case["bf16"] else 4 if case["lookahead"] else 0
    dense = 8 + g + 8 * moments + fwd + (g if case["clip"] else 0)
    return {"bytes": n * R * (case["K"] * dense + case["p"] * sparse), "flops": n * R * case["K"] * (12 + 8 * moments)}


def tolerance(case):
    if case["call"] == "indices":
        return "exact"
    if case.get("bf16"):
        # bf16 results round to 2^-9 of the value; another rounding of the fp32 sums moves few of them by one step
        return {"rel": 5e-4, "max": 0.01}
    # fp32 state.  The EMA entries are differences of weights some sixty times their size: 3e-6 off the
    # result in 64 bits, everything else 2e-7.
    return {"rel": 1.2e-5 if case.get("corr") == "ema" else 8e-7}


# ---------------------------------------------------------------------------------------------
# the same in 64 bits
# ---------------------------------------------------------------------------------------------
def _f32(x):
    return float(np.float32(x))


def _members(n, p, seed, step):
    """The subset of one step: coordinate mu is in it when word mu mod 4 of Philox4x32-10 at counter
    (mu / 4, step), key seed, is below floor(p 2^32)."""
    mask32 = 0xFFFFFFFF
    groups = (n + 3) // 4
    c0 = torch.arange(groups, dtype=torch.int64, device="cuda")
    c1 = torch.zeros_like(c0)
    c2 = torch.full_like(c0, step & mask32)
    c3 = torch.full_like(c0, step >> 32)
    k0, k1 = seed & mask32, seed >> 32

    def product(m, c):                   # high and low words of a 32 x 32 bit product
        low, high = (c & 0xFFFF) * m, (c >> 16) * m
        return (high + (low >> 16)) >> 16, (c * m) & mask32

    for _ in range(10):
        h0, l0 = product(0xD2511F53, c0)
        h1, l1 = product(0xCD9E8D57, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & mask32, (k1 + 0xBB67AE85) & mask32
    return (torch.stack((c0, c1, c2, c3), dim=1).reshape(-1)[:n] < int(math.floor(p * 2.0**32))).nonzero().reshape(-1)


class _Exact:
    """The stage update on whole replicas in fp64."""

    def __init__(self, case, seed):
        self.case, self.seed, self.n, self.R = case, seed, case["n"], case["R"]
        opt, b1, b2 = OPT[case.get("opt", "adamw")]
        self.b1, self.b2 = _f32(b1), _f32(b2)
        w0 = _normal(self.n, W_STD, seed, 0).double()
        self.w = [w0.clone() for _ in range(self.R)]
        self.m = [torch.zeros_like(w0) for _ in range(self.R)]
        self.v = [torch.zeros_like(w0) for _ in range(self.R)] if case.get("opt", "adamw") != "sgd" else None
        self.d = [torch.zeros_like(w0) for _ in range(self.R)] if case["corr"] == "ema" else None
        self.fwd = None
        self.sent, self.t, self.mu_product = {}, 0, 1.0

    def _average(self):
        """Send this round's subset and receive the one sent tau rounds ago; self.w holds the stepped weights."""
        K, tau, lam = self.case.get("K", 1), self.case.get("tau", 1), _f32(LAMBDA)
        if self.t % K:
            return
        at = _members(self.n, self.case.get("p", 0.05), self.seed, self.t)
        self.sent[self.t] = (at, [w[at] for w in self.w])
        if self.t - tau * K < 1:
            return
        at, old = self.sent.pop(self.t - tau * K)
        mean = sum(old) / self.R
        for i in range(self.R):
            if self.d is None:
                self.w[i][at] = mean
                continue
            d = (1 - lam) * self.d[i][at] + lam * (self.w[i][at] - old[i])
            self.d[i][at] = d
            self.w[i][at] = mean + d

    def average(self, moves=None):
        self.t += 1
        if moves is not None:
            self.move(moves)
        self._average()

    def move(self, moves):
        for w, move in zip(self.w, moves):
            w.add_(move)

    def step(self, grads):
        case = self.case
        self.t += 1
        lr, wd, eps, t = _f32(_lr(case)), _f32(WEIGHT_DECAY), _f32(EPS), self.t
        norms = None
        if case.get("clip"):
            norms = torch.stack([sum((x.double()**2).sum() for x in g.split(1 << 26)) for g in grads])
        scale = norms.rsqrt().clamp(max=1.0) if norms is not None else None
        opt = case.get("opt", "adamw")
        if opt == "nadamw":
            mu_t = self.b1 * (1 - 0.5 * 0.96**(t * MOMENTUM_DECAY))
            mu_next = self.b1 * (1 - 0.5 * 0.96**((t + 1) * MOMENTUM_DECAY))
            self.mu_product *= mu_t
            c_g, c_m = lr * (1 - mu_t) / (1 - self.mu_product), lr * mu_next / (1 - self.mu_product * mu_next)
        elif opt == "adamw":
            c_g, c_m = 0.0, lr / (1 - self.b1**t)
        else:
            c_g, c_m = 0.0, lr
        before, stepped = [], []
        for i in range(self.R):
            g = grads[i].double()
            if scale is not None:
                g = g * scale[i]
            self.m[i].mul_(self.b1).add_(g, alpha=1.0 if opt == "sgd" else 1 - self.b1)
            move = c_m * self.m[i] + c_g * g
            if opt != "sgd":
                self.v[i].mul_(self.b2).addcmul_(g, g, value=1 - self.b2)
                move = move / ((self.v[i] / (1 - self.b2**t)).sqrt() + eps)
            if case.get("lookahead"):
                before.append(self.w[i].clone())
            self.w[i] -= lr * wd * self.w[i] + move
            if case.get("lookahead"):
                stepped.append(self.w[i].clone())
        self._average()
        if case.get("lookahead"):
            self.fwd = [w + _f32(GAMMA) * (a - b) for w, a, b in zip(self.w, stepped, before)]
        elif case.get("bf16"):
            self.fwd = [w.clone() for w in self.w]
        return norms

    def d_storage(self):
        """The EMA entries as the layout of the case holds them."""
        if not self.case.get("interleaved"):
            return self.d
        rb = 1
        while rb < min(8, self.R):
            rb *= 2
        out = []
        for b in range(0, self.R, rb):
            block = torch.zeros((self.n + 255) // 256 * 256, rb, dtype=torch.float64, device="cuda")
            for k in range(min(rb, self.R - b)):
                block[:self.n, k] = self.d[b + k]
            out.append(block.reshape(-1))
        return out


def exact(case, seed):
    n, call = case["n"], case["call"]
    if call == "indices":
        return None
    if call == "lookahead":
        w_prev = _normal(n, W_STD, seed, 0)
        w = w_prev + _normal(n, LR, seed, 2)
        return w.double() + _f32(GAMMA) * (w.double() - w_prev.double())
    x = _Exact(case, seed)
    if call == "average":
        moves = [_normal(n, LR, seed, 2, i) for i in range(case["R"])]
        for _ in range(_warm_steps(case)):
            x.average(moves)
        x.move(moves)
        x.average()
        return {"w": x.w, **({"d": x.d_storage()} if x.d is not None else {})}
    if call == "diagnostics":
        case = dict(case, bf16=False)
    grads = [_grads(case, seed, k) for k in range(2)]
    norms = None
    for _ in range(_warm_steps(case) + (0 if call == "diagnostics" else case["K"])):
        norms = x.step(grads[(x.t + 1) % 2])
    if call == "diagnostics":
        mean = sum(x.w) / x.R
        consensus = sum(float(((w - mean)**2).sum()) for w in x.w)
        if x.d is None:
            return (consensus, 0.0, 0.0)
        mean = sum(x.d) / x.R
        variance = sum((d - mean)**2 for d in x.d) / x.R
        return (consensus, float(variance.mean()), float(variance.max()))
    out = {k: v for k, v in (("w", x.w), ("m", x.m), ("v", x.v), ("d", x.d_storage() if x.d is not None else None), ("fwd", x.fwd)) if v is not None}
    if norms is not None:
        out["norms"] = norms
    return out
