"""The calls whose speed is measured: what a training or serving program asks of
the shared-readout loss, through the binding's public entry points.

A case is a dict of plain values:
  op     "train" (readout_fwd_bwd: losses, dh, dW, dgain), "heads" (the same with
         final_module_dW=False: a rank that owns no terminal), "general"
         (temperatures, biases, per-module gains, all their gradients), "priv"
         (one trained readout per head), "rot" (the shared readout in a fixed
         orthogonal basis per head), "eval" (exit evaluation, forward only)
  dtype  "bf16" or "f32"
  K, T, d, V   modules, tokens per module, width, vocabulary
  w_sigma, h_step, hot   the spread of the readout, the growth of the hidden
         states per module and the share of one hot token, as in
         solo_inputs.CONFIGS

Hidden states, readouts, gains, temperatures, biases and Zipf targets have the
distributions of solo_inputs, drawn on the GPU.
"""
import math

import torch

from paper_2609_35440_amd import binding

EPS = 1e-6


def _case(name, op, K, T, d, V, dtype="bf16", w_sigma=0.02, h_step=0.0, hot=0.0):
    return dict(name=name, op=op, dtype=dtype, K=K, T=T, d=d, V=V, w_sigma=w_sigma, h_step=h_step, hot=hot)


def listed():
    return [
        # the smallest training call: the fp32 correctness shape of the workload table
        _case("train_tiny_f32", "train", 2, 256, 64, 512, dtype="f32"),
        # fp32 training of a small model: odd token count and vocabulary
        _case("train_f32", "train", 2, 1001, 768, 8003, dtype="f32"),
        # the four bf16 workloads of the table, whole: 340M-, 1B- and 2B-class models
        # at their micro-batches, and the large-vocabulary shape with large logits
        _case("train_340m", "train", 4, 8192, 1024, 32000),
        _case("train_1b", "train", 4, 16384, 2048, 32000),
        _case("train_2b", "train", 8, 16384, 2560, 32000, h_step=0.25),
        _case("train_large_vocab", "train", 2, 32768, 2048, 128256, w_sigma=0.05, hot=0.01),
        # a 7B-class width (the widest the interface takes), half a sequence
        _case("train_4096", "train", 2, 1024, 4096, 32000),
        # Algorithm 1 with every option, one sequence of a 340M-class model, odd sizes
        _case("general_340m", "general", 4, 2047, 1024, 32001),
        # one private readout per head on the ladder of small models: a width that
        # is no multiple of 256
        _case("priv_640", "priv", 2, 1999, 640, 8192),
        # ROT heads, one sequence of a 1B-class model
        _case("rot_1b", "rot", 4, 2048, 2048, 32000),
        # validation: every exit's loss and top-1 over a 1B-class micro-batch
        _case("eval_1b", "eval", 4, 16384, 2048, 32000),
        # serving: one decode step of 16 sequences through every exit
        _case("eval_decode", "eval", 4, 16, 2048, 32000),
    ]


# Drawn cases: widths up to the interface's limit, multiples of 256 (what models
# mostly use) as often as other multiples of 8; tokens from one to a micro-batch;
# vocabularies from a toy's to the largest of the table.
_OPS = ["train", "train", "train", "heads", "general", "priv", "rot", "eval", "eval"]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(c):
    """Rough seconds: the matrix-core rate where the width is a multiple of 256, a
    vector-ALU rate elsewhere, and the time to allocate and touch the state."""
    fl = _exec_flops(c)
    fast = c["dtype"] == "bf16" and c["d"] % 256 == 0 and (c["d"] <= 2048 or c["d"] == 2560)
    # a call of few rows leaves most of the chip idle
    fill = min(1.0, c["K"] * c["T"] / (32 * 256.0 if fast else 8 * 512.0))
    return fl / ((0.5e15 if fast else 3e12) * fill)


def draw(rng):
    while True:
        f32 = rng.random() < 0.2
        op = rng.choice(_OPS)
        if f32:
            d = 8 * _log_int(rng, 3, 128)
        elif rng.random() < 0.6:
            d = 256 * rng.choice([1, 2, 2, 3, 4, 4, 5, 6, 8, 8, 10, 12, 16])
        else:
            d = 8 * _log_int(rng, 8, 511)
        K = rng.choice([2, 2, 3, 4, 4, 8]) if op != "eval" else rng.choice([1, 2, 4, 8])
        T = _log_int(rng, 1, 16384)
        V = _log_int(rng, 500, 131072)
        if op in ("priv", "rot"):
            K = min(K, 4)
            V = min(V, 65536)
        c = dict(op=op, dtype="f32" if f32 else "bf16", K=K, T=T, d=d, V=V, w_sigma=rng.choice([0.02, 0.02, 0.05]),
                 h_step=0.0, hot=0.0)
        if _cost(c) <= 0.1 and _state_bytes(c) <= 6 << 30:
            return c


def _elem(c):
    return 2 if c["dtype"] == "bf16" else 4


def _exec_flops(c):
    passes = {"train": 2 * c["K"] + 2, "heads": 2 * c["K"], "general": 3 * c["K"] + 1, "priv": 4 * c["K"],
              "rot": 2 * c["K"] + 2, "eval": c["K"]}[c["op"]]
    return 2.0 * passes * c["T"] * c["V"] * c["d"]


def _state_bytes(c):
    nr = c["K"] if c["op"] == "priv" else 1
    return 3 * c["K"] * c["T"] * c["d"] * _elem(c) + nr * c["V"] * c["d"] * (2 * _elem(c) + 4)


def _gen(seed, tag):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * (seed + 1) + tag)
    return g


def _normal(seed, tag, shape, sigma=1.0, mean=0.0, dtype=torch.float32):
    x = torch.randn(shape, generator=_gen(seed, tag), device="cuda", dtype=torch.float32)
    return x.mul_(sigma).add_(mean).to(dtype)


def _targets(c, seed):
    """Bounded Zipf(1.1) token ids by inverse CDF, with the hot token V - 1."""
    K, T, V = c["K"], c["T"], c["V"]
    pmf = torch.arange(1, V + 1, dtype=torch.float64, device="cuda").pow_(-1.1)
    cdf = torch.cumsum(pmf, 0)
    cdf /= cdf[-1].clone()
    u = torch.rand((K, T), generator=_gen(seed, 3), device="cuda", dtype=torch.float64)
    t = torch.searchsorted(cdf, u, right=True).clamp_(max=V - 1).to(torch.int32)
    if c["hot"] > 0.0:
        hit = torch.rand((K, T), generator=_gen(seed, 4), device="cuda") < c["hot"]
        t = torch.where(hit, torch.full_like(t, V - 1), t)
    return t.contiguous()


def _inputs(c, seed):
    K, T, d, V = c["K"], c["T"], c["d"], c["V"]
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    h = torch.empty((K, T, d), device="cuda", dtype=dt)
    for k in range(K):
        h[k] = _normal(seed, 100 + k, (T, d), 1.0 + c["h_step"] * k)
    x = dict(h=h, W=_normal(seed, 1, (V, d), c["w_sigma"], dtype=dt), targets=_targets(c, seed))
    per_module = c["op"] == "general"
    x["gain"] = _normal(seed, 2, (K, d) if per_module else (d,), 0.1, 1.0, dtype=dt)
    if c["op"] in ("general", "priv", "rot"):
        tau = torch.rand((K,), generator=_gen(seed, 5), device="cuda") * 1.5 + 0.5
        tau[K - 1] = 1.0  # the terminal has none
        x["tau"] = tau
    if c["op"] in ("general", "priv"):
        x["bias"] = _normal(seed, 6, (K, V), 0.5)
    if c["op"] == "priv":
        x["Wbar"] = _normal(seed, 7, (K - 1, V, d), c["w_sigma"], dtype=dt)
    if c["op"] == "rot":
        # random orthogonal matrices: products of Householder reflections
        R = torch.eye(d, device="cuda").repeat(K - 1, 1, 1)
        for k in range(K - 1):
            for i in range(8):
                v = _normal(seed, 200 + 8 * k + i, (d,))
                v /= v.norm()
                R[k] -= 2.0 * torch.outer(R[k] @ v, v)
        x["rot"] = R.to(dt)
    return x


def prepare(case, seed):
    return dict(case=dict(case), x=_inputs(case, seed))


def run(state):
    op, x = state["case"]["op"], state["x"]
    if op in ("train", "heads"):
        r = binding.readout_fwd_bwd(x["h"], x["gain"], x["W"], x["targets"], op == "train", EPS)
    elif op == "eval":
        r = binding.exit_eval(x["h"], x["gain"], x["W"], x["targets"], eps=EPS)
    else:
        r = binding.readout_general(x["h"], x["gain"], x["W"], x["targets"], Wbar=x.get("Wbar"), tau=x["tau"],
                                    bias=x.get("bias"), rot=x.get("rot"), heads_train_readout=op == "priv",
                                    want_dtau=True, want_dbias=op != "rot", eps=EPS)
    return r._asdict()


def work(case):
    K, T, d, V, e = case["K"], case["T"], case["d"], case["V"], _elem(case)
    op = case["op"]
    r = 2.0 * T * V * d  # one product of a module's rows with a readout
    flops = {"train": (2 * K + 1) * r, "heads": 2 * K * r, "general": (2 * K + 1) * r, "priv": 3 * K * r,
             "rot": (2 * K + 1) * r + 4.0 * (K - 1) * T * d * d, "eval": K * r}[op]
    b = K * T * d * e + d * e + V * d * e + 4 * K * T + 4 * K  # h, gain, W, targets, losses
    if op == "eval":
        b += 8 * K * T  # per-token losses and top-1
    else:
        b += K * T * d * e  # dh
    if op not in ("heads", "eval"):
        b += 4 * V * d + 4 * d  # dW, dgain
    if op in ("general", "priv"):
        b += 8 * K * V  # biases and their gradients
    if op == "priv":
        b += (K - 1) * V * d * (e + 4)
    if op == "rot":
        b += (K - 1) * d * d * e
    return {"bytes": float(b), "flops": float(flops)}


def tolerance(case):
    # about four times the distance from exact(): fp32 outputs are up to 9e-7 off it
    # (dW; its largest entry 6e-5), bf16 ones up to 2.5e-3 (dW, whose rare tokens'
    # rows lie far below its root mean square: 0.6 at the largest entry)
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-4}
    return {"rel": 1e-2, "max": 0.9, "differ": 0.01}


def exact(case, seed):
    """The definitions in 64 bits: logits, log-sum-exp, residual, transposes, norm
    backward, over blocks of rows."""
    x = _inputs(case, seed)
    K, T, d, V = case["K"], case["T"], case["d"], case["V"]
    op = case["op"]
    f8 = torch.float64
    W = x["W"].to(f8)
    losses = torch.zeros(K, dtype=f8, device="cuda")
    row_loss = torch.zeros((K, T), dtype=f8, device="cuda")
    bwd = op != "eval"
    dh = torch.zeros((K, T, d), dtype=f8, device="cuda") if bwd else None
    dR = {}
    dg = torch.zeros((K, d), dtype=f8, device="cuda")
    dtau = torch.zeros(K, dtype=f8, device="cuda")
    db = torch.zeros((K, V), dtype=f8, device="cuda") if op in ("general", "priv") else None
    block = max(1, min(T, (1 << 28) // V))
    for k in range(K):
        head = k < K - 1
        R = W
        if head and "Wbar" in x:
            R = x["Wbar"][k].to(f8)
        if head and "rot" in x:
            R = W @ x["rot"][k].to(f8)
        g = (x["gain"][k] if x["gain"].dim() == 2 else x["gain"]).to(f8)
        tau = x["tau"][k].to(f8) if "tau" in x else 1.0
        if bwd and ((not head and op != "heads") or op == "priv"):
            dR[k] = torch.zeros((V, d), dtype=f8, device="cuda")
        for t0 in range(0, T, block):
            hb = x["h"][k, t0:t0 + block].to(f8)
            y = x["targets"][k, t0:t0 + block].long()
            r = torch.rsqrt(hb.square().mean(1, keepdim=True) + EPS)
            n = hb * r
            u = (n * g) @ R.t()
            z = u * tau
            if "bias" in x:
                z += x["bias"][k].to(f8)
            lse = torch.logsumexp(z, 1)
            row_loss[k, t0:t0 + block] = lse - z.gather(1, y[:, None])[:, 0]
            if not bwd:
                continue
            delta = torch.exp_(z.sub_(lse[:, None]))
            delta.scatter_add_(1, y[:, None], torch.full((y.numel(), 1), -1.0, dtype=f8, device="cuda"))
            delta /= T
            dtau[k] += (delta * u).sum()
            if db is not None:
                db[k] += delta.sum(0)
            dhat = tau * (delta @ R)
            if k in dR:
                dR[k] += tau * (delta.t() @ (n * g))
            dg[k] += (dhat * n).sum(0)
            dn = dhat * g
            dh[k, t0:t0 + block] = r * (dn - n * (dn * n).mean(1, keepdim=True))
        losses[k] = row_loss[k].mean()
    if op == "eval":
        return dict(losses=losses, row_loss=row_loss, top1=None)
    out = dict(losses=losses, dh=dh, dW=dR.get(K - 1), row_loss=None)
    if op == "heads":
        return dict(out, dgain=None)
    if op == "train":
        return dict(out, dgain=dg[K - 1])
    return dict(out, dgain=dg if op == "general" else dg[K - 1], dtau=dtau, dbias=db,
                dWbar=torch.stack([dR[k] for k in range(K - 1)]) if op == "priv" else None)
