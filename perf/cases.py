"""Performance cases of the RFF linear attention library: the calls a user's
program makes, over the sizes it makes them at.

A case is a dict of plain values.  ``call`` names the entry point(s) of one
pass:

  forward   flex_linattn_fwd: inference of one attention layer
  train     flex_linattn_fwd, then flex_linattn_bwd on the same workspace:
            one attention layer of a training step (all gradients returned)
  prefill   flex_linattn_prefill: a prompt, leaving the decode state
  decode    flex_decode_step: one token of every running sequence
  distill   flex_awd_loss with gradients: one step of kernel distillation
  features  flex_feature_map: the features themselves

B, H, N: batch, heads, tokens; d: head size of Q, K and V; m: frequencies per
matrix; variant, causal and io ("bf16" or "f32") as in make_desc.

Inputs are those of a layer whose kernel is in use: Q, K and V have the
d^-1/4 scaling of the softmax bandwidth, and the frequencies have standard
deviation d^-1/4, so that a phase W x has a standard deviation of one radian
(the kernel then decays over the distance between typical rows, and its row
sums stay positive, as those of a layer that has been trained must).
Workspaces are kept by the caller; outputs are allocated by the call.
"""
from __future__ import annotations

import math

import torch

import paper_2606_27748_amd as flex


def _case(name, call, B, H, N, d, m, variant, causal, io="bf16"):
    return {"name": name, "call": call, "B": B, "H": H, "N": N, "d": d, "m": m,
            "variant": variant, "causal": causal, "io": io}


def listed():
    return [
        # the smallest call: one fp32 head over a short sequence (unit tests,
        # notebooks, single-example evaluation); launch latency counts
        _case("encode_tiny_f32", "forward", 1, 1, 256, 32, 64, "stationary", False, "f32"),
        # one layer of a language model scoring a batch of 1024-token blocks
        _case("lm_forward", "forward", 8, 12, 1024, 64, 128, "stationary", True),
        # one layer of a long-document encoder at inference
        _case("long_encode", "forward", 16, 8, 16384, 64, 64, "stationary", False),
        # one layer of language-model training, 8192-token sequences, heads of 64
        _case("train_lm", "train", 2, 16, 8192, 64, 128, "nonstationary", True),
        # the same with heads of 128 and 256 frequencies: the largest layer
        _case("train_lm_d128", "train", 2, 16, 8192, 128, 256, "nonstationary", True),
        # one layer of encoder training on 4000-token documents (bidirectional;
        # not a whole number of 64-token chunks)
        _case("train_encoder", "train", 8, 8, 4000, 64, 64, "nonstationary", False),
        # training in full fp32 (small models, gradient checks), ragged length
        _case("train_f32", "train", 4, 8, 1023, 32, 64, "nonstationary", True, "f32"),
        # one layer of the prefill of a single 3001-token prompt
        _case("prefill_one", "prefill", 1, 16, 3001, 64, 128, "nonstationary", True),
        # one layer of a decode step of a full serving batch: bound by the state
        _case("decode_batch", "decode", 256, 16, 1, 64, 128, "nonstationary", True),
        # one layer of a decode step of a single sequence: bound by latency
        _case("decode_one", "decode", 1, 12, 1, 64, 128, "stationary", True),
        # one layer of a distillation step, encoder batch of 512-token sequences
        _case("distill", "distill", 32, 8, 512, 64, 64, "nonstationary", False),
        # the features of one layer's queries, for a caller's own contraction
        _case("features", "features", 8, 12, 1000, 64, 128, "nonstationary", False),
    ]


def _cost(c):
    """Rough cost of a pass, to keep drawn cases within the listed ones."""
    tokens = c["B"] * c["H"] * c["N"]
    if c["call"] == "distill":
        return tokens * c["N"] * c["m"] / 16
    return tokens * c["m"] * c["d"] * (4 if c["call"] == "train" else 1) * (3 if c["io"] == "f32" else 1)


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    call = rng.choice(["forward", "forward", "train", "train", "train", "prefill", "decode", "distill", "features"])
    variant = rng.choice(["stationary", "nonstationary"])
    while True:
        io = "bf16" if call == "prefill" else rng.choice(["bf16", "bf16", "bf16", "f32"])
        d = 32 if io == "f32" else rng.choice([32, 64, 64, 128])
        m = rng.choice([48, 64, 64, 80, 128, 128, 192, 256])
        causal = call == "prefill" or (call in ("forward", "train") and rng.random() < 0.6)
        B, H = log_int(1, 32), rng.choice([2, 4, 8, 12, 16])
        N = log_int(100, 20000)
        if call == "prefill":
            B = log_int(1, 4)
        elif call == "decode":
            B, N, causal = log_int(1, 256), 1, True
        elif call == "distill":
            d, m = (32, 64) if io == "f32" else rng.choice([(32, 64), (64, 64), (64, 128)])
            N = log_int(64, 600)
        c = {"call": call, "B": B, "H": H, "N": N, "d": d, "m": m, "variant": variant,
             "causal": causal, "io": io}
        if _cost(c) <= _cost(_case("", "train", 2, 16, 8192, 128, 256, variant, True)):
            return c


def _inputs(c, seed):
    """The tensors of a case, on the GPU, from its seed alone."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(int(seed))

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=dev, dtype=torch.float32)

    B, H, N, d, m = c["B"], c["H"], c["N"], c["d"], c["m"]
    io = torch.bfloat16 if c["io"] == "bf16" else torch.float32
    ns = c["variant"] == "nonstationary"
    x = {}
    if c["call"] == "distill":
        # a kernel near a wide Gaussian before distillation: rows of unit
        # variance, phases within about a radian, every kernel weight positive
        scale, wstd, tau = 1.0, 0.5 / math.sqrt(d), math.log(2.0 * d)
    else:
        scale, wstd, tau = d ** -0.25, d ** -0.25, math.log(2.0)
    x["W1"] = normal(H, m, d) * wstd
    x["W2"] = normal(H, m, d) * wstd if ns else None
    x["tau"] = tau + 0.05 * normal(H)
    rows = (B, H, d) if c["call"] == "decode" else (B, H, N, d)
    x["Q"] = (normal(*rows) * scale).to(io)
    if c["call"] != "features":
        x["K"] = (normal(*rows) * scale).to(io)
    if c["call"] not in ("features", "distill"):
        x["V"] = (normal(*rows) * scale).to(io)
    if c["call"] == "train":
        # rows with larger keys carry a value along the mean of the upstream
        # gradient, so that the norm scale has a gradient, as while it is learned
        u = 0.06 * normal(H, 1, d)
        size = (x["K"].float().square().sum(-1, keepdim=True) - math.sqrt(d)) / math.sqrt(2.0)
        x["V"] = (x["V"].float() + scale * size * u).to(io)
        x["dO"] = (normal(*rows) + u).to(io)
    if c["call"] == "decode":
        # the state of a prefix of some hundreds of tokens: sums of features
        # (z, the cos block of positive mean) and of features times values
        F = 2 * m
        s = torch.empty(B, H, F * (d + 1), device=dev, dtype=torch.float32)
        s.normal_(generator=gen).mul_(8.0)
        s[..., F * d:F * d + m] += 200.0
        x["state"] = s
    return x


def _desc(c):
    return flex.make_desc(c["B"], c["H"], c["N"], c["d"], c["m"], c["variant"], c["causal"], c["io"])


def prepare(case, seed):
    x = _inputs(case, seed)
    desc = _desc(case)
    s = {"call": case["call"], "desc": desc, "x": x}

    def ws(pass_):
        return torch.empty(max(flex.workspace_size(desc, pass_), 256), dtype=torch.uint8, device="cuda")

    if case["call"] in ("forward", "train", "prefill"):
        s["ws"] = ws(flex.FLEX_PASS_FWD)
    if case["call"] == "train":
        s["ws_bwd"] = ws(flex.FLEX_PASS_BWD)
    if case["call"] == "distill":
        s["ws"] = ws(flex.FLEX_PASS_AWD)
    return s


def run(s):
    x, desc, call = s["x"], s["desc"], s["call"]
    if call == "decode":
        o, den = flex.flex_decode_step(desc, x["Q"], x["K"], x["V"], x["W1"], x["W2"], x["tau"], x["state"])
        return {"o": o, "den": den, "state": x["state"]}
    if call == "features":
        return {"phi": flex.flex_feature_map(desc, x["Q"], x["W1"], x["W2"], x["tau"])}
    if call == "distill":
        out = flex.flex_awd_loss(desc, x["Q"], x["K"], x["W1"], x["W2"], x["tau"], ws=s["ws"])
        return {k: v for k, v in out.items() if v is not None}
    args = (desc, x["Q"], x["K"], x["V"], x["W1"], x["W2"], x["tau"])
    if call == "prefill":
        O, den, state = flex.flex_linattn_prefill(*args, ws=s["ws"])
        return {"O": O, "den": den, "state": state}
    O, den = flex.flex_linattn_fwd(*args, ws=s["ws"])
    out = {"O": O, "den": den}
    if call == "train":
        g = flex.flex_linattn_bwd(*args, O, den, x["dO"], ws=s["ws_bwd"], fwd_ws=s["ws"])
        out.update({k: v for k, v in g.items() if v is not None})
    return out


def work(case):
    """Inputs read once, outputs written once; the projections and the state
    contractions (the pairwise tiles for the distillation loss)."""
    BH, H, N, d, m = case["B"] * case["H"], case["H"], case["N"], case["d"], case["m"]
    io = 2 if case["io"] == "bf16" else 4
    nmat = 2 if case["variant"] == "nonstationary" else 1
    F, meff, W = 2 * m, nmat * m, 4 * nmat * case["H"] * m * d
    call, rows = case["call"], BH * N
    if call == "features":
        return {"bytes": rows * (d + F) * io + W, "flops": rows * 2 * d * meff}
    if call == "decode":
        return {"bytes": 2 * BH * F * (d + 1) * 4 + BH * (4 * d * io + 4) + W,
                "flops": BH * (4 * d * meff + 4 * F * (d + 1))}
    if call == "distill":
        # logit and kernel tiles, G phi for either side; the rows' chain rule
        return {"bytes": rows * 2 * d * io + 2 * W + 4 * BH + 4 * H,
                "flops": rows * N * (2 * d + 3 * 2 * F) + 2 * rows * 4 * d * meff}
    b = rows * (4 * d * io + 4) + W
    f = rows * (4 * d * meff + 4 * F * (d + 1))
    if call == "prefill":
        b += BH * F * (d + 1) * 4
    if call == "train":
        # dO read; dQ, dK, dV (fp32) and the parameter gradients written
        b += rows * (d * io + 3 * d * 4) + W + 4 * H
        f += rows * (8 * F * (d + 1) + 8 * d * meff)
    return {"bytes": b, "flops": f}


def tolerance(case):
    """About four times the error against float64 of the outputs (exact)."""
    if case["io"] == "f32":
        if case["call"] == "distill":
            return {"rel": 3e-4, "max": 5e-3}  # measured: 1e-6, dtau (terms that cancel) 6e-5
        return {"rel": 1e-5, "max": 1e-3}      # measured: 1e-7 to 8e-7
    if case["call"] == "train":
        # measured: dQ 4e-3 to 1e-2 (single elements up to 0.3 of the root mean
        # square: rows of small gradient against delta), dW 2e-3 to 4e-3, the
        # others 2e-3 and below
        return {"rel": 3e-2, "max": 0.9}
    if case["call"] == "distill":
        return {"rel": 4e-3, "max": 0.05}      # measured: 1.5e-4 to 3e-4, more over short sequences
    return {"rel": 7e-3, "max": 0.1}           # measured: 1.8e-3 (the output's own rounding)


# ---------------------------------------------------------------------------
# The same outputs in float64, one head at a time.
# ---------------------------------------------------------------------------
def _phi(X, W1, W2, tau, m):
    """Feature rows [..., 2m] of X for one head's frequencies."""
    e = torch.exp((X * X).sum(-1, keepdim=True) / torch.exp(tau))
    if W2 is None:
        P = X @ W1.T
        return e / math.sqrt(m) * torch.cat([torch.cos(P), torch.sin(P)], -1)
    P1, P2 = X @ (0.5 * (W1 + W2)).T, X @ (0.5 * (W1 - W2)).T
    c2 = torch.cos(P2)
    return e / (2 * math.sqrt(m)) * torch.cat([torch.cos(P1) * c2, torch.sin(P1) * c2], -1)


def _attend(pq, pk, V, causal):
    """O, den and the final state [.., 2m, d+1] from feature rows [B, N, 2m]."""
    V1 = torch.cat([V, torch.ones_like(V[..., :1])], -1)
    if not causal:
        S = pk.transpose(-1, -2).contiguous() @ V1
        y = pq @ S
        return y[..., :-1] / y[..., -1:], y[..., -1], S
    B, N, F = pq.shape
    C = 128
    n = (N + C - 1) // C

    def chunks(t):
        return torch.nn.functional.pad(t, (0, 0, 0, n * C - N)).reshape(B, n, C, t.shape[-1])

    q, k, v = chunks(pq), chunks(pk), chunks(V1)
    kt = k.transpose(-1, -2).contiguous()
    local = kt @ v
    total = torch.cumsum(local, 1)
    y = torch.tril(q @ kt) @ v + q @ (total - local)
    y = y.reshape(B, n * C, -1)[:, :N]
    return y[..., :-1] / y[..., -1:], y[..., -1], total[:, -1]


def exact(case, seed):
    x = _inputs(case, seed)
    call, H, m, d, N = case["call"], case["H"], case["m"], case["d"], case["N"]
    x = {k: None if v is None else v.double() for k, v in x.items()}
    ns = x["W2"] is not None
    heads = []
    for h in range(H):
        W1, W2, tau = x["W1"][h], x["W2"][h] if ns else None, x["tau"][h]
        Q = x["Q"][:, h]
        if call == "features":
            heads.append({"phi": _phi(Q, W1, W2, tau, m)})
            continue
        K = x["K"][:, h]
        if call == "decode":
            F = 2 * m
            st = x["state"][:, h]
            pk = _phi(K, W1, W2, tau, m)
            S = st[:, :F * d].reshape(-1, F, d) + pk[:, :, None] * x["V"][:, h, None, :]
            z = st[:, F * d:] + pk
            pq = _phi(Q, W1, W2, tau, m)
            den = (pq * z).sum(-1)
            heads.append({"o": (pq[:, None, :] @ S)[:, 0] / den[:, None], "den": den,
                          "state": torch.cat([S.reshape(len(st), -1), z], -1)})
            continue
        grads = call in ("train", "distill")
        leaf = {"dW1": W1, "dW2": W2, "dtau": tau}
        if call == "train":
            leaf.update(dQ=Q, dK=K, dV=x["V"][:, h])
        leaf = {k: v.clone().requires_grad_(grads) for k, v in leaf.items() if v is not None}
        W1, W2, tau = leaf["dW1"], leaf.get("dW2"), leaf["dtau"]
        Q, K = leaf.get("dQ", Q), leaf.get("dK", K)
        if call == "distill":
            out = {"loss": torch.empty(case["B"], dtype=torch.float64, device=Q.device)}
            step = max(1, (1 << 25) // (N * N))
            for b in range(0, case["B"], step):
                q, k = Q[b:b + step], K[b:b + step]
                P = torch.softmax(q @ k.transpose(-1, -2).contiguous() / math.sqrt(d), -1)
                pq, pk = _phi(q, W1, W2, tau, m), _phi(k, W1, W2, tau, m)
                A = pq @ pk.transpose(-1, -2).contiguous()
                loss = -(P * torch.log(A / A.sum(-1, keepdim=True))).sum((-1, -2)) / N
                loss.sum().backward()
                out["loss"][b:b + step] = loss.detach()
        else:
            pq, pk = _phi(Q, W1, W2, tau, m), _phi(K, W1, W2, tau, m)
            O, den, S = _attend(pq, pk, leaf.get("dV", x["V"][:, h]), case["causal"])
            out = {"O": O.detach(), "den": den.detach()}
            if call == "prefill":
                out["state"] = torch.cat([S[..., :-1].reshape(len(S), -1), S[..., -1]], -1)
            if call == "train":
                (O * x["dO"][:, h]).sum().backward()
        if grads:
            out.update({k: v.grad for k, v in leaf.items()})
        heads.append(out)
    per_head = ("dW1", "dW2", "dtau")   # [H, ...]; every other output is [B, H, ...]
    return {k: torch.stack([o[k] for o in heads], 0 if k in per_head else 1) for k in heads[0]}
