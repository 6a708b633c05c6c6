"""The workloads whose speed is measured: the GLA layer's calls as training,
prompt and generation programs make them, through the package's entry points.

A case is one call pattern ("kind") at one size:
  train     chunk_fwd, then chunk_bwd on the same workspace (the layer in one
            training step); with "state" also S0, S_T, dS_T and dS0
  prefill   chunk_fwd alone, keeping the final state (a prompt)
  decode    recurrent_fwd over a few steps from a state (generation)
  output    output_gate_fwd and output_gate_bwd (the layer's output side)
"gate" is the key gate's form: feature (log alpha per key feature), tau (its
pre-activation, alpha = sigmoid(z)^(1/16)), scalar (one log gamma per step and
head), none (alpha = 1), beta (feature, and a value-side gate as well).
Inputs follow the distributions of workloads.py, drawn on the GPU: q, k, v, dO
standard normal, k scaled by d_k^-1/2, log alpha = logsigmoid(x) / 16.
"""
import math

import torch

import paper_2312_06635_amd as gla

TAU = 16.0
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, kind, B, H, T, dk, dv, io="bf16", gate="feature", chunk=64, subchunk=16, state=False):
    c = dict(kind=kind, B=B, H=H, T=T, dk=dk, dv=dv, io=io, gate=gate, chunk=chunk, subchunk=subchunk, state=state)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # one layer of the 1.3B model in a training step of 8 sequences of 2048 (the benchmark's workload)
        _case("train_1p3b", "train", 8, 4, 2048, 256, 512),
        # one layer of the 340M model, 32 sequences, fed the gate's pre-activation as the model's projection gives it
        _case("train_340m_tau", "train", 32, 4, 2048, 128, 256, gate="tau"),
        # many narrow heads (16 of 128), 32768 tokens: the middle of the length sweep
        _case("train_heads_d128", "train", 16, 16, 2048, 128, 128),
        # one long document in few heads, its state carried in and out with gradients (truncated BPTT across segments)
        _case("train_long_state", "train", 1, 4, 16384, 256, 512, state=True),
        # ungated linear attention at head dimension 64 (the shape of the paper's kernel comparison)
        _case("train_ungated_d64", "train", 32, 16, 2048, 64, 64, gate="none"),
        # scalar gates (retention, Mamba-2 style) at widths and a length that fit no tile
        _case("train_scalar_ragged", "train", 4, 6, 1999, 144, 304, gate="scalar"),
        # single-precision training, shorter chunks
        _case("train_f32", "train", 2, 4, 1024, 128, 256, io="f32", chunk=32),
        # the smallest layer of the test workloads: launches and latency
        _case("train_tiny_f32", "train", 1, 1, 64, 16, 32, io="f32", chunk=16, subchunk=8),
        # the general gated form (gates on keys and values)
        _case("train_value_gate", "train", 4, 4, 1024, 128, 256, gate="beta"),
        # one user's prompt of odd length through a 1.3B layer, keeping the state for generation
        _case("prefill_1p3b", "prefill", 1, 4, 4003, 256, 512, state=True),
        # one generation step of 16 users through a 1.3B layer
        _case("decode_1p3b", "decode", 16, 4, 1, 256, 512, state=True),
        # the output side of the 1.3B layer in a training step: LayerNorm and Swish gate, and their reverse
        _case("output_1p3b", "output", 8, 4, 2048, 256, 512),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _width(rng, hi):
    """A width of 16 .. hi: the usual powers of two, and every other multiple of 16 as well."""
    usual = [w for w in (64, 128, 256, 512) if w <= hi]
    return rng.choice(usual) if rng.random() < 0.5 else 16 * max(1, round(_log(rng, 1, hi / 16)))


def draw(rng):
    kind = rng.choice(["train"] * 8 + ["prefill"] * 3 + ["decode"] * 3 + ["output"] * 2)
    gate = "feature" if kind == "output" else rng.choice(["feature"] * 5 + ["tau"] * 2 + ["scalar", "none", "beta"])
    io = "f32" if rng.random() < 0.2 else "bf16"
    dk, dv = _width(rng, 128 if io == "f32" else 256), _width(rng, 512)
    B, H = round(_log(rng, 1, 32)), round(_log(rng, 1, 16))
    chunk = rng.choice([64, 64, 64, 32, 16])
    T = round(_log(rng, 1, 8)) if kind == "decode" else round(_log(rng, 16, 16384))
    if kind != "decode" and rng.random() < 0.5:
        T = max(chunk, T // 64 * 64)  # else any length
    # no more work than the largest listed case: a tenth of it where single precision or the general form is slower
    most = (32 * 4 * 2048 * 128 * 256) // (10 if io == "f32" or gate == "beta" else 2)
    while B * H * T * dk * dv > most:
        if B > 1:
            B //= 2
        elif H > 1:
            H //= 2
        else:
            T //= 2
    state = kind in ("prefill", "decode") or rng.random() < 0.3
    return _case(None, kind, B, H, T, dk, dv, io, gate, chunk, 16, state)


def _inputs(case, seed):
    """The tensors of a case, made on the GPU from the seed alone."""
    B, H, T, dk, dv = (case[n] for n in ("B", "H", "T", "dk", "dv"))
    dt = DTYPES[case["io"]]
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape, scale=1.0, shift=0.0):
        x = torch.randn(*shape, generator=gen, device="cuda")
        return x.mul_(scale).add_(shift) if (scale, shift) != (1.0, 0.0) else x

    def log_gate(*shape):
        return (torch.nn.functional.logsigmoid(normal(*shape)) / TAU).to(dt)

    if case["kind"] == "output":
        return dict(o=normal(B, H, T, dv).to(dt), g=normal(B, H, T, dv).to(dt), dy=normal(B, H, T, dv).to(dt),
                    ln_w=normal(H, dv, scale=0.1, shift=1.0), ln_b=normal(H, dv, scale=0.1))
    d = dict(q=normal(B, H, T, dk).to(dt), k=normal(B, H, T, dk, scale=dk ** -0.5).to(dt), v=normal(B, H, T, dv).to(dt),
             la=None, lb=None, S0=None, dST=None)
    gate = case["gate"]
    if gate in ("feature", "beta"):
        d["la"] = log_gate(B, H, T, dk)
    elif gate == "scalar":
        d["la"] = log_gate(B, H, T)
    elif gate == "tau":
        d["la"] = normal(B, H, T, dk, scale=2.0, shift=1.0).to(dt)
    if gate == "beta":
        d["lb"] = log_gate(B, H, T, dv)
    if case["kind"] == "train":
        d["dO"] = normal(B, H, T, dv).to(dt)
    if case["state"]:
        if case["kind"] != "prefill":
            d["S0"] = normal(B, H, dk, dv, scale=0.1)
        if case["kind"] == "train":
            d["dST"] = normal(B, H, dk, dv, scale=0.1)
    return d


def prepare(case, seed):
    s = dict(case=case, **_inputs(case, seed))
    if case["kind"] in ("train", "prefill"):
        # one workspace for every step of the program, as a training loop keeps it
        p = (case["B"], case["H"], case["T"], case["dk"], case["dv"], case["chunk"], case["subchunk"], DTYPES[case["io"]])
        if case["kind"] == "train" and case["gate"] == "beta":
            n = gla.general_workspace_bytes(*p)
        else:
            n = gla.workspace_bytes(*p, op=1 if case["kind"] == "train" else 0, scalar_gate=case["gate"] == "scalar")
        s["workspace"] = torch.empty(max(n, 1), dtype=torch.uint8, device="cuda")
    elif case["kind"] == "output":
        s["workspace"] = torch.empty(max(gla.output_gate_workspace_bytes(s["o"]), 1), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "output":
        y, _ = gla.output_gate_fwd(s["o"], s["g"], s["ln_w"], s["ln_b"])
        g = gla.output_gate_bwd(s["o"], s["g"], s["dy"], s["ln_w"], s["ln_b"], workspace=s["workspace"])
        return dict(y=y, **g)
    tau = TAU if case["gate"] == "tau" else 0.0
    if case["kind"] == "decode":
        o, ST = gla.recurrent_fwd(s["q"], s["k"], s["v"], s["la"], S0=s["S0"], output_final_state=True, gate_tau=tau,
                                  log_beta=s["lb"])
        return dict(o=o, ST=ST)
    o, ST = gla.chunk_fwd(s["q"], s["k"], s["v"], s["la"], case["chunk"], case["subchunk"], S0=s["S0"],
                          output_final_state=case["state"], workspace=s["workspace"], gate_tau=tau, log_beta=s["lb"])
    if case["kind"] == "prefill":
        return dict(o=o, ST=ST)
    g = gla.chunk_bwd(s["q"], s["k"], s["v"], s["la"], s["dO"], case["chunk"], case["subchunk"], S0=s["S0"],
                      dST=s["dST"], want_dS0=case["state"], workspace=s["workspace"], reuse_fwd_workspace=True,
                      gate_tau=tau, log_beta=s["lb"], o=o if case["gate"] == "beta" else None)
    return dict(o=o, ST=ST, **g)


def work(case):
    """Each input read once and each output written once; the operations of the chunk form (of the recurrence for decode)."""
    B, H, T, dk, dv, C = (case[n] for n in ("B", "H", "T", "dk", "dv", "chunk"))
    s, rows = (2 if case["io"] == "bf16" else 4), B * H * T
    if case["kind"] == "output":
        return {"bytes": rows * dv * s * 8 + 4 * H * dv * 4, "flops": rows * dv * 36}
    gate = {"feature": dk, "tau": dk, "scalar": 1, "none": 0, "beta": dk + dv}[case["gate"]]
    states = B * H * dk * dv * 4
    fwd = rows * s * (2 * dk + gate + 2 * dv)
    if case["kind"] == "decode":
        return {"bytes": fwd + 2 * states, "flops": rows * 5 * dk * dv}
    flops = rows * (4 * dk * dv + (C + 1) * (dk + dv))
    if case["kind"] == "prefill":
        return {"bytes": fwd + states, "flops": flops}
    # backward: q, k, v, dO and the gates (and o, for the value-side gate) in; dq, dk, dv and the gates' gradients out
    bwd = rows * s * (4 * dk + 2 * gate + 3 * dv + (dv if case["gate"] == "beta" else 0))
    flops += rows * (8 * dk * dv + (C + 1) * (3 * dk + 2 * dv))
    return {"bytes": fwd + bwd + (5 * states if case["state"] else 0), "flops": flops}


def tolerance(case):
    # about four times the relative errors seen against 64-bit results: up to 3e-3 with bf16 inputs and outputs (8e-3 to 1e-2 in
    # the value-side gate's gradient), up to 4e-6 in single precision (the gate gradient's long sums)
    if case["io"] == "f32":
        return {"rel": 1.5e-5}
    return {"rel": 3e-2 if case["gate"] == "beta" else 1.2e-2}


def _exact_output(d):
    o, g, dy, w, b = (d[n].double() for n in ("o", "g", "dy", "ln_w", "ln_b"))
    w, b = w[:, None, :], b[:, None, :]
    rstd = (o.var(-1, unbiased=False, keepdim=True) + 1e-5).rsqrt()
    xh = (o - o.mean(-1, keepdim=True)) * rstd
    ln, sg = xh * w + b, torch.sigmoid(g)
    dln = dy * g * sg
    dx = dln * w
    do = rstd * (dx - dx.mean(-1, keepdim=True) - xh * (dx * xh).mean(-1, keepdim=True))
    return dict(y=g * sg * ln, do=do, dg=dy * ln * sg * (1 + g * (1 - sg)), dln_w=(dln * xh).sum((0, 2)), dln_b=dln.sum((0, 2)))


def exact(case, seed):
    """run()'s results by the recurrence step by step in 64 bits, and its reverse; the gates' gradients in closed form:
    dlog alpha_t = sum_{i >= t} (q_i dq_i - k_i dk_i) + rowsum(S_T dS_T), dlog beta_t likewise from o dO - v dv."""
    B, H, T, dk, dv = (case[n] for n in ("B", "H", "T", "dk", "dv"))
    if T * (600e-6 + B * H * dk * dv * 8 * 12 / 2e12) > 20:
        return None
    d = _inputs(case, seed)
    if case["kind"] == "output":
        return _exact_output(d)
    q, k, v = (d[n].double().flatten(0, 1) for n in ("q", "k", "v"))
    n, gate = B * H, case["gate"]
    z = d["la"].double().flatten(0, 1) if d["la"] is not None else None
    if gate == "none":
        la = torch.zeros(n, T, 1, dtype=torch.float64, device=q.device)
    elif gate == "scalar":
        la = z[:, :, None]
    else:
        la = torch.nn.functional.logsigmoid(z) / TAU if gate == "tau" else z
    a = la.exp().expand(n, T, dk)
    b = d["lb"].double().flatten(0, 1).exp() if d["lb"] is not None else None

    def state(x):
        return x.double().flatten(0, 1).clone() if x is not None else torch.zeros(n, dk, dv, dtype=torch.float64, device=q.device)

    def decay(S, t):
        S = S.mul_(a[:, t, :, None])
        return S.mul_(b[:, t, None, :]) if b is not None else S

    train = case["kind"] == "train"
    dO = d["dO"].double().flatten(0, 1) if train else None
    o = torch.empty_like(v)
    dq, dkk, dvv = (torch.empty_like(x) for x in (q, k, v))
    S = state(d["S0"])
    for t in range(T):
        decay(S, t).addcmul_(k[:, t, :, None], v[:, t, None, :])
        o[:, t] = (S * q[:, t, :, None]).sum(1)
        if train:
            dq[:, t] = (S * dO[:, t, None, :]).sum(2)

    def shape(x):
        return x.unflatten(0, (B, H))

    out = dict(o=shape(o), ST=shape(S) if case["state"] else None)
    if not train:
        return out
    dS = state(d["dST"])
    ca, cb = (S * dS).sum(2), (S * dS).sum(1)
    for t in reversed(range(T)):
        dS.addcmul_(q[:, t, :, None], dO[:, t, None, :])
        dkk[:, t] = (dS * v[:, t, None, :]).sum(2)
        dvv[:, t] = (dS * k[:, t, :, None]).sum(1)
        decay(dS, t)

    def reverse_sum(x):
        return x.flip(1).cumsum(1).flip(1)

    dla = dlb = None
    if gate != "none":
        dla = reverse_sum(q * dq - k * dkk) + ca[:, None]
        if gate == "scalar":
            dla = dla.sum(-1)
        elif gate == "tau":
            dla = dla * torch.sigmoid(-z) / TAU
        dla = shape(dla)
    out.update(dq=shape(dq), dk=shape(dkk), dv=shape(dvv), dlog_alpha=dla, dS0=shape(dS) if case["state"] else None)
    if b is not None:
        out["dlog_beta"] = shape(reverse_sum(o * dO - v * dvv) + cb[:, None])
    return out
