"""Performance cases of the FP32 GPT-2 training library.

What a user has the library do: a linear layer's three products, an MLP, the
language-model head with its loss, causal attention, one ring of
context-parallel attention, a LayerNorm, and the whole training step.  Every
case runs the forward and the backward of its layer through the public calls
(`paper_2606_24780_amd.bt`, `.ring`) on seeded inputs with the scales that
training has: normalised activations, weights N(0, 0.02), small upstream
gradients whose size differs from token to token.  Everything is FP32, the
library's only floating-point type.
"""
from __future__ import annotations

import math

import torch

from paper_2606_24780_amd import bt, ring, synth


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # one layer of the tiny models of the tests: launches and latency
        {"name": "linear_small", "kind": "linear", "M": 128, "K": 64, "N": 192},
        # a projection whose sizes fill no tile: ragged batches, other widths
        {"name": "linear_ragged", "kind": "linear", "M": 1036, "K": 780, "N": 2308},
        # QKV projection of the 2.42B configuration (B = 2, T = 1024)
        {"name": "linear_2b_qkv", "kind": "linear", "M": 2048, "K": 3072, "N": 9216},
        # MLP of GPT-2 124M at the benchmark's batch (B = 16, T = 1024)
        {"name": "mlp_124m", "kind": "mlp", "M": 16384, "C": 768},
        # tied LM head with the cross-entropy, half the benchmark's batch
        {"name": "head_124m", "kind": "head", "M": 8192, "C": 768, "V": 50257, "Vp": 50304},
        # attention of GPT-2 124M at the benchmark's batch
        {"name": "attention_124m", "kind": "attention", "B": 16, "T": 1024, "H": 12, "hd": 64},
        # attention of the long-context configuration, one sequence
        {"name": "attention_long", "kind": "attention", "B": 1, "T": 16384, "H": 12, "hd": 64},
        # odd length, head dim between the padded sizes: the recomputing backward
        {"name": "attention_ragged", "kind": "attention", "B": 3, "T": 777, "H": 6, "hd": 80},
        # context parallelism, both ranks of a ring of two, head dim of the 2.42B model
        {"name": "ring_2_ranks", "kind": "ring", "W": 2, "B": 1, "T": 4096, "H": 8, "hd": 128},
        # LayerNorm of GPT-2 124M: bound by memory
        {"name": "norm_124m", "kind": "norm", "M": 16384, "C": 768},
        # the tests' tiny model: a step of many short launches
        {"name": "step_tiny", "kind": "step", "B": 4, "T": 32, "L": 2, "H": 4, "C": 64, "V": 256, "Vp": 256},
        # the benchmark's step: GPT-2 124M, 16 sequences of 1024 tokens
        {"name": "step_124m", "kind": "step", "B": 16, "T": 1024, "L": 12, "H": 12, "C": 768, "V": 50257,
         "Vp": 50304},
    ]


def _log(rng, lo, hi, unit=4):
    """A multiple of `unit` in [lo, hi], spread over the logarithm; one in three is a multiple of 128."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    if v >= 256 and rng.random() < 1 / 3:
        unit = 128
    return int(min(hi, max(lo, unit * round(v / unit))))


def draw(rng):
    kind = rng.choice(["linear", "linear", "mlp", "head", "attention", "attention", "ring", "norm", "step"])
    if kind == "linear":
        return {"kind": kind, "M": _log(rng, 64, 16384), "K": _log(rng, 64, 3072), "N": _log(rng, 64, 9216)}
    if kind == "mlp":
        return {"kind": kind, "M": _log(rng, 64, 16384), "C": _log(rng, 64, 1536)}
    if kind == "head":
        V = rng.randint(256, 50257)
        return {"kind": kind, "M": _log(rng, 64, 8192), "C": _log(rng, 64, 1024), "V": V, "Vp": (V + 63) // 64 * 64}
    if kind == "attention":
        T = int(round(math.exp(rng.uniform(math.log(16), math.log(4096)))))
        if rng.random() < 0.5:
            T = (T + 31) // 32 * 32
        B = max(1, min(rng.randint(1, 16), (16 << 20) // (T * T)))
        return {"kind": kind, "B": B, "T": T, "H": rng.randint(1, 16), "hd": rng.choice([32, 64, 64, 80, 96, 128])}
    if kind == "ring":
        W = rng.choice([2, 4])
        return {"kind": kind, "W": W, "B": rng.randint(1, 2), "T": 256 * W * rng.randint(1, 8), "H": rng.randint(1, 12),
                "hd": rng.choice([32, 64, 128])}
    if kind == "norm":
        return {"kind": kind, "M": _log(rng, 64, 32768), "C": _log(rng, 64, 4096)}
    hd = rng.choice([32, 64, 64, 128])
    H = rng.randint(1, 768 // hd)
    V = rng.randint(256, 20000)
    return {"kind": "step", "B": rng.randint(1, 8), "T": _log(rng, 32, 1024), "L": rng.randint(1, 6), "H": H, "C": H * hd,
            "V": V, "Vp": (V + 63) // 64 * 64}


# ---------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(0x5EED + 7919 * int(seed))


def _randn(g, shape, std=1.0, mean=0.0):
    x = torch.randn(shape, generator=g, device="cuda")
    return x.mul_(std).add_(mean) if mean else x.mul_(std)


def _grad(g, rows, cols):
    """Upstream gradient: rows (tokens) of different size, 1e-5 to 1e-3."""
    scale = torch.exp(torch.rand((rows, 1), generator=g, device="cuda") * math.log(100.0)) * 1e-5
    return torch.randn((rows, cols), generator=g, device="cuda") * scale


def _zipf(g, n, V):
    """Token ids with P(k) ~ (k + 1)^-1.1, the frequencies of text."""
    w = torch.arange(1, V + 1, dtype=torch.float64, device="cuda") ** -1.1
    cdf = torch.cumsum(w, 0)
    u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * cdf[-1]
    return torch.searchsorted(cdf, u).clamp_(max=V - 1).to(torch.int32)


def _inputs(c, seed):
    """The case's inputs, from the seed alone."""
    g = _gen(seed)
    k = c["kind"]
    if k == "linear":
        M, K, N = c["M"], c["K"], c["N"]
        return {"X": _randn(g, (M, K)), "W": _randn(g, (K, N), 0.02), "b": _randn(g, (N,), 0.02), "dY": _grad(g, M, N)}
    if k == "mlp":
        M, C = c["M"], c["C"]
        return {"X": _randn(g, (M, C)), "R": _randn(g, (M, C)), "W1": _randn(g, (C, 4 * C), 0.02),
                "b1": _randn(g, (4 * C,), 0.02), "W2": _randn(g, (4 * C, C), 0.02), "b2": _randn(g, (C,), 0.02),
                "dY": _grad(g, M, C)}
    if k == "head":
        wte = _randn(g, (c["Vp"], c["C"]), 0.02)
        wte[c["V"]:] = 0
        return {"X": _randn(g, (c["M"], c["C"])), "wte": wte, "targets": _zipf(g, c["M"], c["V"])}
    if k in ("attention", "ring"):
        rows, C = c["B"] * c["T"], c["H"] * c["hd"]
        return {"qkv": _randn(g, (rows, 3 * C)), "dout": _grad(g, rows, C)}
    if k == "norm":
        M, C = c["M"], c["C"]
        return {"x": _randn(g, (M, C), 1.5, 0.1), "gamma": _randn(g, (C,), 0.02, 1.0), "beta": _randn(g, (C,), 0.02),
                "dy": _grad(g, M, C), "dres": _grad(g, M, C)}
    cfg = _config(c)
    parts = []
    for name, shape, _ in synth.param_specs(cfg):
        base = name.split(".")[-1]
        if base in ("ln1g", "ln2g", "lnfg"):
            t = _randn(g, shape, 0.02, 1.0)
        else:
            t = _randn(g, shape, 0.02 / math.sqrt(2 * cfg.L) if base in ("Wo", "Wfp") else 0.02)
        if base == "wte":
            t[cfg.V:] = 0
        parts.append(t.reshape(-1))
    params = torch.cat(parts)
    ids = _zipf(g, c["B"] * c["T"] + 1, cfg.V)
    # AdamW moments as in the middle of a run: v well above eps^2
    m = torch.randn(params.numel(), generator=g, device="cuda") * 1e-4
    v = (torch.rand(params.numel(), generator=g, device="cuda") + 0.5) * 1e-6
    return {"params": params, "moments": torch.cat([m, v]), "tokens": ids[:-1].reshape(c["B"], c["T"]).contiguous(),
            "targets": ids[1:].reshape(c["B"], c["T"]).contiguous()}


_STEPS_TAKEN = 1000  # optimizer steps before the one that is run


def _config(c):
    return synth.GPT2Config(V=c["V"], Vp=c["Vp"], max_T=c["T"], L=c["L"], H=c["H"], C=c["C"])


def _empty(*shape):
    return torch.empty(shape, device="cuda")


def _gemm_ws(products):
    """One scratch buffer for the split products of a layer: (opA, opB, M, N, K, epi)."""
    need = max(bt.lib().bt_gemm_ws_bytes(*p) for p in products)
    return torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    c, s = case, dict(_inputs(case, seed))
    s["case"] = c
    k = c["kind"]
    if k == "linear":
        M, K, N = c["M"], c["K"], c["N"]
        s.update(Y=_empty(M, N), dX=_empty(M, K), dW=_empty(K, N), db=_empty(N))
        s["ws"] = _gemm_ws([(0, 0, M, N, K, bt.EPI_BIAS), (0, 1, M, K, N, 0), (1, 0, K, N, M, 0)])
    elif k == "mlp":
        M, C, F = c["M"], c["C"], 4 * c["C"]
        s.update(pre=_empty(M, F), act=_empty(M, F), Y=_empty(M, C), dh=_empty(M, F), dX=_empty(M, C), dW1=_empty(C, F),
                 dW2=_empty(F, C), db1=_empty(F), db2=_empty(C))
        s["ws"] = _gemm_ws([(0, 0, M, F, C, bt.EPI_BIAS_GELU), (0, 0, M, C, F, bt.EPI_BIAS), (0, 1, M, F, C, bt.EPI_DGELU),
                            (0, 1, M, C, F, 0), (1, 0, F, C, M, 0), (1, 0, C, F, M, 0)])
    elif k == "head":
        M, C, Vp = c["M"], c["C"], c["Vp"]
        s.update(logits=_empty(M, Vp), loss=_empty(M), lse=_empty(M), dX=_empty(M, C), dwte=_empty(Vp, C))
        s["ws"] = _gemm_ws([(0, 1, M, Vp, C, 0), (0, 0, M, C, Vp, 0), (1, 0, Vp, C, M, 0)])
    elif k == "attention":
        B, T, H, hd = c["B"], c["T"], c["H"], c["hd"]
        s.update(out=_empty(B * T, H * hd), lse=_empty(B, H, T), dqkv=_empty(B * T, 3 * H * hd))
        s["ws"] = torch.empty(bt.lib().bt_attention_bwd_ws_bytes(B, T, H, hd), dtype=torch.uint8, device="cuda")
    elif k == "ring":
        W, B, T, H, hd = c["W"], c["B"], c["T"], c["H"], c["hd"]
        C, Tl = H * hd, T // W
        rows = [_ring_rows(c, r) for r in range(W)]
        qkv, dout = s.pop("qkv").reshape(B, T, 3 * C), s.pop("dout").reshape(B, T, C)
        s["qkv"] = [qkv[:, r].reshape(B * Tl, 3 * C).contiguous() for r in rows]
        s["dout"] = [dout[:, r].reshape(B * Tl, C).contiguous() for r in rows]
        s.update(out=[_empty(B * Tl, C) for _ in rows], lse=[_empty(B, H, Tl) for _ in rows],
                 D=[_empty(B, H, Tl) for _ in rows], dqkv=[_empty(B * Tl, 3 * C) for _ in rows])
        s["ws"] = torch.empty(max(ring.ws_bytes(W, T, B, H, hd), 16), dtype=torch.uint8, device="cuda")
    elif k == "norm":
        M, C = c["M"], c["C"]
        s.update(y=_empty(M, C), mean=_empty(M), rstd=_empty(M), dx=_empty(M, C), dgamma=_empty(C), dbeta=_empty(C))
        s["ws"] = torch.empty(bt.lib().bt_layernorm_bwd_ws_bytes(M, C), dtype=torch.uint8, device="cuda")
    else:
        net = bt.GPT2(_config(c), synth.HP_124M, c["B"], c["T"])
        net.params.copy_(s.pop("params"))
        net.opt_state.copy_(s.pop("moments"))
        net.step_count = _STEPS_TAKEN
        s["net"] = net
    return s


def _ring_rows(c, rank):
    """Global token positions of a rank's rows: chunks r and 2W-1-r of 2W."""
    seg = c["T"] // (2 * c["W"])
    a = torch.arange(seg, device="cuda")
    return torch.cat([rank * seg + a, (2 * c["W"] - 1 - rank) * seg + a])


# ---------------------------------------------------------------- one pass
def run(s):
    c = s["case"]
    k = c["kind"]
    if k == "linear":
        M, K, N, ws = c["M"], c["K"], c["N"], s["ws"]
        bt.bt_gemm(0, 0, M, N, K, s["X"], K, s["W"], N, 0.0, s["Y"], N, bias=s["b"], epi=bt.EPI_BIAS, ws=ws)
        bt.bt_gemm(0, 1, M, K, N, s["dY"], N, s["W"], N, 0.0, s["dX"], K, ws=ws)
        bt.bt_gemm(1, 0, K, N, M, s["X"], K, s["dY"], N, 0.0, s["dW"], N, colsum_B=s["db"], ws=ws)
        return {n: s[n] for n in ("Y", "dX", "dW", "db")}
    if k == "mlp":
        M, C, F, ws = c["M"], c["C"], 4 * c["C"], s["ws"]
        bt.bt_gemm(0, 0, M, F, C, s["X"], C, s["W1"], F, 0.0, s["act"], F, bias=s["b1"], epi=bt.EPI_BIAS_GELU,
                   preact_out=s["pre"], ws=ws)
        bt.bt_gemm(0, 0, M, C, F, s["act"], F, s["W2"], C, 0.0, s["Y"], C, bias=s["b2"], epi=bt.EPI_BIAS,
                   residual=s["R"], ws=ws)
        bt.bt_gemm(1, 0, F, C, M, s["act"], F, s["dY"], C, 0.0, s["dW2"], C, colsum_B=s["db2"], ws=ws)
        bt.bt_gemm(0, 1, M, F, C, s["dY"], C, s["W2"], C, 0.0, s["dh"], F, epi=bt.EPI_DGELU, gelu_in=s["pre"], ws=ws)
        bt.bt_gemm(1, 0, C, F, M, s["X"], C, s["dh"], F, 0.0, s["dW1"], F, colsum_B=s["db1"], ws=ws)
        bt.bt_gemm(0, 1, M, C, F, s["dh"], F, s["W1"], F, 0.0, s["dX"], C, ws=ws)
        return {n: s[n] for n in ("Y", "dX", "dW1", "db1", "dW2", "db2")}
    if k == "head":
        M, C, Vp, ws = c["M"], c["C"], c["Vp"], s["ws"]
        bt.bt_gemm(0, 1, M, Vp, C, s["X"], C, s["wte"], C, 0.0, s["logits"], Vp, ws=ws)
        bt.bt_softmax_xent_fused(s["logits"], s["targets"], s["loss"], s["lse"], 1.0 / M, M, c["V"], Vp)
        bt.bt_gemm(0, 0, M, C, Vp, s["logits"], Vp, s["wte"], C, 0.0, s["dX"], C, ws=ws)
        bt.bt_gemm(1, 0, Vp, C, M, s["logits"], Vp, s["X"], C, 0.0, s["dwte"], C, ws=ws)
        return {"loss": s["loss"], "lse": s["lse"], "dlogits": s["logits"], "dX": s["dX"], "dwte": s["dwte"]}
    if k == "attention":
        shape = (c["B"], c["T"], c["H"], c["hd"])
        bt.bt_attention_fwd(s["qkv"], s["out"], s["lse"], *shape)
        bt.bt_attention_bwd(s["dout"], s["qkv"], s["out"], s["lse"], s["dqkv"], *shape, ws=s["ws"])
        return {n: s[n] for n in ("out", "lse", "dqkv")}
    if k == "ring":
        C = c["H"] * c["hd"]
        ring.emulate(c["W"], c["T"], c["B"], c["H"], c["hd"], s["qkv"], s["out"], s["lse"],
                     lambda i: (s["qkv"][i][:, C:], 3 * C), dout=s["dout"], D=s["D"], dqkv=s["dqkv"],
                     dkv_of=lambda i: s["dqkv"][i][:, C:], ws=s["ws"])
        return {n: s[n] for n in ("out", "lse", "dqkv")}
    if k == "norm":
        M, C = c["M"], c["C"]
        bt.bt_layernorm_fwd(s["x"], s["gamma"], s["beta"], s["y"], s["mean"], s["rstd"], M, C)
        bt.bt_layernorm_bwd(s["dy"], s["x"], s["gamma"], s["mean"], s["rstd"], s["dx"], s["dgamma"], s["dbeta"], 0.0, 0.0,
                            M, C, ws=s["ws"])
        return {n: s[n] for n in ("y", "mean", "rstd", "dx", "dgamma", "dbeta")}
    net = s["net"]
    loss = net.train_step(s["tokens"], s["targets"])
    return {"loss": loss, "grads": net.grads, "params": net.params, "moments": net.opt_state}


# ---------------------------------------------------------------- the work
def work(case):
    c = case
    k = c["kind"]
    if k == "linear":
        M, K, N = c["M"], c["K"], c["N"]
        return {"bytes": 4.0 * (2 * M * K + 2 * M * N + 2 * K * N + 2 * N), "flops": 6.0 * M * K * N}
    if k == "mlp":
        M, C = c["M"], c["C"]
        # X, R, dY read, Y, dX written; the hidden pre-activation is kept for
        # the backward (written, read); both weights read, both gradients written
        return {"bytes": 4.0 * (5 * M * C + 2 * 4 * M * C + 4 * 4 * C * C + 10 * C), "flops": 48.0 * M * C * C}
    if k == "head":
        M, C, Vp = c["M"], c["C"], c["Vp"]
        return {"bytes": 4.0 * (2 * M * C + 2 * Vp * C + M * Vp + 3 * M), "flops": 6.0 * M * C * Vp}
    if k in ("attention", "ring"):
        B, T, H, hd = c["B"], c["T"], c["H"], c["hd"]
        pairs = B * H * T * (T + 1) / 2.0
        # forward S and O; backward S, dP, dV, dQ, dK
        return {"bytes": 4.0 * B * T * H * (8 * hd + 1), "flops": 14.0 * hd * pairs}
    if k == "norm":
        M, C = c["M"], c["C"]
        return {"bytes": 4.0 * (4 * M * C + 2 * M + 4 * C), "flops": 16.0 * M * C}
    M, C, L, V = c["B"] * c["T"], c["C"], c["L"], c["Vp"]
    P = synth.num_params(_config(c))
    # products of the layers and the head, three each; attention as above
    flops = 6.0 * M * (12 * C * C * L + C * V) + 14.0 * C * L * c["B"] * c["T"] * (c["T"] + 1) / 2.0
    # parameters read twice, gradients written and read, parameters and
    # moments updated; the activations that the backward needs, written and read
    return {"bytes": 4.0 * (9.0 * P + 2.0 * L * M * (3 * C + C + 4 * C + 2 * C) + 2.0 * M * V), "flops": flops}


# 2-norm errors: about four times the largest difference from 64-bit results
# measured over an output of the kind (1.2e-6, 1.1e-6, 3.9e-6, 2.8e-6, 1.0e-6,
# 1.5e-7 and 7.3e-6), where FP32 sums over up to 50,304 terms set the error
_REL = {"linear": 5e-6, "mlp": 5e-6, "head": 1.6e-5, "attention": 1.2e-5, "ring": 5e-6, "norm": 1e-6, "step": 3e-5}


def tolerance(case):
    return {"rel": _REL[case["kind"]]}


# ---------------------------------------------------------------- 64 bits
def _attention64(qkv, dout, B, T, H, hd):
    """out, lse, dqkv of causal attention, head by head."""
    q, k, v = (t.permute(0, 2, 1, 3) for t in qkv.reshape(B, T, 3, H, hd).unbind(2))
    do = dout.reshape(B, T, H, hd).permute(0, 2, 1, 3)
    out, lse = torch.empty_like(do), torch.empty((B, H, T), dtype=torch.float64, device=qkv.device)
    dqkv = torch.empty((B, T, 3, H, hd), dtype=torch.float64, device=qkv.device)
    dead = torch.ones((T, T), dtype=torch.bool, device=qkv.device).triu(1)
    scale = 1.0 / math.sqrt(hd)
    for b in range(B):
        for h in range(H):
            Q, K, V, G = (t[b, h].contiguous() for t in (q, k, v, do))
            S = (Q @ K.t()).mul_(scale).masked_fill_(dead, -math.inf)
            lse[b, h] = torch.logsumexp(S, 1)
            P = S.sub_(lse[b, h][:, None]).exp_()
            O = P @ V
            out[b, h] = O
            dqkv[b, :, 2, h] = P.t() @ G
            dP = G @ V.t()
            dS = dP.sub_((G * O).sum(1, keepdim=True)).mul_(P).mul_(scale)
            dqkv[b, :, 0, h] = dS @ K
            dqkv[b, :, 1, h] = dS.t() @ Q
    return out.permute(0, 2, 1, 3).reshape(B * T, H * hd), lse, dqkv.reshape(B * T, 3 * H * hd)


def _step64(c, i):
    cfg, hp = _config(c), synth.HP_124M
    F = torch.nn.functional
    offs = synth.param_offsets(cfg)
    p0 = i["params"].double()
    w = {n: p0[offs[j]:offs[j + 1]].reshape(shape).clone().requires_grad_(True)
         for j, (n, shape, _) in enumerate(synth.param_specs(cfg))}
    B, T, H, C, L = c["B"], c["T"], c["H"], c["C"], c["L"]
    dead = torch.ones((T, T), dtype=torch.bool, device="cuda").triu(1)
    ln = lambda x, n: F.layer_norm(x, (C,), w[n + "g"], w[n + "b"], cfg.ln_eps)  # noqa: E731
    total = 0.0
    for b in range(B):  # a sequence at a time: the gradients add up
        x = F.embedding(i["tokens"][b].long(), w["wte"]) + w["wpe"][:T]
        for l in range(L):
            h = f"h{l}."
            q, k, v = (ln(x, h + "ln1") @ w[h + "Wqkv"] + w[h + "bqkv"]).reshape(T, 3, H, C // H).permute(1, 2, 0, 3)
            s = (q @ k.transpose(1, 2) / math.sqrt(C // H)).masked_fill(dead, -math.inf)
            a = (s.softmax(-1) @ v).transpose(0, 1).reshape(T, C)
            x = x + a @ w[h + "Wo"] + w[h + "bo"]
            u = F.gelu(ln(x, h + "ln2") @ w[h + "Wfc"] + w[h + "bfc"], approximate="tanh")
            x = x + u @ w[h + "Wfp"] + w[h + "bfp"]
        logits = ln(x, "lnf") @ w["wte"].t()
        loss = F.cross_entropy(logits[:, :cfg.V], i["targets"][b].long(), reduction="sum") / (B * T)
        loss.backward()
        total += float(loss)
    g = torch.cat([w[n].grad.reshape(-1) for n, _, _ in synth.param_specs(cfg)])
    norm = float(g.norm())
    gc = g * min(1.0, hp.grad_clip / (norm + 1e-6))
    m, v = i["moments"].double().split(p0.numel())
    m = hp.beta1 * m + (1 - hp.beta1) * gc
    v = hp.beta2 * v + (1 - hp.beta2) * gc * gc
    t = _STEPS_TAKEN + 1
    decay = torch.zeros_like(p0)
    decay[:synth.num_decay_params(cfg)] = hp.weight_decay
    upd = (m / (1 - hp.beta1 ** t)) / ((v / (1 - hp.beta2 ** t)).sqrt() + hp.eps)
    p = p0 - hp.lr * decay * p0 - hp.lr * upd
    return {"loss": total, "grads": g, "params": p, "moments": torch.cat([m, v])}


def exact(case, seed):
    c, i = case, _inputs(case, seed)
    k = c["kind"]
    if k == "step":
        return _step64(c, i)
    if k in ("attention", "ring"):
        B, T, H, hd = c["B"], c["T"], c["H"], c["hd"]
        out, lse, dqkv = _attention64(i["qkv"].double(), i["dout"].double(), B, T, H, hd)
        if k == "attention":
            return {"out": out, "lse": lse, "dqkv": dqkv}
        rows = [_ring_rows(c, r) for r in range(c["W"])]
        C = H * hd
        pick = lambda x, n: [x.reshape(B, T, n)[:, r].reshape(-1, n) for r in rows]  # noqa: E731
        return {"out": pick(out, C), "lse": [lse[:, :, r] for r in rows], "dqkv": pick(dqkv, 3 * C)}
    d = {n: t if t.dtype == torch.int32 else t.double() for n, t in i.items()}
    if k == "linear":
        return {"Y": d["X"] @ d["W"] + d["b"], "dX": d["dY"] @ d["W"].t(), "dW": d["X"].t() @ d["dY"], "db": d["dY"].sum(0)}
    if k == "mlp":
        pre = (d["X"] @ d["W1"] + d["b1"]).requires_grad_(True)
        act = torch.nn.functional.gelu(pre, approximate="tanh")
        Y = act.detach() @ d["W2"] + d["b2"] + d["R"]
        dh, = torch.autograd.grad(act, pre, d["dY"] @ d["W2"].t())
        return {"Y": Y, "dX": dh @ d["W1"].t(), "dW1": d["X"].t() @ dh, "db1": dh.sum(0),
                "dW2": act.detach().t() @ d["dY"], "db2": d["dY"].sum(0)}
    if k == "head":
        M, V = c["M"], c["V"]
        z = d["X"] @ d["wte"].t()
        lse = torch.logsumexp(z[:, :V], 1)
        t = d["targets"].long()[:, None]
        loss = lse - z.gather(1, t)[:, 0]
        z[:, :V] = (z[:, :V] - lse[:, None]).exp()
        z[:, V:] = 0
        z.scatter_add_(1, t, torch.full((M, 1), -1.0, dtype=torch.float64, device="cuda"))
        z /= M
        return {"loss": loss, "lse": lse, "dlogits": z, "dX": z @ d["wte"], "dwte": z.t() @ d["X"]}
    x, M, C = d["x"], c["M"], c["C"]
    mean = x.mean(1)
    rstd = (x.var(1, unbiased=False) + 1e-5).rsqrt()
    xh = (x - mean[:, None]) * rstd[:, None]
    gy = d["dy"] * d["gamma"]
    dx = rstd[:, None] * (gy - gy.mean(1, keepdim=True) - xh * (gy * xh).mean(1, keepdim=True))
    return {"y": xh * d["gamma"] + d["beta"], "mean": mean, "rstd": rstd, "dx": dx, "dgamma": (d["dy"] * xh).sum(0),
            "dbeta": d["dy"].sum(0)}
