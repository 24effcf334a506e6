"""The calls that are timed: what a program that uses this package has it do, through its public entry points.

Three kinds of use stand behind the list: serving (decoding with a key/value cache, prefill), training (the forward pass
with its backward pass, bias tensors included) and the recurrent pattern (gated retention, Mamba2's state space module),
forwards and backwards.  Sizes are those of the package's own benchmark (`workloads.py`, `bench.py`) or generic ones of
the same ranges; inputs are N(0, 1) in bfloat16, gates follow the recipes of `workloads.make_gates`.

listed() is the fixed list, draw() gives one more case of the same ranges, prepare() builds what a caller holds before the
call, run() is one call, work() the bytes and operations it cannot do without, exact() the result in 64 bits.
"""
import math

import numpy as np
import torch

from paper_2502_15349_amd import ae_attn as A

CAUSAL = {"mask": "causal"}


def _attention(name, op, B, H_q, H_kv, L_q, L_k, D_qk, D_v, **kw):
    c = dict(name=name, op=op, B=B, H_q=H_q, H_kv=H_kv, L_q=L_q, L_k=L_k, D_qk=D_qk, D_v=D_v, norm="softmax",
             score_mod="none", mask="none", window=0, out="f32", layout="bhld")
    c.update(kw)
    return c


def _gated(name, op, B, H, H_qk, L, D_qk, D_v, **kw):
    c = dict(name=name, op=op, B=B, H=H, H_qk=H_qk, L=L, D_qk=D_qk, D_v=D_v, gates="gated_retention", out="f32",
             segmented=False, state=False)
    c.update(kw)
    return c


def listed():
    return [
        # One new token of one sequence against 8k cached keys, the smallest call of a serving loop (the decoding row of
        # the paper's Table 2): launches and latency count.
        _attention("decode_1x16x8192", "decode", 1, 16, 16, 1, 8192, 192, 128),
        # One new token each of sixteen sequences, grouped heads, an odd number of keys in a cache with room to grow.
        _attention("decode_gqa_16x32x5003", "decode", 16, 32, 8, 1, 5003, 128, 128, out="bf16", layout="cache"),
        # Prefill of a layer with grouped heads at an ordinary size, 16-bit output as the next projection takes it.
        _attention("prefill_gqa_4x32x2048", "forward", 4, 32, 8, 2048, 2048, 128, 128, out="bf16", **CAUSAL),
        # Long prefill with 192/128 heads: the benchmark's largest configuration.
        _attention("prefill_mla_1x128x8192", "forward", 1, 128, 128, 8192, 8192, 192, 128, **CAUSAL),
        # Sigmoid attention of a language model: no row reduction, small heads.
        _attention("sigmoid_8x16x4096", "forward", 8, 16, 16, 4096, 4096, 64, 64, norm="sigmoid", score_mod="bias", **CAUSAL),
        # Retention in its parallel form with the head dims of the paper's Table 2.
        _attention("retention_1x32x4096_256_512", "forward", 1, 32, 32, 4096, 4096, 256, 512, norm="abssum",
                   score_mod="head_decay", **CAUSAL),
        # Backward pass of the layer above at its training size.
        _attention("bwd_gqa_4x32x2048", "backward", 4, 32, 8, 2048, 2048, 128, 128, **CAUSAL),
        # Backward pass of the largest configuration.
        _attention("bwd_mla_1x128x8192", "backward", 1, 128, 128, 8192, 8192, 192, 128, **CAUSAL),
        # Backward pass of an encoder layer with a learned additive bias and ragged sequence lengths, rows of all heads
        # side by side as a fused projection leaves them.
        _attention("bwd_bias_2x12x1023x1201", "backward", 2, 12, 12, 1023, 1201, 64, 64, score_mod="bias_tensor",
                   out="bf16", layout="blhd"),
        # Gated retention over a batch of long sequences.
        _gated("gated_retention_8x32x8192", "gated_forward", 8, 32, 32, 8192, 128, 128),
        # Mamba2's state space module on one sequence (all heads share B and C), the state handed on.
        _gated("mamba2_1x80x8192", "gated_forward", 1, 80, 1, 8192, 128, 64, gates="mamba2", segmented=True, state=True),
        # ... and its backward pass in training, at the longest rows that can be compared (see draw()).
        _gated("mamba2_bwd_8x80x768", "gated_backward", 8, 80, 1, 768, 128, 64, gates="mamba2"),
    ]


def _log_int(rng, lo, hi):
    """Spread over the logarithm; a third of them round, the others as they fall."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if n >= 128 and rng.random() < 0.33:
        n = n // 64 * 64
    return max(lo, min(hi, n))


def draw(rng):
    c = _draw(rng)
    del c["name"]
    return c


def _draw(rng):
    op = rng.choice(["decode", "decode", "forward", "forward", "forward", "backward", "backward", "backward",
                     "gated_forward", "gated_backward", "retention_recurrent"])
    out = rng.choice(["f32", "bf16"])
    if op == "decode":
        B, (H_q, H_kv) = _log_int(rng, 1, 64), rng.choice([(16, 16), (32, 8), (32, 32), (64, 8), (12, 12)])
        D_qk, D_v = rng.choice([(64, 64), (128, 128), (128, 128), (192, 128)])
        L = _log_int(rng, 200, 32768)
        while B * H_q * L * (D_qk + D_v) > 3e9:
            L = L * 2 // 3
        return _attention("", op, B, H_q, H_kv, 1, L, D_qk, D_v, out=out, layout=rng.choice(["bhld", "cache"]))
    if op in ("forward", "backward"):
        D_qk, D_v = rng.choice([(64, 64), (128, 128), (128, 128), (192, 128), (128, 256)] + ([(256, 512)] if op == "forward" else []))
        kinds = [("softmax", "none"), ("softmax", "none"), ("sigmoid", "bias"), ("abssum", "head_decay"), ("none", "relu")]
        if (D_qk, D_v) != (128, 256):
            kinds.append(("softmax", "bias_tensor"))
        norm, mod = rng.choice(kinds) if D_v != 512 else ("abssum", "head_decay")
        masks = {"head_decay": ["causal"], "bias_tensor": ["none", "causal"], "relu": ["none", "causal"]}
        mask = rng.choice(masks.get(mod, ["none", "causal", "causal", "sliding_window"]))
        H_q, H_kv = rng.choice([(16, 16), (32, 8), (12, 12), (24, 6), (6, 6)])
        B, L_q = rng.choice([1, 1, 2, 4, 8]), _log_int(rng, 100, 8192)
        L_k = L_q if rng.random() < 0.7 else max(64, int(L_q * rng.uniform(1.0, 1.5)))
        most = 1.5e12 if op == "forward" else 0.8e12
        if mod == "bias_tensor":
            most = 0.3e12
        while 2.0 * B * H_q * L_q * L_k * (D_qk + D_v) > most:
            L_q, L_k = L_q * 3 // 4, L_k * 3 // 4
        window = _log_int(rng, 64, max(65, L_k)) if mask == "sliding_window" else 0
        return _attention("", op, B, H_q, H_kv, L_q, L_k, D_qk, D_v,
                          norm=norm, score_mod=mod, mask=mask, window=window, out=out, layout=rng.choice(["bhld", "blhd"]))
    # (the gradient of the log-decays is a suffix sum whose rounding grows with the root of the number of later tokens,
    # 0.019 of its norm at 1024 tokens, 0.059 at 8192: from there on two correct results are too far apart to compare)
    L = _log_int(rng, 100, 768 if op == "gated_backward" else 32768)
    if op == "retention_recurrent":
        B, H, D = _log_int(rng, 1, 8), rng.choice([8, 16, 32]), rng.choice([64, 128])
        while B * H * L > 8 * 32 * 8192:
            L = L * 2 // 3
        return _gated("", op, B, H, H, L, D, D, gates="constant", out=out, state=rng.random() < 0.5)
    B, kind = _log_int(rng, 1, 8), rng.choice(["gated_retention", "mamba2"])
    if kind == "mamba2":
        H, H_qk = rng.choice([(80, 1), (64, 1), (24, 1), (32, 8)])
        D_qk, D_v = rng.choice([(128, 64), (128, 64), (64, 64)])
    else:
        H = H_qk = rng.choice([8, 16, 32])
        D_qk, D_v = rng.choice([(128, 128), (128, 128), (64, 64), (64, 128)])
    while B * H * L > 8 * 32 * 8192:
        L = L * 2 // 3
    return _gated("", op, B, H, H_qk, L, D_qk, D_v, gates=kind, out=out if op == "gated_forward" else "f32",
                  segmented=op == "gated_forward" and rng.random() < 0.7, state=op == "gated_forward" and rng.random() < 0.5)


# ---- inputs -------------------------------------------------------------------------------------------------------
def _normal(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(torch.bfloat16)


def _rows(g, layout, B, H, L, D):
    """[B, H, L, D]: contiguous, a view of [B, L, H, D], or the filled part of a cache with room for more rows."""
    if layout == "blhd":
        return _normal(g, B, L, H, D).transpose(1, 2)
    if layout == "cache":
        return _normal(g, B, H, (L + 1024) // 1024 * 1024, D)[:, :, :L]
    return _normal(g, B, H, L, D)


def _gamma(H):
    return [float(np.float32(1.0 - 2.0 ** (-5 - h % 32))) for h in range(H)]


def _inputs(case, seed):
    c, g = case, torch.Generator(device="cuda")
    g.manual_seed(seed)
    bf = torch.bfloat16
    s = {}
    if c["op"] in ("decode", "forward", "backward"):
        q_layout = "blhd" if c["layout"] == "blhd" else "bhld"
        s["Q"] = _rows(g, q_layout, c["B"], c["H_q"], c["L_q"], c["D_qk"])
        s["K"] = _rows(g, c["layout"], c["B"], c["H_kv"], c["L_k"], c["D_qk"])
        s["V"] = _rows(g, c["layout"], c["B"], c["H_kv"], c["L_k"], c["D_v"])
        s["params"] = dict(scale=c["D_qk"] ** -0.5, norm=c["norm"], score_mod=c["score_mod"], mask=c["mask"], window=c["window"])
        if c["score_mod"] == "bias":
            s["params"]["bias"] = float(np.float32(-math.log(c["L_k"])))
        if c["score_mod"] == "head_decay":
            s["params"]["gamma"] = _gamma(c["H_q"])
        if c["score_mod"] == "bias_tensor":  # one bias per head, shared over the batch; rows padded to 8 elements
            s["params"]["bias_tensor"] = _normal(g, 1, c["H_q"], c["L_q"], (c["L_k"] + 7) // 8 * 8)[..., :c["L_k"]]
        if c["op"] == "backward":
            s["dO"] = _normal(g, c["B"], c["H_q"], c["L_q"], c["D_v"])
        return s
    s["Q"] = _normal(g, c["B"], c["H_qk"], c["L"], c["D_qk"])
    s["K"] = _normal(g, c["B"], c["H_qk"], c["L"], c["D_qk"])
    s["V"] = _normal(g, c["B"], c["H"], c["L"], c["D_v"])
    s["scale"] = c["D_qk"] ** -0.5
    s["key_gate"] = None
    if c["gates"] == "constant":
        s["gamma"] = _gamma(c["H"])
    else:
        x = torch.randn((c["B"], c["H"], c["L"]), generator=g, device="cuda", dtype=torch.float32)
        if c["gates"] == "mamba2":
            s["key_gate"] = torch.nn.functional.softplus(x - 4.0)
            s["log_decay"] = s["key_gate"] * -(1.0 + (torch.arange(c["H"], device="cuda") % 16)).float().view(1, -1, 1)
        else:
            s["log_decay"] = torch.nn.functional.logsigmoid(x) / 16.0
    if c["state"]:
        s["h_in"] = torch.randn((c["B"], c["H"], c["D_qk"], c["D_v"]), generator=g, device="cuda", dtype=torch.float32)
    if c["op"] == "gated_backward":
        s["dO"] = _normal(g, c["B"], c["H"], c["L"], c["D_v"])
    s["out_dtype"] = bf if c["out"] == "bf16" else torch.float32
    return s


class _Handle:
    """A serving loop's handle, kept with its output buffer and workspace from token to token."""

    def __init__(self, c, s):
        self.out = torch.empty((c["B"], c["H_q"], c["L_q"], c["D_v"]), device="cuda", dtype=torch.bfloat16 if c["out"] == "bf16" else torch.float32)
        self.handle = A.ae_attn_create(B=c["B"], H_q=c["H_q"], H_kv=c["H_kv"], L_q=c["L_q"], L_k=c["L_k"], D_qk=c["D_qk"], D_v=c["D_v"],
                                       scale=s["params"]["scale"], norm=c["norm"], mask=c["mask"], k_stride=s["K"].stride()[:3],
                                       v_stride=s["V"].stride()[:3], out_dtype=c["out"], kv_splits=-1)
        self.bytes = A.ae_attn_workspace_bytes(self.handle)
        self.workspace = torch.empty(max(self.bytes, 16), dtype=torch.uint8, device="cuda")

    def __del__(self):
        A.ae_attn_destroy(self.handle)


def prepare(case, seed):
    s = dict(_inputs(case, seed), op=case["op"], case=case)
    if case["op"] == "decode":
        s["h"] = _Handle(case, s)
    if case["op"] == "forward":
        s["params"]["out_dtype"] = torch.bfloat16 if case["out"] == "bf16" else torch.float32
    if case["op"] == "backward":  # what the forward pass left behind
        stats = None
        if case["norm"] in ("softmax", "abssum"):
            stats = torch.empty((case["B"], case["H_q"], case["L_q"]), device="cuda", dtype=torch.float32)
        s["O"] = A.attention_forward(s["Q"], s["K"], s["V"], stats=stats, out_dtype=torch.bfloat16 if case["out"] == "bf16" else torch.float32, **s["params"])
        s["stats"] = stats
        if stats is None:
            s["O"] = None
    return s


def run(s):
    op = s["op"]
    if op == "decode":
        h = s["h"]
        A.ae_attn_forward_split(h.handle, s["Q"].data_ptr(), s["K"].data_ptr(), s["V"].data_ptr(), h.out.data_ptr(), 0, h.workspace.data_ptr(),
                                h.workspace.numel(), torch.cuda.current_stream().cuda_stream)
        return h.out
    if op == "forward":
        return A.attention_forward(s["Q"], s["K"], s["V"], **s["params"])
    if op == "backward":
        return A.attention_backward(s["Q"], s["K"], s["V"], s["O"], s["dO"], s["stats"], want_dbias="bias_tensor" in s["params"], **s["params"])
    if op == "gated_forward":
        return A.gated_recurrent(s["Q"], s["K"], s["V"], s["log_decay"], s["key_gate"], scale=s["scale"], h_in=s.get("h_in"), want_state=s["case"]["state"],
                                 out_dtype=s["out_dtype"], segmented=s["case"]["segmented"])
    if op == "gated_backward":
        return A.gated_recurrent_backward(s["Q"], s["K"], s["V"], s["log_decay"], s["key_gate"], s["dO"], scale=s["scale"])
    return A.retention_recurrent(s["Q"], s["K"], s["V"], scale=s["scale"], gamma=s["gamma"], h_in=s.get("h_in"), return_state=s["case"]["state"],
                                 out_dtype=s["out_dtype"])


# ---- the work of a pass -------------------------------------------------------------------------------------------
def _pairs(c):
    """Visible (query, key) pairs of one head."""
    n_q, n_k = c["L_q"], c["L_k"]
    if c["mask"] == "none":
        return n_q * n_k
    last = np.arange(n_q, dtype=np.int64) + n_k - n_q + 1
    first = np.maximum(last - c["window"], 0) if c["mask"] == "sliding_window" else 0
    return int(np.maximum(np.minimum(last, n_k) - first, 0).sum())


def work(case):
    c, out = case, 2 if case["out"] == "bf16" else 4
    if c["op"] in ("decode", "forward", "backward"):
        q, kv, dqk, dv = c["B"] * c["H_q"] * c["L_q"], c["B"] * c["H_kv"] * c["L_k"], c["D_qk"], c["D_v"]
        pairs, bias = c["B"] * c["H_q"] * _pairs(c), 0
        if c["score_mod"] == "bias_tensor":
            bias = 2 * c["H_q"] * c["L_q"] * c["L_k"]
        if c["op"] == "backward":
            rows = 4 * q + out * q * dv if c["norm"] in ("softmax", "abssum") else 0
            return {"bytes": 6 * q * dqk + 6 * kv * (dqk + dv) + 2 * q * dv + rows + bias * (1 + c["B"] if bias else 1),
                    "flops": 2 * (3 * dqk + 2 * dv) * pairs}
        return {"bytes": 2 * q * dqk + 2 * kv * (dqk + dv) + out * q * dv + bias, "flops": 2 * (dqk + dv) * pairs}
    qk, v = c["B"] * c["H_qk"] * c["L"] * c["D_qk"], c["B"] * c["H"] * c["L"] * c["D_v"]
    gates = {"constant": 0, "gated_retention": 1, "mamba2": 2}[c["gates"]] * 4 * c["B"] * c["H"] * c["L"]
    state = 8 * c["B"] * c["H"] * c["D_qk"] * c["D_v"] if c["state"] else 0
    flops = 4 * c["B"] * c["H"] * c["L"] * c["D_qk"] * c["D_v"]
    if c["op"] == "gated_backward":
        return {"bytes": 12 * qk + 8 * v + 2 * gates, "flops": 3 * flops}
    return {"bytes": 4 * qk + (2 + out) * v + gates + state, "flops": flops}


def tolerance(case):
    """bfloat16 weights and carried states in front of 32-bit sums: about four times what the package's results are
    away from those in 64 bits (0.0017 to 0.0029)."""
    if case["op"] == "gated_backward":  # the suffix sums of dlog_decay gather the rounding of every later token
        return {"rel": 0.03, "max": 0.5}
    return {"rel": 0.01, "max": 0.3}


# ---- results in 64 bits ---------------------------------------------------------------------------------------------
def _head(c, s, b, h):
    """(P, row sums for abs-sum, factor between dP and the raw score's gradient) of one head, P normalized."""
    f64 = torch.float64
    p = s["params"]
    hk = h // (c["H_q"] // c["H_kv"])
    q, k, v = s["Q"][b, h].to(f64), s["K"][b, hk].to(f64), s["V"][b, hk].to(f64)
    x = (q @ k.T) * p["scale"]
    i = torch.arange(c["L_q"], device="cuda").view(-1, 1) + (c["L_k"] - c["L_q"])
    j = torch.arange(c["L_k"], device="cuda").view(1, -1)
    hidden = None
    if c["mask"] != "none":
        hidden = j > i
        if c["mask"] == "sliding_window":
            hidden |= j <= i - c["window"]
    decay = None
    if c["score_mod"] == "bias":
        x += p["bias"]
    elif c["score_mod"] == "bias_tensor":
        x += p["bias_tensor"][0, h].to(f64)
    elif c["score_mod"] == "head_decay":
        decay = torch.exp(math.log(p["gamma"][h]) * (i - j).clamp(min=0).to(f64))
        x *= decay
    step = None
    if c["score_mod"] == "relu":
        step = x > 0
        x.clamp_(min=0)
    n = sign = None
    if c["norm"] == "softmax":
        if hidden is not None:
            x.masked_fill_(hidden, -math.inf)
        m = x.amax(dim=1, keepdim=True).clamp(min=-1e300)
        x = torch.exp(x - m)
        x /= x.sum(dim=1, keepdim=True).clamp(min=1e-300)
    elif c["norm"] == "sigmoid":
        x = torch.sigmoid(x)
        if hidden is not None:
            x.masked_fill_(hidden, 0.0)
    else:
        if hidden is not None:
            x.masked_fill_(hidden, 0.0)
        if c["norm"] == "abssum":
            r = x.abs().sum(dim=1, keepdim=True)
            n, sign = r.clamp(min=1.0), torch.sign(x) * (r > 1)
            x /= n
    return q, k, v, x, hidden, decay, step, n, sign, hk


def _exact_attention(c, s):
    dtype = dict(device="cuda", dtype=torch.float64)
    if c["op"] != "backward":
        O = torch.empty((c["B"], c["H_q"], c["L_q"], c["D_v"]), **dtype)
        for b in range(c["B"]):
            for h in range(c["H_q"]):
                _, _, v, P = _head(c, s, b, h)[:4]
                O[b, h] = P @ v
        return O
    dQ = torch.empty((c["B"], c["H_q"], c["L_q"], c["D_qk"]), **dtype)
    dK = torch.zeros((c["B"], c["H_kv"], c["L_k"], c["D_qk"]), **dtype)
    dV = torch.zeros((c["B"], c["H_kv"], c["L_k"], c["D_v"]), **dtype)
    dB = torch.empty((c["B"], c["H_q"], c["L_q"], c["L_k"]), **dtype) if c["score_mod"] == "bias_tensor" else None
    for b in range(c["B"]):
        for h in range(c["H_q"]):
            q, k, v, P, hidden, decay, step, n, sign, hk = _head(c, s, b, h)
            do = s["dO"][b, h].to(torch.float64)
            dV[b, hk] += P.T @ do
            dS = do @ v.T
            if c["norm"] == "softmax":
                dS = P * (dS - (P * dS).sum(dim=1, keepdim=True))
            elif c["norm"] == "sigmoid":
                dS *= P * (1 - P)
            elif c["norm"] == "abssum":
                delta = (P * dS).sum(dim=1, keepdim=True)
                dS = (dS - sign * delta) / n
            if step is not None:
                dS *= step
            if hidden is not None:
                dS.masked_fill_(hidden, 0.0)
            if dB is not None:
                dB[b, h] = dS
            if decay is not None:
                dS *= decay
            dQ[b, h] = dS @ k * s["params"]["scale"]
            dK[b, hk] += dS.T @ q * s["params"]["scale"]
    return (dQ, dK, dV) if dB is None else (dQ, dK, dV, dB)


def _walk(q, k, v, log_decay, h0=None):
    """o_t = q_t h_t, h_t = e^{log_decay_t} h_{t-1} + k_t^T v_t over [H, L, D] in 64 bits, 64 tokens at a time."""
    H, L, _ = v.shape
    o = torch.empty((H, L, v.shape[2]), device="cuda", dtype=torch.float64)
    h = torch.zeros((H, k.shape[2], v.shape[2]), device="cuda", dtype=torch.float64) if h0 is None else h0
    for t in range(0, L, 64):
        qc, kc, vc = q[:, t:t + 64], k[:, t:t + 64], v[:, t:t + 64]
        b = log_decay[:, t:t + 64].cumsum(dim=1)
        w = torch.exp((b.unsqueeze(2) - b.unsqueeze(1)).tril()).tril()
        o[:, t:t + 64] = torch.exp(b).unsqueeze(2) * (qc @ h) + ((qc @ kc.transpose(1, 2).contiguous()) * w) @ vc
        last = b[:, -1:]
        h = torch.exp(last).unsqueeze(2) * h + (kc * torch.exp(last - b).unsqueeze(2)).transpose(1, 2).contiguous() @ vc
    return o, h


def _exact_recurrent(c, s):
    f64 = torch.float64
    B, H, L, G = c["B"], c["H"], c["L"], c["H"] // c["H_qk"]
    dtype = dict(device="cuda", dtype=f64)

    def heads(t):
        return t.to(f64).repeat_interleave(G, dim=0) if G > 1 else t.to(f64)

    if c["gates"] == "constant":
        la_all = torch.tensor(s["gamma"], **dtype).log().view(1, H, 1).expand(B, H, L)
    else:
        la_all = s["log_decay"].to(f64)
    if c["op"] != "gated_backward":
        O = torch.empty((B, H, L, c["D_v"]), **dtype)
        S = torch.empty((B, H, c["D_qk"], c["D_v"]), **dtype)
        for b in range(B):
            k = heads(s["K"][b])
            if s["key_gate"] is not None:
                k *= s["key_gate"][b].to(f64).unsqueeze(2)
            O[b], S[b] = _walk(heads(s["Q"][b]) * s["scale"], k, s["V"][b].to(f64), la_all[b], s["h_in"][b].to(f64) if c["state"] else None)
        return (O, S) if c["state"] else O
    dQ, dK = torch.empty(s["Q"].shape, **dtype), torch.empty(s["K"].shape, **dtype)
    dV, dla = torch.empty(s["V"].shape, **dtype), torch.empty((B, H, L), **dtype)
    dkg = None if s["key_gate"] is None else torch.empty((B, H, L), **dtype)
    for b in range(B):
        q, k, v, do, la = heads(s["Q"][b]) * s["scale"], heads(s["K"][b]), s["V"][b].to(f64), s["dO"][b].to(f64), la_all[b]
        g = torch.ones((H, L), **dtype) if dkg is None else s["key_gate"][b].to(f64)
        g = g.unsqueeze(2)
        back = torch.cat([torch.zeros((H, 1), **dtype), la[:, 1:].flip(1)], dim=1)  # the decay behind each token, last first
        dq = _walk(do, v, k * g, la)[0] * s["scale"]
        x = _walk(v.flip(1), do.flip(1), q.flip(1), back)[0].flip(1)
        dV[b] = _walk(k.flip(1), q.flip(1), do.flip(1), back)[0].flip(1) * g
        dB = (q * dq).sum(2) / s["scale"] - (k * x * g).sum(2)
        dla[b] = dB.flip(1).cumsum(1).flip(1)
        if dkg is not None:
            dkg[b] = (k * x).sum(2)
        dQ[b] = dq.view(c["H_qk"], G, L, -1).sum(1)
        dK[b] = (x * g).view(c["H_qk"], G, L, -1).sum(1)
    return dQ, dK, dV, dla, dkg


def exact(case, seed):
    s = _inputs(case, seed)
    return _exact_attention(case, s) if case["op"] in ("decode", "forward", "backward") else _exact_recurrent(case, s)
