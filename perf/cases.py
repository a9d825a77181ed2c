"""Performance cases of the LeapQuant path: what a serving program has the library do, at the sizes it does it.

Kinds of case
  window      one window of decode steps and the commit that ends it, either as one call per token ("eager") or as a
              HIP graph that was captured once and is replayed ("graph", how a server runs a small batch)
  continuous  one leapquant_decode_step_commit call over requests at different window positions (continuous batching:
              every step some requests end their window)
  quantize    leapquant_quantize_state of given fp32 states (the end of a prefill, or a prefix cache)
  export      leapquant_dequantize_state of states in mid-window (checkpoint, inspection)

Not here: the dense fp32 / bf16 step and the per-window BF16 state, which exist to be compared against.

All inputs are drawn on the GPU from the seed: unit-norm q and k, v ~ N(0, I), beta = sigmoid(N(0, 1)), decays
exp(-0.1 softplus(N(0, 1))), and states of 16 rank-one terms of falling weight plus noise with two outlier rows and
columns (RWKV7: its own decays, removal keys and in-context rates, as two sub-steps per token).
"""
import math

import torch

from paper_2609_38166_amd import binding as B

D = 128
CODES = {"int8": B.LQ_CODE_INT8, "e4m3": B.LQ_CODE_E4M3, "int6": B.LQ_CODE_INT6, "int4": B.LQ_CODE_INT4}
QMAX = {"int8": 127.0, "e4m3": 448.0, "int6": 31.0, "int4": 7.0}
BITS = {"int8": 8, "e4m3": 8, "int6": 6, "int4": 4}
SWEEPS = 4


def _case(kind, batch, heads_v, heads_k, window, n_comp, gate, code="int8", rule="delta", graph=False, name=None):
    c = {"kind": kind, "batch": batch, "heads_v": heads_v, "heads_k": heads_k, "window": window, "n_comp": n_comp,
         "gate": gate, "code": code, "rule": rule, "graph": graph}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one KDA layer (Kimi-Linear shape) at serving batch 256: the headline workload, window by window
        _case("window", 256, 32, 32, 64, 8, "diag", name="kda_batch256"),
        # one GDN layer with grouped key heads (Qwen3-Next shape) at batch 64
        _case("window", 64, 32, 16, 64, 8, "scalar", name="gdn_gqa_batch64"),
        # the method's default window and token count (W = 16, r = 4) at batch 256
        _case("window", 256, 32, 32, 16, 4, "scalar", name="gdn_w16_batch256"),
        # an odd batch and an odd head count with FP8 codes and a window that is no multiple of anything
        _case("window", 37, 12, 4, 21, 4, "scalar", code="e4m3", name="gdn_e4m3_ragged"),
        # one GPU's share of the KDA layer under 8-way tensor parallelism
        _case("window", 256, 4, 4, 64, 8, "diag", graph=True, name="kda_tp8_share"),
        # one request alone: interactive decoding, where latency counts
        _case("window", 1, 32, 32, 64, 8, "diag", graph=True, name="kda_one_request"),
        # the smallest calls, one at a time from Python: launches and host work count
        _case("window", 4, 4, 4, 16, 4, "scalar", name="gdn_tiny_eager"),
        # continuous batching: one fused step over requests at all window positions
        _case("continuous", 128, 32, 32, 64, 8, "diag", name="kda_continuous"),
        # RWKV7 (two sub-steps per token through the general read vector) with the 4-bit codes
        _case("window", 24, 32, 32, 32, 8, "diag", code="int4", rule="general", name="rwkv7_int4"),
        # a prefix cache quantized in bulk
        _case("quantize", 512, 32, 32, 16, 8, "scalar", name="quantize_bulk"),
        # one request admitted after its prefill
        _case("quantize", 1, 32, 32, 64, 8, "diag", name="quantize_one"),
        # a batch exported in mid-window, 6-bit codes
        _case("export", 64, 32, 32, 64, 8, "diag", code="int6", name="export_int6"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["window", "window", "window", "continuous", "quantize", "quantize", "export"])
    window = _log_int(rng, 8, 128)
    heads_k = rng.choice([1, 2, 3, 4, 8, 12, 16, 32])
    heads_v = heads_k * (rng.choice([1, 1, 2, 3]) if heads_k <= 16 else 1)
    most = 16384 if kind == "quantize" else 8192 * 64 // max(window, 64)
    batch = _log_int(rng, 1, max(1, most // heads_v))
    gate = rng.choice(["scalar", "diag"])
    rule = rng.choice(["delta", "delta", "delta", "general"]) if kind == "window" and gate == "diag" else "delta"
    if rule == "general":
        heads_k, window = heads_v, window + window % 2      # whole tokens of two sub-steps
    batch = max(1, min(batch, (8192 * 64) // (window * heads_v)))
    return _case(kind, batch, heads_v, heads_k, window, rng.choice([2, 4, 4, 8, 8]), gate,
                 code=rng.choice(["int8", "int8", "e4m3", "int6", "int4"]), rule=rule,
                 graph=kind == "window" and batch * heads_v <= 2048 and rng.random() < 0.5)


# ---------------------------------------------------------------------------------------------------------- inputs

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _unit(x):
    return x / x.norm(dim=-1, keepdim=True)


def _states(case, g):
    """fp32 states S^T [B][H][d_v][d_k]: 16 rank-one terms of falling weight, noise, two outlier rows and columns."""
    b, h = case["batch"], case["heads_v"]
    n = b * h
    kk = _unit(torch.randn((n, 16, D), generator=g, device="cuda"))
    vv = _unit(torch.randn((n, 16, D), generator=g, device="cuda"))
    vv *= (0.8 ** torch.arange(16, device="cuda", dtype=torch.float32))[None, :, None]
    S = torch.randn((n, D, D), generator=g, device="cuda") * 0.05
    for j in range(16):
        S += vv[:, j, :, None] * kk[:, j, None, :]
    rows = torch.ones((n, D), device="cuda").scatter_(1, torch.randint(0, D, (n, 2), generator=g, device="cuda"), 20.0)
    cols = torch.ones((n, D), device="cuda").scatter_(1, torch.randint(0, D, (n, 2), generator=g, device="cuda"), 20.0)
    S *= torch.maximum(rows[:, None, :], cols[:, :, None])
    return S.view(b, h, D, D)


def _tokens(case, steps, g):
    """Step-major token inputs of `steps` steps."""
    b, hv, hk = case["batch"], case["heads_v"], case["heads_k"]

    def rn(*shape):
        return torch.randn((steps,) + shape, generator=g, device="cuda")

    if case["rule"] == "general":
        # RWKV7: an erase (alpha = w, k = kappa, b = a . kappa, v = 0), then a write (alpha = 1, b = 0), per token
        w = torch.exp(-math.exp(-0.5) * torch.sigmoid(rn(b, hv, D)))
        kap, k, r = _unit(rn(b, hv, D)), _unit(rn(b, hv, D)), _unit(rn(b, hv, D))
        read, v = torch.sigmoid(rn(b, hv, D)) * kap, rn(b, hv, D)
        r[1::2] = r[0::2]
        kap[1::2], w[1::2], read[1::2], v[0::2] = k[1::2], 1.0, 0.0, 0.0
        return {"q": r, "k": kap, "b": read, "v": v, "alpha": w, "beta": torch.ones((steps, b, hv), device="cuda")}
    gate = (b, hv, D) if case["gate"] == "diag" else (b, hv)
    return {"q": _unit(rn(b, hk, D)), "k": _unit(rn(b, hk, D)), "v": rn(b, hv, D),
            "alpha": torch.exp(-0.1 * torch.nn.functional.softplus(rn(*gate))), "beta": torch.sigmoid(rn(b, hv))}


def _inputs(case, seed):
    g = _generator(seed)
    S = _states(case, g)
    steps = {"window": case["window"], "continuous": 16, "quantize": 0, "export": case["window"] // 2 + 1}[case["kind"]]
    return S, _tokens(case, steps, g) if steps else None


def _ending(case, t):
    """The requests whose window is ended after step t of the start-up of a continuous batch: they then sit evenly
    over all positions of the window."""
    return [b for b in range(case["batch"]) if b * case["window"] // case["batch"] == t]


# ------------------------------------------------------------------------------------------------------------ cases

def _dims(case):
    rule = B.LQ_RULE_GENERAL if case["rule"] == "general" else B.LQ_RULE_DELTA
    return B.make_dims(case["batch"], case["heads_v"], case["heads_k"], window=case["window"], n_comp=case["n_comp"],
                       power_iters=SWEEPS, gate=B.LQ_GATE_DIAG if case["gate"] == "diag" else B.LQ_GATE_SCALAR,
                       code=CODES[case["code"]], rule=rule)


def _step(s, t, fused=False):
    x, d, st = s["tokens"], s["dims"], s["st"]
    if s["case"]["rule"] == "general":
        B.leapquant_decode_step_general(d, st, x["q"][t], x["k"][t], x["b"][t], x["v"][t], x["alpha"][t], x["beta"][t],
                                        s["o"][t])
    else:
        f = B.leapquant_decode_step_commit if fused else B.leapquant_decode_step
        f(d, st, x["q"][t], x["k"][t], x["v"][t], x["alpha"][t], x["beta"][t], s["o"][t])


def _window(s):
    for t in range(s["case"]["window"]):
        _step(s, t)
    B.leapquant_window_commit(s["dims"], s["st"])


def prepare(case, seed):
    S, tokens = _inputs(case, seed)
    dims = _dims(case)
    s = {"case": case, "dims": dims, "st": B.State.empty(dims), "tokens": tokens, "S": S}
    if tokens is not None:
        s["o"] = torch.empty((tokens["v"].shape[0], case["batch"], case["heads_v"], D), device="cuda")
    if case["kind"] == "quantize":
        return s
    B.leapquant_quantize_state(dims, S, s["st"])
    if case["kind"] != "export":
        s["S"] = None
    if case["kind"] == "export":
        for t in range(tokens["v"].shape[0]):
            _step(s, t)
    if case["kind"] == "continuous":
        mask = torch.zeros((case["window"], case["batch"]), dtype=torch.int32)
        for t in range(case["window"]):
            mask[t, _ending(case, t)] = 1
        mask = mask.cuda()
        for t in range(case["window"] - 1):
            _step(s, t % 16)
            B.leapquant_window_commit(dims, s["st"], mask[t])
        s["t"] = (case["window"] - 1) % 16
    if case["graph"]:
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            _window(s)
    return s


def run(s):
    st, kind = s["st"], s["case"]["kind"]
    rep = {"codes": st.codes, "scale": st.scale, "smooth": st.smooth, "comp_k": st.comp_k, "comp_u": st.comp_u}
    if kind == "quantize":
        B.leapquant_quantize_state(s["dims"], s["S"], st)
        return rep
    if kind == "export":
        B.leapquant_dequantize_state(s["dims"], st, s["S"])
        return s["S"]
    records = {"rec_k": st.rec_k, "rec_u": st.rec_u, "rec_a": st.rec_a, "rec_len": st.rec_len}
    if kind == "continuous":
        t = s["t"]
        s["t"] = (t + 1) % 16
        _step(s, t, fused=True)
        return {"o": s["o"][t], "rep": rep, "records": records}
    if "graph" in s:
        s["graph"].replay()
    else:
        _window(s)
    return {"o": s["o"], "rep": rep, "records": records}


def work(case):
    tiles, w, r = case["batch"] * case["heads_v"], case["window"], case["n_comp"]
    g = D if case["gate"] == "diag" else 1
    rep = D * D * BITS[case["code"]] // 8 + 8 * D + 4 * r * D
    rec = 4 * D + 2 * g
    # per value head and step: q and k of its share of a key head, v, decay, beta (and b), the output, rec_len
    token = (8 * D * case["heads_k"] / case["heads_v"] + 4 * D + 4 * g + 4
             + (4 * D if case["rule"] == "general" else 0) + 4 * D + 8)
    fit = r * (SWEEPS * 4 * D * D + 6 * D * D) + 6 * D * D
    decode = lambda i: 4 * D * D + (r + i) * 8 * D                                    # noqa: E731
    rebuild = lambda p: 2 * D * D * (r + p + 1)                                       # noqa: E731
    if case["kind"] == "quantize":
        return {"bytes": tiles * (4 * D * D + rep), "flops": tiles * fit}
    if case["kind"] == "export":
        p = w // 2 + 1
        return {"bytes": tiles * (rep + p * rec + 4 * D * D), "flops": tiles * rebuild(p)}
    read = rep * w + rec * w * (w + 1) // 2 + token * w                               # the window's decode steps
    commit = 2 * rep + w * rec
    flops = sum(decode(i) for i in range(w)) + rebuild(w) + fit
    share = w if case["kind"] == "continuous" else 1                                  # one step of w
    return {"bytes": tiles * (read + commit) / share, "flops": tiles * flops / share}


def tolerance(case):
    # fp32 outputs from sums in fp32 (1.1e-7 to 3.3e-7 from exact(), the exported states 2.5e-8); the records, tokens
    # and codes are rounded from sums in fp64, where another order moves a value across a rounding boundary about once
    # in 1e10: they equal exact()'s
    return {"rel": 1e-7 if case["kind"] == "export" else 1.5e-6, "differ": 1e-5}


# ------------------------------------------------------------------------------------- the same results in 64 bits

def _f16(x):
    return x.float().half().double()


def _dot(x, M):
    """x^T M per tile: [n][a], [n][a][b] -> [n][b]."""
    return (M * x[:, :, None]).sum(1)


def _mul(M, y):
    """M y per tile: [n][a][b], [n][b] -> [n][a]."""
    return (M * y[:, None, :]).sum(2)


def _quantized(case, M):
    """Refit, smoothing and codes of the states M [n][d_k][d_v] (fp64): the state that the representation stands for,
    and the representation.  The codes are decided in fp32, as the method's."""
    M = M.clone()
    base = torch.zeros_like(M)
    ks, us = [], []
    for _ in range(case["n_comp"]):
        x = M.square().sum(2).sqrt()
        for sweep in range(SWEEPS + 1):
            n = x.norm(dim=1, keepdim=True)
            x = torch.where(n > 0, x / n, torch.zeros_like(x))
            if sweep < SWEEPS:
                x = _mul(M, _dot(x, M))
        k = _f16(x)
        u = _f16(_dot(k, M))
        pair = k[:, :, None] * u[:, None, :]
        M -= pair
        base += pair
        ks.append(k)
        us.append(u)
    c = M.abs().mean(2).clamp(min=float(torch.tensor(1e-12, dtype=torch.float32))).sqrt().float()
    q = QMAX[case["code"]]
    R = M.float() * (torch.ones_like(c) / c)[:, :, None]
    a = R.abs().amax(1)
    qs = torch.full_like(a, q)          # (a tensor: torch divides by a plain number through its reciprocal)
    delta, inv = a / qs, torch.where(a > 0, qs / a, torch.zeros_like(a))
    Z = (R * inv[:, None, :]).clamp(-q, q) if case["code"] == "e4m3" else (R * inv[:, None, :]).round().clamp(-q, q)
    Z = Z.to(torch.float8_e4m3fn).double() if case["code"] == "e4m3" else Z.double()
    base += c.double()[:, :, None] * (Z * delta.double()[:, None, :])
    shape = (case["batch"], case["heads_v"], -1, D)
    rep = {"scale": delta, "smooth": c, "comp_k": torch.stack(ks, 1), "comp_u": torch.stack(us, 1)}
    return base, rep, shape


def _rep_out(case, rep, shape):
    b, h = shape[:2]
    return {"codes": None, "scale": rep["scale"].double().view(b, h, D), "smooth": rep["smooth"].double().view(b, h, D),
            "comp_k": rep["comp_k"].reshape(shape), "comp_u": rep["comp_u"].reshape(shape)}


def _exact_step(case, S, x, t):
    """One step of the recurrence with the method's FP16 records: state, output, record."""
    b, hv = case["batch"], case["heads_v"]
    n = b * hv

    def head(y):
        return y[t].repeat_interleave(hv // case["heads_k"], dim=1).reshape(n, D)

    q, k = head(x["q"]).double(), head(x["k"])
    v = x["v"][t].reshape(n, D).double()
    a = _f16(x["alpha"][t].reshape(n, -1))
    kt = _f16(x["beta"][t].reshape(n, 1) * k)
    A = S * a[:, :, None]
    read = _dot(x["b"][t].reshape(n, D).double(), S) if case["rule"] == "general" else _dot(k.double(), A)
    u = _f16(v - read)
    A += kt[:, :, None] * u[:, None, :]
    return A, _dot(q, A), kt, u, a


def exact(case, seed):
    S0, x = _inputs(case, seed)
    b, h, w = case["batch"], case["heads_v"], case["window"]
    n = b * h
    S, rep, shape = _quantized(case, S0.reshape(n, D, D).transpose(1, 2).double())
    if case["kind"] == "quantize":
        return _rep_out(case, rep, shape)
    if case["kind"] == "export":
        for t in range(w // 2 + 1):
            S = _exact_step(case, S, x, t)[0]
        return S.transpose(1, 2).reshape(b, h, D, D)
    g = D if case["gate"] == "diag" else 1
    rec = [torch.zeros((n, w, e), dtype=torch.float64, device="cuda") for e in (D, D, g)]
    at = torch.zeros(n, dtype=torch.long, device="cuda")
    every = torch.arange(n, device="cuda")

    def step(t):
        nonlocal S
        S, o, *new = _exact_step(case, S, x, t)
        for to, y in zip(rec, new):
            to[every, at] = y
        at.add_(1)
        return o

    def commit(tiles):
        if len(tiles):
            S[tiles], part, _ = _quantized(case, S[tiles])
            for key, y in part.items():
                rep[key][tiles] = y
            at[tiles] = 0

    if case["kind"] == "window":
        o = torch.stack([step(t) for t in range(w)]).view(w, b, h, D)
        commit(every)
    else:
        tiles_of = lambda bs: torch.tensor([i * h + j for i in bs for j in range(h)], dtype=torch.long, device="cuda")  # noqa: E731
        for t in range(w - 1):
            step(t % 16)
            commit(tiles_of(_ending(case, t)))
        o = step((w - 1) % 16).view(b, h, D)
        commit((at == w).nonzero()[:, 0])
    rk, ru, ra = rec
    ra = ra.view(b, h, w, g)
    return {"o": o, "rep": _rep_out(case, rep, shape),
            "records": {"rec_k": rk.view(b, h, w, D), "rec_u": ru.view(b, h, w, D), "rec_a": ra, "rec_len": None}}
