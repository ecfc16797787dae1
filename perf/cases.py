"""Performance cases of the MoE-decode hot path on one MI355X.

Each case is work that a program using this library has it do through the entry points of
``paper_2608_11688_amd.native`` (routers, expert FFN, decode attention) or through the
decode runner (whole decode steps).  A pass of the single-stage cases takes one token (or
one batch of tokens) through that stage of several layers, each with weights, caches and
inputs of its own, as a decode does: the weights of a layer have then left the caches
before the next token comes to it.

Sizes are those of the workload table in ``paper_2608_11688_amd.configs``; ``draw`` spreads
batch, widths, expert counts, formats, contexts and policies over the ranges between and
around them, sizes that fill no tile among them.
"""
import dataclasses
import math

import torch

from paper_2608_11688_amd import configs, inputs, native
from paper_2608_11688_amd.runtime import DecodeRunner

DEV = "cuda"


# ------------------------------------------------------------------------------ cases
def _route(name, cfg, B, layers, policy=native.SEL_CUMPROB, mode=native.MODE_EXACT):
    return dict(name=name, kind="route", B=B, d=cfg.d, E=cfg.E, k=cfg.k, k_max=cfg.k_max,
                layers=layers, policy=policy, mode=mode, tau=cfg.tau, bias=cfg.bias_skew)


def _ffn(name, cfg, B, layers, weights):
    return dict(name=name, kind="ffn", B=B, d=cfg.d, E=cfg.E, k=cfg.k, I=cfg.I, C=cfg.C,
                layers=layers, weights=weights, bias=cfg.bias_skew)


def _attn(name, cfg, B, layers, ctx_max, pos):
    return dict(name=name, kind="attn", B=B, d=cfg.d, H=cfg.n_heads, G=cfg.n_kv_heads,
                hd=cfg.head_dim, ctx_max=ctx_max, pos=pos, layers=layers)


def _decode(name, cfg, B, layers, steps, C, ctx, mode=native.MODE_EXACT, weights="bf16"):
    return dict(name=name, kind="decode", model=cfg.name, B=B, layers=layers, steps=steps, C=C,
                ctx=ctx, mode=mode, weights=weights)


def listed():
    c = configs
    return [
        # prefetch router and gate of a 64-sequence batch: the two small kernels between
        # attention and experts, many experts, Zipf-like load
        _route("route_olmoe_b64", c.OLMOE, 64, 16),
        # single-user decode, small experts: every launch counts
        _ffn("ffn_granite1b_b1", c.GRANITE_1B, 1, 24, "bf16"),
        # single-user decode, the largest experts: the weight stream
        _ffn("ffn_mixtral_b1", c.MIXTRAL, 1, 2, "bf16"),
        # single-user decode with 4-bit experts, wide and shallow (I = 832)
        _ffn("ffn_phi7b_b1_mxfp4", c.PHI_7B, 1, 32, "mxfp4"),
        # a few users: two or three tokens per expert
        _ffn("ffn_granite3b_b8", c.GRANITE_3B, 8, 16, "bf16"),
        # many users, many experts: about 21 tokens per resident expert
        _ffn("ffn_olmoe_b64", c.OLMOE, 64, 4, "bf16"),
        # 4-bit experts in a batch, I = 1472 (no whole number of row tiles)
        _ffn("ffn_deepseek_b16_mxfp4", c.DEEPSEEK_16B, 16, 8, "mxfp4"),
        # 8-bit experts in a batch, long rows
        _ffn("ffn_mixtral_b32_fp8", c.MIXTRAL, 32, 2, "fp8"),
        # decode attention of one user, 1024 positions: small and latency-bound
        _attn("attn_granite1b_b1", c.GRANITE_1B, 1, 24, 1025, 1024),
        # decode attention of a batch, grouped heads of 128, a context between powers of two
        _attn("attn_mixtral_b32", c.MIXTRAL, 32, 2, 2048, 1999),
        # whole decode steps with every expert in HBM (the host never waits for a router)
        _decode("decode_granite1b_resident", c.GRANITE_1B, 1, 8, 4, 32, 1024),
        # whole decode steps with experts offloaded to host memory: prefetch, copies over
        # the host link, miss correction
        _decode("decode_granite3b_offload", c.GRANITE_3B, 1, 4, 4, 16, 1024),
    ]


def _log_int(rng, lo, hi, mult=1):
    """A multiple of mult, its logarithm spread evenly over [lo, hi]."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(mult, int(round(v / mult)) * mult)


MAX_BYTES = 1.4e9      # a drawn pass moves no more than the largest listed ones
MAX_POOL = 6e9         # slot pools or caches of one state
FORMAT_MULT = {"bf16": 8, "fp8": 16, "mxfp4": 32, "fp32": 4}
FORMAT_BYTES = {"bf16": 2.0, "fp8": 1.0, "mxfp4": 0.53125, "fp32": 4.0}


def draw(rng):
    kind = rng.choice(["route", "ffn", "ffn", "ffn", "ffn", "attn", "attn", "decode"])
    if kind == "decode":
        resident = rng.random() < 0.5
        cfg = rng.choice([configs.GRANITE_1B, configs.GRANITE_3B, configs.TINY])
        B = 1 if cfg is configs.TINY else rng.choice([1, 1, 2, 4])
        return dict(kind="decode", model=cfg.name, B=B, layers=min(cfg.L, rng.randint(2, 4)),
                    steps=rng.randint(2, 4), C=cfg.E if resident else cfg.C,
                    ctx=_log_int(rng, 32, 2048),
                    mode=rng.choice([native.MODE_EXACT, native.MODE_STALL_FREE])
                    if resident else native.MODE_EXACT,
                    weights=rng.choice(["bf16", "fp8"]))
    if kind == "route":
        E = rng.randint(4, 64)
        k = rng.randint(1, min(8, E))
        c = dict(kind="route", B=_log_int(rng, 1, 64), d=_log_int(rng, 256, 4096, 8), E=E, k=k,
                 k_max=rng.randint(k, min(E, 2 * k + 2)), layers=rng.randint(2, 16),
                 policy=rng.choice([native.SEL_CUMPROB, native.SEL_ORDINAL_CDF,
                                    native.SEL_STATIC]),
                 mode=rng.choice([native.MODE_EXACT, native.MODE_STALL_FREE]),
                 tau=rng.choice([0.8, 0.9, 0.95]), bias=rng.random() < 0.5)
        return c
    if kind == "attn":
        hd = rng.choice([64, 128])
        gr = rng.choice([1, 2, 3, 4, 8])
        G = rng.randint(1, max(1, 32 // gr))
        B = _log_int(rng, 1, 64)
        c = dict(kind="attn", B=B, d=_log_int(rng, 256, 4096, 8), H=G * gr, G=G, hd=hd, ctx_max=0,
                 pos=_log_int(rng, 16, 4096), layers=rng.randint(2, 8))
        c["ctx_max"] = c["pos"] + 1 + rng.randint(0, 64)
        while _attn_bytes(c) * c["layers"] > MAX_BYTES / 2 and c["layers"] > 1:
            c["layers"] -= 1
        while _attn_bytes(c) > MAX_BYTES / 2:
            c["pos"] //= 2
            c["ctx_max"] = c["pos"] + 17
        return c
    weights = rng.choice(["bf16", "bf16", "fp8", "mxfp4", "fp32"])
    mult = FORMAT_MULT[weights]
    E = rng.choice([4, 8, 16, 32, 40, 64, rng.randint(4, 64)])
    k = rng.randint(1, min(8, E))
    C = rng.randint(k, E)
    B = 1 if weights == "fp32" or rng.random() < 0.4 else _log_int(rng, 2, 64)
    c = dict(kind="ffn", B=B, d=_log_int(rng, 256, 4096, mult), E=E, k=k,
             I=_log_int(rng, 256, 14336, mult), C=C, layers=rng.randint(1, 16), weights=weights,
             bias=rng.random() < 0.5)
    per = lambda: 3 * c["d"] * c["I"] * FORMAT_BYTES[weights]
    while _distinct(c) * per() > MAX_BYTES or c["C"] * per() > MAX_POOL:
        c["I"] = max(mult, c["I"] // 2 // mult * mult)
    while c["layers"] > 1 and (c["layers"] * _distinct(c) * per() > MAX_BYTES
                               or c["layers"] * c["C"] * per() > MAX_POOL):
        c["layers"] -= 1
    return c


# ----------------------------------------------------------------------------- inputs
def _gen(seed, *more):
    g = torch.Generator(device=DEV)
    s = int(seed) & 0xFFFFFFFF
    for m in more:
        s = (s * 1000003 + int(m) + 12345) & 0x7FFFFFFFFFFF
    g.manual_seed(s)
    return g


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)


def _router(g, E, d):
    """A router matrix with logits of standard deviation 2 on the states below (bf16)."""
    return (_randn(g, E, d) * inputs.router_scale(d) * inputs.W_STD).to(torch.bfloat16)


def _quant_fp8(w):
    """(E4M3 codes, row scales): s_r = fp32(max |row| / 448), codes rounded to nearest even."""
    s = w.abs().amax(-1) / 448.0
    q = (w / s.clamp_min(1e-30).unsqueeze(-1)).to(torch.float8_e4m3fn)
    return q.view(torch.uint8), s


E2M1 = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)


def _quant_mxfp4(w):
    """(E2M1 codes two per byte, block scale bytes) of rows of blocks of 32."""
    R, K = w.shape
    blk = w.view(R, K // 32, 32)
    big = blk.abs().amax(-1)
    _, ex = torch.frexp(big)
    X = torch.where(big > 0, ex - 1 - 2, torch.full_like(ex, -127))
    v = torch.ldexp(blk, -X.unsqueeze(-1).float()).abs()
    # E2M1 steps: 0.5 up to 2, 1 up to 4, 2 beyond; round() takes ties to even steps
    low = torch.round(v * 2)
    mid = torch.round(v) + 2
    high = torch.round(v / 2) + 4
    code = torch.where(v <= 2, low, torch.where(v <= 4, mid, high)).clamp_max(7)
    code = code.to(torch.uint8) | (torch.signbit(blk).to(torch.uint8) << 3)
    code = code.view(R, K)
    return code[:, 0::2] | (code[:, 1::2] << 4), (X + 127).to(torch.uint8)


def _expert(g, d, I, weights):
    """One packed expert (uint8), in the layout that the pack entry points of this format
    write; drawn and packed on the device, where the host packers would take minutes."""
    w13 = (_randn(g, I, 2, d) * inputs.W_STD).to(torch.bfloat16)
    w2 = (_randn(g, d, I) * inputs.W_STD).to(torch.bfloat16)
    if weights == "bf16":
        parts = [w13, w2]
    elif weights == "fp32":
        parts = [w13.float(), w2.float()]
    elif weights == "fp8":
        q13, s13 = _quant_fp8(w13.float())
        q2, s2 = _quant_fp8(w2.float())
        parts = [q13, q2, s13[:, 0].contiguous(), s13[:, 1].contiguous(), s2]
    else:
        q13, x13 = _quant_mxfp4(w13.float().view(2 * I, d))
        q2, x2 = _quant_mxfp4(w2.float())
        x13 = x13.view(I, 2, d // 32)
        parts = [q13, q2, x13[:, 0].contiguous(), x13[:, 1].contiguous(), x2]
    return torch.cat([p.contiguous().view(-1).view(torch.uint8) for p in parts])


def _unpacked(buf, d, I, weights):
    """(W1, W3 [I, d], W2 [d, I]) in float64 of one packed expert."""
    n = 3 * d * I
    if weights in ("bf16", "fp32"):
        w = buf.view(torch.bfloat16 if weights == "bf16" else torch.float32).double()
        w13, w2 = w[:2 * I * d].view(I, 2, d), w[2 * I * d:].view(d, I)
        return w13[:, 0], w13[:, 1], w2
    if weights == "fp8":
        q = buf[:n].view(torch.float8_e4m3fn).double()
        s = buf[n:].view(torch.float32).double()
        w13 = q[:2 * I * d].view(I, 2, d)
        return (w13[:, 0] * s[:I, None], w13[:, 1] * s[I:2 * I, None],
                q[2 * I * d:].view(d, I) * s[2 * I:, None])
    table = torch.tensor(E2M1 + tuple(-v for v in E2M1), dtype=torch.float64, device=buf.device)
    c = buf[:n // 2]
    q = table[torch.stack([c & 15, c >> 4], -1).view(-1).long()]
    x = torch.exp2(buf[n // 2:].double() - 127)
    w13 = q[:2 * I * d].view(I, 2, d)
    nx = I * (d // 32)
    rep = lambda t, r: t.view(r, -1).repeat_interleave(32, 1)
    return (w13[:, 0] * rep(x[:nx], I), w13[:, 1] * rep(x[nx:2 * nx], I),
            q[2 * I * d:].view(d, I) * rep(x[2 * nx:], d))


def _states(g, B, d):
    """Hidden states before and after attention (unit variance, then some noise)."""
    pre = _randn(g, B, d)
    return pre, pre + inputs.POST_NOISE * _randn(g, B, d)


def _prepare_route(case, seed):
    c, layers = case, []
    B, d, E, k, L = c["B"], c["d"], c["E"], c["k"], c["layers"]
    i32 = dict(dtype=torch.int32, device=DEV)
    f32 = dict(dtype=torch.float32, device=DEV)
    out = dict(pf_idx=torch.empty(L, B, c["k_max"], **i32), pf_count=torch.empty(L, B, **i32),
               route_idx=torch.empty(L, B, k, **i32), route_gate=torch.empty(L, B, k, **f32),
               exec_idx=torch.empty(L, B, k, **i32), exec_gate=torch.empty(L, B, k, **f32))
    for l in range(L):
        g = _gen(seed, 1, l)
        pre, post = _states(g, B, d)
        wg = _router(g, E, d)
        wpf = (wg.float() + inputs.PF_NOISE * _router(g, E, d).float()).to(torch.bfloat16)
        layers.append(dict(
            pre=pre, post=post, wg=wg, wpf=wpf, bias=_randn(g, E) if c["bias"] else None,
            avail=(torch.rand(E, generator=g, device=DEV) < 0.7).to(torch.uint8),
            cdf_w=_randn(g, E), cdf_theta=torch.sort(_randn(g, E - k + 1) * 2 + 1).values,
            **{n: t[l] for n, t in out.items()}))
    return dict(case=c, layers=layers, out=out)


def _prepare_ffn(case, seed):
    c, layers = case, []
    B, d, E, k, I, C = (c[n] for n in ("B", "d", "E", "k", "I", "C"))
    _, nbytes, _, ffn = native.weight_format(c["weights"])
    S = nbytes(d, I)
    y = torch.empty(c["layers"], B, d, device=DEV)
    for l in range(c["layers"]):
        g = _gen(seed, 2, l)
        resident = torch.randperm(E, generator=g, device=DEV)[:C]
        table = torch.full((E,), -1, dtype=torch.int32, device=DEV)
        table[resident] = torch.arange(C, dtype=torch.int32, device=DEV)
        # every token runs the k best of the resident experts (stall-free decode)
        z = 2.0 * _randn(g, B, E) + (_randn(g, E) if c["bias"] else 0.0)
        z = z.masked_fill(table < 0, -1e30)
        top = torch.topk(z, k, dim=1)
        slots = torch.empty(C * S, dtype=torch.uint8, device=DEV)
        for s in range(C):
            slots[s * S:(s + 1) * S] = _expert(g, d, I, c["weights"])
        layers.append(dict(x=_states(g, B, d)[1], idx=top.indices.to(torch.int32).contiguous(),
                           gate=torch.softmax(top.values, 1).contiguous(), table=table,
                           slots=slots, y=y[l]))
    ws = native.apex_moe_ffn_workspace_bytes(B, d, I, k)
    return dict(case=c, layers=layers, out=y, ffn=ffn, ws_bytes=ws,
                ws=torch.empty(ws, dtype=torch.uint8, device=DEV))


def _prepare_attn(case, seed):
    c, layers = case, []
    B, d, H, G, hd, n, L = (c[m] for m in ("B", "d", "H", "G", "hd", "ctx_max", "layers"))
    bf16 = dict(dtype=torch.bfloat16, device=DEV)
    out = dict(o=torch.empty(L, B, d, device=DEV), k_cache=torch.empty(L, B, G, n, hd, **bf16),
               v_cache=torch.empty(L, B, G, n, hd, **bf16))
    for l in range(L):
        g = _gen(seed, 3, l)
        out["k_cache"][l] = _randn(g, B, G, n, hd)
        out["v_cache"][l] = _randn(g, B, G, n, hd)
        layers.append(dict(
            h=_states(g, B, d)[0],
            w_qkv=(_randn(g, (H + 2 * G) * hd, d) / math.sqrt(d)).to(torch.bfloat16),
            w_o=(_randn(g, d, H * hd) / math.sqrt(H * hd)).to(torch.bfloat16),
            **{m: t[l] for m, t in out.items()}))
    ws = native.apex_attention_workspace_bytes(B, H, G, hd, n)
    return dict(case=c, layers=layers, out=out, ws_bytes=ws,
                ws=torch.empty(ws, dtype=torch.uint8, device=DEV))


class _Runner(DecodeRunner):
    def __del__(self):
        try:
            self.close()
        except Exception:
            pass


def _prepare_decode(case, seed):
    cfg = dataclasses.replace(configs.get(case["model"]), C=case["C"])
    r = _Runner(cfg, batch=case["B"], mode=case["mode"], seed=seed, steps=case["steps"],
                layers=list(range(case["layers"])), weights=case["weights"], window="attention",
                ctx=case["ctx"])
    return dict(case=case, runner=r, cfg=cfg)


PREPARE = dict(route=_prepare_route, ffn=_prepare_ffn, attn=_prepare_attn, decode=_prepare_decode)


def prepare(case, seed):
    return PREPARE[case["kind"]](case, seed)


# -------------------------------------------------------------------------------- run
def run(state):
    c = state["case"]
    s = torch.cuda.current_stream().cuda_stream
    if c["kind"] == "route":
        for a in state["layers"]:
            native.apex_prefetch_route(
                a["pre"], a["wpf"], a["bias"], c["B"], c["d"], c["E"], c["k"], c["k_max"],
                c["policy"], c["tau"], 2, a["cdf_w"], a["cdf_theta"], a["pf_idx"],
                a["pf_count"], None, s)
            native.apex_gate_topk(
                a["post"], a["wg"], a["bias"], c["B"], c["d"], c["E"], c["k"], c["mode"],
                a["avail"], 0, a["route_idx"], a["route_gate"], a["exec_idx"], a["exec_gate"],
                None, s)
        return state["out"]
    if c["kind"] == "ffn":
        for a in state["layers"]:
            state["ffn"](a["x"], c["B"], c["d"], c["I"], c["E"], c["k"], a["idx"], a["gate"],
                         a["table"], a["slots"], c["C"], a["y"], 0, state["ws"],
                         state["ws_bytes"], s)
        return state["out"]
    if c["kind"] == "attn":
        for a in state["layers"]:
            native.apex_attention_decode(
                a["h"], a["w_qkv"], a["w_o"], c["B"], c["d"], c["H"], c["G"], c["hd"],
                a["k_cache"], a["v_cache"], c["ctx_max"], c["pos"], a["o"], state["ws"],
                state["ws_bytes"], s)
        return state["out"]
    r = state["runner"]
    r.t = 0      # the same tokens again; the expert caches stay as the last pass left them
    out = []
    for _ in range(c["steps"]):
        r.step()
        out.append(r.y.clone())
    return out


# ------------------------------------------------------------------------------- work
def _distinct(c):
    """Experts that B tokens with k of C resident experts each run, on average."""
    return c["C"] * (1.0 - (1.0 - c["k"] / c["C"]) ** c["B"])


def _attn_bytes(c):
    rows = (c["H"] + 2 * c["G"]) * c["hd"]
    return (2 * rows * c["d"] + 2 * c["d"] * c["H"] * c["hd"] + 8 * c["B"] * c["d"]
            + 4 * c["B"] * c["G"] * (c["pos"] + 1) * c["hd"])


def _attn_flops(c):
    rows = (c["H"] + 2 * c["G"]) * c["hd"]
    return 2.0 * c["B"] * (rows * c["d"] + c["d"] * c["H"] * c["hd"]
                           + 2 * c["H"] * (c["pos"] + 1) * c["hd"])


def work(case):
    c = case
    if c["kind"] == "route":
        one = 2 * (2 * c["E"] * c["d"] + 4 * c["B"] * c["d"] + 8 * c["B"] * (c["k_max"] + c["k"]))
        return dict(bytes=c["layers"] * one, flops=c["layers"] * 4.0 * c["B"] * c["E"] * c["d"])
    if c["kind"] == "ffn":
        per = 3 * c["d"] * c["I"]
        one = _distinct(c) * per * FORMAT_BYTES[c["weights"]] + 8 * c["B"] * c["d"]
        return dict(bytes=c["layers"] * one, flops=c["layers"] * 2.0 * c["B"] * c["k"] * per)
    if c["kind"] == "attn":
        return dict(bytes=c["layers"] * _attn_bytes(c), flops=c["layers"] * _attn_flops(c))
    cfg = configs.get(c["model"])
    a = dict(B=c["B"], d=cfg.d, H=cfg.n_heads, G=cfg.n_kv_heads, hd=cfg.head_dim, pos=c["ctx"])
    f = dict(C=cfg.E, k=cfg.k, B=c["B"])
    per = 3 * cfg.d * cfg.I
    one = _attn_bytes(a) + _distinct(f) * per * FORMAT_BYTES[c["weights"]] + 4 * cfg.E * cfg.d
    ops = _attn_flops(a) + 2.0 * c["B"] * cfg.k * per + 4.0 * c["B"] * cfg.E * cfg.d
    n = c["layers"] * c["steps"]
    return dict(bytes=n * one, flops=n * ops)


# -------------------------------------------------------------------- the exact outputs
def _exact_ffn(x, idx, gate, expert):
    """sum over positions of gate * W2 (silu(W1 x) * (W3 x)) in float64; expert(e) gives
    the unpacked weights of expert e."""
    x, gate, idx = x.double(), gate.double(), idx.long()
    y = torch.zeros_like(x)
    for e in torch.unique(idx).tolist():
        rows, pos = torch.nonzero(idx == e, as_tuple=True)
        w1, w3, w2 = expert(e)
        u, v = x[rows] @ w1.T, x[rows] @ w3.T
        y.index_add_(0, rows, gate[rows, pos].unsqueeze(1) * ((u * torch.sigmoid(u) * v) @ w2.T))
    return y


def _top(alpha, k):
    v, i = torch.sort(alpha, dim=1, descending=True, stable=True)
    return i[:, :k], v[:, :k] / v[:, :k].sum(1, keepdim=True)


def _exact_route(a, c):
    z = a["post"].double() @ a["wg"].double().T
    if a["bias"] is not None:
        z = z + a["bias"].double()
    alpha = torch.softmax(z, 1)
    route = _top(alpha, c["k"])[1]
    if c["mode"] == native.MODE_EXACT:
        return route, route
    ex = _top(alpha.masked_fill(a["avail"] == 0, 0.0), c["k"])[1]
    return route, torch.nan_to_num(ex)


def _exact_attn(a, c):
    B, H, G, hd, pos = c["B"], c["H"], c["G"], c["hd"], c["pos"]
    qkv = a["h"].double() @ a["w_qkv"].double().T
    q, k, v = qkv.split([H * hd, G * hd, G * hd], 1)
    kc, vc = a["k_cache"].double(), a["v_cache"].double()
    kc[:, :, pos], vc[:, :, pos] = k.view(B, G, hd), v.view(B, G, hd)
    o = torch.empty(B, H * hd, dtype=torch.float64, device=DEV)
    for b in range(B):   # the new key and value are attended to as the caches hold them
        kb, vb = kc[b, :, :pos + 1].clone(), vc[b, :, :pos + 1].clone()
        kb[:, pos] = kb[:, pos].to(torch.bfloat16).double()
        vb[:, pos] = vb[:, pos].to(torch.bfloat16).double()
        p = torch.softmax(q[b].view(G, H // G, hd) @ kb.transpose(1, 2) / math.sqrt(hd), -1)
        o[b] = (p @ vb).reshape(-1)
    return o @ a["w_o"].double().T, kc, vc


def _exact_decode(st):
    c, cfg, r = st["case"], st["cfg"], st["runner"]
    S, d, I = r.S, cfg.d, cfg.I
    out = [torch.empty(c["layers"], c["B"], d, dtype=torch.float64, device=DEV)
           for _ in range(c["steps"])]
    for l in range(c["layers"]):
        b = r.bufs[l]
        host = b["host"].view(torch.uint8)
        for t in range(c["steps"]):
            x = b["h_post"][t].view(c["B"], d)
            z = x.double() @ b["wg"].view(torch.bfloat16).double().T
            if b["bias"] is not None:
                z = z + b["bias"].double()
            idx, gate = _top(torch.softmax(z, 1), cfg.k)
            out[t][l] = _exact_ffn(x, idx, gate, lambda e: _unpacked(
                host[e * S:(e + 1) * S].to(DEV), d, I, c["weights"]))
    return out


def exact(case, seed):
    """What run() returns, in float64 by plain torch on the same inputs."""
    c, st = case, prepare(case, seed)
    if c["kind"] == "route":
        each = [_exact_route(a, c) for a in st["layers"]]
        return dict(pf_idx=None, pf_count=None, route_idx=None, exec_idx=None,
                    route_gate=torch.stack([e[0] for e in each]),
                    exec_gate=torch.stack([e[1] for e in each]))
    if c["kind"] == "ffn":
        _, nbytes, _, _ = native.weight_format(c["weights"])
        S = nbytes(c["d"], c["I"])
        y = []
        for a in st["layers"]:
            slot = a["table"].tolist()
            y.append(_exact_ffn(a["x"], a["idx"], a["gate"], lambda e: _unpacked(
                a["slots"][slot[e] * S:(slot[e] + 1) * S], c["d"], c["I"], c["weights"])))
        return torch.stack(y)
    if c["kind"] == "attn":
        each = [_exact_attn(a, c) for a in st["layers"]]
        return dict(o=torch.stack([e[0] for e in each]),
                    k_cache=torch.stack([e[1] for e in each]),
                    v_cache=torch.stack([e[2] for e in each]))
    return _exact_decode(st)


def tolerance(case):
    c = case
    if c["kind"] == "route":
        # 32-bit sums; whole values differ where two logits tie within their rounding
        return dict(rel=2e-5, max=1e-2, differ=2e-3)
    if c["kind"] == "attn":
        # 32-bit sums over bf16 weights and caches; a new key or value may round to the
        # other neighbouring bf16 value
        return dict(rel=2e-4, max=2e-2)
    if c["B"] == 1:
        return dict(rel=4e-6, max=1e-4)      # activations stay in 32 bits
    return dict(rel=1e-2, max=8e-2)          # activations rounded to bf16
