"""The performance cases of this repository: what a program does with it, through its entry points.

Four kinds of work: the INT8 SSD layer over a prompt (`prefill`), one token of every sequence on
the persistent int8 state (`decode`), the unquantized FP16 layer (`fp16`) and the static
calibration (`calibrate`).  `listed()` names the cases, `draw()` gives more of the same ranges.
`prepare()` makes what a program holds before the call (activations, parameters, static steps,
workspaces, a captured graph), `run()` is one pass, `exact()` the same pass in 64 bits in plain
torch.  Activations follow the recipe of the package's synthetic layers (normal values with fixed
outlier channels in x and outlier state dimensions in B and C), with outliers small enough that
no output leaves the fp16 range.
"""
import math

import torch

from paper_2608_21952_amd import ssdi8

P, N, Q = 64, 128, 256
LN16 = math.log(16.0)
SHIFT = 7
ETA = 0.15

_DEFAULTS = {
    "kind": "prefill", "B": 1, "L": 0, "H": 24, "G": 1, "dtype": "fp16",
    "a_lo": 0.0,            # A = -exp(U(a_lo, ln 16)): 0 is fast decay, -4 mixes in slow heads
    "dt_mu": -2.0, "dt_sigma": 0.5,
    "xs_per_head": False,   # one X_scaled step per head instead of per channel
    "in_bmm": True,         # B, C handed over unquantized (else quantized first, as two calls)
    "resume": False,        # continue from an int8 state, with per-token steps of C
    "layers": 1,            # decode: layers of one token step; more than 1 is a captured graph
}


def _full(case):
    return {**_DEFAULTS, **case}


def listed():
    return [
        # A short prompt of a small model in fp32: the smallest layer call, where launches and
        # argument handling count.
        {"name": "prefill-tiny", "L": 512, "dtype": "fp32", "in_bmm": False},
        # Batched prefill of a 130M-shaped layer: the ordinary small call.
        {"name": "prefill-130m", "B": 8, "L": 2048},
        # Batched prefill of a 2.7B-shaped layer: the ordinary large call.
        {"name": "prefill-2.7b", "B": 4, "L": 4096, "H": 80},
        # Batched prefill of an 8B-shaped layer: eight groups of B and C, one step per head.
        {"name": "prefill-8b-g8", "B": 2, "L": 8192, "H": 128, "G": 8, "dt_mu": -3.0,
         "dt_sigma": 1.0, "xs_per_head": True},
        # One 64K-token context: the long chain of states, a third of the heads decaying slowly.
        {"name": "prefill-64k", "B": 1, "L": 65536, "H": 80, "a_lo": -4.0},
        # A single prompt on a small model: few sequences, slow heads among them.
        {"name": "prefill-one-prompt", "B": 1, "L": 8192, "H": 24, "a_lo": -4.0,
         "in_bmm": False},
        # The next piece of three conversations: an odd number of chunks and heads per group, an
        # initial int8 state, and C quantized per token.
        {"name": "prefill-resume", "B": 3, "L": 1280, "H": 40, "G": 5, "a_lo": -4.0,
         "resume": True, "in_bmm": False},
        # The SSD steps of one token through 24 layers at a small batch, as a captured graph:
        # the serving loop, bound by launches and latency.
        {"name": "decode-24-layers", "kind": "decode", "B": 8, "H": 24, "layers": 24},
        # One token of a large serving batch in one layer, bound by the states.
        {"name": "decode-large-batch", "kind": "decode", "B": 128, "H": 80},
        # The unquantized layer, small and large: what a program runs where it does not quantize.
        {"name": "fp16-130m", "kind": "fp16", "B": 8, "L": 2048},
        {"name": "fp16-2.7b", "kind": "fp16", "B": 4, "L": 4096, "H": 80, "a_lo": -4.0},
        # Static calibration of one layer from one draw.
        {"name": "calibrate-2.7b", "kind": "calibrate", "B": 4, "L": 2048, "H": 80,
         "a_lo": -4.0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["prefill"] * 7 + ["decode"] * 2 + ["fp16"] * 2 + ["calibrate"])
    G = rng.choice([1, 1, 1, 2, 3, 5, 8])
    H = max(1, _log_int(rng, 8, 128) // G) * G
    case = {"kind": kind, "H": H, "G": G, "dtype": rng.choice(["fp16", "fp16", "fp16", "fp32"]),
            "a_lo": rng.choice([0.0, -4.0])}
    if kind == "decode":
        if rng.random() < 0.5:
            case.update(B=_log_int(rng, 1, 16), layers=rng.choice([8, 16, 24, 48]))
        else:
            case.update(B=max(1, min(_log_int(rng, 8, 256), 10240 // H)))
        return case
    # token-heads up to the largest listed case of the kind (fp32 activations: half of that)
    most = {"prefill": 65536 * 80, "fp16": 4 * 4096 * 80, "calibrate": 4 * 2048 * 80}[kind]
    most //= 2 if case["dtype"] == "fp32" else 1
    chunks = min(_log_int(rng, 1, 256), max(1, most // (H * Q)))
    case.update(L=chunks * Q, B=min(_log_int(rng, 1, 8), max(1, most // (H * Q * chunks))))
    if kind == "prefill":
        case.update(in_bmm=rng.random() < 0.5, xs_per_head=rng.random() < 0.3)
        if rng.random() < 0.3:
            case.update(resume=True, in_bmm=False)
    return case


# ------------------------------------------------------------------------------ inputs
def _dtype(c):
    return torch.float16 if c["dtype"] == "fp16" else torch.float32


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _params(c, gen):
    """A, D, the mean correction and the fixed outlier factors of one layer."""
    H, G = c["H"], c["G"]
    rand = lambda *s: torch.rand(*s, generator=gen, device="cuda")
    randn = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    xs = torch.where(rand(H, P) < 0.02, 20.0, 1.0)
    bs, cs = (torch.where(rand(G, N) < 0.025, 6.0, 1.0) for _ in range(2))
    return {"A": -torch.exp(c["a_lo"] + (LN16 - c["a_lo"]) * rand(H)),
            "D": 1.0 + 0.1 * randn(H), "corr": 0.01 * randn(H, P), "fx": xs, "fb": bs, "fc": cs}


def _acts(c, p, gen, B, L):
    """x, dt (before the softplus), B and C of B sequences of L tokens."""
    H, G, dt = c["H"], c["G"], _dtype(c)
    randn = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    x = torch.empty(B, L, H, P, dtype=dt, device="cuda")
    for b in range(B):
        for l0 in range(0, L, 8192):   # bounds the fp32 temporaries
            x[b, l0:l0 + 8192] = randn(min(8192, L - l0), H, P).mul_(p["fx"])
    return (x, c["dt_mu"] + c["dt_sigma"] * randn(B, L, H),
            (randn(B, L, G, N) * p["fb"]).to(dt), (randn(B, L, G, N) * p["fc"]).to(dt))


def _steps(c, p, gen):
    """Static steps from a calibration draw of the same layer (absmax / 127 per granule), in 64
    bits and rounded once: what a program loads with its weights."""
    x, dt, Bt, Ct = _acts(c, p, gen, 1, min(max(c["L"], Q), 2048))
    return _calibrate64(c, p, x, dt, Bt, Ct)


def _step(amax):
    s = (amax / 127.0).float()
    return torch.where(s == 0, torch.ones_like(s), s)


def _chunks(t, lo, hi):
    """Chunks [lo, hi) of a (1-batch) (L, ...) tensor as (hi - lo, Q, ...)."""
    return t[lo * Q:hi * Q].reshape(hi - lo, Q, *t.shape[1:])


def _dt64(dt):
    """softplus with threshold 20, formed in 64 bits and held in 32."""
    d = dt.double()
    return torch.where(d > 20.0, d, torch.log1p(torch.exp(d.clamp(max=20.0)))).float()


def _calibrate64(c, p, x, dt, Bt, Ct):
    H, G = c["H"], c["G"]
    B, L = x.shape[:2]
    xs = torch.zeros(H, P, dtype=torch.float64, device="cuda")
    sm = torch.zeros(H, P, dtype=torch.float64, device="cuda")
    cb = torch.zeros(G, dtype=torch.float64, device="cuda")
    tril = torch.ones(Q, Q, device="cuda").tril().bool()
    for b in range(B):
        run = torch.zeros(H, P, N, dtype=torch.float64, device="cuda")
        for k in range(L // Q):
            lut, cs = _lut(p, _chunks(dt[b], k, k + 1)[0])
            xl = lut[..., None] * _chunks(x[b], k, k + 1)[0].float()       # (Q, H, P) fp32
            xs = torch.maximum(xs, xl.abs().amax(0).double())
            Bk, Ck = (_chunks(t[b], k, k + 1)[0].double().permute(1, 0, 2).contiguous()
                      for t in (Bt, Ct))                                   # (G, Q, N)
            S = xl.double().permute(1, 2, 0).contiguous() @ _heads(Bk, H)  # (H, P, N)
            run = S + torch.exp(cs[-1])[:, None, None] * run
            sm = torch.maximum(sm, torch.maximum(S.abs(), run.abs()).amax(2))
            CB = Ck @ Bk.transpose(1, 2).contiguous()
            cb = torch.maximum(cb, (CB.abs() * tril).amax((1, 2)))
    am = lambda t: t.abs().amax((0, 1, 3)).double()
    return {"alpha_B": _step(am(Bt)), "alpha_C": _step(am(Ct)),
            "alpha_Xs": _step(xs.amax(1) if c["xs_per_head"] else xs), "alpha_S": _step(sm),
            "alpha_CB": _step(cb)}


def _heads(t, H):
    """(G, ...) -> (H, ...), head h reading group h // (H / G)."""
    return t.repeat_interleave(H // t.shape[0], 0)


def _lut(p, dt):
    """The decay table dt exp(cs_last - cs) of ChunkState (fp32) and cs (64 bits), both (Q, H)."""
    d = _dt64(dt)
    cs = torch.cumsum((d * p["A"]).double(), 0)
    return d * torch.exp(cs[-1:] - cs).float(), cs


def _inputs(c, seed):
    """Everything made from the seed; `prepare` and `exact` share it."""
    gen = _gen(seed)
    if c["kind"] == "decode":
        layers = []
        for _ in range(c["layers"]):
            p = _params(c, gen)
            steps = _steps(c, p, gen)
            x, dt, Bt, Ct = _acts(c, p, gen, c["B"], 1)
            st = torch.randn(c["B"], c["H"], P, N, generator=gen, device="cuda") * 30.0
            layers.append((p, steps, x[:, 0].contiguous(), dt[:, 0].contiguous(), Bt, Ct,
                           st.round_().clamp_(-127, 127).to(torch.int8)))
        return layers
    p = _params(c, gen)
    steps = _steps(c, p, gen) if c["kind"] == "prefill" else None
    acts = _acts(c, p, gen, c["B"], c["L"])
    init = None
    if c["resume"]:
        init = torch.randn(c["B"], c["H"], P, N, generator=gen, device="cuda") * 30.0
        init = init.round_().clamp_(-127, 127).to(torch.int8)
    return p, steps, acts, init


def prepare(case, seed):
    c = _full(case)
    made = _inputs(c, seed)
    if c["kind"] == "decode":
        return _prepare_decode(c, made)
    p, steps, (x, dt, Bt, Ct), init = made
    s = {"c": c, "p": p, "steps": steps, "x": x, "dt": dt, "B": Bt, "C": Ct, "init": init}
    d = ssdi8.dims(c["B"], c["L"], c["H"], c["G"])
    size = {"prefill": ssdi8.workspace_size, "fp16": ssdi8.fp16_workspace_size,
            "calibrate": ssdi8.calibrate_workspace_size}[c["kind"]](d)
    if c["kind"] == "prefill" and not c["resume"]:
        s["layer"] = ssdi8.SSDi8Layer(p["A"], p["D"], p["corr"], steps)
    else:
        s["workspace"] = torch.empty(size, dtype=torch.uint8, device="cuda")
    return s


def _prepare_decode(c, layers):
    B, H, G = c["B"], c["H"], c["G"]
    s = {"c": c, "layers": layers, "graph": None,
         "Bq": torch.empty(B, 1, G, N, dtype=torch.int8, device="cuda"),
         "Cq": torch.empty(B, 1, G, N, dtype=torch.int8, device="cuda"),
         "y": torch.empty(c["layers"], B, H, P, dtype=_dtype(c), device="cuda"),
         "state": torch.stack([l[6] for l in layers])}
    if c["layers"] > 1:
        start = s["state"].clone()
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            _decode_token(s)
        torch.cuda.current_stream().wait_stream(stream)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _decode_token(s)
        s["graph"] = graph
        s["state"].copy_(start)
    return s


# ------------------------------------------------------------------------------ one pass
def _decode_token(s):
    for i, (p, a, x, dt, Bt, Ct, _) in enumerate(s["layers"]):
        ssdi8.quantize_act(Bt, "group", a["alpha_B"], out=s["Bq"])
        ssdi8.quantize_act(Ct, "group", a["alpha_C"], out=s["Cq"])
        ssdi8.decode_step(x, dt, p["A"], s["Bq"][:, 0], s["Cq"][:, 0], a["alpha_B"],
                          a["alpha_C"], a["alpha_Xs"], a["alpha_S"], a["alpha_CB"],
                          s["state"][i], D=p["D"], corr=p["corr"], y=s["y"][i])


def run(s):
    c, p, a = s["c"], s.get("p"), s.get("steps")
    if c["kind"] == "decode":
        if s["graph"] is not None:
            s["graph"].replay()
        else:
            _decode_token(s)
        return {"y": s["y"], "state_q": s["state"]}
    x, dt, Bt, Ct = s["x"], s["dt"], s["B"], s["C"]
    if c["kind"] == "fp16":
        return ssdi8.ssd_chunk_scan_fp16(x, dt, p["A"], Bt, Ct, D=p["D"],
                                         workspace=s["workspace"])
    if c["kind"] == "calibrate":
        return ssdi8.calibrate(x, dt, p["A"], Bt, Ct, D=p["D"], xs_per_head=c["xs_per_head"],
                               eta=ETA, workspace=s["workspace"])
    if c["resume"]:
        Bq, _ = ssdi8.quantize_act(Bt, "group", a["alpha_B"])
        Cq, Cs = ssdi8.quantize_act(Ct, "token")
        return ssdi8.ssd_chunk_scan(x, dt, p["A"], Bq, Cq, a["alpha_B"], Cs.view(Ct.shape[:3]),
                                    a["alpha_Xs"], a["alpha_S"], a["alpha_CB"], D=p["D"],
                                    corr=p["corr"], init_state_q=s["init"],
                                    workspace=s["workspace"])
    # the hand-off count is read once per model pass, not after every layer
    out = s["layer"](x, dt, Bt, Ct, quantize_in_bmm=c["in_bmm"], check=False)
    return {k: out[k] for k in ("y", "final_state_q", "final_state")}


# ------------------------------------------------------------------------------ 64 bits
def _codes(v, step):
    """clamp(rne(fl32(v * fl32(1 / step))), +-127), the quantizer's definition."""
    return (v.float() * (1.0 / step)).round().clamp(-127, 127)


def _requant(i, m):
    return (i.float() * m.float()).round().clamp(-127, 127)


def _layer64(c, p, x, dt, Bt, Ct, a=None, corr=None, init=None, token_c=False):
    """y and the final state of the layer in 64 bits: quantized with steps `a`, or not (a None).
    The integer codes are those of the method; everything else is float64."""
    H, G = c["H"], c["G"]
    B, L = x.shape[:2]
    y = torch.empty(B, L, H, P, dtype=torch.float64, device="cuda")
    fin = torch.empty(B, H, P, N, dtype=torch.float64, device="cuda")
    tril = torch.ones(Q, Q, dtype=torch.float64, device="cuda").tril()
    for b in range(B):
        st = torch.zeros(H, P, N, dtype=torch.float64, device="cuda")
        if init is not None:
            st = init[b].double()
        for k in range(L // Q):
            xk = _chunks(x[b], k, k + 1)[0]
            lut, cs = _lut(p, _chunks(dt[b], k, k + 1)[0])
            d = _dt64(_chunks(dt[b], k, k + 1)[0]).double()
            Bk, Ck = (_chunks(t[b], k, k + 1)[0].permute(1, 0, 2).contiguous() for t in (Bt, Ct))
            E = torch.exp(cs).T                                            # (H, Q)
            if a is None:
                Xs = (d * torch.exp(cs[-1:] - cs))[..., None] * xk.double()
                Bk, Ck = Bk.double(), Ck.double()
                CB = Ck @ Bk.transpose(1, 2).contiguous()
                S = Xs.permute(1, 2, 0).contiguous() @ _heads(Bk, H)
                Y1 = _heads(Ck, H) @ st.transpose(1, 2).contiguous()       # (H, Q, P)
                off = Y1 * E[..., None]
                st = S + torch.exp(cs[-1])[:, None, None] * st
            else:
                aB, aXs, aS, aCB = (a[n] for n in ("alpha_B", "alpha_Xs", "alpha_S", "alpha_CB"))
                aXs = aXs[:, None].expand(H, P) if aXs.dim() == 1 else aXs
                if token_c:
                    aC = _step(Ck.abs().amax(2).double())                  # (G, Q)
                else:
                    aC = a["alpha_C"][:, None].expand(G, Q)
                Bq, Cq = _codes(Bk, aB[:, None, None]).double(), _codes(Ck, aC[..., None]).double()
                Xq = _codes(lut[..., None] * xk.float(), aXs).double()
                mS = (aXs.double() * _heads(aB, H)[:, None].double() / aS.double()).float()
                Sq = _requant(Xq.permute(1, 2, 0).contiguous() @ _heads(Bq, H), mS[..., None])
                mCB = (aC.double() * aB[:, None].double() / aCB[:, None].double()).float()
                CB = _requant(Cq @ Bq.transpose(1, 2).contiguous(), mCB[..., None]).double()
                CB = CB * aCB[:, None, None].double()
                Y1 = _heads(Cq, H) @ st.transpose(1, 2).contiguous()
                off = Y1 * (_heads(aC, H).double() * E)[..., None] * aS[:, None].double()
                qd = (torch.exp(cs[-1]) * (1 << SHIFT)).round()
                r = 1 << (SHIFT - 1)
                st = (Sq.double() + ((qd[:, None, None] * st + r) / (1 << SHIFT)).floor())
                st = st.clamp(-127, 127)
            seg = cs.T[:, :, None] - cs.T[:, None, :]                      # cs_j - cs_i
            W = _heads(CB, H) * d.T[:, None, :] * torch.exp(seg.clamp(max=0.0)) * tril
            yk = off + W @ xk.double().permute(1, 0, 2).contiguous()
            yk = yk.permute(1, 0, 2) + p["D"].double()[:, None] * xk.double()
            y[b, k * Q:(k + 1) * Q] = yk if corr is None else yk + corr.double()
        fin[b] = st
    if a is not None:
        fin = fin * a["alpha_S"].double()[..., None]
    return y, fin


def _decode64(c, p, a, x, dt, Bt, Ct, st):
    H = c["H"]
    x64, st64 = x.double(), st.double()
    d = _dt64(dt)
    dA = (d * p["A"]).double()
    Bq, Cq = (_codes(t[:, 0], a[n][:, None]).double().repeat_interleave(H // c["G"], 1)
              for t, n in ((Bt, "alpha_B"), (Ct, "alpha_C")))              # (B, H, N)
    aB, aC, aCB = (_heads(a[n], H).double() for n in ("alpha_B", "alpha_C", "alpha_CB"))
    aXs = a["alpha_Xs"]
    aXs = aXs[:, None].expand(H, P) if aXs.dim() == 1 else aXs
    Xq = _codes(d[..., None] * x.float(), aXs).double()
    mS = (aXs.double() * aB[:, None] / a["alpha_S"].double()).float()
    Sq = _requant(Xq[..., None] * Bq[:, :, None], mS[..., None]).double()
    qd = (torch.exp(dA) * (1 << SHIFT)).round()[..., None, None]
    new = (Sq + ((qd * st64 + (1 << (SHIFT - 1))) / (1 << SHIFT)).floor()).clamp(-127, 127)
    off = (st64 * Cq[:, :, None]).sum(3) * (aC * torch.exp(dA))[..., None] * a["alpha_S"].double()
    CB = _requant((Cq * Bq).sum(2), (aC * aB / aCB).float()).double() * aCB * d.double()
    y = off + CB[..., None] * x64 + p["D"].double()[:, None] * x64 + p["corr"].double()
    return y, new.to(torch.int8)


def exact(case, seed):
    c = _full(case)
    made = _inputs(c, seed)
    if c["kind"] == "decode":
        outs = [_decode64(c, *layer) for layer in made]
        return {"y": torch.stack([o[0] for o in outs]),
                "state_q": torch.stack([o[1] for o in outs])}
    p, steps, (x, dt, Bt, Ct), init = made
    if c["kind"] == "fp16":
        y, fin = _layer64(c, p, x, dt, Bt, Ct)
        return {"y": y, "final_state": fin}
    if c["kind"] == "calibrate":
        a = _calibrate64(c, p, x, dt, Bt, Ct)
        yf, _ = _layer64(c, p, x, dt, Bt, Ct)
        yq, _ = _layer64(c, p, x, dt, Bt, Ct, a)
        out = {k: v.double() for k, v in a.items()}
        out["corr"] = ETA * (yf - yq).mean((0, 1))
        return out
    y, fin = _layer64(c, p, x, dt, Bt, Ct, steps, p["corr"], init, c["resume"])
    return {"y": y, "final_state_q": None, "final_state": fin}


# ------------------------------------------------------------------------------ figures
def work(case):
    """Minimum bytes (inputs once, outputs once) and multiply-adds times two of one pass."""
    c = _full(case)
    B, L, H, G = c["B"], c["L"], c["H"], c["G"]
    s = 2 if c["dtype"] == "fp16" else 4
    params = 4 * (2 * H + 3 * H * P + 3 * G)
    if c["kind"] == "decode":
        per = B * H * (2 * P * N + 2 * P * s + 4) + 2 * B * G * N * s + params
        return {"bytes": c["layers"] * per, "flops": c["layers"] * B * H * 4 * P * N}
    acts = B * L * (H * P * s + 4 * H + 2 * G * N * s)
    layer = B * L * (H * (4 * P * N + P * (Q + 1)) + G * N * (Q + 1))
    if c["kind"] == "calibrate":
        return {"bytes": acts + 4 * (3 * H * P + 3 * G + 2 * H), "flops": 2 * layer}
    state = B * H * P * N
    if c["kind"] == "fp16":
        return {"bytes": acts + B * L * H * P * s + 4 * state + 8 * H, "flops": layer}
    return {"bytes": acts + B * L * H * P * s + (6 if c["resume"] else 5) * state + params,
            "flops": layer}


def tolerance(case):
    """About four times the error against `exact()` over listed and drawn cases.  Layers and decode
    steps showed 2.3e-4 to 3.1e-4 on y (fp16 weights of ChunkScan2 and, with fp16 outputs, the
    rounding of y itself) and at most 2.1e-4 on the states; integer outputs do not differ.
    Calibration: the steps showed up to 1.2e-4 (fp32 B and C are taken in fp16), the correction,
    a mean of small differences that one code of Y_q moves, 5e-3."""
    if _full(case)["kind"] == "calibrate":
        return {"rel": 1e-2, "max": 0.1}
    return {"rel": 1.2e-3, "max": 0.01}
