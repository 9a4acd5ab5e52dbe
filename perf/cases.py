"""Timing cases of the library's main path: what a program built on it calls, from one decoded token to a training step.

A case is a dict of plain values:
  kind    "fwd": one forward call that continues a sequence (state blob in, state blob out); with L <= 16 that is
                 decoding, with more tokens chunked prefill
          "layer": one forward call from the start of a sequence, gate mask returned
          "train": forward with checkpoints, then backward with every gradient; the lane constants are rebuilt in the
                 forward, as after an optimizer step
          "conv": the Temporal Syntax Cache alone on the magnitude stream, history in and out
  B, L, H, F, conv_k   batch rows, tokens of the call, heads, harmonics per head (J = H * F lanes), conv taps
  gate    "tau" (per-lane threshold) or "valve" (per-head logits);  ret: data-dependent retention
  hconv   the harmonic convolution fused behind the output;  amp: softplus amplitude
  bf16    activations in memory are bfloat16 (state, constants and parameter gradients stay fp32)
  concat  the two planes of the outputs and of their gradients share rows of 2 J elements

Inputs follow the repository's benchmark: activations and upstream gradients N(0, 1), taps N(0, 1/conv_k), retention
U[0.95, 0.9999] (streaming: U[0.999, 0.99999]), rotation angles 10000^(-2 j / J), valve logits N(-3.9, 3^2) (about half of
the valves shut), retention logits N(-2, 1.5^2) with a static bias that falls from +3 to 0 over the harmonics.
"""
import math

import torch

from paper_2604_04250_amd import binding as K

DEV = "cuda:0"
TAU, EPS = 0.1, 0.001
CONV_CLAMP, OUT_CLAMP, GRAD_CLAMP = 50.0, 100.0, 100.0
MOST_LANE_TOKENS = 8 * 8192 * 768       # token-lanes of the largest listed case


def _case(kind, B, L, H, F, conv_k, gate="tau", ret=False, hconv=False, amp=False, bf16=False, concat=False):
    return {"kind": kind, "B": B, "L": L, "H": H, "F": F, "conv_k": conv_k, "gate": gate, "ret": ret, "hconv": hconv,
            "amp": amp, "bf16": bf16, "concat": concat}


_PAPER = {"gate": "valve", "ret": True, "amp": True}      # the layer as the paper states it


def listed():
    """Twelve cases, smallest calls first."""
    return [
        # one token of one sequence: the step of an interactive decoder
        dict(_case("fwd", 1, 1, 12, 64, 4), name="decode 1 token"),
        # one token of each of 64 sequences: a batched decoder of the paper's layer in its network type
        dict(_case("fwd", 64, 1, 4, 64, 3, bf16=True, **_PAPER), name="decode 64 rows, paper, bf16"),
        # a short prompt of odd length through the paper's layer, ending in the harmonic convolution
        dict(_case("fwd", 1, 333, 4, 64, 3, hconv=True, **_PAPER), name="prompt 333, paper, hconv"),
        # one 4096-token chunk of a 2,000,000-token stream, state carried
        dict(_case("fwd", 1, 4096, 12, 64, 4), name="stream chunk 4096"),
        # the paper's chunked-prefill length at the paper's lane shape, bf16
        dict(_case("fwd", 1, 32768, 4, 64, 3, hconv=True, bf16=True, **_PAPER), name="prefill chunk 32768, paper, bf16"),
        # one layer's forward over a batch, gate mask kept (scoring, analysis)
        dict(_case("layer", 4, 2048, 12, 64, 4), name="layer forward"),
        # the conv front-end on its own, in front of a scan that takes its output
        dict(_case("conv", 4, 2048, 12, 64, 4), name="syntax conv alone"),
        # the paper's training micro-batch (7 rows of 1024 tokens) through the layer as the paper states it
        dict(_case("train", 7, 1024, 4, 64, 3, **_PAPER), name="train micro-batch, paper"),
        # odd sizes: heads of 24 harmonics, 120 lanes, 1777 tokens, two taps, planes joined in one row
        dict(_case("train", 3, 1777, 5, 24, 2, concat=True), name="train odd sizes"),
        # long rows of the paper's layer with the harmonic convolution, trained end to end
        dict(_case("train", 8, 8192, 4, 64, 3, hconv=True, **_PAPER), name="train paper layer, hconv"),
        # a wide layer with bfloat16 activations
        dict(_case("train", 2, 4096, 32, 128, 4, bf16=True), name="train wide, bf16"),
        # the headline training step
        dict(_case("train", 8, 8192, 12, 64, 4), name="train step"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the same ranges: every kind, mode and type, sizes spread over their logarithm."""
    kind = rng.choice(["fwd", "fwd", "fwd", "layer", "train", "train", "train", "conv"])
    conv_k = rng.choice([0, 1, 2, 3, 3, 4, 4]) if kind != "conv" else rng.choice([2, 3, 4])
    gate = rng.choice(["tau", "valve"])
    ret, hconv, amp = rng.random() < 0.5, rng.random() < 0.4, rng.random() < 0.5
    bf16, concat = rng.random() < 0.4, rng.random() < 0.3
    if kind == "conv":
        gate, ret, hconv, amp, bf16, concat = "tau", False, False, False, False, False
    if hconv and (gate == "valve" or ret):
        F = rng.choice([32, 64, 64, 128, 256])
    elif hconv:
        F = rng.choice([8, 16, 32, 64, 64, 128, 256])
    elif gate == "valve" or ret:
        F = rng.choice([16, 32, 64, 64, 96, 128])
    else:
        F = rng.choice([16, 24, 32, 40, 64, 64, 100, 128])
    H = _log_int(rng, 1, 32)
    while H * F > 4096:
        H = (H + 1) // 2
    J = H * F
    if kind == "fwd" and rng.random() < 0.4:
        L, B = _log_int(rng, 1, 16), _log_int(rng, 1, 256)
    else:
        L, B = _log_int(rng, 17, 32768), _log_int(rng, 1, 32)
    most = MOST_LANE_TOKENS if kind == "train" else MOST_LANE_TOKENS // 2
    while B * L * J > most:
        if B > 1:
            B = (B + 1) // 2
        else:
            L = L // 2 + 1
    return _case(kind, B, L, H, F, conv_k, gate, ret, hconv, amp, bf16, concat)


# --------------------------------------------------------------------------------------------------- the path
def _desc(c):
    J = c["H"] * c["F"]
    d = K.make_desc(c["B"], c["L"], c["H"], c["F"], conv_k=c["conv_k"], amp_mode=1 if c["amp"] else 0,
                    gate_tau=TAU if c["gate"] == "tau" else 0.0, conv_clamp=CONV_CLAMP, out_clamp=OUT_CLAMP,
                    grad_clamp=GRAD_CLAMP, gate_mode=1 if c["gate"] == "valve" else 0, valve_eps=EPS,
                    ret_mode=1 if c["ret"] else 0, hconv_k=3 if c["hconv"] else 0)
    if c["concat"]:
        d.out_stride_t, d.out_stride_b = 2 * J, c["L"] * 2 * J
    return d


def _inputs(c, seed):
    """Everything a call reads, from the seed alone."""
    B, L, H, F, Kc = c["B"], c["L"], c["H"], c["F"], c["conv_k"]
    J = H * F
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 1000003 + 4250)
    adt = torch.bfloat16 if c["bf16"] else torch.float32
    n = lambda *s: torch.randn(*s, generator=g, device=DEV)
    x = {"mag": n(B, L, J).to(adt), "ang": n(B, L, J).to(adt)}
    lo, hi = (0.999, 0.99999) if c["kind"] == "fwd" else (0.95, 0.9999)
    x["gamma"] = lo + (hi - lo) * torch.rand(J, generator=g, device=DEV)
    j = torch.arange(J, device=DEV, dtype=torch.float64)
    x["theta"] = torch.pow(torch.tensor(10000.0, device=DEV, dtype=torch.float64), -2.0 * j / J).float()
    x["cw"] = n(2, J, Kc) / math.sqrt(Kc) if Kc else None
    x["cb"] = 0.1 * n(2, J) if Kc else None
    x["valve"] = -3.9 + 3.0 * n(B, L, H) if c["gate"] == "valve" else None
    x["ret"] = -2.0 + 1.5 * n(B, L, H) if c["ret"] else None
    x["rb"] = torch.linspace(3.0, 0.0, F, device=DEV) if c["ret"] else None
    x["hw"] = n(2, H, 3) / math.sqrt(3.0) if c["hconv"] else None
    x["hb"] = 0.1 * n(2, H) if c["hconv"] else None
    halo = max(Kc - 1, 0)
    if c["kind"] == "fwd":
        x["state"] = torch.cat([n(B * 2 * J), n(B * halo * 2 * J)])
    if c["kind"] == "conv":
        x["hist"] = n(B, halo, J)
    if c["kind"] == "train":
        if c["concat"]:
            dz = n(B, L, 2 * J).to(adt)
            x["dz_re"], x["dz_im"] = dz[:, :, :J], dz[:, :, J:]
        else:
            x["dz_re"], x["dz_im"] = n(B, L, J).to(adt), n(B, L, J).to(adt)
    return x


def prepare(case, seed):
    """Inputs, output buffers, descriptor and workspace; where the lane constants do not change from call to call
    (every kind but "train") one call has already built them, as in a running program."""
    c = case
    B, L, H, F, Kc = c["B"], c["L"], c["H"], c["F"], c["conv_k"]
    J = H * F
    x = _inputs(c, seed)
    s = {"c": c, "x": x}
    adt = torch.bfloat16 if c["bf16"] else torch.float32
    e = lambda *shape, dt=torch.float32: torch.empty(*shape, device=DEV, dtype=dt)
    d = s["d"] = _desc(c)
    if c["kind"] == "conv":
        s["y"], s["hist_out"] = e(B, L, J), e(B, max(Kc - 1, 0), J)
        return s
    if c["concat"]:
        z = e(B, L, 2 * J, dt=adt)
        s["z"] = (z[:, :, :J], z[:, :, J:])
    else:
        s["z"] = (e(B, L, J, dt=adt), e(B, L, J, dt=adt))
    s["ws"] = K.alloc_workspace(d, DEV)
    s["state_out"] = e(K.cawn_state_bytes(d) // 4) if c["kind"] == "fwd" else None
    s["mask"] = e(B, L, (J + 31) // 32, dt=torch.int32) if c["kind"] == "layer" else None
    if c["kind"] == "train":
        s["ckpt"] = e(K.cawn_ckpt_bytes(d) // 4)
        s["dmag"], s["dang"] = e(B, L, J, dt=adt), e(B, L, J, dt=adt)
        s["dgamma"] = None if c["ret"] else e(J)
        s["dtheta"] = e(J)
        s["dcw"], s["dcb"] = (e(2, J, Kc), e(2, J)) if Kc else (None, None)
        s["dvalve"] = e(B, L, H) if c["gate"] == "valve" else None
        s["dret"] = e(B, L, H) if c["ret"] else None
        s["dhw"], s["dhb"] = (e(2, H, 3), e(2, H)) if c["hconv"] else (None, None)
        s["db"] = _desc(c)
        s["db"].lane_consts_cached = 1
    else:
        _forward(s)
        d.lane_consts_cached = 1
    return s


def _forward(s):
    """The forward call through the entry point of its modes."""
    c, x, d, ws = s["c"], s["x"], s["d"], s["ws"]
    zr, zi = s["z"]
    st, so, ck, mk = x.get("state"), s["state_out"], s.get("ckpt"), s["mask"]
    gamma = None if c["ret"] else x["gamma"]
    if c["hconv"]:
        r = K.cawn_phase_accumulate_hconv_fwd(d, x["mag"], x["ang"], x["valve"], x["ret"], x["rb"], gamma, x["theta"],
                                              x["cw"], x["cb"], x["hw"], x["hb"], st, zr, zi, so, ck, mk, ws,
                                              1 if c["bf16"] else 0)
    elif c["bf16"]:
        r = K.cawn_phase_accumulate_bf16_fwd(d, x["mag"], x["ang"], x["valve"], x["ret"], x["rb"], gamma, x["theta"],
                                             x["cw"], x["cb"], st, zr, zi, so, ck, mk, ws)
    elif c["ret"]:
        r = K.cawn_phase_accumulate_ret_fwd(d, x["mag"], x["ang"], x["valve"], x["ret"], x["rb"], x["theta"], x["cw"],
                                            x["cb"], st, zr, zi, so, ck, mk, ws)
    elif c["gate"] == "valve":
        r = K.cawn_phase_accumulate_valve_fwd(d, x["mag"], x["ang"], x["valve"], gamma, x["theta"], x["cw"], x["cb"],
                                              st, zr, zi, so, ck, mk, ws)
    else:
        r = K.cawn_phase_accumulate_fwd(d, x["mag"], x["ang"], gamma, x["theta"], x["cw"], x["cb"], st, zr, zi, so, ck,
                                        mk, ws)
    K.check(r)


def _backward(s):
    """The backward call through the entry point of its modes."""
    c, x, d, ws = s["c"], s["x"], s["db"], s["ws"]
    gamma = None if c["ret"] else x["gamma"]
    if c["hconv"]:
        r = K.cawn_phase_accumulate_hconv_bwd(d, x["mag"], x["ang"], x["valve"], x["ret"], x["rb"], gamma, x["theta"],
                                              x["cw"], x["cb"], x["hw"], x["hb"], None, s["ckpt"], x["dz_re"], x["dz_im"],
                                              None, s["dmag"], s["dang"], s["dvalve"], s["dret"], s["dgamma"],
                                              s["dtheta"], s["dcw"], s["dcb"], s["dhw"], s["dhb"], None, ws,
                                              1 if c["bf16"] else 0)
    elif c["bf16"]:
        r = K.cawn_phase_accumulate_bf16_bwd(d, x["mag"], x["ang"], x["valve"], x["ret"], x["rb"], gamma, x["theta"],
                                             x["cw"], x["cb"], None, s["ckpt"], x["dz_re"], x["dz_im"], None, s["dmag"],
                                             s["dang"], s["dvalve"], s["dret"], s["dgamma"], s["dtheta"], s["dcw"],
                                             s["dcb"], None, ws)
    elif c["ret"]:
        r = K.cawn_phase_accumulate_ret_bwd(d, x["mag"], x["ang"], x["valve"], x["ret"], x["rb"], x["theta"], x["cw"],
                                            x["cb"], None, s["ckpt"], x["dz_re"], x["dz_im"], None, s["dmag"], s["dang"],
                                            s["dvalve"], s["dret"], s["dtheta"], s["dcw"], s["dcb"], None, ws)
    elif c["gate"] == "valve":
        r = K.cawn_phase_accumulate_valve_bwd(d, x["mag"], x["ang"], x["valve"], gamma, x["theta"], x["cw"], x["cb"],
                                              None, s["ckpt"], x["dz_re"], x["dz_im"], None, s["dmag"], s["dang"],
                                              s["dvalve"], s["dgamma"], s["dtheta"], s["dcw"], s["dcb"], None, ws)
    else:
        r = K.cawn_phase_accumulate_bwd(d, x["mag"], x["ang"], gamma, x["theta"], x["cw"], x["cb"], None, s["ckpt"],
                                        x["dz_re"], x["dz_im"], None, s["dmag"], s["dang"], s["dgamma"], s["dtheta"],
                                        s["dcw"], s["dcb"], None, ws)
    K.check(r)


_GRADS = ["dmag", "dang", "dvalve", "dret", "dgamma", "dtheta", "dcw", "dcb", "dhw", "dhb"]


def run(state):
    s, c = state, state["c"]
    if c["kind"] == "conv":
        x = s["x"]
        K.check(K.cawn_syntax_conv(s["d"], c["H"] * c["F"], x["mag"], x["cw"][0], x["cb"][0], x["hist"], s["y"],
                                   s["hist_out"]))
        return {"y": s["y"], "hist": s["hist_out"]}
    _forward(s)
    out = {"z_re": s["z"][0], "z_im": s["z"][1]}
    if c["kind"] == "fwd":
        out["state"] = s["state_out"]
    if c["kind"] == "layer":
        out["mask"] = s["mask"]
    if c["kind"] == "train":
        _backward(s)
        out.update({k: s[k] for k in _GRADS if s[k] is not None})
    return out


def work(case):
    """Each input read once, each output written once; the operations of one token-lane counted from the equations
    (forward: conv 4 k, clamps and SiLU 12, gate 2, phasor 4, recurrence 8, clamp 2; backward as much again, plus the
    adjoint, the chain rule, the transposed conv and the parameter sums)."""
    c = case
    n, J, k = c["B"] * c["L"] * c["H"] * c["F"], c["H"] * c["F"], c["conv_k"]
    es = 2 if c["bf16"] else 4
    logits = 4 * c["B"] * c["L"] * c["H"] * ((c["gate"] == "valve") + (1 if c["ret"] else 0))
    consts = 4 * J * (2 + 2 * k)
    if c["kind"] == "conv":
        return {"bytes": 8 * n + 4 * J * (k + 1) + 8 * c["B"] * (k - 1) * J, "flops": n * (2 * k + 6)}
    state = 4 * c["B"] * 2 * J * (1 + max(k - 1, 0)) * (2 if c["kind"] == "fwd" else 0)
    by = 4 * es * n + logits + consts + state + (n // 8 if c["kind"] == "layer" else 0)
    fl = n * (4 * k + 28 + (4 if c["ret"] else 0) + (12 if c["hconv"] else 0))
    if c["kind"] == "train":
        by += 6 * es * n + 2 * logits + 2 * consts
        fl += n * (12 * k + 70 + (8 if c["ret"] else 0) + (24 if c["hconv"] else 0))
    return {"bytes": by, "flops": fl}


def tolerance(case):
    """About four times the error that the path shows against exact(): fp32 up to 6e-7 (the scan's roundings and the
    hardware exp, reciprocal, sine and cosine), the conv alone 7e-8, bfloat16 1.9e-3 (the rounding of what is stored)."""
    if case["bf16"]:
        return {"rel": 8e-3}
    return {"rel": 3e-7 if case["kind"] == "conv" else 2.5e-6}


# --------------------------------------------------------------------------------------------------- 64 bits
def _scan(p, lam, s0):
    """S[t] = p[t] + lam[t] S[t-1] over dimension 1 of p [B, L, J] (lam: [J] or [B, L, J]); returns all S."""
    S = torch.empty_like(p)
    cur = s0
    for t in range(p.shape[1]):
        cur = torch.addcmul(p[:, t], lam[:, t] if lam.dim() == 3 else lam, cur)
        S[:, t] = cur
    return S


def _taps(rows, w, b):
    """Causal depth-wise conv of rows [B, k-1+L, J] with w [J, k] and b [J]: in 64 bits, and as the fp32 chain of fused
    multiply-adds on which the gate's decision is defined."""
    k, L = w.shape[1], rows.shape[1] - (w.shape[1] - 1)
    z = b.double().expand(rows.shape[0], L, -1).clone()
    z32 = z.clone()
    for i in range(k):
        t = w[:, i].double() * rows[:, i:i + L].double()
        z += t
        z32 = (t + z32).float().double()      # (the product of two fp32 numbers is exact in 64 bits)
    return z, z32


def _silu(z):
    return z * torch.sigmoid(z)


def _amp(x, amp):
    return torch.clamp(torch.nn.functional.softplus(x, threshold=1e4), max=10.0) if amp else x


def exact(case, seed):
    c = case
    B, L, H, F, Kc = c["B"], c["L"], c["H"], c["F"], c["conv_k"]
    J, halo = H * F, max(c["conv_k"] - 1, 0)
    if B * L * J > MOST_LANE_TOKENS:
        return None
    x = _inputs(c, seed)
    f64 = torch.float64
    if c["kind"] == "conv":
        rows = torch.cat([x["hist"], x["mag"]], 1)
        z, _ = _taps(rows, x["cw"][0], x["cb"][0])
        return {"y": _silu(z.clamp(-CONV_CLAMP, CONV_CLAMP)), "hist": rows[:, L:].double()}
    st = x.get("state")
    hist = st[B * 2 * J:].view(B, halo, 2, J) if st is not None else torch.zeros(B, halo, 2, J, device=DEV)
    rows = [torch.cat([hist[:, :, q], x[k].float()], 1) for q, k in enumerate(("mag", "ang"))]
    cl = lambda v: v.clamp(-CONV_CLAMP, CONV_CLAMP)
    if Kc:
        zm, zm32 = _taps(rows[0], x["cw"][0], x["cb"][0])
        za, _ = _taps(rows[1], x["cw"][1], x["cb"][1])
        xm, phi = _silu(cl(zm)), _silu(cl(za))
    else:
        zm, za = rows[0].double(), rows[1].double()
        zm32, xm, phi = zm, zm, za
    a = _amp(xm, c["amp"])
    head = lambda v: v.double().repeat_interleave(F, dim=2)       # [B, L, H] -> [B, L, J]
    if c["gate"] == "valve":
        sg = torch.sigmoid(x["valve"].double() - 3.0)
        beta = head(torch.where(sg >= float(torch.tensor(EPS)), sg, torch.zeros_like(sg)))
    else:
        x32 = _silu(cl(zm32)) if Kc else zm32
        beta = (_amp(x32, c["amp"]).abs() >= float(torch.tensor(TAU))).double()
        del x32
    del zm32
    p = torch.polar(beta * a, phi)           # (a may be negative: polar takes it as it is)
    rot = torch.polar(torch.ones(J, device=DEV, dtype=f64), x["theta"].double())
    if c["ret"]:
        gam = torch.sigmoid(head(x["ret"]) + x["rb"].double().repeat(H))
        lam = gam * rot
    else:
        gam = x["gamma"].double()
        lam = gam * rot
    s0 = torch.zeros(B, J, device=DEV, dtype=torch.complex128)
    if st is not None:
        s0 = torch.complex(st[:B * 2 * J].view(B, 2, J)[:, 0].double(), st[:B * 2 * J].view(B, 2, J)[:, 1].double())
    S = _scan(p, lam, s0)
    del p
    co = lambda v: v.clamp(-OUT_CLAMP, OUT_CLAMP)
    heads = lambda v: v.view(B, L, H, F)
    shift = lambda v, n: torch.nn.functional.pad(v, (max(-n, 0), max(n, 0)))[..., max(n, 0):max(n, 0) + F]   # v[k + n]
    z = [co(S.real), co(S.imag)]
    out = {}
    if c["hconv"]:
        zc = []
        for q in range(2):
            w, v = x["hw"][q].double(), heads(z[q])
            zc.append(sum(w[:, i, None] * shift(v, i - 1) for i in range(3)) + x["hb"][q].double()[:, None])
        out["z_re"], out["z_im"] = zc[0].reshape(B, L, J), zc[1].reshape(B, L, J)
    else:
        out["z_re"], out["z_im"] = z
    if c["kind"] == "fwd":
        last = torch.stack([S[:, -1].real, S[:, -1].imag], 1)
        tail = torch.stack([r[:, r.shape[1] - halo:] for r in rows], 2).double() if halo else torch.zeros(0, device=DEV, dtype=f64)
        out["state"] = torch.cat([last.flatten(), tail.flatten()])
    if c["kind"] == "layer":
        out["mask"] = None
    if c["kind"] != "train":
        return out
    # ---- backward
    dz = [x["dz_re"].double(), x["dz_im"].double()]
    if c["hconv"]:
        dc = [heads(v.contiguous()) for v in dz]
        out_w, out_b = [], []
        for q in range(2):
            w, v = x["hw"][q].double(), heads(z[q])
            out_w.append(torch.stack([(dc[q] * shift(v, i - 1)).sum((0, 1, 3)) for i in range(3)], 1))
            out_b.append(dc[q].sum((0, 1, 3)))
            dz[q] = sum(w[:, i, None] * shift(dc[q], 1 - i) for i in range(3)).reshape(B, L, J)
        out["dhw"], out["dhb"] = torch.stack(out_w), torch.stack(out_b)
        del dc
    del z
    # the adjoint runs backward in time: G[t] = dZ[t] + conj(lam[t+1]) G[t+1]
    gz = torch.complex(dz[0], dz[1])
    del dz
    G = torch.empty_like(gz)
    cur = torch.zeros(B, J, device=DEV, dtype=torch.complex128)
    lc = lam.conj().resolve_conj()
    for t in range(L - 1, -1, -1):
        if t == L - 1:
            cur = gz[:, t].clone()
        else:
            cur = torch.addcmul(gz[:, t], lc[:, t + 1] if lc.dim() == 3 else lc, cur)
        G[:, t] = cur
    del gz
    cg = lambda v: v.clamp(-GRAD_CLAMP, GRAD_CLAMP)
    Sp = torch.cat([s0[:, None], S[:, :-1]], 1)
    del S
    q = G.conj() * (rot * Sp)                 # Re: d gamma, Im: -(d theta) / gamma
    del Sp
    tg, tt = cg(q.real), cg(-gam * q.imag)
    del q
    if c["ret"]:
        out["dret"] = (tg * gam * (1.0 - gam)).view(B, L, H, F).sum(3)
    else:
        out["dgamma"] = tg.sum((0, 1))
    out["dtheta"] = tt.sum((0, 1))
    del tg, tt
    gr, gi = cg(G.real), cg(G.imag)
    del G
    cs, sn = torch.cos(phi), torch.sin(phi)
    da, dph = gr * cs + gi * sn, (gi * cs - gr * sn) * (beta * a)
    del gr, gi, cs, sn
    if c["gate"] == "valve":
        out["dvalve"] = (a * da).view(B, L, H, F).sum(3) * (sg * (1.0 - sg))
        da = da * beta                        # the threshold gate is straight-through: no factor
    if c["amp"]:
        da = da * torch.where(torch.nn.functional.softplus(xm, threshold=1e4) < 10.0, torch.sigmoid(xm), torch.zeros_like(xm))
    if Kc:
        dsilu = lambda zz: torch.where(zz.abs() <= CONV_CLAMP, torch.sigmoid(zz) * (1.0 + zz * (1.0 - torch.sigmoid(zz))),
                                       torch.zeros_like(zz))
        dzz = [da * dsilu(zm), dph * dsilu(za)]
        del da, dph, zm, za
        du, dw, db = [], [], []
        for sidx in range(2):
            w = x["cw"][sidx].double()
            pad = torch.cat([dzz[sidx], torch.zeros(B, halo, J, device=DEV, dtype=f64)], 1)
            du.append(sum(w[:, k] * pad[:, Kc - 1 - k:Kc - 1 - k + L] for k in range(Kc)))
            dw.append(torch.stack([(dzz[sidx] * rows[sidx][:, k:k + L].double()).sum((0, 1)) for k in range(Kc)], 1))
            db.append(dzz[sidx].sum((0, 1)))
        out["dmag"], out["dang"] = du
        out["dcw"], out["dcb"] = torch.stack(dw), torch.stack(db)
    else:
        out["dmag"], out["dang"] = da, dph
    return out
