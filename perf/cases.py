"""Timed workloads of the library's public entry points.

Each case is one call of a wrapper in ``paper_2512_23068_amd.binding`` on
device tensors, as a program that uses the library makes it: the model's
parameters stay on the GPU between calls, outputs and workspaces come from
torch's allocator inside the call.  Sizes are the repository's own workloads
(``inputs.CONFIGS``, some with a shorter sequence), its model variants on the
same channel counts, and ragged sizes between them.

``exact`` evaluates the same maps in float64 with plain torch: every flow is
a component of a truncated jet (value, directional derivatives, mixed second
derivative), the recurrence is h' = a h + b in jet arithmetic, and a long
sequence is cut into segments that are composed with the product of their
transitions.
"""
from __future__ import annotations

import math

import torch

from paper_2512_23068_amd import binding

DEV = "cuda"

_SSM = dict(kind="scan", B=1, L=1024, D=1536, N=16, K=1, dtype="f32", drive="euler", act="identity", dres=False,
            complex=False, groups=1, rank=0, state=False, a="s4d", dx="normal", lo=1e-3, hi=1e-1)


def _ssm(**kw):
    return {**_SSM, **kw}


def listed():
    return [
        # A toy model: the launch and dependency latency of a call.
        _ssm(name="tiny", L=1024, D=16, dx="impulse0", lo=1e-3, hi=1e-1),
        # A stream that arrives in short blocks: state in, 64 steps, state out.
        _ssm(name="stream_block", B=4, L=64, state=True),
        # One layer of a 130M model on an ordinary context.
        _ssm(name="mamba130m", L=8192),
        # The 128k-step impulse probe (the repository's headline workload).
        _ssm(name="pulse128k", L=131072, dx="impulse", lo=1e-4, hi=1e-2),
        # The stiff regime at the largest width, inputs stored as bfloat16.
        _ssm(name="stiff128k_bf16", L=131072, D=5120, dtype="bf16", a="stiff", hi=10.0),
        # Eight tangent directions against a wide state: Jacobian columns.
        _ssm(name="multidir", B=4, L=8192, D=2048, N=64, K=8, a="s4d8"),
        # A ragged batch through the zero-order hold with the output map.
        _ssm(name="zoh_silu_ragged", B=2, L=10007, D=1000, drive="zoh", act="silu", dres=True),
        # S4D-Lin: a complex diagonal transition.
        _ssm(name="complex_s4d", L=32768, complex=True),
        # Mamba's own block: low-rank step size, SiLU and the residual weight.
        _ssm(name="lowrank_silu", L=32768, rank=48, act="silu", dres=True),
        # Hessian-vector products along two directions.
        _ssm(name="second_order", kind="scan2", L=32768, K=2),
        # Training: every parameter gradient in the forward pass.
        _ssm(name="param_grads", kind="param", L=32768, act="silu", dres=True, delta=True),
        # RWKV-6 style linear attention with its tangent.
        dict(name="rwkv", kind="la", B=1, H=32, L=32768, DK=64, DV=64, K=1, state=False),
    ]


# A drawn case costs no more than the largest listed one: lanes times steps
# times carried flows.
_MAX_FLOW_STEPS = 1.5e10


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["scan", "scan", "scan", "variant", "complex", "wide", "lowrank", "groups", "scan2", "param",
                       "param", "la"])
    if kind == "la":
        B, K = rng.choice([1, 1, 2, 3]), rng.choice([1, 1, 2])
        H, DK, DV = _log_int(rng, 2, 32), rng.choice([16, 32, 64, 64]), rng.choice([64, 64, 128])
        L = _log_int(rng, 100, 32768)
        L = min(L, int(_MAX_FLOW_STEPS / (B * H * DK * DV * (1 + K))))
        return dict(kind="la", B=B, H=H, L=L, DK=DK, DV=DV, K=K, state=rng.random() < 0.3)
    c = _ssm(B=rng.choice([1, 1, 2, 4]), L=_log_int(rng, 64, 131072), D=_log_int(rng, 16, 5120),
             dtype=rng.choice(["f32", "f32", "bf16"]), state=rng.random() < 0.3)
    c["a"], c["hi"] = rng.choice([("s4d", 1e-1), ("s4d", 1e-2), ("stiff", 10.0)])
    out_map = dict(act=rng.choice(["identity", "silu"]), dres=rng.random() < 0.5)
    if kind == "scan":
        c.update(N=rng.choice([4, 8, 16, 16, 16]), K=rng.choice([1, 1, 2]))
    elif kind == "variant":
        c.update(N=rng.choice([8, 16, 16]), K=rng.choice([1, 1, 2]), drive=rng.choice(["euler", "zoh"]), **out_map)
    elif kind == "complex":
        c.update(N=rng.choice([8, 16, 16, 32]), K=rng.choice([1, 1, 2]), complex=True,
                 drive=rng.choice(["euler", "zoh"]))
    elif kind == "wide":
        c.update(N=rng.choice([16, 32, 64, 64]), K=rng.choice([1, 2, 4, 8]), a="s4d8", hi=1e-1)
    elif kind == "lowrank":
        c.update(K=rng.choice([1, 1, 2]), rank=rng.choice([16, 48, 100]), a="s4d", hi=1e-1, **out_map)
    elif kind == "groups":
        g = rng.choice([2, 4])
        c.update(K=rng.choice([1, 1, 2]), groups=g, D=64 * g * rng.randint(1, 1280 // (64 * g)))
    elif kind == "scan2":
        c.update(kind="scan2", N=rng.choice([8, 16, 16, 32]), K=2)
    else:
        c.update(kind="param", N=rng.choice([8, 16, 16, 32]), drive=rng.choice(["euler", "euler", "zoh"]),
                 delta=rng.random() < 0.5, **out_map)
    flows = _flows(c) * (2 if c["complex"] else 1)
    c["L"] = max(1, min(c["L"], int(_MAX_FLOW_STEPS / (c["B"] * c["D"] * c["N"] * flows))))
    return c


def _flows(c):
    """Carried recurrences per lane."""
    if c["kind"] == "scan2":
        return 4
    if c["kind"] == "param":
        return 5 if c["delta"] else 3
    return 1 + c["K"]


# ------------------------------------------------------------------ inputs

def _ssm_params(c, gen):
    D, N, G, R = c["D"], c["N"], c["groups"], c["rank"]
    rand = lambda *s: torch.rand(*s, generator=gen, device=DEV)
    randn = lambda *s: torch.randn(*s, generator=gen, device=DEV)
    n = torch.arange(N, device=DEV, dtype=torch.float32).repeat(D, 1)
    p = {}
    if c["complex"]:
        p["A"] = torch.full((D, N), -0.5, device=DEV)
        p["A_im"] = math.pi * n
    elif c["a"] == "stiff":
        p["A"] = -torch.exp(7.0 * rand(D, N))
    else:
        p["A"] = -(n + 1) / (8.0 if c["a"] == "s4d8" else 1.0)
    v = torch.exp(math.log(c["lo"]) + (math.log(c["hi"]) - math.log(c["lo"])) * rand(D))
    p["b_delta"] = torch.log(torch.expm1(v))
    if R:
        p["W_dx"] = randn(D, R) / math.sqrt(D)
        p["W_dt"] = (2.0 * rand(R, D) - 1.0) / math.sqrt(R)
    else:
        p["w_delta"] = randn(D)
    p["W_B"] = randn(D, G * N) / math.sqrt(D)
    p["W_C"] = randn(D, G * N) / math.sqrt(D)
    if G > 1:
        p["n_groups"] = G
    if c["dres"]:
        p["D_res"] = randn(D)
    return p


def prepare(case, seed):
    c = case
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    randn = lambda *s: torch.randn(*s, generator=gen, device=DEV)
    if c["kind"] == "la":
        B, H, L, DK, DV, K = (c[k] for k in ("B", "H", "L", "DK", "DV", "K"))
        s = 1.0 / math.sqrt(DK)
        rate = math.log(1e-3) + math.log(1e2) * torch.rand(1, H, 1, DK, generator=gen, device=DEV)
        st = {"q": randn(B, H, L, DK) * s, "k": randn(B, H, L, DK) * s, "v": randn(B, H, L, DV),
              "g": -torch.exp(rate + 0.5 * randn(B, H, L, DK)),
              "dq": randn(K, B, H, L, DK) * s, "dk": randn(K, B, H, L, DK) * s, "dv": randn(K, B, H, L, DV)}
        st["dg"] = st["g"] * randn(K, B, H, L, DK)
        if c["state"]:
            st["S_in"], st["dS_in"] = randn(B, H, DK, DV), randn(K, B, H, DK, DV)
        return {"case": c, "in": st}
    B, L, D, N, K = (c[k] for k in ("B", "L", "D", "N", "K"))
    st = {"params": _ssm_params(c, gen)}
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    st["x"] = randn(B, L, D).to(dt)
    if c["kind"] == "param":
        st["gy"] = randn(B, L, D)
    elif c["dx"] == "normal":
        st["dx"] = randn(K, B, L, D).to(dt)
    else:
        st["dx"] = torch.zeros(K, B, L, D, device=DEV, dtype=dt)
        st["dx"][:, :, 0, :1 if c["dx"] == "impulse0" else D] = 1.0
    if c["state"]:
        cd = torch.complex64 if c["complex"] else torch.float32
        rs = lambda *s: torch.randn(*s, generator=gen, device=DEV, dtype=cd)
        nd = {"scan": K, "scan2": 2, "param": _flows(c) - 1}[c["kind"]]
        st["h_in"], st["dh_in"] = 0.1 * rs(B, D, N), 0.1 * rs(nd, B, D, N)
        if c["kind"] == "scan2":
            st["d2h_in"] = 0.1 * rs(B, D, N)
    return {"case": c, "in": st}


def run(state):
    c, i = state["case"], state["in"]
    if c["kind"] == "la":
        return binding.la_scan_jvp(i["q"], i["k"], i["v"], i["g"], i["dq"], i["dk"], i["dv"], i["dg"],
                                   S_in=i.get("S_in"), dS_in=i.get("dS_in"), return_state=c["state"])
    h, dh = i.get("h_in"), i.get("dh_in")
    if c["kind"] == "scan2":
        return binding.scan_jvp2(i["x"], i["dx"], i["params"], h_in=h, dh_in=dh, d2h_in=i.get("d2h_in"),
                                 return_state=c["state"])
    if c["kind"] == "param":
        return binding.param_grads(i["x"], i["gy"], i["params"], h_in=h, gamma_in=dh, return_state=c["state"],
                                   drive=c["drive"], act=c["act"], delta_params=c["delta"])
    return binding.scan_jvp(i["x"], i["dx"], i["params"], h_in=h, dh_in=dh, return_state=c["state"],
                            drive=c["drive"], act=c["act"])


# ------------------------------------------------------------------ size of a pass

def work(case):
    c = case
    if c["kind"] == "la":
        rows = c["B"] * c["H"] * c["L"]
        K = c["K"]
        nbytes = 4 * rows * (1 + K) * (3 * c["DK"] + 2 * c["DV"])
        # per entry of S: decay, k v, q S; per tangent four terms of dS and two of the output
        flops = rows * c["DK"] * c["DV"] * (5 + 11 * K)
        if c["state"]:
            nbytes += 8 * c["B"] * c["H"] * c["DK"] * c["DV"] * (1 + K)
        return {"bytes": nbytes, "flops": flops}
    B, L, D, N, K = (c[k] for k in ("B", "L", "D", "N", "K"))
    s = 2 if c["dtype"] == "bf16" else 4
    tok, lanes = B * L * D, B * L * D * N
    if c["kind"] == "param":
        nbytes, per = tok * (s + 8), 21 + (10 if c["delta"] else 0)
        proj = 1
    elif c["kind"] == "scan2":
        nbytes, per, proj = tok * (3 * s + 16), 54, 3
    else:
        nbytes, proj = tok * (1 + K) * (s + 4), 1 + K
        # complex: the products with Abar and A count four and two real ones
        per = (7 + 11 * K) if not c["complex"] else (24 + 17 * K)
    per += 4 if c["drive"] == "zoh" else 0
    flops = lanes * per + tok * proj * 4 * N * c["groups"]
    if c["rank"]:
        flops += tok * proj * 4 * c["rank"]
    nbytes += 4 * D * N * (1 + 2 * c["groups"]) + 8 * D * (1 + c["rank"])
    if c["state"]:
        nbytes += 8 * B * D * N * _flows(c) * (2 if c["complex"] else 1)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # float32 throughout.  Measured against exact(): 1.1e-6 at most for the
    # scans and linear attention, 2.5e-6 for the parameter gradients (long
    # sums), 5.3e-6 for the complex transition (its rotations accumulate over
    # a weakly damped lane's memory); about four to eight times that.
    if case["kind"] == "param" or case.get("complex"):
        return {"rel": 2e-5}
    return {"rel": 8e-6}


# ------------------------------------------------------------------ float64 reference

def _add(p, q):
    return q if p is None else (p if q is None else p + q)


def _mul(p, q):
    return None if p is None or q is None else p * q


def _jmul(p, q, mixed):
    """Product of two jets: lists (value, derivative per direction), with
    the mixed derivative of directions 1 and 2 as component 3."""
    out = [_mul(p[0], q[0])]
    for k in range(1, len(p)):
        out.append(_add(_mul(p[0], q[k]), _mul(p[k], q[0])))
    if mixed:
        out[3] = _add(out[3], _add(_mul(p[1], q[2]), _mul(p[2], q[1])))
    return out


def _jexp(z, mixed):
    e = torch.exp(z[0])
    out = [e] + [_mul(e, zk) for zk in z[1:]]
    if mixed:
        out[3] = _add(out[3], _mul(e, _mul(z[1], z[2])))
    return out


def _flow(h, T, G, step, seg, read, mixed):
    """Steps h <- a h + b of G segments of T steps, entered in state h (jet
    without a segment axis).  step(t) gives the jets a, b of step t of every
    segment [B,G,...], seg(g) the product of segment g's transitions, and
    read(t, h) sees every state.  Returns the state after the last segment."""
    if G > 1:
        e = None
        for t in range(T):
            a, b = step(t)
            e = list(b) if e is None else [_add(u, v) for u, v in zip(_jmul(a, e, mixed), b)]
        zero = torch.zeros_like(e[0])
        e = [zero if v is None else v for v in e]
        entry = [torch.empty_like(v) for v in e]
        for g in range(G):
            for m, v in zip(entry, h):
                m[:, g] = v
            h = [_add(u, v[:, g]) for u, v in zip(_jmul(seg(g), h, mixed), e)]
    else:
        entry = [v[:, None].clone() for v in h]
    cur = entry
    for t in range(T):
        a, b = step(t)
        cur = [_add(u, v) for u, v in zip(_jmul(a, cur, mixed), b)]
        read(t, cur)
    return [v[:, -1] for v in cur]


def _spans(L, per_seg_bytes):
    """Cuts L steps into (start, T, G) runs of G segments of T steps that
    keep the states of all segments within a few GB."""
    G = int(max(1, min(L // 16 if L >= 32 else 1, 1.5e9 // per_seg_bytes, 2048)))
    T = max(1, L // G)
    G = L // T
    out = [(0, T, G)] if L else []
    if L - T * G:
        out.append((T * G, L - T * G, 1))
    return out


def _silu(v):
    s = torch.sigmoid(v)
    return v * s, s * (1 + v * (1 - s))


def exact(case, seed):
    c = case
    if c["kind"] == "la":
        lanes = c["B"] * c["H"] * c["DK"] * c["DV"]
        flows = 1 + c["K"]
    else:
        flows = _flows(c) * (2 if c["complex"] else 1)
        lanes = c["B"] * c["D"] * c["N"]
    if lanes * c["L"] * flows > 6e10:
        return None
    i = prepare(c, seed)["in"]
    return _exact_la(c, i) if c["kind"] == "la" else _exact_ssm(c, i)


def _exact_ssm(c, i):
    B, L, D, N = (c[k] for k in ("B", "L", "D", "N"))
    kind, mixed = c["kind"], c["kind"] == "scan2"
    f64 = torch.float64
    ldt = torch.complex128 if c["complex"] else f64
    P = {k: v.to(f64) if isinstance(v, torch.Tensor) else v for k, v in i["params"].items()}
    A = torch.complex(P["A"], P["A_im"]) if c["complex"] else P["A"]
    F = _flows(c)
    K = 0 if kind == "param" else c["K"]
    gr = c["groups"]
    x_all = i["x"]
    src = [x_all] + [i["dx"][k] for k in range(K)]
    state = [torch.zeros(B, D, N, device=DEV, dtype=ldt) for _ in range(F)]
    if c["state"]:
        dh = i["dh_in"].to(ldt)
        state = [i["h_in"].to(ldt)] + [dh[k] for k in range(dh.shape[0])]
        if mixed:
            state.append(i["d2h_in"].to(ldt))
    nout = 1 if kind == "param" else F
    outs = [torch.empty(B, L, D, device=DEV, dtype=f64) for _ in range(nout)]
    gA, gB, gC = (torch.zeros(D, N, device=DEV, dtype=f64) for _ in range(3))
    gD, gW, gS = (torch.zeros(D, device=DEV, dtype=f64) for _ in range(3))

    lane = lambda v: None if v is None else v.unsqueeze(-1)
    for t0, T, G in _spans(L, B * D * N * F * 8 * (2 if c["complex"] else 1)):
        rows = [s[:, t0:t0 + T * G].to(f64).reshape(B, G, T, D) for s in src]
        x = rows[0]

        def proj(W):
            # per channel: the columns of its group
            def one(r):
                v = r @ W
                if gr == 1:
                    return v.unsqueeze(-2)
                return v.reshape(B, G, T, gr, N).repeat_interleave(D // gr, dim=3)
            js = [one(r) for r in rows] + [None] * (F - 1 - K)
            return js

        Bj, Cj = proj(P["W_B"]), proj(P["W_C"])
        if c["rank"]:
            zj = [(r @ P["W_dx"]) @ P["W_dt"] for r in rows]
            zj[0] = zj[0] + P["b_delta"]
        else:
            zj = [r * P["w_delta"] for r in rows]
            zj[0] = zj[0] + P["b_delta"]
        sig = torch.sigmoid(zj[0])
        dl = [torch.nn.functional.softplus(zj[0], threshold=1e9)] + [sig * z for z in zj[1:]]
        if mixed:
            dl.append(sig * (1 - sig) * zj[1] * zj[2])
        xj = rows + [None] * (F - 1 - K)
        if kind == "param":   # directions: A, the offset of B, w_delta, b_delta
            dl = [dl[0], None, None] + ([sig * x, sig] if c["delta"] else [])
        dsum = [None if v is None else v.sum(2) for v in dl]

        def zeta(d):
            z = [None if v is None else lane(v) * A for v in d]
            if kind == "param":
                z[1] = lane(d[0])
            return z

        def at(js, t):
            return [None if v is None else v[:, :, t] for v in js]

        def step(t):
            d, xt, bt = at(dl, t), at(xj, t), at(Bj, t)
            z = zeta(d)
            a = _jexp(z, mixed)
            if c["drive"] == "zoh":
                e0 = torch.expm1(z[0]) / A if not c["complex"] else (a[0] - 1) / A
                e = [e0] + [None if v is None else a[0] * lane(v) for v in d[1:]]
                if kind == "param":
                    e[1] = (lane(d[0]) * a[0] - e0) / A
                bx = _jmul(bt, [lane(v) for v in xt], mixed)
                b = _jmul(e, bx, mixed)
                if kind == "param":
                    b[2] = e0 * lane(xt[0])
            else:
                u = _jmul(d, xt, mixed)
                b = _jmul([lane(v) for v in u], bt, mixed)
                if kind == "param":
                    b[2] = lane(u[0]).expand(B, G, D, N)
            return a, b

        def read(t, h):
            ct = at(Cj, t)
            if c["complex"]:
                h = [v.real for v in h]
            view = [o[:, t0:t0 + T * G].view(B, G, T, D) for o in outs]
            xt = x[:, :, t]
            if kind == "param":
                v = (ct[0] * h[0]).sum(-1)
                w = i["gy"][:, t0:t0 + T * G].to(f64).view(B, G, T, D)[:, :, t]
                if c["dres"]:
                    v = v + P["D_res"] * xt
                if c["act"] == "silu":
                    v, dv = _silu(v)
                    w = w * dv
                view[0][:, :, t] = v
                wc = lane(w) * ct[0]
                gA.add_((wc * h[1]).sum((0, 1)))
                gB.add_((wc * h[2]).sum((0, 1)))
                gC.add_((lane(w) * h[0]).sum((0, 1)))
                gD.add_((w * xt).sum((0, 1)))
                if c["delta"]:
                    gW.add_((wc * h[3]).sum((0, 1, 3)))
                    gS.add_((wc * h[4]).sum((0, 1, 3)))
                return
            y = [v.sum(-1) for v in _jmul(ct, h, mixed)]
            if c["dres"]:
                y = [v + P["D_res"] * r[:, :, t] for v, r in zip(y, rows)]
            if c["act"] == "silu":
                f, df = _silu(y[0])
                y = [f] + [v * df for v in y[1:]]
            for o, v in zip(view, y):
                o[:, :, t] = v

        state = _flow(state, T, G, step, lambda g: _jexp(zeta([None if v is None else v[:, g] for v in dsum]), mixed),
                      read, mixed)

    if kind == "param":
        res = [outs[0], gA, gB, gC] + ([gD] if c["dres"] else []) + ([gW, gS] if c["delta"] else [])
    else:
        res = [outs[0], torch.stack(outs[1:1 + c["K"]])] + ([outs[3]] if mixed else [])
    if c["state"]:
        res.append(state[0])
        res.append(torch.stack(state[1:3] if mixed else state[1:]))
        if mixed:
            res.append(state[3])
    return tuple(res)


def _exact_la(c, i):
    B, H, L, DK, DV, K = (c[k] for k in ("B", "H", "L", "DK", "DV", "K"))
    f64 = torch.float64
    jet = lambda p, d: [p.reshape(B * H, L, -1)] + [i_.reshape(B * H, L, -1) for i_ in d]
    q, k, v, g = (jet(i[n], i["d" + n]) for n in ("q", "k", "v", "g"))
    if c["state"]:
        state = [i["S_in"].to(f64).reshape(B * H, DK, DV)]
        state += [s.to(f64).reshape(B * H, DK, DV) for s in i["dS_in"]]
    else:
        state = [torch.zeros(B * H, DK, DV, device=DEV, dtype=f64) for _ in range(1 + K)]
    outs = [torch.empty(B * H, L, DV, device=DEV, dtype=f64) for _ in range(1 + K)]
    for t0, T, G in _spans(L, B * H * DK * DV * (1 + K) * 8):
        cut = lambda js: [r[:, t0:t0 + T * G].to(f64).reshape(B * H, G, T, -1) for r in js]
        qc, kc, vc, gc = cut(q), cut(k), cut(v), cut(g)
        gsum = [r.sum(2) for r in gc]
        at = lambda js, t, dim: [r[:, :, t].unsqueeze(dim) for r in js]

        def step(t):
            return _jexp(at(gc, t, -1), False), _jmul(at(kc, t, -1), at(vc, t, -2), False)

        def read(t, s):
            for o, r in zip(outs, _jmul(at(qc, t, -1), s, False)):
                o[:, t0:t0 + T * G].view(B * H, G, T, DV)[:, :, t] = r.sum(-2)

        state = _flow(state, T, G, step, lambda n: _jexp([r[:, n].unsqueeze(-1) for r in gsum], False), read, False)
    shape = lambda r, n: r.reshape(B, H, n, DV)
    res = [shape(outs[0], L), torch.stack([shape(o, L) for o in outs[1:]])]
    if c["state"]:
        res += [shape(state[0], DK), torch.stack([shape(s, DK) for s in state[1:]])]
    return tuple(res)
