"""The framework's measured workloads.

Each case is one pass through the public entry points of
``paper_2609_36529_amd`` at sizes that its users run: training steps of the
operator, inference forwards (prefill), decode steps, and the whole mixer
around the operator.  ``listed()`` gives the named cases, ``draw(rng)`` one
more of the same ranges, ``prepare`` the inputs that a program has in hand
before the call, ``run`` the pass, ``exact`` the same results in float64 from
plain torch.

Kinds of case:
  train   training forward and backward of the operator.  ``entry`` is
          "autograd" (``attention`` under torch.autograd, a model's layer) or
          "direct" (``fwd`` / ``bwd`` calls, a hand-written training step).
  packed  the direct calls over documents of different lengths stored back to
          back (``cu_seqlens``).
  prefill inference forward: outputs and the final state.
  decode  one token for each sequence, the fp32 state updated in place.
  mixer   input projection with convolution, activations and norms, gate
          heads, operator and output gate, forward and backward.
"""
import math

import torch

import paper_2609_36529_amd as tla

SGLA, GDN = 0, 1


# ------------------------------------------------------------------ the cases
def _op(kind, variant, dtype, B, T, H, K, V, E, chunk, **more):
    return dict(kind=kind, variant=variant, dtype=dtype, B=B, T=T, H=H, K=K, V=V, E=E, chunk=chunk,
                **more)


def listed():
    return [
        # the headline workload: one layer's operator in language-model
        # training at 4k context, hand-written training step
        dict(_op("train", "gdn", "bf16", 4, 4096, 8, 128, 128, 8, 64, entry="direct", s0=True),
             name="train_gdn_4k"),
        # the wide state (E = 16) under autograd, 16 heads of a d_model 2048
        # block, 2k context
        dict(_op("train", "gdn", "bf16", 2, 2048, 16, 128, 128, 16, 64, entry="autograd", s0=False),
             name="train_gdn_e16"),
        # a narrow state (E = 4) without the delta rule, a context length that
        # is no multiple of the chunk
        dict(_op("train", "sgla", "bf16", 2, 1999, 16, 128, 128, 4, 64, entry="autograd", s0=False),
             name="train_sgla_e4_ragged"),
        # documents of uneven lengths packed into one row
        dict(_op("packed", "gdn", "bf16", 13, 8192, 8, 128, 128, 8, 64), name="train_gdn_packed"),
        # fp32 operands at a small head size (numerics work, small models)
        dict(_op("train", "gdn", "f32", 2, 1024, 4, 64, 64, 8, 32, entry="autograd", s0=False),
             name="train_gdn_f32"),
        # the recall (MQAR) model's layer: 64 pairs and 64 queries, 128
        # sequences a step, head dimension 16
        dict(_op("train", "sgla", "bf16", 128, 128, 4, 16, 16, 4, 16, entry="autograd", s0=False),
             name="train_mqar_layer"),
        # batched prefill without the delta rule
        dict(_op("prefill", "sgla", "bf16", 4, 4096, 8, 128, 128, 8, 64, s0=False),
             name="prefill_sgla_4k"),
        # one short user turn continued from a cached state
        dict(_op("prefill", "gdn", "bf16", 1, 777, 16, 128, 128, 8, 64, s0=True),
             name="prefill_gdn_turn"),
        # long-context prefill of one sequence
        dict(_op("prefill", "gdn", "bf16", 1, 65536, 16, 128, 128, 16, 64, s0=False),
             name="prefill_gdn_64k"),
        # a single sequence's decode step
        dict(_op("decode", "gdn", "bf16", 1, 1, 8, 128, 128, 8, 16), name="decode_one"),
        # a serving batch's decode step
        dict(_op("decode", "gdn", "bf16", 256, 1, 16, 128, 128, 16, 16), name="decode_batch"),
        # the mixer of a d_model 2048 block with 16 heads, training
        dict(_op("mixer", "gdn", "bf16", 2, 2048, 16, 128, 128, 8, 64, Dm=2048, W=4),
             name="mixer_train"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["train", "train", "train", "packed", "prefill", "prefill", "prefill", "decode",
                       "decode", "mixer"])
    variant = rng.choice(["gdn", "gdn", "sgla"])
    if kind == "decode":
        H, E = rng.choice([4, 8, 16]), rng.choice([1, 4, 8, 16])
        return _op("decode", variant, "bf16", _log(rng, 1, 256), 1, H, 128, 128, E, 16)
    if kind == "mixer":
        H = rng.choice([4, 8, 16])
        T = _log(rng, 64, 2048)
        return _op("mixer", variant, "bf16", rng.choice([1, 2]), T, H, 128, 128, rng.choice([8, 16]), 64,
                   Dm=8 * rng.randint(64, 256), W=rng.choice([2, 4]))
    if kind == "prefill":
        E, H = rng.choice([1, 4, 8, 8, 16]), rng.choice([4, 8, 16])
        T = _log(rng, 16, 65536)
        B = rng.choice([1, 2, 4]) if T <= 16384 else 1
        return _op("prefill", variant, "bf16", B, T, H, 128, 128, E, 64, s0=rng.random() < 0.5)
    if kind == "packed":
        return _op("packed", variant, "bf16", rng.randint(2, 24), _log(rng, 512, 8192), 8, 128, 128,
                   rng.choice([4, 8]), 64)
    K, chunk, E = rng.choice([(128, 64, 8), (128, 64, 8), (128, 64, 4), (128, 64, 16), (64, 32, 8),
                              (64, 64, 16), (16, 16, 4), (16, 16, 16)])
    small = K < 128
    dtype = rng.choice(["bf16", "f32"]) if K == 64 and chunk == 32 else "bf16"
    T = _log(rng, 64, 1024 if small else 4096)
    B = rng.randint(8, 128) if K == 16 else rng.choice([1, 2, 4])
    return _op("train", variant, dtype, B, T, 4 if small else 8, K, K, E, chunk,
               entry=rng.choice(["autograd", "direct"]), s0=rng.random() < 0.5)


# ----------------------------------------------------------------- the inputs
def _variant(c):
    return GDN if c["variant"] == "gdn" else SGLA


def _dt(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


class _Draws:
    """Seeded normal and uniform tensors on the GPU."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda")
        self.gen.manual_seed(seed)

    def normal(self, *shape):
        return torch.randn(shape, generator=self.gen, device="cuda")

    def uniform(self, *shape):
        return torch.rand(shape, generator=self.gen, device="cuda")

    def unit(self, *shape):
        return torch.nn.functional.normalize(self.normal(*shape), dim=-1)


def _tokens(c, d, lead):
    """q, k, v, q2, k2, g, beta with leading axes `lead`: keys and queries of
    unit length, values N(0, 1), log-gates -softplus(N(0, 1)) / 16, write
    strengths sigmoid(N(0, 1)); for the recall layer (K = 16) unnormalised
    projections, no decay, and a write strength of 1 in the first half of each
    sequence (the pairs) and 0 in the second (the queries)."""
    K, V, E, dt = c["K"], c["V"], c["E"], _dt(c)
    if K == 16:
        q, k, v, q2, k2 = (0.577 * d.normal(*lead, n) for n in (K, K, V, E, E))
        g = torch.zeros(*lead, E, device="cuda")
        beta = torch.ones(lead, device="cuda")
        beta[:, lead[1] // 2:] = 0.0
    else:
        q, k, q2, k2 = (d.unit(*lead, n) for n in (K, K, E, E))
        v = d.normal(*lead, V)
        g = -torch.nn.functional.softplus(d.normal(*lead, E)) / 16.0
        beta = torch.sigmoid(d.normal(*lead)) if c["variant"] == "gdn" else None
    return [x.to(dt) for x in (q, k, v, q2, k2)] + [g, beta]


def _lengths(c):
    """c["B"] document lengths that sum to c["T"], uneven, the same for every
    seed: proportional to 1, 2, .., 5, 1, 2, .. with a remainder on the last."""
    part = [1 + i % 5 for i in range(c["B"])]
    n = [max(1, c["T"] * p // sum(part)) for p in part]
    n[-1] += c["T"] - sum(n)
    return n


def prepare(case, seed):
    c, d = case, _Draws(seed)
    B, T, H, K, V, E, dt = c["B"], c["T"], c["H"], c["K"], c["V"], c["E"], _dt(c)
    st = {"case": c}
    if c["kind"] == "decode":
        st["tok"] = _tokens(c, d, (B, H))
        st["state"] = 0.02 * d.normal(B, H, E, K, V)
        return st
    if c["kind"] == "packed":
        lens = _lengths(c)
        offs = [0]
        for n in lens:
            offs.append(offs[-1] + n)
        st["lens"], st["longest"] = lens, max(lens)
        st["cu"] = torch.tensor(offs, dtype=torch.int32, device="cuda")
        st["tok"] = _tokens(c, d, (1, T, H))
        st["dO"] = d.normal(1, T, H, V).to(dt)
        return st
    if c["kind"] == "mixer":
        Ct = H * (2 * K + V + 2 * E)
        st["u"] = d.normal(B, T, c["Dm"]).to(dt)
        st["Wp"] = (d.normal(Ct, c["Dm"]) / math.sqrt(c["Dm"])).to(dt)
        st["taps"] = (2.0 * d.uniform(c["W"], Ct) - 1.0) / math.sqrt(c["W"])
        st["x"] = d.normal(B, T, H, E).to(dt)
        st["xb"] = d.normal(B, T, H).to(dt) if c["variant"] == "gdn" else None
        st["A"] = torch.log(1.0 + 15.0 * d.uniform(H, E))
        step = torch.exp(math.log(1e-3) + math.log(100.0) * d.uniform(H, E))
        st["b"] = step + torch.log(-torch.expm1(-step))     # softplus(b) = step
        st["z"] = (2.0 * d.normal(B, T, H, V)).to(dt)
        st["gain"] = 1.0 + 0.5 * d.normal(V)
        st["dy"] = d.normal(B, T, H, V).to(dt)
        return st
    st["tok"] = _tokens(c, d, (B, T, H))
    st["s0"] = 0.02 * d.normal(B, H, E, K, V) if c["s0"] else None
    if c["kind"] == "train":
        st["dO"] = d.normal(B, T, H, V).to(dt)
        if c["entry"] == "autograd":
            st["leaves"] = [x for x in st["tok"] + [st["s0"]] if x is not None]
            for x in st["leaves"]:
                x.requires_grad_(True)
    return st


# ------------------------------------------------------------------- the pass
GRADS = ("dq", "dk", "dv", "dq2", "dk2", "dg", "dbeta", "ds0")


def run(state):
    st, c = state, state["case"]
    var = _variant(c)
    if c["kind"] == "decode":
        o = tla.step(var, *st["tok"], st["state"])
        return {"o": o, "state": st["state"]}
    if c["kind"] == "prefill":
        o, sf, _ = tla.fwd(var, *st["tok"], st["s0"], chunk=c["chunk"])
        return {"o": o, "s_final": sf}
    if c["kind"] == "packed":
        q, k, v, q2, k2, g, beta = st["tok"]
        o, sf, saved = tla.fwd(var, q, k, v, q2, k2, g, beta, chunk=c["chunk"], training=True,
                               cu_seqlens=st["cu"], max_seqlen=st["longest"])
        gr = tla.bwd(var, q, k, v, q2, k2, g, beta, None, st["dO"], saved, chunk=c["chunk"],
                     want_ds0=False, cu_seqlens=st["cu"], max_seqlen=st["longest"])
        return {"o": o, "s_final": sf, **{n: gr[n] for n in GRADS if gr[n] is not None}}
    if c["kind"] == "mixer":
        return _run_mixer(st, c, var)
    if c["entry"] == "autograd":
        o, sf = tla.attention(var, *st["tok"], st["s0"], chunk=c["chunk"])
        gr = torch.autograd.grad(o, st["leaves"], st["dO"])
        return {"o": o.detach(), "s_final": sf.detach(), "grads": list(gr)}
    q, k, v, q2, k2, g, beta = st["tok"]
    o, sf, saved = tla.fwd(var, q, k, v, q2, k2, g, beta, st["s0"], chunk=c["chunk"], training=True)
    gr = tla.bwd(var, q, k, v, q2, k2, g, beta, st["s0"], st["dO"], saved, chunk=c["chunk"],
                 want_ds0=st["s0"] is not None)
    return {"o": o, "s_final": sf, "grads": [gr[n] for n in GRADS if gr[n] is not None]}


def _run_mixer(st, c, var):
    H, K, V, E = c["H"], c["K"], c["V"], c["E"]
    q, k, v, q2, k2, y = tla.proj_in_fwd(st["u"], st["Wp"], st["taps"], H, K, V, E, keep_y=True)
    g, beta = tla.gate_heads_fwd(st["x"], st["xb"], st["A"], st["b"])
    o, _, saved = tla.fwd(var, q, k, v, q2, k2, g, beta, chunk=c["chunk"], training=True,
                          want_final=False)
    out = tla.out_gate_fwd(o, st["z"], st["gain"])
    d_o, dz, dgain = tla.out_gate_bwd(o, st["z"], st["gain"], st["dy"])
    gr = tla.bwd(var, q, k, v, q2, k2, g, beta, None, d_o, saved, chunk=c["chunk"], want_ds0=False)
    dx, dxb, dA, db = tla.gate_heads_bwd(st["x"], st["xb"], st["A"], st["b"], gr["dg"], gr["dbeta"])
    du, dWp, dtaps = tla.proj_in_bwd(st["u"], st["Wp"], st["taps"], y, H, K, V, E,
                                     tuple(gr[n] for n in GRADS[:5]))
    res = {"out": out, "dz": dz, "dgain": dgain, "dx": dx, "dA": dA, "db": db, "du": du, "dWp": dWp,
           "dtaps": dtaps}
    if dxb is not None:
        res["dxb"] = dxb
    return res


# ------------------------------------------------------------------- the work
def work(case):
    """Inputs read once, outputs written once; the contractions of the
    chunkwise form (forward: read-outs and state update; backward: the reverse
    recurrence and the state contractions, twice the forward's)."""
    c = case
    B, T, H, K, V, E, C = (c[n] for n in ("B", "T", "H", "K", "V", "E", "chunk"))
    es = 2 if c["dtype"] == "bf16" else 4
    gdn = c["variant"] == "gdn"
    state = B * H * E * K * V
    if c["kind"] == "decode":
        n = B * H
        return {"bytes": 8 * state + n * (es * (2 * K + 2 * V + 2 * E) + 4 * E + 4 * gdn),
                "flops": n * E * K * V * (7 if gdn else 5)}
    th = (T if c["kind"] == "packed" else B * T) * H
    io = es * (2 * K + 2 * V + 2 * E) + 4 * E + 4 * gdn
    fl = (6 if gdn else 4) * K * V * E + 4 * C * K + 2 * C * V * (2 if gdn else 1)
    by = th * io + 4 * state * (2 if c.get("s0") else 1)
    if c["kind"] == "prefill":
        return {"bytes": by, "flops": th * fl}
    by += th * (io + es * (2 * K + V + 2 * E) + 4 * E + 4 * gdn)
    if c.get("s0"):
        by += 4 * state
    fl *= 3
    if c["kind"] == "mixer":
        Ct, N = H * (2 * K + V + 2 * E), B * T
        by = (2 * 2 * N * c["Dm"] + 2 * Ct * c["Dm"] + 4 * Ct * c["Dm"] + 8 * c["W"] * Ct
              + th * (2 * 2 * E + 2 * 2 * gdn + 4 * 2 * V))
        return {"bytes": by, "flops": th * fl + 6 * N * Ct * c["Dm"]}
    return {"bytes": by, "flops": th * fl}


def tolerance(case):
    """About four times the relative error against float64 that was measured:
    bf16 results 1.8e-3 (their own rounding), 5e-3 where layers follow one
    another (mixer) or the operands are not normalised (recall layer), fp32
    operands 3e-7 with up to three times that at other sizes."""
    if case["dtype"] == "f32":
        return {"rel": 4e-6}
    if case["kind"] == "mixer" or case["K"] == 16:
        return {"rel": 2e-2}
    return {"rel": 8e-3}


# ------------------------------------------------------ the results in 64 bits
def _operator64(c, q, k, v, q2, k2, g, beta, s0, C):
    """Chunk by chunk in float64 (autograd goes through it): [B, T, H, .] in,
    (o, final state) out."""
    B, T, H, K = q.shape
    V, E = v.shape[-1], q2.shape[-1]
    gdn = c["variant"] == "gdn"
    if beta is None:
        beta = torch.ones(B, T, H, dtype=torch.float64, device=q.device)
    q, k, v, q2, k2, g = (x.transpose(1, 2) for x in (q, k, v, q2, k2, g))
    beta = beta.transpose(1, 2)
    S = s0 if s0 is not None else torch.zeros(B, H, E, K, V, dtype=torch.float64, device=q.device)
    S = S.reshape(B, H, E * K, V)
    outs = []
    for t in range(0, T, C):
        n = min(C, T - t)
        qc, kc, vc, q2c, k2c, gc = (x[:, :, t:t + n].contiguous() for x in (q, k, v, q2, k2, g))
        bc = beta[:, :, t:t + n, None]
        G = gc.cumsum(2)
        low = torch.ones(n, n, dtype=torch.float64, device=q.device).tril()
        D = torch.exp((G[:, :, :, None] - G[:, :, None]).clamp(max=0.0)) * low[:, :, None]
        Rq = ((q2c[:, :, :, None] * D) * k2c[:, :, None]).sum(-1)
        Aq = torch.matmul(qc, kc.transpose(2, 3).contiguous()) * Rq

        def joint(x2, x):
            return (x2[..., :, None] * x[..., None, :]).reshape(B, H, n, E * K)

        if gdn:
            Rk = ((k2c[:, :, :, None] * D) * k2c[:, :, None]).sum(-1)
            L = (bc * torch.matmul(kc, kc.transpose(2, 3).contiguous()) * Rk).tril(-1)
            rhs = bc * (vc - torch.matmul(joint(k2c * torch.exp(G), kc), S))
            # (I + L)^-1 rhs with L nilpotent: (I - L)(I + L^2)(I + L^4) ..
            U, P, m = rhs - torch.matmul(L, rhs), torch.matmul(L, L), 2
            while m < n:
                U = U + torch.matmul(P, U)
                P, m = torch.matmul(P, P), 2 * m
        else:
            U = bc * vc
        outs.append(torch.matmul(joint(q2c * torch.exp(G), qc), S) + torch.matmul(Aq, U))
        kj = joint(k2c * torch.exp(G[:, :, -1:] - G), kc)
        decay = torch.exp(G[:, :, -1])[..., None].expand(B, H, E, K).reshape(B, H, E * K, 1)
        S = decay * S + torch.matmul(kj.transpose(2, 3).contiguous(), U)
    return torch.cat(outs, 2).transpose(1, 2), S.reshape(B, H, E, K, V)


def _f64(x):
    return None if x is None else x.detach().double()


def exact(case, seed):
    c = case
    st = prepare(c, seed)
    C = 64 if c["K"] > 16 else 16
    if c["kind"] == "decode":
        q, k, v, q2, k2, g, beta = (_f64(x) for x in st["tok"])
        S = _f64(st["state"]) * torch.exp(g)[..., None, None]
        kj = k2[..., :, None] * k[..., None, :]
        w = v if c["variant"] == "sgla" else v - (kj[..., None] * S).sum((2, 3))
        w = w if beta is None else beta[..., None] * w
        S += kj[..., None] * w[:, :, None, None, :]
        qj = q2[..., :, None] * q[..., None, :]
        return {"o": (qj[..., None] * S).sum((2, 3)), "state": S}
    if c["kind"] == "prefill":
        with torch.no_grad():
            o, sf = _operator64(c, *[_f64(x) for x in st["tok"]], _f64(st["s0"]), C)
        return {"o": o, "s_final": sf}
    if c["kind"] == "mixer":
        return _exact_mixer(c, st)
    ins = [_f64(x) for x in st["tok"]]
    s0 = _f64(st.get("s0"))
    leaves = [x.requires_grad_(True) for x in ins + [s0] if x is not None]
    if c["kind"] == "packed":
        names = [n for n, x in zip(GRADS, ins) if x is not None]
        outs, finals, at = [], [], 0
        total = 0.0
        for n in st["lens"]:
            part = [None if x is None else x[:, at:at + n] for x in ins]
            o, sf = _operator64(c, *part, None, C)
            total = total + (o * st["dO"][:, at:at + n].double()).sum()
            outs.append(o.detach())
            finals.append(sf.detach())
            at += n
        gr = torch.autograd.grad(total, leaves)
        return {"o": torch.cat(outs, 1), "s_final": torch.cat(finals, 0), **dict(zip(names, gr))}
    o, sf = _operator64(c, *ins, s0, C)
    gr = torch.autograd.grad(o, leaves, st["dO"].double())
    return {"o": o.detach(), "s_final": sf.detach(), "grads": list(gr)}


def _exact_mixer(c, st):
    B, T, H, K, V, E, W = (c[n] for n in ("B", "T", "H", "K", "V", "E", "W"))
    names = [n for n in ("u", "Wp", "taps", "x", "xb", "A", "b", "z", "gain") if st[n] is not None]
    p = {n: _f64(st[n]).requires_grad_(True) for n in names}
    F = torch.nn.functional
    y = torch.matmul(p["u"].reshape(B * T, -1), p["Wp"].t().contiguous()).reshape(B, T, -1)
    past = F.pad(y, (0, 0, W - 1, 0))
    y = sum(p["taps"][j] * past[:, j:j + T] for j in range(W))
    parts = torch.split(y, [H * K, H * K, H * V, H * E, H * E], dim=-1)
    q, k, v, q2, k2 = (x.reshape(B, T, H, -1) for x in parts)

    def norm(x):
        return x / torch.sqrt((x * x).sum(-1, keepdim=True) + 1e-6)

    q, k, v = norm(F.silu(q)), norm(F.silu(k)), F.silu(v)
    q2, k2 = norm(F.softplus(q2)), norm(F.softplus(k2))
    g = -torch.exp(p["A"]) * F.softplus(p["x"] + p["b"])
    beta = torch.sigmoid(p["xb"]) if "xb" in p else None
    o, _ = _operator64(c, q, k, v, q2, k2, g, beta, None, 64)
    out = o / torch.sqrt((o * o).mean(-1, keepdim=True) + 1e-6) * p["gain"] * torch.sigmoid(p["z"])
    gr = dict(zip(names, torch.autograd.grad(out, [p[n] for n in names], st["dy"].double())))
    return {"out": out.detach(), **{"d" + n: gr[n] for n in names}}
