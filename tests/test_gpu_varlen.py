"""GPU parity of packed variable-length batches (tla_fwd_varlen /
tla_bwd_varlen): every packed sequence must give what the fp64 oracle gives
for that sequence alone, from its own initial state (the state restarts with
each sequence), including empty sequences, ragged last chunks and sequences
of several chunks, in training and in inference; a packed batch of equal lengths
must reproduce the fixed-length entry points bit for bit, and in inference every
packed sequence the call with that sequence alone."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import paper_2609_36529_amd as tla
from paper_2609_36529_amd import synth
from helpers import TOL_BF16, TOL_F32, dev, host64, rel_err

pytestmark = pytest.mark.gpu
SGLA, GDN = tla.SGLA, tla.GDN
NAMES = ("q", "k", "v", "q2", "k2", "g")
GRADS = ("dq", "dk", "dv", "dq2", "dk2", "dg", "dbeta", "ds0")
LENGTHS = [150, 0, 1, 64, 37, 65, 178]


def packed_case(variant, dtype, lengths, chunk=64, H=2, K=128, V=128, E=8, seed=31):
    """Packed inputs [1, total, H, .] for len(lengths) sequences, their
    offsets, per-sequence initial states, dO and final-state gradients."""
    total = int(sum(lengths))
    cfg = synth.Config("varlen", variant, 1, total, H, K, V, E, chunk, dtype, "softplus16",
                       variant == GDN, 0.0, seed)
    inp = synth.make_inputs(cfg)
    n = len(lengths)
    st = synth.make_inputs(dataclasses.replace(cfg, B=n, T=1, s0_std=0.02, seed=seed + 1))["s0"]
    dO = synth.make_dO(cfg, seed=seed + 2)
    rng = np.random.default_rng(seed + 3)
    dSf = torch.from_numpy(rng.standard_normal((n, H, E, K, V))).float()
    cu = torch.tensor(np.concatenate([[0], np.cumsum(lengths)]), dtype=torch.int32)
    return cfg, inp, st, dO, dSf, cu


def seq_slice(x, a, b):
    return None if x is None else synth.to64(x[:, a:b])


def oracle_per_sequence(variant, inp, s0, dO, dSf, cu):
    """Packed fp64 oracle results, each sequence run alone."""
    outs, sfs, grads = [], [], {k: [] for k in GRADS}
    for i in range(len(cu) - 1):
        a, b = int(cu[i]), int(cu[i + 1])
        s0i = synth.to64(s0[i:i + 1])
        dsi = synth.to64(dSf[i:i + 1])
        if b == a:  # an empty sequence passes its state through
            sfs.append(s0i[0])
            grads["ds0"].append(dsi[0])
            continue
        args = [seq_slice(inp[nm], a, b) for nm in NAMES]
        o, sf = oracle.fwd(variant, *args, seq_slice(inp["beta"], a, b), s0i)
        outs.append(o[0])
        sfs.append(sf[0])
        gr = oracle.bwd(variant, *args, seq_slice(inp["beta"], a, b), s0i, seq_slice(dO, a, b), dsi)
        for k in GRADS:
            if gr[k] is None:
                continue
            grads[k].append(gr[k][0])
    o = np.concatenate(outs, axis=0)[None]
    packed = {k: (np.concatenate(v, axis=0)[None] if k != "ds0" else np.stack(v))
              for k, v in grads.items() if v}
    return o, np.stack(sfs), packed


@pytest.mark.parametrize("variant", [SGLA, GDN])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_varlen_matches_each_sequence_alone(variant, dtype):
    cfg, inp, s0, dO, dSf, cu = packed_case(variant, dtype, LENGTHS)
    if dtype == "bf16":
        dSf = torch.zeros_like(dSf)  # as the bf16 backward workloads (bf16 state-gradient operand)
    tol = TOL_F32 if dtype == "f32" else TOL_BF16
    d = {k: dev(v) for k, v in inp.items()}
    cud = dev(cu)
    T = max(LENGTHS)
    o, sf, saved = tla.fwd(variant, d["q"], d["k"], d["v"], d["q2"], d["k2"], d["g"], d["beta"],
                           dev(s0), chunk=cfg.chunk, out_dtype=torch.float32, training=True,
                           cu_seqlens=cud, max_seqlen=T)
    gr = tla.bwd(variant, d["q"], d["k"], d["v"], d["q2"], d["k2"], d["g"], d["beta"], dev(s0),
                 dev(dO), saved, dS_final=dev(dSf), chunk=cfg.chunk, out_dtype=torch.float32,
                 cu_seqlens=cud, max_seqlen=T)
    torch.cuda.synchronize()
    ro, rsf, rg = oracle_per_sequence(variant, inp, s0, dO, dSf, cu)
    errs = {"o": rel_err(host64(o), ro), "s_final": rel_err(host64(sf), rsf)}
    for k in GRADS:
        if gr[k] is None:
            assert k not in rg
            continue
        got = host64(gr[k])
        assert np.all(np.isfinite(got)), k
        errs[k] = rel_err(got, rg[k])
    print(f"varlen variant={variant} {dtype}: " + " ".join(f"{k}={v:.1e}" for k, v in errs.items()),
          flush=True)
    bad = {k: v for k, v in errs.items() if v > tol}
    assert not bad, bad


@pytest.mark.parametrize("variant", [SGLA, GDN])
def test_varlen_equal_lengths_equals_fixed_length_bitwise(variant):
    n, L = 3, 150
    cfg = synth.Config("eq", variant, n, L, 2, 128, 128, 8, 64, "bf16", "softplus16",
                       variant == GDN, 0.02, 41)
    inp = synth.make_inputs(cfg)
    dO = synth.make_dO(cfg, seed=42)
    d = {k: dev(v) for k, v in inp.items()}
    o1, sf1, sv1 = tla.fwd(variant, d["q"], d["k"], d["v"], d["q2"], d["k2"], d["g"], d["beta"],
                           d["s0"], chunk=64, out_dtype=torch.float32, training=True)
    g1 = tla.bwd(variant, d["q"], d["k"], d["v"], d["q2"], d["k2"], d["g"], d["beta"], d["s0"],
                 dev(dO), sv1, chunk=64, out_dtype=torch.float32)
    pk = {k: (None if v is None else v.reshape((1, n * L) + tuple(v.shape[2:])))
          for k, v in d.items() if k != "s0"}
    cu = torch.arange(0, n * L + 1, L, dtype=torch.int32, device="cuda")
    o2, sf2, sv2 = tla.fwd(variant, pk["q"], pk["k"], pk["v"], pk["q2"], pk["k2"], pk["g"],
                           pk["beta"], d["s0"], chunk=64, out_dtype=torch.float32, training=True,
                           cu_seqlens=cu, max_seqlen=L)
    g2 = tla.bwd(variant, pk["q"], pk["k"], pk["v"], pk["q2"], pk["k2"], pk["g"], pk["beta"],
                 d["s0"], dev(dO).reshape(1, n * L, 2, 128), sv2, chunk=64,
                 out_dtype=torch.float32, cu_seqlens=cu, max_seqlen=L)
    torch.cuda.synchronize()
    assert torch.equal(o1.reshape(o2.shape), o2)
    assert torch.equal(sf1, sf2)
    for k in GRADS:
        if g1[k] is None:
            assert g2[k] is None
            continue
        assert torch.equal(g1[k].reshape(g2[k].shape), g2[k]), k


def test_varlen_all_empty_passes_states_through():
    cfg, inp, s0, dO, dSf, cu = packed_case(GDN, "bf16", [1], H=1)
    cu = torch.zeros(4, dtype=torch.int32)
    d = {k: dev(v) for k, v in inp.items()}
    s0 = torch.randn(3, 1, 8, 128, 128) * 0.02
    o, sf, _ = tla.fwd(GDN, d["q"][:, :0], d["k"][:, :0], d["v"][:, :0], d["q2"][:, :0],
                       d["k2"][:, :0], d["g"][:, :0], d["beta"][:, :0], dev(s0), chunk=64,
                       out_dtype=torch.float32, cu_seqlens=dev(cu), max_seqlen=1)
    torch.cuda.synchronize()
    assert torch.equal(sf.cpu(), s0)


# inference: an empty and a one-token sequence, ragged and whole chunks, and one
# longer than 17 chunks of 64
LONG = [150, 0, 1, 64, 37, 1093, 128]


@pytest.mark.parametrize("variant", [SGLA, GDN])
@pytest.mark.parametrize("K,chunk,E,H,V", [(128, 64, 8, 2, 128), (128, 64, 8, 4, 128), (128, 64, 4, 2, 64),
                                           (128, 64, 16, 2, 48), (128, 32, 8, 4, 128), (64, 32, 8, 6, 64)])
def test_varlen_inference(variant, K, chunk, E, H, V):
    """The inference forward over packed sequences (7 of them: 8 value columns a
    workgroup up to 128 / (7 V / 16) heads, 16 beyond; E = 16 always 8) against the
    oracle, and bit for bit against each sequence alone, which takes 8 columns."""
    cfg, inp, s0, _, _, cu = packed_case(variant, "bf16", LONG, chunk=chunk, H=H, K=K, V=V, E=E)
    d = {k: dev(v) for k, v in inp.items()}
    args = ("q", "k", "v", "q2", "k2", "g", "beta")
    s0d = dev(s0)
    o, sf, _ = tla.fwd(variant, *[d[n] for n in args], s0d, chunk=chunk, out_dtype=torch.float32,
                       cu_seqlens=dev(cu), max_seqlen=max(LONG))
    torch.cuda.synchronize()
    assert torch.isfinite(o).all() and torch.isfinite(sf).all()
    for i in range(len(LONG)):
        a, b = int(cu[i]), int(cu[i + 1])
        if a == b:
            assert torch.equal(sf[i], s0d[i])
            continue
        one = [None if d[n] is None else d[n][:, a:b].clone() for n in args]  # (aligned)
        o1, sf1, _ = tla.fwd(variant, *one, s0d[i:i + 1].clone(), chunk=chunk, out_dtype=torch.float32)
        torch.cuda.synchronize()
        assert torch.equal(o[:, a:b], o1) and torch.equal(sf[i:i + 1], sf1), i
        ro, rs = oracle.fwd(variant, *[seq_slice(inp[nm], a, b) for nm in NAMES],
                            seq_slice(inp["beta"], a, b), synth.to64(s0[i:i + 1]))
        eo, es = rel_err(host64(o1), ro), rel_err(host64(sf1), rs)
        print(f"varlen inference {variant=} {K=} {chunk=} {E=} {H=} T={b - a}: o {eo:.1e} s_final {es:.1e}",
              flush=True)
        assert eo <= TOL_BF16 and es <= TOL_BF16, (i, eo, es)
