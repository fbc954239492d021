"""The look-ahead forward (bf16 operands, K >= 64, E >= 4) at the edges of its
dispatch: lengths around a chunk and around the chunks that form W from their own
start state (every 16th), both workgroup widths (16 value columns, and 8 where
those would leave half of the chip idle), both variants, extreme gates, against
the fp64 oracle; the two widths bit for bit; sequences cut and resumed.  Bound
against the oracle: the bf16 parity bound of the other forward tests (max|err| /
RMS 2e-2, one bf16 rounding of the state operand per chunk)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_36529_amd as tla
from paper_2609_36529_amd import synth
from helpers import host64, oracle_fwd_heads, rel_err

pytestmark = pytest.mark.gpu
TOL = 2e-2


def _inputs(variant, B, T, H, K, V, E, C, seed=11):
    cfg = synth.Config("la", variant, B, T, H, K, V, E, C, "bf16", "softplus16", variant == 1, 0.02, seed)
    return synth.make_inputs(cfg)


def _fwd(variant, inp, C, s0=None):
    d = {k: (None if v is None else v.to("cuda")) for k, v in inp.items()}
    if s0 is not None:
        d["s0"] = s0
    o, sf, _ = tla.fwd(variant, d["q"], d["k"], d["v"], d["q2"], d["k2"], d["g"], d["beta"], d["s0"],
                       chunk=C, out_dtype=torch.float32)
    torch.cuda.synchronize()
    return o, sf


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("K,C,E,V", [(128, 64, 8, 128), (128, 64, 4, 48), (128, 64, 16, 32), (64, 32, 8, 64),
                                     (64, 64, 16, 16), (128, 32, 8, 16)])
@pytest.mark.parametrize("T", [1, 65, 1087])
def test_lengths(variant, K, C, E, V, T):
    inp = _inputs(variant, 1, T, 3, K, V, E, C)
    o, sf = _fwd(variant, inp, C)
    ro, rs = oracle.fwd(variant, *[synth.to64(inp[n]) for n in ("q", "k", "v", "q2", "k2", "g")],
                        synth.to64(inp["beta"]), synth.to64(inp["s0"]))
    eo, es = rel_err(host64(o), ro), rel_err(host64(sf), rs)
    print(f"{variant=} {K=} {C=} {E=} {V=} {T=}: o {eo:.2e} s_final {es:.2e}", flush=True)
    assert eo <= TOL and es <= TOL


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("K,C,E,V", [(128, 64, 8, 128), (128, 64, 4, 48), (128, 32, 8, 128), (64, 32, 8, 64)])
@pytest.mark.parametrize("chunks,tail", [(0, 1), (1, 0), (17, 5)])
def test_many_heads(variant, K, C, E, V, chunks, tail):
    """The 16-column workgroups against the oracle on the first and the last
    head: one position, one whole chunk, and past the chunk that forms its W from
    its own start state."""
    T, H = chunks * C + tail, 8
    B = 128 // (H * V // 16) + 1
    assert B * H * V // 16 > 128
    inp = _inputs(variant, B, T, H, K, V, E, C)
    o, sf = _fwd(variant, inp, C)
    assert torch.isfinite(o).all() and torch.isfinite(sf).all()
    for (b, h), (ro, rs) in oracle_fwd_heads(variant, inp, [(0, 0), (B - 1, H - 1)]).items():
        eo, es = rel_err(host64(o[b, :, h]), ro), rel_err(host64(sf[b, h]), rs)
        print(f"{variant=} {K=} {C=} {E=} {V=} {T=} head {(b, h)}: o {eo:.2e} s_final {es:.2e}", flush=True)
        assert eo <= TOL and es <= TOL


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("K,C,E", [(128, 64, 8), (128, 64, 16), (64, 32, 8)])
def test_extreme_gates(variant, K, C, E):
    """Log-gates of -1000 and log(2^-5) per token, inside a chunk, on its last
    position and on the first of the next: the tile factors exp(G_r - G_m),
    exp(G_m - G_c) and the cross-chunk decays stay finite and match the oracle."""
    inp = _inputs(variant, 1, 3 * C + 22, 2, K, 64, E, C)
    g = inp["g"].clone()
    g[:, ::5] = -1000.0
    g[:, 1::5] = float(np.log(2.0 ** -5))
    g[:, C - 1] = g[:, 2 * C] = -1000.0
    inp["g"] = g
    o, sf = _fwd(variant, inp, C)
    ro, rs = oracle.fwd(variant, *[synth.to64(inp[n]) for n in ("q", "k", "v", "q2", "k2", "g")],
                        synth.to64(inp["beta"]), synth.to64(inp["s0"]))
    eo, es = rel_err(host64(o), ro), rel_err(host64(sf), rs)
    print(f"{variant=} {K=} {C=} {E=}: o {eo:.2e} s_final {es:.2e}", flush=True)
    assert np.all(np.isfinite(host64(o))) and np.all(np.isfinite(host64(sf)))
    assert eo <= TOL and es <= TOL


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("K,C,E", [(128, 64, 8), (128, 64, 4), (128, 32, 8), (64, 32, 8)])
def test_widths_agree(variant, K, C, E):
    """The 8-column workgroups (few heads) and the 16-column ones run the same
    chunk recurrence, with the sums over slices in one order: a sequence gives
    the same bits alone (8 columns) and among others (16 columns), here past
    the chunk that forms its W from its own start state."""
    B, T, H, V = 5, 16 * C + 70, 8, 128
    inp = _inputs(variant, B, T, H, K, V, E, C)
    assert B * H * V // 16 > 128 >= H * V // 16  # the two sides of the rule
    o, sf = _fwd(variant, inp, C)
    one = {k: (None if v is None else v[1:2].contiguous()) for k, v in inp.items()}
    o1, sf1 = _fwd(variant, one, C)
    assert torch.equal(o[1:2], o1) and torch.equal(sf[1:2], sf1)


@pytest.mark.parametrize("C", [64, 32])
def test_resume_at_sync(C):
    """A sequence cut at a multiple of 16 chunks and resumed from the handed-on
    state repeats the uncut one bit for bit."""
    T = 16 * C
    inp = _inputs(1, 1, 2 * T + 37, 2, 128, 128, 8, C)
    o, sf = _fwd(1, inp, C)
    first = {k: (v if v is None or k == "s0" else v[:, :T].contiguous()) for k, v in inp.items()}
    _, mid = _fwd(1, first, C)
    rest = {k: (v if v is None or k == "s0" else v[:, T:].contiguous()) for k, v in inp.items()}
    o2, sf2 = _fwd(1, rest, C, s0=mid)
    assert torch.equal(o[:, T:], o2) and torch.equal(sf, sf2)
    assert np.all(np.isfinite(host64(o)))


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("path,E", [("inference", 8), ("inference", 16), ("training", 8), ("training", 16),
                                    ("f32", 8)])
def test_resume_elsewhere(variant, path, E):
    """Cut at another chunk boundary (8 chunks of 64) a sequence repeats the uncut
    one bit for bit, but for the GDN look-ahead forward: it forms the W of the first
    chunk from the bf16 operands of another state (that chunk's own start instead of
    the one before), each element of which is within 2^-9 of the fp32 state:
    operands at most 2^-8 apart, and so the results in the 2-norm (measured 4e-5)."""
    C, cut = 64, 512
    cfg = synth.Config("la", variant, 1, cut + 300, 4, 128, 128, E, C, "f32" if path == "f32" else "bf16",
                       "softplus16", variant == 1, 0.02, 11)
    inp = synth.make_inputs(cfg)

    def run(sl, s0):
        d = [None if inp[n] is None else inp[n][:, sl].contiguous().to("cuda")
             for n in ("q", "k", "v", "q2", "k2", "g", "beta")]
        o, sf, _ = tla.fwd(variant, *d, s0, chunk=C, out_dtype=torch.float32, training=path == "training")
        torch.cuda.synchronize()
        return o, sf

    s0 = inp["s0"].to("cuda")
    o, sf = run(slice(None), s0)
    _, mid = run(slice(0, cut), s0)
    o2, sf2 = run(slice(cut, None), mid)
    for x, y in ((o[:, cut:], o2), (sf, sf2)):
        d = ((x.double() - y.double()).norm() / x.double().norm()).item()
        print(f"{variant=} {path} {E=}: {d:.2e}", flush=True)
        assert d <= (2.0 ** -8 if variant == 1 and path == "inference" else 0.0)
