"""The look-ahead forward (bf16 operands, K >= 64) at the edges of its dispatch:
lengths around a chunk and around the chunks that form W from their own start
state (every 16th), both workgroup widths (16 value columns, and 8 where those
would leave half of the chip idle), both variants, against the fp64 oracle.
Bound: the bf16 parity bound of the other forward tests (max|err| / RMS 2e-2,
one bf16 rounding of the state operand per chunk)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_36529_amd as tla
from paper_2609_36529_amd import synth
from helpers import host64, rel_err

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
