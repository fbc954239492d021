"""The reverse recurrence with two key slices a tile (bf16 operands, E = 16,
K >= 64) where its 8-column tiles meet the edges: one and an odd number of
16-column blocks, both variants, with and without a final-state gradient, a
ragged last chunk; and the sGLA state contractions without dW.  Bound: the bf16
parity bound of the other backward tests (max|err| / RMS 2e-2)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_36529_amd as tla
from paper_2609_36529_amd import synth
from helpers import host64, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("variant", [0, 1])
@pytest.mark.parametrize("final", [False, True])
@pytest.mark.parametrize("K,C,E,V", [(128, 64, 16, 16), (128, 64, 16, 48), (64, 64, 16, 32), (128, 64, 8, 16)])
def test_backward(variant, final, K, C, E, V):
    B, T, H = 1, 139, 2
    cfg = synth.Config("pk", variant, B, T, H, K, V, E, C, "bf16", "softplus16", variant == 1, 0.02, 31)
    inp = synth.make_inputs(cfg)
    d = {k: (None if v is None else v.to("cuda")) for k, v in inp.items()}
    dO = synth.make_dO(cfg, seed=5)
    rng = np.random.Generator(np.random.PCG64(9))
    dSf = torch.from_numpy(rng.standard_normal((B, H, E, K, V))).float() if final else None
    args = (d["q"], d["k"], d["v"], d["q2"], d["k2"], d["g"], d["beta"], d["s0"])
    _, _, saved = tla.fwd(variant, *args, chunk=C, out_dtype=torch.float32, training=True)
    gr = tla.bwd(variant, *args, dO.to("cuda"), saved, dS_final=None if dSf is None else dSf.to("cuda"),
                 chunk=C, out_dtype=torch.float32)
    torch.cuda.synchronize()
    ref = oracle.bwd(variant, *[synth.to64(inp[n]) for n in ("q", "k", "v", "q2", "k2", "g")],
                     synth.to64(inp["beta"]), synth.to64(inp["s0"]), synth.to64(dO), synth.to64(dSf))
    for key in ("dq", "dk", "dv", "dq2", "dk2", "dg", "dbeta", "ds0"):
        if gr[key] is None:
            continue
        err = rel_err(host64(gr[key]), ref[key])
        print(f"{variant=} {final=} {K=} {E=} {V=} {key}: {err:.2e}", flush=True)
        assert err <= 2e-2, (key, err)


@pytest.mark.parametrize("variant", [0, 1])
def test_widths_agree(variant):
    """K = 64 without a final-state gradient takes 8-column workgroups for few
    heads and 16-column ones for many: the gradients of a sequence have the same
    bits alone and among others."""
    K, C, E, V, H, B, T = 64, 64, 16, 64, 8, 5, 139
    cfg = synth.Config("pk", variant, B, T, H, K, V, E, C, "bf16", "softplus16", variant == 1, 0.02, 37)
    assert B * H * V // 16 > 128 >= H * V // 16  # the two sides of the rule
    inp = synth.make_inputs(cfg)
    inp["dO"] = synth.make_dO(cfg, seed=5)
    got = []
    for pick in (slice(0, B), slice(1, 2)):
        d = {k: (None if v is None else v[pick].contiguous().to("cuda")) for k, v in inp.items()}
        args = (d["q"], d["k"], d["v"], d["q2"], d["k2"], d["g"], d["beta"], d["s0"])
        _, _, saved = tla.fwd(variant, *args, chunk=C, training=True)
        got.append(tla.bwd(variant, *args, d["dO"], saved, chunk=C, out_dtype=torch.float32))
    torch.cuda.synchronize()
    for key, x in got[0].items():
        if x is not None:
            assert torch.equal(x[1:2], got[1][key]), key
