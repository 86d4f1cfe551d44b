"""The GLA forward whose state pass runs in several segments: parity with the oracle where segments
end in a cut chunk, with initial states, gates in either type and packed batches that leave segments
empty.  Bar: max |gpu - ref| / max |ref| <= 2e-2 per tensor (bf16 io).  And one segment where the
rule gives one."""
import numpy as np
import pytest
import torch

from bench import gla_seg  # the library's rule
from gpu_helpers import TOL, nerr, np64
from oracle import ccq_oracle as O
from paper_2606_01294_amd import ccq
from paper_2606_01294_amd.inputs import GLA, make_inputs, to_device, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,H,dk,dv,gate,cont", [
    ([577, 0, 300, 64], 2, 64, 128, torch.bfloat16, True), ([1025], 4, 128, 256, torch.float32, False),
    ([520, 511, 1], 2, 128, 512, torch.bfloat16, False), ([2000] * 4, 8, 128, 256, torch.bfloat16, True)])
def test_segments_match_oracle(lens, H, dk, dv, gate, cont):
    print("gla segments", lens, H, dk, dv, gate, cont, flush=True)
    T = max(lens)
    assert gla_seg(len(lens) * H, -(-T // 64), dk, dv) > 0
    d = make_inputs(GLA, len(lens), T, H, dk, dv, torch.bfloat16, gate_dtype=gate, seed=T, keys="aniso", lam="random")
    p = {n: torch.cat([x[b, :L] for b, L in enumerate(lens)], dim=0).contiguous() for n, x in d.items()}
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    kw, gkw = {}, {}
    if cont:
        rng = np.random.default_rng(1)
        keys = rng.standard_normal((len(lens), H, 30, dk)) / dk ** 0.5
        kw = dict(S0=(rng.standard_normal((len(lens), H, dv, dk)) * 0.2).astype(np.float32),
                  C0=(np.einsum("bhnc,bhnd->bhcd", keys, keys) / 30).astype(np.float32),
                  mu0=keys.mean(axis=2).astype(np.float32))
        gkw = dict({n: torch.from_numpy(x).cuda() for n, x in kw.items()}, t0=30)
        kw["t0"] = 30
    g, f = {n: x.cuda() for n, x in p.items()}, to_f64(p)
    out = ccq.ccq_gla_fwd_varlen(g["q"], g["k"], g["v"], g["g"], g["lam"], torch.from_numpy(cu).cuda(), T, **gkw)
    torch.cuda.synchronize()
    ref = O.varlen_fwd(f["q"], f["k"], f["v"], f["g"], f["lam"], cu, backbone=O.GLA, **kw)
    for key in ("o", "ST"):
        e = nerr(np64(out[key]), ref[key])
        print("  ", key, "%.2e" % e, flush=True)
        assert e <= TOL[torch.bfloat16], (key, e)


def test_training_output_equals_a_forward_of_one_segment_bit_for_bit():
    """A training step runs one segment.  So does the forward at 64 heads of 28 chunks (dk = 128, dv =
    256), where a second segment would round the later states to bf16 in two parts."""
    assert gla_seg(64, 28, 128, 256) == 0
    print("gla one segment", flush=True)
    d = make_inputs(GLA, 8, 1792, 8, 128, 256, torch.bfloat16, seed=28, keys="aniso", lam="random", with_dO=True)
    g = to_device(d)
    fwd = ccq.ccq_gla_fwd(g["q"], g["k"], g["v"], g["g"], g["lam"])
    out = ccq.ccq_fwd_bwd(g["q"], g["k"], g["v"], g["g"], g["lam"], g["dO"])
    torch.cuda.synchronize()
    assert torch.equal(out["o"], fwd["o"])
