"""The training step on packed batches read in place: parity of every gradient with the oracle
on lengths that mix empty, one-token, whole-chunk and many-chunk sequences, a bound above the
longest length, and a bound below it (the sequence is cut there; its later rows are neither
read for the result nor written).  Bar as every training test: max |gpu - ref| / max |ref| <=
1e-4 (fp32 io) or 2e-2 (bf16 io) per tensor."""
import numpy as np
import pytest
import torch

from gpu_helpers import TOL, nerr, np64
from oracle import ccq_oracle as O
from paper_2606_01294_amd import ccq
from paper_2606_01294_amd.inputs import GDN, GLA, make_inputs, to_f64

pytestmark = pytest.mark.gpu
F32, BF16 = torch.float32, torch.bfloat16

# backbone, dtype, lengths, H, dk, dv, length bound
CASES = [(GLA, BF16, [300, 0, 64, 129, 1], 2, 128, 256, 337), (GLA, F32, [65, 190, 0, 3], 3, 64, 64, 190),
         (GDN, BF16, [300, 64, 0, 1, 450], 2, 256, 256, 450), (GDN, BF16, [129, 600, 63], 3, 128, 128, 640),
         (GDN, F32, [0, 130, 64], 2, 64, 128, 130),
         (GLA, BF16, [200, 150, 220], 2, 64, 128, 130), (GDN, BF16, [400, 70, 333], 1, 128, 64, 100)]


@pytest.mark.parametrize("backbone", [GLA, GDN])
@pytest.mark.parametrize("side", [False, True])
def test_outputs_may_take_the_place_of_inputs(backbone, side):
    """Every gradient over the input it belongs to, o over dO: the same results as into new tensors,
    on the current stream and on another one."""
    print("packed training in place", backbone, side, flush=True)
    lens, H, dk, dv = [300, 64, 0, 450], 2, 128, 256
    d = make_inputs(backbone, len(lens), max(lens), H, dk, dv, BF16, seed=3, keys="aniso", lam="random", with_dO=True)
    g = {n: torch.cat([x[b, :L] for b, L in enumerate(lens)], dim=0).contiguous().cuda() for n, x in d.items()}
    cu = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)).cuda()
    gate = "g" if backbone == GLA else "logalpha"

    def step(t, **kw):
        return ccq.ccq_fwd_bwd_varlen(t["q"], t["k"], t["v"], t[gate], t["lam"], t["dO"], cu, max(lens),
                                      backbone=backbone, beta=t.get("beta"), **kw)
    want = step(g)
    t = {n: x.clone() for n, x in g.items()}
    out = dict(o=t["dO"], dq=t["q"], dk=t["k"], dv=t["v"], dg=t[gate], dlam=t["lam"])
    if backbone == GDN:
        out["dbeta"] = t["beta"]
    torch.cuda.synchronize()
    got = step(t, out=out, stream=torch.cuda.Stream() if side else None)
    torch.cuda.synchronize()
    for n in want:
        assert got[n].data_ptr() == out[n].data_ptr()
        assert torch.equal(got[n], want[n]), n


@pytest.mark.parametrize("backbone,dtype,lens,H,dk,dv,bound", CASES)
def test_packed_training_matches_oracle(backbone, dtype, lens, H, dk, dv, bound):
    print("packed training", backbone, dtype, lens, H, dk, dv, bound, flush=True)
    T = max(lens)
    d = make_inputs(backbone, len(lens), T, H, dk, dv, dtype, seed=T, keys="aniso", lam="random", with_dO=True)
    p = {n: torch.cat([x[b, :L] for b, L in enumerate(lens)], dim=0).contiguous() for n, x in d.items()}
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    g = {n: x.cuda() for n, x in p.items()}
    gate = g["g"] if backbone == GLA else g["logalpha"]
    like = dict(o=g["v"], dq=g["q"], dk=g["k"], dv=g["v"], dg=gate, dlam=g["lam"])
    if backbone == GDN:
        like["dbeta"] = g["beta"]
    mark = 7.0
    out = {n: torch.full_like(x, mark) for n, x in like.items()}
    out = ccq.ccq_fwd_bwd_varlen(g["q"], g["k"], g["v"], gate, g["lam"], g["dO"], torch.from_numpy(cu).cuda(), bound,
                                 backbone=backbone, beta=g.get("beta"), out=out)
    torch.cuda.synchronize()
    # the reference on each sequence cut at the bound
    f = to_f64(p)
    rows = np.concatenate([np.arange(cu[b], cu[b] + min(L, bound)) for b, L in enumerate(lens)]).astype(np.int64)
    cut = {n: x[rows] for n, x in f.items()}
    cuc = np.concatenate([[0], np.cumsum([min(L, bound) for L in lens])])
    ref = O.varlen_fwd_bwd(cut["q"], cut["k"], cut["v"], cut["g" if backbone == GLA else "logalpha"], cut["lam"],
                           cut["dO"], cuc, beta=cut.get("beta"), backbone=O.GLA if backbone == GLA else O.GDN)
    rest = np.setdiff1d(np.arange(cu[-1]), rows)
    for key in like:
        got = np64(out[key])
        e = nerr(got[rows], ref[key])
        print("  ", key, "%.2e" % e, flush=True)
        assert e <= TOL[dtype], (key, e)
        assert np.all(got[rest] == mark), key
