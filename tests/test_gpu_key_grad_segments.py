"""The contraction's key gradient where a segment holds three chunks and the last one is cut: the
statistics' blocks, H = X + X^T at a segment's start, its update inside the segment and none after
the segment's first chunk.  12 x 8 heads of 5 chunks make segments of 3 and 2.  Bar of the training
step: max |gpu - ref| / max |ref| <= 2e-2 (bf16 io) or 1e-4 (fp32 io)."""
import pytest
import torch

from gpu_helpers import TOL, nerr, np64
from oracle import ccq_oracle as O
from paper_2606_01294_amd import ccq
from paper_2606_01294_amd.inputs import GDN, make_inputs, to_device, to_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,dk", [(torch.bfloat16, 64), (torch.bfloat16, 128), (torch.bfloat16, 256),
                                      (torch.float32, 64)])
@pytest.mark.parametrize("centered", [True, False])
def test_key_gradient_over_segments(dtype, dk, centered):
    print("key gradient", dtype, dk, centered, flush=True)
    d = make_inputs(GDN, 12, 290, 8, dk, 64, dtype, seed=dk, keys="meanshift", lam="random", with_dO=True)
    g = to_device(d)
    out = ccq.ccq_fwd_bwd(g["q"], g["k"], g["v"], g["logalpha"], g["lam"], g["dO"], backbone=ccq.CCQ_GDN,
                          beta=g["beta"], centered=centered)
    torch.cuda.synchronize()
    # two of the sequences against the oracle: each is independent of the others
    for b in (0, 11):
        f = {n: x[b:b + 1] for n, x in to_f64(d).items()}
        ref = O.gdn_fwd_bwd(f["q"], f["k"], f["v"], f["logalpha"], f["beta"], f["lam"], f["dO"], centered=centered)
        e = nerr(np64(out["dk"][b:b + 1]), ref["dk"])
        print("  ", b, "%.2e" % e, flush=True)
        assert e <= TOL[dtype], (b, e)
