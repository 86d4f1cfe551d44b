"""Kernels that split their work differently where there is little of it: the segment prefix of
the key statistics (segments over the waves of a workgroup with few heads) and the
pre-processing pass (one token per wave up to 2048 tokens, or 1024 with the most heads, and the
order of its loads above 8192).  Parity with the oracle on both
sides of each rule; fp32 io is held to 1e-4 and bf16 rows to 2e-2 of the largest value, as in
the other parity tests."""
import numpy as np
import pytest
import torch

from gpu_helpers import nerr, np64
from oracle import ccq_oracle as O
from paper_2606_01294_amd import ccq
from paper_2606_01294_amd.inputs import GLA, make_inputs, to_f64

pytestmark = pytest.mark.gpu


# lengths (packed), heads, dk: four segments or more of two chunks, in counts that eight waves
# share evenly and unevenly, an empty and a one-token sequence; at most 256 workgroups of the
# plain form (B H dk^2 / 1024), and more (the plain form)
@pytest.mark.parametrize("lens,H,dk", [([1205, 0, 1, 449], 1, 64), ([1024], 2, 128), ([130, 513], 16, 64),
                                       ([700] * 5, 13, 64)])
@pytest.mark.parametrize("cont", [False, True])
def test_segment_prefix(lens, H, dk, cont):
    print("segment prefix", lens, H, dk, cont, flush=True)
    T = max(lens)
    d = make_inputs(GLA, len(lens), T, H, dk, 64, torch.float32, seed=T, keys="meanshift", lam="random")
    p = {n: torch.cat([x[b, :L] for b, L in enumerate(lens)], dim=0).contiguous() for n, x in d.items()}
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    kw, gkw = {}, {}
    if cont:
        rng = np.random.default_rng(1)
        keys = rng.standard_normal((len(lens), H, 30, dk)) / dk ** 0.5
        kw = dict(S0=(rng.standard_normal((len(lens), H, 64, dk)) * 0.2).astype(np.float32),
                  C0=(np.einsum("bhnc,bhnd->bhcd", keys, keys) / 30).astype(np.float32),
                  mu0=keys.mean(axis=2).astype(np.float32))
        gkw = dict({n: torch.from_numpy(x).cuda() for n, x in kw.items()}, t0=30)
        kw["t0"] = 30
    g, f = {n: x.cuda() for n, x in p.items()}, to_f64(p)
    out = ccq.ccq_gla_fwd_varlen(g["q"], g["k"], g["v"], g["g"], g["lam"], torch.from_numpy(cu).cuda(), T, **gkw)
    torch.cuda.synchronize()
    ref = O.varlen_fwd(f["q"], f["k"], f["v"], f["g"], f["lam"], cu, backbone=O.GLA, **kw)
    for key in ("o", "ST", "CT", "muT"):
        e = nerr(np64(out[key]), ref[key])
        print("  ", key, "%.2e" % e, flush=True)
        assert e <= 1e-4, (key, e)


@pytest.mark.parametrize("T,H,dk", [(T, H, dk) for H, dk in ((8, 256), (3, 64)) for T in (1, 3, 5, 2048, 2049, 2061)] +
                         [(1024, 16, 64), (1025, 15, 64), (8192, 2, 64), (8193, 4, 128)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_preprocessing_token_split(T, H, dk, dtype):
    print("preprocessing", T, H, dk, dtype, flush=True)
    gen = torch.Generator().manual_seed(T)
    q = torch.randn(1, T, H, dk, generator=gen).to(dtype)
    k = torch.randn(1, T, H, dk, generator=gen).to(dtype)
    w = torch.randn(H, H * dk, generator=gen) / (H * dk) ** 0.5
    b = torch.randn(H, generator=gen)
    out = ccq.ccq_prep(q.cuda(), k.cuda(), w.cuda(), b.cuda())
    torch.cuda.synchronize()
    ref = O.prep(q.double().numpy(), k.double().numpy(), w.double().numpy(), b.double().numpy())
    bar = 2e-2 if dtype == torch.bfloat16 else 1e-4
    for key in ("q", "k"):
        assert nerr(np64(out[key]), ref[key]) <= bar, key
    assert nerr(np64(out["lam"]), ref["lam"]) <= 1e-4
