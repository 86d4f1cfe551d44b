"""The WY form of the Gated DeltaNet state pass (gdn_wy_state_kernel): parity of the calls
that take it (from 4 chunks at dk = 128, 8 or 16 at dk = 256) with the oracle, at the edges
of its rule and of its tiles, and the load counts its loaders wait on.

Bar: max |gpu - ref| / max |ref| <= 2e-2 (bf16 io) per tensor, as every bf16 call; the
statistics, which do not go through this pass, have bars of their own elsewhere.
"""
import os
import re
import subprocess
import sys
import tempfile

import numpy as np
import pytest
import torch

from gpu_helpers import TOL, nerr, np64
from oracle import ccq_oracle as O
from paper_2606_01294_amd import build as B
from paper_2606_01294_amd import ccq
from paper_2606_01294_amd.inputs import GDN, make_inputs, to_device, to_f64

BF16 = torch.bfloat16
BAR = TOL[BF16]


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def init(rng, n, H, dk, dv):
    keys = rng.standard_normal((n, H, 30, dk))
    keys /= np.linalg.norm(keys, axis=-1, keepdims=True)
    return [x.astype(np.float32) for x in (rng.standard_normal((n, H, dv, dk)) * 0.2,
                                           np.einsum("bhnc,bhnd->bhcd", keys, keys) / 30,
                                           keys.mean(axis=2))]


# B, T, H, dk, dv, initial states: the first chunk count of the rule (and one below it), one,
# two and four value tiles per workgroup, whole and cut last chunks
CASES = [
    (1, 192, 2, 128, 64, False), (1, 193, 2, 128, 64, True), (1, 256, 3, 128, 128, False),
    (1, 448, 2, 256, 256, False), (1, 449, 2, 256, 256, True), (3, 513, 5, 256, 64, True),
    (3, 1023, 8, 256, 256, False), (1, 600, 3, 256, 512, False), (5, 320, 8, 128, 128, True),
    (5, 257, 8, 128, 256, False),
]


@pytest.mark.gpu
@pytest.mark.parametrize("B_,T,H,dk,dv,cont", CASES)
def test_forward_matches_oracle(B_, T, H, dk, dv, cont):
    say("gdn_wy forward", B_, T, H, dk, dv, cont)
    d = make_inputs(GDN, B_, T, H, dk, dv, BF16, seed=T + dv, keys="aniso", lam="random")
    kw = {}
    if cont:
        S0, C0, mu0 = init(np.random.default_rng(T), B_, H, dk, dv)
        kw = dict(S0=S0, C0=C0, mu0=mu0, t0=37)
    g, f = to_device(d), to_f64(d)
    out = ccq.ccq_gdn_fwd(g["q"], g["k"], g["v"], g["logalpha"], g["beta"], g["lam"],
                          **{n: torch.from_numpy(x).cuda() if n != "t0" else x for n, x in kw.items()})
    torch.cuda.synchronize()
    ref = O.fwd(f["q"], f["k"], f["v"], f["logalpha"], f["lam"], beta=f["beta"], backbone=O.GDN, **kw)
    for key in ("o", "ST", "CT", "muT"):
        e = nerr(np64(out[key]), ref[key])
        say("  ", key, "%.2e" % e)
        assert e <= BAR, (key, e)


@pytest.mark.gpu
@pytest.mark.parametrize("lens,H,dk,dv", [([600, 0, 1, 512, 64, 513], 2, 256, 256),
                                          ([300, 256, 3, 0, 255], 4, 128, 256)])
def test_packed_batch_matches_oracle(lens, H, dk, dv):
    say("gdn_wy packed", lens, H, dk, dv)
    T = max(lens)
    d = make_inputs(GDN, len(lens), T, H, dk, dv, BF16, seed=7, keys="aniso", lam="random")
    p = {n: torch.cat([x[b, :L] for b, L in enumerate(lens)], dim=0).contiguous() for n, x in d.items()}
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    S0, C0, mu0 = init(np.random.default_rng(3), len(lens), H, dk, dv)
    g, f = to_device(p), to_f64(p)
    out = ccq.ccq_gdn_fwd_varlen(g["q"], g["k"], g["v"], g["logalpha"], g["beta"], g["lam"],
                                 torch.from_numpy(cu).cuda(), T, S0=torch.from_numpy(S0).cuda(),
                                 C0=torch.from_numpy(C0).cuda(), mu0=torch.from_numpy(mu0).cuda(), t0=30)
    torch.cuda.synchronize()
    ref = O.varlen_fwd(f["q"], f["k"], f["v"], f["logalpha"], f["lam"], cu, beta=f["beta"],
                       backbone=O.GDN, S0=S0, C0=C0, mu0=mu0, t0=30)
    for key in ("o", "ST", "CT", "muT"):
        e = nerr(np64(out[key]), ref[key])
        say("  ", key, "%.2e" % e)
        assert e <= BAR, (key, e)


@pytest.mark.gpu
@pytest.mark.parametrize("T,H,dk,dv", [(520, 3, 256, 256), (270, 2, 128, 64)])
def test_raw_keys_match_the_two_passes(T, H, dk, dv):
    """The row scales enter W through the normalised rows and K through the coefficients: the
    same results as normalising first, up to bf16 roundings of either."""
    say("gdn_wy raw", T, H, dk, dv)
    gen = torch.Generator().manual_seed(T)
    d = make_inputs(GDN, 2, T, H, dk, dv, BF16, seed=T, keys="iso", lam="random")
    q = torch.randn(2, T, H, dk, generator=gen).to(BF16).cuda()
    k = (3.0 * torch.randn(2, T, H, dk, generator=gen)).to(BF16).cuda()
    w = (torch.randn(H, H * dk, generator=gen) / (H * dk) ** 0.5).cuda()
    b = torch.randn(H, generator=gen).cuda()
    g = to_device(d)
    raw = ccq.ccq_fwd_raw(q, k, w, b, g["v"], g["logalpha"], beta=g["beta"], backbone=ccq.CCQ_GDN)
    p = ccq.ccq_prep(q, k, w, b)
    two = ccq.ccq_gdn_fwd(p["q"], p["k"], g["v"], g["logalpha"], g["beta"], p["lam"])
    torch.cuda.synchronize()
    for key in ("o", "ST"):
        e = nerr(np64(raw[key]), np64(two[key]))
        say("  ", key, "%.2e" % e)
        assert e <= BAR, (key, e)


@pytest.mark.gpu
@pytest.mark.parametrize("B_,T,H,dk,dv", [(1, 577, 2, 256, 128), (2, 300, 3, 128, 64), (1, 512, 1, 256, 64)])
def test_training_step_matches_oracle(B_, T, H, dk, dv):
    say("gdn_wy training", B_, T, H, dk, dv)
    d = make_inputs(GDN, B_, T, H, dk, dv, BF16, seed=T, keys="aniso", lam="random", with_dO=True)
    g, f = to_device(d), to_f64(d)
    out = ccq.ccq_fwd_bwd(g["q"], g["k"], g["v"], g["logalpha"], g["lam"], g["dO"],
                          backbone=ccq.CCQ_GDN, beta=g["beta"])
    torch.cuda.synchronize()
    ref = O.gdn_fwd_bwd(f["q"], f["k"], f["v"], f["logalpha"], f["beta"], f["lam"], f["dO"])
    ref["dg"] = ref.pop("dlogalpha")
    for key in ("o", "dq", "dk", "dv", "dg", "dbeta", "dlam"):
        e = nerr(np64(out[key]), ref[key])
        say("  ", key, "%.2e" % e)
        assert e <= BAR, (key, e)


@pytest.mark.parametrize("dk,npr", [(128, 1), (128, 2), (128, 4), (256, 1), (256, 2)])
def test_loader_loops_issue_the_counted_loads(dk, npr, wy_asm):
    """The loaders wait on counts of loads in flight (per wave: NWL of a W slot and NKL of a K
    slot, or NVL of a V slot), so their chunk loops must hold exactly those loads and no other
    vector memory instruction, and no register may be spilled anywhere in the kernel."""
    sym = "_ZN3ccq19gdn_wy_state_kernelILi%dELi%dEEEvNS_7GdnArgsE" % (dk, npr)
    body = wy_asm.split("\n" + sym + ":", 1)[1].split(".Lfunc_end", 1)[0].split("\n")
    assert not any(x.strip().startswith(("scratch_", "buffer_")) for x in body)
    nwl, nkl, nvl = 64 * dk * 2 // 4096 + 2, 64 * dk * 2 // 4096, 2 * npr + 1
    label = {m.group(1): i for i, x in enumerate(body) for m in [re.match(r"(\.LBB\d+_\d+):", x)] if m}
    loops = {}
    for i, x in enumerate(body):
        m = re.search(r"s_c?branch\w*\s+(\.LBB\d+_\d+)", x)
        if m and label[m.group(1)] <= i:
            loops[label[m.group(1)]] = max(i, loops.get(label[m.group(1)], 0))
    counts = []
    for h, e in loops.items():
        ins = [x.split(";")[0].split() for x in body[h:e + 1]]
        ins = [x[0] for x in ins if x and not x[0].startswith(".")]
        if not any("mfma" in x for x in ins):
            vm = [x for x in ins if x.startswith(("global_", "flat_"))]
            counts.append((vm.count("global_load_lds_dwordx4"), len(vm)))
    assert (nwl + nkl, nwl + nkl) in counts, counts  # loaders of W and K
    assert (nvl, nvl) in counts, counts              # V loader


@pytest.fixture(scope="module")
def wy_asm():
    src = os.path.join(B.CSRC, "ccq_gdn_wy.hip")
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "wy.s")
        cmd = [B._hipcc()] + B.COMMON + B.DEVICE + ["--cuda-device-only", "-S", src, "-o", out]
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            pytest.skip("hipcc unavailable for gfx950 here: " + res.stderr[-300:])
        return open(out).read()
