"""The Gated DeltaNet state pass with the waves in roles (gdn_state_roles_kernel, bf16 with dk = 128
and 256): parity with the oracle from one chunk on and at the edges of its tiles; the same bits
whatever the value split and in a training step as in the forward; and its error where the state
predicts the values.

Bar: max |gpu - ref| / max |ref| <= 2e-2 (bf16 io) per tensor, as every bf16 call; the
statistics, which do not go through this pass, have bars of their own elsewhere.
"""
import sys

import numpy as np
import pytest
import torch

from gpu_helpers import TOL, nerr, np64
from oracle import ccq_oracle as O
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


# B, T, H, dk, dv, initial states: one, two (fewer than the ring's slots) and more chunks, whole and
# cut last ones; one, two and four value tiles per workgroup
CASES = [
    (1, 1, 2, 256, 64, True), (1, 65, 2, 128, 64, True), (2, 128, 8, 256, 512, False), (8, 100, 8, 128, 256, True),
    (1, 192, 2, 128, 64, False), (1, 193, 2, 128, 64, True), (1, 256, 3, 128, 128, False),
    (1, 448, 2, 256, 256, False), (1, 449, 2, 256, 256, True), (3, 513, 5, 256, 64, True),
    (3, 1023, 8, 256, 256, False), (1, 600, 3, 256, 512, False), (5, 320, 8, 128, 128, True),
    (5, 257, 8, 128, 256, False),
]


@pytest.mark.gpu
@pytest.mark.parametrize("B_,T,H,dk,dv,cont", CASES)
def test_forward_matches_oracle(B_, T, H, dk, dv, cont):
    say("gdn_roles forward", B_, T, H, dk, dv, cont)
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
    say("gdn_roles packed", lens, H, dk, dv)
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
    """The row scales enter through the coefficients that multiply key rows: the same results as
    normalising first, up to bf16 roundings of either."""
    say("gdn_roles raw", T, H, dk, dv)
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
    say("gdn_roles training", B_, T, H, dk, dv)
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


def gdn_call(d):
    g = to_device(d)
    out = ccq.ccq_gdn_fwd(g["q"], g["k"], g["v"], g["logalpha"], g["beta"], g["lam"])
    torch.cuda.synchronize()
    return out


# One value tile per workgroup, and two or four with more heads: the first sequence's final state is
# the same bit for bit (at dk = 128 below 1024 tiles, from where the features' sum has another order).
@pytest.mark.gpu
@pytest.mark.parametrize("B_,T,H,dk,dv", [(5, 330, 4, 256, 256), (5, 191, 8, 128, 128), (5, 256, 8, 128, 256)])
def test_final_state_does_not_depend_on_the_value_split(B_, T, H, dk, dv):
    say("gdn_roles bits", B_, T, H, dk, dv)
    d = make_inputs(GDN, B_, T, H, dk, dv, BF16, seed=T + dv, keys="aniso", lam="random")
    one = gdn_call({n: x[:1].contiguous() for n, x in d.items()})
    assert torch.equal(gdn_call(d)["ST"][:1], one["ST"])


# A training step stores every state, a forward one per output group; the rest is the same kernels.
@pytest.mark.gpu
@pytest.mark.parametrize("B_,T,H,dk,dv", [(4, 1030, 8, 256, 256), (1, 600, 2, 256, 256), (5, 260, 8, 128, 256),
                                          (8, 300, 8, 128, 256)])
def test_training_output_equals_the_forward_bit_for_bit(B_, T, H, dk, dv):
    say("gdn_roles training bits", B_, T, H, dk, dv)
    d = make_inputs(GDN, B_, T, H, dk, dv, BF16, seed=T, keys="aniso", lam="random", with_dO=True)
    g = to_device(d)
    fwd = ccq.ccq_gdn_fwd(g["q"], g["k"], g["v"], g["logalpha"], g["beta"], g["lam"])
    out = ccq.ccq_fwd_bwd(g["q"], g["k"], g["v"], g["logalpha"], g["lam"], g["dO"], backbone=ccq.CCQ_GDN,
                          beta=g["beta"])
    torch.cuda.synchronize()
    assert torch.equal(out["o"], fwd["o"])


def emulated_state(k, v, beta):
    """S_T of one head without decay, in 64 bits but for the roundings to bf16 that the state pass
    has by design: Tm, S_r and R as operands, U as the update's operand."""
    def bf(x):
        return torch.from_numpy(x).to(BF16).double().numpy()
    T, dk = k.shape
    S = np.zeros((v.shape[1], dk))
    for r in range(0, T, 64):
        K, V, b = k[r:r + 64], v[r:r + 64], beta[r:r + 64, None]
        A = np.tril(b * (K @ K.T), -1)
        Tm = np.linalg.inv(np.eye(len(K)) + A)
        U = bf(Tm) @ bf(b * (V - K @ bf(S).T))
        S = S + bf(U).T @ K
    return S


# Values that the state predicts, v = M k, and no decay: V - K S^T cancels, so a rounding of either
# term ahead of the cancellation shows.  The bar is the error of the emulation above plus a tenth
# (this pass measures 0.99 to 1.01 of it; with W = -Tm diag(beta e^gamma) K rounded to bf16, U =
# Tb V + W S^T, it is 1.3 to 1.4).
@pytest.mark.gpu
@pytest.mark.parametrize("dk", [128, 256])
def test_error_where_the_state_predicts_the_values(dk):
    say("gdn_roles precision", dk)
    T, H, dv = 1024, 4, 64
    rng = np.random.default_rng(dk)
    k = rng.standard_normal((1, T, H, dk))
    k = torch.from_numpy(k / np.linalg.norm(k, axis=-1, keepdims=True)).to(BF16)
    M = rng.standard_normal((H, dv, dk))
    v = torch.from_numpy(np.einsum("hvc,bthc->bthv", M, k.double().numpy())).to(BF16)
    beta = torch.from_numpy(rng.uniform(0.3, 1.0, (1, T, H))).float()
    d = dict(q=k.clone(), k=k, v=v, logalpha=torch.zeros(1, T, H), beta=beta, lam=torch.zeros(1, T, H))
    ST = np64(gdn_call(d)["ST"])
    f = to_f64(d)
    ref = O.fwd(f["q"], f["k"], f["v"], f["logalpha"], f["lam"], beta=f["beta"], backbone=O.GDN)["ST"]
    emu = np.stack([emulated_state(f["k"][0, :, h], f["v"][0, :, h], f["beta"][0, :, h]) for h in range(H)])
    e, bar = np.linalg.norm(ST - ref), np.linalg.norm(emu[None] - ref)
    say("   S_T error / emulated %.3f" % (e / bar), "relative %.2e" % (e / np.linalg.norm(ref)))
    assert e <= 1.1 * bar, (e, bar)
