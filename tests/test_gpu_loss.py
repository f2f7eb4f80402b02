"""GPU parity of the objectives that consume a rollout (ff_loss.h) against the oracle.

Tolerances: the noised latent is one fused multiply-add per element in float32,
stored in the tensor's dtype (bf16: half an ulp of bf16; f32: a few float32
ulps).  The matching losses read bf16 / f32 values that the oracle sees
exactly; per element the difference and its square are float32 (relative
error ~1e-7), summed in float32 over 8 elements and in float64 beyond, so the
per-sample sums agree to ~1e-6 relative: the bound used is 1e-5.  The GRPO
objective is float64 throughout (bound 1e-12); the clip count is an integer
and must match exactly.
"""
import math

import numpy as np
import pytest
import torch

from oracle import losses as OL
from paper_2602_12529_amd import configs as C

from gpu_util import TOL, best_us, dev, host, normal, rel, say

pytestmark = pytest.mark.gpu

SHAPES = [(8, 256), (3, 1000), (1, 1), (2, 7), (5, 12345), (4, 65536), (2, 8 * 2048 + 8)]
LOSS_REL = 1e-5


@pytest.mark.parametrize("dt", [C.F32, C.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("B,D", SHAPES)
def test_flow_noise_parity(gpu_lib, dt, B, D):
    say("flow_noise", dt, B, D)
    x0, eps = normal(300, (B, D), dt), normal(301, (B, D), dt)
    t = np.linspace(0.05, 0.95, B).astype(np.float32)
    Xt = gpu_lib.flow_noise(dev(x0, dt), dev(eps, dt), torch.from_numpy(t).cuda())
    torch.cuda.synchronize()
    ref = OL.flow_noise(x0, eps, t.astype(np.float64))
    got = host(Xt)
    assert rel(got, ref) <= TOL[dt]
    # one float32 fma (error ~2^-24 of the two terms) then rounding to the stored dtype
    half_ulp = 2.0 ** -8 if dt == C.BF16 else 2.0 ** -24
    tb = t.astype(np.float64)[:, None]
    bound = half_ulp * np.abs(ref) + 4 * 2.0 ** -24 * (np.abs((1 - tb) * x0) + np.abs(tb * eps))
    assert np.all(np.abs(got - ref) <= bound)


@pytest.mark.parametrize("dt", [C.F32, C.BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("B,D", SHAPES)
def test_awm_and_nft_loss_parity(gpu_lib, dt, B, D):
    say("awm/nft", dt, B, D)
    v, vn, eps, x0 = (normal(310 + i, (B, D), dt) for i in range(4))
    adv = normal(320, (B,), C.F32)
    r = np.linspace(0.0, 1.0, B).astype(np.float32)
    V, VN, E, X0 = (dev(a, dt) for a in (v, vn, eps, x0))
    per, loss = gpu_lib.awm_loss(V, E, X0, dev(adv))
    per2, loss2 = gpu_lib.nft_loss(V, VN, E, X0, torch.from_numpy(r).cuda())
    per_again, loss_again = gpu_lib.awm_loss(V, E, X0, dev(adv))
    torch.cuda.synchronize()
    ref_per, ref_loss = OL.awm_loss(v, eps, x0, adv)
    np.testing.assert_allclose(host(per), ref_per, rtol=LOSS_REL, atol=1e-12)
    assert host(loss)[0] == pytest.approx(ref_loss, rel=LOSS_REL, abs=LOSS_REL * np.mean(np.abs(ref_per)))
    ref_per2, ref_loss2 = OL.nft_loss(v, vn, eps, x0, r)
    np.testing.assert_allclose(host(per2), ref_per2, rtol=LOSS_REL, atol=1e-12)
    assert host(loss2)[0] == pytest.approx(ref_loss2, rel=LOSS_REL)
    # fixed-order reductions: repetition is bitwise identical
    assert torch.equal(per, per_again) and torch.equal(loss, loss_again)


# One workgroup finishes up to 4096 samples, with 64 lanes a sample down to one; more take two launches.
@pytest.mark.parametrize("B,D", [(1, 200000), (3, 30000), (300, 2056), (4096, 8), (4097, 8)])
def test_matching_loss_sample_counts(gpu_lib, B, D):
    test_awm_and_nft_loss_parity(gpu_lib, C.F32, B, D)


# Of few partial sums (of 2048 elements) a lane one workgroup finishes everything, of more two launches; the first of
# each pair is the last that NFT or AWM finishes in one.
@pytest.mark.parametrize("B,sums", [(192, 16), (192, 17), (192, 32), (192, 33), (32, 64), (33, 63), (16, 512), (17, 482)])
def test_matching_loss_partial_sums(gpu_lib, B, sums):
    say("awm/nft", B, sums)
    gen = torch.Generator(device="cuda").manual_seed(B)
    v, vn, eps, x0 = (torch.randn((B, sums * 2048 - 8), device="cuda", generator=gen).to(torch.bfloat16) for _ in range(4))
    adv, r = torch.randn(B, device="cuda", generator=gen), torch.linspace(0, 1, B, device="cuda")
    per, loss = gpu_lib.awm_loss(v, eps, x0, adv)
    per2, loss2 = gpu_lib.nft_loss(v, vn, eps, x0, r)
    target = eps.double() - x0.double()
    s1, s2 = (((a.double() - target) ** 2).sum(-1) for a in (v, vn))
    ref, ref2 = adv.double() * s1, r.double() * s1 + (1 - r.double()) * s2
    np.testing.assert_allclose(host(per), host(ref), rtol=LOSS_REL)
    np.testing.assert_allclose(host(per2), host(ref2), rtol=LOSS_REL)
    assert loss.item() == pytest.approx(ref.mean().item(), rel=LOSS_REL, abs=LOSS_REL * ref.abs().mean().item())
    assert loss2.item() == pytest.approx(ref2.mean().item(), rel=LOSS_REL)


def test_matching_loss_of_one_long_sample(gpu_lib):
    """One sample of 16384 partial sums: the sums against float64, and NFT, which reads four tensors where AWM
    reads three (4/3 of the traffic), takes no more than 1.6 times as long."""
    gen = torch.Generator(device="cuda").manual_seed(5)
    v, vn, eps, x0 = (torch.randn((1, 1 << 26), device="cuda", generator=gen).to(torch.bfloat16) for _ in range(4))
    adv, r = torch.tensor([0.7], device="cuda"), torch.tensor([0.25], device="cuda")
    per, loss = gpu_lib.awm_loss(v, eps, x0, adv)
    per2, loss2 = gpu_lib.nft_loss(v, vn, eps, x0, r)
    target = eps.double() - x0.double()
    s1, s2 = (((a.double() - target) ** 2).sum().item() for a in (v, vn))
    assert per.item() == pytest.approx(float(adv[0]) * s1, rel=LOSS_REL) and loss.item() == per.item()
    assert per2.item() == pytest.approx(0.25 * s1 + 0.75 * s2, rel=LOSS_REL) and loss2.item() == per2.item()
    ws = torch.empty(gpu_lib.loss_workspace_size(1, 1 << 26), dtype=torch.uint8, device="cuda")
    awm = best_us(lambda: gpu_lib.awm_loss(v, eps, x0, adv, per, loss, ws))
    nft = best_us(lambda: gpu_lib.nft_loss(v, vn, eps, x0, r, per2, loss2, ws))
    say(f"one long sample: AWM {awm:.1f} us, NFT {nft:.1f} us")
    assert nft < 1.6 * awm


def test_awm_loss_of_the_exact_velocity_is_zero(gpu_lib):
    """With v = eps - x0 formed on the device the AWM loss vanishes (the sign convention of the target)."""
    B, D = 4, 4096
    x0, eps = normal(330, (B, D), C.F32), normal(331, (B, D), C.F32)
    X0, E = dev(x0), dev(eps)
    per, loss = gpu_lib.awm_loss(E - X0, E, X0, torch.ones(B, device="cuda"))
    torch.cuda.synchronize()
    assert np.all(host(per) == 0.0) and host(loss)[0] == 0.0


@pytest.mark.parametrize("S,B", [(1, 2), (3, 16), (10, 8), (7, 1000)])
def test_grpo_loss_parity(gpu_lib, S, B):
    rng = np.random.default_rng(S * 1000 + B)
    lpo = rng.standard_normal((S, B)) * 100.0 - 2e5
    lpn = lpo + rng.uniform(-0.6, 0.6, (S, B))
    adv = rng.standard_normal(B).astype(np.float32)
    w = rng.uniform(0.5, 2.0, S).astype(np.float32)
    ec = 0.2
    # keep the ratio away from the clip boundaries so the integer count is unambiguous
    r = np.exp(lpn - lpo)
    lpn = np.where(np.abs(np.abs(r - 1.0) - ec) < 1e-9, lpn + 1e-6, lpn)
    LPN, LPO = (torch.from_numpy(a).cuda() for a in (lpn, lpo))
    for wt in (None, w):
        loss, n = gpu_lib.grpo_loss(LPN, LPO, torch.from_numpy(adv).cuda(),
                                    None if wt is None else torch.from_numpy(wt).cuda(), ec)
        torch.cuda.synchronize()
        ref_loss, ref_n = OL.grpo_loss(lpn, lpo, adv, wt, ec)
        assert host(loss)[0] == pytest.approx(ref_loss, rel=1e-12, abs=1e-14)
        assert int(n.cpu()[0]) == ref_n


def test_grpo_on_policy_recompute(gpu_lib):
    """Recomputing the log-probs of a stored SDE step with ff_logprob reproduces ff_sde_step's bits,
    so the on-policy ratio is exactly 1: no element is clipped and the loss is -mean(A)."""
    B, D, S = 8, 5000, 3
    adv = normal(340, (B,), C.F32)
    old, new = [], []
    for k in range(S):
        x, v, e = (normal(341 + 3 * k + i, (B, D), C.BF16) for i in range(3))
        X, V, E = dev(x, C.BF16), dev(v, C.BF16), dev(e, C.BF16)
        Xn = torch.empty_like(X)
        lp_old = torch.empty(B, dtype=torch.float64, device="cuda")
        gpu_lib.sde_step(X, V, E, Xn, 0.8 - 0.1 * k, 0.7 - 0.1 * k, 0.7, logp=lp_old)
        lp_new = torch.empty_like(lp_old)
        gpu_lib.logprob(X, V, Xn, lp_new, 0.8 - 0.1 * k, 0.7 - 0.1 * k, 0.7)
        old.append(lp_old)
        new.append(lp_new)
    loss, n = gpu_lib.grpo_loss(torch.stack(new), torch.stack(old), dev(adv), None, 0.2)
    torch.cuda.synchronize()
    assert int(n.cpu()[0]) == 0
    assert host(loss)[0] == pytest.approx(-float(np.mean(adv.astype(np.float64))), rel=1e-12, abs=1e-15)
