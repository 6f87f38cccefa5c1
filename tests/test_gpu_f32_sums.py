"""Results held in float32 keep the accuracy of blocked sums.

The low-rank denominator d_lr (float32 storage), a sum of positive terms over
the features and the tokens: 2-norm error <= 2 u of the result (u = 2^-24, half a unit in the last
place).  A value carries the roundings of its features (three products and a
sigmoid pair of a few u each, averaged over the r features and N tokens that
enter it), of short chains of sums and of the final scaling: 0.9e-7 measured.
One chain over all r products adds about sqrt(r / 3) u / 2 at r = 64, which
is past the bar (1.43e-7 measured)."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2607_20214_amd as E
from gpu_util import cfg_of, head_cfg_of, run_gpu_fwd, say
from paper_2607_20214_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,d,r,causal", [(784, 64, 64, False), (784, 128, 64, True), (512, 64, 128, False)])
def test_low_rank_denominator(N, d, r, causal):
    w = W.Workload(f"f32-sums-{N}-{d}-{r}", 2, 2, N, d, 64, r, causal, "f32", recipe="iid", qk_scale=d ** -0.25, seed=97)
    cfg, inp = cfg_of(w), W.make_inputs(w)
    got, _ = run_gpu_fwd(cfg, inp)
    num = den = 0.0
    for b in range(2):
        for h in range(2):
            ref = oracle.forward(head_cfg_of(cfg), inp["Q"][b, h], inp["K"][b, h], inp["V"][b, h], inp["W_sort"][h],
                                 inp["W_race"][h])["d_lr"]
            num += float(np.sum((got["d_lr"][b, h].astype(np.float64) - ref) ** 2))
            den += float(np.sum(ref ** 2))
    say(f"[f32 sums] N={N} d={d} r={r} causal={causal}: {(num / den) ** 0.5:.3e}")
    assert (num / den) ** 0.5 <= 2 * 2.0 ** -24


@pytest.mark.parametrize("N,d,causal", [(784, 64, False), (600, 128, True)])
def test_fusion_rounds_once(N, d, causal):
    """Without gates O = m O_s + O_lr from the saved parts with one rounding:
    the 64-bit sum rounded to float32 (which can differ from the fused
    product's single rounding only next to a tie of the 64-bit sum)."""
    w = W.Workload(f"f32-fuse-{N}-{d}", 1, 2, N, d, 64, 32, causal, "f32", recipe="iid", qk_scale=d ** -0.25, seed=98)
    got, _ = run_gpu_fwd(cfg_of(w), W.make_inputs(w))
    m, o_s, o_lr = (got[k].astype(np.float64) for k in ("m", "O_s", "O_lr"))
    once = (m[..., None] * o_s + o_lr).astype(np.float32)
    assert (got["O"] != once).mean() < 1e-4


@pytest.mark.parametrize("N,H,d", [(1024, 64, 128), (2560, 52, 64)])
def test_wide_leaf_denominator(N, H, d):
    """One key of weight 1 and the others of 2^-25.5, each of them less than
    half a unit in the last place of 1: a chain that starts with the first key
    loses every one it adds, 31 of a lane's first tile (6.5e-7 = 11 u); sums
    of eight lose three of them (1.1 u).  Rows of the first tile, bar 8 u for
    log d: those, at most u for each later addition to the first key's sum
    (the second four, three more eights, the other half wave) and 2 u for the
    logarithm."""
    q = torch.zeros(1, H, N, d, device="cuda", dtype=torch.bfloat16)
    k = torch.zeros_like(q)
    q[..., 0] = 16.0
    k[:, :, 1:, 0] = -25.5 * math.log(2.0) * d ** 0.5 / 16.0
    v = torch.randn(1, H, N, d, device="cuda").bfloat16()
    cfg = E.Config(B=1, H=H, N=N, d_h=d, k=128, r=32, causal=True, n0=N)
    E.profile_enable(True)
    try:
        lse = E.fwd(cfg, q, k, v, torch.randn(H, 5, d, device="cuda"), torch.randn(H, 2, 4, d, device="cuda"))[1]
        names = set(E.profile_read())
    finally:
        E.profile_enable(False)
    assert "sparse_fwd_leaf_wide" in names, names
    s = float(q[0, 0, 1, 0]) * float(k[0, 0, 1, 0]) * d ** -0.5
    ref = torch.log1p(torch.arange(64, dtype=torch.float64) * math.exp(s))
    err = (lse[0, :, :64].double().cpu() - ref).abs().max().item()
    say(f"[f32 sums] wide leaf N={N} d={d}: log d off by {err:.3e}")
    assert err <= 8 * 2.0 ** -24


@pytest.mark.parametrize("B,H,N,G", [(2, 8, 4096, 64), (2, 8, 4096, 0), (1, 4, 16384, 64)])
def test_token_rule_parameter_sums(B, H, N, G):
    """dlam_c = sum of dlambda over the tokens: the workgroups' partial sums
    (32 to 128 per head here) are added in blocks.  An addition's rounding is
    about 0.4 u of the sum so far, so a chain of K of them gives 0.4 u
    sqrt(K / 3): 0.7 u for eight blocks and as much inside a workgroup, but
    1.3 u to 2.6 u for the partial sums in one chain.  Bar 1.4 u."""
    errs = []
    for seed in range(4):
        g = torch.Generator(device="cuda").manual_seed(seed)

        def rand(*shape):
            return torch.randn(*shape, generator=g, device="cuda")
        p = dict(lam_w=rand(H, 64) * 0.1, lam_b=rand(H) * 0.1, lam_c=rand(H).abs() + 0.1)
        if G:
            p.update(W1=rand(H, G, 64) * 0.1, b1=rand(H, G) * 0.1, W2=rand(H, 2, G) * 0.1, b2=rand(H, 2) * 0.1)
        q, dl = rand(B, H, N, 64).bfloat16(), rand(B, H, N) + 2
        cfg = E.Config(B=B, H=H, N=N, d_h=64, k=64, r=32, causal=True)
        got = E.token_rules_bwd(cfg, E.TokenRules(**p), q, rand(B, H, N, 2) if G else None, dl)["dlam_c"]
        ref = dl.double().sum((0, 2))
        errs.append(((got.double() - ref) / ref).pow(2).mean().item())
    err = float(np.mean(errs)) ** 0.5
    say(f"[f32 sums] dlam_c B={B} H={H} N={N} G={G}: {err:.3e}")
    assert err <= 1.4 * 2.0 ** -24


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_token_rule_sigmoid(dtype):
    """With W2 = 0 the gates are sigmoid(b2) and nothing else.  For x in [-1, 0]
    the rounding of 1 + e (2.1e-8 of it, rms), of the quotient (2.4e-8) and
    of the exponential (2.4e-8 of what is left of it) come to 4.0e-8; one more
    rounded product, as in e times a reciprocal, to 4.7e-8.  Bar 4.3e-8."""
    H = 512
    b2 = torch.linspace(-1, 0, 2 * H, device="cuda").view(H, 2)
    zero = [torch.zeros(*s, device="cuda") for s in ((H, 64, 64), (H, 64), (H, 2, 64))]
    cfg = E.Config(B=1, H=H, N=64, d_h=64, k=64, r=32, causal=True, dtype=dtype)
    q = torch.zeros(1, H, 64, 64, device="cuda", dtype=cfg.torch_dtype)
    gates, _ = E.token_rules_fwd(cfg, E.TokenRules(W1=zero[0], b1=zero[1], W2=zero[2], b2=b2), q)
    ref = torch.sigmoid(b2.double())
    err = ((gates[0, :, 0].double() - ref) / ref).pow(2).mean().sqrt().item()
    say(f"[f32 sums] sigmoid {dtype}: {err:.3e}")
    assert err <= 4.3e-8
