"""float32 storage keeps the accuracy of blocked sums: the low-rank
denominator d_lr, a sum of positive terms over the features and the tokens.

Bar: 2-norm error <= 2 u of the result (u = 2^-24, half a unit in the last
place).  A value carries the roundings of its features (three products and a
sigmoid pair of a few u each, averaged over the r features and N tokens that
enter it), of short chains of sums and of the final scaling: 0.9e-7 measured.
One chain over all r products adds about sqrt(r / 3) u / 2 at r = 64, which
is past the bar (1.43e-7 measured)."""
import numpy as np
import pytest

import oracle
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
