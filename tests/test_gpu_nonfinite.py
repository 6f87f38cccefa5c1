"""Infinities and NaN stay where the operator's own sums take them: values
that a kernel loads only to mask them out change no other row.  Each case
runs the same inputs twice, clean and poisoned, and compares bit for bit the
rows that do not depend on the poisoned values."""
import numpy as np
import pytest

from gpu_util import cfg_of, run_gpu_fwd, run_gpu_fwd_bwd, say
import paper_2607_20214_amd as E
from paper_2607_20214_amd import workloads as W

pytestmark = pytest.mark.gpu


def _w(name, H, N, d, k, r, dtype, n0=0, causal=True):
    return W.Workload(name, 1, H, N, d, k, r, causal, dtype, recipe="iid", qk_scale=d ** -0.25, seed=95, n0=n0)


# odd recursions, whose last query lists hold zero tokens: as loads they are
# token 0's rows.  b = 64 and 128 take the whole-block kernel, b = 256 and 96 the two passes
PADDED = [
    _w("bf16-d64-k64-777", 1, 777, 64, 64, 32, "bf16"),
    _w("bf16-d128-k128-1111", 2, 1111, 128, 128, 64, "bf16"),
    _w("bf16-d64-k128-2051", 1, 2051, 64, 128, 32, "bf16", 130),
    _w("bf16-d64-k256-1001", 1, 1001, 64, 256, 32, "bf16", 130),
    _w("bf16-d64-k96-777", 1, 777, 64, 96, 32, "bf16", 100),
    _w("f32-d64-k64-387", 2, 387, 64, 64, 32, "f32"),
    _w("f32-d128-k64-387", 1, 387, 128, 64, 32, "f32"),
]


@pytest.mark.parametrize("poison", ["score", "dO", "Q"])
@pytest.mark.parametrize("w", PADDED, ids=[w.name for w in PADDED])
def test_zero_tokens_do_not_read_token_0(w, poison):
    """Token 0 is a query of its leaf alone, so its Q and dO, and its score
    against later keys, reach no later row."""
    cfg = cfg_of(w)
    leaf = w.N
    while leaf > (w.n0 or 2 * w.k):
        leaf = (leaf + 1) // 2
    t0 = max(64, leaf)                       # later rows share no leaf and no 64-token chunk with token 0
    assert E.num_levels(cfg) > 0 and t0 < w.N // 2
    inp = W.make_inputs(w, with_grad=True)
    if poison == "score":                    # Q_0 . K_j overflows for every j >= t0, no other product does
        inp["Q"][..., 3] = 0
        inp["K"][..., :t0, 3] = 0
        inp["K"][..., t0:, 3] = 1e20
    _, clean = run_gpu_fwd_bwd(cfg, inp)
    if poison == "score":
        inp["Q"][..., 0, 3] = 1e20
    else:
        inp[poison][..., 0, :] = np.nan
    say(f"[nonfinite] {w.name} {poison}: rows from {t0}")
    _, got = run_gpu_fwd_bwd(cfg, inp)
    for name in ("dQ", "dK", "dV"):
        assert np.isfinite(clean[name]).all(), name
        bad = ~(got[name][:, :, t0:] == clean[name][:, :, t0:])
        assert not bad.any(), f"{name}: {bad.sum()} of {bad.size} differ"


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,r", [(64, 16), (64, 48), (128, 48), (64, 80)])
def test_padded_feature_tables_stay_zero(d, r, causal):
    """float32, a feature count that fills no padded size: an infinite entry
    of a key saturates its features like a huge one, and the tables that pad
    the count stay out of the low-rank branch."""
    w = _w(f"f32-d{d}-r{r}", 2, 200, d, 64, r, "f32", causal=causal)
    cfg, inp = cfg_of(w), W.make_inputs(w)
    inp["K"][..., 17, 5] = 1e30
    huge, _ = run_gpu_fwd(cfg, inp)
    inp["K"][..., 17, 5] = np.inf
    inf, _ = run_gpu_fwd(cfg, inp)
    for name in ("d_lr", "O_lr"):
        assert np.isfinite(huge[name]).all(), name
        assert np.array_equal(huge[name], inf[name]), name
