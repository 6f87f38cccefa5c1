"""GPU parity of the RACE output and dV passes where eight waves share a segment's
state (d_h 128, 129 to 256 features): feature tables that fill one group of four
waves and part of the other, lengths around a chunk, both causalities."""
import numpy as np
import pytest

import oracle
from gpu_util import TOL, cfg_of, head_cfg_of, rel_err, run_gpu_fwd_bwd, say
from paper_2607_20214_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,r,causal", [(65, 144, True), (200, 208, True), (333, 256, True), (129, 144, False),
                                        (320, 256, False)])
def test_wide_state(N, r, causal):
    w = W.Workload(f"wide-state-{N}-{r}", 1, 2, N, 128, 64, r, causal, "bf16", recipe="iid", qk_scale=128 ** -0.25, seed=91)
    cfg, inp = cfg_of(w), W.make_inputs(w, with_grad=True)
    gates = np.zeros((1, 2, N, 2), np.float32)
    gates[..., 0], gates[..., 1] = 0.25, 0.75              # the low-rank branch dominates
    say(f"[wide-state] N={N} r={r} causal={causal}")
    fwd, got = run_gpu_fwd_bwd(cfg, inp, gates)
    hc, tol = head_cfg_of(cfg), TOL["bf16"]
    for h in (0, 1):
        ref = oracle.backward(hc, inp["Q"][0, h], inp["K"][0, h], inp["V"][0, h], inp["W_sort"][h], inp["W_race"][h],
                              inp["dO"][0, h], gates=gates[0, h])
        ref["O"] = oracle.forward(hc, inp["Q"][0, h], inp["K"][0, h], inp["V"][0, h], inp["W_sort"][h],
                                  inp["W_race"][h], gates=gates[0, h])["O"]
        got["O"] = fwd["O"]
        for name in ("O", "dQ", "dK", "dV"):
            e = rel_err(got[name][0, h], ref[name])
            assert e <= tol, f"{name} (h={h}): {e:.3e}"
