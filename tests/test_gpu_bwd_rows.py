"""GPU parity of the backward's row scalars where the state pass forms them (d_h
64: up to 131072 rows; d_h 128: bf16, up to 64 features and 65536 rows) and
where the row pass does, on either side of those lines: the gate and lambda
gradients, dQ and dV against the oracle on sampled rows; a row is covered by 8
lanes (bf16, d_h 64) or 16."""
import numpy as np
import pytest

import oracle
import paper_2607_20214_amd as E
from gpu_util import TOL, cfg_of, head_cfg_of, rel_err, run_gpu_fwd_bwd, say
from paper_2607_20214_amd import workloads as W

pytestmark = pytest.mark.gpu


def _w(name, B, H, N, d, r, causal, dtype):
    return W.Workload(name, B, H, N, d, 64, r, causal, dtype, recipe="iid", qk_scale=d ** -0.25, seed=90)


CASES = [
    _w("bf16-d64-77", 1, 2, 77, 64, 32, True, "bf16"),          # one full chunk and a ragged one
    _w("bf16-d128-r128-200", 2, 1, 200, 128, 128, False, "bf16"),
    _w("f32-d64-r128-130", 1, 1, 130, 64, 128, True, "f32"),
    _w("f32-d128-65", 1, 2, 65, 128, 32, False, "f32"),
    _w("bf16-d128-r64-77", 1, 2, 77, 128, 64, True, "bf16"),
    _w("bf16-d128-r32-16x4096", 2, 8, 4096, 128, 32, False, "bf16"),   # 65536 rows
    _w("bf16-d128-r32-16x4097", 2, 8, 4097, 128, 32, False, "bf16"),
    _w("bf16-d64-16x8192", 2, 8, 8192, 64, 32, False, "bf16"),   # 131072 rows: the last fused length
    _w("bf16-d64-16x8193", 2, 8, 8193, 64, 32, False, "bf16"),   # one token more
]


def _fused(w):
    rows = w.B * w.H * w.N
    return rows <= 131072 if w.d == 64 else w.dtype == "bf16" and w.r <= 64 and rows <= 65536


@pytest.mark.parametrize("w", CASES, ids=[w.name for w in CASES])
def test_row_scalars(w):
    cfg = cfg_of(w)
    inp = W.make_inputs(w, with_grad=True)
    gates, lam = W.make_gates(w), W.make_lambda_rows(w)
    say(f"[rows] {w.name}: B={w.B} H={w.H} N={w.N} d={w.d} r={w.r} causal={w.causal} {w.dtype}")
    E.profile_enable(True)
    try:
        _, got = run_gpu_fwd_bwd(cfg, inp, gates, want_dgates=True, lam_rows=lam, want_dlambda=True)
        names = set(E.profile_read())
    finally:
        E.profile_enable(False)
    assert ("race_rows_bwd" in names) == _fused(w) and ("bwd_rows" in names) != _fused(w), names
    hc, tol = head_cfg_of(cfg), TOL[w.dtype]
    mask = None
    if w.N > 4096:
        mask = np.zeros(w.N, np.uint8)
        mask[np.r_[:40, w.N - 70:w.N]] = 1
    rows = slice(None) if mask is None else mask > 0
    for b, h in {(0, 0), (w.B - 1, w.H - 1)}:
        ref = oracle.backward(hc, inp["Q"][b, h], inp["K"][b, h], inp["V"][b, h], inp["W_sort"][h], inp["W_race"][h],
                              inp["dO"][b, h], gates=gates[b, h], lam_rows=lam[b, h], q_mask=mask, k_mask=mask)
        for name in ("dgates", "dlambda", "dQ", "dV"):
            e = rel_err(got[name][b, h][rows], ref[name][rows])
            assert e <= tol, f"{name} (b={b}, h={h}): {e:.3e}"
