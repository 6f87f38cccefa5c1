"""bench.py's byte accounting (host logic, no GPU): the algorithmic bytes of
the 16K causal workload written out by hand from the per-token terms of the
complexity model, the per-kernel model exceeding them by exactly the level
partials, and the choice of the dominant kernel."""
import bench
from paper_2607_20214_amd import workloads as W


def test_survey_units_16k_by_hand():
    w = W.CAUSAL_16K
    Lv, s, N, d, heads = 6, 2, 16384, 128, 16
    u = bench.survey_units(w, Lv)
    # sparse backward leaf: Q, K, V, dO read (4Nds), dQ, dK, dV at 4 bytes (12Nd), 8N row scalars
    assert u["sparse_bwd_leaf"][0] == heads * (4 * N * d * s + 12 * N * d + 8 * N)
    # one level: half of the tokens as queries (Q, dO) and half as keys (K, V): 2Nds + 4N
    assert u["sparse_bwd_levels"][0] == heads * Lv * (2 * N * d * s + 4 * N)
    # forward level: 1.5 Nds + 4N per level
    assert u["sparse_fwd_levels"][0] == heads * Lv * (3 * (N // 2) * d * s + 4 * N)
    # 10 d flops per sparse interaction backward; leaf interactions n0 (n0 + 1) / 2 per leaf
    n0 = N >> Lv
    assert u["sparse_bwd_leaf"][1] == heads * (N // n0) * (n0 * (n0 + 1) // 2) * 10 * d
    # the whole step's bytes quoted in the documentation
    assert sum(v[0] for v in u.values()) == 4126670848


def test_kernel_model_adds_exactly_the_level_partials():
    w = W.CAUSAL_16K
    Lv, s, N, d, heads = 6, 2, 16384, 128, 16
    u, km = bench.survey_units(w, Lv), bench.kernel_model(w, Lv)
    slots = Lv * heads * (N // 2)               # one partial row per level list entry
    # the level kernel also writes the dQ, dK, dV partial rows (storage
    # dtype) and reads the two index lists and the row scalars per entry
    assert km["sparse_bwd_levels"] - u["sparse_bwd_levels"][0] == slots * (3 * d * s + 12)


def test_units_that_share_a_launch_are_charged_together():
    """The sort that runs beside the RACE scan, and the row scalars formed in
    the state pass: one figure each, nothing lost from the step's total."""
    for w, Lv in ((W.TINY_FP32, 0), (W.CAUSAL_16K, 6)):
        u = bench.survey_units(w, Lv)
        m = bench.merge_shared(u, {"sort_scan", "race_rows_bwd", "race_out"})
        assert set(u) - set(m) == {"sort", "lowrank_fwd", "bwd_rows", "lowrank_bwd"}
        assert {"race_state_fwd", "race_out", "sort_scan"} <= set(m["sort+lowrank_fwd"][2])
        assert {"race_rows_bwd", "race_bwd"} <= set(m["bwd_rows+lowrank_bwd"][2])
        for i in (0, 1):
            assert sum(v[i] for v in m.values()) == sum(v[i] for v in u.values())
        assert bench.merge_shared(u, {"sort", "race_scan_fwd", "bwd_rows", "race_state_bwd"}) == u


def test_kernel_model_matches_the_counted_traffic():
    """The committed rocprofv3 FETCH_SIZE / WRITE_SIZE summaries, where they
    were taken on the current kernel source, agree with the model within 5%."""
    import os
    w = W.CAUSAL_16K
    km = bench.kernel_model(w, 6)
    checked = 0
    for k in ("sparse_leaf_bwd", "sparse_bwd_levels"):
        counted = bench.read_traffic(k, w.name)
        if counted is None:
            continue
        checked += 1
        assert abs(counted / km[k] - 1) < 0.05, (k, counted, km[k])
    if not checked:
        import pytest
        pytest.skip("no counter summary taken on the current kernel source")


def test_dominant_unit_follows_the_largest_kernel():
    rows = {"lowrank_bwd": (0.40, 1, 1, ["race_dq", "race_dk", "race_dv"]),
            "sparse_bwd_leaf": (0.35, 1, 1, ["sparse_leaf_bwd"]),
            "sort": (0.05, 1, 1, ["sort"])}
    per = {"race_dq": 0.14, "race_dk": 0.15, "race_dv": 0.11, "sparse_leaf_bwd": 0.35, "sort": 0.05}
    # the unit with the largest sum is not the one of the largest kernel
    assert bench.dominant_unit(rows, per) == "sparse_bwd_leaf"
    per["race_dk"] = 0.36
    assert bench.dominant_unit(rows, per) == "lowrank_bwd"
