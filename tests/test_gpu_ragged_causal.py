"""GPU parity of the causal recursion when segment and leaf lengths are not
multiples of the 64-row tile, and of the paper's causal text setting
(block size 256, base length 4096), against the oracle."""
import numpy as np
import pytest

import oracle
from gpu_util import TOL, cfg_of, head_cfg_of, rel_err, run_gpu_fwd_bwd, say
import paper_2607_20214_amd as E
from paper_2607_20214_amd import workloads as W

pytestmark = pytest.mark.gpu


def _w(name, B, H, N, d, k, r, dtype, n0, recipe="iid", seed=80):
    qs = d ** -0.25 if recipe == "iid" else 1.0
    return W.Workload(name, B, H, N, d, k, r, True, dtype, recipe=recipe, qk_scale=qs, seed=seed,
                      centres=16, n0=n0)


CASES = [
    # levels of 1000 / 500 / 250 sorted queries, leaves of 250 tokens
    _w("c-bf16-d128-2000-leaf250", 1, 2, 2000, 128, 64, 128, "bf16", 300),
    # odd leaves of 125 tokens
    _w("c-f32-d64-1000-leaf125", 1, 1, 1000, 64, 32, 32, "f32", 130),
    _w("c-bf16-d64-1000-leaf125-clustered", 1, 2, 1000, 64, 64, 64, "bf16", 130, recipe="clustered"),
    # leaf shorter than one tile
    _w("c-bf16-d128-800-leaf50", 2, 1, 800, 128, 32, 64, "bf16", 60),
    # the text setting's block and base length, scaled: levels 4000 / 2000 / 1000, leaves 1000
    _w("c-bf16-text-8000-b256-leaf1000", 1, 1, 8000, 128, 256, 64, "bf16", 1000),
    # leaves of 9 tiles (odd: the last workgroup of a long leaf holds one query tile), d_h 64
    _w("c-bf16-d64-2080-leaf520", 1, 2, 2080, 64, 64, 64, "bf16", 520),
    # the text setting's own leaf of 4096 tokens
    _w("c-bf16-text-8192-b256-n04096", 1, 1, 8192, 128, 256, 64, "bf16", 4096),
]


def _check(w, neighbors=0, heads=None, q_mask=None, launches=()):
    """launches: kernels that the call has to run."""
    cfg = cfg_of(w, neighbors=neighbors)
    Lv = E.num_levels(cfg)
    say(f"[ragged] {w.name}: N={w.N} k={w.k} n0={w.n0} levels={Lv} leaf={w.N >> Lv} {w.dtype} nbr={neighbors}")
    inp = W.make_inputs(w, with_grad=True)
    E.profile_enable(True)
    try:
        fwd, bwd = run_gpu_fwd_bwd(cfg, inp)
        names = set(E.profile_read())
    finally:
        E.profile_enable(False)
    assert set(launches) <= names, names
    tol = TOL[w.dtype]
    hc = head_cfg_of(cfg)
    errs = {}
    for b in range(w.B):
        for h in range(w.H):
            if heads is not None and (b, h) not in heads:
                continue
            args = (inp["Q"][b, h], inp["K"][b, h], inp["V"][b, h], inp["W_sort"][h], inp["W_race"][h])
            pq, pk = oracle.select(hc, args[0], args[1], args[3])
            assert np.array_equal(fwd["perm_q"][b, h], pq) and np.array_equal(fwd["perm_k"][b, h], pk)
            ref = oracle.forward(hc, *args, row_mask=q_mask)
            rows = slice(None) if q_mask is None else (q_mask > 0)
            for name in ("O", "O_s", "m"):
                e = rel_err(fwd[name][b, h][rows], ref[name][rows])
                errs[name] = max(errs.get(name, 0.0), e)
                assert e <= tol, f"{name} (b={b}, h={h}): {e:.3e}"
            rb = oracle.backward(hc, *args, inp["dO"][b, h], q_mask=q_mask, k_mask=q_mask)
            for name in ("dQ", "dK", "dV"):
                e = rel_err(bwd[name][b, h][rows], rb[name][rows])
                errs[name] = max(errs.get(name, 0.0), e)
                assert e <= tol, f"{name} (b={b}, h={h}): {e:.3e}"
    say("   errors:", {k: f"{v:.2e}" for k, v in errs.items()})


@pytest.mark.parametrize("w", CASES, ids=[w.name for w in CASES])
def test_ragged_causal(w):
    _check(w)


# the whole-block level backward on lists that end in a short block and on
# (b = 64, 128) on padded ones (zero tokens in the query lists), and the two
# passes that padded lists of b = 256 take: halves shorter than a block, a last
# block of one entry, several zero tokens
BLOCK_CASES = [
    _w("c-bf16-d128-k64-777-padded", 1, 2, 777, 128, 64, 64, "bf16", 0),
    _w("c-bf16-d64-k64-1155-padded", 1, 1, 1155, 64, 64, 32, "bf16", 0, recipe="clustered"),
    _w("c-bf16-d128-k128-1111-padded", 1, 2, 1111, 128, 128, 64, "bf16", 0, recipe="clustered"),
    _w("c-bf16-d64-k128-1032-one-entry-block", 1, 2, 1032, 64, 128, 64, "bf16", 130),
    _w("c-bf16-d128-k128-300-half-shorter", 2, 1, 300, 128, 128, 64, "bf16", 80),
    _w("c-bf16-d128-k256-2051-padded", 1, 2, 2051, 128, 256, 64, "bf16", 0),
    _w("c-bf16-d64-k256-1001-half-shorter", 1, 1, 1001, 64, 256, 64, "bf16", 130),
    _w("c-f32-d64-k64-387-padded", 1, 2, 387, 64, 64, 32, "f32", 0),
    _w("c-f32-d128-k64-650", 1, 1, 650, 128, 64, 64, "f32", 0, recipe="clustered"),
]


@pytest.mark.parametrize("w", BLOCK_CASES, ids=[w.name for w in BLOCK_CASES])
def test_ragged_causal_whole_blocks(w):
    _check(w)


# 256-key blocks of a padded recursion keep a dQ summed over the block's keys in
# float32 (the two passes); the whole-block kernel's two halves, which round the
# first half's sum to bf16, take unpadded lists only
@pytest.mark.parametrize("N,halves", [(2051, False), (1001, False), (2048, True), (1040, True)])
def test_padded_256_key_blocks_keep_float32_sums(N, halves):
    w = _w(f"c-bf16-d64-k256-{N}", 1, 1, N, 64, 256, 32, "bf16", 130)
    inp = W.make_inputs(w, with_grad=True)
    E.profile_enable(True)
    try:
        run_gpu_fwd_bwd(cfg_of(w), inp)
        names = set(E.profile_read())
    finally:
        E.profile_enable(False)
    assert ("sparse_bwd_levels" in names) == halves, names
    assert ({"sparse_dq_levels", "sparse_dkv_levels"} <= names) == (not halves), names


# the forward's 128-query tiles: levels of b >= 128 (from 160 tiles; the first
# three have fewer and take the 64-query form) whose lists end anywhere in a
# tile and whose blocks straddle tiles (b = 160, 200), neighbouring blocks,
# zero tokens; leaves of 1024 and more (from 512 tiles; d_h 64: of 2560 and
# more, from 1024 tiles, the case below that line takes the 64-query form)
# that end in a tile's first, third and last wave
LEVELS, LEAF = "sparse_fwd_levels_wide", "sparse_fwd_leaf_wide"
WIDE_CASES = [
    (_w("c-bf16-d128-k160-1500", 1, 2, 1500, 128, 160, 64, "bf16", 0), 0, "sparse_fwd_levels"),
    (_w("c-bf16-d64-k200-1111-padded", 2, 1, 1111, 64, 200, 64, "bf16", 0, recipe="clustered"), 0, "sparse_fwd_levels"),
    (_w("c-bf16-d64-k128-1300-nbr1", 1, 1, 1300, 64, 128, 64, "bf16", 0), 1, "sparse_fwd_levels"),
    (_w("c-bf16-d128-k160-10x1500", 1, 10, 1500, 128, 160, 64, "bf16", 0), 0, LEVELS),
    (_w("c-bf16-d64-k200-18x1111-padded", 2, 9, 1111, 64, 200, 64, "bf16", 0, recipe="clustered"), 0, LEVELS),
    (_w("c-bf16-d64-k128-10x1300-nbr1", 1, 10, 1300, 64, 128, 64, "bf16", 0), 1, LEVELS),
    (_w("c-bf16-d128-leaf1025", 1, 32, 2049, 128, 128, 64, "bf16", 1100), 0, LEAF),
    (_w("c-bf16-d64-leaf1110", 3, 20, 1110, 64, 128, 64, "bf16", 1200, recipe="clustered"), 0, "sparse_fwd_leaf"),
    (_w("c-bf16-d64-leaf2570", 7, 7, 2570, 64, 128, 64, "bf16", 2600, recipe="clustered"), 0, LEAF),
    (_w("c-bf16-d128-leaf1152-k64", 2, 29, 1152, 128, 64, 64, "bf16", 1152, recipe="clustered"), 0, LEAF),
]


@pytest.mark.parametrize("w,nbr,kernel", WIDE_CASES, ids=[c[0].name for c in WIDE_CASES])
def test_ragged_causal_wide_tiles(w, nbr, kernel):
    _check(w, neighbors=nbr, heads={(0, 0), (w.B - 1, w.H - 1)}, launches=[kernel])


# the leaf's dQ in 128-query tiles (d_h 64: leaves from 224 and 512 tiles; d_h
# 128: from 1024 and 256 tiles, or 448 and 2048 tiles): W' of 64 columns (r >
# 128), leaves of one query past a tile, a leaf whose last tiles hold no token,
# d_h 64 and 128; the last case, below the line, takes the 64-query form
WIDE_LEAF_BWD_CASES = [
    _w("c-bf16-d64-r32-leaf225", 4, 16, 900, 64, 64, 32, "bf16", 230, recipe="clustered"),
    _w("c-bf16-d64-r64-leaf257", 4, 22, 514, 64, 64, 64, "bf16", 260),
    _w("c-bf16-d128-r256-leaf1153", 1, 26, 1153, 128, 128, 256, "bf16", 1200),
    _w("c-bf16-d64-r192-leaf1024", 2, 16, 2047, 64, 64, 192, "bf16", 1030, recipe="clustered"),
    _w("c-bf16-d128-r16-leaf513", 3, 22, 4099, 128, 64, 16, "bf16", 520),
    _w("c-bf16-d64-r32-leaf193", 2, 16, 772, 64, 64, 32, "bf16", 200, recipe="clustered"),
]


@pytest.mark.parametrize("w", WIDE_LEAF_BWD_CASES, ids=[w.name for w in WIDE_LEAF_BWD_CASES])
def test_ragged_causal_wide_leaf_backward(w):
    wide = "leaf193" not in w.name
    _check(w, heads={(0, 0), (w.B - 1, w.H - 1)}, launches=["sparse_leaf_bwd_wide" if wide else "sparse_leaf_bwd"])


def test_ragged_causal_with_neighbours():
    _check(_w("c-bf16-d128-2000-leaf250-nbr1", 1, 1, 2000, 128, 64, 128, "bf16", 300, seed=81), neighbors=1)


@pytest.mark.timeout(900)
def test_text_setting_full_size_sampled_rows():
    """All 16 heads of the text setting at N = 32000 on 368 sampled rows each."""
    # N = 32000 (the ArXiv length): the oracle computes sampled rows only
    w = W.TEXT_32K
    mask = np.zeros(w.N, np.uint8)
    rng = np.random.default_rng(8)
    mask[rng.choice(w.N, 200, replace=False)] = 1
    mask[:64] = 1
    mask[-64:] = 1
    mask[3990:4010] = 1        # across the first leaf boundary
    mask[15990:16010] = 1      # across the top-level halves
    _check(w, q_mask=mask)
