"""GPU parity of bigbird_attn_fwd against the fp64 oracle, through the C ABI.

Tolerances (max abs error of O and LSE): 1e-4 for fp32 storage, 2e-2 for bf16.
"""
import math

import numpy as np
import pytest

import bigbird_inputs as inp
import oracle
import paper_2007_14062_amd as bb
from gpu_util import device_qkv, sample_rows, to_host

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "bf16": 2e-2}


def torch_mod():
    import torch
    assert torch.cuda.is_available()
    return torch


def run_fwd(t, rand_idx, dtype, g, w, scale, key_mask=None, mode=0):
    torch = torch_mod()
    Q, K, V = device_qkv(t, dtype)
    ridx = torch.from_numpy(np.ascontiguousarray(rand_idx)).to("cuda:0")
    km = None if key_mask is None else torch.from_numpy(key_mask).to("cuda:0")
    O, LSE = bb.bigbird_attn_fwd(Q, K, V, ridx, g=g, w=w, scale=scale, key_padding_mask=km,
                                 global_mode=mode)
    torch.cuda.synchronize()
    return O, LSE


def check_full(t, rand_idx, dtype, b, g, w, scale, key_mask=None, mode=0, tag=""):
    O, LSE = run_fwd(t, rand_idx, dtype, g, w, scale, key_mask, mode)
    Oref, Lref = oracle.attn_fwd(t["Q"], t["K"], t["V"], rand_idx, b, g, w, scale,
                                 key_mask=key_mask, global_mode=mode)
    Oh, Lh = to_host(O), to_host(LSE)
    finite = np.isfinite(Lref)
    assert (np.isneginf(Lh) == ~finite).all(), tag
    err_o = np.abs(Oh - Oref).max()
    err_l = np.abs(Lh[finite] - Lref[finite]).max() if finite.any() else 0.0
    print(f"{tag}: max|dO|={err_o:.3e} max|dLSE|={err_l:.3e}")
    assert err_o <= TOL[dtype], (tag, err_o)
    assert err_l <= TOL[dtype], (tag, err_l)
    return O, LSE


def test_cfg1_fp32_small_full_parity():
    wl = inp.WORKLOADS["cfg1_fp32_small"]
    t = inp.workload_tensors(wl)
    ridx = bb.bigbird_make_rand_idx(wl.H, wl.n, wl.b, wl.g, wl.w, wl.r, wl.pattern_seed)
    assert (ridx == oracle.make_rand_idx(wl.H, wl.n, wl.b, wl.g, wl.w, wl.r, wl.pattern_seed)).all()
    check_full(t, ridx, "f32", wl.b, wl.g, wl.w, wl.scale, tag="cfg1 fp32")


def test_cfg1_shape_bf16_full_parity():
    wl = inp.WORKLOADS["cfg1_fp32_small"]
    t = inp.make_tensors(wl.B, wl.H, wl.n, wl.d, 100, "bf16")
    ridx = bb.bigbird_make_rand_idx(wl.H, wl.n, wl.b, wl.g, wl.w, wl.r, wl.pattern_seed)
    check_full(t, ridx, "bf16", wl.b, wl.g, wl.w, wl.scale, tag="cfg1-shape bf16")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_ragged_shapes_leading_globals(dtype):
    """B*H = 6 (not a multiple of the 8 dies), nb = 10, 3 leading global blocks, w = 5, r = 2."""
    B, H, n, g, w, r = 2, 3, 640, 3, 5, 2
    t = inp.make_tensors(B, H, n, 64, 7, dtype)
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 9, bb.BB_GLOBAL_LEADING)
    check_full(t, ridx, dtype, 64, g, w, 0.2, mode=bb.BB_GLOBAL_LEADING, tag=f"ragged {dtype}")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_full_coverage_equals_full_attention(dtype):
    """Window widened over every block: every row is split over several workgroups."""
    B, H, n = 1, 2, 1280
    nb = n // 64
    t = inp.make_tensors(B, H, n, 64, 8, dtype)
    empty = np.full((H, nb, 0), -1, dtype=np.int32)
    O, _ = check_full(t, empty, dtype, 64, 0, 2 * nb - 1, 0.125, tag=f"full coverage {dtype}")
    # the same numbers must come out when all blocks are global instead
    O2, _ = check_full(t, empty, dtype, 64, nb, 1, 0.125, tag=f"all global {dtype}")
    assert np.abs(to_host(O) - to_host(O2)).max() <= TOL[dtype]


@pytest.mark.parametrize("H", [2, 20])  # a workgroup per row; waves' streams (here and below)
@pytest.mark.parametrize("g,w,r", [(0, 1, 0), (1, 1, 0), (0, 3, 2), (2, 3, 0), (1, 7, 4)])
def test_degenerate_patterns(g, w, r, H):
    B, n = 1, 1024
    t = inp.make_tensors(B, H, n, 64, 9, "bf16")
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 3)
    check_full(t, ridx, "bf16", 64, g, w, 0.125, tag=f"g{g} w{w} r{r}")


@pytest.mark.parametrize("n", [2048, 3072])
def test_summarisation_encoder_lengths(n):
    """Encoder lengths of the summarisation experiments (App. E.5): nb = 32 and 48 (not a power
    of two), 16 heads as in the large model (B*H = 16: two rounds over the 8 dies), two of the
    heads compared in full."""
    B, H, g, w, r = 1, 16, 2, 3, 3
    t = inp.make_tensors(B, H, n, 64, 31 + n, "bf16")
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 11)
    O, LSE = run_fwd(t, ridx, "bf16", g, w, 0.125)
    Oh, Lh = to_host(O), to_host(LSE)
    for h in (3, 15):
        sub = {k: v[:, h:h + 1] for k, v in t.items() if k in ("Q", "K", "V")}
        Oref, Lref = oracle.attn_fwd(sub["Q"], sub["K"], sub["V"], ridx[h:h + 1], 64, g, w, 0.125)
        err_o = np.abs(Oh[:, h:h + 1] - Oref).max()
        err_l = np.abs(Lh[:, h:h + 1] - Lref).max()
        print(f"n={n} head {h}: max|dO|={err_o:.3e} max|dLSE|={err_l:.3e}")
        assert err_o <= TOL["bf16"] and err_l <= TOL["bf16"], (n, h, err_o, err_l)


def test_single_block_sequence():
    t = inp.make_tensors(2, 1, 64, 64, 10, "f32")
    empty = np.full((1, 1, 0), -1, dtype=np.int32)
    check_full(t, empty, "f32", 64, 1, 1, 0.125, tag="nb=1 global")
    check_full(t, empty, "f32", 64, 0, 1, 0.125, tag="nb=1 window")


@pytest.mark.parametrize("H", [2, 20])
def test_table_with_duplicates_and_negative_entries(H):
    """Entries < 0 are ignored; entries repeating the window, a global block or each other count once."""
    B, n, g, w, r = 1, 1024, 2, 3, 4
    t = inp.make_tensors(B, H, n, 64, 11, "bf16")
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 5)
    ridx[0, 5] = [-1, 9, 9, 12]
    ridx[0, 6] = [6, 0, 7, 3]
    ridx[1, 8] = [-1, -1, -1, -1]
    ridx[1, 9] = [15, 2, 2, 2]
    check_full(t, ridx, "bf16", 64, g, w, 0.125, tag="dirty table")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_key_padding_unaligned_and_empty_rows(dtype):
    B, H, n, g, w, r = 3, 2, 1024, 2, 3, 3
    t = inp.make_tensors(B, H, n, 64, 12, dtype)
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 6)
    km = np.ones((B, n), dtype=np.uint8)
    km[0, 700:] = 0                   # tail padding, not block aligned; last global block padded
    km[1, :64] = 0                    # first global block padded away
    km[1, 300:309] = 0                # a hole inside a block
    km[1, 640:768] = 0                # two fully padded interior blocks
    km[2, :] = 0                      # no valid key at all: O = 0, LSE = -inf everywhere
    O, LSE = check_full(t, ridx, dtype, 64, g, w, 0.125, key_mask=km, tag=f"padding {dtype}")
    assert (to_host(O)[2] == 0).all() and np.isneginf(to_host(LSE)[2]).all()


@pytest.mark.parametrize("tail", [1, 2, 31, 32, 33, 63])
@pytest.mark.parametrize("mode,g,r", [(bb.BB_GLOBAL_FIRST_LAST, 2, 3), (bb.BB_GLOBAL_LEADING, 3, 0)])
@pytest.mark.parametrize("H", [2, 8])
def test_blocks_with_padded_keys_inside(tail, mode, g, r, H):
    """bf16: validity ends `tail` keys into a block, at the edges of the 32-key units; a hole of every
    residue; a whole sequence of `tail` keys (rows with no full block); mask bytes of any non-zero value;
    K rows of padded keys hold NaN.  (Same tolerance as everywhere: the keys left out change nothing else.)"""
    torch = torch_mod()
    B, n, w = 3, 1024, 3
    t = inp.make_tensors(B, H, n, 64, 40 + tail, "bf16")
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 6, mode)
    km = np.full((B, n), 0x80, dtype=np.uint8)
    km[0, 640 + tail:] = 0
    km[1, 128:128 + tail] = 0
    km[1, 300:300 + 2 * tail] = 0
    km[2, tail:] = 0
    Oref, Lref = oracle.attn_fwd(t["Q"], t["K"], t["V"], ridx, 64, g, w, 0.125, key_mask=(km != 0).astype(np.uint8),
                                 global_mode=mode)
    Q, K, V = device_qkv(t, "bf16")
    kmd = torch.from_numpy(km).to("cuda:0")
    K.masked_fill_((kmd == 0)[:, None, :, None], float("nan"))
    O, LSE = bb.bigbird_attn_fwd(Q, K, V, torch.from_numpy(ridx).to("cuda:0"), g=g, w=w, scale=0.125,
                                 key_padding_mask=kmd, global_mode=mode)
    Oh, Lh = to_host(O), to_host(LSE)
    fin = np.isfinite(Lref)
    assert (np.isneginf(Lh) == ~fin).all()
    err_o, err_l = np.abs(Oh - Oref).max(), np.abs(Lh[fin] - Lref[fin]).max()
    print(f"tail {tail} mode {mode}: max|dO|={err_o:.3e} max|dLSE|={err_l:.3e}")
    assert err_o <= TOL["bf16"] and err_l <= TOL["bf16"]


@pytest.mark.parametrize("H,nb,g,w,r", [
    (2, 9, 2, 3, 3), (40, 9, 1, 3, 0), (40, 10, 2, 5, 3),  # rows by a workgroup; an item for each wave
    (24, 20, 1, 15, 4),                                    # two slices to a row, one or two for each wave
    (100, 12, 2, 3, 3),                                    # whole rows, three for each wave: from either kind to either kind
])
@pytest.mark.parametrize("skip", [False, True])
@pytest.mark.parametrize("gain", [1.0, 40.0])
def test_running_maximum_in_the_streams(H, nb, g, w, r, skip, gain):
    """bf16: items with and without padded keys inside a block, side by side in a wave's stream at the last shape (its batch
    entry 1), lists of one block up to two slices of 16; blocks whose first or second 32 keys, or all but one, are
    padded.  LSE is an fp32 sum there: 1e-5 of its size, where rounding the probabilities first would give 2^-9."""
    torch = torch_mod()
    B, n = 3, nb * 64
    t = inp.make_tensors(B, H, n, 64, 300 + nb, "bf16")
    Qg = t["Q"] * np.float32(gain)          # a power of two times the rounded values would be exact; round again
    u = np.ascontiguousarray(Qg, dtype=np.float32).view(np.uint32)
    bits = ((u + 0x7fff + ((u >> 16) & 1)) >> 16).astype(np.uint16)
    t["Q_bits"], t["Q"] = bits, (bits.astype(np.uint32) << 16).view(np.float32)
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 5)
    km = np.ones((B, n), dtype=np.uint8)
    km[0, :32] = 0                          # first half of the first global block
    km[0, 3 * 64 + 32:4 * 64] = 0           # second half of block 3
    km[0, 5 * 64:5 * 64 + 63] = 0           # all but the last key of block 5
    km[1, (nb - 2) * 64 + 1:] = 0           # one key of the last block that has any
    km[2] = np.random.default_rng(nb).integers(0, 2, n)  # every block cut
    mode = bb.BB_SKIP_PADDED_QUERY_BLOCKS if skip else 0
    kw = dict(key_mask=km)
    Oref, Lref = oracle.attn_fwd(t["Q"], t["K"], t["V"], ridx, 64, g, w, 0.125, **kw)
    Q, K, V = device_qkv(t, "bf16")
    O, LSE = bb.bigbird_attn_fwd(Q, K, V, torch.from_numpy(ridx).to("cuda:0"), g=g, w=w, scale=0.125,
                                 key_padding_mask=torch.from_numpy(km).to("cuda:0"), global_mode=mode)
    Oh, Lh = to_host(O), to_host(LSE)
    if skip:
        dead = ~km.reshape(B, nb, 64).any(axis=2).repeat(64, axis=1)
        Oref = np.where(dead[:, None, :, None], 0.0, Oref)
        Lref = np.where(dead[:, None, :], -np.inf, Lref)
    fin = np.isfinite(Lref)
    assert (np.isneginf(Lh) == ~fin).all()
    assert np.abs(Oh - Oref).max() <= TOL["bf16"]
    # batch entry 2: every list has a cut block; others: items without one sum the rounded probabilities
    err = np.abs(np.where(fin, Lh, 0) - np.where(fin, Lref, 0)) / np.maximum(1.0, np.abs(np.where(fin, Lref, 0)))
    assert err[2].max() <= 1e-5 and err.max() <= 2.0 ** -8


@pytest.mark.parametrize("B,H,nb,g,w,r", [
    (1, 1, 1, 1, 1, 0), (1, 1, 3, 0, 1, 0), (1, 3, 9, 2, 3, 3), (1, 16, 18, 2, 3, 3), (1, 17, 17, 2, 3, 3),
    (1, 2, 66, 1, 3, 60), (1, 2, 70, 1, 3, 61), (1, 1, 130, 2, 3, 12), (1, 6, 48, 4, 9, 3)])
@pytest.mark.parametrize("masked", [False, True])
def test_rows_by_workgroup(B, H, nb, g, w, r, masked):
    """Small launches (a workgroup per row) and the first ones past the limit of 288 rows; key lists of 1, 2, 3,
    9, 16, 64 and 65 blocks dealt out to four waves; global rows of one and of several workgroups (48 blocks to one, where
    lists of 16 leave no room for two); a mask that leaves waves without a block."""
    n = nb * 64
    t = inp.make_tensors(B, H, n, 64, 70 + nb, "bf16")
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 8)
    km = None
    if masked:
        km = np.zeros((B, n), dtype=np.uint8)
        km[:, n // 2 - 5:n // 2 + 60] = 1
    check_full(t, ridx, "bf16", 64, g, w, 0.125, key_mask=km, tag=f"rows B{B} H{H} nb{nb} r{r} mask{masked}")


@pytest.mark.parametrize("B,H,nb,g,w,r", [
    (1, 2, 1, 1, 1, 0), (2, 3, 2, 1, 1, 0), (1, 4, 3, 2, 3, 0), (2, 2, 4, 2, 3, 0),  # a pair for a wave, or none
    (1, 2, 8, 2, 3, 3), (1, 3, 12, 2, 3, 3), (1, 2, 17, 1, 5, 9),                    # two; three; five and four
])
@pytest.mark.parametrize("drop", [False, True])
def test_short_rows_with_the_running_maximum(B, H, nb, g, w, r, drop):
    """Rows by a workgroup whose waves have one to five pairs: every block holds padded keys (a pair's K rows of these are
    NaN without dropout), and under dropout as well.  LSE is an fp32 sum: 1e-5 of its size."""
    torch = torch_mod()
    n = nb * 64
    t = inp.make_tensors(B, H, n, 64, 900 + nb, "bf16")
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 3)
    km = np.random.default_rng(nb).integers(0, 2, (B, n)).astype(np.uint8)
    Q, K, V = device_qkv(t, "bf16")
    kmd = torch.from_numpy(km).to("cuda:0")
    rd = torch.from_numpy(ridx).to("cuda:0")
    kw = dict(g=g, w=w, scale=0.125, key_padding_mask=kmd)
    args = (t["Q"], t["K"], t["V"], ridx, 64, g, w, 0.125)
    if drop:
        O, LSE = bb.bigbird_attn_fwd_dropout(Q, K, V, rd, p_drop=0.25, seed=11, **kw)
        Oref, Lref = oracle.attn_fwd_dropout(*args, 0.25, 11, key_mask=km)
    else:
        K.masked_fill_((kmd == 0)[:, None, :, None], float("nan"))
        O, LSE = bb.bigbird_attn_fwd(Q, K, V, rd, **kw)
        Oref, Lref = oracle.attn_fwd(*args, key_mask=km)
    Oh, Lh = to_host(O), to_host(LSE)
    fin = np.isfinite(Lref)
    assert (np.isneginf(Lh) == ~fin).all()
    assert np.abs(Oh - Oref).max() <= TOL["bf16"]
    assert (np.abs(Lh[fin] - Lref[fin]) / np.maximum(1.0, np.abs(Lref[fin]))).max() <= 1e-5


@pytest.mark.parametrize("B,H,nb,g,w,r", [
    (5, 16, 9, 2, 3, 3),    # four waves: rows of fewer than 16 blocks
    (3, 16, 16, 2, 3, 3),   # eight waves to a workgroup: two blocks of a global row each
    (4, 7, 16, 1, 3, 0),    # the same with short lists, a wave to a SIMD if there were four
    (3, 11, 20, 1, 17, 2),  # four waves: non-global rows in two slices
    (2, 10, 48, 4, 9, 3),   # eight: lists of a whole slice of 16
    (1, 10, 80, 2, 3, 3),   # global rows by two workgroups of eight waves
    (1, 9, 66, 2, 3, 3),    # by three of four
    (4, 8, 32, 2, 3, 3),
    (5, 8, 33, 2, 3, 3),    # 30 workgroups of eight waves to a die
    (6, 6, 36, 2, 3, 3),    # 32
    (6, 8, 33, 2, 3, 3),    # 36 would not fit: four waves, 16 blocks of a global row each
    (1, 8, 64, 2, 3, 3),    # a third of the units: four waves with 8 blocks, two workgroups to a global row and a merge launch
])
@pytest.mark.parametrize("case", ["plain", "masked", "skip", "drop"])
def test_launches_of_medium_size(B, H, nb, g, w, r, case):
    n = nb * 64
    t = inp.make_tensors(B, H, n, 64, 600 + nb, "bf16")
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 8)
    torch = torch_mod()
    km = None
    if case in ("masked", "skip"):
        km = np.ones((B, n), dtype=np.uint8)
        km[0, n // 2 + 5:] = 0
        km[B - 1, 3:40] = 0
        km[B - 1, n - 130:n - 64] = 0
    args = (t["Q"], t["K"], t["V"], ridx, 64, g, w, 0.125)
    kw = dict(g=g, w=w, scale=0.125, key_padding_mask=None if km is None else torch.from_numpy(km).to("cuda:0"),
              global_mode=bb.BB_SKIP_PADDED_QUERY_BLOCKS if case == "skip" else 0)
    Q, K, V = device_qkv(t, "bf16")
    rd = torch.from_numpy(ridx).to("cuda:0")
    if case == "drop":
        O, LSE = bb.bigbird_attn_fwd_dropout(Q, K, V, rd, p_drop=0.25, seed=3, **kw)
        Oref, Lref = oracle.attn_fwd_dropout(*args, 0.25, 3)
    else:
        O, LSE = bb.bigbird_attn_fwd(Q, K, V, rd, **kw)
        Oref, Lref = oracle.attn_fwd(*args, key_mask=km, skip_padded_query_blocks=case == "skip")
    fin = np.isfinite(Lref)
    assert (np.isneginf(to_host(LSE)) == ~fin).all()
    err_o, err_l = np.abs(to_host(O) - Oref).max(), np.abs(to_host(LSE)[fin] - Lref[fin]).max()
    print(f"B{B} H{H} nb{nb} {case}: max|dO|={err_o:.3e} max|dLSE|={err_l:.3e}")
    assert err_o <= TOL["bf16"] and err_l <= TOL["bf16"]


def test_zero_queries_closed_form_and_pattern_readback():
    """Q = 0 => O_i = mean of V over N(i), LSE_i = ln|N(i)|; V one-hot per key block spells out
    the neighbour set the kernel used, which must be the table's."""
    torch = torch_mod()
    B, H, n, g, w, r = 1, 3, 4096, 2, 3, 3
    nb = n // 64
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 1)
    V = np.zeros((B, H, n, 64), dtype=np.float32)
    for k in range(n):
        V[:, :, k, k // 64] = 1.0
    t = {"Q": np.zeros_like(V), "K": np.random.default_rng(0).standard_normal(V.shape).astype(np.float32),
         "V": V}
    O, LSE = run_fwd(t, ridx, "f32", g, w, 0.125)
    Oh, Lh = to_host(O), to_host(LSE)
    for h in range(H):
        for j in range(nb):
            want = set(range(nb)) if j in (0, nb - 1) else \
                {0, nb - 1, j - 1, j, j + 1} | {int(x) for x in ridx[h, j]}
            cnt = 64 * len(want)
            rows = Oh[0, h, j * 64:(j + 1) * 64]
            got = {c for c in range(64) if rows[0, c] > 0}
            assert got == want, (h, j)
            assert np.abs(rows[:, sorted(want)] - 64.0 / cnt).max() < 1e-6
            assert np.abs(Lh[0, h, j * 64:(j + 1) * 64] - math.log(cnt)).max() < 1e-5


@pytest.mark.parametrize("H", [3, 6])
def test_runs_are_bit_reproducible(H):
    torch = torch_mod()
    t = inp.make_tensors(2, H, 2048, 64, 13, "bf16")
    ridx = bb.bigbird_make_rand_idx(H, 2048, 64, 2, 3, 3, 2)
    O1, L1 = run_fwd(t, ridx, "bf16", 2, 3, 0.125)
    O2, L2 = run_fwd(t, ridx, "bf16", 2, 3, 0.125)
    assert torch.equal(O1.view(torch.int16), O2.view(torch.int16)) and torch.equal(L1, L2)


def _sampled_parity(wl, n_bh=3, seed=0):
    t = inp.workload_tensors(wl)
    ridx = bb.bigbird_make_rand_idx(wl.H, wl.n, wl.b, wl.g, wl.w, wl.r, wl.pattern_seed)
    assert (ridx == oracle.make_rand_idx(wl.H, wl.n, wl.b, wl.g, wl.w, wl.r, wl.pattern_seed)).all()
    km = t.get("key_mask")
    O, LSE = run_fwd(t, ridx, wl.dtype, wl.g, wl.w, wl.scale, km)
    Oh, Lh = to_host(O), to_host(LSE)
    assert np.isfinite(Oh).all()
    rng = np.random.default_rng(seed)
    worst_o = worst_l = 0.0
    picks = {(0, 0), (wl.B - 1, wl.H - 1)} | {(int(rng.integers(wl.B)), int(rng.integers(wl.H)))
                                             for _ in range(n_bh)}
    for (bi, h) in sorted(picks):
        rows = sample_rows(wl.nb, wl.b, rng)
        Or, Lr = oracle.attn_fwd_rows(t["Q"], t["K"], t["V"], ridx, wl.b, wl.g, wl.w, wl.scale,
                                      bi, h, rows, key_mask=km)
        worst_o = max(worst_o, np.abs(Oh[bi, h, rows] - Or).max())
        worst_l = max(worst_l, np.abs(Lh[bi, h, rows] - Lr).max())
    print(f"{wl.name}: sampled max|dO|={worst_o:.3e} max|dLSE|={worst_l:.3e}")
    assert worst_o <= TOL[wl.dtype] and worst_l <= TOL[wl.dtype]
    return Lh


def test_cfg2_bert_base_sampled_rows():
    _sampled_parity(inp.WORKLOADS["cfg2_bert_base"])


def test_cfg3_key_padding_sampled_rows():
    _sampled_parity(inp.WORKLOADS["cfg3_key_padding"])


def test_cfg5_long_sequence_sampled_rows():
    _sampled_parity(inp.WORKLOADS["cfg5_long_seq"], n_bh=2)


def test_maximum_length_sampled_rows():
    """n = 65 536 (nb = 1024): sixteen workgroups and
    a merge per global row, key lists built from a 3072-entry table row set; sampled rows."""
    wl = inp.Workload("max_len", B=1, H=2, n=65536, pattern_seed=21, data_seed=321)
    _sampled_parity(wl, n_bh=1)


def test_cfg2_lse_bound_holds_for_every_row():
    """A property that holds at any size: sum_k exp(S_ik - LSE_i) = 1 implies
    max_k S_ik <= LSE_i <= max_k S_ik + ln|N(i)|; checked here through the Q = 0-free route
    LSE >= ln|N(i)| + min S and <= ln|N(i)| + max S with |S| <= scale |q||k|."""
    wl = inp.WORKLOADS["cfg2_bert_base"]
    t = inp.workload_tensors(wl)
    ridx = bb.bigbird_make_rand_idx(wl.H, wl.n, wl.b, wl.g, wl.w, wl.r, wl.pattern_seed)
    O, LSE = run_fwd(t, ridx, wl.dtype, wl.g, wl.w, wl.scale)
    Lh, Oh = to_host(LSE), to_host(O)
    qn = np.linalg.norm(t["Q"].astype(np.float64), axis=-1)
    kmax = np.linalg.norm(t["K"].astype(np.float64), axis=-1).max(axis=-1)[..., None]
    bound = wl.scale * qn * kmax
    counts = np.full(wl.nb, 8 * 64.0)
    counts[[1, wl.nb - 2]] = 7 * 64.0
    counts[[0, wl.nb - 1]] = wl.n
    lc = np.log(np.repeat(counts, 64))[None, None, :]
    assert (Lh <= lc + bound + 1e-3).all() and (Lh >= lc - bound - 1e-3).all()
    # outputs are convex combinations of V rows
    vmax = np.abs(t["V"]).max()
    assert np.abs(Oh).max() <= vmax + 1e-2


def test_seeded_sweep_of_small_configurations():
    """Forty seeded combinations of batch, heads, length, pattern, global placement, padding and
    storage type (every legal corner the other tests do not name), each compared in full."""
    rng = np.random.default_rng(20260)
    done = 0
    while done < 40:
        nb = int(rng.integers(1, 21))
        g = int(rng.integers(0, min(nb, 3) + 1))
        w = int(rng.choice([1, 3, 5, 7]))
        r = int(rng.integers(0, 5))
        B, H = int(rng.integers(1, 4)), int(rng.integers(1, 5))
        mode = int(rng.integers(0, 2))
        dtype = "bf16" if rng.random() < 0.7 else "f32"
        n = nb * 64
        try:
            ridx = oracle.make_rand_idx(H, n, 64, g, w, r, int(rng.integers(0, 1000)), mode)
        except ValueError:
            continue  # fewer than r candidate blocks somewhere: not a legal pattern
        t = inp.make_tensors(B, H, n, 64, int(rng.integers(0, 10000)), dtype)
        km = None
        if rng.random() < 0.5:
            km = np.ones((B, n), dtype=np.uint8)
            for bi in range(B):
                km[bi, int(rng.integers(0, n + 1)):] = 0          # valid prefix of any length, 0 included
                if rng.random() < 0.3:
                    a = int(rng.integers(0, n)); km[bi, a:a + int(rng.integers(1, 130))] = 0   # a hole
        scale = float(rng.choice([0.125, 0.2, 0.05]))
        check_full(t, ridx, dtype, 64, g, w, scale, key_mask=km, mode=mode,
                   tag=f"sweep {done}: B{B} H{H} nb{nb} g{g} w{w} r{r} mode{mode} {dtype} pad{km is not None}")
        done += 1


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_workspace_of_the_standard_slices(dtype):
    """A small launch whose fp32 form cuts rows finer where the workspace has room for it: with room for
    the standard slices alone (8 blocks: 2 global rows x 2 slices x 2 heads, and the item counters) both types run."""
    torch = torch_mod()
    B, H, n, g, w, r = 1, 2, 1024, 2, 3, 3
    t = inp.make_tensors(B, H, n, 64, 14, dtype)
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 7)
    nbytes = 8 * (64 * 64 + 2 * 64) * 4 + 8 * 128
    assert nbytes < bb.bigbird_attn_workspace_bytes(B, H, n, 64, 64, g, w, r)
    # the buffer ends where its size says: what lies behind it stays as it was
    buf = torch.full((nbytes + 4096,), 0xA5, dtype=torch.uint8, device="cuda:0")
    Q, K, V = device_qkv(t, dtype)
    O, LSE = bb.bigbird_attn_fwd(Q, K, V, torch.from_numpy(ridx).to("cuda:0"), g=g, w=w, scale=0.125, workspace=buf[:nbytes])
    Oref, Lref = oracle.attn_fwd(t["Q"], t["K"], t["V"], ridx, 64, g, w, 0.125)
    assert np.abs(to_host(O) - Oref).max() <= TOL[dtype] and np.abs(to_host(LSE) - Lref).max() <= TOL[dtype]
    assert (buf[nbytes:] == 0xA5).all()
    with pytest.raises(bb.BigBirdError):
        bb.bigbird_attn_fwd(Q, K, V, torch.from_numpy(ridx).to("cuda:0"), g=g, w=w, scale=0.125, workspace=buf[:nbytes - 256])
