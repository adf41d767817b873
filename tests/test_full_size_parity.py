"""GPU parity at the full sizes of the benchmark workloads, compared in full (not sampled),
and cases that leave the comfortable range of the logits.

Tolerances as everywhere: max abs error 2e-2 for bf16 outputs and gradients (1e-4 for fp32).
The dense fp64 oracle takes about a tenth of a second per (batch, head) slice at n = 4096 and
about fifteen seconds per slice at n = 16 384 on the GPU machine's host cores.
"""
import math

import numpy as np
import pytest

import bigbird_inputs as inp
import oracle
import paper_2007_14062_amd as bb
from gpu_util import device_qkv, device_tensor, to_host

pytestmark = pytest.mark.gpu

TOL = 2e-2


def _fwd(t, ridx, g, w, scale, km=None, mode=0):
    import torch
    assert torch.cuda.is_available()
    Q, K, V = device_qkv(t, "bf16")
    r_d = torch.from_numpy(np.ascontiguousarray(ridx)).to("cuda:0")
    km_d = None if km is None else torch.from_numpy(km).to("cuda:0")
    O, LSE = bb.bigbird_attn_fwd(Q, K, V, r_d, g=g, w=w, scale=scale, key_padding_mask=km_d, global_mode=mode)
    torch.cuda.synchronize()
    return (Q, K, V, r_d, km_d), O, LSE


def _bwd(dev, O, LSE, t, g, w, scale, mode=0):
    import torch
    Q, K, V, r_d, km_d = dev
    dO = device_tensor(t, "dO", "bf16")
    dQ, dK, dV = bb.bigbird_attn_bwd(Q, K, V, O, LSE, dO, r_d, g=g, w=w, scale=scale, key_padding_mask=km_d,
                                     global_mode=mode)
    torch.cuda.synchronize()
    return to_host(dQ), to_host(dK), to_host(dV)


def _fwd_errors(Oh, Lh, Oref, Lref):
    finite = np.isfinite(Lref)
    assert (np.isneginf(Lh) == ~finite).all()
    return np.abs(Oh - Oref).max(), (np.abs(Lh[finite] - Lref[finite]).max() if finite.any() else 0.0)


def test_cfg2_every_slice_in_full():
    """The benchmark workload itself, in the launch the benchmark times: all 48 (batch, head)
    slices, every row, against the dense oracle."""
    wl = inp.WORKLOADS["cfg2_bert_base"]
    t = inp.workload_tensors(wl)
    ridx = bb.bigbird_make_rand_idx(wl.H, wl.n, wl.b, wl.g, wl.w, wl.r, wl.pattern_seed)
    _, O, LSE = _fwd(t, ridx, wl.g, wl.w, wl.scale)
    Oh, Lh = to_host(O), to_host(LSE)
    worst_o = worst_l = 0.0
    for bi in range(wl.B):
        sl = slice(bi, bi + 1)
        Oref, Lref = oracle.attn_fwd(t["Q"][sl], t["K"][sl], t["V"][sl], ridx, wl.b, wl.g, wl.w, wl.scale)
        eo, el = _fwd_errors(Oh[sl], Lh[sl], Oref, Lref)
        worst_o, worst_l = max(worst_o, eo), max(worst_l, el)
    print(f"cfg2, all {wl.B * wl.H} slices in full: max|dO|={worst_o:.3e} max|dLSE|={worst_l:.3e}")
    assert worst_o <= TOL and worst_l <= TOL


def test_cfg3_one_full_slice_per_batch_entry():
    """Key-padding workload: every batch entry has its own valid length, so one (batch, head)
    slice of each is compared in full (heads spread over the twelve)."""
    wl = inp.WORKLOADS["cfg3_key_padding"]
    t = inp.workload_tensors(wl)
    km = t["key_mask"]
    ridx = bb.bigbird_make_rand_idx(wl.H, wl.n, wl.b, wl.g, wl.w, wl.r, wl.pattern_seed)
    _, O, LSE = _fwd(t, ridx, wl.g, wl.w, wl.scale, km)
    Oh, Lh = to_host(O), to_host(LSE)
    worst_o = worst_l = 0.0
    for bi in range(wl.B):
        h = (5 * bi + 1) % wl.H
        sl = (slice(bi, bi + 1), slice(h, h + 1))
        Oref, Lref = oracle.attn_fwd(t["Q"][sl], t["K"][sl], t["V"][sl], ridx[h:h + 1], wl.b, wl.g, wl.w, wl.scale,
                                     key_mask=km[bi:bi + 1])
        eo, el = _fwd_errors(Oh[sl], Lh[sl], Oref, Lref)
        print(f"cfg3 (b={bi}, len={int(km[bi].sum())}, h={h}): max|dO|={eo:.3e} max|dLSE|={el:.3e}")
        worst_o, worst_l = max(worst_o, eo), max(worst_l, el)
    assert worst_o <= TOL and worst_l <= TOL


def test_cfg5_one_head_every_row():
    """n = 16 384: one of the sixteen heads against the dense oracle, all rows."""
    wl = inp.WORKLOADS["cfg5_long_seq"]
    t = inp.workload_tensors(wl)
    ridx = bb.bigbird_make_rand_idx(wl.H, wl.n, wl.b, wl.g, wl.w, wl.r, wl.pattern_seed)
    _, O, LSE = _fwd(t, ridx, wl.g, wl.w, wl.scale)
    h = 11
    sl = (slice(0, 1), slice(h, h + 1))
    Oref, Lref = oracle.attn_fwd(t["Q"][sl], t["K"][sl], t["V"][sl], ridx[h:h + 1], wl.b, wl.g, wl.w, wl.scale)
    eo, el = _fwd_errors(to_host(O)[sl], to_host(LSE)[sl], Oref, Lref)
    print(f"cfg5 head {h}, all {wl.n} rows: max|dO|={eo:.3e} max|dLSE|={el:.3e}")
    assert eo <= TOL and el <= TOL


def test_cfg4_backward_every_slice_in_full():
    """Forward + backward workload: dQ, dK, dV of all 24 (batch, head) slices."""
    wl = inp.WORKLOADS["cfg4_fwd_bwd"]
    t = inp.workload_tensors(wl)
    ridx = bb.bigbird_make_rand_idx(wl.H, wl.n, wl.b, wl.g, wl.w, wl.r, wl.pattern_seed)
    dev, O, LSE = _fwd(t, ridx, wl.g, wl.w, wl.scale)
    hQ, hK, hV = _bwd(dev, O, LSE, t, wl.g, wl.w, wl.scale)
    worst = [0.0, 0.0, 0.0]
    rel = [0.0, 0.0, 0.0]
    for bi in range(wl.B):
        sl = slice(bi, bi + 1)
        ref = oracle.attn_bwd(t["Q"][sl], t["K"][sl], t["V"][sl], t["dO"][sl], ridx, wl.b, wl.g, wl.w, wl.scale)
        for u, (got, want) in enumerate(zip((hQ[sl], hK[sl], hV[sl]), ref)):
            worst[u] = max(worst[u], np.abs(got - want).max())
            rel[u] = max(rel[u], np.abs(got - want).max() / np.abs(want).max())
    print(f"cfg4, all {wl.B * wl.H} slices in full: max|ddQ|={worst[0]:.3e} max|ddK|={worst[1]:.3e} "
          f"max|ddV|={worst[2]:.3e}; relative to the largest entry {rel[0]:.2e} {rel[1]:.2e} {rel[2]:.2e}")
    assert max(worst) <= TOL


def test_backward_at_the_longest_supported_sequence():
    """n = 16 384 (nb = 256, the backward's limit): 32 slices per global row and per global key
    column through the fixed-order reduction; one head compared in full.  One block more is refused."""
    import torch
    B, H, n, g, w, r = 1, 2, 16384, 2, 3, 3
    t = inp.make_tensors(B, H, n, 64, 611, "bf16", with_dO=True)
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 29)
    dev, O, LSE = _fwd(t, ridx, g, w, 0.125)
    hQ, hK, hV = _bwd(dev, O, LSE, t, g, w, 0.125)
    h = 1
    sl = (slice(0, 1), slice(h, h + 1))
    ref = oracle.attn_bwd(t["Q"][sl], t["K"][sl], t["V"][sl], t["dO"][sl], ridx[h:h + 1], 64, g, w, 0.125)
    errs = [np.abs(got[sl] - want).max() for got, want in zip((hQ, hK, hV), ref)]
    rels = [e / np.abs(want).max() for e, want in zip(errs, ref)]
    print(f"bwd n=16384 head {h}: max|ddQ|={errs[0]:.3e} max|ddK|={errs[1]:.3e} max|ddV|={errs[2]:.3e}; "
          f"relative to the largest entry {rels[0]:.2e} {rels[1]:.2e} {rels[2]:.2e}")
    assert max(errs) <= TOL
    # 257 blocks: refused, not computed wrongly
    n2 = 257 * 64
    z = torch.zeros((1, 1, n2, 64), dtype=torch.bfloat16, device="cuda:0")
    l = torch.zeros((1, 1, n2), dtype=torch.float32, device="cuda:0")
    r2 = torch.from_numpy(bb.bigbird_make_rand_idx(1, n2, 64, g, w, r, 1)).to("cuda:0")
    with pytest.raises(bb.BigBirdError):
        bb.bigbird_attn_bwd(z, z, z, z, l, z, r2, g=g, w=w, scale=0.125)


@pytest.mark.parametrize("n", [4096, 16384])
def test_bf16_zero_queries_pattern_readback(n):
    """Q = 0 through the bf16 kernel: every probability is exactly 1 / |N(i)|, so V one-hot per key
    block (64 blocks at a time, the others zero) spells out, column by column, which key blocks
    the kernel used for each query block: they must be the table's, at nb = 64 and at nb = 256
    (global rows over several workgroups and the merge kernel)."""
    B, H, g, w, r = 1, 2, 2, 3, 3
    nb = n // 64
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 41)
    K = np.random.default_rng(3).standard_normal((B, H, n, 64)).astype(np.float32)
    Kv, Kb = inp.round_to_bf16(K)
    zeros = np.zeros((B, H, n, 64), dtype=np.float32)
    got = [[set() for _ in range(nb)] for _ in range(H)]
    for base in range(0, nb, 64):
        V = np.zeros((B, H, n, 64), dtype=np.float32)
        for kb in range(base, min(base + 64, nb)):
            V[:, :, kb * 64:(kb + 1) * 64, kb - base] = 1.0
        Vv, Vb = inp.round_to_bf16(V)
        t = {"Q": zeros, "Q_bits": np.zeros((B, H, n, 64), dtype=np.uint16), "K": Kv, "K_bits": Kb,
             "V": Vv, "V_bits": Vb}
        _, O, LSE = _fwd(t, ridx, g, w, 0.125)
        Oh, Lh = to_host(O), to_host(LSE)
        for h in range(H):
            for j in range(nb):
                want = set(range(nb)) if j in (0, nb - 1) else \
                    {0, nb - 1, j - 1, j, j + 1} | {int(x) for x in ridx[h, j]}
                rows = Oh[0, h, j * 64:(j + 1) * 64]
                cols = {c for c in range(64) if rows[0, c] > 0}
                assert all((rows[:, c] > 0).all() == (c in cols) for c in range(64)), (h, j)
                got[h][j] |= {base + c for c in cols}
                share = 1.0 / len(want)                      # a block's 64 keys weigh 64 / (64 |blocks|)
                present = sorted(c for c in cols)
                if present:
                    assert np.abs(rows[:, present] - share).max() <= share * 2.0 ** -8, (h, j)
                assert np.abs(Lh[0, h, j * 64:(j + 1) * 64] - math.log(64 * len(want))).max() < 1e-4, (h, j)
    for h in range(H):
        for j in range(nb):
            want = set(range(nb)) if j in (0, nb - 1) else \
                {0, nb - 1, j - 1, j, j + 1} | {int(x) for x in ridx[h, j]}
            assert got[h][j] == want, (h, j)


def _scaled_key_blocks(t, factors):
    """K with key block k multiplied by factors[k] (bf16 again after the multiplication)."""
    K = t["K"].astype(np.float32).copy()
    for k, f in enumerate(factors):
        K[:, :, k * 64:(k + 1) * 64] *= np.float32(f)
    vals, bits = inp.round_to_bf16(K)
    out = dict(t)
    out["K"], out["K_bits"] = vals, bits
    return out


@pytest.mark.parametrize("H,mask", [(2, ""), (20, ""), (20, "masked"), (20, "skip")])  # a workgroup per row; waves' streams
@pytest.mark.parametrize("case", ["growing", "decreasing", "growing_hot", "decreasing_hot"])
def test_row_maxima_that_move_along_the_key_list(case, H, mask):
    """Logits whose size changes from key block to key block, so that a row's maximum moves (up or
    down) several times along its key list.  At scale 0.125 the sums stay in the range of the
    fixed-reference path; the `hot` cases (scale 1.0: logits up to about +-150) leave it, the
    items are redone by the running-maximum recurrence, block after block with a finite running
    maximum, and the backward has to reproduce probabilities from LSE values of that size.
    Forward and backward compared in full.  Masked: a cut block, a padded tail and whole blocks in front."""
    B, n, g, w, r = 1, 1024, 2, 3, 3
    nb = n // 64
    t = inp.make_tensors(B, H, n, 64, 77, "bf16", with_dO=True)
    up = [1.0 + k / 4.0 for k in range(nb)]
    t = _scaled_key_blocks(t, up if case.startswith("growing") else up[::-1])
    scale = 1.0 if case.endswith("hot") else 0.125
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 5)
    km, mode, ref_kw = None, 0, {}
    if mask:
        km = np.ones((B, n), dtype=np.uint8)
        km[0, 128:256] = 0
        km[0, 900:] = 0
        mode = bb.BB_SKIP_PADDED_QUERY_BLOCKS if mask == "skip" else 0
        ref_kw = dict(key_mask=km, skip_padded_query_blocks=mask == "skip")
    dev, O, LSE = _fwd(t, ridx, g, w, scale, km, mode)
    Oref, Lref = oracle.attn_fwd(t["Q"], t["K"], t["V"], ridx, 64, g, w, scale, **ref_kw)
    eo, el = _fwd_errors(to_host(O), to_host(LSE), Oref, Lref)
    print(f"{case}: |LSE|max={np.abs(Lref).max():.1f} max|dO|={eo:.3e} max|dLSE|={el:.3e}")
    assert eo <= TOL and el <= TOL
    hQ, hK, hV = _bwd(dev, O, LSE, t, g, w, scale, mode)
    ref = oracle.attn_bwd(t["Q"], t["K"], t["V"], t["dO"], ridx, 64, g, w, scale, **ref_kw)
    errs = [np.abs(got - want).max() for got, want in zip((hQ, hK, hV), ref)]
    mags = [np.abs(want).max() for want in ref]
    print(f"{case}: max|ddQ|={errs[0]:.3e} max|ddK|={errs[1]:.3e} max|ddV|={errs[2]:.3e} "
          f"(|dQ|max={mags[0]:.2f} |dK|max={mags[1]:.2f} |dV|max={mags[2]:.2f})")
    assert all(np.isfinite(x).all() for x in (hQ, hK, hV))
    # gradients grow with the logits' scale: the absolute bar holds where they are of order one,
    # beyond that it is taken relative to the largest entry of each gradient
    for e, m in zip(errs, mags):
        assert e <= TOL * max(1.0, m), (case, errs, mags)
