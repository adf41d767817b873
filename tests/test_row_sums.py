"""GPU test: row sums of the bf16 forward on calls whose softmax is summed in fp32 before the
probabilities are rounded: rows that attend a block with padded keys inside, and all rows under dropout.

One key holds nearly all of every row, with a probability of another size in every row, so that the
rounding of that probability to bf16 (up to 2^-8 of it) shows in whatever is summed or divided after it.
The values are closed forms: q = (8 l, 0, ..), the key k* = (1, 0, ..), every other key 0, scale 1/8: the
logits of a row are l for k* and 0 for the other attended keys.
"""
import numpy as np
import pytest

import oracle
import paper_2007_14062_amd as bb
from gpu_util import to_host

pytestmark = pytest.mark.gpu

KEY = 17  # k*: in block 0, a global block of every pattern here


def dominated(B, H, n, lo, hi, seed):
    """Q, K, V (bf16, device) and the logits l [B, H, n] of k*; V rows of +-1."""
    import torch
    assert torch.cuda.is_available()
    rng = np.random.default_rng(seed)
    q0 = torch.from_numpy(rng.uniform(8 * lo, 8 * hi, (B, H, n)).astype(np.float32)).to(torch.bfloat16)
    Q = torch.zeros((B, H, n, 64), dtype=torch.bfloat16)
    Q[..., 0] = q0
    K = torch.zeros_like(Q)
    K[:, :, KEY, 0] = 1
    V = torch.from_numpy(rng.choice([-1.0, 1.0], (B, H, n, 64)).astype(np.float32)).to(torch.bfloat16)
    return tuple(x.to("cuda:0") for x in (Q, K, V)), q0.double().numpy() / 8


@pytest.mark.parametrize("B,H,n,w,r,skip,cut", [
    (1, 2, 1024, 3, 3, False, 980),    # a workgroup per row; the cut block and k* in different waves
    (2, 10, 1664, 3, 3, False, 20),    # items in the waves' streams, global rows in shares of 16 blocks
    (2, 10, 1664, 3, 3, True, 20),
    (1, 10, 2048, 15, 4, False, 20),   # non-global rows of more than 16 blocks
    (1, 2, 8192, 3, 3, False, 20),     # global rows of several workgroups
])
def test_lse_of_rows_with_a_cut_block(B, H, n, w, r, skip, cut):
    """20 keys from `cut` on are padded, in the first or in the last block: every row attends both.  (Where the
    waves' shares of a row, or its slices, are 16 blocks, those without a cut block are summed as without a mask:
    k* is in the share of the cut block there.)
    LSE = ln(e^l + m - 1), m the number of attended valid keys; fp32 sums leave an error of some 2^-22 of l
    and of the sum: 2e-5 here."""
    import torch
    (Q, K, V), l = dominated(B, H, n, 6.0, 9.0, 5)
    ridx = bb.bigbird_make_rand_idx(H, n, 64, 2, w, r, 4)
    km = torch.ones((B, n), dtype=torch.uint8, device="cuda:0")
    km[:, cut:cut + 20] = 0
    O, LSE = bb.bigbird_attn_fwd(Q, K, V, torch.from_numpy(ridx).to("cuda:0"), g=2, w=w, scale=0.125, key_padding_mask=km,
                                 global_mode=bb.BB_SKIP_PADDED_QUERY_BLOCKS if skip else 0)
    got = to_host(LSE)
    for h in range(H):
        A = oracle.dense_mask(ridx[h], n, 64, 2, w)
        m = A.sum(axis=1) - A[:, cut:cut + 20].sum(axis=1)
        err = np.abs(got[:, h] - np.log(np.exp(l[:, h]) + m - 1)).max()
        assert err <= 2e-5, (h, err)


@pytest.mark.parametrize("B,H,n,w,r", [
    (1, 2, 1024, 3, 3),    # a workgroup per row
    (2, 10, 1664, 3, 3),   # non-global rows by single waves
    (1, 10, 2048, 15, 4),  # cut rows: non-global rows of more than 16 blocks,
    (1, 2, 8192, 3, 3),    # global rows of more than 64,
    (2, 12, 4096, 3, 3),   # global rows of 64 at a size where they are cut finer
])
def test_dropout_output_of_dominated_rows(B, H, n, w, r):
    """Attention dropout at its smallest rate (2^-15): wherever k* is kept, O is V[k*] but for 1e-4 (the other
    keys: up to 8191 e^-18), so that its bf16 value is +-1 exactly; a numerator and a divisor that round the
    probability of k* differently would give 1 -+ 2^-8.  LSE in fp32 as without dropout."""
    import torch
    (Q, K, V), l = dominated(B, H, n, 18.0, 21.0, 6)
    ridx = bb.bigbird_make_rand_idx(H, n, 64, 2, w, r, 4)
    O, LSE = bb.bigbird_attn_fwd_dropout(Q, K, V, torch.from_numpy(ridx).to("cuda:0"), g=2, w=w, scale=0.125,
                                         p_drop=2.0 ** -15, seed=99)
    want = V[:, :, KEY:KEY + 1, :].float()
    wrong = (O.float() != want).any(dim=3).cpu().numpy()  # [B, H, n]
    for b, h, i in zip(*np.nonzero(wrong)):  # few: the rows that dropped k*
        keep, _ = bb.bigbird_dropout_keep_mask(2.0 ** -15, 99, b * H + h, n, int(i), 1)
        assert not keep[0, KEY], (b, h, i, O[b, h, i, :4])
    assert wrong.sum() <= 16 + wrong.size // 4096
    assert np.abs(to_host(LSE) - l).max() <= 2e-4
