"""GPU parity of the fp32 kernels of small launches (a workgroup per eight positions), forward and backward, at the
edges of their range: one block up to the last launch that takes them and the first ones past it, lists of one and of two
entries a wave, padded keys inside blocks, skipped query blocks, attention
dropout.  Tolerance 1e-4 (fp32 sums of up to 64 * 16 terms of order one: 2^-24 * 1024 = 6e-5)."""
import numpy as np
import pytest

import bigbird_inputs as inp
import paper_2007_14062_amd as bb
import test_dropout_parity
import test_skip_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,nb,g,w,r", [
    (1, 1, 1, 0, 1, 0),     # one block, a list of one
    (1, 3, 2, 1, 1, 0),
    (1, 4, 8, 2, 3, 3),     # 32 blocks: the last launch of both passes
    (1, 5, 8, 2, 3, 3),     # past it: forward alone
    (1, 12, 8, 2, 3, 2),    # last forward
    (1, 13, 8, 1, 3, 2),    # past it
    (1, 8, 8, 0, 3, 3),     # lists of 6, no global block: last forward
    (1, 12, 8, 0, 3, 2),    # of 5: past it
    (2, 1, 10, 1, 3, 3),    # 20 blocks, lists of 10: past it under dropout
    (1, 10, 6, 1, 3, 1),    # 60 blocks of 6: forward alone
    (1, 3, 9, 2, 3, 3),     # two entries for wave 0 of a global block
    (2, 1, 12, 0, 5, 4),    # no global block
    (1, 1, 12, 2, 3, 3),
    (1, 1, 13, 2, 3, 3),    # one slice of more than 12 blocks: slices of the list
    (1, 2, 16, 2, 3, 3),    # two entries for every wave of a global block
    (1, 2, 16, 2, 9, 5),    # lists of all 16
    (2, 1, 16, 4, 13, 0),   # of all 16, no random blocks
    (1, 3, 11, 2, 3, 3),    # 33 blocks
])
@pytest.mark.parametrize("case", ["plain", "padded", "skip", "drop", "drop padded"])
def test_parity(B, H, nb, g, w, r, case):
    n = nb * 64
    rng = np.random.default_rng(nb * 100 + H)
    t = inp.make_tensors(B, H, n, 64, 700 + nb, "f32", with_dO=True)
    ridx = bb.bigbird_make_rand_idx(H, n, 64, g, w, r, 5)
    tag = f"fp32 rows B{B} H{H} nb{nb} {case}"
    if case in ("plain", "drop"):
        test_dropout_parity.check(t, ridx, 64, g, w, 0.125, 0.0 if case == "plain" else 0.25, 11, "f32", tag=tag)
        return
    km = np.ones((B, n), dtype=np.uint8)
    km[0, n - n // 3 - 5:] = 0                      # ends inside a block; whole blocks after it
    km[B - 1, 7:7 + int(rng.integers(1, 50))] = 0   # a hole in the first block
    if case == "drop padded":
        test_dropout_parity.check(t, ridx, 64, g, w, 0.125, 0.25, 11, "f32", key_mask=km, tag=tag)
    elif case == "skip":
        test_skip_parity.check(t, ridx, 64, g, w, 0.125, "f32", km, tag=tag)
    else:
        test_dropout_parity.check(t, ridx, 64, g, w, 0.125, 0.0, 11, "f32", key_mask=km, tag=tag)
