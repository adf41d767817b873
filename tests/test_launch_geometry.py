"""How launches are cut up, on the CPU: the host rules of the kernel headers, compiled into a small program.

Every key block of a row is somebody's, lists fit where they are kept, partial results fit the workspace -- over all
forms the entry points take, small and large, with many or no global blocks."""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include "bwd_kernels.h"
#include "f32_rows.h"
#include "fwd_kernels.h"
#include <cstdio>
int main() {
  int BH, nb, g, w, r, masked, drop;
  while (scanf("%d %d %d %d %d %d %d", &BH, &nb, &g, &w, &r, &masked, &drop) == 7) {
    const bb::Bf16Geom q = bb::make_bf16_geom(BH, nb, g, w, r, masked != 0);
    const bb::RowSplit s = bb::make_row_split(BH, nb, g, w, r);
    printf("%d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d\n", q.waves, q.by_row, q.sw_len, q.gw_len, q.ng, q.cs, q.n_sitems, q.p_wgs,
           q.g_wgs, q.bh_rounds, bb::longest_sparse_list(nb, g, w, r), bb::kListedItems, s.slots_per_bh,
           bb::rows_f32_fwd(BH, nb, g, w, r, masked != 0, drop != 0), bb::rows_f32_bwd(BH, nb), bb::dkv_global_slice(BH, nb, g, w, r, masked != 0, drop != 0),
           bb::dq_global_slice(BH, nb, g, w, r, masked != 0), bb::make_key_split(nb, g, w, r, 0, 8).slots_per_bh, bb::bwd_by_row(BH, nb, g, w, r),
           bb::dkv_two_teams(BH, nb, bb::make_key_split(nb, g, w, r, 0, bb::dkv_global_slice(BH, nb, g, w, r, masked != 0, drop != 0))));
  }
}
"""
FIELDS = "waves by_row sw_len gw_len ng cs n_sitems p_wgs g_wgs bh_rounds sparse listed slots_per_bh rows_f32_fwd rows_f32_bwd dkv_slice dq_slice kv_slots_per_bh bwd_by_row two_teams".split()


@pytest.fixture(scope="module")
def geometry(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("geometry")
    src, exe = d / "geometry.hip", d / "geometry"
    src.write_text(PROGRAM)
    subprocess.run([hipcc, "--offload-host-only", "-std=c++17", "-O1", "-w", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2007_14062_amd", "csrc"), str(src), "-o", str(exe)], check=True)

    def ask(cases):
        """cases: (BH, nb, g, w, r[, masked[, drop]]) each; a dict of the fields for each."""
        text = "".join(" ".join(str(int(x)) for x in (tuple(c) + (0, 0))[:7]) + "\n" for c in cases)
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
        return [dict(zip(FIELDS, map(int, line.split()))) for line in out.splitlines()]

    return ask


def any_forms(count, seed):
    rng = random.Random(seed)
    out = []
    for _ in range(count):
        nb = max(1, round(2 ** rng.uniform(0, 9)))
        g = rng.choice((0, 1, 2, 2, 2, 4, 7, nb // 2, nb))
        w = rng.choice((1, 3, 3, 3, 7, 15, 33, 2 * nb + 1))
        out.append((max(1, round(2 ** rng.uniform(0, 9))), nb, min(g, nb), w, rng.choice((0, 2, 3, 3, 12)), rng.randrange(2), rng.randrange(2)))
    return out


def test_every_block_has_a_wave_and_every_list_a_place(geometry):
    cases = any_forms(4000, 1)
    for c, q in zip(cases, geometry(cases)):
        BH, nb, g = c[:3]
        assert q["waves"] in (4, 8) and 1 <= q["gw_len"] <= 16, (c, q)
        assert q["waves"] * q["gw_len"] * q["ng"] >= nb, (c, q)                  # global rows
        if q["by_row"]:
            assert q["waves"] == 4 and q["sw_len"] <= 16 and 4 * q["sw_len"] >= q["sparse"], (c, q)
            assert q["g_wgs"] == g * q["ng"] + nb - g and q["cs"] == 1, (c, q)
        else:
            assert 16 * q["cs"] >= q["sparse"] and q["g_wgs"] == g * q["ng"], (c, q)
            assert q["n_sitems"] == (nb - g) * q["cs"], (c, q)
            assert q["p_wgs"] * q["waves"] * q["listed"] >= q["bh_rounds"] * q["n_sitems"], (c, q)
        slots = (g * q["ng"] if q["ng"] > 1 else 0) + ((nb - g) * q["cs"] if q["cs"] > 1 else 0)
        assert slots <= q["slots_per_bh"], (c, q)
        # backward: slices of global blocks as long as the standard 8 or longer, a query block's in a list of 16
        assert q["dkv_slice"] >= 8 and 8 <= q["dq_slice"] <= 16, (c, q)
        cut = -(-nb // q["dkv_slice"])
        assert (g * cut if cut > 1 else 0) <= q["kv_slots_per_bh"], (c, q)


@pytest.mark.parametrize("BH,nb,waves", [
    (48, 15, 4), (56, 12, 4), (72, 8, 4),                # a workgroup of four waves to a compute unit
    (64, 12, 4), (72, 10, 4), (56, 15, 4), (64, 15, 4),  # global rows of fewer than 16 blocks
    (44, 16, 8), (48, 16, 8), (64, 16, 8), (36, 20, 8), (24, 64, 8), (12, 64, 8), (40, 33, 8),
    (36, 36, 8), (48, 28, 8),                            # 32 workgroups of eight waves to a die: every unit has one
    (64, 20, 4), (48, 33, 4), (48, 64, 4), (8, 64, 4),   # past that; too few
    (80, 9, 4), (32, 32, 8), (36, 36, 8),                # (with the ones above: what the GPU tests of medium launches run)
    (10, 80, 8), (9, 66, 4),                             # longer than 64 blocks: 51 and 44 workgroups of four waves
])
def test_workgroups_of_eight_waves(geometry, BH, nb, waves):
    """The count that decides is the one that is launched: the items of a die's slices together, not slice by slice."""
    (q,) = geometry([(BH, nb, 2, 3, 3)])
    assert q["waves"] == waves and not q["by_row"]
    if waves == 8:
        assert q["bh_rounds"] * q["g_wgs"] + q["p_wgs"] <= 32


@pytest.mark.parametrize("BH,nb,g,w,r,masked,waves", [
    (28, 16, 1, 3, 0, 0, 8), (28, 16, 1, 3, 0, 1, 8),    # lists of 4: also with a wave to a SIMD
    (28, 20, 1, 3, 3, 0, 8), (28, 20, 1, 3, 3, 1, 4),    # of 7: not under a mask
    (28, 20, 2, 3, 3, 0, 4), (28, 48, 1, 3, 0, 0, 8), (10, 36, 1, 3, 0, 0, 4),
    (36, 20, 2, 1, 8, 0, 4), (44, 20, 2, 1, 8, 0, 8),    # of 11
    (36, 24, 4, 9, 3, 0, 4), (20, 48, 4, 9, 3, 0, 8), (10, 48, 4, 9, 3, 0, 4),  # of 16
    (10, 80, 2, 3, 3, 1, 4), (10, 80, 1, 3, 0, 0, 4),    # longer than 64 blocks: under a mask, short lists
    (64, 24, 0, 3, 3, 0, 4),                             # no global rows
    (33, 20, 1, 17, 2, 0, 4), (20, 56, 4, 9, 5, 0, 4),   # two slices to a row
])
def test_workgroups_of_eight_waves_by_lists(geometry, BH, nb, g, w, r, masked, waves):
    (q,) = geometry([(BH, nb, g, w, r, masked)])
    assert q["waves"] == waves and not q["by_row"], q


@pytest.mark.parametrize("BH,nb,masked,ng,gw_len", [
    (1, 128, 0, 4, 8), (2, 128, 0, 4, 8), (1, 200, 0, 7, 8), (3, 80, 0, 3, 8), (2, 65, 1, 3, 8),  # longer than 64 blocks
    (4, 64, 0, 2, 8), (4, 50, 0, 2, 8), (4, 45, 0, 2, 8), (4, 50, 1, 2, 8), (8, 33, 1, 2, 8),
    (4, 44, 0, 1, 11), (8, 35, 0, 1, 9), (8, 33, 0, 1, 9),                                        # dealt out in quarters
    (12, 16, 0, 1, 4), (12, 16, 1, 1, 4), (4, 32, 1, 1, 8),
])
def test_global_rows_of_launches_by_rows(geometry, BH, nb, masked, ng, gw_len):
    (q,) = geometry([(BH, nb, 2, 3, 3, masked)])
    assert q["by_row"] and (q["ng"], q["gw_len"]) == (ng, gw_len), q


@pytest.mark.parametrize("BH,nb,masked,wide,by_row", [
    (5, 56, 0, 0, 0), (8, 35, 1, 0, 0), (7, 40, 1, 0, 0), (12, 24, 0, 0, 1),
    (6, 48, 0, 1, 1), (6, 48, 1, 1, 1), (6, 49, 0, 1, 0), (4, 56, 0, 1, 1),  # lists of a whole slice
])
def test_launches_just_past_those_by_rows(geometry, BH, nb, masked, wide, by_row):
    (q,) = geometry([(BH, nb, 4, 9, 3, masked) if wide else (BH, nb, 2, 3, 3, masked)])
    assert q["by_row"] == by_row and q["waves"] == 4, q
    if by_row and wide:
        assert (q["ng"], q["gw_len"]) == ((1, 12) if BH == 6 else (2, 8)), q


@pytest.mark.parametrize("BH,nb,fwd,bwd", [
    (1, 1, 1, 1), (32, 1, 1, 1), (33, 1, 0, 0), (2, 2, 1, 1), (4, 8, 1, 1), (5, 8, 1, 0), (12, 8, 1, 0), (13, 8, 0, 0), (10, 6, 1, 0), (11, 6, 0, 0),
    (3, 9, 1, 1), (1, 12, 1, 1), (1, 13, 0, 0), (2, 16, 1, 1), (3, 11, 0, 0), (1, 17, 0, 0),
])
def test_fp32_launches_by_eight_positions(geometry, BH, nb, fwd, bwd):
    (q,) = geometry([(BH, nb, min(2, nb), 3, 0)])
    assert (q["rows_f32_fwd"], q["rows_f32_bwd"]) == (fwd, bwd)


@pytest.mark.parametrize("BH,nb,g,r,masked,drop,fwd", [
    (12, 8, 0, 2, 0, 0, 0), (12, 8, 1, 2, 0, 0, 1), (8, 8, 0, 3, 0, 0, 1), (10, 8, 0, 3, 0, 0, 0), (5, 8, 0, 2, 0, 0, 0),  # of 5, 6, 8
    (12, 8, 1, 2, 1, 0, 0), (9, 8, 1, 2, 1, 0, 0), (8, 8, 1, 2, 1, 1, 1),                # under a mask
    (1, 1, 1, 0, 0, 1, 0), (32, 1, 0, 0, 1, 1, 0), (32, 1, 0, 0, 1, 0, 1), (2, 2, 1, 0, 0, 1, 1),   # a single block under dropout
    (2, 10, 1, 3, 0, 0, 1), (2, 10, 1, 3, 0, 1, 0), (2, 10, 1, 3, 1, 1, 1), (3, 10, 2, 3, 0, 1, 0), (2, 16, 2, 3, 0, 1, 1),
    (3, 9, 2, 3, 0, 1, 1), (1, 12, 0, 3, 0, 1, 1),                   # no list is that long without global blocks
])
def test_fp32_forward_launches_by_their_lists(geometry, BH, nb, g, r, masked, drop, fwd):
    (q,) = geometry([(BH, nb, g, 3, r, masked, drop)])
    assert q["rows_f32_fwd"] == fwd, q


@pytest.mark.parametrize("BH,nb,masked,drop,dkv", [
    (24, 101, 0, 1, 12), (24, 90, 0, 1, 12), (24, 128, 0, 1, 12), (40, 72, 0, 1, 12),  # under dropout, a smaller last group
    (48, 64, 0, 1, 24), (48, 48, 0, 1, 24), (24, 64, 0, 1, 24), (16, 256, 0, 1, 32),   # equal groups, or one
    (24, 101, 0, 0, 24), (24, 101, 1, 1, 16), (24, 101, 1, 0, 16), (20, 128, 0, 1, 12), (20, 128, 0, 0, 12), (24, 48, 0, 0, 8),
])
def test_slices_of_global_key_blocks(geometry, BH, nb, masked, drop, dkv):
    (q,) = geometry([(BH, nb, 2, 3, 3, masked, drop)])
    assert q["dkv_slice"] == dkv


@pytest.mark.parametrize("BH,nb,g,two", [
    (384, 1, 0, 0), (512, 1, 1, 0),                                  # lists of one
    (96, 3, 1, 0), (72, 4, 2, 0), (48, 6, 2, 0), (97, 3, 1, 1), (64, 6, 2, 1), (160, 2, 1, 1),   # short lists: 288 items, more
    (48, 8, 2, 1), (32, 9, 0, 1), (32, 10, 2, 1), (24, 16, 2, 1), (32, 16, 0, 1), (33, 16, 0, 0),
])
def test_pairs_of_waves_per_key_block(geometry, BH, nb, g, two):
    (q,) = geometry([(BH, nb, g, 3, 3)])
    assert q["two_teams"] == two and not q["bwd_by_row"], q


@pytest.mark.parametrize("BH,nb,masked,items", [
    (300, 12, 1, 2.5),       # the GPU tests of streams with several items to a wave
    (520, 256, 1, 62),       # and of lists that are full
])
def test_items_of_a_wave(geometry, BH, nb, masked, items):
    g = 2 if nb == 12 else 1
    (q,) = geometry([(BH, nb, g, 3 if nb == 12 else 1, 3 if nb == 12 else 0, masked)])
    assert not q["by_row"] and q["cs"] == 1 and q["waves"] == 4
    resident = min(q["p_wgs"], 64) * q["waves"]
    assert q["bh_rounds"] * q["n_sitems"] / resident > items, q
