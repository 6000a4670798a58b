"""How the workgroups of a head-wise call are dealt to its groups of heads (csrc/work_share.h), and into how many parts the band units
of the backward are split, and which calls run dQ and dK/dV in one launch (csrc/bwd_common.h, csrc/attn_fp32.h), in a host build, no GPU."""
import shutil
import subprocess

import pytest

from paper_2412_12094_amd import build
from test_gpu_attn_shapes import JOINT_CASES, JOINT_ROWS
from test_gpu_fp32_backward import CASES as FP32_CASES

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "work_share.h"
using namespace sepattn;
// L d gp TP slots windows...: the split's threshold, then per group its window, workgroups and pieces of work
int main(int argc, char **argv) {
    auto arg = [&](int i) { return atoi(argv[i]); };
    sepattn_params p = {};
    p.B = 1, p.L = arg(1), p.d = arg(2);
    const int gp = arg(3), TP = arg(4), slots = arg(5);
    p.Hq = p.Hkv = argc - 6;
    for (int h = 0; h < p.Hq; ++h) p.n = arg(6 + h) > p.n ? arg(6 + h) : p.n;
    HeadWin hw = {};
    for (int h = 0; h < p.Hq; ++h) hw.delta[h] = p.n - arg(6 + h);
    const int keys = split_keys(p, hw, gp, TP, slots, (size_t)1 << 40), tiles = (p.L + TP - 1) / TP;
    printf("%d\n", keys);
    const WorkShare w = share_queries(p, hw, gp, TP, slots, keys);
    for (int i = 0; i < w.n; ++i) {
        const int n = p.n - group_delta(hw, w.group[i] * gp, gp);
        printf("%d %d %d\n", n, w.first[i + 1] - w.first[i], tiles + split_tiles(tiles, TP, n, keys).n);
    }
}
"""


PARTS_PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "bwd_common.h"
using namespace sepattn;
int sepattn::compute_units() { return 256; }
// B Hq Hkv L d a n: parts of a band unit, workgroups per (batch, KV head), parts that the workspace has room for
int main(int, char **argv) {
    auto arg = [&](int i) { return atoi(argv[i]); };
    sepattn_params p = {};
    p.B = arg(1), p.Hq = arg(2), p.Hkv = arg(3), p.L = arg(4), p.d = arg(5), p.a = arg(6), p.n = arg(7);
    const int wpg = dkv_workgroups_per_head(p, 2);
    printf("%d %d %d\n", band_split(p, wpg, 2), wpg, band_split(p, wpg, 2, true));
}
"""


JOINT_PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "attn_fp32.h"
#include "bwd_common.h"
using namespace sepattn;
int sepattn::compute_units() { return 256; }
// fp32 docs B Hq Hkv L d a n: fp32, bytes from word to word of the one launch (0: two), of all words, of the place they take.  bf16, dQ
// workgroups per group of the one launch (0: two), workgroups per (batch, KV head) and bytes of the partials that dK/dV has there, and at most
int main(int, char **argv) {
    auto arg = [&](int i) { return atoi(argv[i]); };
    sepattn_params p = {};
    const bool docs = arg(2);
    p.B = arg(3), p.Hq = arg(4), p.Hkv = arg(5), p.L = arg(6), p.d = arg(7), p.a = arg(8), p.n = arg(9), p.cap = p.L;
    if (arg(1)) {
        const Fp32Workspace w = fp32_workspace(p);
        printf("%d %ld %ld\n", fp32_one_launch(p, w), w.n_counters * fp32_one_launch(p, w), (long)w.d_bytes);
        return 0;
    }
    const int dq = joint_dq_workgroups(p, HeadWin{}, docs), wpg = dq ? joint_dkv_workgroups(p, dq) : 0;
    const long rows = dq ? far_geom(p, wpg, 2, band_split(p, wpg, 2)).rows : 0;
    printf("%d %d %d %ld %ld\n", dq, wpg, dkv_workgroups_per_head(p, 2), rows * p.B * p.Hkv * p.d * 4, (long)bwd_workspace(p).far_bytes);
}
"""


def host_program(d, source):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    (d / "share.hip").write_text(source)
    cmd = ["hipcc", *build.FLAGS, "--offload-host-only", "-c", str(d / "share.hip"), "-o", str(d / "share.o")]
    subprocess.run(cmd, check=True, capture_output=True)
    subprocess.run(["g++", str(d / "share.o"), "-o", str(d / "share")], check=True)
    return lambda *args: [list(map(int, line.split())) for line in
                          subprocess.run([str(d / "share"), *map(str, args)], check=True, capture_output=True, text=True).stdout.splitlines()]


@pytest.fixture(scope="module")
def dealt(tmp_path_factory):
    return host_program(tmp_path_factory.mktemp("work_share"), PROGRAM)


@pytest.fixture(scope="module")
def parts(tmp_path_factory):
    return host_program(tmp_path_factory.mktemp("band_parts"), PARTS_PROGRAM)


@pytest.fixture(scope="module")
def joint(tmp_path_factory):
    return host_program(tmp_path_factory.mktemp("one_launch"), JOINT_PROGRAM)


@pytest.mark.parametrize("L,d,gp,TP,slots,windows,is_split", [
    (2600, 128, 4, 32, 512, [2600] * 4 + [40, 7, 1, 64], True),      # more workgroups than pieces
    (2600, 128, 4, 32, 100, [2600] * 4 + [40, 7, 1, 64], True),      # fewer
    (2600, 64, 1, 128, 512, [2600] * 4 + [2000, 7, 1, 64], True),
    (4096, 128, 4, 32, 512, ([4096] * 4 + [128] * 12) * 2, True),
    (1300, 128, 4, 32, 512, [600] * 4 + [40, 7, 1, 64], False),
    (66, 64, 1, 128, 16, [66, 5, 20, 1] * 8, False),                 # more groups than slots
])
def test_no_group_gets_more_workgroups_than_it_has_pieces(dealt, L, d, gp, TP, slots, windows, is_split):
    (keys,), *groups = dealt(L, d, gp, TP, slots, *windows)
    tiles = -(-L // TP)
    assert (keys > 0) == is_split and len(groups) == len(windows) // gp
    for window, count, pieces in groups:
        assert pieces == tiles if not is_split or window < keys else tiles < pieces <= 2 * tiles
        assert 1 <= count <= pieces
    total = sum(count for _, count, _ in groups)
    assert total <= max(slots, len(groups))
    # what one group cannot use goes to the others
    if slots >= sum(pieces for _, _, pieces in groups):
        assert all(count == pieces for _, count, pieces in groups)


@pytest.mark.parametrize("B,Hq,Hkv,L,d,a,n,want", [
    (1, 8, 2, 600, 128, 4, 96, 4),     # few units, nothing beside them: as many parts as there are heads
    (1, 8, 1, 527, 64, 8, 32, 4),      # a part has four steps at least
    (1, 28, 4, 600, 128, 4, 96, 7),
    (1, 8, 1, 3803, 64, 0, 32, 1),     # far work, whose slices get as short as the parts: four parts took 1.44 times as long
    (2, 8, 1, 2820, 64, 8, 58, 2),     # 1.05 times
    (1, 8, 1, 2921, 128, 3, 19, 2),    # 1.25 times
    (1, 32, 8, 869, 128, 3, 86, 1),    # more parts than compute units: four took 1.25 times as long
    (1, 8, 2, 600, 128, 4, 600, 4),    # the whole sequence in the window: no far work
    (21, 4, 1, 384, 128, 4, 360, 4),   # as many parts as workgroups
    (21, 4, 1, 385, 128, 4, 360, 2),   # one key more
    (1, 8, 8, 600, 128, 4, 96, 1),     # one head per KV head
])
def test_band_units_are_split_where_the_parts_have_room(parts, B, Hq, Hkv, L, d, a, n, want):
    ((split, wpg, room),) = parts(B, Hq, Hkv, L, d, a, n)
    assert split == want and split <= room
    assert split == 1 or -(-L // 64) * split <= wpg


@pytest.mark.parametrize("case", JOINT_CASES, ids=str)
def test_small_backward_in_one_launch(joint, case):
    """The calls of the GPU test of the same line: 192 query tiles (of 512 workgroups) are the most, and dK/dV has no more workgroups and
    partials there than the workspace is laid out for."""
    B, Hq, Hkv, L, d, a, n, p, docs, one = case
    ((dq, wpg, most, rows, room),) = joint(0, int(docs), B, Hq, Hkv, L, d, 0 if docs else a, n)
    gp = next(g for g in (4, 2, 1) if Hq // Hkv % g == 0)
    tiles = -(-L * gp // 128)
    assert (dq > 0) == one == (B * Hq // gp * tiles <= 192)
    assert not one or (dq == tiles and 1 <= wpg <= most and B * Hkv * wpg + B * Hq // gp * dq <= 512 and 0 < rows <= room)


@pytest.mark.parametrize("Hq,Hkv,L,d,a,n", JOINT_ROWS)
def test_small_backward_of_a_row_and_of_four(joint, Hq, Hkv, L, d, a, n):
    assert joint(0, 0, 1, Hq, Hkv, L, d, a, n)[0][0] > 0 and joint(0, 0, 4, Hq, Hkv, L, d, a, n)[0][0] == 0


@pytest.mark.parametrize("B,Hq,Hkv,L,d,n,docs,one", [
    (1, 8, 8, 24, 64, 8, False, True),      # fewer tiles than workgroups per KV head
    (191, 1, 1, 40, 64, 8, False, True),    # more KV heads than it has workgroups left over for two each
    (1, 7, 1, 500, 128, 64, False, False),  # seven waves
    (1, 4, 1, 3000, 128, 3000, False, False),  # split streams
    (1, 4, 1, 1100, 128, 1100, False, False),  # the list of all keys
    (1, 4, 1, 1100, 128, 1100, True, True),    # which packed rows do not have
])
def test_small_backward_other_rules(joint, B, Hq, Hkv, L, d, n, docs, one):
    ((dq, wpg, most, rows, room),) = joint(0, int(docs), B, Hq, Hkv, L, d, 0 if docs else 4, n)
    assert (dq > 0) == one
    assert not one or (1 <= wpg <= most and 0 < rows <= room)


@pytest.mark.parametrize("case", FP32_CASES, ids=str)
def test_fp32_backward_in_one_launch(joint, case):
    """The calls of the GPU test that compares one launch with two: on which side of the line each is, and that the words have room."""
    B, Hq, Hkv, L, d, a, n, p, one = case
    ((stride, words, room),) = joint(1, 0, B, Hq, Hkv, L, d, a, n)
    assert (stride > 0) == one and words <= room
    assert not one or stride == (128 if words // stride * 128 <= room else 8)
