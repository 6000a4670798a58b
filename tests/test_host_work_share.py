"""How the workgroups of a head-wise call are dealt to its groups of heads (csrc/work_share.h), in a host build, no GPU."""
import shutil
import subprocess

import pytest

from paper_2412_12094_amd import build

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


@pytest.fixture(scope="module")
def dealt(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("work_share")
    (d / "share.hip").write_text(PROGRAM)
    cmd = ["hipcc", *build.FLAGS, "--offload-host-only", "-c", str(d / "share.hip"), "-o", str(d / "share.o")]
    subprocess.run(cmd, check=True, capture_output=True)
    subprocess.run(["g++", str(d / "share.o"), "-o", str(d / "share")], check=True)
    return lambda *args: [list(map(int, line.split())) for line in
                          subprocess.run([str(d / "share"), *map(str, args)], check=True, capture_output=True, text=True).stdout.splitlines()]


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
