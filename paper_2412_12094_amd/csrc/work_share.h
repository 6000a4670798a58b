// How the workgroups of a head-wise call are dealt out to its groups of heads (the heads that share K/V tiles).
//
// A group runs with the largest window among ITS heads, so the groups' work differs by up to L / n: with heads that
// see everything next to heads with a window of 128, an even deal leaves all but the longest groups' workgroups
// idle, and running every group with the call's largest window made each as long as the longest (32/8 heads,
// d = 128, L = 4096, every fourth KV head full, the others 128: forward 180 -> 102 us, dQ 228 -> 170, dK/dV 581 -> 170,
// what is left in the first two being the last query tile, whose stream no deal shortens).  Workgroups are dealt so that
// the largest work of any one of them is least (share_out), the longest groups first in dispatch order, so that two
// of them share a compute unit only when there are more long workgroups than compute units.
#pragma once

#include "common.h"

namespace sepattn {

// groups of one batch row in order of falling work: `group[i]` owns the workgroups first[i] .. first[i+1]-1 of the row
struct WorkShare {
    int32_t n;  // number of groups; 0: an ordinary call, every group gets the same number
    int32_t first[kMaxHeadwise + 1];
    int32_t group[kMaxHeadwise];
    int32_t all[kMaxHeadwise];  // every head of the group sees every earlier key
};

struct ShareOf {
    int b, pos, rank, count;  // batch row, index into the tables, workgroup's number within its group and their number
};
__device__ inline ShareOf share_of(const WorkShare &w, int id, int B) {
    ShareOf s;
    s.b = id % B;
    const int r = id / B;
    int lo = 0, hi = w.n;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (w.first[mid] <= r) lo = mid;
        else hi = mid;
    }
    s.pos = lo;
    s.rank = r - w.first[lo];
    s.count = w.first[lo + 1] - w.first[lo];
    return s;
}

// how much shorter than p.n the largest window of the heads h0 .. h0 + n - 1 is
__host__ __device__ inline int group_delta(const HeadWin &hw, int h0, int n) {
    int d = head_delta(hw, h0);
    for (int i = 1; i < n; ++i) d = head_delta(hw, h0 + i) < d ? head_delta(hw, h0 + i) : d;
    return d;
}

// What a forward or dQ kernel is given about head-wise windows.  An ordinary call has nothing of it: reading the tables (a round
// trip to the arguments, behind that for the group's number) would stand at the start of every workgroup.
template <bool HW>
struct HeadArgs {
    HeadWin hw;
    WorkShare share;
    __device__ int of_group(int h0, int n) const { return group_delta(hw, h0, n); }
    __device__ int of_head(int h) const { return head_delta(hw, h); }
};
template <>
struct HeadArgs<false> {
    __device__ static int of_group(int, int) { return 0; }
    __device__ static int of_head(int) { return 0; }
};

inline bool any_delta(const HeadWin &hw) {
    for (int h = 0; h < kMaxHeadwise; ++h)
        if (hw.delta[h]) return true;
    return false;
}

// share of the keys that are separators, for the estimate of a group's work only (the count is on the device): text
// holds about one in ten
constexpr double kSepShare = 0.1;

// Deals at most `slots` workgroups of a batch row to the groups of `heads` query heads each, between 1 and cap(window) per
// group, so that the largest cost(window, all) per workgroup is as small as it can be (bisection over that value; dealing by
// rounded shares left groups with one workgroup where two per group were to be had: 219 -> 274 us at 8 x 32
// heads, L = 512).  More groups than slots get one each, the longest ones dispatched first.
template <typename Cap, typename Cost>
inline WorkShare share_out(const sepattn_params &p, const HeadWin &hw, int heads, int slots, Cap cap, Cost cost) {
    WorkShare w;
    w.n = p.Hq / heads;
    int limit[kMaxHeadwise];
    double c[kMaxHeadwise], sum = 0.;
    for (int g = 0; g < w.n; ++g) {
        const int dmin = group_delta(hw, g * heads, heads);
        bool all = p.n - dmin >= p.L;
        for (int i = 0; i < heads; ++i) all = all && head_delta(hw, g * heads + i) == dmin;
        const double x = cost(p.n - dmin, all);
        sum += x;
        int i = g;
        for (; i > 0 && c[i - 1] < x; --i) {
            c[i] = c[i - 1];
            limit[i] = limit[i - 1];
            w.group[i] = w.group[i - 1];
            w.all[i] = w.all[i - 1];
        }
        c[i] = x;
        limit[i] = cap(p.n - dmin);
        w.group[i] = g;
        w.all[i] = all;
    }
    auto wanted = [&](int i, double most) {
        const double k = c[i] / most + 0.999;
        return k >= limit[i] ? limit[i] : (k < 1. ? 1 : (int)k);
    };
    double lo = sum / (slots > 0 ? slots : 1) / 2, hi = c[0];  // hi: one workgroup each
    for (int it = 0; it < 12; ++it) {
        const double mid = (lo + hi) / 2;
        long total = 0;
        for (int i = 0; i < w.n; ++i) total += wanted(i, mid);
        if (total <= slots) hi = mid;
        else lo = mid;
    }
    w.first[0] = 0;
    for (int i = 0; i < w.n; ++i) w.first[i + 1] = w.first[i] + wanted(i, hi);
    return w;
}

// keys streamed by the query tiles of TP positions of a forward or dQ group, and what its segments' starts cost
inline double query_cost(const sepattn_params &p, int TP, int n) {
    const double L = p.L, w = n < p.L ? n : p.L, out = L - w;
    return w * (L - w / 2) + L * (TP + 128) + kSepShare * out * out / 2;
}

// Query tiles whose key streams go in two halves to two workgroups.  A tile's stream is a serial chain of one workgroup,
// and where windows are long and tiles few it is what the kernel waits for.  Of the tiles, longest first, the first `n`
// are split: those whose first row has at least `keys` keys in its window (0: none).
struct SplitTiles {
    int n, most, tiles;  // split tiles of the group; of any group; all tiles
    // rank in the order of falling work -> tile and part (-1: whole).  Lengths fall linearly from the longest to its half over
    // the split tiles and from there to nothing, so four halves (two tiles) go with one whole tile.
    __host__ __device__ void find(int rank, int &tile, int &part) const {
        const int fives = n / 2 < tiles - n ? n / 2 : tiles - n;
        int half = -1;
        tile = rank - n;
        if (rank < 5 * fives) {
            if (rank % 5) half = rank / 5 * 4 + rank % 5 - 1;
            else tile = n + rank / 5;
        } else if (rank < 2 * n + fives) {
            half = rank - fives;
        }
        part = half < 0 ? -1 : half & 1;
        if (half >= 0) tile = half >> 1;
    }
};
__host__ __device__ inline SplitTiles split_tiles(int tiles, int TP, int window, int keys) {
    SplitTiles s;
    s.tiles = tiles;
    s.most = keys && tiles > keys / TP ? tiles - keys / TP : 0;
    s.n = keys && window >= keys ? s.most : 0;
    return s;
}

// From which window length on tiles are split, 0: none are.  Half of the longest (p.n is that of the call), if that shortens the
// longest chain by kWorthSplitting keys, given the workgroups' mean work, and there is `room` for the parts of so many
// tiles.  A split costs the second part's start, fp32 sums and a launch that adds them (6 us for 128 tiles at
// d = 128).  Over 270 calls with full windows of 1300 to 2500 positions the step is, by what a split saves, 1.00 times as fast at 800 to
// 1200 keys (0.96 to 1.06), 1.04 at 1200 to 1600 (0.97 to 1.10), 1.07 above (1.01 to 1.12).  Forward and backward in us, whole / split
// streams.  Above the line: every fourth KV head full, the others 128 (32/8 heads, d = 128, L = 4096) 363 / 352, the same with 8/8 heads
// 245 / 213; 8/1 heads, L = 3000, n = L 193 / 179; 12/12 heads, d = 64, L = n = 2048 123 / 116, 1300 91 / 88; 8/2 heads, L = 4096, n = L 273 / 254.
// Below it: 32/8 heads, L = n = 2048 225 / 228; 12/12 heads, d = 64, 4 x L = 2048 194 / 207.  Windows that end before the sequence and
// are shorter than twice the line stay whole: from there on all tiles are equally long, and it is half of them or more that
// are split (8/2 heads, L = 4096, n = 2048, 1330 keys saved, 201 / 208; 6/3 heads, 1570 keys, 222 / 221).
constexpr int kWorthSplitting = 1280;
inline int split_keys(const sepattn_params &p, const HeadWin &hw, int gp, int TP, long slots, size_t room) {
    const int longest = p.n < p.L ? p.n : p.L, start = TP + 128;
    if (p.n < p.L && longest < 2 * kWorthSplitting) return 0;
    double sum = 0.;
    for (int h = 0; h < p.Hq; h += gp) sum += query_cost(p, TP, p.n - group_delta(hw, h, gp)) / TP * p.B;
    const int keys = (longest / 2 + TP - 1) / TP * TP;
    if (longest + start - sum / slots < kWorthSplitting) return 0;
    const SplitTiles s = split_tiles((p.L + TP - 1) / TP, TP, p.n, keys);
    return (size_t)p.B * (p.Hq / gp) * s.most <= room ? keys : 0;
}

// pieces of work of a forward or dQ group whose largest window is `n`: its query tiles, split ones twice
inline int query_pieces(const sepattn_params &p, int TP, int n, int part_keys) {
    const int tiles = (p.L + TP - 1) / TP;
    return tiles + split_tiles(tiles, TP, n, part_keys).n;
}
// the workgroups of a head-wise forward or dQ: no group gets more than it has pieces
inline WorkShare share_queries(const sepattn_params &p, const HeadWin &hw, int gp, int TP, int slots, int part_keys) {
    return share_out(p, hw, gp, slots, [&](int n) { return query_pieces(p, TP, n, part_keys); }, [&](int n, bool) { return query_cost(p, TP, n); });
}

}  // namespace sepattn
