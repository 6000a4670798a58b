// The dense key stream of one query tile (used by the forward and the dQ kernels).
//
// For query positions [i0, i0+TP) the visible keys are enumerated as one stream
//     [ initial tokens j < min(a, bs) | separators in [min(a,bs), bs) | band keys bs .. i0+TP-1 ]
// with bs = max(0, i0-n+1), the first key of the first row's neighbour window (Sec. 3.1).  Elements
// of the first two parts are visible to every row of the tile; a band key j is visible to query i
// iff  j <= i  and  (i-j < n  or  j is an initial token or a separator)  (Eq. 2).  Each stream
// element carries the inclusive query range [lo, hi] that sees it, so the test is lo <= i <= hi.
#pragma once

#include "common.h"
#include "mfma_common.h"

namespace sepattn {

constexpr int kBN = 64;  // keys per LDS tile

// The workgroups of a forward or dQ launch.  A group is one (batch, KV head, packed query heads) and owns its own K/V rows; `wpg`
// workgroups share its query tiles.
// Consecutive workgroup ids (x first) are dealt round-robin to the 8 XCDs, each with a private L2.  When the
// number of groups is a multiple of 8, the grid is 8 x wpg x groups/8, so that XCD x only ever sees groups congruent to
// x and the K/V rows of a group stay in one L2 instead of being streamed through all eight.  Otherwise groups x wpg.
struct QueryGrid {
    int gx;      // groups side by side in the grid
    int groups;  // head groups per KV head
    FastDiv by_groups, by_hkv;
};
struct GroupOf {
    int hg, kv, b;  // head group, KV head, batch row
};
__device__ inline GroupOf group_of(const QueryGrid &g, int group, int Hkv) {
    GroupOf r;
    const int bkv = quotient(group, g.by_groups);
    r.hg = group - bkv * g.groups;
    r.b = quotient(bkv, g.by_hkv);
    r.kv = bkv - r.b * Hkv;
    return r;
}
inline QueryGrid query_grid(const sepattn_params &p, int gp, long n_groups) {
    QueryGrid g;
    g.groups = p.Hq / p.Hkv / gp;
    g.gx = n_groups % 8 == 0 && n_groups / 8 <= 65535 ? 8 : (int)n_groups;
    g.by_groups = fast_div((uint32_t)g.groups);
    g.by_hkv = fast_div((uint32_t)p.Hkv);
    return g;
}

// Shape of a forward / dQ workgroup: nw waves of 32 query rows each, gp query heads of one KV head packed into
// the rows, i.e. 32 nw / gp positions.  Fewer positions mean fewer keys that only some rows see (a tile
// streams the window of its first row AND its own length), more heads mean fewer tiles.
//   Four waves, so that two (d = 64: three) independent workgroups share a compute unit: one's segment change, row
//     stores and barriers overlap the others' matrix work, and the split of a group is finer.
//   Seven heads per KV head: seven waves, one head each (one head per workgroup streamed 456 band keys for a
//     window of 200; seven stream 232: B=3, L=3077, d=128 forward 113 -> 72 us).  Three, five and six heads per KV
//     head run with one or two per tile; shapes with all of them in one tile have not been built or measured.
//   Eight waves at d = 128 with four heads where the work is large (eight rounds of four-wave workgroups per compute
//     unit and more): half the tile loads per matrix instruction (L = 64K: 3.67 ms against 4.0; level at L = 4096).
struct QueryShape {
    int gp, nw;
};
inline QueryShape query_shape(const sepattn_params &p) {
    const int G = p.Hq / p.Hkv;
    if (G % 7 == 0) return {7, 7};
    const int gp = G % 4 == 0 ? 4 : (G % 2 == 0 ? 2 : 1);
    const long tiles = (long)p.B * p.Hkv * (G / gp) * (((long)p.L * gp + 127) / 128);  // of four waves
    return {gp, p.d == 128 && gp == 4 && tiles >= 8l * compute_units() ? 8 : 4};
}

struct Stream {
    int n_init, n_dense, n_total, sep_lo, bs;
};

__device__ inline Stream make_stream(const sepattn_params &p, const int32_t *__restrict__ prefix, int i0,
                                     int tile_positions) {
    Stream st;
    st.bs = max(0, i0 - p.n + 1);
    st.n_init = min(p.a, st.bs);
    st.sep_lo = load_uniform(prefix, st.n_init);
    st.n_dense = st.n_init + (load_uniform(prefix, st.bs) - st.sep_lo);
    st.n_total = st.n_dense + (min(p.L, i0 + tile_positions) - st.bs);
    return st;
}

// Packed documents: the row holds several documents and a query sees nothing outside its own.  The
// first tokens of every document are marked like separators beforehand (the kernels then run with
// a = 0), so the keys of the first row's document that are older than its window are still one
// contiguous range of the compacted list, now starting at that document's first position `ds`; the
// band starts no earlier than `ds`.  Rows of later documents in the same tile find all their keys in
// the band part; who sees what is decided by the per-key range [lo, hi] with hi cut at the end of
// the key's document.
__device__ inline Stream make_stream_docs(const sepattn_params &p, const int32_t *__restrict__ prefix, int i0,
                                          int tile_positions, int ds) {
    Stream st;
    st.bs = max(ds, i0 - p.n + 1);
    st.n_init = 0;
    st.sep_lo = load_uniform(prefix, ds);
    st.n_dense = load_uniform(prefix, st.bs) - st.sep_lo;
    st.n_total = st.n_dense + (min(p.L, i0 + tile_positions) - st.bs);
    return st;
}
// key position of stream element k, and the query range [lo, hi] that sees it
__device__ inline int stream_key(const Stream &s, int k, const sepattn_params &p,
                                 const int32_t *__restrict__ idx, const int32_t *__restrict__ prefix,
                                 int &lo, int &hi) {
    if (k >= s.n_total) {  // padding of the last tile: never visible, any valid row to load
        lo = kIntMax;
        hi = -1;
        return 0;
    }
    int j;
    if (k < s.n_init) {
        j = k;
        hi = kIntMax;
    } else if (k < s.n_dense) {
        // the clamps keep a stale list tail (caller broke sep_count <= cap) from faulting
        j = min(max(idx[min(s.sep_lo + k - s.n_init, p.cap - 1)], 0), p.L - 1);
        hi = kIntMax;
    } else {
        j = s.bs + (k - s.n_dense);
        bool always = (j < p.a) || (prefix[j + 1] != prefix[j]);
        hi = always ? kIntMax : j + p.n - 1;
    }
    lo = j;
    return j;
}

// Whether every pair of a block of 32 stream elements is visible to a wave with rows [pw, pw+31], as three comparisons
// against thresholds that are computed once per wave: a block of 32 stream elements starting at k0
// needs no mask test iff it lies in the dense part (k0 <= dense_last) or is a band block whose keys
// are inside every row's window and not in any row's future (band_first <= k0 <= band_last).
struct FullBlocks {
    int dense_last, band_first, band_last;
};
__device__ inline FullBlocks full_blocks(const Stream &st, int pw, int n) {
    FullBlocks f;
    const int pmax = pw + 31;
    f.dense_last = st.n_dense - 32;
    f.band_first = max(st.n_dense, st.n_dense + (pmax - n + 1) - st.bs);  // jmin + n - 1 >= pmax
    f.band_last = min(st.n_dense + (pw - 31) - st.bs, st.n_total - 32);   // jmax <= pw, no padding
    return f;
}
// no block of the tile is free of the mask test (a wave whose rows reach into the next document)
__device__ inline FullBlocks no_full_blocks() {
    FullBlocks f;
    f.dense_last = -(1 << 30);
    f.band_first = 1 << 30;
    f.band_last = -1;
    return f;
}
__device__ inline bool block_is_full(const FullBlocks &f, int k0) {
    return (k0 <= f.dense_last) | ((k0 >= f.band_first) & (k0 <= f.band_last));
}

}  // namespace sepattn
