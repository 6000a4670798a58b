// Geometry shared by the backward kernels: the compacted list of "far" keys (initial tokens and
// separators, the only keys a query can see beyond its neighbour window, Sec. 3.1) and the split of
// the far pass of dK/dV among persistent workgroups.
#pragma once

#include "common.h"
#include "key_stream.h"
#include "work_share.h"

namespace sepattn {

// A dK/dV workgroup holds KW key blocks of 32 keys, two waves each (32 KW keys, 128 KW threads), in one
// of two shapes:
//   KW = 4: 8 waves, one workgroup per compute unit.  Fewest tile loads per matrix instruction; the
//           better shape when a workgroup's pieces are long: d = 128, sequences from 8K on with
//           grouped heads.  dK/dV and the sum of its partials in us, KW = 4 / 2 (means of two runs, 1 to 2 % apart): 32/8 heads, L = 8192,
//           n = 256 196.7 / 198.5, n = 1024 348 / 382, two of them 408 / 418; 28/4 heads, L = 8192, n = 256 168 / 174, n = 1024 305 / 333; 16/4
//           heads, L = 8192, n = 256 109 / 112; 32/8 heads, L = 16384, n = 512 (dK/dV) 674 / 710; 8/2 heads, L = 16384 (dK/dV) 138 / 150.  Short
//           windows at 8K, where pieces are shorter, are on the wrong side of the line: 32/8 heads, n = 64 (dK/dV) 150 / 145.  Beyond
//           it: 16/4 heads, L = 4096, n = 256 52.7 / 47.5; 32/8 heads 89.1 / 89.2, but n = 1024 161 / 177; 32/32 heads, L = 8192, n = 256 265 / 255.
//   KW = 2: 4 waves, two workgroups per compute unit (three at d = 64, where the registers and the ring
//           of query tiles allow it) that run independently: one's piece start-up and partial stores
//           overlap the others' matrix work, the split of a (batch, KV head) is finer (it fills the
//           chip where 256 / (B Hkv) is not a whole number), and the workgroups' barriers do not lock
//           each other's phases.
// With packed documents the far pieces end with their documents, so the pieces are short at any
// length.  The launcher chooses (docs: the call has document bounds) and hands KW to both kernels;
// the workspace is laid out for the larger of the two shapes' needs, so its size does not depend
// on the choice.
inline int dkv_key_blocks(const sepattn_params &p, bool docs) {
    const long G = p.Hq / p.Hkv;
    return (p.d == 128 && !docs && p.L >= 8192 && G * p.L >= 32768) ? 4 : 2;
}
// workgroups of a shape that share a compute unit
inline int dkv_workgroups_per_cu(const sepattn_params &p, int kw) { return kw == 4 ? 1 : (p.d == 64 ? 3 : 2); }

__host__ __device__ inline int align_down32(int x) { return x & ~31; }

// x / y of numbers >= 0: a 64-bit division is some 150 instructions, and four or five of them stand at the start of a
// dK/dV kernel
__device__ inline long quotient(long x, long y) { return ((x | y) >> 31) ? x / y : (long)((uint32_t)x / (uint32_t)y); }

// Inclusive sums over the lanes of a wave, in registers (row_shr by 1, 2, 4, 8, then the rows' last lanes handed on).
__device__ inline int lanes_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 to rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31 to rows 2 and 3
    return v;
}

// The far work of one (batch, KV head): for list tile ft (bk = 32 KW consecutive list entries) the
// "items" (query tile, query head) from the first query that can see the tile's first key
// to the end of the sequence.  The items of all list tiles, in this order, are cut into slices, at
// most one per workgroup (`wpg` of them; workgroups with fewer band units get longer ones, see dkv_kernel); the
// part of a slice that lies in one list tile is a "piece" and produces one fp32 partial of that tile's dK / dV rows.  Piece (w, ft) uses partial slot w + ft
// (along the pieces either w or ft grows, so the slot numbers are distinct).
struct FarGeom {
    int wpg;     // workgroups per (batch, KV head)
    int bk;      // keys per workgroup and entries per list tile: 32 KW
    int NFcap;   // capacity of the far list, a multiple of bk
    int NFTcap;  // list tiles at full capacity
    int NP;      // partial slots per (batch, KV head)
    long rows;   // fp32 partial rows per (batch, KV head): NP slots of bk rows, then one band row per list entry (band units
                 // that are split among workgroups, see band_split: bk rows per part)
};
inline int dkv_workgroups_per_head(const sepattn_params &p, int kw) {
    const long n_bkv = (long)p.B * p.Hkv;
    const long w = dkv_workgroups_per_cu(p, kw) * (long)compute_units() / n_bkv;
    return (int)(w < 1 ? 1 : w);
}
// Among how many workgroups a band unit (32 KW keys and their windows, all query heads of the KV head) is split, by query
// heads.  A unit is a chain of G ((n + 30) / 32 + 1) steps of 0.7 us on one workgroup; where there are fewer units than
// workgroups it sets the time of the kernel.  Split, every key's sums pass through fp32 partials and the combine
// kernel, and the parts, with the slices of far work, which are cut as short as they are (see min_slice), share the compute units.
// Only units longer than three times the workgroups' mean work are split, into a number that divides the heads, gives no
// workgroup two parts, leaves a part four steps and spares eight: the number for which the steps of a part, 12 for each part and 6
// for each far slice that a compute unit gets, and 3 for the combine kernel where there is a split, are fewest together.
// Over 1760 calls with grouped heads and room for parts, 668 are split; of these 17 take more than 2 % longer than whole (at most 11 %), and
// the backward of all takes 0.87 of the time.  By the largest divisor alone it was 65 of 703, at most 44 %.  Backward in us, whole / 2 / 4 / 8
// parts, and what is chosen: 8/1 heads, d = 64, L = 3803, n = 32 45.3 / 47.8 / 65.2 / 54.3 (whole); L = 3662, n = 36 49.2 / 44.8 / 56.4 / 55.7
// (two); L = 527, n = 32 32.3 / 26.1 / 25.4 / 26.8 (four); d = 128, L = 2921, n = 19 51.7 / 52.0 / 64.8 / 55.4 (two); 32/8 heads, d = 128, L = 869,
// n = 86 43.7 / 47.6 / 54.7 (whole); 8/2 heads, L = 600, n = 96 dK/dV and combine 22.3 + 4.5 whole, 13.6 + 5.3 in four.
// (any_n: for the workspace, whose size does not depend on the window: the largest split of any window.)
inline int band_split(const sepattn_params &p, int wpg, int kw, bool any_n = false) {
    const int G = p.Hq / p.Hkv, steps = any_n ? 1 << 20 : ((p.n < p.L ? p.n : p.L) + 30) / 32 + 1;
    const long units = ((long)p.L + 32 * kw - 1) / (32 * kw);
    // far work in steps of 32 query rows, from the share of separators that work_share.h assumes
    const double out = any_n || p.n >= p.L ? 0. : p.L - p.n, far = (p.a + kSepShare * out / 2) * out / (1024. * kw) * G;
    if (3. * (far + (double)units * G * steps) > (double)wpg * G * steps) return 1;
    const double share = (double)p.B * p.Hkv / compute_units();  // of the workgroups of a (batch, KV head), per compute unit
    auto cost = [&](int s) {
        const long part = (long)G / s * steps, slice = part < 4 ? 4 : (part > 16 ? 16 : part), left = wpg - units * s;
        return part + (12. * units * s + 6. * (far / slice < left ? far / slice : left)) * share + (s > 1 ? 3. : 0.);
    };
    int split = 1;
    for (int s = 2; s <= G; ++s)
        if (G % s == 0 && units * s <= wpg && (long)G / s * steps >= 4 && (long)(G - G / s) * steps >= 8 && cost(s) < cost(split)) split = s;
    return split;
}
__host__ __device__ inline FarGeom far_geom(const sepattn_params &p, int wpg, int kw, int split = 1) {
    FarGeom g;
    g.wpg = wpg;
    g.bk = 32 * kw;
    g.NFcap = (p.a + p.cap + g.bk - 1) / g.bk * g.bk;
    g.NFTcap = g.NFcap / g.bk;
    g.NP = wpg + g.NFTcap;
    g.rows = (long)g.NP * g.bk + g.NFcap;
    if (split > 1) {
        const long band = ((long)p.L + g.bk - 1) / g.bk * g.bk * split;
        if (band > g.NFcap) g.rows = (long)g.NP * g.bk + band;
    }
    return g;
}

// backward workspace: D_i [B,Hq,L] fp32 | LSE_i * log2(e) [B,Hq,L] fp32 | dK partials | dV partials |
// first and last workgroup of every list tile [B,Hkv,NFTcap,2] int32
struct BwdWorkspace {
    size_t d_bytes, far_bytes, tab_bytes, total;
};
inline BwdWorkspace bwd_workspace(const sepattn_params &p) {
    BwdWorkspace w;
    w.d_bytes = align_up((size_t)p.B * p.Hq * p.L * sizeof(float), 256);
    w.far_bytes = w.tab_bytes = 0;
    // the eight-wave shape exists at d = 128 only
    for (int kw = 2; kw <= (p.d == 128 ? 4 : 2); kw += 2) {
        const int wpg = dkv_workgroups_per_head(p, kw);
        const FarGeom fg = far_geom(p, wpg, kw, band_split(p, wpg, kw, true));
        const size_t far = align_up((size_t)p.B * p.Hkv * fg.rows * p.d * sizeof(float), 256);
        const size_t tab = align_up((size_t)p.B * p.Hkv * fg.NFTcap * 2 * sizeof(int32_t), 256);
        w.far_bytes = far > w.far_bytes ? far : w.far_bytes;
        w.tab_bytes = tab > w.tab_bytes ? tab : w.tab_bytes;
    }
    w.total = 2 * w.d_bytes + 2 * w.far_bytes + w.tab_bytes;
    return w;
}

// Whether KV heads that see every earlier key work through the list of all keys (see dkv_kernel).  As band units their
// work is q = units / workgroups walks per workgroup, the longest about 1 + 1/q times the mean; as slices it is even, but
// every key's gradients pass through fp32 partials.  That pays where a workgroup has about one unit (eight waves,
// with nothing beside it on the compute unit to fill the gap: two) and the walks are long, with grouped heads, or
// next to KV heads with shorter windows, which leave the full ones more workgroups.
// Measured, a step in us, band units / slices, n = L.  Taken: 32/8 heads, d = 128, L = 8192 (q = 2, eight waves) 2716 / 2311,
// L = 2048 (q = 1/2) 339 / 235, 16/8 heads, d = 64, L = 4096 (q = 2/3) 320 / 270 and twice that batch (q = 4/3) 442 / 429, every
// other of 8/8 heads full, d = 64, L = 4096 246 / 205.  Not taken: 4 x 32/8 heads, L = 2048 (q = 2) 694 / 716, 2 x 12/12
// heads, d = 64, L = 4096 (q = 2) 367 / 399 and one (q = 1) 242 / 247; every other of 8 x 12/12 heads full, L = 300 54 / 82.
inline bool list_of_all_keys(const sepattn_params &p, int kw, int wpg, const FarGeom &fg, bool headwise) {
    const long units = (p.L + fg.bk - 1) / fg.bk, G = p.Hq / p.Hkv;
    const bool fits = p.cap + p.a >= p.L;  // the list has to fit where the far list does
    return fits && 3 * units <= (kw == 4 ? 6 : 4) * (long)wpg && G * p.L >= 4096 && (G >= 2 || headwise);
}

// Whether dQ and dK/dV of a call share a launch (bwd_joint.h), and with how many dQ workgroups per group; 0: they do not.  They do in
// four-wave shapes without split streams and without a list of all keys, whose query tiles are at most three eighths as many
// as the workgroups that fit the chip.  Beyond that, the tiles take from dK/dV the workgroups that its longest units and slices need.  Backward, two launches' time over one's, over 137 calls of two head sizes: up to 64 tiles 1.22 to 1.59 (1.34 in
// the mean), up to 128 1.22 to 1.56 (1.33), up to 192 1.01 to 1.36 (1.20), up to 256 0.74 to 1.29 (1.08), up to 320 0.48 to 1.22 (1.01).
// In us, two / one: 8/2 heads, L = 600, n = 96, d = 128 (38 tiles) 27.1 / 20.6, d = 64 22.2 / 17.2; 32/8 heads, L = 768, n = 100 (192) 40.0 /
// 31.9, d = 64 24.5 / 24.2; 12/12 heads, L = 2011, n = 64 (192) 42.1 / 37.7; 4 x 8/2 heads, L = 936, n = 657 (240) 59.4 / 80.3.
inline int joint_dq_workgroups(const sepattn_params &p, const HeadWin &hw, bool docs) {
    const QueryShape shape = query_shape(p);
    if (any_delta(hw) || shape.nw != 4 || dkv_key_blocks(p, docs) != 2) return 0;
    const int TP = 32 * shape.nw / shape.gp, tiles = (p.L + TP - 1) / TP;
    const long slots = 2l * compute_units(), n_groups = (long)p.B * (p.Hq / shape.gp), n_bkv = (long)p.B * p.Hkv;
    if (n_groups * tiles > slots * 3 / 8 || n_groups * tiles + n_bkv > slots) return 0;
    if (!docs && split_keys(p, hw, shape.gp, TP, slots, (size_t)-1)) return 0;
    const int wpg = dkv_workgroups_per_head(p, 2);
    if (!docs && p.n >= p.L && list_of_all_keys(p, 2, wpg, far_geom(p, wpg, 2), false)) return 0;
    return tiles;
}
// Workgroups per (batch, KV head) that dQ leaves dK/dV there: no more than dK/dV has by itself, which the workspace is laid out for.
inline int joint_dkv_workgroups(const sepattn_params &p, int dq_wpg) {
    const long n_dq = (long)p.B * (p.Hq / query_shape(p).gp) * dq_wpg, wpg = (2l * compute_units() - n_dq) / ((long)p.B * p.Hkv);
    return (int)(wpg < 1 ? 1 : wpg);
}

struct FarList {
    int a_eff, sep_base, NF;
};
// every_key: the list of all keys (see dkv_kernel), which far_pos and far_index treat as initial tokens
__device__ inline FarList far_list(const sepattn_params &p, const int32_t *__restrict__ prefix, bool every_key = false) {
    FarList f;
    if (every_key) {
        f.a_eff = f.NF = p.L;
        f.sep_base = 0;
        return f;
    }
    f.a_eff = p.a;  // already clamped to L by the host
    f.sep_base = load_uniform(prefix, f.a_eff);
    int cnt = min(load_uniform(prefix, p.L), p.cap);
    f.NF = f.a_eff + max(cnt - f.sep_base, 0);
    return f;
}
__device__ inline int far_pos(const FarList &fl, int f, const int32_t *__restrict__ idx, int L) {
    if (f < fl.a_eff) return f;
    return min(max(idx[fl.sep_base + f - fl.a_eff], 0), L - 1);
}
// index of key position j on the far list, -1 if it is neither an initial token nor a listed separator
__device__ inline int far_index(const FarList &fl, const int32_t *__restrict__ prefix, int j) {
    int f = -1;
    if (j < fl.a_eff)
        f = j;
    else if (prefix[j + 1] != prefix[j])
        f = fl.a_eff + prefix[j] - fl.sep_base;
    return f < fl.NF ? f : -1;
}
// first query row the far pieces of list entry f's tile cover (>= L: the entry has no far piece)
__device__ inline int far_first_query(const FarList &fl, int f, const int32_t *__restrict__ idx,
                                      const sepattn_params &p, int bk) {
    return align_down32(far_pos(fl, (f / bk) * bk, idx, p.L) + p.n);
}

// one past the last query row the far pieces of list entry f's tile cover: the end of the sequence,
// or, with packed documents (dend: one past the last position of each position's document, else
// nullptr), the end of the document of the tile's last entry.  A tile whose first query row
// (far_first_query) is not below this has no far piece.
__device__ inline int far_last_query(const FarList &fl, int f, const int32_t *__restrict__ idx,
                                     const sepattn_params &p, const int32_t *__restrict__ dend, int bk) {
    if (!dend) return p.L;
    const int last = min((f / bk + 1) * bk, fl.NF) - 1;
    return min(max(dend[far_pos(fl, last, idx, p.L)], 0), p.L);
}

// Adds the partials of a dK/dV pass of the four-wave shape with `wpg` workgroups per (batch, KV head).
int launch_dkv_combine_bf16(const sepattn_params &p, const int32_t *sep_idx, const int32_t *sep_prefix, const int32_t *doc_end,
                            uint16_t *dK, uint16_t *dV, const float *farK, const float *farV, const int32_t *piece_tab, int wpg, int split,
                            hipStream_t st);

// The backward of a small call: dQ and dK/dV in one launch (bwd_joint.h).  dq_wpg: workgroups per group of the dQ part.
int launch_joint_64(const sepattn_params &p, int dq_wpg, const uint16_t *Q, const uint16_t *K, const uint16_t *V, const uint16_t *O, const float *LSE,
                    const uint16_t *dO, const int32_t *sep_idx, const int32_t *sep_prefix, const int32_t *doc_start, const int32_t *doc_end,
                    uint16_t *dQ, uint16_t *dK, uint16_t *dV, float *Dws, float *Lws, float *farK, float *farV, int32_t *piece_tab, hipStream_t st);
int launch_joint_128(const sepattn_params &p, int dq_wpg, const uint16_t *Q, const uint16_t *K, const uint16_t *V, const uint16_t *O, const float *LSE,
                     const uint16_t *dO, const int32_t *sep_idx, const int32_t *sep_prefix, const int32_t *doc_start, const int32_t *doc_end,
                     uint16_t *dQ, uint16_t *dK, uint16_t *dV, float *Dws, float *Lws, float *farK, float *farV, int32_t *piece_tab, hipStream_t st);

// doc_end: packed documents ([B, L], p.a == 0), or nullptr
int launch_dkv_bf16(const sepattn_params &p, const HeadWin &hw, const uint16_t *Q, const uint16_t *K, const uint16_t *V,
                    const float *lse2, const uint16_t *dO, const float *Dws, const int32_t *sep_idx,
                    const int32_t *sep_prefix, const int32_t *doc_end, uint16_t *dK, uint16_t *dV, float *farK,
                    float *farV, int32_t *piece_tab, hipStream_t st);

}  // namespace sepattn
