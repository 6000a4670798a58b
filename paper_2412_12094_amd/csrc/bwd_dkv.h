// dK and dV (bf16 MFMA): the work of a workgroup, for the kernel that does nothing else (bwd_dkv_bf16.hip, which describes it) and for
// the one that runs it beside dQ (bwd_joint.h).
#pragma once

#include "bwd_common.h"
#include "mfma_common.h"
#include "work_share.h"

namespace sepattn {

namespace {

// First partial row of a KV head whose workgroups are dealt by work: slots for its workgroups and list tiles, then one
// band row per list entry, one KV head after the other.  The workgroups of a batch row are no more than with an
// even deal, so this fits the same workspace.
__device__ inline long shared_part_row(const FarGeom &even, const WorkShare &w, const ShareOf &s, const sepattn_params &p) {
    return (long)s.b * p.Hkv * even.rows + (long)w.first[s.pos] * even.bk + (long)s.pos * ((long)even.NFTcap * even.bk + even.NFcap);
}

// DOCS: packed documents (doc_end [B, L]: one past the last position of each position's document;
// p.a == 0, the documents' initial tokens are list entries): a key's query range ends with its
// document, and the far pieces of a list tile end with the document of the tile's last entry.
// HW: head-wise windows.  p.n becomes the largest window of the KV head's query heads: it fixes the far / band
// split and the schedule; in a band unit a key that is neither an initial token nor a separator is visible to
// query i of head h only while i <= j + p.n - 1 - delta[h] (a third comparison in the blocks that need the mask
// test).  The workgroups are dealt to the KV heads by their work (work_share.h).
// A KV head whose query heads all see every earlier key (n >= L) may have no band (`share.all`, see list_of_all_keys):
// its list is then that of ALL keys and its far pairs are i >= j, so that this work is cut into equal slices too; as
// a band unit the first keys' walk through the whole sequence is one workgroup's.
// What the slices of the far work depend on, per launch (head-wise windows: per KV head, worked out on the device).  The start of
// a workgroup, from its arguments to its first piece, is in the way of every call: with these numbers from the host, divisions
// by multiplication, sums over lanes in registers and the head-wise tables left to the head-wise kernel it takes 2900 cycles instead
// of 4900 at 8/2 heads, L = 600 (the kernel 11.2 -> 9.4 us, the step 45.4 -> 44.4), 8 x L = 2048 a step 157 -> 155 us.
struct DkvSlices {
    int G, Gs;              // query heads per KV head, per part of a band unit
    int every_key;
    int heavy;              // workgroups with one band unit more than the others
    int min_slice;          // items of the shortest slice
    int unit_items;         // what a band unit costs, in items
    FastDiv by_bkv, by_hkv, by_G, by_split, by_wpg, by_min_slice;  // by_bkv: (batch, KV head)s of the call
    __host__ __device__ void set(int n_band, int wpg, int Gs, int n, bool every_key, int blocks_per_tile) {
        constexpr int kUnitStart = 8;  // steps of 32 query rows
        const int unit_steps = Gs * ((n + 30) / 32 + 1), least = unit_steps < 4 ? 4 : (unit_steps > 16 ? 16 : unit_steps);
        heavy = n_band % wpg;
        min_slice = (every_key ? 16 : least) / blocks_per_tile;
        unit_items = (unit_steps + kUnitStart) / blocks_per_tile;
    }
};

inline DkvSlices dkv_slices(const sepattn_params &p, int kw, int wpg, int split, bool every_key) {
    DkvSlices sl;
    sl.G = p.Hq / p.Hkv;
    sl.Gs = sl.G / split;
    sl.every_key = every_key;
    sl.set(every_key ? 0 : (p.L + 32 * kw - 1) / (32 * kw) * split, wpg, sl.Gs, every_key ? 0 : p.n, every_key, kw == 2 ? 1 : 2);
    sl.by_bkv = fast_div((uint32_t)(p.B * p.Hkv));
    sl.by_hkv = fast_div((uint32_t)p.Hkv);
    sl.by_G = fast_div((uint32_t)sl.G);
    sl.by_split = fast_div((uint32_t)split);
    sl.by_wpg = fast_div((uint32_t)wpg);
    sl.by_min_slice = fast_div((uint32_t)sl.min_slice);
    return sl;
}

// Query rows per LDS tile.  Workgroups that share a compute unit (two at d = 128 with 80 KB each,
// three at d = 64 with 53 KB and 168 registers) stream tiles of 32 rows (one block) through the
// ring of four, the single workgroup tiles of 64 rows (two blocks).
template <int D, int KW>
struct DkvLds {
    static constexpr int kRows = KW == 2 ? 32 : 64, kTiles = 4;
    alignas(1024) uint16_t Qs[kTiles][kRows * D];
    alignas(1024) uint16_t dOs[kTiles][kRows * D];
    alignas(256) float row_s[2][kTiles][2][64];  // LSE*log2e, -D of a tile's one or two blocks: 32 values twice
    alignas(1024) uint16_t Pex[KW][2][2][64 * 8];  // [key block][step parity][k-half][lane*8], bf16
};
// bkv, w_id: (batch, KV head) and number of the workgroup (head-wise windows: bkv is the block's number)
template <int D, bool DOCS, bool HW, int KW, bool PARTS>
__device__ __forceinline__ void dkv_work(
    DkvLds<D, KW> &lds, int bkv, int w_id, sepattn_params p, const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K,
    const uint16_t *__restrict__ V, const float *__restrict__ LSE2, const uint16_t *__restrict__ dO,
    const float *__restrict__ Dws, const int32_t *__restrict__ sep_idx,
    const int32_t *__restrict__ sep_prefix, const int32_t *__restrict__ doc_end,
    uint16_t *__restrict__ dK, uint16_t *__restrict__ dV,
    float *__restrict__ farK, float *__restrict__ farV, int32_t *__restrict__ piece_tab, int wpg, int n_band,
    int split, DkvSlices sl, HeadArgs<HW> ha) {
    constexpr int NW = 2 * KW;               // waves per workgroup
    constexpr int BK = 32 * KW;              // keys per workgroup
    constexpr int CH = D / 8;                // 16-byte chunks per row
    constexpr int RPL = 64 / CH;             // rows covered by one wave-wide 1 KB load
    constexpr int BQ = DkvLds<D, KW>::kRows;  // query rows per LDS tile
    constexpr int BPT = BQ / 32;             // blocks of 32 query rows per tile
    // The loads of a tile (36 wave-wide ones per compute unit, 16 cycles each, and the waves that issue them stand still
    // meanwhile) are issued where there is time to spare.  With eight waves each role loads the tensor that it reads first, the
    // P-waves in front of their softmax, the dS-waves in front of the barrier: with all loads on the P-waves these came 300 cycles later to
    // the barrier of a step of 2000.  With four waves the dS-waves load, in front of the barrier (see refill), although they are the later
    // ones: the two workgroups of a compute unit fill each other's gaps.  By all waves right behind the barrier, where every wave has
    // the longest way to go, the loads cost 325 - 590 of 2400 cycles per step.  dK/dV, us, P-waves / each its own: 32/8 heads, d = 128, L = 8192,
    // n = 256 205.4 / 202.5, L = 12000, n = 128 312 / 300, L = 16384, n = 512 655 / 645, 28/4 heads, L = 8192, n = 1024 297 / 291.  Four waves,
    // dS-waves / each its own: 28/4 heads, 3 x L = 3077 133 / 136, 32/8 heads, L = 4096, n = 256 82.3 / 83.1.
    constexpr bool EACH = KW == 4;           // each role loads its own tensor, else the dS-waves both
    constexpr int TILE_LOADS[2] = {EACH ? 16 / RPL : 0, (EACH ? 1 : 2) * (16 / RPL) + 1};  // wave-wide loads per tile, by role
    constexpr int LOADS = BQ / (RPL * KW);   // wave-wide loads per loading wave per tensor per tile
    constexpr int KSTEPS = D / 16;
    constexpr int DB = D / 32;
    constexpr int TILE = BQ * D;
    constexpr int NBUF = DkvLds<D, KW>::kTiles;
    static_assert(LOADS * RPL * KW == BQ && 2 * BPT == KW, "tile must divide among the waves");

    auto &Qs = lds.Qs;
    auto &dOs = lds.dOs;
    auto &Pex = lds.Pex;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int role = wave / KW;  // 0: P-wave (S, dV), 1: dS-wave (dP, dK)
    const int kbw = wave % KW;   // key block of the wave
    const int kj = lane & 31, hh = lane >> 5;
    const int G = sl.G;
    if constexpr (!PARTS) split = 1;
    const int Gs = PARTS ? sl.Gs : G;  // query heads per part of a band unit (see band_split); n_band counts the parts
    // Consecutive workgroups belong to consecutive (batch, KV head) pairs (the grid's first dimension), so with 8 KV heads
    // each head's K, V, Q, dO rows stay in the L2 of one XCD.
    long part0 = bkv * far_geom(p, wpg, KW, split).rows;  // first partial row of the (batch, KV head)
    int gdelta = 0;
    bool every_key = false;
    if constexpr (HW) {
        const ShareOf s = share_of(ha.share, bkv, p.B);
        bkv = s.b * p.Hkv + ha.share.group[s.pos];
        part0 = shared_part_row(far_geom(p, wpg, KW), ha.share, s, p);
        w_id = s.rank;
        wpg = s.count;
        gdelta = ha.of_group((bkv - s.b * p.Hkv) * G, G);
        every_key = ha.share.all[s.pos] != 0;
        p.n = every_key ? 0 : p.n - gdelta;
        if (every_key) n_band = 0;
        sl.set(n_band, wpg, Gs, p.n, every_key, BPT);
    } else if constexpr (!DOCS) {
        every_key = sl.every_key != 0;
        if (every_key) p.n = n_band = 0;
    }
    const int b = quotient(bkv, sl.by_hkv), kv = bkv - b * p.Hkv;
    const int32_t *prefix = sep_prefix + (long)b * (p.L + 1);
    const int32_t *idx = sep_idx + (long)b * p.cap;
    const int32_t *dend = DOCS ? doc_end + (long)b * p.L : nullptr;
    const long kvrow0 = ((long)b * p.Hkv + kv) * (long)p.L;
    const float sl2 = p.scale * kLog2e_f;
    const FarGeom fg = far_geom(p, wpg, KW);
    const FarList fl = far_list(p, prefix, every_key);
    const int a_row = pi_row(kj);
    const int my_pc = lane % CH, my_sub = lane / CH;
    // byte offset within a tile of Q or dO of what this lane fetches of the wave's first rows; those RPL rows on differ by
    // them and by a chunk bit each (kSwzBoth; the wave's rows start at a multiple of 16)
    constexpr uint32_t ROWB = D * 2;
    static_assert(LOADS * RPL == 16, "a loading wave's rows");
    const uint32_t my_off = (uint32_t)(16 * kbw + my_sub) * ROWB + swz_chunk<kSwzBoth, D>(my_pc, my_sub) * 16;
    // Per-lane byte offsets of the operand fragments inside a tile, computed once.  The first
    // contraction reads rows of T1 (Q for the P-wave, dO for the dS-wave), the second reads the other
    // tensor (T2) transposed.  Row-major fragments: the XOR permutation acts on the 16-byte chunk
    // index 2*ks + hh and the k-step only enters through bits 1..3 of it, so fragment ks sits at
    // (fragment 0) ^ (32 * ks); tile and block bases are multiples of 1 KB, so the XOR commutes with
    // adding them.
    const uint32_t q_base = lds_addr(&Qs[0][0]), do_base = lds_addr(&dOs[0][0]), row_base = lds_addr(&lds.row_s[0][0][0][0]);
    const uint32_t t1_base = (role == 0 ? q_base : do_base) + lds_off_a<kSwzBoth, D>(a_row, hh);
    const uint32_t t2_base = role == 0 ? do_base : q_base;
    uint32_t ktr0[DB], ktr1[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) {
        ktr0[db] = t2_base + lds_off_a_tr<kSwzBoth, D>(db * 32, lane);
        ktr1[db] = t2_base + lds_off_a_tr_second<kSwzBoth, D>(db * 32, lane);
    }

    // ---- the far work of this (batch, KV head) and this workgroup's slice [s0, s1) of it.
    // Lane t of a group of 64 list tiles describes tile t: first query row and number of items.
    const int NFT = (fl.NF + BK - 1) / BK;
    auto tile_items = [&](int t, int &fq) __attribute__((always_inline)) {
        fq = p.L;
        int qe = p.L;
        if (t < NFT) {
            fq = align_down32(far_pos(fl, t * BK, idx, p.L) + p.n);
            qe = far_last_query(fl, t * BK, idx, p, dend, BK);
        }
        return fq < qe ? G * ((qe - fq + BQ - 1) / BQ) : 0;
    };
    // the first group of 64 list tiles is worked out once, for the total and for the pieces
    int first_fq, first_nq = tile_items(lane, first_fq), first_inc = lanes_scan(first_nq);
    long far_total = __builtin_amdgcn_readlane(first_inc, 63);
    for (int base = 64; base < NFT; base += 64) {
        int fq;
        far_total += __builtin_amdgcn_readlane(lanes_scan(tile_items(base + lane, fq)), 63);
    }
    // Slices.  Where the band units do not divide among the workgroups, the first `heavy` have one more than the others,
    // and far work goes to those others first, as much as a band unit costs (in items, with its start).  Without that
    // a workgroup with two units and a full slice sets the time where most have one unit (28/4 heads, 3 x L=3077,
    // 49 units on 42 workgroups: 190 us, 174 with it).  No slice is shorter than min_slice, the steps of a
    // band unit up to 16: the start of a piece and the
    // sum of many partials would cost more than the items (8/2 heads, L = 600: 29 + 12.6 us with slices of one
    // item, 22 + 4 now).  The slices that are not empty belong to consecutive workgroups, which is what the combine
    // kernel relies on.
    auto by = [](long x, FastDiv f, int d) { return x >> 31 ? x / d : (long)quotient((int)x, f); };
    const int heavy = sl.heavy, light = wpg - heavy, min_slice = sl.min_slice;
    const long unit_items = sl.unit_items;
    // What is left when the others have that much goes to all in equal parts; where these would be shorter than min_slice,
    // slices of min_slice go to as many of the first (`n_heavy`, the last of them) as it takes to leave the others no more than
    // one beyond a unit's cost.  All of it to the others, one workgroup of sixteen got the far work of 47 units' keys: dK/dV and
    // combine in us, so / now: 32/32 heads, L = 3000, n = 512 178 / 103, 16/8 heads, L = 3856, n = 156 174 / 57, 4 x 32/8 heads, L = 3000,
    // n = 1024 605 / 483; over 240 calls 1.02 times as fast, level where the units divide evenly.
    // What the equal parts leave over goes to the others too, unless that would be more than two items each: then they get one, and as many
    // of the first (`extra`) as there are more.  All of it to the others, one workgroup of 43 got 39 items where the rest had a unit (10
    // items) and four.  Backward in us, so / now: 8/8 heads, n = 22, L = 2646, d = 64 35 to 45 (with the separators) / 27 to 28, L = 2611,
    // d = 128 47.3 / 39.1.
    long per_heavy = 0, n_heavy = 0;
    int extra = 0;
    if (heavy) {
        const long rest = max(far_total - unit_items * light, 0l);
        per_heavy = HW ? quotient(rest, wpg) : by(rest, sl.by_wpg, wpg);
        n_heavy = heavy;
        if (per_heavy < min_slice) {
            per_heavy = min_slice;
            n_heavy = min(max((HW ? quotient(rest, min_slice) : by(rest, sl.by_min_slice, min_slice)) - light, 0l), (long)heavy);
        } else {
            const int over = (int)(rest - per_heavy * wpg) - light;
            extra = over > light ? over : 0;
        }
    }
    auto heavy_start = [&](int v) __attribute__((always_inline)) { return v * per_heavy + min(v, extra); };  // of workgroup v of those n_heavy
    const long all_heavy = per_heavy * n_heavy + extra, far_light = far_total - all_heavy;
    const long n_light = min(max(HW ? quotient(far_light, min_slice) : by(far_light, sl.by_min_slice, min_slice), 1l), (long)light);
    const int w_light = w_id - heavy;
    // the first of the slices w of n_light equal ones: floor(w far_light / n_light), w <= n_light <= wpg, from one division
    const long whole = quotient(far_light, n_light), over = far_light - whole * n_light;
    auto slice_start = [&](long w) __attribute__((always_inline)) {
        const long x = w * over;  // < n_light^2
        return w * whole + (x < kSmallQuotient ? (long)small_quotient((int)x, reciprocal((int)n_light)) : x / n_light);
    };
    const int v_heavy = w_light + (int)n_heavy;
    const long s0 = w_light < 0 ? heavy_start(max(v_heavy, 0)) : all_heavy + slice_start(min((long)w_light, n_light));
    const long s1 = w_light < 0 ? (v_heavy < 0 ? 0l : heavy_start(v_heavy + 1)) : all_heavy + slice_start(min(w_light + 1l, n_light));

    // iteration state over the pieces: first the far pieces of the slice (list tiles in groups of 64,
    // `pend` = tiles of the current group that overlap the slice and are still to be visited), then
    // the band units
    int it_phase = 0, grp_next = 0, grp_base = 0, band_u = w_id;
    long cum_next = 0, grp_cum = 0;
    int g_fq = 0, g_nq = 0, g_excl = 0;
    unsigned long long pend = 0;
    for (;;) {
        bool FAR = false, have = false;
        int ft = 0, fq0 = 0, item0 = 0, n_items = 0, unit = 0, n_qt = 1;
        while (!have) {
            if (it_phase == 0) {
                if (pend == 0) {
                    if (grp_next >= NFT || cum_next >= s1) {
                        it_phase = 1;
                        continue;
                    }
                    grp_base = grp_next;
                    grp_cum = cum_next;
                    g_nq = first_nq;
                    g_fq = first_fq;
                    int inc = first_inc;
                    if (HW || grp_base > 0) {  // head-wise: once more, rather than registers that d = 64 does not have
                        g_nq = tile_items(grp_base + lane, g_fq);
                        inc = lanes_scan(g_nq);
                    }
                    g_excl = inc - g_nq;
                    pend = __ballot(g_nq > 0 && grp_cum + inc > s0 && grp_cum + g_excl < s1);
                    cum_next = grp_cum + __builtin_amdgcn_readlane(inc, 63);
                    grp_next = grp_base + 64;
                    continue;
                }
                const int l = __ffsll(pend) - 1;
                pend &= pend - 1;
                const long first = grp_cum + __builtin_amdgcn_readlane(g_excl, l);
                const int nq = __builtin_amdgcn_readlane(g_nq, l);
                const long lo_i = s0 > first ? s0 : first, hi_i = s1 < first + nq ? s1 : first + nq;
                ft = grp_base + l;
                fq0 = __builtin_amdgcn_readlane(g_fq, l);
                item0 = (int)(lo_i - first);
                n_items = (int)(hi_i - lo_i);
                n_qt = quotient(nq, sl.by_G);
                // the combine kernel finds the pieces of a list tile through its first and last workgroup
                if (tid == 0) {
                    int32_t *tab = piece_tab + ((long)bkv * fg.NFTcap + ft) * 2;
                    if (item0 == 0) tab[0] = w_id;
                    if (item0 + n_items == nq) tab[1] = w_id;
                }
                FAR = true;
                have = true;
            } else {
                if (band_u >= n_band) break;
                unit = band_u;
                band_u += wpg;
                have = true;
            }
        }
        if (!have) break;
        // the previous piece's last LDS reads are done in every wave before its buffers are refilled
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();

        // ---- this wave's 32 keys and the query range of the piece.  Item i of the piece is query tile
        // i % n_qt (64 rows from q_lo on) of query head i / n_qt.
        int j, lo, hi, q_lo, q_hi, fidx = 0;
        int hi2 = 1 << 29;  // HW: last query row of the head with the LARGEST window that sees the key as a neighbour
        bool valid;
        if (FAR) {
            q_lo = fq0;
            q_hi = far_last_query(fl, ft * BK, idx, p, dend, BK);
            fidx = ft * BK + 32 * kbw + kj;
            valid = fidx < fl.NF;
            j = valid ? far_pos(fl, fidx, idx, p.L) : 0;
            lo = j + p.n;
            hi = q_hi - 1;
            if constexpr (DOCS) hi = min(hi, dend[j] - 1);
        } else {
            const int j0 = (PARTS ? quotient(unit, sl.by_split) : unit) * BK;
            j = j0 + 32 * kbw + kj;
            valid = j < p.L;
            q_lo = j0;
            q_hi = min(p.L, j0 + BK + p.n - 1);
            lo = j;
            hi = min(j + p.n - 1, p.L - 1);
            if constexpr (HW) {
                const int jj = valid ? j : 0;
                if (!(jj < p.a || prefix[jj + 1] != prefix[jj])) hi2 = jj + p.n - 1;
            }
            if (!valid) j = 0;
            if constexpr (DOCS) hi = min(hi, dend[j] - 1);
            item0 = 0;
            n_qt = (q_hi - q_lo + BQ - 1) / BQ;
            n_items = Gs * n_qt;
        }
        if (!valid) {
            lo = kIntMax;
            hi = -1;
        }
        // visibility of query row i for this lane's key: lo <= i <= hi, tested with one comparison as
        // (unsigned)(i - lo) <= hi - lo; an empty range (hi < lo) becomes lo = max int, span 0
        const int lo_m = hi >= lo ? lo : kIntMax;
        const uint32_t span_m = hi >= lo ? (uint32_t)(hi - lo) : 0u;
        // wave-uniform bounds of the keys' query ranges, in scalar registers so that the per-block
        // decisions below are scalar branches
        // (the keys ascend with the lane, invalid ones come last: the extremes sit in the first and the last lane, that of
        // hi2 in the first key that is neither an initial token nor a separator)
        const int lo_max = __builtin_amdgcn_readlane(lo, 31);
        const int hi_min = min(__builtin_amdgcn_readlane(hi, 0), __builtin_amdgcn_readlane(hi, 31));
        int hi2_min = 1 << 29;
        if constexpr (HW) {
            const unsigned long long near = __ballot(hi2 < (1 << 29));
            if (near) hi2_min = __builtin_amdgcn_readlane(hi2, __ffsll(near) - 1);
        }

        // Resident B operand: K rows for the P-wave, V rows for the dS-wave.  They come through LDS, into the half of the ring
        // that the piece's third and fourth tile will take (8 KB per wave at d = 128, its own): a load straight into the
        // operand layout is 64 scattered 16-byte pieces per instruction, and the number of such pieces is what it
        // costs (with them, the start of a piece spent 7000 to 11000 cycles issuing its loads).
        const uint32_t row_lds = (role == 0 ? q_base : do_base) + 2 * (TILE * 2) + kbw * (32 * D * 2);
        {
            const char *rows = reinterpret_cast<const char *>((role == 0 ? K : V) + kvrow0 * D);
            static_for<32 / RPL>([&](auto U) {
                const int r = decltype(U)::value * RPL + my_sub;
                const uint32_t off = (uint32_t)__shfl(j, r) * (uint32_t)(D * 2) + swz_chunk<kSwzRow, D>(my_pc, r) * 16;
                dma_to_lds_16(rows, off, row_lds + decltype(U)::value * 1024);
            });
        }
        bf16x8 breg[KSTEPS];
        f32x16 acc[DB];  // dV^T (P-wave) or dK^T (dS-wave) of the wave's keys
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[db][i] = 0.f;

        // The piece as a sequence of steps; in every step a wave works on one block of 32 query rows.
        // Far piece: block s of its tiles in step s.  Band unit: a key block of 32 keys needs only NBK
        // of the nbh blocks of a head (the queries j <= i < j+n of its keys), key block kb the blocks
        // kb .. kb+NBK-1; all waves walk through a head's blocks together, but the last ov = nbh-NBK
        // steps of a head are merged with the first ov steps of the next head: in merged step b the
        // key blocks kb > b finish the old head (block NBK+b, which the others cannot see) while the
        // key blocks kb <= b start the new one (block b, which the others cannot see either: its
        // queries come before their keys).  A head then costs NBK steps instead of nbh.
        const int n_tiles = n_items;
        const int nbh = FAR ? BPT * n_tiles : BPT * n_qt;        // blocks per "head" (a far piece is one run)
        const int NBK = (p.n + 30) / 32 + 1;
        // steps from one head's start to the next's: at least NBK; at most KW-1 merged steps;
        // and more than half a head, so that a head's tail only overlaps the head that follows it and
        // the ring of NBUF tiles always holds what two consecutive steps need
        int st_P = NBK > nbh / 2 + 1 ? NBK : nbh / 2 + 1;
        st_P = st_P > nbh - (KW - 1) ? st_P : nbh - (KW - 1);
        // a tile is requested one barrier before the barrier that waits for it, so the tiles of three
        // consecutive steps must fit the ring: with one block per tile a head's first step needs two
        // plain steps behind it
        if (BPT == 1 && st_P < 3) st_P = 3;
        if (FAR || st_P > nbh) st_P = nbh;
        const int st_ov = nbh - st_P;                            // 0 .. KW-1
        const int st_G = FAR ? 1 : Gs;
        const int n_blocks = (st_G - 1) * st_P + nbh;            // steps of the piece
        const int tiles_per_head = FAR ? 0 : n_qt;

        // tile tt -> LDS buffer tt%4: a loading wave of key block kbw fills rows (LOADS*kbw + u)*RPL ..
        // +RPL-1 with one wave-wide direct load per tensor; a lane owns physical chunk lane%CH of its row and
        // fetches the logical chunk the permutation maps there, and the 32 row values (LSE*log2e or -D) of one block with one
        // load.  Tiles are issued in order, head by head: the next one is query tile iss_qt of the head iss_g (at first) and
        // begins iss_off bytes into Q and dO.  Its address is the same for all lanes, the lanes' parts are constants: 40
        // instructions a tile, where one address per load took 125, on the path of the wave that the others wait for.  A tile that
        // reaches past the sequence's end clamps its rows (they are masked by the [lo, hi] test: hi <= L-1).
        // dK/dV in us, before / now: 32/8 heads, d = 128, n = 256, L = 8192 218 / 210, L = 4096 86.5 / 83.7, n = 512, L = 16384 681 / 662; 28/4
        // heads, 3 x L = 3077 137.7 / 132.4; 8 x 12/12 heads, L = 2048, d = 64 61.2 / 59.4.
        int iss_tt = 0, iss_g = item0 < kSmallQuotient ? __builtin_amdgcn_readfirstlane(small_quotient(item0, reciprocal(n_qt))) : item0 / n_qt;
        const int q0_tile = item0 - iss_g * n_qt;
        int iss_qt = q0_tile;
        if (PARTS && !FAR) iss_g = (unit - quotient(unit, sl.by_split) * split) * Gs;  // the part's first head
        size_t iss_off = ((((long)b * p.Hq + kv * G + iss_g) * (long)p.L) + q_lo + iss_qt * BQ) * ROWB;
        const int n_whole = (p.L - q_lo) / BQ;  // tiles of a head that end within the sequence
        const size_t to_next_head = ((size_t)p.L - (size_t)(n_qt - 1) * BQ) * ROWB;
        auto issue_tile = [&]() {
            if (EACH || role == 1) {
                const uint32_t buf = iss_tt & (NBUF - 1);
                const uint32_t to = buf * (TILE * 2) + kbw * (LOADS * RPL * ROWB);
                const char *qp = reinterpret_cast<const char *>(Q) + iss_off, *dop = reinterpret_cast<const char *>(dO) + iss_off;
                uint32_t off[LOADS];
#pragma unroll
                for (int u = 0; u < LOADS; ++u) off[u] = my_off ^ (u * (D == 128 ? 16u : 32u));
                const bool whole = iss_qt < n_whole;
                const uint32_t last = p.L - q_lo - iss_qt * BQ - 1;  // not whole: row of the tile that is the sequence's last
                if (whole) {
                    if (!EACH || role == 0) dma_to_lds_16_rows(qp, off, q_base + to);
                    if (role == 1) dma_to_lds_16_rows(dop, off, do_base + to);
                } else {
                    static_for<LOADS>([&](auto U) {
                        constexpr int u = U;
                        off[u] = min(off[u] + u * 1024u, last * ROWB | (off[u] & (ROWB - 1)));
                        if (!EACH || role == 0) dma_to_lds_16(qp, off[u], q_base + to + u * 1024u);
                        if (role == 1) dma_to_lds_16(dop, off[u], do_base + to + u * 1024u);
                    });
                }
                if (role == 1) {
                    const int which = kbw / BPT, half = kbw % BPT;
                    const char *rp = reinterpret_cast<const char *>(which ? Dws : LSE2) + iss_off / (ROWB / 4);
                    const uint32_t row = 4u * (32 * half + kj);
                    dma_to_lds_4(rp, whole ? row : min(row, 4u * last), row_base + ((which * NBUF + buf) * 2 + half) * 256);
                }
            }
            ++iss_tt;
            ++iss_qt;
            iss_off += iss_qt == n_qt ? to_next_head : (size_t)(BQ * ROWB);
            if (iss_qt == n_qt) iss_qt = 0;
        };
        // wait until at most the wave's loads of the n_out newest tiles are still in flight: loads complete in the
        // order they were issued, TILE_LOADS of them per tile.  (A wave that issues none waits here for its resident rows at the
        // start of a piece.)
        auto wait_tiles = [&](int n_out) __attribute__((always_inline)) {
            auto of = [&](auto LW) __attribute__((always_inline)) {  // LW: the wave's loads of a tile
                constexpr int lw = decltype(LW)::value;
                if (n_out <= 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                else if (n_out == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(lw) : "memory");
                else if (n_out == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * lw) : "memory");
                else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * lw) : "memory");
            };
            if (role == 0) of(IntC<TILE_LOADS[0]>{});
            else of(IntC<TILE_LOADS[1]>{});
        };

        // ---- per-step pieces.  What a wave needs to know about a step (the LDS offset of its block, the
        // block's first query row, whether the block needs the mask test, which tiles the step and its
        // successor touch) is computed for 64 steps at a time, one step per lane, and fetched with
        // three v_readlane per step: scalar bookkeeping inside the loop costs issue slots that the
        // matrix instructions need.  Tiles are numbered in load order (head-major).
        struct Blk {
            int dlt;         // HW: how much shorter the window of the block's head is than p.n
            int r0, ps, rv;  // first query row; parity of the step (P exchange slot); float offset of the row values
            uint32_t off;    // byte offset of the block's first row from the start of the ring
            bool full;       // every (query, key) pair of the block is visible: no mask test needed
        };
        // step s: the tile and block this wave (key block kbw) works on, lowest / highest tile of any wave
        int step_head = 0;  // head (within the group) of the block step_of was last asked about (band units)
        const bool few = n_blocks + n_qt < kSmallQuotient;  // steps and tiles are divided by reciprocals
        const float by_P = reciprocal(st_P), by_qt = reciprocal(n_qt);
        auto step_of = [&](int s, int &tile, int &blk, int &lo_t, int &hi_t) __attribute__((always_inline)) {
            const int g = FAR ? 0 : few ? small_quotient(s, by_P) : s / st_P, b = s - g * st_P;
            const int base_t = g * tiles_per_head;
            const bool mg = g > 0 && b < st_ov;
            const int own = base_t + b / BPT, old = base_t - tiles_per_head + (b + st_P) / BPT;
            const bool prev = mg && (kbw > b || g == st_G);
            step_head = prev ? g - 1 : g;
            tile = prev ? old : own;
            blk = prev ? b + st_P : b;
            lo_t = mg ? old : own;
            hi_t = (mg && g == st_G) ? old : own;
        };
        uint32_t sch_off = 0;
        int sch_r0 = 0, sch_t = 0, sch_d = 0;
        auto fill_schedule = [&](int first) __attribute__((always_inline)) {
            const int sidx = first + lane;
            int tile, blk, lo_t, hi_t, tile_n, blk_n, lo_n, hi_n;
            step_of(sidx, tile, blk, lo_t, hi_t);
            int dl = 0;
            if constexpr (HW) {
                // the head's delta: the table is indexed with wave-uniform numbers only
                const int hd = step_head;
                for (int g = 0; g < G; ++g) {
                    const int sd = ha.of_head(kv * G + g) - gdelta;
                    dl = (!FAR && hd == g) ? sd : dl;
                }
            }
            step_of(sidx + 1, tile_n, blk_n, lo_n, hi_n);
            if (sidx + 1 >= n_blocks) hi_n = n_tiles - 1;
            const int buf = tile % NBUF, qb = blk % BPT;
            const int q = q0_tile + blk / BPT, q_head = few ? small_quotient(q, by_qt) : q / n_qt;
            const int r0 = q_lo + (q - q_head * n_qt) * BQ + 32 * qb;
            bool full = (r0 >= lo_max) && (r0 + 31 <= hi_min);
            if constexpr (HW) full = full && (r0 + 31 + dl <= hi2_min);
            sch_d = dl;
            sch_off = (uint32_t)buf * (TILE * 2) + (uint32_t)qb * (32 * D * 2);
            sch_r0 = r0 | (buf << 2) | (qb << 1) | (full ? 1 : 0);  // r0 is a multiple of 32
            sch_t = (lo_t << 2) | max(0, min(hi_n - lo_t, 3));
        };
        int st_n = -1;                            // number of the step handed out last
        int lo_cur = 0, hi_next = 0;              // lowest tile of that step; highest tile of the step after it
        int lo_free = 0;                          // tiles below this one are read by no wave any more
        int hi_landed = 0;                        // highest tile this wave has waited for
        auto next_block = [&]() __attribute__((always_inline)) {
            ++st_n;
            const int l = st_n & 63;
            if (l == 0) fill_schedule(st_n);
            Blk k;
            k.off = __builtin_amdgcn_readlane(sch_off, l);
            const int r0p = __builtin_amdgcn_readlane(sch_r0, l);
            const int tp = __builtin_amdgcn_readlane(sch_t, l);
            k.r0 = r0p & ~31;
            k.full = r0p & 1;
            k.rv = (r0p & 14) << 5;
            k.ps = st_n & 1;
            k.dlt = HW ? __builtin_amdgcn_readlane(sch_d, l) : 0;
            lo_cur = tp >> 2;
            hi_next = lo_cur + (tp & 3);
            return k;
        };
        // fragment reads by precomputed address: one vector instruction per read forms the address
        auto rd_row = [&](uint32_t rbase, int ks) __attribute__((always_inline)) {
            return lds_read_b128_at(rbase ^ (32u * ks));
        };
        // rows 16*stp .. +15 of the block, columns 32*db .. +31, transposed.  For d = 128 the second
        // 64-bit read is the first with chunk bit 0 flipped, four rows on.
        auto rd_tr = [&](uint32_t boff, int stp, int db) __attribute__((always_inline)) {
            const uint32_t first = boff + ktr0[db];
            const uint32_t second = D == 128 ? (first ^ 16u) + 4u * D * 2u : boff + ktr1[db];
            return lds_read_tr_at2(first + stp * 16 * D * 2, second + stp * 16 * D * 2);
        };
        auto read_rows = [&](const Blk &k, bf16x8 (&afr)[KSTEPS]) __attribute__((always_inline)) {
            const uint32_t rbase = t1_base + k.off;
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) afr[ks] = rd_row(rbase, ks);
        };
        auto read_transposed = [&](const Blk &k, bf16x8 (&tfr)[2][DB]) __attribute__((always_inline)) {
#pragma unroll
            for (int stp = 0; stp < 2; ++stp)
#pragma unroll
                for (int db = 0; db < DB; ++db) tfr[stp][db] = rd_tr(k.off, stp, db);
        };
        // The two contractions of one pipeline step, with the LDS reads of the later one placed
        // between the MFMA groups of the earlier one: a fragment is requested four MFMAs (128 cycles)
        // before its use, and at most 32 fragment registers are live.  The scheduling fences keep the
        // compiler from hoisting all reads to the top (which would spill).
        auto zero = [&](f32x16 &x) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = 0.f;
        };
        // acc += T2^T(cur) x_b(cur), then x = T1(nxt) B        (P-wave order)
        auto gemm2_then_gemm1 = [&](const Blk &cur, const bf16x8 (&xb)[2], const Blk &nxt, f32x16 &x) __attribute__((always_inline)) {
            const uint32_t rbase = t1_base + nxt.off;
            bf16x8 t0[DB], t1[DB], a0[KSTEPS / 2], a1[KSTEPS / 2];
#pragma unroll
            for (int db = 0; db < DB; ++db) t0[db] = rd_tr(cur.off, 0, db);
#pragma unroll
            for (int db = 0; db < DB; ++db) t1[db] = rd_tr(cur.off, 1, db);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int db = 0; db < DB; ++db) acc[db] = mfma_bf16(t0[db], xb[0], acc[db]);
#pragma unroll
            for (int ks = 0; ks < KSTEPS / 2; ++ks) a0[ks] = rd_row(rbase, ks);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int db = 0; db < DB; ++db) acc[db] = mfma_bf16(t1[db], xb[1], acc[db]);
#pragma unroll
            for (int ks = 0; ks < KSTEPS / 2; ++ks) a1[ks] = rd_row(rbase, ks + KSTEPS / 2);
            __builtin_amdgcn_sched_barrier(0);
            zero(x);
#pragma unroll
            for (int ks = 0; ks < KSTEPS / 2; ++ks) x = mfma_bf16(a0[ks], breg[ks], x);
#pragma unroll
            for (int ks = 0; ks < KSTEPS / 2; ++ks) x = mfma_bf16(a1[ks], breg[ks + KSTEPS / 2], x);
            __builtin_amdgcn_sched_barrier(0);
        };
        // xn += T1(nxt) B (fragments a0, a1 already requested; xn comes in holding -D of the block's rows,
        // so that it leaves as dP - D), then acc += T2^T(cur) x_b(cur)   (dS-wave order)
        auto gemm1_then_gemm2 = [&](const Blk &nxt, const bf16x8 (&a0)[KSTEPS / 2], const bf16x8 (&a1)[KSTEPS / 2],
                                    f32x16 &xn, const Blk &cur, const bf16x8 (&xb)[2]) __attribute__((always_inline)) {
            bf16x8 t0[DB], t1[DB];
#pragma unroll
            for (int ks = 0; ks < KSTEPS / 2; ++ks) xn = mfma_bf16(a0[ks], breg[ks], xn);
#pragma unroll
            for (int db = 0; db < DB; ++db) t0[db] = rd_tr(cur.off, 0, db);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 0; ks < KSTEPS / 2; ++ks) xn = mfma_bf16(a1[ks], breg[ks + KSTEPS / 2], xn);
#pragma unroll
            for (int db = 0; db < DB; ++db) t1[db] = rd_tr(cur.off, 1, db);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int db = 0; db < DB; ++db) acc[db] = mfma_bf16(t0[db], xb[0], acc[db]);
#pragma unroll
            for (int db = 0; db < DB; ++db) acc[db] = mfma_bf16(t1[db], xb[1], acc[db]);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto read_rows_halves = [&](const Blk &k, bf16x8 (&a0)[KSTEPS / 2], bf16x8 (&a1)[KSTEPS / 2]) __attribute__((always_inline)) {
            const uint32_t rbase = t1_base + k.off;
#pragma unroll
            for (int ks = 0; ks < KSTEPS / 2; ++ks) {
                a0[ks] = rd_row(rbase, ks);
                a1[ks] = rd_row(rbase, ks + KSTEPS / 2);
            }
        };
        auto gemm1 = [&](const bf16x8 (&afr)[KSTEPS], f32x16 &x) {  // x += T1 B
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks) x = mfma_bf16(afr[ks], breg[ks], x);
        };
        auto gemm2 = [&](const bf16x8 (&tfr)[2][DB], const bf16x8 (&xb)[2]) {
#pragma unroll
            for (int stp = 0; stp < 2; ++stp)
#pragma unroll
                for (int db = 0; db < DB; ++db) acc[db] = mfma_bf16(tfr[stp][db], xb[stp], acc[db]);
        };
        // the sixteen per-row values (LSE*log2e or D) of the block's rows held by this lane
        auto read_rowvals = [&](const Blk &k, f32x16 &rv) __attribute__((always_inline)) {
            const float *rowval = &lds.row_s[role == 0 ? 0 : 1][0][0][0] + k.rv;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int base = 16 * half + 8 * hh;
                const float4 l0 = *reinterpret_cast<const float4 *>(rowval + base);
                const float4 l1 = *reinterpret_cast<const float4 *>(rowval + base + 4);
                rv[8 * half + 0] = l0.x, rv[8 * half + 1] = l0.y, rv[8 * half + 2] = l0.z, rv[8 * half + 3] = l0.w;
                rv[8 * half + 4] = l1.x, rv[8 * half + 5] = l1.y, rv[8 * half + 6] = l1.z, rv[8 * half + 7] = l1.w;
            }
        };
        // P-wave: P = exp2(S*scale*log2e - LSE*log2e), zero where masked, rounded to bf16 (the form its
        // own second contraction needs) and handed to the dS-wave in that form
        auto softmax_and_publish = [&](const Blk &k, f32x16 &x, bf16x8 (&xb)[2]) __attribute__((always_inline)) {
            f32x16 ls;
            read_rowvals(k, ls);
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = __builtin_amdgcn_exp2f(fmaf(x[i], sl2, -ls[i]));
            if (!k.full) {
                const int rel = k.r0 + 8 * hh - lo_m;  // row of element i, relative to lo: rel + 16*(i/8) + i%8
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    bool vis = (uint32_t)(rel + (16 * (i >> 3) + (i & 7))) <= span_m;
                    if constexpr (HW) vis = vis && (k.r0 + 16 * (i >> 3) + 8 * hh + (i & 7) + k.dlt <= hi2);
                    x[i] = vis ? x[i] : 0.f;
                }
            }
            xb[0] = pack_bf16x8(x, 0);
            xb[1] = pack_bf16x8(x, 8);
            *reinterpret_cast<bf16x8 *>(&Pex[kbw][k.ps][0][lane * 8]) = xb[0];
            *reinterpret_cast<bf16x8 *>(&Pex[kbw][k.ps][1][lane * 8]) = xb[1];
        };
        // dS-wave: dS = P (dP - D); x holds dP - D (the accumulator started from -D), the result is
        // rounded to bf16 in the form the second contraction needs
        auto fetch_p = [&](const Blk &k, u32x4 (&pw2)[2]) __attribute__((always_inline)) {
#pragma unroll
            for (int h = 0; h < 2; ++h) pw2[h] = *reinterpret_cast<const u32x4 *>(&Pex[kbw][k.ps][h][lane * 8]);
        };
        auto form_ds = [&](const u32x4 (&pw2)[2], const f32x16 &x, bf16x8 (&xb)[2]) __attribute__((always_inline)) {
            f32x16 ds;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const u32x4 pw = pw2[h];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float p_lo = __uint_as_float(pw[e] << 16), p_hi = __uint_as_float(pw[e] & 0xFFFF0000u);
                    ds[8 * h + 2 * e] = p_lo * x[8 * h + 2 * e];
                    ds[8 * h + 2 * e + 1] = p_hi * x[8 * h + 2 * e + 1];
                }
            }
            xb[0] = pack_bf16x8(ds, 0);
            xb[1] = pack_bf16x8(ds, 8);
        };
        // Barrier after the first contraction (and publication of P) of the step handed out last.  The
        // interval after it reads the blocks of that step (second contraction) and of the next one
        // (first contraction): every wave first waits for its share of the tiles the next step needs,
        // and in that interval the buffers of the tiles below the lowest one still in use are refilled.
        auto block_barrier = [&](auto ROLE) __attribute__((always_inline)) {
            if constexpr (TILE_LOADS[decltype(ROLE)::value] != 0) {
                if (hi_next != hi_landed) {
                    wait_tiles(iss_tt - 1 - hi_next);
                    hi_landed = hi_next;
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            lo_free = lo_cur;
        };
        auto refill = [&]() __attribute__((always_inline)) {
            while (iss_tt < n_tiles && iss_tt - NBUF < lo_free) issue_tile();
            __builtin_amdgcn_sched_barrier(0);
        };

        // start-up: two tiles, the resident rows (requested before them) out of the other half of the ring, and when every
        // wave has those, the rest of the ring.  Step 0 needs tile 0 only.
        while (iss_tt < n_tiles && iss_tt < 2) issue_tile();
        wait_tiles(iss_tt);
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks)
            breg[ks] = lds_read_b128_at(row_lds + lds_off_a<kSwzRow, D>(kj, 2 * ks + hh));
        wait_tiles(iss_tt - 1);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        while (iss_tt < n_tiles && iss_tt < NBUF) issue_tile();

        // ---- software pipeline over the steps.  Between the barriers of steps s and s+1 a wave runs
        // the second contraction of its block of step s and the first of its block of step s+1, with
        // the LDS operands of both requested up front; the P-wave puts its softmax arithmetic last (it
        // overlaps the other wave's MFMAs on the same SIMD), the dS-wave puts its arithmetic first.
        // A wave also runs the blocks of a far piece or of its head in which its keys see no query
        // (their P is zero through the mask): the waves meet at a barrier per step anyway, and a loop
        // body without alternatives keeps the accumulators in place.
        auto pipeline = [&](auto ROLE) {
            constexpr int R = ROLE;
            f32x16 x, y;  // P-wave: scores (x only); dS-wave: dP - D of the current and of the next block, in turn
            bf16x8 xb[2];
            Blk cur = next_block();
            {
                bf16x8 afr[KSTEPS];
                read_rows(cur, afr);
                if constexpr (R == 0)
                    zero(x);
                else
                    read_rowvals(cur, x);
                gemm1(afr, x);
                if constexpr (R == 0) softmax_and_publish(cur, x, xb);
            }
            block_barrier(ROLE);
            // one step of the dS-wave: xc holds dP - D of block cur, xn receives that of block nxt
            auto ds_step = [&](f32x16 &xc, f32x16 &xn) __attribute__((always_inline)) {
                const Blk nxt = next_block();
                bf16x8 a0[KSTEPS / 2], a1[KSTEPS / 2];
                // LDS reads return in the order they were requested, and behind the barrier all waves request theirs: P first,
                // because the dS arithmetic needs nothing else (last: dK/dV 216 us instead of 212 at 32/8 heads, d = 128,
                // L = 8192, 28/4 heads, 3 x L = 3077 153 instead of 150; at d = 64, with half the reads, level or slower)
                u32x4 pw[2];
                if constexpr (D == 128) {
                    fetch_p(cur, pw);
                    __builtin_amdgcn_sched_barrier(0);
                }
                read_rows_halves(nxt, a0, a1);  // in flight during the dS arithmetic
                read_rowvals(nxt, xn);
                if constexpr (D == 128) __builtin_amdgcn_sched_barrier(0);
                else fetch_p(cur, pw);
                form_ds(pw, xc, xb);
                __builtin_amdgcn_sched_barrier(0);
                gemm1_then_gemm2(nxt, a0, a1, xn, cur, xb);
                refill();
                block_barrier(ROLE);
                cur = nxt;
            };
            if constexpr (R == 0) {
                for (int gb = 0; gb + 1 < n_blocks; ++gb) {
                    const Blk nxt = next_block();
                    gemm2_then_gemm1(cur, xb, nxt, x);
                    refill();
                    softmax_and_publish(nxt, x, xb);
                    block_barrier(ROLE);
                    cur = nxt;
                }
            } else {
                // two steps per trip, so that the two accumulators swap roles without copies
                int gb = 0;
                for (; gb + 2 < n_blocks; gb += 2) {
                    ds_step(x, y);
                    ds_step(y, x);
                }
                if (gb + 1 < n_blocks) {
                    ds_step(x, y);
                    x = y;
                }
            }
            {
                bf16x8 tfr[2][DB];
                read_transposed(cur, tfr);
                if constexpr (R == 1) {
                    u32x4 pw[2];
                    fetch_p(cur, pw);
                    form_ds(pw, x, xb);
                }
                gemm2(tfr, xb);
            }
        };
        if (role == 0)
            pipeline(IntC<0>{});
        else
            pipeline(IntC<1>{});

        // ---- epilogue: the P-wave owns dV, the dS-wave owns dK (times scale).  A far piece writes its
        // partial (slot w + ft, row = entry within the list tile); a band unit finishes keys that are
        // not on the far list and writes the band partial (one row per list entry, after the slots)
        // of those that are.
        // The sums go through LDS (the ring, 32 fp32 rows per wave, chunks of 16 bytes permuted by the row) and leave as whole
        // rows: stored as they lie in the accumulators, an instruction is 64 scattered pieces of 16 bytes, which took 3400 to
        // 9400 cycles a piece and held up the next piece's loads behind them.  dK/dV in us, scattered / whole rows: 32/8 heads,
        // d = 128, n = 256, L = 8192 212 / 206, 28/4 heads, 3 x L = 3077 133.4 / 131.2, 8 x 12/12 heads, L = 2048, d = 64 59.6 / 55.8.
        const float oscale = role == 0 ? 1.f : p.scale;
        float *farX = role == 0 ? farV : farK;
        uint16_t *outX = role == 0 ? dV : dK;
        int f = -1;  // entry of the far list whose band partial this key's row is
        if (!FAR && !PARTS && valid) {
            f = far_index(fl, prefix, j);
            if (f >= 0 && far_first_query(fl, f, idx, p, BK) >= far_last_query(fl, f, idx, p, dend, BK)) f = -1;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        {
            constexpr int RCH = D / 4, RPI = 64 / RCH;  // chunks of a row, rows per instruction
            const uint32_t stage = q_base + wave * (32 * D * 4);
            int ln = lane;
            asm volatile("" : "+v"(ln));  // the addresses are formed here, not kept through the loop above
            const uint32_t to = stage + (ln & 31) * (D * 4) + (((ln >> 5) ^ (ln & 31 & (RCH - 1))) * 16);
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4)
                    lds_write_b128_at(to ^ ((db * 8 + 2 * i4) * 16), f32x4{acc[db][4 * i4] * oscale, acc[db][4 * i4 + 1] * oscale,
                                                                           acc[db][4 * i4 + 2] * oscale, acc[db][4 * i4 + 3] * oscale});
            if (FAR || PARTS) {
                // whole slots: rows of no key are written with them and read by nobody
                const uint32_t from = stage + ln / RCH * (D * 4) + ((ln % RCH ^ ln / RCH) * 16);  // row ln / RCH
                float *dst = farX + (part0 + (FAR ? (long)(w_id + ft) * BK : ((long)fg.NP + unit) * BK) + 32 * kbw) * D + 4 * ln;
#pragma unroll
                for (int it = 0; it < 32 / RPI; ++it)
                    *reinterpret_cast<f32x4 *>(dst + it * 256) = lds_read_f32x4_at((from ^ (RPI * it % RCH * 16)) + it * 1024);
            } else {
                // all rows but those of keys on the list (and past the end) as bf16, eight columns a lane
                constexpr int RB = 512 / D;  // rows per instruction
                const int sub = ln / (D / 8), c = ln % (D / 8);
                const uint32_t from = stage + sub * (D * 4) + ((2 * c ^ sub) * 16);
                uint16_t *dst = outX + (kvrow0 + unit * BK + 32 * kbw) * D + 8 * ln;
                const uint32_t listed = (uint32_t)__ballot(f >= 0), own = (uint32_t)__ballot(valid && f < 0) >> sub;
#pragma unroll
                for (int it = 0; it < 32 / RB; ++it) {
                    const uint32_t at = (from ^ (RB * it % RCH * 16)) + it * (RB * D * 4);
                    const f32x4 x = lds_read_f32x4_at(at), y = lds_read_f32x4_at(at ^ 16);
                    if ((own >> (RB * it)) & 1) {
                        const uint2 u = pack_bf16x4(x[0], x[1], x[2], x[3]), v = pack_bf16x4(y[0], y[1], y[2], y[3]);
                        *reinterpret_cast<uint4 *>(dst + it * 512) = uint4{u.x, u.y, v.x, v.y};
                    }
                }
                for (uint32_t m = listed; m; m &= m - 1) {
                    const int r = __ffs(m) - 1;
                    float *row = farX + (part0 + (long)fg.NP * BK + __builtin_amdgcn_readlane(f, r)) * D;
                    if (ln < RCH) *reinterpret_cast<f32x4 *>(row + 4 * ln) = lds_read_f32x4_at(stage + r * (D * 4) + ((ln ^ (r % RCH)) * 16));
                }
            }
        }
    }  // pieces
}

}  // namespace

}  // namespace sepattn
