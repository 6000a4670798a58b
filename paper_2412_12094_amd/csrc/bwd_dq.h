// dQ (bf16 MFMA): the work of a workgroup, for the kernel that does nothing else (bwd_bf16.hip) and for the one that runs it beside
// dK/dV (bwd_joint.h).
#pragma once

#include "bwd_common.h"
#include "mfma_common.h"
#include "key_stream.h"
#include "work_share.h"

namespace sepattn {

namespace {

__device__ inline float bf16_dot8(u32x4 a, u32x4 b) {
    float s = 0.f;
    const uint32_t *x = reinterpret_cast<const uint32_t *>(&a);
    const uint32_t *y = reinterpret_cast<const uint32_t *>(&b);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        s = fmaf(__uint_as_float(x[k] << 16), __uint_as_float(y[k] << 16), s);
        s = fmaf(__uint_as_float(x[k] & 0xFFFF0000u), __uint_as_float(y[k] & 0xFFFF0000u), s);
    }
    return s;
}

// ---------------------------------------------------------------------------------------------
// dQ
//
// Same workgroup shapes, key stream and load scheme as the forward (fwd_bf16.hip): every wave has 32 query rows (one
// head, 32 positions) whose Q and dO rows stay in registers as B operands; K/V tiles of 64 stream elements
// pass through LDS.  Per block of 32 keys a wave runs
//     S^T = K Q^T,  dP^T = V dO^T   (2 D/16 matrix instructions, operands row-major from LDS)
//     dS = exp2(S*scale*log2e - LSE*log2e) * (dP - D), masked pairs zero, rounded to bf16
//     dQ^T += K^T dS^T              (2 D/32 matrix instructions, K read transposed from the same tile)
// A tile is four straight runs of matrix instructions,
//     S, dP of block 0 | S, dP of block 1 | dQ update of block 0 | dQ update of block 1,
// with the dS arithmetic of block 0 issued between the matrix instructions of the second run and that of block 1
// between those of the third (a fixed share after each, held there by scheduling fences), so that it executes
// while the matrix pipe is busy; the row loads ride on the first run.  Nothing is carried from one tile to the
// next, so two stages of K and V (AH = 1) are enough for four waves and two workgroups share a compute unit
// (three at d = 64, with 168 registers, spill: 65 us against 50 at 12 heads, 8 x L=2048).  K and V tiles are stored
// with the XOR permutation that serves row-major and transposed reads.
// Bounds: the matrix pipe and issue slots on long streams, the start of a workgroup and of a segment on short ones.
// Measured (us; before: dS between two runs with nothing beside it, eight waves at d = 128, one head per tile for
// seven, loads and their index work on four waves): 32/8 heads, d = 128, L = 8192, n = 256 171 -> 158, packed from eight
// documents 137 -> 124; 28/4 heads, 3 x L=3077 173 -> 127; 8/2 heads, L = 600 19 -> 14; 12 heads, d = 64, 8 x L=2048 54.6 -> 51;
// every fourth KV head full at L = 4096 170 -> 133.  Since then (K and V tiles interleaved with shared operand addresses, nothing in
// scratch memory, waves that end with their own stream, split streams), in the same order: 158 -> 131, 124 -> 102, 127 -> 104,
// 14 -> 12, 51 -> 44, 133 -> 96 + 6.
// ---------------------------------------------------------------------------------------------
// DOCS: packed documents, as in the forward kernel (doc_start / doc_end [B, L]; p.a == 0).
// PARTS: streams of windows of part_keys and more keys go in two parts (split_tiles), whose sums go to `parts`
// [group][split tile][part][wave][32 D].
// HW: head-wise windows.
// ROWS: -D and LSE*log2e are there already (row_values_kernel); otherwise they are formed and written here.
// block: number of the group (head-wise windows: of the workgroup); rank0: of the workgroup within its group.
template <int D, int NW, bool DOCS>
struct DqLds {
    static constexpr int kStages = NW == 4 ? 2 : 4, kMarks = 8;
    alignas(1024) uint16_t KVs[kStages][2][kBN * D];  // K and V rows of a tile, a constant apart
    alignas(256) int lo_s[kMarks][kBN];
    alignas(256) int hi_s[kMarks][kBN];
    alignas(256) uint32_t off_s[4][kBN];           // byte offset of a tile's rows in K and V
    alignas(256) int ent_s[4][DOCS ? 3 : 2][kBN];  // index entries of a tile
    // staging of one 32-column block of a wave's 32 rows (see the start and the end of a segment)
    alignas(16) uint16_t ostage[NW][32 * 32];
};
template <int D, int GP, bool DOCS, int NW, bool PARTS, bool HW, bool ROWS>
__device__ __forceinline__ void dq_work(
    DqLds<D, NW, DOCS> &lds, int block, int rank0, sepattn_params p, const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K,
    const uint16_t *__restrict__ V, const uint16_t *__restrict__ O, const float *__restrict__ LSE,
    const uint16_t *__restrict__ dO, const int32_t *__restrict__ sep_idx,
    const int32_t *__restrict__ sep_prefix, const int32_t *__restrict__ doc_start,
    const int32_t *__restrict__ doc_end, uint16_t *__restrict__ dQ, float *__restrict__ Dws,
    float *__restrict__ Lws, float *__restrict__ parts, int part_keys, int wpg, QueryGrid qg, HeadArgs<HW> ha) {
    constexpr int TP = 32 * NW / GP;
    constexpr bool OWN_END = TP > 32;  // the waves' streams end at different tiles (as in the forward)
    constexpr int CH = D / 8;
    constexpr int RPL = 64 / CH;      // rows covered by one wave-wide 1 KB load
    constexpr int NLD = kBN / RPL;    // wave-wide loads per tensor per tile
    constexpr int LOADS = (NLD + NW - 1) / NW;
    constexpr int KSTEPS = D / 16;
    constexpr int DB = D / 32;
    // tiles the rows are requested ahead, and tiles between two workgroup barriers (as in the forward)
    constexpr int AH = NW == 4 ? 1 : 2;
    constexpr int KST = 2 * AH, MKS = 8;
    constexpr int TILE = kBN * D;

    static_assert(DqLds<D, NW, DOCS>::kStages == KST && DqLds<D, NW, DOCS>::kMarks == MKS, "stages");
    auto &KVs = lds.KVs;
    auto &lo_s = lds.lo_s;
    auto &hi_s = lds.hi_s;
    auto &off_s = lds.off_s;
    auto &ent_s = lds.ent_s;
    auto &ostage = lds.ostage;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qi = lane & 31, hh = lane >> 5;
    // Persistent workgroups as in the forward kernel: a workgroup belongs to one (batch, KV head, head
    // group) and walks through several query tiles of it ("segments") in zig-zag order, `wpg`
    // workgroups per group; rank 0 is the last tile, the one with the longest key stream.
    const int n_pos_tiles = (p.L + TP - 1) / TP;
    int y = block;
    GroupOf at;
    if constexpr (HW) {  // see work_share.h
        const ShareOf s = share_of(ha.share, block, p.B);
        rank0 = s.rank;
        wpg = s.count;
        const int g = ha.share.group[s.pos], k = quotient(g, qg.by_groups);
        at = {g - k * qg.groups, k, s.b};
        y = s.b * p.Hkv * qg.groups + g;
    } else {
        at = group_of(qg, y, p.Hkv);
    }
    const int kv = at.kv, b = at.b, head0 = (kv * qg.groups + at.hg) * GP;
    const int head = head0 + (wave % GP);
    const int gdelta = ha.of_group(head0, GP);  // head-wise windows: see the forward kernel
    p.n -= gdelta;
    const int hdelta = ha.of_head(head) - gdelta;

    const int32_t *prefix = sep_prefix + (long)b * (p.L + 1);
    const int32_t *idx = sep_idx + (long)b * p.cap;
    const int32_t *dstart = DOCS ? doc_start + (long)b * p.L : nullptr;
    const int32_t *dend = DOCS ? doc_end + (long)b * p.L : nullptr;

    // state of the segment being multiplied (the lambdas below refer to it)
    int iq = 0, iq_h = 0;
    FullBlocks fullb = {};
    bf16x8 qreg[KSTEPS], doreg[KSTEPS];
    float Di = 0.f, neg_lse2 = 0.f;
    const float sl2 = p.scale * kLog2e_f;
    f32x16 acc[DB];

    // ---- segments and the look-ahead over the concatenation of their tiles, as in the forward kernel: what a tile
    // holds is worked out four tiles ahead of the multiplications by wave 0 (even tiles) and wave 1 (odd
    // tiles; tiles 0 .. 3 by the first four waves), one row per lane, from index entries requested two tiles before.  Past the last segment the stream
    // is empty: its tiles are "loaded" too (row 0, never visible).
    struct Seg {
        Stream st;
        int t0, n_tiles, i0, de;  // tiles t0 .. n_tiles-1 of the stream
        int slot;                 // where the sums of a part go, -1: not a part
    };
    const SplitTiles split = split_tiles(n_pos_tiles, TP, p.n, PARTS ? part_keys : 0);  // of this group (its p.n)
    auto rank_of = [&](int round) { return round * wpg + ((round & 1) ? wpg - 1 - rank0 : rank0); };
    const int n_pieces = n_pos_tiles + split.n;
    auto segment_at = [&](int rank) {  // rank < n_pieces; no branches, as in the forward
        Seg g;
        int tile = rank, part = -1;
        if constexpr (PARTS) split.find(rank, tile, part);
        g.i0 = (n_pos_tiles - 1 - tile) * TP;
        if constexpr (DOCS) {
            // the clamps keep inconsistent bounds (caller error) from faulting
            const int ds = min(max(load_uniform(dstart, g.i0), 0), g.i0);
            g.de = min(max(load_uniform(dend, g.i0), g.i0 + 1), p.L);
            g.st = make_stream_docs(p, prefix, g.i0, TP, ds);
        } else {
            g.de = kIntMax;
            g.st = make_stream(p, prefix, g.i0, TP);
        }
        g.n_tiles = (g.st.n_total + kBN - 1) / kBN;
        g.t0 = 0;
        g.slot = -1;
        if (PARTS && part >= 0) {
            g.slot = (y * split.most + tile) * 2 + part;
            if (part) g.t0 = g.n_tiles / 2;
            else g.n_tiles /= 2;
        }
        return g;
    };
    auto past_the_last = []() { return Seg{Stream{0, 0, 0, 0, 0}, 0, kIntMax, -1, kIntMax, -1}; };
    auto open_segment = [&](int round) {
        const int rank = rank_of(round);
        return rank >= n_pieces ? past_the_last() : segment_at(rank);
    };
    struct Cursor {
        Seg cur, next;
        int round, t;  // segment of this workgroup and tile of its stream
    };
    auto advance = [&](Cursor &c) __attribute__((always_inline)) {
        if (++c.t == c.cur.n_tiles) {
            c.cur = c.next;
            ++c.round;
            c.t = PARTS ? c.cur.t0 : 0;
            c.next = open_segment(c.round + 1);
        }
    };
    // where a lane's entries of tile t of stream ss stand
    struct EntryAt {
        const int32_t *of_row, *behind, *doc_end;
    };
    auto entry_at = [&](const Stream &ss, int t) __attribute__((always_inline)) {
        const int k = t * kBN + lane;
        const int e = min(max(ss.sep_lo - ss.n_init + k, 0), p.cap - 1);
        const int j = min(max(ss.bs - ss.n_dense + k, 0), p.L - 1);
        return EntryAt{k < ss.n_dense ? idx + e : prefix + j, prefix + j + 1, DOCS ? dend + j : nullptr};
    };
    // entries of tile t (global number g) of stream ss
    auto issue_entries = [&](const Stream &ss, int t, int g) __attribute__((always_inline)) {
        const EntryAt at = entry_at(ss, t);
        const uint32_t dst = lds_addr(&ent_s[g & 3][0][0]);
        dma_to_lds_4_addr(at.of_row, dst);
        dma_to_lds_4_addr(at.behind, dst + kBN * 4);
        if constexpr (DOCS) dma_to_lds_4_addr(at.doc_end, dst + 2 * kBN * 4);  // where the key's document ends
    };
    auto write_entries = [&](const Cursor &c, int g, int e0, int e1, int doc_end) __attribute__((always_inline)) {
        const Stream &ss = c.cur.st;
        const int k = c.t * kBN + lane;
        const bool dense = k < ss.n_dense, pad = k >= ss.n_total;
        const int jb = ss.bs + (k - ss.n_dense);
        // the clamp keeps a stale list tail (caller broke sep_count <= cap) from faulting
        int j = dense ? min(max(e0, 0), p.L - 1) : jb;
        j = k < ss.n_init ? k : j;
        int hi = (dense | (jb < p.a) | (e1 != e0)) ? kIntMax : jb + p.n - 1;
        if constexpr (DOCS) hi = min(hi, (dense ? c.cur.de : doc_end) - 1);
        lo_s[g % MKS][lane] = pad ? kIntMax : j;
        hi_s[g % MKS][lane] = pad ? -1 : hi;
        off_s[g & 3][lane] = pad ? 0u : (uint32_t)j * (uint32_t)(D * 2);
    };
    auto write_rows = [&](const Cursor &c, int g) __attribute__((always_inline)) {
        write_entries(c, g, ent_s[g & 3][0][lane], ent_s[g & 3][1][lane], DOCS ? ent_s[g & 3][DOCS ? 2 : 0][lane] : 0);
    };
    // start of tile step g: positions of a tile four further on, entries of one six further on (AH = 2: of two
    // tiles every other step)
    Cursor lc;
    auto look_ahead = [&](int g) __attribute__((always_inline)) {
        if (AH == 1 ? wave == (g & 1) : ((g & 1) == 0 && wave < 2)) {
            const int t = g + (AH == 1 ? 0 : wave);
            write_rows(lc, t + 4);
            advance(lc);
            advance(lc);
            issue_entries(lc.cur.st, lc.t, t + 6);
        }
    };

    // ---- row loads: load n of a tile fills rows n*RPL .. +RPL-1 with one wave-wide direct global->LDS load per
    // tensor; wave w issues loads LOADS*w + u (the last one again where the waves do not divide the tile)
    const char *Kb = reinterpret_cast<const char *>(K + ((long)b * p.Hkv + kv) * (long)p.L * D);
    const char *Vb = reinterpret_cast<const char *>(V + ((long)b * p.Hkv + kv) * (long)p.L * D);
    const int my_pc = lane % CH, my_sub = lane / CH;
    const uint32_t kv_base = lds_addr(&KVs[0][0][0]);
    uint32_t gofs[LOADS];  // byte offset of this lane's piece of the rows it helps to fill next
    auto read_offsets = [&](int g) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            const int r = min(LOADS * wave + u, NLD - 1) * RPL + my_sub;
            gofs[u] = off_s[g & 3][r] + swz_chunk<kSwzBoth, D>(my_pc, r) * 16;
        }
    };
    auto issue_row = [&](int g, auto N) __attribute__((always_inline)) {  // the K (even n) or V (odd n) rows of load n / 2
        constexpr int n = decltype(N)::value, u = n / 2;
        const uint32_t at = kv_base + (unsigned)(g % KST) * (TILE * 4) + (uint32_t)min(LOADS * wave + u, NLD - 1) * 1024u;
        if constexpr (n % 2 == 0) dma_to_lds_16(Kb, gofs[u], at);
        else dma_to_lds_16(Vb, gofs[u], at + TILE * 2);
    };
    // publishes every load and LDS write of the wave
    auto wg_barrier = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // per-lane byte offsets of the operand fragments inside a tile
    const int a_row = pi_row(qi);
    // Row-major fragments: the XOR permutation acts on the 16-byte chunk index 2*ks + hh, and the
    // k-step only enters through bits 1..3 of it, so fragment ks sits at (fragment 0) ^ (32 * ks):
    // one register instead of KSTEPS.  (Tile bases are multiples of 1 KB, so the XOR commutes with
    // adding the base.)  K and V tiles share one layout and therefore these offsets.
    const uint32_t koff0 = lds_off_a<kSwzBoth, D>(a_row, hh);
    uint32_t ktr0[DB], ktr1[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) {
        ktr0[db] = lds_off_a_tr<kSwzBoth, D>(db * 32, lane);
        ktr1[db] = lds_off_a_tr_second<kSwzBoth, D>(db * 32, lane);
    }
    // for d = 128 the second transposed read is the first with chunk bit 0 flipped, four rows on
    auto tr_second = [&](uint32_t first, int db) __attribute__((always_inline)) {
        if constexpr (D == 128)
            return (first ^ 16u) + 4u * D * 2u;
        else
            return first - ktr0[db] + ktr1[db];
    };

    // ---- one straight run of tile X of the current segment (global number gbase + X).  SP: S and dP of block SP into
    // s_new, p_new; DQ: dQ update with block DQ's keys and ds_old; DS: dS of block DS from s_old, p_old into
    // ds_new (-1: not in this run); LD: the rows of tile X + AH are requested.
    int gbase = 0;
    constexpr int LA = 4;
    // d = 64 has the registers to start every dP accumulator from -D: no subtraction per element
    constexpr bool FROM_D = D == 64;
    f32x16 d_start;
    auto run = [&](int X, auto SP_, auto DQ_, auto DS_, auto LD_, f32x16 &s_new, f32x16 &p_new, const bf16x8 (&ds_old)[2],
                   f32x16 &s_old, f32x16 &p_old, bf16x8 (&ds_new)[2]) __attribute__((always_inline)) {
        constexpr int SP = decltype(SP_)::value, DQ = decltype(DQ_)::value, DS = decltype(DS_)::value;
        constexpr bool DO_LD = decltype(LD_)::value != 0;
        constexpr int NS = SP >= 0 ? 2 * KSTEPS : (DQ >= 0 ? 2 * DB : 0);
        static_assert(SP < 0 || DQ < 0, "one kind of matrix work per run");
        constexpr int E = NS ? 16 / (NS ? NS : 1) : 16;  // elements of dS per matrix instruction
        // Block and matrix (K or V) are added after the XOR: they become the instructions' offsets, and a K and a V fragment, or
        // those of both blocks, share an address.
        const uint32_t stage = kv_base + (unsigned)(gbase + X) % KST * (TILE * 4);
        constexpr uint32_t BO = (SP >= 0 ? SP : (DQ >= 0 ? DQ : 0)) * 32 * D * 2;
        bf16x8 frag[LA];
        auto request = [&](auto S) __attribute__((always_inline)) {
            constexpr int s = decltype(S)::value;
            if constexpr (s < NS) {
                if constexpr (SP >= 0) {
                    frag[s % LA] = lds_read_b128_at(((stage + koff0) ^ (32u * (s / 2))) + (BO + (s % 2) * TILE * 2));
                } else {
                    constexpr int stp = s / DB, db = s % DB;
                    frag[s % LA] = lds_read_tr_at2(stage + ktr0[db] + (BO + stp * 16 * D * 2),
                                                   tr_second(stage + ktr0[db], db) + (BO + stp * 16 * D * 2));
                }
            }
        };
        static_for<LA>([&](auto S) { request(S); });
        if constexpr (DS >= 0) {
            if (!block_is_full(fullb, X * kBN + DS * 32)) {
                const int ms_ = (unsigned)(gbase + X) % MKS;
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    const int base = DS * 32 + 16 * half + 8 * hh;
                    const int4 lo0 = *reinterpret_cast<const int4 *>(&lo_s[ms_][base]);
                    const int4 lo1 = *reinterpret_cast<const int4 *>(&lo_s[ms_][base + 4]);
                    const int4 hi0 = *reinterpret_cast<const int4 *>(&hi_s[ms_][base]);
                    const int4 hi1 = *reinterpret_cast<const int4 *>(&hi_s[ms_][base + 4]);
                    const int los[8] = {lo0.x, lo0.y, lo0.z, lo0.w, lo1.x, lo1.y, lo1.z, lo1.w};
                    const int his[8] = {hi0.x, hi0.y, hi0.z, hi0.w, hi1.x, hi1.y, hi1.z, hi1.w};
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const bool vis = (los[k] <= iq) & (iq_h <= his[k]);
                        s_old[8 * half + k] = vis ? s_old[8 * half + k] : -INFINITY;
                    }
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // elements e0 .. e0+E-1 get their exponentials in a slot, and their factor dP - D in the next one, when the
        // transcendental unit has delivered
        auto exps = [&](int e0) __attribute__((always_inline)) {
#pragma unroll
            for (int i = e0; i < e0 + E; ++i)
                if (i < 16) s_old[i] = __builtin_amdgcn_exp2f(fmaf(s_old[i], sl2, neg_lse2));
        };
        auto products = [&](int e0) __attribute__((always_inline)) {
#pragma unroll
            for (int i = e0; i < e0 + E; ++i)
                if (i >= 0 && i < 16) s_old[i] *= FROM_D ? p_old[i] : p_old[i] - Di;
        };
        static_for<NS>([&](auto S) {
            constexpr int s = decltype(S)::value;
            if constexpr (SP >= 0) {
                const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                if constexpr (s % 2 == 0) s_new = mfma_bf16(frag[s % LA], qreg[s / 2], s == 0 ? zero : s_new);
                else p_new = mfma_bf16(frag[s % LA], doreg[s / 2], s == 1 ? (FROM_D ? d_start : zero) : p_new);
            } else {
                acc[s % DB] = mfma_bf16(frag[s % LA], ds_old[s / DB], acc[s % DB]);
            }
            request(IntC<s + LA>{});
            if constexpr (DS >= 0) {
                constexpr int e0 = E * s;
                exps(e0);
                products(e0 - E);
                if constexpr (e0 - E < 8 && e0 >= 8) ds_new[0] = pack_bf16x8(s_old, 0);
            }
            if constexpr (DO_LD && s >= 1) {
                constexpr int LPS = (2 * LOADS + NS - 2) / (NS - 1);  // row loads per slot
                static_for<LPS>([&](auto J) {
                    constexpr int n = (s - 1) * LPS + decltype(J)::value;
                    if constexpr (n < 2 * LOADS) issue_row(gbase + X + AH, IntC<n>{});
                });
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (DS >= 0) {
            if constexpr (NS == 0) exps(0);
            products(16 - E);
            if constexpr (E > 8) ds_new[0] = pack_bf16x8(s_old, 0);
            ds_new[1] = pack_bf16x8(s_old, 8);
            u32x4 &x0 = reinterpret_cast<u32x4 &>(ds_new[0]), &x1 = reinterpret_cast<u32x4 &>(ds_new[1]);
            asm volatile("" : "+v"(x0), "+v"(x1));
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    const IntC<0> first, off;
    const IntC<1> second, on;
    const IntC<-1> none;
    // The wave's 32 rows of Q, dO and O of a segment.  The operand layout wants, per lane, 16-byte pieces
    // of ONE row; fetched that way every load instruction is 64 scattered pieces, and their number (1536
    // per wave and segment) is what such loads cost.  They are fetched instead so that four consecutive
    // lanes cover 64 contiguous bytes of a row (column block cb of 32 columns, rows 16 t + lane / 4,
    // piece lane % 4), and they are requested one segment ahead, before the previous segment's dQ rows
    // are stored, so that the store path hides their latency.  (Past the last segment: row 0, unused.)
    constexpr int CB = D / 32;  // column blocks of 32 columns (64 bytes of a row)
    const long head_row0 = ((long)b * p.Hq + head) * p.L;  // rows of this wave's head
    u32x4 q4[CB][2], do4[CB][2], o4[ROWS ? 1 : CB][2];
    float row_d = 0.f;  // ROWS: -D of the lane's row
    // What the start and the end of a segment derive from the lane's number is worked out anew each time: kept over the loop
    // between them, where no register is free, it went to scratch memory.
    auto lane_anew = [&]() __attribute__((always_inline)) {
        int l = lane;
        asm volatile("" : "+v"(l));
        return l;
    };
    auto fetch_rows = [&](const Seg &sg) __attribute__((always_inline)) {
        const int lane = lane_anew();
        const char *qb = reinterpret_cast<const char *>(Q + head_row0 * D);
        const char *dob = reinterpret_cast<const char *>(dO + head_row0 * D);
        const char *ob = reinterpret_cast<const char *>(O + head_row0 * D);
        const int pwn = max(sg.i0, 0) + 32 * (wave / GP);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const uint32_t roff = (uint32_t)min(pwn + 16 * t + (lane >> 2), p.L - 1) * (uint32_t)(D * 2) + 16u * (lane & 3);
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                q4[cb][t] = *reinterpret_cast<const u32x4 *>(qb + (roff + 64u * cb));
                do4[cb][t] = *reinterpret_cast<const u32x4 *>(dob + (roff + 64u * cb));
                if constexpr (!ROWS) o4[cb][t] = *reinterpret_cast<const u32x4 *>(ob + (roff + 64u * cb));
            }
        }
        if constexpr (ROWS) row_d = Dws[head_row0 + min(pwn + (lane & 31), p.L - 1)];
    };
    // ---- start-up, once per workgroup, as in the forward: positions of tiles 0 .. 3, a wave each, then the first rows (the entries
    // of tiles 4 and 5 are on their way).  The first segment's rows of Q, dO and O are requested behind the entries,
    // which alone are waited for (they come into registers: the compiler counts the loads that it has placed behind them).
    Seg cseg = segment_at(rank0);
    {
        Seg next = segment_at(min(rank_of(1), n_pieces - 1));
        if (rank_of(1) >= n_pieces) next = past_the_last();
        lc = {cseg, next, 0, cseg.t0};
    }
    int e0 = 0, e1 = 0, e_doc = 0;
    if (wave < 4) {
        for (int t = 0; t < wave; ++t) advance(lc);
        const EntryAt at = entry_at(lc.cur.st, lc.t);
        e0 = *at.of_row, e1 = *at.behind;
        if constexpr (DOCS) e_doc = *at.doc_end;
    }
    __builtin_amdgcn_sched_barrier(0);
    fetch_rows(cseg);
    __builtin_amdgcn_sched_barrier(0);
    if (wave < 4) {
        const Cursor own = lc;
        if (wave < 2)
            for (int t = 0; t < 4; ++t) advance(lc);
        asm volatile("" : "+v"(e0), "+v"(e1), "+v"(e_doc));  // looked at from here on
        write_entries(own, wave, e0, e1, e_doc);
        if (wave < 2) issue_entries(lc.cur.st, lc.t, 4 + wave);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // only what write_rows wrote is published here
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    static_for<AH>([&](auto T) {
        read_offsets(decltype(T)::value);
        static_for<2 * LOADS>([&](auto N) { issue_row(decltype(T)::value, N); });
    });
    for (int round = 0; cseg.i0 >= 0; ++round) {
        const int pw = cseg.i0 + 32 * (wave / GP);
        iq = pw + qi;
        iq_h = iq + hdelta;
        fullb = full_blocks(cseg.st, pw, p.n - hdelta);
        if (DOCS && pw + 31 >= cseg.de) fullb = no_full_blocks();
        {
            const int lane = lane_anew(), qi = lane & 31, hh = lane >> 5;
            // Q and dO reach their operand layout through the wave's 2 KB staging area, one column block
            // at a time (16-byte piece c of row r at piece position c ^ ((r / 4) % 4); the LDS operations
            // of a wave execute in order).  D_i = sum_k dO_ik O_ik needs no particular layout: partial
            // sums per lane, then over the four lanes of a row, then handed to the lane pair that owns
            // the row.
            if constexpr (ROWS) {
                Di = -row_d;
            } else {
                float part[2] = {0.f, 0.f};
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) part[t] += bf16_dot8(do4[cb][t], o4[cb][t]);
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    part[t] += __shfl_xor(part[t], 1);
                    part[t] += __shfl_xor(part[t], 2);
                }
                // row qi is held by the lanes 4 (qi % 16) .. +3 in part[qi / 16]
                const float d0 = __shfl(part[0], 4 * (qi & 15)), d1 = __shfl(part[1], 4 * (qi & 15));
                Di = qi < 16 ? d0 : d1;
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) d_start[i] = -Di;
            uint16_t *stg = &ostage[wave][0];
            const int wr0 = (lane >> 2), wc = lane & 3;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                static_for<2>([&](auto X) {
                    constexpr bool is_q = decltype(X)::value == 0;
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const int r = 16 * t + wr0;
                        *reinterpret_cast<u32x4 *>(stg + r * 32 + ((wc ^ ((r >> 2) & 3)) * 8)) = is_q ? q4[cb][t] : do4[cb][t];
                    }
#pragma unroll
                    for (int k2 = 0; k2 < 2; ++k2) {
                        const u32x4 v = *reinterpret_cast<const u32x4 *>(stg + qi * 32 + (((2 * k2 + hh) ^ ((qi >> 2) & 3)) * 8));
                        if constexpr (is_q) qreg[2 * cb + k2] = as_bf16x8(v);
                        else doreg[2 * cb + k2] = as_bf16x8(v);
                    }
                });
            }
            const uint32_t soff = (uint32_t)min(iq, p.L - 1) * 4u;
            const float lse2 = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(LSE + head_row0) + soff) * kLog2e_f;
            neg_lse2 = -lse2;
            if (!ROWS && hh == 0 && iq < p.L && (!PARTS || cseg.t0 == 0)) {
                // stored negated: the dK/dV kernel starts its dP accumulator from -D
                *reinterpret_cast<float *>(reinterpret_cast<char *>(Dws + head_row0) + soff) = -Di;
                // the dK/dV kernels work in the log2 domain too
                *reinterpret_cast<float *>(reinterpret_cast<char *>(Lws + head_row0) + soff) = lse2;
            }
        }
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[db][i] = 0.f;

        // Step X reads tile gbase+X and requests tile gbase+X+AH, whose stages held tile gbase+X-AH; barriers stand in
        // front of every AH-th tile of the concatenated stream, where everything requested before has landed.  The
        // second block of the wave's last tile is left out when it is all padding or beyond the wave's last position; in
        // tiles beyond that (OWN_END) the wave only takes part in the loads.
        // (A tail after the loop: alternatives inside it would cost a copy of the accumulators per tile.)
        const int t0 = PARTS ? cseg.t0 : 0, n_tiles = cseg.n_tiles;
        gbase -= t0;
        int my_total = OWN_END ? min(cseg.st.n_total, cseg.st.n_dense + pw + 32 - cseg.st.bs) : cseg.st.n_total;
        if constexpr (PARTS) my_total = max(min(my_total, n_tiles * kBN), t0 * kBN);
        const int n_whole = (my_total + 31) / kBN, my_tiles = OWN_END ? (my_total + kBN - 1) / kBN : n_tiles;
        auto begin_tile = [&](int X) __attribute__((always_inline)) {
            if ((gbase + X) % AH == 0) wg_barrier();
            look_ahead(gbase + X);
            read_offsets(gbase + X + AH);
        };
        f32x16 s0, p0, s1, p1;
        bf16x8 ds0[2], ds1[2];
        for (int X = t0; X < n_whole; ++X) {
            begin_tile(X);
            run(X, first, none, none, on, s0, p0, ds0, s0, p0, ds0);
            run(X, second, none, first, off, s1, p1, ds0, s0, p0, ds0);
            run(X, none, first, second, off, s0, p0, ds0, s1, p1, ds1);
            run(X, none, second, none, off, s0, p0, ds1, s1, p1, ds1);
        }
        if (n_whole < my_tiles) {
            begin_tile(n_whole);
            run(n_whole, first, none, none, on, s0, p0, ds0, s0, p0, ds0);
            run(n_whole, none, none, first, off, s1, p1, ds0, s0, p0, ds0);
            run(n_whole, none, first, none, off, s1, p1, ds0, s0, p0, ds0);
        }
        if constexpr (OWN_END) {
            for (int X = my_tiles; X < n_tiles; ++X) {
                begin_tile(X);
                static_for<2 * LOADS>([&](auto N) { issue_row(gbase + X + AH, N); });
            }
        }
        gbase += n_tiles;
        const Seg nseg = open_segment(round + 1);
        fetch_rows(nseg);
        __builtin_amdgcn_sched_barrier(0);

        // A lane holds 4-column pieces of ONE dQ row: stored straight from the accumulators they are 64
        // scattered 8-byte pieces per instruction, and their number is what the stores cost.  Each
        // 32-column block of the wave's 32 rows goes through a 2 KB staging area of the wave instead
        // and leaves as 16-byte pieces of which four consecutive lanes cover 64 contiguous bytes of a
        // row.  8-byte chunk ch of row r sits at chunk position ch ^ (2 * ((r / 4) % 4)); the LDS
        // operations of a wave execute in order, so a block's reads precede the next block's writes.
        if (PARTS && cseg.slot >= 0) {
            // fp32 sums of a part, in the accumulators' own order: every store covers 1 KB
            const int lane = lane_anew();
            float *out = parts + ((long)cseg.slot * NW + wave) * (32 * D) + lane * 4;
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const float4 v = {acc[db][4 * i4] * p.scale, acc[db][4 * i4 + 1] * p.scale,
                                      acc[db][4 * i4 + 2] * p.scale, acc[db][4 * i4 + 3] * p.scale};
                    *reinterpret_cast<float4 *>(out + (db * 4 + i4) * 256) = v;
                }
        } else {
            const int lane = lane_anew(), qi = lane & 31, hh = lane >> 5;
            uint16_t *stg = &ostage[wave][0];
            const int wsw = ((qi >> 2) & 3) << 1;
#pragma unroll
            for (int db = 0; db < DB; ++db) {
#pragma unroll
                for (int i4 = 0; i4 < 4; ++i4) {
                    const uint2 v = pack_bf16x4(acc[db][4 * i4] * p.scale, acc[db][4 * i4 + 1] * p.scale,
                                                acc[db][4 * i4 + 2] * p.scale, acc[db][4 * i4 + 3] * p.scale);
                    *reinterpret_cast<uint2 *>(stg + qi * 32 + (((2 * i4 + hh) ^ wsw) * 4)) = v;
                }
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int r = 16 * t + (lane >> 2), c = lane & 3;
                    const int pos = (2 * c) ^ (((r >> 2) & 3) << 1);
                    const uint4 v = *reinterpret_cast<const uint4 *>(stg + r * 32 + pos * 4);
                    if (pw + r < p.L) *reinterpret_cast<uint4 *>(dQ + (head_row0 + pw + r) * D + db * 32 + c * 8) = v;
                }
                __builtin_amdgcn_sched_barrier(0);  // one block at a time: keeps the register pressure down
            }
        }
        cseg = nseg;
    }
    // the loads of the padding tiles past the last segment must have landed before the workgroup
    // ends and its LDS is handed on
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

}  // namespace

}  // namespace sepattn
