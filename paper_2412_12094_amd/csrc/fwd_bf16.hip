// SepAttention forward, bf16 MFMA (Eq. 1 with the mask of Eq. 2), flash-style with online softmax.
//
// A workgroup (NW waves; see query_shape in key_stream.h) owns
// TP = 32 NW / GP consecutive query positions of GP query heads that share one KV
// head (grouped-query attention: the heads are packed into the row dimension, so K/V tiles and the
// mask are shared).  Each wave owns 32 rows: one head, 32 positions.  The keys a tile can see are
// turned into ONE dense stream,
//     [ initial tokens j < min(a, bs) | separators in [min(a,bs), bs) | band keys bs .. i0+TP-1 ]
// with bs = max(0, i0-n+1) the first key of the first row's neighbour window (Sec. 3.1).  The first
// two parts are visible to every row of the tile (they are older than every window and are initial
// tokens / separators) and are gathered through the compacted separator index list; only band keys
// need the per-element test  j <= i and (i-j < n or j is an initial token or a separator).
//
// Bounds: long streams the matrix pipe and, with it, the power limit (per 64-key tile and SIMD 2048 cycles of
// matrix instructions in about 3500, at 1.9 GHz), short ones also the start of a workgroup and of a segment.
// Tiles are filled by direct global->LDS loads
// (global_load_lds_dwordx4, no staging registers), unpadded with XOR-swizzled
// 16-byte chunks (see mfma_common.h).  V^T operands are read with ds_read_b64_tr_b16.  A wave drops
// the mask test on blocks every one of its rows sees in full.  The running maximum is only raised
// when it grows by more than 2^8 (all terms carry the same stale maximum, so the result is
// unchanged), which removes almost every rescale of the output accumulators; whether it has is seen from
// the exponentials, so that a block's maximum is not formed at all unless they are too large (raise_max).
// Measured (forward call with its index step, us; before: eight waves, vector work outside the shadow of the matrix
// instructions, loads and index work on four of the waves): 32/8 heads, d = 128: L=8192 n=256 109 -> 98, L=64K
// n=1024 3990 -> 3650, 4 x L=1531 n=256 84 -> 75; 28/4 heads, 3 x L=3077 119 -> 78; 12 heads, d = 64, 8 x L=2048 51 -> 40.  The kernel alone (scalar
// loads of a segment's bounds, no maximum per block, operands of a tile's second half requested in its first): 113 -> 94 (L=8192),
// 3625 -> 3385 (64K), 88 -> 76 (3 x 3077), 38 -> 34 (d = 64), 86 -> 76 (8192 packed from eight documents).
// The start of a workgroup (arguments -> bounds of its segments -> index entries -> rows) lasted 6800 cycles in a small call and 14000
// where all compute units start at once; with the tables of head-wise calls left to these, divisions by multiplication, both
// segments' bounds in one round trip and four waves for the first tiles' entries, here and in dQ, a step in us: 8/2 heads, L = 600
// 47.3 -> 45.4, 8 x L = 2048 157 -> 154, 4 prompts of 1531 65.5 -> 62.2.
#include "common.h"
#include "mfma_common.h"
#include "key_stream.h"
#include "work_share.h"

namespace sepattn {

namespace {

constexpr float kRescaleThreshold = 8.f;  // log2 units
constexpr float kMaxTerm = 256.f;         // 2^kRescaleThreshold

// DOCS: packed documents (see make_stream_docs); doc_start / doc_end [B, L] give, per position, the
// first position of its document and one past its last.  Requires p.a == 0.
// NW: waves per workgroup (4, 7 or 8, see query_shape); about two waves per SIMD in all shapes, three at d = 64 with four.
// HW: head-wise windows (see below); the workgroups are dealt to the groups by their work (work_share.h).
template <int D, int GP, bool DOCS, int NW, bool HW>
__global__ __launch_bounds__(64 * NW, D == 64 && NW == 4 ? 3 : 2) void fwd_bf16_kernel(
    sepattn_params p, const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K,
    const uint16_t *__restrict__ V, const int32_t *__restrict__ sep_idx,
    const int32_t *__restrict__ sep_prefix, const int32_t *__restrict__ doc_start,
    const int32_t *__restrict__ doc_end, uint16_t *__restrict__ O, float *__restrict__ LSE, int wpg, QueryGrid qg, HeadArgs<HW> ha) {
    constexpr int TP = 32 * NW / GP;  // query positions per workgroup
    // The waves' streams end at different tiles: a wave that is past its last position leaves the arithmetic of the rest out
    // (12 heads, d = 64, 8 x L = 2048, n = 64, four waves of 32 positions each: forward and backward 170.0 -> 165.1 us, of
    // which the forward 2.6; with TP = 32 there is nothing to leave out, and the code for it is not there).
    constexpr bool OWN_END = TP > 32;
    constexpr int CH = D / 8;         // 16-byte chunks per row
    constexpr int RPL = 64 / CH;      // rows covered by one wave-wide 1 KB load
    constexpr int NLD = kBN / RPL;    // wave-wide loads per tensor per tile
    constexpr int LOADS = (NLD + NW - 1) / NW;  // ... of which each wave issues this many (K and V each)
    constexpr int KSTEPS = D / 16;
    constexpr int DB = D / 32;
    // How many tiles ahead the rows are requested, and tiles between two workgroup barriers (see the
    // pipeline): 1 with four waves, so that two (d = 64: three) workgroups fit a compute unit, else 2.
    constexpr int AH = NW == 4 ? 1 : 2;
    constexpr int KST = 2 * AH, VST = 2 * AH, MKS = 8;
    constexpr int TILE = kBN * D;    // elements per LDS tile (unpadded, XOR-swizzled chunks)

    __shared__ __attribute__((aligned(1024))) uint16_t Ks[KST][TILE];
    __shared__ __attribute__((aligned(1024))) uint16_t Vs[VST][TILE];
    __shared__ __attribute__((aligned(256))) int lo_s[MKS][kBN];
    __shared__ __attribute__((aligned(256))) int hi_s[MKS][kBN];
    __shared__ __attribute__((aligned(256))) uint32_t off_s[4][kBN];  // byte offset of a tile's rows in K and V
    __shared__ __attribute__((aligned(256))) int ent_s[4][DOCS ? 3 : 2][kBN];      // index entries of a tile (see issue_entries)
    // staging of one 32-column block of a wave's 32 output rows (see the epilogue)
    __shared__ __attribute__((aligned(16))) uint16_t ostage[NW][32 * 32];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keeps branches scalar
    const int qi = lane & 31, hh = lane >> 5;
    // A workgroup is persistent: it belongs to one (batch, KV head, head group) and walks through
    // several query tiles of it ("segments"), `wpg` workgroups per group sharing the tiles in zig-zag
    // order (round r: rank r*wpg + j for even r, r*wpg + wpg-1-j for odd r; rank 0 = the last tile,
    // the one with the longest key stream), so that with an even spread of separators every
    // workgroup gets about the same number of stream tiles.  Launch gaps, the tail of a grid of
    // unequal workgroups and most of the per-tile start-up cost are paid once per workgroup.
    const int n_pos_tiles = (p.L + TP - 1) / TP;
    int rank0 = blockIdx.y;
    GroupOf at;
    if constexpr (HW) {
        const ShareOf s = share_of(ha.share, blockIdx.x, p.B);
        rank0 = s.rank;
        wpg = s.count;
        const int g = ha.share.group[s.pos], k = quotient(g, qg.by_groups);
        at = {g - k * qg.groups, k, s.b};
    } else {
        at = group_of(qg, blockIdx.x + qg.gx * blockIdx.z, p.Hkv);
    }
    const int kv = at.kv, b = at.b, head0 = (kv * qg.groups + at.hg) * GP;
    const int head = head0 + (wave % GP);
    // head-wise windows: the stream is that of the largest window of the group's heads (p.n from here on); this
    // head's window is shorter by hdelta, which only enters the visibility test of band keys (hi was computed
    // with p.n) and the decision which blocks need no test
    const int gdelta = ha.of_group(head0, GP);
    p.n -= gdelta;
    const int hdelta = ha.of_head(head) - gdelta;

    const int32_t *prefix = sep_prefix + (long)b * (p.L + 1);
    const int32_t *idx = sep_idx + (long)b * p.cap;
    const int32_t *dstart = DOCS ? doc_start + (long)b * p.L : nullptr;
    const int32_t *dend = DOCS ? doc_end + (long)b * p.L : nullptr;

    // state of the current segment (the lambdas below refer to it)
    int i0 = 0, pw = 0, iq = 0, iq_h = 0, n_tiles = 0;
    Stream st = {};
    FullBlocks fullb = {};
    bf16x8 qreg[KSTEPS];  // this wave's queries as B operands
    const float sl2 = p.scale * kLog2e_f;

    f32x16 oacc[DB];
    float m_run = -INFINITY, l_run = 0.f;  // m_run in the log2 domain (scores times scale*log2e)
    float neg_m = 0.f;                     // -m_run, 0 as long as no key has been seen
    float alpha_pending = 1.f;             // rescale of oacc decided by a softmax, applied before the next output update
    bool rescale = false;                  // alpha_pending != 1 in some lane (wave-uniform)
    bool no_max = true;                    // some lane has seen no key yet (wave-uniform)

    // ---- segments of this workgroup, as the loads see them.  The tiles of all segments form ONE stream
    // of loads that runs ahead of the multiplications also across segment borders, so that only the
    // first segment of a workgroup pays the start-up latencies.
    struct Seg {
        Stream st;
        int n_tiles, i0, de;
    };
    auto rank_of = [&](int round) { return round * wpg + ((round & 1) ? wpg - 1 - rank0 : rank0); };
    auto segment_at = [&](int rank) {  // rank < n_pos_tiles; no branches, so that the loads of two segments go out together
        Seg g;
        g.i0 = (n_pos_tiles - 1 - rank) * TP;
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
        return g;
    };
    // no more work: an empty stream of padding tiles
    auto past_the_last = []() { return Seg{Stream{0, 0, 0, 0, 0}, kIntMax, -1, kIntMax}; };
    auto open_segment = [&](int round) {
        const int rank = rank_of(round);
        return rank >= n_pos_tiles ? past_the_last() : segment_at(rank);
    };

    // ---- what a tile holds: worked out four tiles ahead of the multiplications, one row per lane, by wave
    // 0 (even tiles) and wave 1 (odd tiles; tiles 0 .. 3 by the first four waves) for all waves, which only read the rows' byte offsets back.  Two
    // steps: the index entries of the rows (issue_entries: list entry or prefix count of the row's
    // position, and the next prefix count) are requested with 4-byte global->LDS loads, and two tiles
    // later turned into key position and visibility range (write_rows).  Past the last segment the
    // stream is empty: its tiles are "loaded" too (row 0, never visible).
    struct Cursor {
        Seg cur, next;
        int round, t;  // segment of this workgroup and tile of its stream
    };
    auto advance = [&](Cursor &c) __attribute__((always_inline)) {
        if (++c.t == c.cur.n_tiles) {
            c.cur = c.next;
            ++c.round;
            c.t = 0;
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

    // ---- row loads: load n of a tile fills rows n*RPL .. +RPL-1 with one wave-wide direct global->LDS
    // load per tensor; wave w issues loads LOADS*w + u (the last one again where the waves do not
    // divide the tile: same bytes to the same place).  A lane owns physical chunk lane%CH of its row.
    const char *Kb = reinterpret_cast<const char *>(K + ((long)b * p.Hkv + kv) * (long)p.L * D);
    const char *Vb = reinterpret_cast<const char *>(V + ((long)b * p.Hkv + kv) * (long)p.L * D);
    const int my_pc = lane % CH, my_sub = lane / CH;
    const uint32_t ks_base = lds_addr(&Ks[0][0]), vs_base = lds_addr(&Vs[0][0]);
    uint32_t kgo[LOADS], vgo[LOADS];  // byte offset of this lane's 16-byte piece inside a K / V row
    uint32_t koffs[LOADS], voffs[LOADS];  // byte offsets of the rows this lane helps to fill next
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
        const int r = min(LOADS * wave + u, NLD - 1) * RPL + my_sub;
        kgo[u] = swz_chunk<kSwzRow, D>(my_pc, r) * 16;
        vgo[u] = swz_chunk<kSwzTr, D>(my_pc, r) * 16;
    }
    // the rows of K one tile further on than those of V
    auto read_offsets = [&](int g) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < LOADS; ++u) {
            voffs[u] = koffs[u];
            koffs[u] = off_s[g & 3][min(LOADS * wave + u, NLD - 1) * RPL + my_sub];
        }
    };
    auto issue_k = [&](int g, auto U) __attribute__((always_inline)) {
        constexpr int u = decltype(U)::value;
        dma_to_lds_16(Kb, koffs[u] + kgo[u], ks_base + (uint32_t)(g % KST) * (TILE * 2) + (uint32_t)min(LOADS * wave + u, NLD - 1) * 1024u);
    };
    auto issue_v = [&](int g, auto U) __attribute__((always_inline)) {
        constexpr int u = decltype(U)::value;
        dma_to_lds_16(Vb, voffs[u] + vgo[u], vs_base + (uint32_t)(g % VST) * (TILE * 2) + (uint32_t)min(LOADS * wave + u, NLD - 1) * 1024u);
    };

    const int a_row = pi_row(qi);
    // per-lane byte offsets of the operand fragments inside a tile (constant for the whole kernel).  The
    // XOR permutation of a K row acts on the chunk index 2*ks + hh and ks enters through its bits 1..3 only,
    // so fragment ks sits at (fragment 0) ^ (32 * ks).
    const uint32_t koff0 = lds_off_a<kSwzRow, D>(a_row, hh);
    uint32_t voff[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) voff[db] = lds_off_a_tr<kSwzTr, D>(db * 32, lane);

    // Workgroup barrier without the compiler's memory fence; what it publishes is waited for explicitly:
    // every row and entry load and every LDS write of the wave.
    auto wg_barrier = [&]() __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // ---- The pipeline.  Every wave runs the same instruction stream.  Work is cut into blocks of 32 keys
    // (block c = 2*tile + half).  Tile step X consists of two halves:
    //   half 1:  S(2X)   = K_X[ 0..31] Q^T      O^T += V_{X-1}[ 0..31]^T P(2X-2)^T    softmax of block 2X-1
    //   half 2:  S(2X+1) = K_X[32..63] Q^T      O^T += V_{X-1}[32..63]^T P(2X-1)^T    softmax of block 2X
    // A half begins with what branches (mask, rescaling) and then is ONE straight run of matrix
    // instructions, after each of which a fixed share of the rest (exponentials, row sum and rounding to
    // bf16 of one block, row loads, operand requests LA matrix instructions ahead) is
    // issued and executes while the matrix pipe is busy.  Branches inside the run, or results that are only
    // used beyond it, let the compiler move the vector work out of the shadow of the matrix
    // instructions: hence the scheduling fences and the empty asm statements that use the results in place.
    //
    // Step X reads K_X and V_{X-1} and requests K_{X+AH} and V_{X+AH-1}, whose stages held K_{X-AH} and
    // V_{X-AH-1}; barriers stand in front of every AH-th tile (of the concatenated stream), where everything
    // requested before has landed.  AH = 2 lets the two waves of a SIMD drift apart between barriers, so that one's
    // start of a half falls into the other's run; with AH = 1 they belong to different workgroups and do so anyway.
    f32x16 s_a, s_b;          // scores: first / second block of a tile
    bf16x8 p_a[2], p_b[2];    // probabilities (bf16, B-operand layout) of the first / second block
    constexpr int LA = D == 128 ? 6 : 4;
    constexpr int NQK = KSTEPS, NPV = 2 * DB;  // matrix instructions per half

    // largest score of a block for each of the wave's queries (log2 domain)
    auto block_max = [&](const f32x16 &s) __attribute__((always_inline)) {
        float m = fmaxf(fmaxf(s[0], s[1]), s[2]);
#pragma unroll
        for (int i = 3; i < 15; i += 2) m = fmaxf(fmaxf(m, s[i]), s[i + 1]);
        return pair_max(fmaxf(m, s[15]) * sl2);
    };
    // Raises the running maximum to that of a block where it has grown.  This happens where a query has no maximum yet
    // (before the block's exponentials), and afterwards only where the exponentials turn out too large (their sum
    // over a lane says so): the maximum of every block need not be known then.
    auto raise_max = [&](const f32x16 &s) __attribute__((always_inline)) {
        const float m = block_max(s);
        const bool grow = m > m_run + kRescaleThreshold;
        const float alpha = grow ? __builtin_amdgcn_exp2f(m_run - m) : 1.f;
        alpha_pending = rescale ? alpha_pending * alpha : alpha;
        m_run = grow ? m : m_run;
        neg_m = (m_run == -INFINITY) ? 0.f : -m_run;
        l_run *= alpha;
        rescale = true;
    };
    // softmax of a block, the part that branches: mask, first maximum
    auto softmax_head = [&](f32x16 &s, int tile, int gtile, int kb) __attribute__((always_inline)) {
        if (!block_is_full(fullb, tile * kBN + kb * 32)) {
            const int vs_ = (unsigned)gtile % MKS;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const int base = kb * 32 + 16 * half + 8 * hh;
                const int4 lo0 = *reinterpret_cast<const int4 *>(&lo_s[vs_][base]);
                const int4 lo1 = *reinterpret_cast<const int4 *>(&lo_s[vs_][base + 4]);
                const int4 hi0 = *reinterpret_cast<const int4 *>(&hi_s[vs_][base]);
                const int4 hi1 = *reinterpret_cast<const int4 *>(&hi_s[vs_][base + 4]);
                const int los[8] = {lo0.x, lo0.y, lo0.z, lo0.w, lo1.x, lo1.y, lo1.z, lo1.w};
                const int his[8] = {hi0.x, hi0.y, hi0.z, hi0.w, hi1.x, hi1.y, hi1.z, hi1.w};
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const bool vis = (los[k] <= iq) & (iq_h <= his[k]);
                    s[8 * half + k] = vis ? s[8 * half + k] : -INFINITY;
                }
            }
        }
        if (no_max) {
            raise_max(s);
            no_max = __builtin_amdgcn_ballot_w64(m_run == -INFINITY) != 0ull;
        }
    };
    auto apply_rescale = [&]() __attribute__((always_inline)) {
        if (rescale) {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int i = 0; i < 16; ++i) oacc[db][i] *= alpha_pending;
            rescale = false;
        }
    };
    auto pin = [&](bf16x8 (&x)[2]) __attribute__((always_inline)) {
        u32x4 &x0 = reinterpret_cast<u32x4 &>(x[0]), &x1 = reinterpret_cast<u32x4 &>(x[1]);
        asm volatile("" : "+v"(x0), "+v"(x1));
    };

    // one half of a tile step.  HB: which block of the tile (0 or 1).  DO_QK: S(2X+HB) of tile X into
    // s_new; DO_PV: O^T += V_{X-1}[32 HB ..]^T p_old^T; DO_SM: softmax of the block whose scores are
    // s_old (tile sm_tile, block sm_kb) into p_new; DO_LD: V rows of tile X+AH-1 and K rows of tile X+AH are requested.
    // NEXT: the last LA slots request the first operands of the tile's second block, which the following half then finds on
    // their way (READY) instead of waiting for them.
    int gbase = 0;  // global number of tile 0 of the segment being multiplied
    bf16x8 frag[LA];
    auto half_step = [&](int X, auto HB_, auto DO_QK_, auto DO_PV_, auto DO_SM_, auto DO_LD_, auto READY_, auto NEXT_, f32x16 &s_new,
                         const bf16x8 (&p_old)[2], f32x16 &s_old, bf16x8 (&p_new)[2], int sm_tile,
                         int sm_kb) __attribute__((always_inline)) {
        constexpr int HB = decltype(HB_)::value;
        constexpr bool DO_QK = decltype(DO_QK_)::value != 0, DO_PV = decltype(DO_PV_)::value != 0;
        constexpr bool DO_SM = decltype(DO_SM_)::value != 0, DO_LD = decltype(DO_LD_)::value != 0;
        constexpr bool READY = decltype(READY_)::value != 0, NEXT = decltype(NEXT_)::value != 0;
        constexpr int N1 = DO_QK ? NQK : 0, N2 = DO_PV ? NPV : 0, NS = N1 + N2;
        constexpr int E = (16 + NS - 1) / NS;              // elements of the softmax per matrix instruction
        // (which half is added after the XOR, so that it becomes the instruction's offset and both halves share the addresses)
        const uint32_t vst = vs_base + ((unsigned)(gbase + X + VST - 1) % VST) * (TILE * 2);
        const uint32_t kst = ks_base + ((unsigned)(gbase + X) % KST) * (TILE * 2) + koff0;
        constexpr uint32_t HO = HB * 32 * D * 2;
        constexpr int OFF = READY ? (NQK + NPV) % LA : 0;  // where the half before put the first operand
        auto request = [&](auto S) __attribute__((always_inline)) {
            constexpr int s = decltype(S)::value;
            if constexpr (s < N1) {
                frag[(s + OFF) % LA] = lds_read_b128_at((kst ^ (32u * s)) + HO);
            } else if constexpr (s < NS) {
                constexpr int q_ = s - N1, stp = q_ / DB, db = q_ % DB;
                frag[(s + OFF) % LA] = lds_read_tr_at(vst + voff[db] + (HO + stp * 16 * D * 2), 4 * D * 2);
            } else if constexpr (NEXT) {
                static_assert(HB == 0 && DO_QK && LA <= NQK, "the next half begins with K rows 32 .. 63 of the same tile");
                constexpr int n = s - NS;
                frag[s % LA] = lds_read_b128_at((kst ^ (32u * n)) + 32 * D * 2);
            }
        };
        auto multiply = [&](auto S) __attribute__((always_inline)) {
            constexpr int s = decltype(S)::value;
            if constexpr (s < N1) {
                const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                s_new = mfma_bf16(frag[(s + OFF) % LA], qreg[s], s == 0 ? zero : s_new);
            } else {
                constexpr int q_ = s - N1, stp = q_ / DB, db = q_ % DB;
                oacc[db] = mfma_bf16(frag[(s + OFF) % LA], p_old[stp], oacc[db]);
            }
        };
        if constexpr (DO_LD) read_offsets(gbase + X + AH);
        if constexpr (!READY) static_for<(LA < NS ? LA : NS)>([&](auto S) { request(S); });
        if constexpr (DO_PV) apply_rescale();
        if constexpr (DO_SM) softmax_head(s_old, sm_tile, gbase + sm_tile, sm_kb);
        float psum = 0.f;
        f32x16 pe;  // exponentials; the scores stay, in case they turn out too large
        __builtin_amdgcn_sched_barrier(0);
        static_for<NS>([&](auto S) {
            constexpr int s_ = decltype(S)::value;
            multiply(S);
            request(IntC<s_ + LA>{});
            if constexpr (DO_SM) {
                // the sum takes an element one slot later, when the transcendental unit has delivered
                constexpr int e0 = E * s_;
#pragma unroll
                for (int i = e0; i < e0 + E && i < 16; ++i) pe[i] = __builtin_amdgcn_exp2f(fmaf(s_old[i], sl2, neg_m));
#pragma unroll
                for (int i = e0 - E; i < e0; ++i)
                    if (i >= 0) psum += pe[i];
                if constexpr (e0 - E < 8 && e0 >= 8) p_new[0] = pack_bf16x8(pe, 0);
            }
            if constexpr (DO_LD && s_ >= 1) {
                constexpr int LPS = (2 * LOADS + NS - 2) / (NS - 1), n0 = (s_ - 1) * LPS;  // row loads per slot
                static_for<LPS>([&](auto J) {
                    constexpr int n = n0 + decltype(J)::value;
                    if constexpr (n < LOADS) issue_v(gbase + X + AH - 1, IntC<n>{});
                    else if constexpr (n < 2 * LOADS) issue_k(gbase + X + AH, IntC<n - LOADS>{});
                });
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (DO_SM) {
#pragma unroll
            for (int i = 16 - E; i < 16; ++i) psum += pe[i];
            p_new[1] = pack_bf16x8(pe, 8);
            if (__builtin_amdgcn_ballot_w64(psum > 16.f * kMaxTerm) != 0ull) {
                raise_max(s_old);
                psum = 0.f;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    pe[i] = __builtin_amdgcn_exp2f(fmaf(s_old[i], sl2, neg_m));
                    psum += pe[i];
                }
                p_new[0] = pack_bf16x8(pe, 0);
                p_new[1] = pack_bf16x8(pe, 8);
            }
            l_run += psum;
            pin(p_new);
            asm volatile("" : "+v"(l_run));
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    Seg cseg = segment_at(rank0), cnext = segment_at(min(rank_of(1), n_pos_tiles - 1));
    if (rank_of(1) >= n_pos_tiles) cnext = past_the_last();
    auto load_queries = [&](int seg_i0) __attribute__((always_inline)) {
        const int row = min(seg_i0 + 32 * (wave / GP) + qi, p.L - 1);
        const uint16_t *qrow = Q + (((long)b * p.Hq + head) * p.L + row) * D;
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks)
            qreg[ks] = as_bf16x8(*reinterpret_cast<const u32x4 *>(qrow + ks * 16 + 8 * hh));
    };

    // ---- start-up, once per workgroup: positions of tiles 0 .. 3, a wave each, then the first rows (the entries of tiles 4
    // and 5 are on their way).  The queries are requested behind the entries, which alone are waited for: they come into registers, so
    // that the compiler counts the loads that it has placed behind them.
    Cursor lc = {cseg, cnext, 0, 0};
    int e0 = 0, e1 = 0, e_doc = 0;
    if (wave < 4) {
        for (int t = 0; t < wave; ++t) advance(lc);
        const EntryAt at = entry_at(lc.cur.st, lc.t);
        e0 = *at.of_row, e1 = *at.behind;
        if constexpr (DOCS) e_doc = *at.doc_end;
    }
    __builtin_amdgcn_sched_barrier(0);
    load_queries(cseg.i0);
    __builtin_amdgcn_sched_barrier(0);
    if (wave < 4) {
        const Cursor own = lc;
        if (wave < 2)
            for (int t = 0; t < 4; ++t) advance(lc);
        asm volatile("" : "+v"(e0), "+v"(e1), "+v"(e_doc));  // looked at from here on
        write_entries(own, wave, e0, e1, e_doc);
        if (wave < 2) issue_entries(lc.cur.st, lc.t, 4 + wave);
    }
    // start of tile step g: positions of a tile four further on, entries of one six further on (AH = 2: of two
    // tiles every other step)
    auto look_ahead = [&](int g) __attribute__((always_inline)) {
        if (AH == 1 ? wave == (g & 1) : ((g & 1) == 0 && wave < 2)) {
            const int t = g + (AH == 1 ? 0 : wave);
            write_rows(lc, t + 4);
            advance(lc);
            advance(lc);
            issue_entries(lc.cur.st, lc.t, t + 6);
        }
    };
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // only what write_rows wrote is published here
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    read_offsets(0);
    static_for<LOADS>([&](auto U) { issue_k(0, U); });
    if constexpr (AH == 2) {
        read_offsets(1);
        static_for<LOADS>([&](auto U) { issue_v(0, U); });
        static_for<LOADS>([&](auto U) { issue_k(1, U); });
    }
    wg_barrier();

    const IntC<1> yes;
    const IntC<0> no;
    const IntC<0> first_block;
    const IntC<1> second_block;
    // a tile step of a wave that is through with its own blocks
    auto loads_only = [&](int X) __attribute__((always_inline)) {
        look_ahead(gbase + X);
        read_offsets(gbase + X + AH);
        static_for<LOADS>([&](auto U) { issue_v(gbase + X + AH - 1, U); });
        static_for<LOADS>([&](auto U) { issue_k(gbase + X + AH, U); });
    };
    for (int round = 0; cseg.i0 >= 0; ++round) {
    i0 = cseg.i0;
    pw = i0 + 32 * (wave / GP);  // first position of this wave
    iq = pw + qi;                // this lane's query position
    iq_h = iq + hdelta;          // ... as the upper ends of the keys' query ranges (computed with p.n) see it
    st = cseg.st;
    n_tiles = cseg.n_tiles;
    // tiles up to the wave's last position; in those beyond it only takes part in the loads
    const int my_tiles = OWN_END ? (min(st.n_total, st.n_dense + pw + 32 - st.bs) + kBN - 1) / kBN : n_tiles;
    fullb = full_blocks(st, pw, p.n - hdelta);
    if (DOCS && pw + 31 >= cseg.de) fullb = no_full_blocks();
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[db][i] = 0.f;
    m_run = -INFINITY;
    l_run = 0.f;
    neg_m = 0.f;
    rescale = false;
    no_max = true;

    // step 0: no output update yet, no softmax in the first half.  Its barrier was that of the start-up or
    // of the previous segment's last step.
    look_ahead(gbase);
    half_step(0, first_block, yes, no, no, yes, no, no, s_a, p_a, s_b, p_b, 0, 0);
    half_step(0, second_block, yes, no, yes, no, no, no, s_b, p_b, s_a, p_a, 0, 0);
    int X = 1;
    for (; X < my_tiles; ++X) {
        if ((gbase + X) % AH == 0) wg_barrier();
        look_ahead(gbase + X);
        half_step(X, first_block, yes, yes, yes, yes, no, yes, s_a, p_a, s_b, p_b, X - 1, 1);
        half_step(X, second_block, yes, yes, yes, no, yes, no, s_b, p_b, s_a, p_a, X, 0);
    }
    // last step: output updates of the last tile, softmax of its second block; the queries of the
    // next segment are fetched meanwhile (the registers are free: no score block in this step)
    if ((gbase + X) % AH == 0) wg_barrier();
    if (OWN_END && X < n_tiles) loads_only(X);
    if (cnext.i0 >= 0) load_queries(cnext.i0);
    half_step(X, first_block, no, yes, yes, no, no, no, s_a, p_a, s_b, p_b, X - 1, 1);
    half_step(X, second_block, no, yes, no, no, no, no, s_b, p_b, s_a, p_a, X, 0);
    if constexpr (OWN_END) {
        while (++X <= n_tiles) {
            if ((gbase + X) % AH == 0) wg_barrier();
            if (X < n_tiles) loads_only(X);
        }
    }
    gbase += n_tiles;

    // epilogue: normalise, store O (bf16) and LSE (natural log)
    float l_tot = pair_sum(l_run);
    float inv = 1.f / l_tot;
    // A lane holds 4-column pieces of ONE output row, so a store straight from the accumulators would
    // write 64 scattered 8-byte pieces per instruction, and the number of such pieces (1024 per wave
    // and segment) is what the stores cost.  Each 32-column block of the wave's 32 rows therefore goes
    // through a 2 KB staging area of the wave and leaves as 16-byte pieces of which four consecutive
    // lanes cover 64 contiguous bytes of a row (16 rows per store instruction).  8-byte chunk ch of
    // row r sits at chunk position ch ^ (2 * ((r / 4) % 4)): 16-byte pairs stay together, and the
    // writes (one chunk of 32 rows) spread over the banks.  The LDS operations of a wave execute in
    // order, so a block's reads are issued before the next block's writes without a wait in between.
    {
        // d = 64: worked out anew from the lane's number each time (kept over the loop it would go to scratch memory there)
        int ln = lane;
        if constexpr (D == 64) asm volatile("" : "+v"(ln));
        const int lane = ln, qi = lane & 31, hh = lane >> 5;
        uint16_t *stg = &ostage[wave][0];
        const long orow0 = ((long)b * p.Hq + head) * p.L + pw;  // output row of the wave's first query
        const int wsw = ((qi >> 2) & 3) << 1;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const uint2 v = pack_bf16x4(oacc[db][4 * i4] * inv, oacc[db][4 * i4 + 1] * inv,
                                            oacc[db][4 * i4 + 2] * inv, oacc[db][4 * i4 + 3] * inv);
                *reinterpret_cast<uint2 *>(stg + qi * 32 + (((2 * i4 + hh) ^ wsw) * 4)) = v;
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int r = 16 * t + (lane >> 2), c = lane & 3;
                const int pos = (2 * c) ^ (((r >> 2) & 3) << 1);
                const uint4 v = *reinterpret_cast<const uint4 *>(stg + r * 32 + pos * 4);
                if (pw + r < p.L) *reinterpret_cast<uint4 *>(O + (orow0 + r) * D + db * 32 + c * 8) = v;
            }
            __builtin_amdgcn_sched_barrier(0);  // one block at a time: keeps the register pressure of the epilogue down
        }
    }
    if (iq < p.L && hh == 0) LSE[((long)b * p.Hq + head) * p.L + iq] = (m_run + __builtin_amdgcn_logf(l_tot)) * kLn2_f;
    cseg = cnext;
    cnext = open_segment(round + 2);
    }  // segments
    // the loads of the padding tiles past the last segment are still in flight: they must have
    // landed before the workgroup ends and its LDS is handed on
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

template <int D, bool DOCS>
int launch_fwd(const sepattn_params &p, const uint16_t *Q, const uint16_t *K, const uint16_t *V,
               const int32_t *sep_idx, const int32_t *sep_prefix, const int32_t *doc_start, const int32_t *doc_end,
               uint16_t *O, float *LSE, const HeadWin &hw, hipStream_t st) {
    const QueryShape shape = query_shape(p);
    const int TP = 32 * shape.nw / shape.gp;
    const int n_pos_tiles = (p.L + TP - 1) / TP;
    const long n_groups = (long)p.B * (p.Hq / shape.gp);
    // persistent workgroups, spread evenly over the groups; never more than a group has tiles
    int wpg = (int)((shape.nw > 4 ? 1 : D == 64 ? 3 : 2) * (long)compute_units() / n_groups);
    wpg = wpg < 1 ? 1 : (wpg > n_pos_tiles ? n_pos_tiles : wpg);
    if (n_groups * wpg > 0x7FFFFFFFL) return SEPATTN_ERR_SHAPE;
    WorkShare share = {};
    long n_wg = n_groups * wpg;
    const bool headwise = !DOCS && any_delta(hw);  // (packed calls have no windows per head)
    if (headwise) {
        share = share_queries(p, hw, shape.gp, TP, (shape.nw > 4 ? 1 : D == 64 ? 3 : 2) * compute_units() / p.B, 0);
        n_wg = (long)p.B * share.first[share.n];
    }
    const QueryGrid qg = query_grid(p, shape.gp, n_groups);
    const dim3 block(64 * shape.nw), grid = headwise ? dim3((unsigned)n_wg) : dim3((unsigned)qg.gx, (unsigned)wpg, (unsigned)(n_groups / qg.gx));
    {
    ProfScope prof(SEPATTN_K_FORWARD, st);
    auto go = [&](auto NW_, auto GP_) {
        constexpr int NW = decltype(NW_)::value, GP = decltype(GP_)::value;
        if constexpr (!DOCS) {
            if (headwise) {
                hipLaunchKernelGGL((fwd_bf16_kernel<D, GP, false, NW, true>), grid, block, 0, st, p, Q, K, V, sep_idx, sep_prefix, doc_start, doc_end, O, LSE, wpg, qg, (HeadArgs<true>{hw, share}));
                return;
            }
        }
        hipLaunchKernelGGL((fwd_bf16_kernel<D, GP, DOCS, NW, false>), grid, block, 0, st, p, Q, K, V, sep_idx, sep_prefix, doc_start, doc_end, O, LSE, wpg, qg, HeadArgs<false>{});
    };
    if (shape.gp == 7) go(IntC<7>{}, IntC<7>{});
    else if (D == 128 && shape.nw == 8) go(IntC<D == 128 ? 8 : 4>{}, IntC<4>{});
    else if (shape.gp == 4) go(IntC<4>{}, IntC<4>{});
    else if (shape.gp == 2) go(IntC<4>{}, IntC<2>{});
    else go(IntC<4>{}, IntC<1>{});
    }
    return launch_status();
}

}  // namespace

size_t forward_bf16_workspace(const sepattn_params &) { return 0; }

int launch_forward_bf16(const sepattn_params &p, const HeadWin &hw, const void *Q, const void *K, const void *V,
                        const int32_t *sep_idx, const int32_t *sep_prefix, const int32_t *doc_start,
                        const int32_t *doc_end, void *O, float *LSE, void *, hipStream_t st) {
    auto q = static_cast<const uint16_t *>(Q), k = static_cast<const uint16_t *>(K),
         v = static_cast<const uint16_t *>(V);
    auto o = static_cast<uint16_t *>(O);
    if (doc_start) {
        if (p.d == 64) return launch_fwd<64, true>(p, q, k, v, sep_idx, sep_prefix, doc_start, doc_end, o, LSE, hw, st);
        return launch_fwd<128, true>(p, q, k, v, sep_idx, sep_prefix, doc_start, doc_end, o, LSE, hw, st);
    }
    if (p.d == 64) return launch_fwd<64, false>(p, q, k, v, sep_idx, sep_prefix, nullptr, nullptr, o, LSE, hw, st);
    return launch_fwd<128, false>(p, q, k, v, sep_idx, sep_prefix, nullptr, nullptr, o, LSE, hw, st);
}

}  // namespace sepattn
