// fp32 path of SepAttention forward and backward (Eq. 1 with the mask of Eq. 2): the path that a bf16
// run is checked against.
//
// All contractions run on v_mfma_f32_16x16x4_f32 (fp32 operands, fp32 accumulation: a fused
// multiply-add per product, no reduced precision anywhere) in blocks of 16 queries x 16 keys of one query head.  Operand layouts
// (lane l, m = l%16, g = l/16):
//   A (16 x 4): row m, k = g          B (4 x 16): column m, k = g
//   C (16 x 16): column m, register i holds row 4 g + i
// The k slots of a contraction may be dealt in any order as long as both operands agree, so a row
// operand is read as 16-byte pieces (piece c of a lane: elements 16 c + 4 g .. +3 of its row, one
// element per matrix instruction), and a lane's four accumulator registers of one contraction are,
// as they stand, its B operand of the next one (step i: k slot g is accumulator row 4 g + i).
//
// At the sizes this path is used at, a call lasts about as long as its chain of memory latencies, so
// the work of a tile is spread over the four waves of a workgroup (16-key blocks, or query blocks, dealt round-robin; the waves'
// partial results meet once in LDS), operands go straight from memory to registers, and what can
// share a launch does: dQ and dK/dV (fp32_one_launch), and the far keys' partial sums are added by the
// last workgroup to finish a list tile instead of by a kernel of their own.
//
// A masked pair enters the contractions over streamed rows with weight 0, and 0 times an infinity or a NaN is NaN: a
// non-finite value in a row would reach every row of the other side that shares a block with it.  As all that such a
// pair can do to a sum is to make it NaN, a wave looks at its finished sums and, if one is NaN, forms them once more
// with vector arithmetic over the visible pairs only.  Finite inputs pay for the look: 43.9 -> 44.6 us for the call
// below; B=1, 32/8 heads, L=4096, d=128, n=256 451 us forward and 1858 backward with it, 452 and 1866 without.
// B=1, 2 heads per KV head, L=512, d=64, n=64: forward 22 -> 7 us, D_i and dQ 5 + 23 -> 8, dK/dV 168 -> 16, against one
// wave per row on the vector ALU.
#include "attn_fp32.h"
#include "bwd_common.h"
#include "key_stream.h"
#include "mfma_common.h"

namespace sepattn {

namespace {

constexpr int kWaves = 4;  // waves per workgroup
// (query block, head) items per far slice: one per wave, more where a list tile of the whole sequence would be shared among
// more than kMaxShare slices, whose sums one workgroup adds.  Backward, us, with 4 / 8 / the rule: 2 heads per KV head,
// L=512, d=64 23.0 / 23.9 / 23.0; 4 and 4 heads, 2 x L=300, d=128 32.7 / 36.4 / 32.7; 4 heads per KV head, 2 x L=1000, d=64
// 34.0 / 30.7 / 30.7.
constexpr int kMinItems = 4, kMaxShare = 32;

__device__ inline f32x4 mfma_f32(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

template <int D>
__device__ inline void load_row(f32x4 (&f)[D / 16], const float *__restrict__ row, int g) {
#pragma unroll
    for (int c = 0; c < D / 16; ++c) f[c] = *reinterpret_cast<const f32x4 *>(row + 16 * c + 4 * g);
}
// x = A B over D, two interleaved accumulators
template <int D>
__device__ inline f32x4 row_product(const f32x4 (&a)[D / 16], const f32x4 (&b)[D / 16]) {
    f32x4 x = {0.f, 0.f, 0.f, 0.f}, y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < D / 16; ++c) {
        x = mfma_f32(a[c][0], b[c][0], x);
        y = mfma_f32(a[c][1], b[c][1], y);
        x = mfma_f32(a[c][2], b[c][2], x);
        y = mfma_f32(a[c][3], b[c][3], y);
    }
    return x + y;
}
__device__ inline float group_max(float v) {
    v = fmaxf(v, __shfl_xor(v, 16));
    return fmaxf(v, __shfl_xor(v, 32));
}
__device__ inline float group_sum(float v) {
    v += __shfl_xor(v, 16);
    return v + __shfl_xor(v, 32);
}

// Divisors that a launch has in common.
struct Fp32Plan {
    FastDiv by_tiles, by_hq, by_g, by_bkv, by_hkv, by_min_slice;
    int n_tiles, G, min_slice;
};
// A query tile: 16 positions from i0 on of one query head, and its key stream (key_stream.h).
struct QueryTile {
    int b, h, kv, i0;
    long row0;  // first row of the head in [B, Hq, L]
    sepattn_params p;  // p.n: the head's own window
    const int32_t *prefix, *idx, *dend;
    Stream st;
    int de;
};
template <bool HW>
__device__ inline QueryTile query_tile(const sepattn_params &p, const Fp32Plan &pl, const HeadArgs<HW> &ha, int block, const int32_t *sep_idx,
                                       const int32_t *sep_prefix, const int32_t *doc_start, const int32_t *doc_end) {
    QueryTile t;
    const int bh = quotient(block, pl.by_tiles);
    t.b = quotient(bh, pl.by_hq), t.h = bh - t.b * p.Hq, t.kv = quotient(t.h, pl.by_g);
    t.i0 = (block - bh * pl.n_tiles) * kT;
    t.row0 = (long)bh * p.L;
    t.p = p;
    t.p.n = p.n - ha.of_head(t.h);
    t.prefix = sep_prefix + (long)t.b * (p.L + 1);
    t.idx = sep_idx + (long)t.b * p.cap;
    t.dend = doc_end ? doc_end + (long)t.b * p.L : nullptr;
    if (doc_start) {
        // the clamps keep inconsistent bounds (caller error) from faulting
        t.st = make_stream_docs(t.p, t.prefix, t.i0, kT, min(max(doc_start[(long)t.b * p.L + t.i0], 0), t.i0));
        t.de = min(max(t.dend[t.i0], t.i0 + 1), p.L);
    } else {
        t.st = make_stream(t.p, t.prefix, t.i0, kT);
        t.de = kIntMax;
    }
    return t;
}
// position and visible query range of stream element k
__device__ inline int tile_key(const QueryTile &t, int k, int &lo, int &hi) {
    const int j = stream_key(t.st, k, t.p, t.idx, t.prefix, lo, hi);
    if (t.dend) hi = min(hi, (k < t.st.n_dense ? t.de : t.dend[j]) - 1);
    return j;
}
// the four keys whose scores this lane holds: element 4 g + i of a block, described by lane 4 g + i
struct Keys4 {
    int j[4];
    bool vis[4];
};
__device__ inline Keys4 keys_of_lane(int j, int lo, int hi, int g, int iq) {
    Keys4 k;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int src = 4 * g + i;
        k.j[i] = __shfl(j, src);
        const int l = __shfl(lo, src), h = __shfl(hi, src);  // every lane takes part in both
        k.vis[i] = l <= iq && iq <= h;
    }
    return k;
}
// element (column block cb * 16 + m, streamed row i of the lane's four) of a row-major matrix, transposed operand
template <int D>
__device__ inline void load_columns(float (&f)[D / 16][4], const float *__restrict__ base, const int (&row)[4], int m) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int cb = 0; cb < D / 16; ++cb) f[cb][i] = base[(long)row[i] * D + 16 * cb + m];
}

template <int C>
__device__ inline bool any_nan(const f32x4 (&x)[C]) {
    bool n = false;
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) n |= x[c][e] != x[c][e];
    return __ballot(n) != 0ull;
}
// acc (column m, rows 16 c + 4 g + e: dimensions) += sum over the 16 streamed rows of weight * row, visible pairs only:
// what load_columns and the matrix instructions add where every value is finite.  w, vis, row: the lane's four.
template <int D>
__device__ inline void add_visible(f32x4 (&acc)[D / 16], const f32x4 &w, const bool (&vis)[4], const float *__restrict__ base,
                                   const int (&row)[4], int m, int g) {
#pragma unroll 1
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int src = 16 * s + m, r = __shfl(row[i], src);  // every lane takes part in all three
            const float f = __shfl(w[i], src);
            const bool v = __shfl((int)vis[i], src) != 0;
            asm volatile("" ::: "memory");  // one row at a time: no more registers than the matrix path
            f32x4 x[D / 16];
            load_row<D>(x, base + (long)r * D, g);
            if (!v) continue;
#pragma unroll
            for (int c = 0; c < D / 16; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[c][e] = fmaf(f, x[c][e], acc[c][e]);
        }
}

// ---- forward -----------------------------------------------------------------------------------
template <int D, bool HW>
__global__ __launch_bounds__(64 * kWaves, D == 64 ? 4 : 3) void fwd_fp32_kernel(sepattn_params p, const float *__restrict__ Q,
                                                               const float *__restrict__ K, const float *__restrict__ V,
                                                               const int32_t *__restrict__ sep_idx,
                                                               const int32_t *__restrict__ sep_prefix,
                                                               const int32_t *__restrict__ doc_start,
                                                               const int32_t *__restrict__ doc_end,
                                                               float *__restrict__ O, float *__restrict__ LSE, Fp32Plan pl, HeadArgs<HW> ha) {
    constexpr int C = D / 16;
    __shared__ float os[kWaves][kT][D + 4];
    __shared__ float ms[kWaves][kT], ls[kWaves][kT];
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform: scalar loads and branches
    const QueryTile t = query_tile<HW>(p, pl, ha, blockIdx.x, sep_idx, sep_prefix, doc_start, doc_end);
    const long kv0 = ((long)t.b * p.Hkv + t.kv) * (long)p.L * D;
    const float *Kh = K + kv0, *Vh = V + kv0;
    const int iq = t.i0 + m;
    f32x4 qf[C], o[C];
    load_row<D>(qf, Q + (t.row0 + min(iq, p.L - 1)) * D, g);
    float mx, l;
    auto run = [&](auto VISIBLE_ONLY) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < C; ++c) o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
        mx = -INFINITY, l = 0.f;
        for (int k0 = wave * kT; k0 < t.st.n_total; k0 += kWaves * kT) {
            int lo, hi;
            const int j = tile_key(t, k0 + m, lo, hi);
            f32x4 kf[C];
            load_row<D>(kf, Kh + (long)j * D, g);
            const Keys4 kk = keys_of_lane(j, lo, hi, g, iq);
            float vf[C][4];
            if constexpr (!VISIBLE_ONLY) load_columns<D>(vf, Vh, kk.j, m);
            f32x4 s = row_product<D>(kf, qf);
            float mb = -INFINITY;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s[i] = kk.vis[i] ? s[i] * p.scale : -INFINITY;
                mb = fmaxf(mb, s[i]);
            }
            const float m_new = fmaxf(mx, group_max(mb));
            const float ref = m_new == -INFINITY ? 0.f : m_new;  // a row that has seen no key yet
            const float alpha = expf(mx - ref);
            float ps = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s[i] = expf(s[i] - ref);
                ps += s[i];
            }
            l = l * alpha + group_sum(ps);
            mx = m_new;
#pragma unroll
            for (int c = 0; c < C; ++c) o[c] *= alpha;
            if constexpr (VISIBLE_ONLY) {
                add_visible<D>(o, s, kk.vis, Vh, kk.j, m, g);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int c = 0; c < C; ++c) o[c] = mfma_f32(vf[c][i], s[i], o[c]);
            }
        }
    };
    run(IntC<0>{});
    if (any_nan(o)) run(IntC<1>{});
#pragma unroll
    for (int c = 0; c < C; ++c) *reinterpret_cast<f32x4 *>(&os[wave][m][16 * c + 4 * g]) = o[c];
    if (g == 0) ms[wave][m] = mx, ls[wave][m] = l;
    __syncthreads();
    for (int e = threadIdx.x; e < kT * D / 4; e += 64 * kWaves) {
        const int r = e / (D / 4), col = (e % (D / 4)) * 4;
        float mt = ms[0][r], lt = 0.f;
        for (int w = 1; w < kWaves; ++w) mt = fmaxf(mt, ms[w][r]);
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const float f = expf(ms[w][r] - mt);
            lt += ls[w][r] * f;
            x += *reinterpret_cast<const f32x4 *>(&os[w][r][col]) * f;
        }
        if (t.i0 + r < p.L) {
            *reinterpret_cast<f32x4 *>(O + (t.row0 + t.i0 + r) * D + col) = x / lt;
            if (col == 0) LSE[t.row0 + t.i0 + r] = mt + logf(lt);
        }
    }
}

// ---- dQ, and D_i = <dO_i, O_i> (stored where Dws is given) ------------------------------------------
template <int D, bool HW>
__device__ inline void dq_tile(float (&xs)[kWaves][kT][D + 4], int block, const sepattn_params &p, const float *__restrict__ Q,
                               const float *__restrict__ K, const float *__restrict__ V, const float *__restrict__ O,
                               const float *__restrict__ LSE, const float *__restrict__ dO, const int32_t *__restrict__ sep_idx,
                               const int32_t *__restrict__ sep_prefix, const int32_t *__restrict__ doc_start,
                               const int32_t *__restrict__ doc_end, float *__restrict__ dQ, float *__restrict__ Dws,
                               const Fp32Plan &pl, const HeadArgs<HW> &ha) {
    constexpr int C = D / 16;
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform: scalar loads and branches
    const QueryTile t = query_tile<HW>(p, pl, ha, block, sep_idx, sep_prefix, doc_start, doc_end);
    const long kv0 = ((long)t.b * p.Hkv + t.kv) * (long)p.L * D;
    const float *Kh = K + kv0, *Vh = V + kv0;
    const int iq = t.i0 + m;
    const long row = t.row0 + min(iq, p.L - 1);
    f32x4 qf[C], gf[C], acc[C];
    load_row<D>(qf, Q + row * D, g);
    load_row<D>(gf, dO + row * D, g);
    float Di = 0.f;
    {
        f32x4 of[C];
        load_row<D>(of, O + row * D, g);
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) Di = fmaf(gf[c][e], of[c][e], Di);
        Di = group_sum(Di);
    }
    const float lse = LSE[row];
    if (Dws && wave == 0 && g == 0 && iq < p.L) Dws[row] = Di;
    auto run = [&](auto VISIBLE_ONLY) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < C; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int k0 = wave * kT; k0 < t.st.n_total; k0 += kWaves * kT) {
            int lo, hi;
            const int j = tile_key(t, k0 + m, lo, hi);
            f32x4 kf[C], vf[C];
            load_row<D>(kf, Kh + (long)j * D, g);
            load_row<D>(vf, Vh + (long)j * D, g);
            const Keys4 kk = keys_of_lane(j, lo, hi, g, iq);
            float kt[C][4];
            if constexpr (!VISIBLE_ONLY) load_columns<D>(kt, Kh, kk.j, m);
            const f32x4 s = row_product<D>(kf, qf), dp = row_product<D>(vf, gf);
            f32x4 ds;
#pragma unroll
            for (int i = 0; i < 4; ++i) ds[i] = kk.vis[i] ? expf(s[i] * p.scale - lse) * (dp[i] - Di) : 0.f;
            if constexpr (VISIBLE_ONLY) {
                add_visible<D>(acc, ds, kk.vis, Kh, kk.j, m, g);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int c = 0; c < C; ++c) acc[c] = mfma_f32(kt[c][i], ds[i], acc[c]);
            }
        }
    };
    run(IntC<0>{});
    if (any_nan(acc)) run(IntC<1>{});
#pragma unroll
    for (int c = 0; c < C; ++c) *reinterpret_cast<f32x4 *>(&xs[wave][m][16 * c + 4 * g]) = acc[c];
    __syncthreads();
    for (int e = threadIdx.x; e < kT * D / 4; e += 64 * kWaves) {
        const int r = e / (D / 4), col = (e % (D / 4)) * 4;
        f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kWaves; ++w) x += *reinterpret_cast<const f32x4 *>(&xs[w][r][col]);
        if (t.i0 + r < p.L) *reinterpret_cast<f32x4 *>(dQ + (t.row0 + t.i0 + r) * D + col) = x * p.scale;
    }
}

// ---- dK, dV ------------------------------------------------------------------------------------
// Keys come in two kinds of tiles of 16: consecutive positions, of which only those that are neither
// initial tokens nor separators count (a band unit: the queries of their window), and consecutive
// entries of the far list (every query from the tile's first key to the end of the sequence or
// document).  The items (query block, head) of all list tiles of a (batch, KV head), in order, are
// cut into equal slices, one per workgroup, at most `wpg` of them and none shorter than kMinItems (and see kMaxShare); a
// list tile that lies in one slice is finished there, otherwise each slice writes a partial (slot
// slice + tile) and the workgroup that is the last to count itself in adds them in slice order.
// Every wave of a workgroup keeps the tile's K and V rows and its own dK and dV sums in registers.
// OWN_D: D_i is formed here, from the rows of dO, which an item reads anyway, and of O, so that the launch need not wait for dQ;
// and slices are counted in words that nobody has to clear (common.h; `one`) instead of in counters.
template <int D, bool HW, bool OWN_D>
__device__ inline void dkv_unit(float (&xs)[kWaves][kT][D + 4], const sepattn_params &p, const float *__restrict__ Q, const float *__restrict__ K,
                                const float *__restrict__ V, const float *__restrict__ O, const float *__restrict__ LSE,
                                const float *__restrict__ dO, const float *__restrict__ Drow, const int32_t *__restrict__ sep_idx,
                                const int32_t *__restrict__ sep_prefix, const int32_t *__restrict__ doc_end, float *__restrict__ dK,
                                float *__restrict__ dV, float *__restrict__ partials, void *__restrict__ counters, int n_far_tiles, int wpg,
                                int word_stride, uint64_t one, const Fp32Plan &pl, const HeadArgs<HW> &ha) {
    constexpr int C = D / 16;
    __shared__ int last_s, js[kT];  // js: the keys of a list tile
    const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform: scalar loads and branches
    const int G = pl.G, n_bkv = p.B * p.Hkv;
    const int unit = quotient(blockIdx.x, pl.by_bkv), bkv = blockIdx.x - unit * n_bkv;  // units: wpg far slices, then the band units
    const int b = quotient(bkv, pl.by_hkv), kv = bkv - b * p.Hkv;
    const int32_t *prefix = sep_prefix + (long)b * (p.L + 1);
    const int32_t *idx = sep_idx + (long)b * p.cap;
    const int32_t *dend = doc_end ? doc_end + (long)b * p.L : nullptr;
    const long kvrow0 = (long)bkv * p.L;
    const FarList fl = far_list(p, prefix);
    f32x4 kf[C], vf[C], ak[C], av[C];

    // items [first, last) of the tile's keys, item i = (query block i % n_qb from q_lo on, head i / n_qb), added to ak, av
    auto run_items = [&](int first, int last, int q_lo, int n_qb, int j, bool valid, int end, bool far) __attribute__((always_inline)) {
        const int jr = valid ? j : 0;
        load_row<D>(kf, K + (kvrow0 + jr) * D, g);
        load_row<D>(vf, V + (kvrow0 + jr) * D, g);
        const float by_qb = reciprocal(n_qb);
        auto run = [&](auto VISIBLE_ONLY) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < C; ++c) ak[c] = av[c] = f32x4{0.f, 0.f, 0.f, 0.f};
            for (int it = first + wave; it < last; it += kWaves) {
                const int head = last < kSmallQuotient ? __builtin_amdgcn_readfirstlane(small_quotient(it, by_qb)) : it / n_qb;
                const int h = kv * G + head, q0 = q_lo + (it - head * n_qb) * kT;
                // last query that sees the key: end of the sequence (document), or of head h's window
                const int hi = valid ? (far ? end : (int)min((long)end, (long)j + p.n - ha.of_head(h))) - 1 : -1;
                if (__ballot(hi >= q0) == 0ull) continue;
                const long hrow = ((long)b * p.Hq + h) * p.L;
                f32x4 qf[C], gf[C];
                const long qrow = hrow + min(q0 + m, p.L - 1);
                load_row<D>(qf, Q + qrow * D, g);
                load_row<D>(gf, dO + qrow * D, g);
                int qi[4];
                float lse[4], Dq[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    qi[i] = min(q0 + 4 * g + i, p.L - 1);
                    lse[i] = LSE[hrow + qi[i]];
                    if constexpr (!OWN_D) Dq[i] = Drow[hrow + qi[i]];
                }
                f32x4 of[C];
                if constexpr (OWN_D) load_row<D>(of, O + qrow * D, g);
                // requested with the rows: one memory round trip per item
                float gt[C][4], qt[C][4];
                if constexpr (!VISIBLE_ONLY) {
                    load_columns<D>(gt, dO + hrow * D, qi, m);
                    load_columns<D>(qt, Q + hrow * D, qi, m);
                }
                const f32x4 s = row_product<D>(qf, kf), dp = row_product<D>(gf, vf);
                if constexpr (OWN_D) {  // as in dq_tile, handed to the lanes that hold the row's scores
                    float Di = 0.f;
#pragma unroll
                    for (int c = 0; c < C; ++c)
#pragma unroll
                        for (int e = 0; e < 4; ++e) Di = fmaf(gf[c][e], of[c][e], Di);
                    Di = group_sum(Di);
#pragma unroll
                    for (int i = 0; i < 4; ++i) Dq[i] = __shfl(Di, 4 * g + i);
                }
                f32x4 pr, ds;
                bool vis[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int q = q0 + 4 * g + i;
                    vis[i] = j <= q && q <= hi;
                    pr[i] = vis[i] ? expf(s[i] * p.scale - lse[i]) : 0.f;
                    ds[i] = vis[i] ? pr[i] * (dp[i] - Dq[i]) : 0.f;
                }
                if constexpr (VISIBLE_ONLY) {
                    add_visible<D>(av, pr, vis, dO + hrow * D, qi, m, g);
                    add_visible<D>(ak, ds, vis, Q + hrow * D, qi, m, g);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int c = 0; c < C; ++c) av[c] = mfma_f32(gt[c][i], pr[i], av[c]);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int c = 0; c < C; ++c) ak[c] = mfma_f32(qt[c][i], ds[i], ak[c]);
                }
            }
        };
        run(IntC<0>{});
        if (any_nan(av) || any_nan(ak)) run(IntC<1>{});
    };
    // sum over the waves of x (dK or dV of the tile's 16 keys), handed out as out(row, column, four values)
    auto add_waves = [&](const f32x4 (&x)[C], auto out) __attribute__((always_inline)) {
        __syncthreads();
#pragma unroll
        for (int c = 0; c < C; ++c) *reinterpret_cast<f32x4 *>(&xs[wave][m][16 * c + 4 * g]) = x[c];
        __syncthreads();
        for (int e = threadIdx.x; e < kT * D / 4; e += 64 * kWaves) {
            const int r = e / (D / 4), col = (e % (D / 4)) * 4;
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < kWaves; ++w) v += *reinterpret_cast<const f32x4 *>(&xs[w][r][col]);
            out(r, col, v);
        }
    };

    if (unit >= wpg) {  // band unit
        const int j0 = (unit - wpg) * kT, j = j0 + m, jc = min(j, p.L - 1);
        const bool valid = j < p.L && far_index(fl, prefix, jc) < 0;
        if (__ballot(valid) == 0ull) return;
        const int end = dend ? min(dend[jc], p.L) : p.L;
        const int n_qb = (min(p.L, j0 + kT + p.n - 1) - j0 + kT - 1) / kT;
        run_items(0, G * n_qb, j0, n_qb, j, valid, end, false);
        auto finish = [&](float *dst, float f) {
            return [=](int r, int col, f32x4 v) {
                if (j0 + r < p.L && far_index(fl, prefix, j0 + r) < 0)
                    *reinterpret_cast<f32x4 *>(dst + (kvrow0 + j0 + r) * D + col) = v * f;
            };
        };
        add_waves(ak, finish(dK, p.scale));
        add_waves(av, finish(dV, 1.f));
        return;
    }

    const int NFT = (fl.NF + kT - 1) / kT;
    // lane t of a group of 64 list tiles: first query block and number of items of tile t
    auto tile_items = [&](int t, int &fq) {
        fq = 0;
        if (t >= NFT) return 0;
        fq = far_pos(fl, t * kT, idx, p.L) & ~(kT - 1);
        return max(0, G * ((far_last_query(fl, t * kT, idx, p, dend, kT) - fq + kT - 1) / kT));
    };
    // the first group of 64 list tiles (all of them up to 1024 list entries) is worked out once for both passes
    int fq, nq = tile_items(lane, fq), inc = lanes_scan(nq);
    long total = __shfl(inc, 63);
    for (int t0 = 64; t0 < NFT; t0 += 64) {
        int unused;
        total += __shfl(lanes_scan(tile_items(t0 + lane, unused)), 63);
    }
    const long least = total >> 31 ? total / pl.min_slice : (long)quotient((int)total, pl.by_min_slice);
    const long slices = min((long)wpg, max(1l, least));
    if (unit >= slices || total == 0) return;
    // slice u is [u total / slices, (u + 1) total / slices); u < slices <= wpg
    const long whole = quotient(total, slices), over = total - whole * slices;
    const float by_slices = reciprocal((int)slices), by_total = reciprocal((int)min(total, (long)kSmallQuotient));
    auto slice_start = [&](long u) { return u * whole + (u * over < kSmallQuotient ? (long)small_quotient((int)(u * over), by_slices) : u * over / slices); };
    const long s0 = slice_start(unit), s1 = slice_start(unit + 1);
    auto slice_of = [&](long item) {  // the slice that holds an item
        const long x = (item + 1) * slices - 1;
        return (int)(x < kSmallQuotient ? (long)small_quotient((int)x, by_total) : quotient(x, total));
    };
    long cum = 0;
    for (int t0 = 0; t0 < NFT && cum < s1; t0 += 64) {
        if (t0 > 0) {
            nq = tile_items(t0 + lane, fq);
            inc = lanes_scan(nq);
        }
        unsigned long long pend = __ballot(nq > 0 && cum + inc > s0 && cum + inc - nq < s1);
        for (; pend; pend &= pend - 1) {
            const int src = __ffsll(pend) - 1, ft = t0 + src, items = __shfl(nq, src), q_lo = __shfl(fq, src);
            const long F = cum + __shfl(inc, src) - items;  // the tile's first item
            const int f = ft * kT + m;
            const bool valid = f < fl.NF;
            const int j = valid ? far_pos(fl, f, idx, p.L) : 0;
            const int end = dend ? min(dend[j], p.L) : p.L;
            __syncthreads();  // the tile before has been written out
            if (threadIdx.x < kT) js[m] = j;
            uint64_t *const word = OWN_D ? reinterpret_cast<uint64_t *>(static_cast<char *>(counters) + ((long)bkv * n_far_tiles + ft) * word_stride) : nullptr;
            uint64_t seen = 0;
            if constexpr (OWN_D) {
                if (threadIdx.x == 0) seen = arrival_seen(word);
            }
            run_items((int)(max(s0, F) - F), (int)(min(s1, F + items) - F), q_lo, quotient(items, pl.by_g), j, valid, end, true);
            // slices w0 .. w1 hold the tile
            const int w0 = slice_of(F), w1 = slice_of(F + items - 1);
            auto to_row = [&](float *dst, float fac) {
                return [=](int r, int col, f32x4 v) {
                    if (ft * kT + r < fl.NF)
                        *reinterpret_cast<f32x4 *>(dst + (kvrow0 + js[r]) * D + col) = v * fac;
                };
            };
            if (w0 == w1) {
                add_waves(ak, to_row(dK, p.scale));
                add_waves(av, to_row(dV, 1.f));
                continue;
            }
            // slot: [dK rows | dV rows] of 16 keys
            float *slots = partials + (long)bkv * (wpg + n_far_tiles) * (2 * kT * D);
            auto slot_of = [=](int w, int which) { return slots + ((long)(w + ft) * 2 + which) * (kT * D); };
            auto to_slot = [&](int which) {
                float *dst = slot_of(unit, which);
                return [=](int r, int col, f32x4 v) {
                    publish(dst + r * D + col, float2{v[0], v[1]});
                    publish(dst + r * D + col + 2, float2{v[2], v[3]});
                };
            };
            add_waves(ak, to_slot(0));
            add_waves(av, to_slot(1));
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's part of the slot is where every XCD sees it
            __syncthreads();
            if constexpr (OWN_D) {
                if (threadIdx.x == 0) {
                    arrival_ready(word, seen, one, w1 - w0 + 1);
                    last_s = arrives_last(word, one, w1 - w0 + 1);
                    if (last_s) arrival_reset(word);
                }
            } else {
                if (threadIdx.x == 0) last_s = atomicAdd(static_cast<int32_t *>(counters) + (long)bkv * n_far_tiles + ft, 1) == w1 - w0;
            }
            __syncthreads();
            if (!last_s) continue;
            for (int e = threadIdx.x; e < kT * D / 4; e += 64 * kWaves) {
                const int r = e / (D / 4), col = (e % (D / 4)) * 4;
                f32x4 v[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
                constexpr int NB = 8;  // slots requested together, dK and dV
                for (int w = w0; w <= w1; w += NB) {
                    float2 x[NB][2], y[NB][2];
#pragma unroll
                    for (int k = 0; k < NB; ++k)
#pragma unroll
                        for (int which = 0; which < 2; ++which) {
                            const float *src = slot_of(min(w + k, w1), which) + r * D + col;
                            x[k][which] = fetch_published(src), y[k][which] = fetch_published(src + 2);
                        }
#pragma unroll
                    for (int k = 0; k < NB; ++k)
                        if (w + k <= w1)
#pragma unroll
                            for (int which = 0; which < 2; ++which)
                                v[which] += f32x4{x[k][which].x, x[k][which].y, y[k][which].x, y[k][which].y};
                }
                to_row(dK, p.scale)(r, col, v[0]);
                to_row(dV, 1.f)(r, col, v[1]);
            }
        }
        cum += __shfl(inc, 63);
    }
}

// dQ by itself, with D_i for the dK/dV kernel, whose counters it clears too
template <int D, bool HW>
__global__ __launch_bounds__(64 * kWaves, D == 64 ? 4 : 2) void dq_fp32_kernel(
    sepattn_params p, const float *__restrict__ Q, const float *__restrict__ K, const float *__restrict__ V, const float *__restrict__ O,
    const float *__restrict__ LSE, const float *__restrict__ dO, const int32_t *__restrict__ sep_idx,
    const int32_t *__restrict__ sep_prefix, const int32_t *__restrict__ doc_start, const int32_t *__restrict__ doc_end,
    float *__restrict__ dQ, float *__restrict__ Dws, int32_t *__restrict__ counters, long n_counters, Fp32Plan pl, HeadArgs<HW> ha) {
    __shared__ float xs[kWaves][kT][D + 4];
    for (long c = (long)blockIdx.x * (64 * kWaves) + threadIdx.x; c < n_counters; c += (long)gridDim.x * (64 * kWaves)) counters[c] = 0;
    dq_tile<D, HW>(xs, blockIdx.x, p, Q, K, V, O, LSE, dO, sep_idx, sep_prefix, doc_start, doc_end, dQ, Dws, pl, ha);
}
// MERGED: the blocks behind the dK/dV units are dQ tiles (see fp32_one_launch).
template <int D, bool HW, bool MERGED>
__global__ __launch_bounds__(64 * kWaves, D == 64 ? 2 : 1) void dkv_fp32_kernel(
    sepattn_params p, const float *__restrict__ Q, const float *__restrict__ K, const float *__restrict__ V, const float *__restrict__ O,
    const float *__restrict__ LSE, const float *__restrict__ dO, const float *__restrict__ Drow, const int32_t *__restrict__ sep_idx,
    const int32_t *__restrict__ sep_prefix, const int32_t *__restrict__ doc_start, const int32_t *__restrict__ doc_end,
    float *__restrict__ dQ, float *__restrict__ dK, float *__restrict__ dV, float *__restrict__ partials, void *__restrict__ counters,
    int n_far_tiles, int wpg, int word_stride, uint64_t one, int n_units, Fp32Plan pl, HeadArgs<HW> ha) {
    __shared__ float xs[kWaves][kT][D + 4];
    if (MERGED && (int)blockIdx.x >= n_units)
        dq_tile<D, HW>(xs, blockIdx.x - n_units, p, Q, K, V, O, LSE, dO, sep_idx, sep_prefix, doc_start, doc_end, dQ, nullptr, pl, ha);
    else
        dkv_unit<D, HW, MERGED>(xs, p, Q, K, V, O, LSE, dO, Drow, sep_idx, sep_prefix, doc_end, dK, dV, partials, counters, n_far_tiles, wpg,
                                word_stride, one, pl, ha);
}

}  // namespace

size_t backward_fp32_workspace(const sepattn_params &p) { return fp32_workspace(p).total; }

static Fp32Plan fp32_plan(const sepattn_params &p) {
    Fp32Plan pl;
    pl.n_tiles = (p.L + kT - 1) / kT;
    pl.G = p.Hq / p.Hkv;
    pl.min_slice = (int)(pl.G * (long)pl.n_tiles / kMaxShare > kMinItems ? pl.G * (long)pl.n_tiles / kMaxShare : kMinItems);
    pl.by_tiles = fast_div((uint32_t)pl.n_tiles);
    pl.by_hq = fast_div((uint32_t)p.Hq);
    pl.by_g = fast_div((uint32_t)pl.G);
    pl.by_bkv = fast_div((uint32_t)(p.B * p.Hkv));
    pl.by_hkv = fast_div((uint32_t)p.Hkv);
    pl.by_min_slice = fast_div((uint32_t)pl.min_slice);
    return pl;
}

int launch_forward_fp32(const sepattn_params &p, const HeadWin &hw, const float *Q, const float *K, const float *V,
                        const int32_t *sep_idx, const int32_t *sep_prefix, const int32_t *doc_start,
                        const int32_t *doc_end, float *O, float *LSE, hipStream_t st) {
    const long tiles = (long)p.B * p.Hq * ((p.L + kT - 1) / kT);
    if (tiles > 0x7FFFFFFFL) return SEPATTN_ERR_SHAPE;
    auto go = [&](auto kernel, auto ha) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(64 * kWaves), 0, st, p, Q, K, V, sep_idx, sep_prefix, doc_start, doc_end, O, LSE,
                           fp32_plan(p), ha);
    };
    if (any_delta(hw)) go(p.d == 64 ? fwd_fp32_kernel<64, true> : fwd_fp32_kernel<128, true>, HeadArgs<true>{hw, {}});
    else go(p.d == 64 ? fwd_fp32_kernel<64, false> : fwd_fp32_kernel<128, false>, HeadArgs<false>{});
    return launch_status();
}

template <int D, bool HW>
int launch_backward_shape(const sepattn_params &p, const HeadArgs<HW> &ha, const float *Q, const float *K, const float *V,
                          const float *O, const float *LSE, const float *dO, const int32_t *sep_idx, const int32_t *sep_prefix,
                          const int32_t *doc_start, const int32_t *doc_end, float *dQ, float *dK, float *dV, void *ws, hipStream_t st) {
    const Fp32Workspace w = fp32_workspace(p);
    const Fp32Plan pl = fp32_plan(p);
    char *base = static_cast<char *>(ws);
    float *Dws = reinterpret_cast<float *>(base);
    int32_t *counters = reinterpret_cast<int32_t *>(base + w.d_bytes);
    float *partials = reinterpret_cast<float *>(base + w.d_bytes + w.counter_bytes);
    const long q_tiles = (long)p.B * p.Hq * pl.n_tiles, k_units = (long)p.B * p.Hkv * (w.wpg + pl.n_tiles);
    if (q_tiles > 0x7FFFFFFFL || k_units > 0x7FFFFFFFL) return SEPATTN_ERR_SHAPE;
    const dim3 block(64 * kWaves);
    const int stride = fp32_one_launch(p, w);
    if (stride && !being_captured(st)) {
        hipLaunchKernelGGL((dkv_fp32_kernel<D, HW, true>), dim3((unsigned)(k_units + q_tiles)), block, 0, st, p, Q, K, V, O, LSE, dO, nullptr, sep_idx,
                           sep_prefix, doc_start, doc_end, dQ, dK, dV, partials, Dws, w.n_far_tiles, w.wpg, stride, launch_number(), (int)k_units, pl, ha);
        return launch_status();
    }
    hipLaunchKernelGGL((dq_fp32_kernel<D, HW>), dim3((unsigned)q_tiles), block, 0, st, p, Q, K, V, O, LSE, dO, sep_idx, sep_prefix, doc_start,
                       doc_end, dQ, Dws, counters, w.n_counters, pl, ha);
    if (hipGetLastError() != hipSuccess) return SEPATTN_ERR_HIP;
    hipLaunchKernelGGL((dkv_fp32_kernel<D, HW, false>), dim3((unsigned)k_units), block, 0, st, p, Q, K, V, O, LSE, dO, Dws, sep_idx, sep_prefix,
                       doc_start, doc_end, dQ, dK, dV, partials, counters, w.n_far_tiles, w.wpg, 0, 0ull, (int)k_units, pl, ha);
    return launch_status();
}

int launch_backward_fp32(const sepattn_params &p, const HeadWin &hw, const float *Q, const float *K, const float *V,
                         const float *O, const float *LSE, const float *dO, const int32_t *sep_idx,
                         const int32_t *sep_prefix, const int32_t *doc_start, const int32_t *doc_end, float *dQ,
                         float *dK, float *dV, void *ws, hipStream_t st) {
    auto go = [&](auto launch, auto ha) {
        return launch(p, ha, Q, K, V, O, LSE, dO, sep_idx, sep_prefix, doc_start, doc_end, dQ, dK, dV, ws, st);
    };
    if (any_delta(hw)) return go(p.d == 64 ? launch_backward_shape<64, true> : launch_backward_shape<128, true>, HeadArgs<true>{hw, {}});
    return go(p.d == 64 ? launch_backward_shape<64, false> : launch_backward_shape<128, false>, HeadArgs<false>{});
}

}  // namespace sepattn
