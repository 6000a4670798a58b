// SepAttention backward, dK and dV (bf16 MFMA): the analytic gradient of Eq. 1 under the mask of Eq. 2,
//   dV_j = sum_i P_ij dO_i,   dK_j = scale sum_i dS_ij Q_i,   dS_ij = P_ij (<dO_i, V_j> - D_i),
//   P_ij = exp(scale <Q_i, K_j> - LSE_i),  summed over the query heads of the KV head.
//
// The visible pairs split into band pairs (i-j < n) and far pairs (i-j >= n, j an initial token or a
// separator, Sec. 3.1).  dkv_kernel runs persistent workgroups, `wpg` per (batch, KV head), each of
// which works through
//   its far pieces: far pairs on the COMPACTED list of such keys.  For list tile ft (128 or 64 consecutive
//              list entries, gathered K/V rows) the work is the sequence of items (query tile of 64 or 32
//              rows, query head) from the first query that sees the tile's first key to the end of
//              the sequence; the items of all list tiles, concatenated, are cut into slices, up to
//              one per workgroup, and the part of a slice inside one list tile is a piece.  A piece
//              writes an fp32 partial dK/dV of the tile's rows to the workspace (slot w + ft).
//   its band units: 128 or 64 consecutive keys against the queries j <= i < j+n (units w, w+wpg, ...).
//              Keys that are not on the far list are finished here (rounded once to bf16); for the
//              others the band unit writes one more fp32 partial.
// dkv_combine_kernel then adds, in fixed order, the partials of every far-list key and rounds once to
// bf16.  One workgroup owns each partial row: no atomics, results are bit-reproducible.  Every
// workgroup gets (up to one) the same number of band units, and those with one less get more far work, so
// the compute units finish together.
// A workgroup is KW = 4 or 2 (dkv_key_blocks) key blocks of 32 keys x 2 roles = 8 or 4 waves.  The two waves of a key block split
// the four contractions so that each keeps only one operand matrix and one accumulator resident:
//   P-wave :  S = Q K^T   -> P = exp2(.)      -> dV^T += dO^T P     (holds K rows, dV^T)
//   dS-wave:  dP = dO V^T -> dS = P (dP - D)  -> dK^T += Q^T dS     (holds V rows, dK^T)
// P travels from the first to the second through a small LDS buffer (same lane, same register:
// both are 32x32 accumulator layouts), once per block of 32 queries, fenced by the block's
// workgroup barrier (P is exchanged in bf16, the form it has in the second contraction anyway).  Query
// tiles (64 or 32 rows of Q and dO, plus LSE*log2e and -D) stream through a ring of four LDS buffers filled
// by direct global->LDS loads, issued in the step in which a buffer becomes free; with the ring the block barriers
// are the only barriers.  The tiles are stored unpadded with XOR-permuted 16-byte
// chunks so that both the row-major reads (first contraction) and the transposed reads (second
// contraction) are free of bank conflicts.  The G query heads of a KV head are just G times as many
// query tiles.
#include "bwd_dkv.h"

namespace sepattn {

namespace {

template <int D, bool DOCS, bool HW, int KW, bool PARTS>
__global__ __launch_bounds__(128 * KW, KW == 4 ? 1 : (D == 64 ? 3 : 2)) void dkv_kernel(
    sepattn_params p, const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K,
    const uint16_t *__restrict__ V, const float *__restrict__ LSE2, const uint16_t *__restrict__ dO,
    const float *__restrict__ Dws, const int32_t *__restrict__ sep_idx,
    const int32_t *__restrict__ sep_prefix, const int32_t *__restrict__ doc_end,
    uint16_t *__restrict__ dK, uint16_t *__restrict__ dV,
    float *__restrict__ farK, float *__restrict__ farV, int32_t *__restrict__ piece_tab, int wpg, int n_band,
    int split, DkvSlices sl, HeadArgs<HW> ha) {
    __shared__ DkvLds<D, KW> lds;
    dkv_work<D, DOCS, HW, KW, PARTS>(lds, blockIdx.x, blockIdx.y, p, Q, K, V, LSE2, dO, Dws, sep_idx, sep_prefix, doc_end, dK, dV, farK, farV, piece_tab,
                                     wpg, n_band, split, sl, ha);
}

// Sum of the partials of every far-list key (the far pieces of its list tile in ascending workgroup
// order, then the band partial), rounded once to bf16.  One thread per (key, 4 consecutive columns).  Bounds: the chain
// list length -> list entry -> piece table -> partials, then their bytes.  The list's length is on the device and
// its capacity is that of all keys: a grid for an eighth of the capacity, which walks on where there are more
// entries, starts an eighth of the workgroups that only find out that they have nothing to do.
template <int D, int KW, bool HW>
__global__ __launch_bounds__(256) void dkv_combine_kernel(sepattn_params p, const int32_t *__restrict__ sep_idx,
                                                          const int32_t *__restrict__ sep_prefix,
                                                          const int32_t *__restrict__ doc_end,
                                                          uint16_t *__restrict__ dK, uint16_t *__restrict__ dV,
                                                          const float *__restrict__ farK,
                                                          const float *__restrict__ farV,
                                                          const int32_t *__restrict__ piece_tab, int wpg,
                                                          DkvSlices sl, HeadArgs<HW> ha) {
    constexpr int TPR = D / 4, RPB = 256 / TPR;  // threads per row, rows per workgroup
    constexpr int kw = KW;
    int bkv = HW ? blockIdx.y : blockIdx.x;
    const int row_block = HW ? blockIdx.x : blockIdx.y, row_blocks = HW ? gridDim.x : gridDim.y;
    long base = bkv * far_geom(p, wpg, kw).rows;
    bool every_key = sl.every_key != 0;
    if constexpr (HW) {  // as in dkv_kernel
        ShareOf s;
        s.b = quotient(bkv, sl.by_hkv);
        s.pos = bkv - s.b * p.Hkv;
        bkv = s.b * p.Hkv + ha.share.group[s.pos];
        base = shared_part_row(far_geom(p, wpg, kw), ha.share, s, p);
        wpg = ha.share.first[s.pos + 1] - ha.share.first[s.pos];
        every_key = ha.share.all[s.pos] != 0;
        p.n -= ha.of_group((bkv - s.b * p.Hkv) * sl.G, sl.G);
    }
    if (every_key) p.n = 0;
    const int b = quotient(bkv, sl.by_hkv), kv = bkv - b * p.Hkv;
    const int32_t *prefix = sep_prefix + (long)b * (p.L + 1);
    const int32_t *idx = sep_idx + (long)b * p.cap;
    const FarGeom fg = far_geom(p, wpg, kw);
    const FarList fl = far_list(p, prefix, every_key);
    const int col = (threadIdx.x % TPR) * 4;
    constexpr int lt = 32 * KW;  // entries per list tile
    const int32_t *dend = doc_end ? doc_end + (long)b * p.L : nullptr;
    for (int f = row_block * RPB + threadIdx.x / TPR; f < fl.NF; f += row_blocks * RPB) {
        // everything that does not depend on a loaded value is requested before the first use
        const int ft = f / lt;
        const int32_t *tab = piece_tab + ((long)bkv * fg.NFTcap + ft) * 2;
        const int t0 = tab[0], t1 = tab[1];
        const long brow = (base + (long)fg.NP * lt + f) * D + col;
        float4 bk = {0.f, 0.f, 0.f, 0.f}, bv = {0.f, 0.f, 0.f, 0.f};
        if (!every_key) {
            bk = *reinterpret_cast<const float4 *>(farK + brow);
            bv = *reinterpret_cast<const float4 *>(farV + brow);
        }
        const int j = far_pos(fl, f, idx, p.L);
        // no far piece for this list tile: the band unit has written the row
        if (far_first_query(fl, f, idx, p, lt) >= far_last_query(fl, f, idx, p, dend, lt)) continue;
        // the clamps keep a table that the far pass did not write (it always does) from faulting
        const int w0 = min(max(t0, 0), wpg - 1), w1 = min(max(t1, w0), wpg - 1);
        float4 sk = {0.f, 0.f, 0.f, 0.f}, sv = {0.f, 0.f, 0.f, 0.f};
        // eight pieces at a time (clamped slots) are requested together, so that a list tile with up to eight
        // pieces costs one memory round trip; the sum runs in slot order
        constexpr int NB = 8;
        for (int w = w0; w <= w1; w += NB) {
            float4 pk[NB], pv[NB];
#pragma unroll
            for (int c = 0; c < NB; ++c) {
                const int ww = min(w + c, w1);
                const long prow = (base + (long)(ww + ft) * lt + (f - ft * lt)) * D + col;
                pk[c] = *reinterpret_cast<const float4 *>(farK + prow);
                pv[c] = *reinterpret_cast<const float4 *>(farV + prow);
            }
#pragma unroll
            for (int c = 0; c < NB; ++c) {
                if (w + c <= w1) {
                    sk.x += pk[c].x, sk.y += pk[c].y, sk.z += pk[c].z, sk.w += pk[c].w;
                    sv.x += pv[c].x, sv.y += pv[c].y, sv.z += pv[c].z, sv.w += pv[c].w;
                }
            }
        }
        sk.x += bk.x, sk.y += bk.y, sk.z += bk.z, sk.w += bk.w;
        sv.x += bv.x, sv.y += bv.y, sv.z += bv.z, sv.w += bv.w;
        const long orow = (((long)b * p.Hkv + kv) * (long)p.L + j) * D + col;
        *reinterpret_cast<uint2 *>(dK + orow) = pack_bf16x4(sk.x, sk.y, sk.z, sk.w);
        *reinterpret_cast<uint2 *>(dV + orow) = pack_bf16x4(sv.x, sv.y, sv.z, sv.w);
    }
}

// The same where band units are split among workgroups (band_split): every key is finished here, from the parts of its band
// unit and, if it is on the list, its far pieces.
template <int D, int KW>
__global__ __launch_bounds__(256) void dkv_combine_parts_kernel(sepattn_params p, const int32_t *__restrict__ sep_idx,
                                                                const int32_t *__restrict__ sep_prefix,
                                                                const int32_t *__restrict__ doc_end,
                                                                uint16_t *__restrict__ dK, uint16_t *__restrict__ dV,
                                                                const float *__restrict__ farK,
                                                                const float *__restrict__ farV,
                                                                const int32_t *__restrict__ piece_tab, int wpg,
                                                                int split, FastDiv by_hkv) {
    constexpr int TPR = D / 4, RPB = 256 / TPR;  // threads per row, rows per workgroup
    constexpr int kw = KW;
    const int bkv = blockIdx.x, b = quotient(bkv, by_hkv);
    const FarGeom fg = far_geom(p, wpg, kw, split);
    const int32_t *prefix = sep_prefix + (long)b * (p.L + 1);
    const int32_t *idx = sep_idx + (long)b * p.cap;
    const int32_t *dend = doc_end ? doc_end + (long)b * p.L : nullptr;
    constexpr int lt = 32 * KW;
    const int j = blockIdx.y * RPB + threadIdx.x / TPR, col = (threadIdx.x % TPR) * 4;
    if (j >= p.L) return;
    const long row0 = bkv * fg.rows;
    float4 sk = {0.f, 0.f, 0.f, 0.f}, sv = {0.f, 0.f, 0.f, 0.f};
    // `count` partial rows `step` rows apart from `first` on, NB at a time (the last one again past the end), in order
    auto request = [&](auto NB_, long first, long step, int h, int count, auto &x, auto &y) __attribute__((always_inline)) {
        constexpr int NB = decltype(NB_)::value;
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            const long at = (first + min(h + c, count - 1) * step) * D + col;
            x[c] = *reinterpret_cast<const float4 *>(farK + at);
            y[c] = *reinterpret_cast<const float4 *>(farV + at);
        }
    };
    auto add = [&](auto NB_, int h, int count, const auto &x, const auto &y) __attribute__((always_inline)) {
        constexpr int NB = decltype(NB_)::value;
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            if (h + c < count) {
                sk.x += x[c].x, sk.y += x[c].y, sk.z += x[c].z, sk.w += x[c].w;
                sv.x += y[c].x, sv.y += y[c].y, sv.z += y[c].z, sv.w += y[c].w;
            }
        }
    };
    // the parts are in flight while the far pieces are found (two more round trips)
    const long part0 = row0 + (long)(fg.NP + j / lt * split) * lt + j % lt;
    const IntC<4> four;
    const IntC<8> eight;
    float4 bk[4], bv[4], x[8], y[8];
    request(four, part0, lt, 0, split, bk, bv);
    const FarList fl = far_list(p, prefix);
    const int f = far_index(fl, prefix, j);
    if (f >= 0) {
        const int ft = f / lt;
        const int32_t *tab = piece_tab + ((long)bkv * fg.NFTcap + ft) * 2;
        const int t0 = tab[0], t1 = tab[1];
        if (far_first_query(fl, f, idx, p, lt) < far_last_query(fl, f, idx, p, dend, lt)) {
            // the clamps keep a table that the far pass did not write (it always does) from faulting
            const int w0 = min(max(t0, 0), wpg - 1), n = min(max(t1, w0), wpg - 1) - w0 + 1;
            for (int h = 0; h < n; h += 8) {
                request(eight, row0 + (long)(w0 + ft) * lt + (f - ft * lt), lt, h, n, x, y);
                add(eight, h, n, x, y);
            }
        }
    }
    add(four, 0, split, bk, bv);
    for (int h = 4; h < split; h += 4) {
        request(four, part0, lt, h, split, bk, bv);
        add(four, h, split, bk, bv);
    }
    const long orow = ((long)bkv * p.L + j) * D + col;
    *reinterpret_cast<uint2 *>(dK + orow) = pack_bf16x4(sk.x, sk.y, sk.z, sk.w);
    *reinterpret_cast<uint2 *>(dV + orow) = pack_bf16x4(sv.x, sv.y, sv.z, sv.w);
}

// adds the partials that a dK/dV launch with these slices has left
template <int D, int KW>
int launch_combine(const sepattn_params &p, const HeadWin &hw, bool headwise, const int32_t *sep_idx, const int32_t *sep_prefix,
                   const int32_t *doc_end, uint16_t *dK, uint16_t *dV, const float *farK, const float *farV, const int32_t *piece_tab,
                   int wpg, int split, bool any_all, const DkvSlices &sl, const WorkShare &share, hipStream_t st) {
    ProfScope prof(SEPATTN_K_BWD_COMBINE, st);
    const FarGeom fg = far_geom(p, wpg, KW);
    const int rows_per_block = 256 / (D / 4);
    const int list_rows = split > 1 ? p.L : any_all ? fg.NFcap : (fg.NFcap + 7) / 8;
    // (batch, KV head) first: with eight KV heads, or a multiple, a head's partials lie in the L2 of the XCD that has written them
    // (32/8 heads, L = 8192, n = 256 13.8 -> 10.9 us, packed from eight documents 14.4 -> 11.6, other counts level).  Head-wise calls, where a
    // few heads have most of the rows, spread a head's rows over the XCDs (12.4; 17 the other way).
    const int row_blocks = (list_rows + rows_per_block - 1) / rows_per_block;
    const dim3 grid = headwise ? dim3(row_blocks, p.B * p.Hkv) : dim3(p.B * p.Hkv, row_blocks < 65535 ? row_blocks : 65535);
    auto go = [&](auto kernel, auto ha) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, p, sep_idx, sep_prefix, doc_end, dK, dV, farK, farV, piece_tab, wpg, sl, ha);
    };
    if (split > 1)
        hipLaunchKernelGGL((dkv_combine_parts_kernel<D, KW>), grid, dim3(256), 0, st, p, sep_idx, sep_prefix, doc_end, dK, dV, farK, farV, piece_tab, wpg, split, sl.by_hkv);
    else if (headwise) go(dkv_combine_kernel<D, KW, true>, HeadArgs<true>{hw, share});
    else go(dkv_combine_kernel<D, KW, false>, HeadArgs<false>{});
    return launch_status();
}

template <int D, int KW>
int launch_dkv_shape(const sepattn_params &p, const HeadWin &hw, bool headwise, const uint16_t *Q, const uint16_t *K,
                     const uint16_t *V, const float *lse2, const uint16_t *dO, const float *Dws, const int32_t *sep_idx,
                     const int32_t *sep_prefix, const int32_t *doc_end, uint16_t *dK, uint16_t *dV, float *farK,
                     float *farV, int32_t *piece_tab, int wpg, int split, const WorkShare &share, hipStream_t st) {
    const int n_band = (p.L + 32 * KW - 1) / (32 * KW) * split;
    bool any_all = share.all[0] != 0;  // some KV head works through the list of all keys
    for (int i = 1; i < share.n; ++i) any_all = any_all || share.all[i] != 0;
    const DkvSlices sl = dkv_slices(p, KW, wpg, split, !headwise && any_all);
    {
        const dim3 block(128 * KW), grid = headwise ? dim3((unsigned)(p.B * share.first[share.n])) : dim3((unsigned)(p.B * p.Hkv), (unsigned)wpg);
        ProfScope prof(SEPATTN_K_BWD_DKV, st);
        auto go = [&](auto kernel, auto ha) {
            hipLaunchKernelGGL(kernel, grid, block, 0, st, p, Q, K, V, lse2, dO, Dws, sep_idx, sep_prefix, doc_end, dK, dV, farK, farV, piece_tab, wpg,
                               n_band, split, sl, ha);
        };
        const HeadArgs<false> none;
        if (doc_end && split == 1) go(dkv_kernel<D, true, false, KW, false>, none);
        else if (headwise) go(dkv_kernel<D, false, true, KW, false>, HeadArgs<true>{hw, share});
        else if (split == 1) go(dkv_kernel<D, false, false, KW, false>, none);
        else if (doc_end) go(dkv_kernel<D, true, false, KW, true>, none);
        else go(dkv_kernel<D, false, false, KW, true>, none);
    }
    if (hipGetLastError() != hipSuccess) return SEPATTN_ERR_HIP;
    return launch_combine<D, KW>(p, hw, headwise, sep_idx, sep_prefix, doc_end, dK, dV, farK, farV, piece_tab, wpg, split, any_all, sl, share, st);
}

template <int D>
int launch_dkv(const sepattn_params &p, const HeadWin &hw, bool headwise, const uint16_t *Q, const uint16_t *K, const uint16_t *V,
               const float *lse2, const uint16_t *dO, const float *Dws, const int32_t *sep_idx,
               const int32_t *sep_prefix, const int32_t *doc_end, uint16_t *dK, uint16_t *dV, float *farK,
               float *farV, int32_t *piece_tab, hipStream_t st) {
    const int kw = dkv_key_blocks(p, doc_end != nullptr);
    const int wpg = dkv_workgroups_per_head(p, kw);
    const FarGeom fg = far_geom(p, wpg, kw);
    if ((long)wpg * p.B * p.Hkv > 0x7FFFFFFFL) return SEPATTN_ERR_SHAPE;
    WorkShare share = {};
    const bool list_all = !doc_end && list_of_all_keys(p, kw, wpg, fg, headwise);
    if (headwise) {
        const int G = p.Hq / p.Hkv;
        // pairs multiplied, and the start of a piece as 320 / G queries
        share = share_out(p, hw, G, wpg * p.Hkv, [](int) { return kIntMax; }, [&](int n, bool all) {
            const double L = p.L, out = L - n;
            return all && list_all ? L * L / 2 : n * (L - n / 2.) + L * (fg.bk + 320. / G) + kSepShare * out * out / 2;
        });
        if (!list_all)
            for (int i = 0; i < share.n; ++i) share.all[i] = 0;
    } else {
        share.all[0] = list_all && p.n >= p.L;
    }
    const int split = headwise || share.all[0] ? 1 : band_split(p, wpg, kw);
    // the eight-wave shape exists for d = 128 only (dkv_key_blocks)
    auto go = [&](auto launch) {
        return launch(p, hw, headwise, Q, K, V, lse2, dO, Dws, sep_idx, sep_prefix, doc_end, dK, dV, farK, farV, piece_tab, wpg, split, share, st);
    };
    if (D == 128 && kw == 4) return go(launch_dkv_shape<128, 4>);
    return go(launch_dkv_shape<D, 2>);
}

}  // namespace

int launch_dkv_combine_bf16(const sepattn_params &p, const int32_t *sep_idx, const int32_t *sep_prefix, const int32_t *doc_end,
                            uint16_t *dK, uint16_t *dV, const float *farK, const float *farV, const int32_t *piece_tab, int wpg, int split,
                            hipStream_t st) {
    const DkvSlices sl = dkv_slices(p, 2, wpg, split, false);
    const HeadWin hw = {};
    const WorkShare share = {};
    auto go = [&](auto launch) {
        return launch(p, hw, false, sep_idx, sep_prefix, doc_end, dK, dV, farK, farV, piece_tab, wpg, split, false, sl, share, st);
    };
    return p.d == 64 ? go(launch_combine<64, 2>) : go(launch_combine<128, 2>);
}

int launch_dkv_bf16(const sepattn_params &p, const HeadWin &hw, const uint16_t *Q, const uint16_t *K, const uint16_t *V,
                    const float *lse2, const uint16_t *dO, const float *Dws, const int32_t *sep_idx,
                    const int32_t *sep_prefix, const int32_t *doc_end, uint16_t *dK, uint16_t *dV, float *farK,
                    float *farV, int32_t *piece_tab, hipStream_t st) {
    const bool headwise = any_delta(hw);
    if (p.d == 64)
        return launch_dkv<64>(p, hw, headwise, Q, K, V, lse2, dO, Dws, sep_idx, sep_prefix, doc_end, dK, dV, farK, farV, piece_tab, st);
    return launch_dkv<128>(p, hw, headwise, Q, K, V, lse2, dO, Dws, sep_idx, sep_prefix, doc_end, dK, dV, farK, farV, piece_tab, st);
}

}  // namespace sepattn
