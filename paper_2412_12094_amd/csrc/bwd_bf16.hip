// SepAttention backward, bf16 MFMA: the analytic gradient of Eq. 1 under the mask of Eq. 2.
//
//   D_i = <dO_i, O_i>,  P_ij = exp(scale*<Q_i,K_j> - LSE_i),  dP_ij = <dO_i, V_j>,
//   dS_ij = P_ij (dP_ij - D_i),  dQ_i = scale sum_j dS_ij K_j,  dK_j = scale sum_i dS_ij Q_i,
//   dV_j = sum_i P_ij dO_i   (dK, dV summed over the query heads of the KV head).
//
// Three launches, no floating-point atomics (results are bit-reproducible; a small call has 1. and 2. side by side in one launch behind a
// kernel that forms -D_i and LSE_i*log2(e) of all rows: bwd_joint.h, joint_dq_workgroups):
//  1. dq_kernel (this file; its work: bwd_dq.h): persistent workgroups over the query tiles, same dense key stream as the forward
//     [initial | separators older than the window | band].  Also writes -D_i and LSE_i*log2(e).
//     (Where few tiles have long streams, these go in two parts to two workgroups and dq_parts_kernel adds their
//     fp32 sums: see split_tiles.)
//  2. dkv_kernel (bwd_dkv_bf16.hip; its work: bwd_dkv.h): the visible pairs split into band pairs (i-j < n) and far
//     pairs (i-j >= n, j an initial token or a separator); far units work on the COMPACTED list of
//     such keys and write fp32 partials, band units finish the keys that are not on that list.
//  3. dkv_combine_kernel: adds, in fixed order, the partials of every far-list key and rounds once.
#include "bwd_dkv.h"
#include "bwd_dq.h"

namespace sepattn {

namespace {

template <int D, int GP, bool DOCS, int NW, bool PARTS, bool HW>
__global__ __launch_bounds__(64 * NW, 2) void dq_kernel(
    sepattn_params p, const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K,
    const uint16_t *__restrict__ V, const uint16_t *__restrict__ O, const float *__restrict__ LSE,
    const uint16_t *__restrict__ dO, const int32_t *__restrict__ sep_idx,
    const int32_t *__restrict__ sep_prefix, const int32_t *__restrict__ doc_start,
    const int32_t *__restrict__ doc_end, uint16_t *__restrict__ dQ, float *__restrict__ Dws,
    float *__restrict__ Lws, float *__restrict__ parts, int part_keys, int wpg, QueryGrid qg, HeadArgs<HW> ha) {
    __shared__ DqLds<D, NW, DOCS> lds;
    dq_work<D, GP, DOCS, NW, PARTS, HW, false>(lds, blockIdx.x + (HW ? 0 : qg.gx * blockIdx.z), blockIdx.y, p, Q, K, V, O, LSE, dO, sep_idx, sep_prefix,
                                               doc_start, doc_end, dQ, Dws, Lws, parts, part_keys, wpg, qg, ha);
}

// dQ of the query tiles whose streams went in two parts (see split_tiles): the sum of the parts, rounded once.  One workgroup
// per tile and column block; thread = lane of the dq kernel's wave.  Bounds: the bytes of the parts.
template <int D, int GP, int NW>
__global__ __launch_bounds__(64 * NW) void dq_parts_kernel(sepattn_params p, const float *__restrict__ parts, uint16_t *__restrict__ dQ,
                                                           int part_keys, HeadWin hw) {
    constexpr int TP = 32 * NW / GP, DB = D / 32;
    const int G = p.Hq / p.Hkv, groups = G / GP, n_pos_tiles = (p.L + TP - 1) / TP;
    const int tile = blockIdx.x / DB, db = blockIdx.x % DB, y = blockIdx.y;
    const int hg = y % groups, kv = (y / groups) % p.Hkv, b = y / (groups * p.Hkv);
    const SplitTiles split = split_tiles(n_pos_tiles, TP, p.n - group_delta(hw, kv * G + hg * GP, GP), part_keys);
    if (tile >= split.n) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, qi = lane & 31, hh = lane >> 5;
    const float *src = parts + (((long)y * split.most + tile) * 2 * NW + wave) * (32 * D) + db * 1024 + lane * 4;
    const int row = (n_pos_tiles - 1 - tile) * TP + 32 * (wave / GP) + qi;
    float4 u[4], v[4];
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4) {
        u[i4] = *reinterpret_cast<const float4 *>(src + i4 * 256);
        v[i4] = *reinterpret_cast<const float4 *>(src + (long)NW * (32 * D) + i4 * 256);
    }
    if (row >= p.L) return;
    uint16_t *out = dQ + (((long)b * p.Hq + kv * G + hg * GP + wave % GP) * p.L + row) * D + db * 32 + 4 * hh;
#pragma unroll
    for (int i4 = 0; i4 < 4; ++i4)
        *reinterpret_cast<uint2 *>(out + 8 * i4) = pack_bf16x4(u[i4].x + v[i4].x, u[i4].y + v[i4].y, u[i4].z + v[i4].z, u[i4].w + v[i4].w);
}

template <int D, bool DOCS>
int launch_bwd(const sepattn_params &p, const uint16_t *Q, const uint16_t *K, const uint16_t *V,
               const uint16_t *O, const float *LSE, const uint16_t *dO, const int32_t *sep_idx,
               const int32_t *sep_prefix, const int32_t *doc_start, const int32_t *doc_end, uint16_t *dQ,
               uint16_t *dK, uint16_t *dV, void *ws, const HeadWin &hw, hipStream_t st) {
    const BwdWorkspace w = bwd_workspace(p);
    char *base = static_cast<char *>(ws);
    float *Dws = reinterpret_cast<float *>(base);
    float *Lws = reinterpret_cast<float *>(base + w.d_bytes);
    float *farK = reinterpret_cast<float *>(base + 2 * w.d_bytes);
    float *farV = reinterpret_cast<float *>(base + 2 * w.d_bytes + w.far_bytes);
    int32_t *piece_tab = reinterpret_cast<int32_t *>(base + 2 * w.d_bytes + 2 * w.far_bytes);

    if (const int dq_wpg = joint_dq_workgroups(p, hw, DOCS))
        return (D == 64 ? launch_joint_64 : launch_joint_128)(p, dq_wpg, Q, K, V, O, LSE, dO, sep_idx, sep_prefix, doc_start, doc_end, dQ, dK, dV, Dws, Lws,
                                                              farK, farV, piece_tab, st);
    const QueryShape shape = query_shape(p);
    const int TP = 32 * shape.nw / shape.gp;
    const int n_pos_tiles = (p.L + TP - 1) / TP;
    const long n_groups = (long)p.B * (p.Hq / shape.gp);
    // persistent workgroups, spread evenly over the groups; never more than a group has tiles, or parts of tiles
    const int per_cu = shape.nw > 4 ? 1 : 2;
    const long slots = per_cu * (long)compute_units();
    // the parts' sums lie where the dK/dV kernel puts its partials later
    const int part_keys = DOCS || shape.nw != 4 ? 0 : split_keys(p, hw, shape.gp, TP, slots, 2 * w.far_bytes / (2 * TP * shape.gp * D * sizeof(float)));
    const int n_pieces = query_pieces(p, TP, p.n, part_keys);  // of the group with the longest window
    int wpg = (int)(slots / n_groups);
    wpg = wpg < 1 ? 1 : (wpg > n_pieces ? n_pieces : wpg);
    if (n_groups * wpg > 0x7FFFFFFFL) return SEPATTN_ERR_SHAPE;
    WorkShare share = {};
    long n_wg = n_groups * wpg;
    const bool headwise = !DOCS && any_delta(hw);  // (packed calls have no windows per head)
    if (headwise) {
        share = share_queries(p, hw, shape.gp, TP, (int)(slots / p.B), part_keys);
        n_wg = (long)p.B * share.first[share.n];
    }
    const QueryGrid qg = query_grid(p, shape.gp, n_groups);
    const dim3 block(64 * shape.nw), grid = headwise ? dim3((unsigned)n_wg) : dim3((unsigned)qg.gx, (unsigned)wpg, (unsigned)(n_groups / qg.gx));
    {
    ProfScope prof(SEPATTN_K_BWD_DQ, st);
    auto go = [&](auto NW_, auto GP_, auto PARTS_) {
        constexpr int GP = decltype(GP_)::value, NW = decltype(NW_)::value;
        constexpr bool PARTS = decltype(PARTS_)::value != 0;
        auto run = [&](auto kernel, auto ha) {
            hipLaunchKernelGGL(kernel, grid, block, 0, st, p, Q, K, V, O, LSE, dO, sep_idx, sep_prefix, doc_start, doc_end, dQ, Dws, Lws, farK, part_keys, wpg, qg, ha);
        };
        if constexpr (!DOCS) {
            if (headwise) run(dq_kernel<D, GP, false, NW, PARTS, true>, HeadArgs<true>{hw, share});
        }
        if (!headwise) run(dq_kernel<D, GP, DOCS, NW, PARTS, false>, HeadArgs<false>{});
        if constexpr (PARTS)
            hipLaunchKernelGGL((dq_parts_kernel<D, GP, NW>), dim3((n_pieces - n_pos_tiles) * (D / 32), (unsigned)n_groups), block, 0, st, p, farK, dQ, part_keys, hw);
    };
    auto go4 = [&](auto GP_) {
        if constexpr (!DOCS) {
            if (part_keys) return go(IntC<4>{}, GP_, IntC<1>{});
        }
        go(IntC<4>{}, GP_, IntC<0>{});
    };
    if (shape.gp == 7) go(IntC<7>{}, IntC<7>{}, IntC<0>{});
    else if (D == 128 && shape.nw == 8) go(IntC<D == 128 ? 8 : 4>{}, IntC<4>{}, IntC<0>{});
    else if (shape.gp == 4) go4(IntC<4>{});
    else if (shape.gp == 2) go4(IntC<2>{});
    else go4(IntC<1>{});
    }
    if (hipGetLastError() != hipSuccess) return SEPATTN_ERR_HIP;
    return launch_dkv_bf16(p, hw, Q, K, V, Lws, dO, Dws, sep_idx, sep_prefix, doc_end, dK, dV, farK, farV, piece_tab, st);
}

}  // namespace

size_t backward_bf16_workspace(const sepattn_params &p) { return bwd_workspace(p).total; }

int launch_backward_bf16(const sepattn_params &p, const HeadWin &hw, const void *Q, const void *K, const void *V,
                         const void *O, const float *LSE, const void *dO, const int32_t *sep_idx,
                         const int32_t *, const int32_t *sep_prefix, const int32_t *doc_start,
                         const int32_t *doc_end, void *dQ, void *dK, void *dV, void *ws, hipStream_t st) {
    auto u = [](const void *x) { return static_cast<const uint16_t *>(x); };
    auto w = [](void *x) { return static_cast<uint16_t *>(x); };
    if (doc_start) {
        if (p.d == 64)
            return launch_bwd<64, true>(p, u(Q), u(K), u(V), u(O), LSE, u(dO), sep_idx, sep_prefix, doc_start, doc_end,
                                        w(dQ), w(dK), w(dV), ws, hw, st);
        return launch_bwd<128, true>(p, u(Q), u(K), u(V), u(O), LSE, u(dO), sep_idx, sep_prefix, doc_start, doc_end,
                                     w(dQ), w(dK), w(dV), ws, hw, st);
    }
    if (p.d == 64)
        return launch_bwd<64, false>(p, u(Q), u(K), u(V), u(O), LSE, u(dO), sep_idx, sep_prefix, nullptr, nullptr,
                                     w(dQ), w(dK), w(dV), ws, hw, st);
    return launch_bwd<128, false>(p, u(Q), u(K), u(V), u(O), LSE, u(dO), sep_idx, sep_prefix, nullptr, nullptr,
                                  w(dQ), w(dK), w(dV), ws, hw, st);
}

}  // namespace sepattn
