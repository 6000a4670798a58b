// SepAttention backward of small calls (bf16): dQ and dK/dV side by side in one launch.
//
// dK/dV needs of dQ only -D_i and LSE_i*log2(e).  Where the query tiles are few, the dQ kernel leaves most of the chip idle for as
// long as its chain of round trips and its few key tiles take, and dK/dV, as short, waits for it.  Here a kernel of its own
// forms the row values first (row_values_kernel: the bytes of O and dO, once), and the next launch holds the workgroups of both:
// first those of dK/dV, whose chains are the longer ones, then those of dQ, which find the row values there and need no
// rows of O.  The sums and their order are those of the separate kernels, so the results are the same bits up to where dK/dV is
// cut: its slices follow the number of workgroups that dQ leaves it.
// Bounds: the latency of its chains (row values -> a unit's or slice's rows and tiles -> its steps -> partials).  The backward at 8/2 heads,
// L = 600, n = 96, d = 128: 27.1 us with two launches (in a trace, which adds a few tenths to each kernel: dQ 11.3, dK/dV 12.1, sum of the parts
// 5.1), 20.6 here (row values 2.7, this 13.5, sum 5.2).
#pragma once

#include "bwd_dq.h"
#include "bwd_dkv.h"

namespace sepattn {

namespace {

// -D_i and LSE_i*log2(e) of all rows: four lanes per row, sixteen rows per wave, as dq_work forms them.
template <int D>
__global__ __launch_bounds__(256) void row_values_kernel(long rows, const uint16_t *__restrict__ O, const float *__restrict__ LSE,
                                                         const uint16_t *__restrict__ dO, float *__restrict__ Dws, float *__restrict__ Lws) {
    constexpr int CB = D / 32;  // 64-byte blocks of a row
    const int lane = threadIdx.x & 63;
    const long row = ((long)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16 + (lane >> 2), at = min(row, rows - 1);
    const char *ob = reinterpret_cast<const char *>(O + at * D) + 16 * (lane & 3), *dob = reinterpret_cast<const char *>(dO + at * D) + 16 * (lane & 3);
    u32x4 o4[CB], do4[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        o4[cb] = *reinterpret_cast<const u32x4 *>(ob + 64 * cb);
        do4[cb] = *reinterpret_cast<const u32x4 *>(dob + 64 * cb);
    }
    const float lse = LSE[at];
    float part = 0.f;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) part += bf16_dot8(do4[cb], o4[cb]);
    part += __shfl_xor(part, 1);
    part += __shfl_xor(part, 2);
    if ((lane & 3) == 0 && row < rows) {
        Dws[row] = -part;
        Lws[row] = lse * kLog2e_f;
    }
}

struct JointPlan {
    int n_kv, kv_wpg, dq_wpg, n_band, split;  // dK/dV workgroups, in all and per (batch, KV head); dQ workgroups per group
    FastDiv by_gx, by_dq_wpg;
};
template <int D, int GP, bool DOCS, bool PARTS>
__global__ __launch_bounds__(256, 2) void bwd_joint_kernel(
    sepattn_params p, const uint16_t *__restrict__ Q, const uint16_t *__restrict__ K, const uint16_t *__restrict__ V,
    const float *__restrict__ LSE, const uint16_t *__restrict__ dO, const int32_t *__restrict__ sep_idx,
    const int32_t *__restrict__ sep_prefix, const int32_t *__restrict__ doc_start, const int32_t *__restrict__ doc_end,
    uint16_t *__restrict__ dQ, uint16_t *__restrict__ dK, uint16_t *__restrict__ dV, float *__restrict__ Dws, float *__restrict__ Lws,
    float *__restrict__ farK, float *__restrict__ farV, int32_t *__restrict__ piece_tab, JointPlan jp, QueryGrid qg, DkvSlices sl) {
    union Lds {
        DqLds<D, 4, DOCS> q;
        DkvLds<D, 2> kv;
    };
    __shared__ Lds lds;
    const int id = blockIdx.x;
    if (id < jp.n_kv) {
        const int w = quotient(id, sl.by_bkv);
        dkv_work<D, DOCS, false, 2, PARTS>(lds.kv, id - w * (p.B * p.Hkv), w, p, Q, K, V, Lws, dO, Dws, sep_idx, sep_prefix, doc_end, dK, dV, farK, farV,
                                           piece_tab, jp.kv_wpg, jp.n_band, jp.split, sl, HeadArgs<false>{});
    } else {
        // gx x dq_wpg x groups/gx, the first dimension fastest, as in the grid of dq_kernel
        const int t = id - jp.n_kv, r = quotient(t, jp.by_gx), z = quotient(r, jp.by_dq_wpg);
        dq_work<D, GP, DOCS, 4, false, false, true>(lds.q, t - r * qg.gx + qg.gx * z, r - z * jp.dq_wpg, p, Q, K, V, nullptr, LSE, dO, sep_idx, sep_prefix,
                                                    doc_start, doc_end, dQ, Dws, Lws, nullptr, 0, jp.dq_wpg, qg, HeadArgs<false>{});
    }
}

template <int D>
int launch_joint(const sepattn_params &p, int dq_wpg, const uint16_t *Q, const uint16_t *K, const uint16_t *V, const uint16_t *O, const float *LSE,
                 const uint16_t *dO, const int32_t *sep_idx, const int32_t *sep_prefix, const int32_t *doc_start, const int32_t *doc_end,
                 uint16_t *dQ, uint16_t *dK, uint16_t *dV, float *Dws, float *Lws, float *farK, float *farV, int32_t *piece_tab, hipStream_t st) {
    const QueryShape shape = query_shape(p);
    const long n_groups = (long)p.B * (p.Hq / shape.gp), n_dq = n_groups * dq_wpg, n_bkv = (long)p.B * p.Hkv, rows = (long)p.B * p.Hq * p.L;
    const QueryGrid qg = query_grid(p, shape.gp, n_groups);
    JointPlan jp;
    jp.kv_wpg = joint_dkv_workgroups(p, dq_wpg);
    jp.n_kv = (int)(n_bkv * jp.kv_wpg);
    jp.dq_wpg = dq_wpg;
    jp.split = band_split(p, jp.kv_wpg, 2);
    jp.n_band = (p.L + 63) / 64 * jp.split;
    jp.by_gx = fast_div((uint32_t)qg.gx);
    jp.by_dq_wpg = fast_div((uint32_t)dq_wpg);
    const DkvSlices sl = dkv_slices(p, 2, jp.kv_wpg, jp.split, false);
    {
        ProfScope prof(SEPATTN_K_BWD_DQ, st);
        hipLaunchKernelGGL((row_values_kernel<D>), dim3((unsigned)((rows + 63) / 64)), dim3(256), 0, st, rows, O, LSE, dO, Dws, Lws);
    }
    {
        ProfScope prof(SEPATTN_K_BWD_DKV, st);
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3((unsigned)(jp.n_kv + n_dq)), dim3(256), 0, st, p, Q, K, V, LSE, dO, sep_idx, sep_prefix, doc_start, doc_end, dQ, dK,
                               dV, Dws, Lws, farK, farV, piece_tab, jp, qg, sl);
        };
        auto pick = [&](auto GP_) {
            constexpr int GP = decltype(GP_)::value;
            if (doc_start) jp.split > 1 ? go(bwd_joint_kernel<D, GP, true, true>) : go(bwd_joint_kernel<D, GP, true, false>);
            else jp.split > 1 ? go(bwd_joint_kernel<D, GP, false, true>) : go(bwd_joint_kernel<D, GP, false, false>);
        };
        if (shape.gp == 4) pick(IntC<4>{});
        else if (shape.gp == 2) pick(IntC<2>{});
        else pick(IntC<1>{});
    }
    if (hipGetLastError() != hipSuccess) return SEPATTN_ERR_HIP;
    return launch_dkv_combine_bf16(p, sep_idx, sep_prefix, doc_end, dK, dV, farK, farV, piece_tab, jp.kv_wpg, jp.split, st);
}

}  // namespace

}  // namespace sepattn
