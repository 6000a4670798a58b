// Pieces shared by the decode kernels (decode_wide.hip: bf16, up to 16 query heads per KV head; decode_mfma.hip: bf16,
// 17 to 32; decode.hip: fp32 and wider groups on the vector ALU): the map from logical cache entries to slots, and the partial record merge.
#pragma once

#include "common.h"

namespace sepattn {

// The state of one sequence's cache, read from its row of `sizes` and clamped so that no value can
// lead outside the buffers: counts of valid entries and the ring heads of the two ring regions.
//   slots [0,a) Initial Cache | [a,a+s) Separator Cache (ring) | [a+s,c) window (ring)
//   separator k (oldest first) sits in slot a + (sep_head + k) mod s,
//   window entry u (oldest first: Past Window, then Local Window) in slot a+s + (win_head + u) mod (c-a-s)
struct CacheMap {
    int n_init, n_sep, n_past, n_loc, sep_head, win_head, a, s, wcap;
};
__device__ inline CacheMap cache_map(const sepkv_params &p, const int32_t *__restrict__ sz) {
    CacheMap m;
    m.a = p.a;
    m.s = p.s;
    m.wcap = p.c - p.a - p.s;
    const int init = sz[0], sep = sz[1], past = sz[2], loc = sz[3], sep_head = sz[4], win_head = sz[5];
    m.n_init = min(max(init, 0), p.a);
    m.n_sep = min(max(sep, 0), p.s);
    m.n_past = min(max(past, 0), m.wcap);
    m.n_loc = min(max(loc, 0), m.wcap - m.n_past);
    m.sep_head = max(min(max(sep_head, 0), p.s - 1), 0);
    m.win_head = min(max(win_head, 0), m.wcap - 1);
    return m;
}
__device__ inline int sep_slot(const CacheMap &m, int k) {
    const int t = m.sep_head + k;
    return m.a + (t >= m.s ? t - m.s : t);
}
__device__ inline int win_index(const CacheMap &m, int u) {  // index into the window region (and its flag array)
    const int t = m.win_head + u;
    return t >= m.wcap ? t - m.wcap : t;
}
// logical valid entry e (oldest first over Initial, Separator, Past Window, Local Window) -> slot
__device__ inline int decode_slot_of(const CacheMap &m, int e) {
    if (e < m.n_init) return e;
    if (e < m.n_init + m.n_sep) return sep_slot(m, e - m.n_init);
    return m.a + m.s + win_index(m, e - m.n_init - m.n_sep);
}

__device__ inline uint16_t decode_f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

bool decode_mfma_applicable(const sepkv_params &p);
int decode_mfma_nsplit(const sepkv_params &p);
// rope: table of cos / sin by position [n_pos][2][d/2], or nullptr for keys that carry their encoding
int launch_decode_mfma(const sepkv_params &p, int nsplit, const uint16_t *q, const uint16_t *Kc, const uint16_t *Vc,
                       const int32_t *sizes, const float *rope, int n_pos, uint16_t *out, float *lse, float *part,
                       hipStream_t st);

bool decode_wide_applicable(const sepkv_params &p);
struct DecodeWideShape {
    int nsplit, nw;  // slices per (sequence, KV head), waves per workgroup
    bool add;        // the slices are added by decode_wide_kernel itself, not by a merge launch
};
DecodeWideShape decode_wide_shape(const sepkv_params &p, bool rope, int units);  // units: compute_units()
// where decode_wide_kernel has several slices the workspace holds one word per (sequence, KV head), in which they are counted
__host__ __device__ inline size_t decode_wide_arrival_bytes(const sepkv_params &p) { return align_up((size_t)p.S * p.Hkv * sizeof(uint64_t), 256); }
int launch_decode_wide(const sepkv_params &p, const DecodeWideShape &shape, const uint16_t *q, const uint16_t *Kc, const uint16_t *Vc,
                       const int32_t *sizes, const float *rope, int n_pos, uint16_t *out, float *lse, float *part,
                       hipStream_t st);

}  // namespace sepattn
