// Internal declarations shared by the HIP sources of libsepattn (not part of the public ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "sepattn.h"

namespace sepattn {

constexpr int kWave = 64;

inline int launch_status() { return hipGetLastError() == hipSuccess ? SEPATTN_OK : SEPATTN_ERR_HIP; }
// An error that an earlier, unrelated runtime call of the caller left pending would otherwise be read
// (and blamed on this call) by the first launch_status(): every entry point discards it first.
inline void discard_stale_hip_error() { (void)hipGetLastError(); }

__host__ __device__ inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// 16-byte loads and stores with the non-temporal hint, for rows that are touched once
typedef unsigned int nt_u32x4 __attribute__((ext_vector_type(4)));
__device__ inline uint4 nt_load(const uint4 *p) {
    const nt_u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const nt_u32x4 *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ inline void nt_store(uint4 v, uint4 *p) {
    const nt_u32x4 t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, reinterpret_cast<nt_u32x4 *>(p));
}

// Element i (the same in every lane) of an array that no running kernel writes, through the scalar cache.  As an ordinary
// load it would be a vector load here (the statements that write LDS behind the compiler's back keep it from
// proving that nothing has changed), whose result is waited for behind every row load and row store in flight.
__device__ inline int load_uniform(const int32_t *__restrict__ a, int i) {
    return ((const __attribute__((address_space(4))) int32_t *)(uintptr_t)a)[__builtin_amdgcn_readfirstlane(i)];
}

// Values that pass between workgroups of one launch, which may run on different XCDs, whose L2 caches are not coherent with
// each other: stored and loaded as device-scope atomics of 8 bytes, which go past the L2 (a fence would write back all of
// it).  The publisher waits for its stores (s_waitcnt vmcnt(0)) before it counts itself in.
__device__ inline void publish(float *dst, float2 v) {
    __hip_atomic_store(reinterpret_cast<uint64_t *>(dst), __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline float2 fetch_published(const float *src) {
    return __builtin_bit_cast(float2, __hip_atomic_load(reinterpret_cast<const uint64_t *>(src), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// How many slices of one piece of work (the caches of a (sequence, KV head), a list tile) have published their records: a word in
// the caller's workspace, which nobody clears.  Each slice adds `one`, the number of this launch in the upper 56 bits and 1 in the lower 8; the last one finds
// (slices - 1) of them and sets the word to 0, so that the next launch finds it so.  Whatever else may stand there
// (memory never used for this, the sum that calls left which overlapped on one workspace) is no multiple of this
// launch's `one`: every slice looks at the word before it counts itself in and, if it saw such a value, replaces that by 0;
// if the exchange fails, another slice of this launch has done so.  Nobody waits for another workgroup.  (A word that
// every launch has to set first: 0.1 to 0.2 us more.)
__device__ inline uint64_t arrival_seen(uint64_t *word) { return __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void arrival_ready(uint64_t *word, uint64_t seen, uint64_t one, int nsplit) {
    const uint64_t n = seen & 0xFF;
    if (n >= (uint64_t)nsplit || seen != n * one)
        __hip_atomic_compare_exchange_strong(word, &seen, 0ull, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline bool arrives_last(uint64_t *word, uint64_t one, int nsplit) {
    return __hip_atomic_fetch_add(word, one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint64_t)(nsplit - 1) * one;
}
__device__ inline void arrival_reset(uint64_t *word) { __hip_atomic_store(word, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

uint64_t launch_number();  // `one` of a launch (api.hip)
// A captured launch runs with the same arguments at every replay, so it has no number of its own to count its slices under.
bool being_captured(hipStream_t st);

// number of compute units of the current device (queried once per device; 256 if the query fails)
int compute_units();

// Measurement hook: brackets launches of the selected kernel with HIP events (see sepattn.h).
void profile_mark(int kernel, hipStream_t st, bool stop);
struct ProfScope {
    int kernel;
    hipStream_t st;
    ProfScope(int k, hipStream_t s) : kernel(k), st(s) { profile_mark(kernel, st, false); }
    ~ProfScope() { profile_mark(kernel, st, true); }
};

// Division of 0 <= x < 2^31 by a number known on the host: x / d = x m >> s with s = 31 + l, l = ceil(log2 d), m = ceil(2^s / d) (m d
// exceeds 2^s by less than d <= 2^l).  Four scalar instructions; a division on the device is forty, and the start of a
// workgroup had up to eight of them.
struct FastDiv {
    uint32_t m;
    int32_t s;
};
inline FastDiv fast_div(uint32_t d) {
    int l = 0;
    while ((1ull << l) < d) ++l;
    return {(uint32_t)(((1ull << (31 + l)) + d - 1) / d), 31 + l};
}
__device__ inline int quotient(int x, FastDiv f) { return (int)(((uint64_t)(uint32_t)x * f.m) >> f.s); }
// The same with a divisor d that only the device knows, by its reciprocal (v_rcp_f32, one unit in the last place): x + 1/2 is at
// least 1/(2d) of a whole number off, and the product's relative error is below 2^-22, so this holds for 0 <= x < 2^21.
constexpr int kSmallQuotient = 1 << 21;
__device__ inline float reciprocal(int d) { return __builtin_amdgcn_rcpf((float)d); }
__device__ inline int small_quotient(int x, float rcp) { return (int)(((float)x + 0.5f) * rcp); }

// Head-wise neighbour windows (the head-wise variant of Sec. 4.6): every attention kernel is given
// p.n = the LARGEST window of the call and, by value, how much shorter each query head's own window
// is.  The key streams and the far / band split of a group of heads that share K/V tiles are those of
// the group's largest window (work_share.h); within it only the visibility test of a band key uses
// the head's own window:  key j, not an initial token or a separator, is visible to query i of head
// h iff j <= i <= j + p.n - 1 - delta[h].  All zeros for an ordinary call.
constexpr int kMaxHeadwise = SEPATTN_MAX_HEADWISE_HEADS;
struct HeadWin {
    int32_t delta[kMaxHeadwise];
};
__host__ __device__ inline int head_delta(const HeadWin &hw, int h) {
    return hw.delta[h < kMaxHeadwise ? h : kMaxHeadwise - 1];
}

// ---- integer kernels -------------------------------------------------------------------------
struct SepIdSet {
    int n;
    int ids[SEPATTN_MAX_SEP_IDS];
};
int launch_mark(const int32_t *token_ids, long n_tokens, const SepIdSet &set, uint8_t *is_sep,
                hipStream_t st);
int launch_mark_interval(int B, int L, int delta, int phase, uint8_t *is_sep, hipStream_t st);
constexpr int kCompactChunk = 2048;  // tokens per workgroup of the compaction kernels
// fill: what the entries behind a list's last separator are set to, or nullptr (left alone)
int launch_compact(const uint8_t *is_sep, int B, int L, int32_t *sep_idx, int cap, int32_t *sep_count,
                   int32_t *sep_prefix, int32_t *chunk_counts, const int32_t *fill, hipStream_t st);
int launch_mark_compact(const int32_t *token_ids, int B, int L, const SepIdSet &set, uint8_t *is_sep,
                        int32_t *sep_idx, int cap, int32_t *sep_count, int32_t *sep_prefix,
                        int32_t *chunk_counts, const int32_t *fill, hipStream_t st);

// ---- fp32 path ---------------------------------------------------------------------------------
// doc_start / doc_end: packed documents (per-position bounds [B, L]), or nullptr
int launch_forward_fp32(const sepattn_params &p, const HeadWin &hw, const float *Q, const float *K, const float *V,
                        const int32_t *sep_idx, const int32_t *sep_prefix, const int32_t *doc_start,
                        const int32_t *doc_end, float *O, float *LSE, hipStream_t st);
size_t backward_fp32_workspace(const sepattn_params &p);
int launch_backward_fp32(const sepattn_params &p, const HeadWin &hw, const float *Q, const float *K, const float *V,
                         const float *O, const float *LSE, const float *dO, const int32_t *sep_idx,
                         const int32_t *sep_prefix, const int32_t *doc_start, const int32_t *doc_end, float *dQ,
                         float *dK, float *dV, void *ws, hipStream_t st);

// ---- bf16 MFMA path ----------------------------------------------------------------------------
size_t forward_bf16_workspace(const sepattn_params &p);
// doc_start / doc_end: packed documents (per-position bounds [B, L]; p.a must be 0), or nullptr
int launch_forward_bf16(const sepattn_params &p, const HeadWin &hw, const void *Q, const void *K, const void *V,
                        const int32_t *sep_idx, const int32_t *sep_prefix, const int32_t *doc_start,
                        const int32_t *doc_end, void *O, float *LSE, void *ws, hipStream_t st);
int launch_doc_bounds(const int32_t *cu_seqlens, int n_docs, int L, int a, int32_t *doc_start, int32_t *doc_end,
                      uint8_t *is_sep, hipStream_t st);
size_t backward_bf16_workspace(const sepattn_params &p);
int launch_backward_bf16(const sepattn_params &p, const HeadWin &hw, const void *Q, const void *K, const void *V,
                         const void *O, const float *LSE, const void *dO, const int32_t *sep_idx,
                         const int32_t *sep_count, const int32_t *sep_prefix, const int32_t *doc_start,
                         const int32_t *doc_end, void *dQ, void *dK, void *dV, void *ws, hipStream_t st);

// ---- streaming cache ---------------------------------------------------------------------------
int check_kv_params(const sepkv_params *p);  // host validation shared by every cache call
size_t decode_workspace(const sepkv_params &p);
// rope: table of cos / sin by position [n_pos][2][d/2] (keys stored without position encoding), or nullptr
int launch_decode(const sepkv_params &p, const void *q, const void *Kc, const void *Vc,
                  const int32_t *sizes, const float *rope, int n_pos, void *out, float *lse, void *ws,
                  hipStream_t st);
int launch_rope_table(int n_pos, int d, double base, float *table, hipStream_t st);
int launch_cache_append(const sepkv_params &p, const void *k_new, const void *v_new, const uint8_t *is_sep_new,
                        void *Kc, void *Vc, uint8_t *win_is_sep, int32_t *sizes, hipStream_t st);
size_t evict_workspace(const sepkv_params &p);
int launch_evict(const sepkv_params &p, void *Kc, void *Vc, const uint8_t *win_is_sep, int32_t *sizes,
                 void *ws, hipStream_t st);
int launch_cache_fill(const sepkv_params &p, int L, int nw, const void *K, const void *V, const uint8_t *is_sep,
                      const int32_t *sep_idx, int cap, const int32_t *sep_prefix, void *Kc, void *Vc,
                      uint8_t *win_is_sep, int32_t *sizes, bool zero_rest, hipStream_t st);

}  // namespace sepattn
