// Separator marking and compaction (integer kernels).
//
// mark:    is_sep[t] = token_ids[t] in S, S = the caller's separator id set (Sec. 4.1 "Parameter
//          Setting").  One thread per four tokens, the id set travels in the kernel arguments.
// compact: the index form of the separator part of mask M (Eq. 2): ascending separator positions,
//          their count and the exclusive prefix count per sequence.  Two passes over chunks of
//          2048 tokens: (1) per-chunk separator counts, (2) each chunk sums the counts of the
//          chunks before it, ranks its own separators with wave ballots + a block prefix sum over
//          the per-wave counts, and writes prefix / index entries.  No atomics, so the output
//          order is the position order by construction.  Sequences of up to 32768 tokens take
//          one launch: pass (2) then counts the flags of the earlier chunks itself.
// mark + compact in one launch (sequences of up to 8192 tokens): pass (2) reads the token ids, tests
//          them against the id set itself and also writes the marker bitmap; at these sizes each
//          of the two kernels lasts no longer than its launch.
#include "common.h"

namespace sepattn {

__global__ __launch_bounds__(256) void mark_kernel(const int32_t *__restrict__ ids, long n,
                                                   SepIdSet set, uint8_t *__restrict__ out) {
    long t4 = ((long)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (t4 >= n) return;
    if (t4 + 4 <= n) {
        int4 v = *reinterpret_cast<const int4 *>(ids + t4);
        unsigned f0 = 0, f1 = 0, f2 = 0, f3 = 0;
        for (int k = 0; k < set.n; ++k) {
            int s = set.ids[k];
            f0 |= (v.x == s);
            f1 |= (v.y == s);
            f2 |= (v.z == s);
            f3 |= (v.w == s);
        }
        *reinterpret_cast<uint32_t *>(out + t4) = f0 | (f1 << 8) | (f2 << 16) | (f3 << 24);
    } else {
        for (long t = t4; t < n; ++t) {
            unsigned f = 0;
            for (int k = 0; k < set.n; ++k) f |= (ids[t] == set.ids[k]);
            out[t] = (uint8_t)f;
        }
    }
}

int launch_mark(const int32_t *token_ids, long n_tokens, const SepIdSet &set, uint8_t *is_sep,
                hipStream_t st) {
    long threads = (n_tokens + 3) / 4;
    unsigned blocks = (unsigned)((threads + 255) / 256);
    ProfScope prof(SEPATTN_K_MARK, st);
    hipLaunchKernelGGL(mark_kernel, dim3(blocks), dim3(256), 0, st, token_ids, n_tokens, set, is_sep);
    return launch_status();
}

// Fixed-interval variant ("FixLLM", the appendix on the fixed-interval variant): one token in every
// `delta` is marked instead of the separators: position j of every sequence iff j % delta == phase.
__global__ __launch_bounds__(256) void mark_interval_kernel(int L, long n, int delta, int phase,
                                                            uint8_t *__restrict__ out) {
    const long t4 = ((long)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (t4 >= n) return;
    int r = (int)((t4 % L) % delta);  // residue of the first of this thread's four positions
    int j = (int)(t4 % L);
    unsigned f[4];
    for (int k = 0; k < 4; ++k) {
        f[k] = (r == phase);
        ++j;
        r = (r + 1 == delta) ? 0 : r + 1;
        if (j == L) {  // next sequence
            j = 0;
            r = 0;
        }
    }
    if (t4 + 4 <= n) {
        *reinterpret_cast<uint32_t *>(out + t4) = f[0] | (f[1] << 8) | (f[2] << 16) | (f[3] << 24);
    } else {
        for (int k = 0; t4 + k < n; ++k) out[t4 + k] = (uint8_t)f[k];
    }
}

int launch_mark_interval(int B, int L, int delta, int phase, uint8_t *is_sep, hipStream_t st) {
    const long n = (long)B * L, threads = (n + 3) / 4;
    const unsigned blocks = (unsigned)((threads + 255) / 256);
    ProfScope prof(SEPATTN_K_MARK_INTERVAL, st);
    hipLaunchKernelGGL(mark_interval_kernel, dim3(blocks), dim3(256), 0, st, L, n, delta, phase, is_sep);
    return launch_status();
}

// ---- compaction --------------------------------------------------------------------------------
// Bounds: the launch and one round trip of loads; nothing here comes near the memory's rate.  Sixteen waves per chunk, so that
// a thread has two tokens of its own and at most six in front of the chunk, all requested together, and one barrier in
// all.  Kernel time in us, before (four waves, eight tokens per thread, three or four barriers, one scalar load per id) /
// now: mark and compact of 600 tokens 5.8 / 5.3, 8 x 2048 7.2 / 6.1, 3 x 3077 9.5 / 6.7, 8192 8.8 / 7.3;
// compaction alone of 8192 flags 7.2 / 4.9.
constexpr int kCompactThreads = 1024;
constexpr int kCompactSingleLaunch = 32768;  // longest sequence compacted with one launch
constexpr int kMarkCompactSingleLaunch = 8192;  // longest sequence marked and compacted with one launch
constexpr int kCompactIters = kCompactChunk / kCompactThreads;  // ballots per wave per chunk
constexpr int kCompactWaves = kCompactThreads / kWave;
constexpr int kCompactGroups = kCompactIters * kCompactWaves;  // a ballot each, in position order
static_assert(kCompactGroups + kCompactWaves <= kWave, "the counts are added with one per lane");

// pass 1: chunk_counts[b, chunk] = number of separators in the chunk
__global__ __launch_bounds__(kCompactThreads) void compact_count_kernel(
    const uint8_t *__restrict__ is_sep, int L, int n_chunks, int32_t *__restrict__ chunk_counts) {
    __shared__ int wave_cnt[kCompactWaves];
    int b = blockIdx.y, chunk = blockIdx.x;
    const uint8_t *row = is_sep + (long)b * L;
    int base = chunk * kCompactChunk;
    int cnt = 0;
    for (int it = 0; it < kCompactIters; ++it) {
        int j = base + it * kCompactThreads + threadIdx.x;
        bool f = (j < L) && row[j] != 0;
        cnt += __popcll(__ballot(f));
    }
    int wave = threadIdx.x / kWave;
    if (threadIdx.x % kWave == 0) wave_cnt[wave] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        int s = 0;
        for (int w = 0; w < kCompactWaves; ++w) s += wave_cnt[w];
        chunk_counts[(long)b * n_chunks + chunk] = s;
    }
}

// What the list holds behind its last separator: left alone, or set to `value`
struct ListRest {
    bool set;
    int32_t value;
};

// pass 2: ranks and writes.  FUSED: the flags are not read from is_sep but formed from the token ids
// (and written to marks_out for the chunk's own positions); chunk_counts is nullptr then.
template <bool FUSED>
__global__ __launch_bounds__(kCompactThreads) void compact_write_kernel(
    const uint8_t *__restrict__ is_sep, const int32_t *__restrict__ token_ids, SepIdSet set,
    uint8_t *__restrict__ marks_out, int L, int n_chunks, const int32_t *__restrict__ chunk_counts,
    int32_t *__restrict__ sep_idx, int cap, int32_t *__restrict__ sep_count,
    int32_t *__restrict__ sep_prefix, ListRest rest) {
    __shared__ int part[kCompactGroups + kCompactWaves];  // counts of the chunk's groups; of what each wave saw in front of it
    const int b = blockIdx.y, chunk = blockIdx.x, tid = threadIdx.x;
    const int base = chunk * kCompactChunk;
    const int lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);

    // the flags of the thread's own tokens, and the number of separators it finds in the earlier chunks of the sequence: from
    // the counts of pass 1, or (short sequences, single launch) counted here
    bool flag[kCompactIters];
    int early = 0;
    if constexpr (FUSED) {
        // token q * kCompactThreads + tid, from the sequence's first to the chunk's own ones.  The id set (padded by the host
        // with ids of its own) is walked in the outer loop, eight ids per scalar load; a token's matches are
        // collected as a bit and counted once, so that an id given twice does not count twice.
        constexpr int kTokens = kMarkCompactSingleLaunch / kCompactThreads;
        static_assert(SEPATTN_MAX_SEP_IDS % 8 == 0, "ids are read eight at a time");
        const int32_t *row = token_ids + (long)b * L;
        const int own = chunk * kCompactIters;
        int v[kTokens];
#pragma unroll
        for (int q = 0; q < kTokens; ++q)
            if (q < own + kCompactIters) v[q] = row[min(q * kCompactThreads + tid, L - 1)];
        uint32_t hit = 0;
        for (int k0 = 0; k0 < set.n; k0 += 8) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int sid = set.ids[k0 + k];
#pragma unroll
                for (int q = 0; q < kTokens; ++q)
                    if (q < own + kCompactIters) hit |= (uint32_t)(v[q] == sid) << q;
            }
        }
        early = __popc(hit & ((1u << own) - 1u));
#pragma unroll
        for (int it = 0; it < kCompactIters; ++it) {
            const int j = base + it * kCompactThreads + tid;
            flag[it] = j < L && ((hit >> (own + it)) & 1u);
            if (j < L) marks_out[(long)b * L + j] = flag[it] ? 1 : 0;
        }
    } else {
        const uint8_t *row = is_sep + (long)b * L;
#pragma unroll
        for (int it = 0; it < kCompactIters; ++it) {
            const int j = base + it * kCompactThreads + tid;
            flag[it] = j < L && row[j] != 0;
        }
        if (chunk_counts != nullptr) {
            for (int c = tid; c < chunk; c += kCompactThreads) early += chunk_counts[(long)b * n_chunks + c];
        } else if ((reinterpret_cast<uintptr_t>(row) & 3u) == 0) {  // base is a multiple of 4
            for (int j = tid * 4; j < base; j += kCompactThreads * 4) {
                const uint32_t w = *reinterpret_cast<const uint32_t *>(row + j);
                // one bit per non-zero byte
                early += __popc((((w & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | w) & 0x80808080u);
            }
        } else {
            for (int j = tid; j < base; j += kCompactThreads) early += row[j] != 0;
        }
    }
    for (int off = 32; off > 0; off >>= 1) early += __shfl_xor(early, off);
    if (lane == 0) part[kCompactGroups + wave] = early;
    const unsigned long long lt_mask = (1ull << lane) - 1ull;
    int rank_in_wave[kCompactIters];
#pragma unroll
    for (int it = 0; it < kCompactIters; ++it) {
        const unsigned long long m = __ballot(flag[it]);
        rank_in_wave[it] = __popcll(m & lt_mask);
        if (lane == 0) part[it * kCompactWaves + wave] = __popcll(m);
    }
    __syncthreads();
    // every wave: inclusive sums over the groups (position order), then over what lies in front of the chunk
    const int v = lane < kCompactGroups + kCompactWaves ? part[lane] : 0;
    int incl = v;
    for (int off = 1; off < kWave; off <<= 1) {
        const int t = __shfl_up(incl, off);
        if (lane >= off) incl += t;
    }
    const int chunk_base = __builtin_amdgcn_readlane(incl, kWave - 1) - __builtin_amdgcn_readlane(incl, kCompactGroups - 1);
    int32_t *list = sep_idx + (long)b * cap;
#pragma unroll
    for (int it = 0; it < kCompactIters; ++it) {
        const int g = it * kCompactWaves + wave, j = base + it * kCompactThreads + tid;
        const int group_base = chunk_base + __builtin_amdgcn_readlane(incl - v, g);  // in front of the branch: lane g may lie past L
        if (j < L) {
            const int r = group_base + rank_in_wave[it];
            if (sep_prefix) sep_prefix[(long)b * (L + 1) + j] = r;
            // token j is separator r, or one of the others, j - r of which lie in front of it: these take the entries behind
            // the list's last, from L - 1 downwards, so that nobody needs to know how long the list is
            const int e = flag[it] ? r : L - 1 - (j - r);
            if (e < cap && (flag[it] || rest.set)) list[e] = flag[it] ? j : rest.value;
            if (j == L - 1) {
                const int total = r + (flag[it] ? 1 : 0);
                if (sep_prefix) sep_prefix[(long)b * (L + 1) + L] = total;
                sep_count[b] = total;
            }
        }
    }
    if (rest.set)
        for (long e = (long)L + chunk * kCompactThreads + tid; e < cap; e += (long)n_chunks * kCompactThreads) list[e] = rest.value;
}

int launch_compact(const uint8_t *is_sep, int B, int L, int32_t *sep_idx, int cap,
                   int32_t *sep_count, int32_t *sep_prefix, int32_t *chunk_counts, const int32_t *fill, hipStream_t st) {
    int n_chunks = (L + kCompactChunk - 1) / kCompactChunk;
    dim3 grid(n_chunks, B);
    // Up to kCompactSingleLaunch positions a workgroup counts the separators in front of its chunk
    // itself (at most that many flag bytes, read once more): one launch instead of two, which matters
    // because at these sizes the kernels last no longer than their launch.
    const bool single = L <= kCompactSingleLaunch;
    if (!single) {
        ProfScope prof(SEPATTN_K_COMPACT_COUNT, st);
        hipLaunchKernelGGL(compact_count_kernel, grid, dim3(kCompactThreads), 0, st, is_sep, L, n_chunks,
                           chunk_counts);
        if (hipGetLastError() != hipSuccess) return SEPATTN_ERR_HIP;
    }
    ProfScope prof(SEPATTN_K_COMPACT_WRITE, st);
    hipLaunchKernelGGL(compact_write_kernel<false>, grid, dim3(kCompactThreads), 0, st, is_sep, nullptr, SepIdSet{},
                       nullptr, L, n_chunks, single ? nullptr : chunk_counts, sep_idx, cap, sep_count, sep_prefix,
                       ListRest{fill != nullptr, fill ? *fill : 0});
    return launch_status();
}

// marking and compaction together: one launch for sequences of up to kMarkCompactSingleLaunch tokens
// (a workgroup then tests the ids in front of its chunk once more to count them), the separate
// kernels beyond
int launch_mark_compact(const int32_t *token_ids, int B, int L, const SepIdSet &set, uint8_t *is_sep,
                        int32_t *sep_idx, int cap, int32_t *sep_count, int32_t *sep_prefix,
                        int32_t *chunk_counts, const int32_t *fill, hipStream_t st) {
    if (L > kMarkCompactSingleLaunch) {
        int rc = launch_mark(token_ids, (long)B * L, set, is_sep, st);
        if (rc != SEPATTN_OK) return rc;
        return launch_compact(is_sep, B, L, sep_idx, cap, sep_count, sep_prefix, chunk_counts, fill, st);
    }
    int n_chunks = (L + kCompactChunk - 1) / kCompactChunk;
    ProfScope prof(SEPATTN_K_MARK_COMPACT, st);
    hipLaunchKernelGGL(compact_write_kernel<true>, dim3(n_chunks, B), dim3(kCompactThreads), 0, st, nullptr, token_ids,
                       set, is_sep, L, n_chunks, nullptr, sep_idx, cap, sep_count, sep_prefix,
                       ListRest{fill != nullptr, fill ? *fill : 0});
    return launch_status();
}

}  // namespace sepattn
