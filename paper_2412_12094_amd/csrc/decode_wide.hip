// Single-query attention over the four-block KV cache (Sec. 3.2 "Generation", Sec. 3.3), bf16, up to 16
// query heads per KV head: the decode kernel of every such call (more heads: decode_mfma.hip).
//
// A short cache, or one of few, is bound by the chain  sizes -> slots -> rows -> scores -> softmax -> output
// -> sum over the slices and by the instructions a wave issues along it; many long ones by the rate of the memory.  A
// workgroup owns one (sequence, KV head) and one of `nsplit` slices of its valid entries:
//   - eight waves or four (see decode_wide_shape), one block of
//     32 entries each at a time.  A wave has one LDS stage of K and V rows, filled with direct global->LDS
//     loads; the K half is refilled as soon as the scores' operands sit in registers, the V half one step
//     later, so 128 KB per compute unit are in flight nearly all the time and no workgroup barrier is needed;
//   - v_mfma_f32_16x16x32_bf16: a block's scores are 8 values per lane (16 with 32-column operands), the
//     output 4 registers per 16 dimensions, the merge records half as many;
//   - a row's slot is worked out once per row (lane r has row r's) and handed to the lanes that fetch it with
//     ds_bpermute, instead of once per 16-byte piece;
//   - positions within the cache (ROPE, Sec. 3.3 "Positional Encoding", Sec. 4.6): every key is turned by its
//     distance to the query, so that the query needs no turning.  Row r of a block is r entries closer than the
//     block's first, so its angle is that of the first entry's distance (one table row per block, read by all
//     lanes alike) minus that of r (rows 0 .. 31 of the table, fetched once per workgroup into LDS, kept in
//     registers); dimension i pairs with i + D/2 in another fragment of the same lane.  (Reading each row's own
//     table row from memory is 64 separate 16-byte pieces per instruction: 3.5 us per round of eight blocks.)
//   - where the slices' records are few, the workgroup of a cache that finishes last adds them (arrives_last): 1 to 2 us of
//     device-scope round trips (the records stored, the count, the records fetched: 0.4 us each), as long as a merge launch takes on the device, but a launch less on the host, which
//     costs 3 us there (append + decode of a streaming generation step, 32/8 heads, 4 sequences of 800 entries: 12.3 us -> 9.9).
// Measured (MI355X, 32/8 heads, d = 128, one call of a stream of calls, us without / with ROPE; before: four
// waves, 32-column operands, two stages per wave, the angle carried from block to block in registers):
//   1 sequence, 64 entries 5.1 / 6.7 -> 3.6 / 4.8; 800 entries 8.8 / 12.0 -> 6.1 / 7.3
//   32 sequences, 300 entries 9.5 / 13.5 -> 6.9 / 8.4; 3332 entries (436.7 MB) 67.7 / 73.1 -> 64.6 / 65.8 (6.8 TB/s)
// Since then (angles formed while the K rows are on their way, queries through LDS with ROPE, a word per cache line, records of the
// waves in their own stages): 1 sequence, 800 entries 6.5 / 7.5 -> 5.9 / 6.9; 4 sequences 6.8 / 7.8 -> 6.0 / 7.0; 3588 entries 8.7 /
// 10.5 -> 7.6 / 9.0.  Where the 13100 cycles of such a workgroup with ROPE go that adds (one block per wave, 4 sequences): sizes and
// table's requests 1050, rows' requests 700, table in registers 1200, K rows 900, turned and multiplied 1800, V 800,
// waves' records 1400, slices' records published 900, counted 1000, added 2700.
// Then: the counting word looked at while the records are on their way and set back behind the slices' maximum, at d = 64 the slices' pairs along
// rows of lanes.  Calls with slices 0.1 to 0.2 us less, at d = 64 0.3 to 0.6 (4 x 32/8 heads, 1999 entries 6.84 -> 6.43).
//
// Operand layouts of 16x16x32 (lane l, g = l / 16): A row l%16, k = 8g..8g+7; B column l%16, same k; C
// column l%16, rows 4g..4g+3.  Row 4g+i of score tile t (t = 0, 1) is row 8g+4t+i of the block, so that
// the two tiles' registers of lane group g are rows 8g..8g+7, exactly the k-slots the group holds of the
// probabilities as B operand of the output contraction: no exchange between lanes.
#include "common.h"
#include "mfma_common.h"
#include "decode_common.h"

namespace sepattn {

namespace {

constexpr int kDwRows = 32;  // entries per block (one stage of a wave)
constexpr int kDwMostAdded = 16;  // slices that the kernel itself adds, at most

__device__ inline f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

// XOR permutation of the 16-byte chunks of a row (row = 8a + 4t + i): the 16 rows (a, i) of a row-major
// A fragment hit 16 different 16-byte slots of 256 bytes, and the 8 rows (a%2, i) of half a transposed
// read 8 different 32-byte slots
template <int D>
__device__ inline int dw_swz(int row) {
    const int i = row & 3, a = row >> 3;
    if (D == 128) return (i << 1) | ((a & 1) << 3) | (a >> 1);
    return (i & 2) | ((a & 1) << 2) | (a >> 1);  // two rows per 256 bytes: row bit 0 already separates them
}

// maximum / sum over the four lane groups (lanes l, l^16, l^32, l^48)
__device__ inline float groups_max(float x) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return pair_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ inline float groups_sum(float x) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return pair_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// maximum over the eight lanes of half a row of sixteen
__device__ inline float half_row_max(float x) {
    auto with = [&](auto CTRL) {
        x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), decltype(CTRL)::value, 0xF, 0xF, true)));
    };
    with(IntC<0xB1>{});   // quad_perm [1, 0, 3, 2]
    with(IntC<0x4E>{});   // quad_perm [2, 3, 0, 1]
    with(IntC<0x141>{});  // row_half_mirror
    return x;
}

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wint-to-pointer-cast"
__device__ inline f32x4 lds_read_f4(uint32_t addr) { return *(const f32x4 __attribute__((address_space(3))) *)addr; }
#pragma clang diagnostic pop

// ADD: several slices, added by the workgroup that finishes last.  Otherwise one slice, or the records are left to a merge launch.
// The arguments fill 120 bytes, so that what the kernel reads of them, the grid's size behind them included, is two cache
// lines: a third one costs a short eager call 0.1 us.
template <int D, bool ROPE, int NW, bool ADD>
__global__ __launch_bounds__(64 * NW, D == 64 ? 4 : 2) void decode_wide_kernel(
    sepkv_params p, int G, int n_pos, const uint16_t *__restrict__ q, const uint16_t *__restrict__ Kc,
    const uint16_t *__restrict__ Vc, const int32_t *__restrict__ sizes, const float *__restrict__ rope, uint64_t one,
    float *__restrict__ part, uint16_t *__restrict__ out, float *__restrict__ lse) {
    constexpr int CH = D / 8;           // 16-byte chunks per row
    constexpr int RPL = 64 / CH;        // rows covered by one wave-wide 1 KB load
    constexpr int NLD = kDwRows / RPL;  // wave-wide loads per tensor per stage
    constexpr int KSTEPS = D / 32;
    constexpr int KS2 = KSTEPS / 2;     // dimensions of k-step ks pair with those of k-step ks + KS2
    constexpr int DB = D / 16;          // output blocks of 16 dimensions
    constexpr int TILE = kDwRows * D;
    constexpr int PF = D + 2;           // partial record: max (log2 domain), sum, D unnormalised outputs
    constexpr int RF = D + 4;           // the same in LDS, padded to whole 16-byte pieces

    __shared__ __attribute__((aligned(1024))) uint16_t smem[2][NW][TILE];  // K rows, V rows of every wave's stage

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, g = lane >> 4;
    const int nsplit = gridDim.x, split = blockIdx.x, kv = blockIdx.y, sq = blockIdx.z;
    const int h0 = kv * G;
    const uint16_t *Kh = Kc + ((long)sq * p.Hkv + kv) * (long)p.c * D;
    const uint16_t *Vh = Vc + ((long)sq * p.Hkv + kv) * (long)p.c * D;

    // Waited for only when the queries and the table's rows have been requested: those requests are up to 256 scattered pieces of 16 bytes per
    // wave, which go out during this round trip; behind it the rows queue up behind them (28/4 heads, 1 sequence of 447
    // entries 6.46 -> 6.35 us, 16/1 heads 7.75 -> 7.66)
    int32_t sz[SEPKV_SIZES_COLS];
#pragma unroll
    for (int i = 0; i < SEPKV_SIZES_COLS; ++i) sz[i] = sizes[SEPKV_SIZES_COLS * sq + i];
    // queries: B operand, column = head of the group (zero beyond G).  With ROPE fragment ks is fetched by wave ks for all waves,
    // through LDS, every lane's 16 bytes to the lane's own place: loads into registers are waited for by the compiler, which
    // does not see the row loads behind them, with all of those, while the angles could be formed.  Without ROPE there
    // is nothing to do meanwhile, and the barrier costs more than the wait (1 sequence of 384 entries 5.7 -> 6.1 us).
    const uint16_t *const qh = q + ((long)sq * p.Hq + h0) * D;
    const uint32_t q_off = (uint32_t)(min(col, G - 1) * D + 8 * g) * 2;  // of fragment 0; the next one is 64 bytes on
    __shared__ __attribute__((aligned(1024))) uint16_t q_s[ROPE ? KSTEPS : 1][ROPE ? 64 * 8 : 8];
    u32x4 qraw[KSTEPS];
    if constexpr (ROPE) {
        static_assert(KSTEPS <= NW, "one fragment per wave");
        if (wave < KSTEPS)
            dma_to_lds_16(qh, q_off + 64u * wave, lds_addr(&q_s[wave][0]));
    } else {
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) qraw[ks] = *reinterpret_cast<const u32x4 *>(reinterpret_cast<const char *>(qh) + (q_off + 64u * ks));
    }
    __builtin_amdgcn_sched_barrier(0);
    // ROPE: the table rows 0 .. 31 (cos, sin of a row's place within a block), shared by the waves, with the chunks
    // of a row permuted; and per wave the table row of the block's first entry (two, in turn)
    // four waves: the table lies over the V stages, whose first rows are requested once it has been read, so that
    // two workgroups fit a compute unit (where each has one to itself, V rows requested at once bring nothing: 6.66 us against 6.63)
    constexpr bool OVER = NW == 4;
    __shared__ __attribute__((aligned(1024))) float tab_s[ROPE && !OVER ? kDwRows * D : 4];
    __shared__ __attribute__((aligned(1024))) float base_s[ROPE ? NW : 1][ROPE ? 2 * D : 4];
    const uint32_t t_lds = OVER ? lds_addr(&smem[1][0][0]) : lds_addr(&tab_s[0]), b_lds = lds_addr(&base_s[ROPE ? wave : 0][0]);
    if constexpr (ROPE) {
        constexpr int TCH = D / 4, TRPL = 64 / TCH, TLD = kDwRows / TRPL / NW;  // chunks per row, rows and loads per wave
        static_assert(TLD >= 1 && TLD * TRPL * NW == kDwRows, "the table rows must divide among the waves");
        static_for<TLD>([&](auto U) {
            const int r = (wave * TLD + U) * TRPL + lane / TCH;
            dma_to_lds_16(rope, (uint32_t)(min(r, n_pos - 1) * D * 4) + (uint32_t)(((lane % TCH) ^ dw_swz<128>(r)) * 16),
                          t_lds + (wave * TLD + U) * 1024);
        });
        __builtin_amdgcn_sched_barrier(0);
    }
    // the word of the (sequence, KV head), and its records [head][slice].  Every word stands in front of its own records: side by
    // side the words share a few cache lines, and the counting of all caches waits in one queue (4 sequences x 8 KV heads, seven
    // slices: 0.9 to 1.4 us for the count, 0.4 now).  Records that a merge launch adds lie in one piece, behind where as many words would stand.
    const long pair = (long)sq * p.Hkv + kv, pair_bytes = (long)G * nsplit * (PF * 4);
    char *const arrived_at = reinterpret_cast<char *>(part) + pair * ((long)sizeof(uint64_t) + pair_bytes);
    uint64_t *const arrived = reinterpret_cast<uint64_t *>(arrived_at);
    char *const recs = ADD ? arrived_at + sizeof(uint64_t) : reinterpret_cast<char *>(part) + decode_wide_arrival_bytes(p) + pair * pair_bytes;
    // requested in front of the rows, by the wave with the fewest of them, and looked at while the records are on their way (requested behind
    // the rows, 0.1 us more)
    uint64_t seen = 0;
    if constexpr (ADD) {
        if (tid == 64 * (NW - 1)) seen = arrival_seen(arrived);
    }
    const CacheMap cm = cache_map(p, sz);
    const int nv = cm.n_init + cm.n_sep + cm.n_past + cm.n_loc;
    // slices of whole blocks; wave w takes blocks w, w + NW, ... of the slice
    const int nb = (nv + kDwRows - 1) / kDwRows;
    // blocks per slice, rounded up (c d < 2^30, so nb < 2^19; an integer division is on the way to the first row)
    const int share = small_quotient(nb + nsplit - 1, reciprocal(nsplit));
    const int per = (nsplit == 1 ? nb : __builtin_amdgcn_readfirstlane(share)) * kDwRows;
    const int e0 = min(split * per, nv), e1 = min(nv, e0 + per);

    const uint32_t k_lds = lds_addr(&smem[0][wave][0]), v_lds = lds_addr(&smem[1][wave][0]);
    const int my_pc = lane % CH, my_sub = lane / CH;
    // The rows of one block, in two steps (the K rows' half of the stage is free as soon as the scores' operands
    // sit in registers, the V rows' half one step later): byte offsets of the rows, the K rows (with ROPE after the
    // table row of the first entry's distance, D fp32 unpermuted: all lanes of a group read the same pieces), the V rows.
    uint32_t off[NLD];
    auto issue_keys = [&](int eb, int par) __attribute__((always_inline)) {
        const int slot = decode_slot_of(cm, min(eb + (lane & 31), e1 - 1));  // entries past the end: the last one (masked)
        static_for<NLD>([&](auto U) {
            constexpr int u = U;
            const int r = u * RPL + my_sub;
            const int sl = __builtin_amdgcn_ds_bpermute(r * 4, slot);
            off[u] = (uint32_t)sl * (uint32_t)(D * 2) + (uint32_t)((my_pc ^ dw_swz<D>(r)) * 16);
        });
        if constexpr (ROPE) {
            if (lane < D / 4) dma_to_lds_16(rope + (long)(nv - 1 - eb) * D, lane * 16, b_lds + par * D * 4);
        }
        static_for<NLD>([&](auto U) { dma_to_lds_16_nt(Kh, off[U], k_lds + U * RPL * D * 2); });
    };
    auto issue_values = [&]() __attribute__((always_inline)) {
        static_for<NLD>([&](auto U) { dma_to_lds_16_nt(Vh, off[U], v_lds + U * RPL * D * 2); });
    };
    auto wait_loads = [&](auto N) __attribute__((always_inline)) {  // at most N loads are still in flight
        constexpr int n = decltype(N)::value;
        static_assert(n == 4 || n == 5 || n == 8 || n == 9 || n == 16 || n == 17, "wait counts are written for d = 64 and 128");
        if constexpr (n == 4) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        if constexpr (n == 5) asm volatile("s_waitcnt vmcnt(5)" ::: "memory");
        if constexpr (n == 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        if constexpr (n == 9) asm volatile("s_waitcnt vmcnt(9)" ::: "memory");
        if constexpr (n == 16) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
        if constexpr (n == 17) asm volatile("s_waitcnt vmcnt(17)" ::: "memory");
    };

    const float sl2 = p.scale * kLog2e_f;
    f32x4 oacc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) oacc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = -INFINITY, l_run = 0.f;
    bf16x8 qreg[KSTEPS];

    // byte offsets of this lane's fragments in a stage: K row 8 (col/4) + col%4 (+ 4t), chunk 4 ks + g;
    // V rows 8g + p/4 (+ 4), columns 16 db + 4 (p%4) with p = lane % 16
    const int krow = 8 * (col >> 2) + (col & 3), vrow = 8 * g + (col >> 2);
    const uint32_t kswz = dw_swz<D>(krow), vswz = dw_swz<D>(vrow);  // the same for rows + 4
    const uint32_t kbase = k_lds + krow * D * 2, vbase = v_lds + vrow * D * 2 + ((col & 1) << 3);

    int eb = e0 + wave * kDwRows;
    const bool any = eb < e1;
    if (any) {
        issue_keys(eb, 0);
        if (!(ROPE && OVER)) issue_values();
    }
    // cos / sin of the lane's two rows r = krow + 4t within a block, 8 frequencies per k-step
    f32x4 rc[2][KS2][2], rs[2][KS2][2];
    if constexpr (ROPE) {
        // this wave's share of the queries and of the table (requested before its first stage) has landed
        if (any) wait_loads(IntC<(OVER ? 1 : 2) * NLD + 1>{});
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int ks = 0; ks < KS2; ++ks)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t row = t_lds + (krow + 4 * t) * D * 4, tswz = dw_swz<128>(krow);
                    rc[t][ks][h] = lds_read_f4(row + (((uint32_t)(8 * ks + 2 * g + h) ^ tswz) << 4));
                    rs[t][ks][h] = lds_read_f4(row + (((uint32_t)(D / 8 + 8 * ks + 2 * g + h) ^ tswz) << 4));
                }
        if constexpr (OVER) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            if (any) issue_values();
        }
    }
#pragma unroll
    for (int ks = 0; ks < KSTEPS; ++ks) {
        if constexpr (ROPE) qraw[ks] = *reinterpret_cast<const u32x4 *>(&q_s[ks][lane * 8]);
        qreg[ks] = as_bf16x8(col < G ? qraw[ks] : u32x4{0u, 0u, 0u, 0u});
    }

    for (int par = 0; eb < e1; eb += NW * kDwRows, par ^= 1) {
        // R(-distance): (x, y) -> (x cos + y sin, y cos - x sin), dimension i with i + D/2; the distance of row r
        // is that of the block's first entry minus r.  The angles need the block's table row only, which arrives in front of the K
        // rows, and are formed while these are on their way (d = 64 has no registers for that).
        auto base_row = [&](int ks, f32x4 (&bc)[2], f32x4 (&bs)[2]) __attribute__((always_inline)) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                bc[h] = lds_read_f4(b_lds + par * D * 4 + (8 * ks + 2 * g + h) * 16);
                bs[h] = lds_read_f4(b_lds + par * D * 4 + (D / 8 + 8 * ks + 2 * g + h) * 16);
            }
        };
        auto angle = [&](int t, int ks, int e, const f32x4 (&bc)[2], const f32x4 (&bs)[2], float &c, float &s) __attribute__((always_inline)) {
            const float c0 = bc[e >> 2][e & 3], s0 = bs[e >> 2][e & 3];
            const float cr = rc[t][ks][e >> 2][e & 3], sr = rs[t][ks][e >> 2][e & 3];
            c = fmaf(s0, sr, c0 * cr);
            s = fmaf(-c0, sr, s0 * cr);
        };
        constexpr bool EARLY = D == 128;
        float ac[2][KS2][8], as[2][KS2][8];
        if constexpr (ROPE && EARLY) {
            wait_loads(IntC<2 * NLD>{});
#pragma unroll
            for (int ks = 0; ks < KS2; ++ks) {
                f32x4 bc[2], bs[2];
                base_row(ks, bc, bs);
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int e = 0; e < 8; ++e) angle(t, ks, e, bc, bs, ac[t][ks][e], as[t][ks][e]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        wait_loads(IntC<NLD>{});  // the K rows; the V rows may be in flight
        bf16x8 ka[2][KSTEPS];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int ks = 0; ks < KSTEPS; ++ks)
                ka[t][ks] = lds_read_b128_at(kbase + 4 * t * D * 2 + (((uint32_t)(4 * ks + g) ^ kswz) << 4));
        const bool more = eb + NW * kDwRows < e1;
        if (more) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            issue_keys(eb + NW * kDwRows, par ^ 1);
        }
        if constexpr (ROPE) {
#pragma unroll
            for (int ks = 0; ks < KS2; ++ks) {
                f32x4 bc[2], bs[2];
                if constexpr (!EARLY) base_row(ks, bc, bs);
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const f32x8 x = __builtin_convertvector(ka[t][ks], f32x8), y = __builtin_convertvector(ka[t][ks + KS2], f32x8);
                    f32x8 u, v;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        float c, s;
                        if constexpr (EARLY) c = ac[t][ks][e], s = as[t][ks][e];
                        else angle(t, ks, e, bc, bs, c, s);
                        u[e] = fmaf(y[e], s, x[e] * c);
                        v[e] = fmaf(-x[e], s, y[e] * c);
                    }
                    ka[t][ks] = __builtin_convertvector(u, bf16x8);
                    ka[t][ks + KS2] = __builtin_convertvector(v, bf16x8);
                }
            }
        }
        f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KSTEPS; ++ks) {
            s0 = mfma16(ka[0][ks], qreg[ks], s0);
            s1 = mfma16(ka[1][ks], qreg[ks], s1);
        }
        if (more) wait_loads(IntC<NLD + (ROPE ? 1 : 0)>{});  // the V rows (only the next block's K rows are in flight)
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        bf16x8 va[DB];
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const uint32_t a0 = vbase + (((uint32_t)(2 * db + ((col & 3) >> 1)) ^ vswz) << 4);
            va[db] = lds_read_tr_at(a0, 4 * D * 2);
        }
        if (more) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            issue_values();
        }
        float s[8] = {s0[0], s0[1], s0[2], s0[3], s1[0], s1[1], s1[2], s1[3]};  // rows 8g .. 8g+7 of the block
        const int n_valid = e1 - eb;  // >= 1
        if (n_valid < kDwRows) {
#pragma unroll
            for (int i = 0; i < 8; ++i) s[i] = 8 * g + i < n_valid ? s[i] : -INFINITY;
        }
        float m_loc = fmaxf(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])), fmaxf(fmaxf(s[4], s[5]), fmaxf(s[6], s[7])));
        const float m_new = fmaxf(m_run, groups_max(m_loc) * sl2);  // finite: row 0 of a block is valid
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        m_run = m_new;
        float psum = 0.f;
        f32x8 pr;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            pr[i] = __builtin_amdgcn_exp2f(fmaf(s[i], sl2, -m_new));
            psum += pr[i];
        }
        l_run = l_run * alpha + psum;
        const bf16x8 pb = __builtin_convertvector(pr, bf16x8);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            oacc[db] *= alpha;
            oacc[db] = mfma16(va[db], pb, oacc[db]);
        }
    }

    // ---- merge the waves' states through LDS: D outputs, max, sum of a head.  A wave's records lie in its own stage, whose rows
    // nobody else reads: heads 0 .. 7 in the K half, the others in the V half
    const float l_tot = groups_sum(l_run);
    static_assert(8 * RF * sizeof(float) <= TILE * sizeof(uint16_t), "the records of eight heads in half a stage");
    auto record = [&](int h, int w) __attribute__((always_inline)) { return reinterpret_cast<float *>(&smem[h >> 3][w][0]) + (h & 7) * RF; };
    if (col < G) {
        float *r = record(col, wave);
        if (g == 0) *reinterpret_cast<float2 *>(r + D) = float2{m_run, l_tot};
#pragma unroll
        for (int db = 0; db < DB; ++db) *reinterpret_cast<f32x4 *>(r + 16 * db + 4 * g) = oacc[db];
    }
    __syncthreads();
    for (int item = tid; item < G * (D / 2); item += 64 * NW) {  // two columns per thread
        const int h = item / (D / 2), c2 = item % (D / 2);
        float2 ml[NW], o[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float *r = record(h, w);
            ml[w] = *reinterpret_cast<const float2 *>(r + D);
            o[w] = *reinterpret_cast<const float2 *>(r + 2 * c2);
        }
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) M = fmaxf(M, ml[w].x);
        float lsum = 0.f, o0 = 0.f, o1 = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float wgt = (ml[w].x == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(ml[w].x - M);
            lsum = fmaf(wgt, ml[w].y, lsum);
            o0 = fmaf(wgt, o[w].x, o0);
            o1 = fmaf(wgt, o[w].y, o1);
        }
        const long sh = (long)sq * p.Hq + h0 + h;
        if (!ADD && nsplit == 1) {
            const float inv = lsum > 0.f ? 1.f / lsum : 0.f;
            typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
            typedef float f32x2 __attribute__((ext_vector_type(2)));
            const f32x2 v = {lsum > 0.f ? o0 * inv : 0.f, lsum > 0.f ? o1 * inv : 0.f};
            *reinterpret_cast<bf16x2 *>(out + sh * D + 2 * c2) = __builtin_convertvector(v, bf16x2);
            if (lse && c2 == 0) lse[sh] = (lsum > 0.f) ? (M + __builtin_amdgcn_logf(lsum)) * kLn2_f : -INFINITY;
        } else {
            float *dst = reinterpret_cast<float *>(recs + (uint32_t)(h * nsplit + split) * (PF * 4));
            if constexpr (ADD) {
                publish(dst + 2 + 2 * c2, float2{o0, o1});
                if (c2 == 0) publish(dst, float2{M, lsum});
            } else {
                *reinterpret_cast<float2 *>(dst + 2 + 2 * c2) = float2{o0, o1};
                if (c2 == 0) *reinterpret_cast<float2 *>(dst) = float2{M, lsum};
            }
        }
    }
    if constexpr (!ADD) return;

    // ---- the workgroup that finishes last adds the slices' records, in slice order, whichever it is
    __shared__ int last_s;
    if (tid == 64 * (NW - 1)) arrival_ready(arrived, seen, one, nsplit);  // while the record is on its way
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's part of the record is where every XCD sees it
    __syncthreads();
    if (tid == 0) last_s = arrives_last(arrived, one, nsplit);
    // (a __syncthreads would also wait for stores)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (!last_s) return;
    // The lanes of a head (64, or 32 at d = 64) have two columns each.  Maximum and sum of slice k are fetched by lane k of the head's
    // lanes (d = 128) or of every row of sixteen (d = 64, where a wave has two heads) and handed on, as scalars or along the row:
    // fetched by every lane, they are half of the requests, whose number is what the fetch costs.  A call in us, every lane for itself / handed
    // on: d = 128, one head per KV head, 2 x 8 KV heads, 1130 entries 6.66 / 6.63, two heads 6.85 / 6.78, four (4 x 8 KV heads, 800 entries)
    // 6.71 / 6.51, seven (2 x 2 KV heads, 1400 entries) 7.36 / 7.00; d = 64, 7 x 12/12 heads, 1750 entries 9.17 / 9.11, 1 x 4/2 heads, 5200
    // entries 6.56 / 6.19 (there as scalars, two and a choice per value: 9.38, 6.83).
    // The arithmetic, and so every bit, is that of decode_merge_kernel: eight records at a time, in slice order, and exp2f, whose results
    // reach below 2^-126 where the bare instruction's end.
    static_assert(kDwMostAdded <= 16, "a slice per lane of a row of sixteen, in two batches");
    const int lk = lane % (D == 128 ? 64 : 16);
    // what lane S0 + K of this lane's head or row holds
    auto of_slice = [&](float x, auto S0, auto K) __attribute__((always_inline)) {
        if constexpr (D == 128) return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(x), S0 + K));
        else return __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x150 + S0 + K, 0xF, 0xF, false));  // row_newbcast
    };
    for (int item = tid; item < G * (D / 2); item += 64 * NW) {
        const int h = item / (D / 2), c2 = item % (D / 2);
        const uint32_t at = (uint32_t)(h * nsplit) * (PF * 4);
        float2 ml = {-INFINITY, 0.f};
        float M = -INFINITY, lsum = 0.f, o0 = 0.f, o1 = 0.f;
        // the slices s0 .. s0 + 7, those past the last as the last again with weight 0
        auto batch = [&](auto s0) __attribute__((always_inline)) {
            float2 o[8];
            auto record_at = [&](int slice) { return at + (uint32_t)(min(slice, nsplit - 1) * (PF * 4)); };
#pragma unroll
            for (int k = 0; k < 8; ++k) o[k] = fetch_published(reinterpret_cast<const float *>(recs + (record_at(s0 + k) + 8u + 8u * c2)));
            __builtin_amdgcn_sched_barrier(0);
            if (s0 == 0) {  // the last of the requests, because its answer is waited for first
                ml = fetch_published(reinterpret_cast<const float *>(recs + record_at(lk)));
                if (lk >= nsplit) ml = float2{-INFINITY, 0.f};
            }
            // (the largest of the batch is in all of its eight lanes)
            const float Mn = fmaxf(M, of_slice(half_row_max(ml.x), s0, IntC<0>{}));
            if (s0 == 0 && tid == 0) arrival_reset(arrived);  // (in front of the maximum: 0.1 us more)
            const float keep = (M == -INFINITY) ? 0.f : exp2f(M - Mn);
            lsum *= keep, o0 *= keep, o1 *= keep;
            M = Mn;
            const float wgt = (ml.x == -INFINITY) ? 0.f : exp2f(ml.x - M);  // used of the batch's lanes
            static_for<8>([&](auto KK) __attribute__((always_inline)) {
                constexpr int k = decltype(KK)::value;
                const float w = of_slice(wgt, s0, KK);
                lsum = fmaf(w, of_slice(ml.y, s0, KK), lsum);
                o0 = fmaf(w, o[k].x, o0);
                o1 = fmaf(w, o[k].y, o1);
            });
        };
        if constexpr (D == 128) {
            for (int s0 = 0; s0 < nsplit; s0 += 8) batch(s0);
        } else {  // the lane is part of the instruction
            batch(IntC<0>{});
            if (nsplit > 8) batch(IntC<8>{});
        }
        const long sh = (long)sq * p.Hq + h0 + h;
        const uint32_t b0 = decode_f32_to_bf16(lsum > 0.f ? o0 / lsum : 0.f), b1 = decode_f32_to_bf16(lsum > 0.f ? o1 / lsum : 0.f);
        *reinterpret_cast<uint32_t *>(out + sh * D + 2 * c2) = b0 | (b1 << 16);
        // (the bare logarithm: the largest slice counts with weight 1, so the sum is no denormal number)
        if (lse && c2 == 0) lse[sh] = (lsum > 0.f) ? (M + __builtin_amdgcn_logf(lsum)) * kLn2_f : -INFINITY;
    }
}

}  // namespace

bool decode_wide_applicable(const sepkv_params &p) {
    return p.dtype == SEPATTN_BF16 && (p.d == 64 || p.d == 128) && p.Hq / p.Hkv <= 16;
}

// Slices per cache, waves per workgroup, and who adds the slices.  Times below: one call of a stream of calls in us, 32/8 heads,
// d = 128, caches that are full, without / with ROPE, unless noted.
//   Slices are at most one workgroup per compute unit, four blocks each (one per wave; d = 64 with more than 32 blocks:
//     eight): the rows that one compute unit has to fetch are what a short call waits for.  1 sequence of 800 entries
//     (25 blocks): seven slices of four waves 6.8 / 7.7, four of eight with a merge launch 8.3 / 9.4; 4 sequences
//     8.0 / 8.8 against 9.0 / 10.0.  Never two workgroups on some compute units: d = 64, 32 sequences of 2300 entries,
//     one slice 22.5 / 23.0, two 24.4 / 25.1.
//   Eight slices, whose records are fetched in one round trip (1 sequence of 1400 entries: 6.7 / 8.6, eleven 7.7 / 8.8); more
//     for long caches, in proportion to the root of their length, because what a slice more costs does not depend on
//     the length and what it spares does.  16/4 heads, 3332 entries: sixteen 8.8 / 10.1, eight 9.5 / 11.7 (d = 64, whose blocks take
//     half the time: fourteen 8.2 / 8.7, eight 7.1 / 7.8); 16/2 heads, 8192 entries: thirty-two 11.2 / 12.0, sixteen 11.6 / 13.3; 16384: 13.7 /
//     14.9 and 16.4 / 18.9; 65536: sixty-four 22.8 / 24.2, thirty-two 27.8 / 31.5, sixteen 44 / 48.  With more than four pairs, whose
//     sixteen slices are half a chip, the second line lies later: 32/8 heads, 8192 entries: thirty-two 13.3 / 13.8, sixteen
//     12.4 / 13.4; 16384: 17.7 / 18.3 and 18.1 / 19.1.
//   The kernel adds the slices where their records are few, as one workgroup fetches them all, past the L2: 33 KB at the line.
//     A merge launch takes the device 0.6 us longer for three records of 4 x 128, as long for twelve, 2 us less for eight of
//     16 x 128 and 1.6 for thirty-two of 4 x 128.  16/1 heads, 3332 entries, sixteen: 14.6 / 15.9, with a merge launch 9.5 / 10.8; 16/2
//     heads 10.8 / 12.1 and 9.2 / 10.4; 32/8 heads, 16384 entries, thirty-two: 18.9 / 19.4 and 17.8 / 18.3.  It also costs the host 3 us, which
//     append + decode per token wait for: 28/4 heads, 4 sequences, caches of 1600, 13.3 us per token with eight slices added in
//     the kernel, 14.7 with a merge launch.
//   Slices pay when the blocks that a workgroup is spared take longer than adding the records (1 to 2 us; a block costs
//     a lone workgroup 0.2 us, with ROPE 0.3 us, half of that at d = 64).  The slices follow the capacity c, as only the
//     device knows how much of it is in use.  One slice / sliced, 32/8 and 28/4 heads, 1 to 6 sequences, full caches and half-full
//     ones: without ROPE 13 blocks 6.7 / 6.4 and 5.3 / 5.8, 16 blocks 7.5 / 6.5 and 5.6 / 5.9 (28/4 heads, 12 to 16 of them in use, 6.9 / 7.9), 20 blocks 8.6 / 6.6 and 6.0 / 6.0;
//     with ROPE 13 blocks 9.1 / 7.3 and 6.6 / 7.0, 20 blocks 10.1 / 7.5 and 7.8 / 7.2; d = 64: 20 blocks 5.7 / 5.4 and 4.1 / 5.1, 25 blocks
//     6.4 / 5.6 and 4.8 / 5.3.  Two or three slices of four waves have hardly more waves than the one of eight, and have to spare
//     more: two, 16 sequences of 28 blocks 13.2 / 13.9 and (0.6 full) 9.5 / 11.1, with ROPE 14.8 / 14.8 and 11.1 / 12.1, of 38 blocks with
//     ROPE 19.2 / 17.5 and 13.2 / 12.9; three, 10 sequences of 15 blocks with ROPE 9.8 / 10.1, of 19 blocks 10.9 / 10.2.
//   Four waves per slice at d = 128 (two slices for 16 sequences of 2300 entries 24.6 / 25.6, of eight waves 24.8 / 25.6)
//     and where each has one block; eight at d = 64 (8 sequences of 2300 entries 8.2 / 8.8 against 8.7 / 9.5).
//   One slice: eight waves (more bytes in flight); four for caches of up to four blocks (1 sequence of 128 entries
//     3.6 / 4.8 against 4.2 / 5.1; of eight blocks, which four waves take in two rounds, 0.14 us slower), and where more workgroups wait than the compute units hold at once: half the LDS, so
//     that two (d = 64: four) share a compute unit and one's start and merge overlap another's stream (64 sequences x
//     8 heads of 100 entries 8.9 -> 5.4, of 1000 entries 40.7 -> 39.2).
DecodeWideShape decode_wide_shape(const sepkv_params &p, bool rope, int units) {
    const long pairs = (long)p.S * p.Hkv, fit = units / pairs;
    const int nb = (p.c + kDwRows - 1) / kDwRows, d64 = p.d == 64 ? 2 : 1, row = p.Hq / p.Hkv * p.d;
    const int want = d64 == 2 && nb > 32 ? 8 : 4;  // blocks per slice
    const int most = nb <= (d64 == 1 ? 80 : 128) ? 8 : nb <= (pairs > 4 ? 400 : 200) * d64 ? 16 : nb <= 800 * d64 ? 32 : 64;
    int ns = (nb + want - 1) / want;
    if (ns > most) ns = most;
    if (ns > fit) ns = (int)fit;
    if (ns > 1) {
        const int per = (nb + ns - 1) / ns;
        const int pays = (rope ? 9 * d64 : d64 == 1 ? 13 : 22) + (ns == 2 ? 8 : ns == 3 ? 3 : 0) * d64;
        if (nb - per >= pays) return {ns, d64 == 1 || per <= 4 ? 4 : 8, ns <= kDwMostAdded && row <= 1024 && ns * row <= 8192};
    }
    return {1, nb <= 4 || pairs > (long)units * d64 ? 4 : 8, false};
}

int launch_decode_wide(const sepkv_params &p, const DecodeWideShape &shape, const uint16_t *q, const uint16_t *Kc, const uint16_t *Vc,
                       const int32_t *sizes, const float *rope, int n_pos, uint16_t *out, float *lse, float *part,
                       hipStream_t st) {
    if (p.Hkv > 65535 || p.S > 65535) return SEPATTN_ERR_SHAPE;
    const int G = p.Hq / p.Hkv;
    ProfScope prof(SEPATTN_K_DECODE_SPLIT, st);
    const uint64_t one = shape.add ? launch_number() : 0;
    auto go = [&](auto D_, auto NW_, auto ADD_) {
        constexpr int D = decltype(D_)::value, NW = decltype(NW_)::value;
        constexpr bool ADD = decltype(ADD_)::value;
        const dim3 grid(shape.nsplit, p.Hkv, p.S), block(64 * NW);
        if (rope)
            hipLaunchKernelGGL((decode_wide_kernel<D, true, NW, ADD>), grid, block, 0, st, p, G, n_pos, q, Kc, Vc, sizes, rope, one, part, out, lse);
        else
            hipLaunchKernelGGL((decode_wide_kernel<D, false, NW, ADD>), grid, block, 0, st, p, G, n_pos, q, Kc, Vc, sizes, rope, one, part, out, lse);
    };
    auto pick = [&](auto D_, auto NW_) { shape.add ? go(D_, NW_, IntC<1>{}) : go(D_, NW_, IntC<0>{}); };
    if (p.d == 64) shape.nw == 4 ? pick(IntC<64>{}, IntC<4>{}) : pick(IntC<64>{}, IntC<8>{});
    else shape.nw == 4 ? pick(IntC<128>{}, IntC<4>{}) : pick(IntC<128>{}, IntC<8>{});
    return launch_status();
}

}  // namespace sepattn
