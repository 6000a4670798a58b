// The fp32 path's blocks, its backward's workspace, and the rule for one launch or two: what the host needs to know of attn_fp32.hip.
#pragma once

#include "common.h"

namespace sepattn {

constexpr int kT = 16;  // queries / keys per block

// backward workspace: D_i [B,Hq,L] (where dQ and dK/dV share a launch: the words that count the slices) | one counter per list tile |
// the slots of the partial sums
struct Fp32Workspace {
    int wpg, n_far_tiles;
    long n_counters;
    size_t d_bytes, counter_bytes, total;
};
inline Fp32Workspace fp32_workspace(const sepattn_params &p) {
    Fp32Workspace w;
    const long n_bkv = (long)p.B * p.Hkv, wpg = 2 * (long)compute_units() / n_bkv;
    w.wpg = (int)(wpg < 1 ? 1 : wpg);
    w.n_far_tiles = (p.a + p.cap + kT - 1) / kT;
    w.n_counters = n_bkv * w.n_far_tiles;
    w.d_bytes = align_up((size_t)p.B * p.Hq * p.L * sizeof(float), 256);
    w.counter_bytes = align_up((size_t)w.n_counters * sizeof(int32_t), 256);
    w.total = w.d_bytes + w.counter_bytes + (size_t)n_bkv * (w.wpg + w.n_far_tiles) * (2 * kT * p.d) * sizeof(float);
    return w;
}

// One launch or two.  dK/dV needs nothing of dQ but D_i.  Where the blocks are few, both kinds run side by side in one launch and
// dK/dV forms D_i itself (one more row per item); where they fill the chip anyway, dQ comes first, by itself.  The line, in dQ
// tiles and band units per compute unit, of which the joint kernel has two at a time at d = 64 and one at d = 128 (registers):
// backward in us, two launches / one.  d = 64: 2/1 heads, L = 512 (0.4) 21.3 / 15.0, 4 x 4/1 heads, L = 1000 (1.2) 48.0 / 38.1, 8/2
// heads, L = 1024 (2.5) 49.8 / 40.0, 32/32 heads, L = 200 (3.3) 30.6 / 27.9, 2/2 heads, L = 4000 (3.9) 53.5 / 51.1, 1/1 heads, L = 8192 (4)
// 90.1 / 93.6, 2 x 8/8 heads, L = 1024 (8) 59.8 / 61.9, 4 x 12/12 heads 167 / 190.  d = 128: 4/4 heads, L = 300 (0.6) 33.7 / 21.2, L = 1024 (2)
// 34.3 / 31.9, 8/2 heads, L = 1024 (2.5) 89.9 / 79.4, 32/32 heads, L = 200 (3.3) 56.2 / 63.0, 8/8 heads, L = 1024 (4) 79.8 / 88.9.
// Returned: 0, two launches; otherwise one, and the bytes from one of the words that count slices to the next: a cache line where there
// is room.  (A captured call has two launches whatever this says, see being_captured.)
inline int fp32_one_launch(const sepattn_params &p, const Fp32Workspace &w) {
    const long tiles = (p.L + kT - 1) / kT, most = (p.d == 64 ? 15 : 10) * (long)compute_units() / 4;
    const int stride = (size_t)w.n_counters * 128 <= w.d_bytes ? 128 : 8;
    return (long)p.B * (p.Hq + p.Hkv) * tiles <= most && (size_t)w.n_counters * stride <= w.d_bytes ? stride : 0;
}

}  // namespace sepattn
