// The joint backward kernels at d = 128 (see bwd_joint.h).
#include "bwd_joint.h"

namespace sepattn {

int launch_joint_128(const sepattn_params &p, int dq_wpg, const uint16_t *Q, const uint16_t *K, const uint16_t *V, const uint16_t *O, const float *LSE,
                     const uint16_t *dO, const int32_t *sep_idx, const int32_t *sep_prefix, const int32_t *doc_start, const int32_t *doc_end,
                     uint16_t *dQ, uint16_t *dK, uint16_t *dV, float *Dws, float *Lws, float *farK, float *farV, int32_t *piece_tab, hipStream_t st) {
    return launch_joint<128>(p, dq_wpg, Q, K, V, O, LSE, dO, sep_idx, sep_prefix, doc_start, doc_end, dQ, dK, dV, Dws, Lws, farK, farV, piece_tab, st);
}

}  // namespace sepattn
