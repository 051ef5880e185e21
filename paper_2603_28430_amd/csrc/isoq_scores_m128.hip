// Attention-logit kernels with the stage-2 residual correction of m = 128 sign
// bits per key (the kernel template is in isoq_scores_m.h).
#include "isoq_scores_m_pick.h"

namespace isoq {

ScoreKernel score_m_kernel_m128(int d, int bits, int group, bool wide)
{
    return score_m_d<128>(d, bits, group, wide);
}

}  // namespace isoq
