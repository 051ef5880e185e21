// Attention-logit kernels with the stage-2 residual correction of m = 64 sign
// bits per key (the kernel template is in isoq_scores_m.h).
#include "isoq_scores_m_pick.h"

namespace isoq {

ScoreKernel score_m_kernel_m64(int d, int bits, int group, bool wide)
{
    return score_m_d<64>(d, bits, group, wide);
}

}  // namespace isoq
