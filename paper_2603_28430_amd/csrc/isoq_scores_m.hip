// Attention-logit kernels without the stage-2 sketch (the kernel template is
// in isoq_scores_m.h), and the dispatch over the sketch size.
#include "isoq_scores_m_pick.h"

namespace isoq {

ScoreKernel score_m_kernel_m64(int d, int bits, int group, bool wide);
ScoreKernel score_m_kernel_m128(int d, int bits, int group, bool wide);

ScoreKernel score_m_kernel_for(int d, int bits, int group, int m, bool wide)
{
    switch (m) {
    case 0: return score_m_d<0>(d, bits, group, wide);
    case 64: return score_m_kernel_m64(d, bits, group, wide);
    case 128: return score_m_kernel_m128(d, bits, group, wide);
    }
    return {nullptr, 0};
}

}  // namespace isoq
