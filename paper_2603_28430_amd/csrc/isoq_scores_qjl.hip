// Attention-logit kernels with the stage-2 residual correction (the kernel
// template is in isoq_scores.h): m = 64 or 128 sign bits at the decoding
// widths up to 192, 64 at d = 256 and 512.
#include "isoq_scores.h"

namespace isoq {
namespace {

template <int VAR, int D, int BITS, bool F16>
ScoreKernel pick_m(int m)
{
    if constexpr (score_by_tables(D, BITS, 1)) {
        if (m == 64)
            return {reinterpret_cast<const void *>(&score_kernel<VAR, D, BITS, F16, 64>), 0};
        if constexpr (D <= 192) {
            if (m == 128)
                return {reinterpret_cast<const void *>(&score_kernel<VAR, D, BITS, F16, 128>), 0};
        }
    }
    return {nullptr, 0};
}

template <int VAR, int D>
ScoreKernel pick_bits(int bits, bool f16, int m)
{
    switch (bits) {
    case 2: return f16 ? pick_m<VAR, D, 2, true>(m) : pick_m<VAR, D, 2, false>(m);
    case 3: return f16 ? pick_m<VAR, D, 3, true>(m) : pick_m<VAR, D, 3, false>(m);
    case 4: return f16 ? pick_m<VAR, D, 4, true>(m) : pick_m<VAR, D, 4, false>(m);
    }
    return {nullptr, 0};
}

template <int VAR>
ScoreKernel pick_d(int d, int bits, bool f16, int m)
{
    switch (d) {
    case 64: return pick_bits<VAR, 64>(bits, f16, m);
    case 80: return pick_bits<VAR, 80>(bits, f16, m);
    case 96: return pick_bits<VAR, 96>(bits, f16, m);
    case 128: return pick_bits<VAR, 128>(bits, f16, m);
    case 160: return pick_bits<VAR, 160>(bits, f16, m);
    case 192: return pick_bits<VAR, 192>(bits, f16, m);
    case 256: return pick_bits<VAR, 256>(bits, f16, m);
    case 512: return pick_bits<VAR, 512>(bits, f16, m);
    }
    return {nullptr, 0};
}

}  // namespace

ScoreKernel score_qjl_kernel_for(int variant, int d, int bits, bool f16, int m)
{
    switch (variant) {
    case VAR_FULL: return pick_d<VAR_FULL>(d, bits, f16, m);
    case VAR_FAST: return pick_d<VAR_FAST>(d, bits, f16, m);
    case VAR_PLANAR2D: return pick_d<VAR_PLANAR2D>(d, bits, f16, m);
    }
    return {nullptr, 0};
}

}  // namespace isoq
