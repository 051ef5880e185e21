// Attention-logit kernels with the stage-2 residual correction (the kernel
// template is in isoq_scores.h): m = 64 or 128 sign bits at the decoding
// widths up to 192, 64 at d = 256 and 512.
#include "isoq_scores.h"

namespace isoq {
namespace {

template <int VAR, int D, int BITS, bool F16, bool FILL>
ScoreKernel pick_m(int m)
{
    if constexpr (score_by_tables(D, BITS, 1)) {
        if (m == 64)
            return {reinterpret_cast<const void *>(&score_kernel<VAR, D, BITS, F16, 64, FILL>), 0};
        if constexpr (D <= 192) {
            if (m == 128)
                return {reinterpret_cast<const void *>(&score_kernel<VAR, D, BITS, F16, 128, FILL>), 0};
        }
    }
    return {nullptr, 0};
}

template <int VAR, int D, int BITS>
ScoreKernel pick_dtype(bool f16, int m, bool fill)
{
    if (f16)
        return fill ? pick_m<VAR, D, BITS, true, true>(m) : pick_m<VAR, D, BITS, true, false>(m);
    return fill ? pick_m<VAR, D, BITS, false, true>(m) : pick_m<VAR, D, BITS, false, false>(m);
}

template <int VAR, int D>
ScoreKernel pick_bits(int bits, bool f16, int m, bool fill)
{
    switch (bits) {
    case 2: return pick_dtype<VAR, D, 2>(f16, m, fill);
    case 3: return pick_dtype<VAR, D, 3>(f16, m, fill);
    case 4: return pick_dtype<VAR, D, 4>(f16, m, fill);
    }
    return {nullptr, 0};
}

template <int VAR>
ScoreKernel pick_d(int d, int bits, bool f16, int m, bool fill)
{
    switch (d) {
    case 64: return pick_bits<VAR, 64>(bits, f16, m, fill);
    case 80: return pick_bits<VAR, 80>(bits, f16, m, fill);
    case 96: return pick_bits<VAR, 96>(bits, f16, m, fill);
    case 128: return pick_bits<VAR, 128>(bits, f16, m, fill);
    case 160: return pick_bits<VAR, 160>(bits, f16, m, fill);
    case 192: return pick_bits<VAR, 192>(bits, f16, m, fill);
    case 256: return pick_bits<VAR, 256>(bits, f16, m, fill);
    case 512: return pick_bits<VAR, 512>(bits, f16, m, fill);
    }
    return {nullptr, 0};
}

}  // namespace

ScoreKernel score_qjl_kernel_for(int variant, int d, int bits, bool f16, int m, bool fill)
{
    switch (variant) {
    case VAR_FULL: return pick_d<VAR_FULL>(d, bits, f16, m, fill);
    case VAR_FAST: return pick_d<VAR_FAST>(d, bits, f16, m, fill);
    case VAR_PLANAR2D: return pick_d<VAR_PLANAR2D>(d, bits, f16, m, fill);
    }
    return {nullptr, 0};
}

}  // namespace isoq
