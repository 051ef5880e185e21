// Compile-time dispatch of the attention-logit kernels without the stage-2
// sketch over width, bits, query type and filling (the kernel template is in
// isoq_scores.h), shared by the translation units that instantiate it for
// the rotation variants (isoq_scores.hip, isoq_scores_8d.hip).
#pragma once

#include "isoq_scores.h"

namespace isoq {
namespace {

template <int VAR, int D, int BITS, bool F16>
ScoreKernel pick_fill(bool fill)
{
    if constexpr (score_by_tables(D, BITS, 1))
        return {fill ? reinterpret_cast<const void *>(&score_kernel<VAR, D, BITS, F16, 0, true>)
                     : reinterpret_cast<const void *>(&score_kernel<VAR, D, BITS, F16, 0, false>), 0};
    return {nullptr, 0};
}

template <int VAR, int D, int BITS>
ScoreKernel pick_dtype(bool f16, bool fill)
{
    return f16 ? pick_fill<VAR, D, BITS, true>(fill) : pick_fill<VAR, D, BITS, false>(fill);
}

template <int VAR, int D>
ScoreKernel pick_bits(int bits, bool f16, bool fill)
{
    switch (bits) {
    case 2: return pick_dtype<VAR, D, 2>(f16, fill);
    case 3: return pick_dtype<VAR, D, 3>(f16, fill);
    case 4: return pick_dtype<VAR, D, 4>(f16, fill);
    }
    return {nullptr, 0};
}

template <int VAR>
ScoreKernel pick_d(int d, int bits, bool f16, bool fill)
{
    switch (d) {
    case 64: return pick_bits<VAR, 64>(bits, f16, fill);
    case 80: return pick_bits<VAR, 80>(bits, f16, fill);
    case 96: return pick_bits<VAR, 96>(bits, f16, fill);
    case 128: return pick_bits<VAR, 128>(bits, f16, fill);
    case 160: return pick_bits<VAR, 160>(bits, f16, fill);
    case 192: return pick_bits<VAR, 192>(bits, f16, fill);
    case 256: return pick_bits<VAR, 256>(bits, f16, fill);
    case 512: return pick_bits<VAR, 512>(bits, f16, fill);
    }
    return {nullptr, 0};
}

}  // namespace
}  // namespace isoq
