// Compile-time dispatch of the attention-logit kernels without the stage-2
// sketch over width, bits and query type (the kernel template is in
// isoq_scores.h), shared by the translation units that instantiate it for
// the rotation variants (isoq_scores.hip, isoq_scores_8d.hip).
#pragma once

#include "isoq_scores.h"

namespace isoq {
namespace {

template <int VAR, int D, int BITS>
ScoreKernel pick_dtype(bool f16)
{
    if constexpr (score_by_tables(D, BITS, 1))
        return {f16 ? reinterpret_cast<const void *>(&score_kernel<VAR, D, BITS, true, 0>)
                    : reinterpret_cast<const void *>(&score_kernel<VAR, D, BITS, false, 0>), 0};
    return {nullptr, 0};
}

template <int VAR, int D>
ScoreKernel pick_bits(int bits, bool f16)
{
    switch (bits) {
    case 2: return pick_dtype<VAR, D, 2>(f16);
    case 3: return pick_dtype<VAR, D, 3>(f16);
    case 4: return pick_dtype<VAR, D, 4>(f16);
    }
    return {nullptr, 0};
}

template <int VAR>
ScoreKernel pick_d(int d, int bits, bool f16)
{
    switch (d) {
    case 64: return pick_bits<VAR, 64>(bits, f16);
    case 80: return pick_bits<VAR, 80>(bits, f16);
    case 96: return pick_bits<VAR, 96>(bits, f16);
    case 128: return pick_bits<VAR, 128>(bits, f16);
    case 160: return pick_bits<VAR, 160>(bits, f16);
    case 192: return pick_bits<VAR, 192>(bits, f16);
    case 256: return pick_bits<VAR, 256>(bits, f16);
    case 512: return pick_bits<VAR, 512>(bits, f16);
    }
    return {nullptr, 0};
}

}  // namespace
}  // namespace isoq
