// Compile-time dispatch of the matrix-core logit kernels over width, bits and
// group size for one sketch size, shared by the translation units that
// instantiate them (isoq_scores_m.hip: no sketch; isoq_scores_m64.hip and
// isoq_scores_m128.hip: m = 64 and 128 sign bits).
#pragma once

#include "isoq_scores_m.h"

namespace isoq {
namespace {

// Heads per tile and tiles per pass: two heads (up to d = 256; the two copies
// of their query digits take d / 8 registers) share the row groups of the
// matrix instruction between 16-key groups; up to four take one tile; more
// loop, eight at a time up to d = 192.  Wide codebooks loop,
// four at a time, except for two heads (two sets, d = 128, 3 bits, 8 x 8 key
// heads, 8,192 keys: 18.0 us in the loop, 15.8 by pairs; 14.7 with lookup
// tables.  One set: 12.7 -> 11.2 us).
template <int D, int BITS, int QM>
ScoreKernel score_m_entry(int group, bool wide)
{
    using S = ScoreMShape<D, BITS, QM>;
    const size_t lds = sizeof(uint32_t) * (kOddWords + (size_t)group * S::head_words());
    if constexpr (D <= 256) {
        if (wide && group == 2)
            return {reinterpret_cast<const void *>(&score_m_kernel<D, BITS, QM, 2, 1, false, true>), lds};
    }
    if (wide)
        return {reinterpret_cast<const void *>(&score_m_kernel<D, BITS, QM, 4, 1, true, true>), lds};
    if constexpr (D <= 256) {
        if (group == 2)
            return {reinterpret_cast<const void *>(&score_m_kernel<D, BITS, QM, 2, 1, false, false>), lds};
    }
    if (group <= 4)
        return {reinterpret_cast<const void *>(&score_m_kernel<D, BITS, QM, 4, 1, false, false>), lds};
    return {reinterpret_cast<const void *>(&score_m_kernel<D, BITS, QM, 4, D <= 192 ? 2 : 1, true, false>), lds};
}

template <int D, int QM>
ScoreKernel score_m_bits(int bits, int group, bool wide)
{
    switch (bits) {
    case 2: return score_m_entry<D, 2, QM>(group, wide);
    case 3: return score_m_entry<D, 3, QM>(group, wide);
    case 4: return score_m_entry<D, 4, QM>(group, wide);
    }
    return {nullptr, 0};
}

template <int QM>
ScoreKernel score_m_d(int d, int bits, int group, bool wide)
{
    switch (d) {
    case 64: return score_m_bits<64, QM>(bits, group, wide);
    case 80: return score_m_bits<80, QM>(bits, group, wide);
    case 96: return score_m_bits<96, QM>(bits, group, wide);
    case 128: return score_m_bits<128, QM>(bits, group, wide);
    case 160: return score_m_bits<160, QM>(bits, group, wide);
    case 192: return score_m_bits<192, QM>(bits, group, wide);
    }
    if constexpr (QM < 128) {
        if (d == 256)
            return score_m_bits<256, QM>(bits, group, wide);
        if (d == 512)
            return score_m_bits<512, QM>(bits, group, wide);
    }
    return {nullptr, 0};
}

}  // namespace
}  // namespace isoq
