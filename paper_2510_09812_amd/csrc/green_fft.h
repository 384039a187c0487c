// The elastic preconditioner's own grid transforms (green_fft.hip).
#pragma once

#include "common.h"

namespace gspm {

constexpr int kFftSlots = 3;           // values of k a wave of a stage takes at once
// k = 0 .. R / 2, padded to whole slots
__host__ __device__ constexpr int fft_columns(int R) { return (R / 2 + kFftSlots) / kFftSlots * kFftSlots; }

// One axis: length n1 n2, for each of the two lengths R (cos, sin)(2 pi k t /
// R) as [t <= R / 2][fft_columns(R)], the twiddles exp(-2 pi i n2' k1 / N) as
// [n2'][k1], and by position the frequency and the position of its negative.
struct FftAxis {
    int32_t n1, n2;
    const void *cs1, *cs2, *tw;        // pairs of T
    const int32_t *freq, *neg;
};

struct FftPlan {
    FftAxis x, y, z;
    const int32_t *pairs;              // [npairs][4]: positions of a column and of its mirror; its kx, ky (kx <= gx / 2)
    int32_t npairs, wg_pairs;          // wg_pairs: pairs of a workgroup of the z pass
};

// The pairs of a workgroup of the z pass; 0 when the library's transforms serve:
// planes or columns do not fit LDS or a stage's outputs a wave's registers, or
// the library is the faster.
int green_fft_pairs(const GreenView &gv, const int n1[3], const int n2[3], bool f32, size_t lds_max);
// gv.grid (two packed complex fields) replaced by A_g^+ of itself over G;
// returns at once when the scalar set has converged.
template <class T>
void launch_pc_fft(const GreenView &gv, const FftPlan &fp, const CGScalars &cg, hipStream_t s);

}  // namespace gspm
