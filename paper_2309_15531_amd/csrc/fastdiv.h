// Correctly rounded fp32 quotient w/s from a precomputed reciprocal.
//
// The quantizer divides every weight of a group by the same scale.  With
// y = RN(1/s) computed once per group by a true IEEE division, the quotient of
// each weight costs three operations instead of a full division sequence:
//     t = RN(w*y);  r = fma(-s, t, w) (the exact residual);  q = fma(r, y, t).
// q equals the correctly rounded w/s for every w that is an fp16 value (at most
// 11 significant bits) and every normal fp32 s for which no intermediate leaves
// the normal range; tests/host/fastdiv_check.cpp verifies this exhaustively over
// all significand pairs (the operations are invariant under power-of-two
// scaling of w and s).  It also equals RN(w / s) for every fp32 w in
// [2^-60, 2^60] when s is 2^bits - 1, bits 2 to 8 (the same check takes all
// significands of w): a group's range is divided that way.  Callers take the
// plain division when fastdiv_ok(s) is false.
//
// Plain C++ (fmaf), so that the same text compiles for the host-side check and,
// through hipcc, for the device (v_fma_f32 is a single-rounding fused op).
#pragma once

#include <cmath>

#if defined(__HIPCC__)
#define FASTDIV_FN __host__ __device__ __forceinline__
#else
#define FASTDIV_FN inline
#endif

// s in [2^-40, 2^40]: with |w| in {0} U [2^-24, 65504] every intermediate stays normal.
FASTDIV_FN bool fastdiv_ok(float s) { return s >= 9.094947e-13f && s <= 1.0995116e12f; }

FASTDIV_FN float fastdiv(float w, float s, float y) {
    const float t = w * y;
    const float r = fmaf(-s, t, w);
    return fmaf(r, y, t);
}

// For numerators of any significand fastdiv's quotient is within one unit in the last place of a / b (its error before rounding
// is about 2^-46 relative), and correcting it once more rounds to RN(a / b): the residual a - b q is then exact (Markstein's
// theorem on division with a correctly rounded reciprocal).  So a quotient q of fastdiv's is RN(a / b) if this
// leaves it as it is.  Holds while no intermediate leaves the normal range: b and y = RN(1 / b) in [2^-40, 2^40], and |a| = 0 or
// in [2^-80, 2^61].
FASTDIV_FN float fastdiv_corrected(float a, float b, float y, float q) {
    return fmaf(fmaf(-b, q, a), y, q);
}
