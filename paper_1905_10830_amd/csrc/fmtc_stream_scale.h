// The scale of the streaming projection's operands (k_project_quantize_stream).  Plain C++, for the model of its sums on the
// CPU.
#pragma once
#include <cmath>

namespace fmtc {

// S for a step delta at a bit depth and a basis whose longest row has the norm row_norm.  Pixels whose coefficients fill the
// quantizer's range A = delta 2^(bits-1) have |x - mu|_2 = A / row_norm, which S brings to 64 .. 128:
//   - f16 holds pixels of up to 468 A / row_norm.  (A pixel beyond is decided exactly in all coefficients.)
//   - v_lo and 2^-11 v_hi lose up to 2^-25 of a value each in the subnormals, over all channels at most 2^-24 sqrt(160)
//     row_norm of S y, which is less than 2^-5 of what the floor of the distance from a rounding boundary, 2^-21 of the range
//     (tau_min), leaves: 2^-21 S A = 2^-15 row_norm at least.
// (With S from A alone, the basis taken for one of unit rows: rows of norm 16384, pixels of a tenth of the range, 128
// channels, 8 bits: 60 of a million values wrong and not decided exactly; rows of norm 2^-9: every value decided exactly.)
inline float stream_scale(float delta, int bits, float row_norm) {
    const double reach = std::ldexp((double)delta, bits - 1) / (double)row_norm;
    if (!(reach > 0.0) || std::isinf(reach)) return 1.f;  // (no row but zeros, or rows beyond fp32)
    int e = 0;
    (void)std::frexp(reach, &e);  // reach in [2^(e-1), 2^e)
    const int k = 7 - e;
    return std::ldexp(1.f, k < -100 ? -100 : (k > 100 ? 100 : k));  // (what fp32 and its reciprocal hold)
}

}  // namespace fmtc
