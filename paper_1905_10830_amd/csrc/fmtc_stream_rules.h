// Rules of the streaming projection (k_project_quantize_stream) that can be checked without a device: the scale of its
// operands, the distance to a rounding boundary from which its sums decide, and the order of its tiles.  Plain C++.
#pragma once
#include <stdint.h>

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
    return std::ldexp(1.f, k < -126 ? -126 : (k > 126 ? 126 : k));  // (what fp32 holds)
}

// What a coefficient's sum over `steps` steps of 16 channels is off by at most, in units of 2^-24 |T_k|_2.
// band_of_roundings, per sqrt(v_1^2 + v_2^2 + ...) with v_j the length of the pixel's part S (x - mu) in the first j steps:
//   - three matrix instructions a step, each of which adds two times eight products to the sum and rounds it to nearest both
//     times, where the sum so far is no larger than |T_k|_2 v_j (1 + 2^-10): 6 (v_1 + v_2 + ...), which is 6 sqrt(steps) of these
//     at most.  (6 steps |v|_2 as a whole is 1.3 times that where all channels are alike: planar tensor of 256 x 128 x 28 x 28,
//     6 bits, 49.1 us for the kernel, 47.8 this way.)
// kBandOfRest, per the whole pixel's length:
//   - 8: before each of these additions the eight products (exact in fp32) are cut off, and the sum so far rounded down, at
//     2^-24 of the largest of them or less, and over all steps these largest ones add up to |T_k|_2 |S (x - mu)|_2 at most
//     (those of the lower parts to 2^-11 of it);
//   - 4 for the two f16 parts of T, 4 for those of x - mu, 4 for the product of the two lower parts, left out; 1 for the
//     rounding of x - mu;
//   - 1 for that of 1 / delta;
//   - 4 that cover the subnormals (see above), the sum of squares behind |x - mu|_2 and 2^-10 of all this.
// (The instruction's arithmetic as measured: with the cut at 2^(e - 24), e the largest sum of the factors' exponents, and one
// rounding to nearest, all of 60000 sums of eight products of like size are reproduced bit by bit, and 99.99 % of those of
// sizes over 2^12.)
inline float band_of_roundings(int steps) { return 6.f * std::sqrt((float)steps) * (1.f / 16777216.f); }
constexpr float kBandOfRest = 26.f / 16777216.f;

// The tiles that a wavefront takes, one after the other.  Whole rounds, and a tensor's only one, go to the wavefronts of the
// grid in order, neighbouring tiles to one workgroup: dealt to the workgroups first, planar tiles lose the lines that they
// share (144 channels, 255 images of 14 x 14, 1562 tiles 17.8 -> 21.4 us; 160 channels, 61 of 28 x 28 19.9 -> 22.4).  The tiles
// of a last round that is not full go to the workgroups first: a few of them have a compute unit each.
struct TileWalk {
    int64_t n, stride, whole, last, first;
    constexpr TileWalk(int64_t n_tiles, uint32_t grid, uint32_t waves, uint32_t block, uint32_t wave)
        : n(n_tiles), stride((int64_t)grid * waves),
          whole(n_tiles <= stride ? n_tiles : n_tiles - (int64_t)((uint32_t)n_tiles % (uint32_t)stride)),
          last(whole + (int64_t)wave * grid + block), first((int64_t)block * waves + wave) {}
    // (n or more: none)
    constexpr int64_t after(int64_t tile) const { return tile + stride < whole ? tile + stride : (tile < whole ? last : n); }
};

}  // namespace fmtc
