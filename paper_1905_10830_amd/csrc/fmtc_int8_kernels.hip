// 8-bit basis and 8-bit activations (paper section 3.1 "Linear transform": the PCA matrix is stored at 8 bits;
// section 5: the hardware moves 8-bit activations).  Both contractions run on the integer matrix cores
// (v_mfma_i32_32x32x16_i8) and are exact; every rounding decision is one fp64 operation on exact operands, so the
// results are defined bit for bit:
//   forward  n = 256 sum_c Tq[k][c] xq[c] - sum_c Tq[k][c] mf[c],  level = rne(n * g),  g = s_T s_x / (256 Delta)
//   inverse  m = sum_k Tq[k][c] (s[k] - 2^(b-1)),  v = fma(m, h, mf[c]),  xq^ = clamp(rne(v / 256), 0, 255),
//            h = 256 s_T Delta / s_x   (computed as rne(fma(m, h / 256, mf[c] / 256)): scaling by 2^-8 is exact)
// The matrix instruction multiplies signed bytes; unsigned activations and symbols enter as (value - 128) (one XOR)
// and the difference is folded into per-row integer offsets prepared with the basis.
//
// A wavefront owns 32 pixels (k_int8_tiles: up to 128 channels) or a workgroup 64 (k_int8_wide).  Operand order (both operands): lane l holds row/pixel l % 32 and the 8 bytes
// 16 s + 8 (l / 32) .. + 7 of contraction step s.  The rows of a 32-row tile of the basis are stored permuted so
// that a lane's 16 results are 16 consecutive coefficients (channels): one 16-byte store.
#include "fmtc_device.h"
#include "fmtc_internal.h"

namespace fmtc {

typedef int v16i __attribute__((ext_vector_type(16)));
typedef int v4i __attribute__((ext_vector_type(4)));

// 8 consecutive bytes row[c0 .. c0 + 7] of a row-major byte matrix with rows of n_cols bytes; zeros outside.
// wide: n_cols is a multiple of 8 and base is 8-byte aligned, so the group is either whole or absent.
__device__ __forceinline__ unsigned long long load8_row(const uint8_t* __restrict__ base, int64_t row, int64_t n_rows,
                                                        int c0, int n_cols, bool wide) {
    if (row >= n_rows || c0 >= n_cols) return 0ull;
    const uint8_t* q = base + (size_t)row * (size_t)n_cols + (size_t)c0;
    if (wide) return *reinterpret_cast<const unsigned long long*>(q);
    unsigned long long v = 0ull;
#pragma unroll
    for (int e = 0; e < 8; e++)
        if (c0 + e < n_cols) v |= (unsigned long long)q[e] << (8 * e);
    return v;
}

// the same bytes of pixel p from a planar (n, c, hw) tensor
__device__ __forceinline__ unsigned long long load8_planar(const uint8_t* __restrict__ base, int64_t p, int64_t P,
                                                           int c0, int C, int64_t HW) {
    if (p >= P || c0 >= C) return 0ull;
    const int64_t n = p / HW, hw = p - n * HW;
    const uint8_t* q = base + ((size_t)n * (size_t)C + (size_t)c0) * (size_t)HW + (size_t)hw;
    unsigned long long v = 0ull;
#pragma unroll
    for (int e = 0; e < 8; e++)
        if (c0 + e < C) v |= (unsigned long long)q[(size_t)e * (size_t)HW] << (8 * e);
    return v;
}

struct Int8Params {
    const uint8_t* in;              // forward: activations in `layout`; inverse: symbols [P][C]
    uint8_t* out;                   // forward: symbols [P][C]; inverse: activations in `layout`
    const unsigned long long* op8;  // [nct][NS][64] basis (forward) or its transpose (inverse), operand order
    const double* row_off;          // forward [nct * 32]: sum_c Tq[k][c] (mf[c] - 256 * 128), an integer below 2^53
    const int* col_sum;             // inverse [nct * 32]: sum_k Tq[k][c]
    const double* mean_d;           // inverse [nct * 32]: the mean in activation units (mean_fix / 256, exact)
    int64_t P, HW, n_tiles;
    int C, NS, nct, bits;
    double factor;                  // g (forward) or h / 256 (inverse)
    // forward, whole encoder only (else null): one partial histogram per workgroup [gridDim.x][2^bits], and the
    // coder's scratch that the first kernel of a call clears
    uint32_t* hist_parts;
    CoderCtrl* ctrl;
    unsigned long long* lookback;
    uint32_t n_groups;
};

struct Int8WideParams {
    Int8Params p;
    int64_t px_tiles;  // of 64 pixels
    int kt_per;        // row tiles per workgroup
    int hist_shift;    // log2 of the histogram copies per wavefront
};

constexpr int kCopies = 16;  // histogram copies per wavefront
constexpr unsigned long long kFlip = 0x8080808080808080ull;  // unsigned byte -> (value - 128) as a signed byte

// The symbol of coefficient r (forward), the activation of channel r (inverse) from the sum of products.  (All integers
// below 2^53, so the fp64 operations before the one rounding product are exact.)
__device__ __forceinline__ uint32_t level_of(int acc, double row_off, double g, int hk) {
    const double n = fma((double)acc, 256.0, -row_off);
    return (uint32_t)(int)(fmin(fmax(rint(n * g), (double)-hk), (double)(hk - 1)) + (double)hk);
}
__device__ __forceinline__ uint32_t activation_of(int acc, int col_sum, double mean, double h, int hk) {
    const int m = acc + (128 - hk) * col_sum;
    return (uint32_t)(int)fmin(fmax(rint(fma((double)m, h, mean)), 0.0), 255.0);
}

// At most 128 channels: the pixel tile's operand (NS <= NSR steps) stays in registers over the coefficient tiles.
template <int LAYOUT, int NSR, bool INVERSE>
__global__ __launch_bounds__(256) void k_int8_tiles(Int8Params p) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    const int C = p.C, NS = p.NS;
    const int hk = 1 << (p.bits - 1);
    const bool wide = (C % 8) == 0;
    // Histogram (forward, whole encoder), in dynamic LDS: kCopies interleaved copies per wavefront (bin s of copy q
    // at word s * kCopies + q, lane l counts in copy l % kCopies), because most symbols of a tile are the same few
    // values and one copy would serialise the lanes on a few words.
    // The basis operand (at most 8 steps, 16 KB) is copied into LDS first.
    extern __shared__ __align__(16) uint32_t s_dyn[];  // basis operand [nct][NS][64] x 8 bytes, then the histogram
                                                       // [4][K * kCopies] if hist
    const int basis_words = p.nct * NS * 128;
    uint32_t* s_hist = s_dyn + basis_words;
    const bool hist = !INVERSE && p.hist_parts != nullptr;
    const int K = 1 << p.bits;
    uint32_t* wh = s_hist + (size_t)wave * K * kCopies + (lane & (kCopies - 1));
    {
        const uint4* src = reinterpret_cast<const uint4*>(p.op8);
        uint4* dst = reinterpret_cast<uint4*>(s_dyn);
        for (int i = threadIdx.x; i < basis_words / 4; i += 256) dst[i] = src[i];
    }
    if (hist) {
        zero_coder_scratch(p.ctrl, p.lookback, p.n_groups);
        for (int i = threadIdx.x; i < 4 * K * kCopies; i += 256) s_hist[i] = 0u;
    }
    __syncthreads();
    const unsigned long long* op8 = reinterpret_cast<const unsigned long long*>(s_dyn);
    for (int64_t tile = (int64_t)blockIdx.x * 4 + wave; tile < p.n_tiles; tile += (int64_t)gridDim.x * 4) {
        const int64_t px = tile * 32 + l32;
        auto operand = [&](int s) -> long {
            const int c0 = 16 * s + 8 * half;
            unsigned long long v;
            if (INVERSE || LAYOUT == FMTC_NHWC) v = load8_row(p.in, px, p.P, c0, C, wide);
            else v = load8_planar(p.in, px, p.P, c0, C, p.HW);
            return (long)(v ^ kFlip);
        };
        long b[NSR];
#pragma unroll
        for (int s = 0; s < NSR; s++) b[s] = s < NS ? operand(s) : 0l;
        for (int kt = 0; kt < p.nct; kt++) {
            v16i acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
            const unsigned long long* a8 = op8 + ((size_t)kt * NS) * 64 + lane;
#pragma unroll
            for (int s = 0; s < NSR; s++)
                if (s < NS) acc = __builtin_amdgcn_mfma_i32_32x32x16_i8((long)a8[(size_t)s * 64], b[s], acc, 0, 0, 0);
            // this lane: pixel px, results r0 .. r0 + 15 (coefficients, or channels for the inverse)
            const int r0 = kt * 32 + 16 * half;
            uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int v = 0; v < 16; v++) {
                const int r = r0 + v;  // < nct * 32: the per-row arrays are padded to that
                uint32_t t;
                if constexpr (INVERSE) t = activation_of(acc[v], p.col_sum[r], p.mean_d[r], p.factor, hk);
                else t = level_of(acc[v], p.row_off[r], p.factor, hk);
                w[v >> 2] |= t << (8 * (v & 3));
            }
            if (hist && px < p.P) {
                if (r0 + 16 <= C) {
#pragma unroll
                    for (int v = 0; v < 16; v++) atomicAdd(&wh[((w[v >> 2] >> (8 * (v & 3))) & 0xffu) * kCopies], 1u);
                } else {
#pragma unroll
                    for (int v = 0; v < 16; v++)
                        if (r0 + v < C) atomicAdd(&wh[((w[v >> 2] >> (8 * (v & 3))) & 0xffu) * kCopies], 1u);
                }
            }
            if (px < p.P && r0 < C) {
                if (INVERSE && LAYOUT == FMTC_NCHW) {
                    const int64_t n = px / p.HW, hw = px - n * p.HW;
#pragma unroll
                    for (int v = 0; v < 16; v++)
                        if (r0 + v < C)
                            p.out[((size_t)n * (size_t)C + (size_t)(r0 + v)) * (size_t)p.HW + (size_t)hw] =
                                (uint8_t)(w[v >> 2] >> (8 * (v & 3)));
                } else {
                    uint8_t* q = p.out + (size_t)px * (size_t)C + (size_t)r0;
                    if ((C % 16) == 0) {
                        *reinterpret_cast<uint4*>(q) = make_uint4(w[0], w[1], w[2], w[3]);
                    } else {
#pragma unroll
                        for (int v = 0; v < 16; v++)
                            if (r0 + v < C) q[v] = (uint8_t)(w[v >> 2] >> (8 * (v & 3)));
                    }
                }
            }
        }
    }
    if (hist) {
        __syncthreads();
        if ((int)threadIdx.x < K) {
            uint32_t sum = 0;
            for (int q = 0; q < 4; q++)
                for (int c = 0; c < kCopies; c++) sum += s_hist[((size_t)q * K + threadIdx.x) * kCopies + c];
            p.hist_parts[(size_t)blockIdx.x * K + threadIdx.x] = sum;
        }
    }
}

// Wider tensors, and planar activations.  A workgroup of four wavefronts brings 64 pixels, all channels, into LDS (one byte each: 8 to 64 KB) and
// its wavefronts share out the 32-row tiles of the workgroup's rows [kt0, kt0 + kt_per) of the basis, which streams from
// L2 in operand order, 256 channels ahead of its use; each of its entries meets two pixel groups.  Rows are split over
// blockIdx.y while pixels alone leave the device idle.  Results that do not leave as aligned pieces of a pixel (planar
// activations, channel counts that are no multiple of 16) go through LDS.
// What bounds it: latency for few pixels (loads of the tile, C / 32 products one after the other per row tile), the fp64
// operations and LDS additions of the results for many.  (Before: a wavefront by itself loaded its 32 pixels again from memory
// for every row tile, byte by byte where they are planar, and waited for each load.  Quantizer and reconstruction, us:
// 512 channels, N = 12, 16 x 15 102 -> 10 and 102 -> 8; 1024, N = 1, 9 x 12, planar 1914 -> 21 and 385 -> 13; 576, N = 2,
// 52 x 52, planar 713 -> 19 and 145 -> 13; 256, N = 250, 14 x 14 49 -> 21 and 47 -> 18; 250, the same 184 -> 40 and 182 -> 35.)
template <int LAYOUT, bool INVERSE, bool STAGED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_int8_wide(Int8WideParams q) {
    const Int8Params& p = q.p;
    constexpr int PG = 2, PX = 32 * PG;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int C = p.C, NS = p.NS, NP = (NS + 1) / 2;
    const int hk = 1 << (p.bits - 1), K = 1 << p.bits, HS = q.hist_shift;
    const int kt0 = (int)blockIdx.y * q.kt_per, kts = p.nct - kt0 < q.kt_per ? p.nct - kt0 : q.kt_per;
    const uint32_t stride = 16u * (uint32_t)NS + 8u;  // of a pixel in LDS: an odd number of 8-byte pieces
    extern __shared__ __align__(16) uint8_t s_wide[];
    // per row of the workgroup: fp64 constant [kt_per * 32], (inverse) column sums; histogram copies [4][K << HS]; staged
    // results [PX][132]; pixels [PX][stride] and 64 bytes that the reads of the last of them may run into
    double* s_const = reinterpret_cast<double*>(s_wide);
    int* s_sum = reinterpret_cast<int*>(s_const + q.kt_per * 32);
    uint32_t* s_hist = reinterpret_cast<uint32_t*>(s_sum + (INVERSE ? q.kt_per * 32 : 0));
    const bool hist = !INVERSE && p.hist_parts != nullptr;
    uint8_t* s_stage = reinterpret_cast<uint8_t*>(s_hist + (hist ? 4 * (K << HS) : 0));
    uint8_t* s_px = s_stage + (STAGED ? PX * 132 : 0);
    for (int i = tid; i < kts * 32; i += 256) {  // (the per-row arrays are padded to whole tiles)
        if constexpr (INVERSE) {
            s_const[i] = p.mean_d[kt0 * 32 + i];
            s_sum[i] = p.col_sum[kt0 * 32 + i];
        } else {
            s_const[i] = p.row_off[kt0 * 32 + i];
        }
    }
    if (hist) {
        zero_coder_scratch(p.ctrl, p.lookback, p.n_groups);
        for (int i = tid; i < 4 * (K << HS); i += 256) s_hist[i] = 0u;
    }
    uint32_t* wh = s_hist + wave * (K << HS) + (lane & ((1 << HS) - 1));

    for (int64_t tile = blockIdx.x; tile < q.px_tiles; tile += gridDim.x) {
        const int64_t px0 = tile * PX;
        const int n_px = p.P - px0 < PX ? (int)(p.P - px0) : PX;
        // ---- the pixels, as signed bytes (whatever stands behind the last channel meets zero basis bytes) ----
        if constexpr (INVERSE || LAYOUT == FMTC_NHWC) {
            // 16 pixels per wavefront; a lane takes four channels of each, eight loads in flight
            const uint8_t* src = p.in + (size_t)px0 * (size_t)C;
            for (int c = 4 * lane; c < C; c += 256) {
                const bool whole = c + 4 <= C;
#pragma unroll
                for (int i0 = 0; i0 < PX / 4; i0 += 8) {
                    uint32_t v[8];
#pragma unroll
                    for (int i = 0; i < 8; i++) {
                        int r = wave * (PX / 4) + i0 + i;
                        r = r < n_px ? r : n_px - 1;  // (rows past the tensor repeat its last pixel; never stored)
                        const uint8_t* at = src + (size_t)r * (size_t)C + c;
                        v[i] = 0u;
                        if (whole) {
                            __builtin_memcpy(&v[i], at, 4);
                        } else {
                            for (int e = 0; c + e < C; e++) v[i] |= (uint32_t)at[e] << (8 * e);
                        }
                    }
#pragma unroll
                    for (int i = 0; i < 8; i++)
                        *reinterpret_cast<uint32_t*>(s_px + (uint32_t)(wave * (PX / 4) + i0 + i) * stride + c) = v[i] ^ 0x80808080u;
                }
            }
        } else {
            // a lane takes four channels of four neighbouring pixels: one load per plane, transposed in registers
            const int quad = tid & 15;
            int64_t at[4];  // channel 0 of the four pixels
            const int64_t pl = px0 + 4 * quad;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int64_t px = pl + i < p.P ? pl + i : p.P - 1;
                const int64_t n = px / p.HW;
                at[i] = n * (int64_t)C * p.HW + (px - n * p.HW);
            }
            const bool whole = at[3] == at[0] + 3 && at[1] == at[0] + 1;  // all in one image, all inside the tensor
#pragma unroll 2
            for (int c = 4 * (tid >> 4); c < C; c += 64) {
                uint32_t v[4];
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const uint8_t* plane = p.in + (int64_t)(c + j < C ? c + j : C - 1) * p.HW;
                    if (whole) {
                        __builtin_memcpy(&v[j], plane + at[0], 4);
                    } else {
                        v[j] = (uint32_t)plane[at[0]] | ((uint32_t)plane[at[1]] << 8) | ((uint32_t)plane[at[2]] << 16) |
                               ((uint32_t)plane[at[3]] << 24);
                    }
                }
                const uint32_t a = __builtin_amdgcn_perm(v[1], v[0], 0x05010400u), b = __builtin_amdgcn_perm(v[1], v[0], 0x07030602u);
                const uint32_t d = __builtin_amdgcn_perm(v[3], v[2], 0x05010400u), e = __builtin_amdgcn_perm(v[3], v[2], 0x07030602u);
                const uint32_t w[4] = {__builtin_amdgcn_perm(d, a, 0x05040100u), __builtin_amdgcn_perm(d, a, 0x07060302u),
                                       __builtin_amdgcn_perm(e, b, 0x05040100u), __builtin_amdgcn_perm(e, b, 0x07060302u)};
#pragma unroll
                for (int i = 0; i < 4; i++)
                    *reinterpret_cast<uint32_t*>(s_px + (uint32_t)(4 * quad + i) * stride + c) = w[i] ^ 0x80808080u;
            }
        }
        __syncthreads();

        for (int rt0 = 0; rt0 < kts; rt0 += 4) {
            const int rt = rt0 + wave;
            if (rt < kts) {  // wavefront-uniform
                const unsigned long long* a8 = p.op8 + (size_t)(kt0 + rt) * NS * 64 + lane;
                // entries of contraction steps 2 pr and 2 pr + 1 (zero past the last)
                auto load_a = [&](int pr0, unsigned long long (&a)[8]) __attribute__((always_inline)) {
#pragma unroll
                    for (int i = 0; i < 8; i++) {
                        const int st = 2 * pr0 + i;
                        a[i] = st < NS ? a8[(size_t)st * 64] : 0ull;  // wavefront-uniform
                    }
                };
                v16i acc[PG];
#pragma unroll
                for (int g = 0; g < PG; g++) acc[g] = v16i{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
                auto multiply = [&](int pr0, const unsigned long long (&a)[8]) __attribute__((always_inline)) {
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        if (pr0 + i >= NP) break;  // wavefront-uniform
                        const v4i av = {(int)(uint32_t)a[2 * i], (int)(a[2 * i] >> 32), (int)(uint32_t)a[2 * i + 1], (int)(a[2 * i + 1] >> 32)};
#pragma unroll
                        for (int g = 0; g < PG; g++) {
                            const uint8_t* row = s_px + (uint32_t)(32 * g + l32) * stride + 32u * (uint32_t)(pr0 + i) + 8u * (uint32_t)half;
                            const uint2 b0 = *reinterpret_cast<const uint2*>(row), b1 = *reinterpret_cast<const uint2*>(row + 16);
                            const v4i bv = {(int)b0.x, (int)b0.y, (int)b1.x, (int)b1.y};
                            acc[g] = __builtin_amdgcn_mfma_i32_32x32x32_i8(av, bv, acc[g], 0, 0, 0);
                        }
                    }
                };
                unsigned long long a0[8], a1[8];
                load_a(0, a0);
                for (int pr = 0; pr < NP; pr += 8) {
                    load_a(pr + 4, a1);
                    multiply(pr, a0);
                    load_a(pr + 8, a0);
                    multiply(pr + 4, a1);
                }
                // this lane: pixels l32 and 32 + l32, results r0 .. r0 + 15 (coefficients, or channels for the inverse)
                const int r0 = (kt0 + rt) * 32 + 16 * half;
                const double* cst = s_const + rt * 32 + 16 * half;
                const int* sums = s_sum + rt * 32 + 16 * half;
#pragma unroll
                for (int g = 0; g < PG; g++) {
                    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                    for (int v = 0; v < 16; v++) {
                        uint32_t t;
                        if constexpr (INVERSE) t = activation_of(acc[g][v], sums[v], cst[v], p.factor, hk);
                        else t = level_of(acc[g][v], cst[v], p.factor, hk);
                        w[v >> 2] |= t << (8 * (v & 3));
                    }
                    const int pxl = 32 * g + l32;
                    if (hist && pxl < n_px) {
#pragma unroll
                        for (int v = 0; v < 16; v++)
                            if (r0 + v < C) atomicAdd(&wh[((w[v >> 2] >> (8 * (v & 3))) & 0xffu) << HS], 1u);
                    }
                    if constexpr (STAGED) {
                        uint32_t* dst = reinterpret_cast<uint32_t*>(s_stage + pxl * 132 + 32 * wave + 16 * half);
#pragma unroll
                        for (int i = 0; i < 4; i++) dst[i] = w[i];
                    } else {
                        if (pxl < n_px && r0 < C)
                            *reinterpret_cast<uint4*>(p.out + (size_t)(px0 + pxl) * (size_t)C + (size_t)r0) = make_uint4(w[0], w[1], w[2], w[3]);
                    }
                }
            }
            if constexpr (STAGED) {
                // rows [base, base + n_rows) of the 64 pixels: whole words, the last of a row byte by byte
                __syncthreads();
                const int base = (kt0 + rt0) * 32;
                int n_rows = 32 * (kts - rt0 < 4 ? kts - rt0 : 4);
                n_rows = base + n_rows <= C ? n_rows : C - base;
                if constexpr (INVERSE && LAYOUT == FMTC_NCHW) {
                    const int quad = tid & 15;
                    int64_t at[4];
                    const int64_t pl = px0 + 4 * quad;
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        const int64_t px = pl + i < p.P ? pl + i : p.P - 1;
                        const int64_t n = px / p.HW;
                        at[i] = n * (int64_t)C * p.HW + (px - n * p.HW);
                    }
                    const bool whole = at[3] == at[0] + 3 && at[1] == at[0] + 1;
                    for (int c = 4 * (tid >> 4); c < n_rows; c += 64) {
                        uint32_t v[4];
#pragma unroll
                        for (int i = 0; i < 4; i++) v[i] = *reinterpret_cast<const uint32_t*>(s_stage + (4 * quad + i) * 132 + c);
                        const uint32_t a = __builtin_amdgcn_perm(v[1], v[0], 0x05010400u), b = __builtin_amdgcn_perm(v[1], v[0], 0x07030602u);
                        const uint32_t d = __builtin_amdgcn_perm(v[3], v[2], 0x05010400u), e = __builtin_amdgcn_perm(v[3], v[2], 0x07030602u);
                        const uint32_t w[4] = {__builtin_amdgcn_perm(d, a, 0x05040100u), __builtin_amdgcn_perm(d, a, 0x07060302u),
                                               __builtin_amdgcn_perm(e, b, 0x05040100u), __builtin_amdgcn_perm(e, b, 0x07060302u)};
#pragma unroll
                        for (int j = 0; j < 4; j++) {
                            if (c + j >= n_rows) break;
                            uint8_t* plane = p.out + (int64_t)(base + c + j) * p.HW;
                            if (whole) {
                                __builtin_memcpy(plane + at[0], &w[j], 4);
                            } else {
#pragma unroll
                                for (int i = 0; i < 4; i++)
                                    if (pl + i < p.P) plane[at[i]] = (uint8_t)(w[j] >> (8 * i));
                            }
                        }
                    }
                } else {
                    for (int i = tid; i < PX * 32; i += 256) {
                        const int pxl = i >> 5, c = 4 * (i & 31);
                        if (pxl < n_px && c < n_rows) {
                            const uint32_t v = *reinterpret_cast<const uint32_t*>(s_stage + pxl * 132 + c);
                            uint8_t* dst = p.out + (size_t)(px0 + pxl) * (size_t)C + (size_t)(base + c);
                            if (c + 4 <= n_rows) __builtin_memcpy(dst, &v, 4);
                            else for (int e = 0; c + e < n_rows; e++) dst[e] = (uint8_t)(v >> (8 * e));
                        }
                    }
                }
                __syncthreads();  // the staged results have been read
            }
        }
        if constexpr (!STAGED) __syncthreads();  // everybody is done with the pixels: the next tile's may overwrite them
    }
    if (hist) {
        __syncthreads();
        if (tid < K) {
            uint32_t sum = 0;
            for (int w = 0; w < 4; w++)
                for (int c = 0; c < (1 << HS); c++) sum += s_hist[(((size_t)w * K + tid) << HS) + c];
            p.hist_parts[((size_t)blockIdx.y * gridDim.x + blockIdx.x) * K + tid] = sum;
        }
    }
}

template <bool INVERSE>
static hipError_t launch_int8_wide(int kernel_id, const Int8Params& p, int layout, int* n_parts, hipStream_t s) {
    Int8WideParams q{};
    q.p = p;
    q.px_tiles = (p.P + 63) / 64;
    // rows over workgroups until there are two of them per compute unit, at least one tile per wavefront
    const int most = (p.nct + 3) / 4;
    int gy = (int)(512 / (q.px_tiles < 512 ? q.px_tiles : 512));
    gy = gy > most ? most : (gy < 1 ? 1 : gy);
    q.kt_per = (((p.nct + gy - 1) / gy) + 3) / 4 * 4;
    gy = (p.nct + q.kt_per - 1) / q.kt_per;
    // (one row of partial counts per workgroup: no more of them than run at once, so that the pack kernel can add them up)
    const int64_t cap = (p.hist_parts ? 512 : 2048) / gy;
    const int64_t gx = q.px_tiles < cap ? q.px_tiles : cap;
    if (n_parts) *n_parts = (int)gx * gy;
    // histogram copies per wavefront: as many as 2 KB of LDS hold, 16 at most
    q.hist_shift = p.bits <= 5 ? 4 : (p.bits == 6 ? 3 : (p.bits == 7 ? 2 : 1));
    const bool planar = layout == FMTC_NCHW;  // of the activations: read by the forward kernel, written by the inverse
    const bool staged = (INVERSE && planar) || p.C % 16 != 0 || (reinterpret_cast<uintptr_t>(p.out) & 15u) != 0;
    const size_t lds = (size_t)q.kt_per * 32 * (INVERSE ? 12 : 8) + (p.hist_parts ? sizeof(uint32_t) * 4 * ((size_t)1 << (p.bits + q.hist_shift)) : 0) +
                       (staged ? 64 * 132 : 0) + (size_t)64 * (16 * p.NS + 8) + 64;
    const dim3 grid((unsigned)gx, (unsigned)gy), block(256);
#define FMTC_INT8_WIDE(LAY, ST)                                                                                 \
    do {                                                                                                        \
        hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_int8_wide<LAY, INVERSE, ST>),      \
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);              \
        if (ea != hipSuccess) return ea;                                                                        \
        return launch(kernel_id, k_int8_wide<LAY, INVERSE, ST>, grid, block, lds, s, q);                        \
    } while (0)
    if (planar) { if constexpr (!INVERSE) if (!staged) FMTC_INT8_WIDE(FMTC_NCHW, false); FMTC_INT8_WIDE(FMTC_NCHW, true); }
    if (staged) FMTC_INT8_WIDE(FMTC_NHWC, true);
    FMTC_INT8_WIDE(FMTC_NHWC, false);
#undef FMTC_INT8_WIDE
}

template <bool INVERSE>
static hipError_t launch_int8(int kernel_id, const Int8Params& p, int layout, int* n_parts, hipStream_t s) {
    if (!p.in || !p.out || !p.op8 || (!INVERSE && !p.row_off) || (INVERSE && (!p.col_sum || !p.mean_d)))
        return hipErrorInvalidValue;
    if (p.P < 1 || p.C < 1 || p.C > 1024 || p.NS != (p.C + 15) / 16 || p.nct != (p.C + 31) / 32 || p.HW < 1 ||
        p.n_tiles != (p.P + 31) / 32 || p.bits < 2 || p.bits > 8)
        return hipErrorInvalidValue;
    if (p.hist_parts && (INVERSE || !p.ctrl || !p.lookback)) return hipErrorInvalidValue;
    // Planar activations of more than 48 channels take the workgroup tile too: its loads are words of four pixels, not bytes
    // (quantizer, us: 64 channels, N = 256, 56 x 56 163 -> 97; 128, N = 256, 28 x 28 84 -> 35; 50, N = 100, 35 x 35 35 -> 28;
    // 64, N = 1 11.8 -> 5.7; but 28 channels, N = 100, 35 x 35 17 -> 22).  Channels last, up to 128 of them fit the registers
    // of one wavefront with the basis in LDS (64 channels, N = 256 38 there, 121 here).
    if (p.NS > 8 || (!INVERSE && layout == FMTC_NCHW && p.NS >= 4)) return launch_int8_wide<INVERSE>(kernel_id, p, layout, n_parts, s);
    int64_t gx = (p.n_tiles + 3) / 4;
    const int64_t cap = p.hist_parts ? kMaxHistParts : 2048;  // one histogram row per workgroup
    if (gx > cap) gx = cap;
    if (n_parts) *n_parts = (int)gx;
    const dim3 grid((unsigned)gx), block(256);
    const size_t lds = (size_t)p.nct * p.NS * 512 + (p.hist_parts ? sizeof(uint32_t) * 4 * kCopies * ((size_t)1 << p.bits) : 0);
#define FMTC_INT8(LAY)                                                                                          \
    do {                                                                                                        \
        if (lds > 32 * 1024) {                                                                                  \
            hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_int8_tiles<LAY, 8, INVERSE>),  \
                                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);          \
            if (ea != hipSuccess) return ea;                                                                    \
        }                                                                                                       \
        return launch(kernel_id, k_int8_tiles<LAY, 8, INVERSE>, grid, block, lds, s, p);                        \
    } while (0)
    if (layout == FMTC_NCHW) FMTC_INT8(FMTC_NCHW);  // (of the activations: read by the forward kernel, written by the inverse)
    FMTC_INT8(FMTC_NHWC);
#undef FMTC_INT8
}

hipError_t launch_quantize_u8(const Basis8Device& b, const uint8_t* d_xq, int64_t P, int64_t HW, int layout,
                              int bits, double g, uint8_t* d_syms, const CoderScratch* cs, int* n_parts,
                              hipStream_t s) {
    Int8Params p{};
    p.in = d_xq;
    p.out = d_syms;
    p.op8 = b.fwd8;
    p.row_off = b.row_off;
    p.col_sum = nullptr;
    p.mean_d = nullptr;
    p.P = P;
    p.HW = HW;
    p.n_tiles = (P + 31) / 32;
    p.C = b.C;
    p.NS = (b.C + 15) / 16;
    p.nct = (b.C + 31) / 32;
    p.bits = bits;
    p.factor = g;
    if (cs) {
        p.hist_parts = cs->hist_parts;
        p.ctrl = cs->ctrl;
        p.lookback = cs->lookback;
        p.n_groups = cs->n_groups;
        if (!p.hist_parts || !n_parts) return hipErrorInvalidValue;
    }
    return launch_int8<false>(K_QUANTIZE_U8, p, layout, n_parts, s);
}

hipError_t launch_reconstruct_u8(const Basis8Device& b, const uint8_t* d_syms, int64_t P, int64_t HW, int layout,
                                 int bits, double h, uint8_t* d_xq_hat, hipStream_t s) {
    Int8Params p{};
    p.in = d_syms;
    p.out = d_xq_hat;
    p.op8 = b.inv8;
    p.row_off = nullptr;
    p.col_sum = b.col_sum;
    p.mean_d = b.mean_d;
    p.P = P;
    p.HW = HW;
    p.n_tiles = (P + 31) / 32;
    p.C = b.C;
    p.NS = (b.C + 15) / 16;
    p.nct = (b.C + 31) / 32;
    p.bits = bits;
    p.factor = h;
    return launch_int8<true>(K_RECONSTRUCT_U8, p, layout, nullptr, s);
}

}  // namespace fmtc
