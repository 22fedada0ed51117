// Encoder front end: y = T(x - mu), uniform quantizer, symbol histogram
// (paper section 3; section 3.1 "Linear transform", "Quantization",
// "Variable length coding" for the statistics).
//
// The projection of all pixels is one dense contraction [C x C] . [C x P].  It
// runs on the f16 matrix cores (v_mfma_f32_32x32x16_f16) with every fp32 operand
// split into two f16 parts, which is as accurate as the fp32 matrix instruction
// and several times as fast; values that land too close to a rounding boundary
// for the fast pass to decide are recomputed in fp64 by the wavefront.  Four
// forms: one wavefront per 32 pixels with the basis in LDS (up to 160 channels),
// a 128 x 128 tile per workgroup (wider, a multiple of 16 channels), a small tile
// whose contraction the workgroup's wavefronts share out (few pixels, other channel
// counts), and 32 pixels with all channels in LDS (many pixels of such counts).
#include <atomic>
#include <cstdio>
#include <type_traits>

#include "fmtc_device.h"
#include "fmtc_internal.h"
#include "fmtc_pack_device.h"
#include "fmtc_stream_rules.h"

namespace fmtc {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Narrow tensors (at most 160 channels after padding to 32).  One wavefront owns 32 pixels
// for all coefficients.  The contraction runs on the f16 matrix cores with every fp32 operand
// split in two f16 parts, v = hi + lo / 2^11 (hi = v rounded to f16, lo = 2^11 times the rest
// rounded to f16: 22 significant bits in all, and the scaling keeps lo out of the subnormals):
//   y = sum T_hi x_hi  +  2^-11 (sum T_hi x_lo + sum T_lo x_hi)
// with exact products and fp32 accumulation (v_mfma_f32_32x32x16_f16, three instructions per
// 16 channels where the fp32 instruction needs eight four times as long).  Measured against
// fp64 the result is as close as the fp32 instruction's; what is left of the error is bounded
// per pixel by a multiple of |x - mu|_2 and handled by the exact decision below.
// Lane (pixel r, half h) loads its pixel's channels 16j + 8h .. 16j + 8h + 7, j = 0 .. Cpad/16 - 1,
// straight from global memory into registers (the contraction index may be walked in any order
// as long as both operands agree, so no transpose through LDS is needed); the next tile's loads
// are issued as soon as this tile's values are converted.  The basis sits in LDS in operand
// order (see pack_operand16 on the host), rows of a tile permuted so that a lane ends up with
// 16 consecutive coefficients of its pixel: one 16-byte store of symbols per tile.  The
// quantizer of tile kt is scheduled between the matrix instructions of tile kt+1.
// Histogram: interleaved LDS copies per wavefront.
// ---------------------------------------------------------------------------
// Bit pattern of u clamped between the patterns of lo and hi (positive floats: their order is the order of their
// patterns as signed integers).  Compared as integers so that every input ends in range: a negative u (sign bit set)
// below lo, a NaN at one end or the other -- the result indexes the histogram.
__device__ __forceinline__ uint32_t clamp_pattern(float u, float lo, float hi) {
    uint32_t c;  // (one instruction, where the compiler, which does not know lo <= hi, takes three)
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(c) : "v"(u), "s"(lo), "v"(hi));
    return c;
}

// The larger of two values, NaN if either is: the largest distance of a tile's values to their levels must not pass over one
// that the f16 parts could not hold (a basis entry beyond f16), so that it is decided exactly.
__device__ __forceinline__ float max_or_nan(float a, float b) { return __builtin_elementwise_maximum(a, b); }

constexpr int kHistLanes = 16;  // histogram copies per wavefront in the narrow-tensor kernel
constexpr int kFixList = 64;    // values per wavefront waiting for their exact decision

// LDS traffic of one wavefront completes in order; this keeps the compiler from moving it across the point
__device__ __forceinline__ void wave_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

struct RowParams {
    const float* x;
    const uint16_t* basis16;  // fwd16 packing
    const float* mu;          // [Cpad]
    const float* Trow;        // [C][C] row major, for the exact decisions
    int64_t P, HW;
    int C, bits;
    int active_tiles;         // 32-coefficient tiles up to the basis' last row that is not all zero
    float inv_delta, delta;
    float kappa;              // distance to a rounding boundary (in steps) below which a value of a pixel with
                              // |x - mu|_2 = 1 is decided exactly
    float tau_min;            // floor of that distance
    int64_t n_tiles;          // 32-pixel tiles
    uint8_t* syms;
    uint32_t* hist_parts;
    CoderCtrl* ctrl;
    unsigned long long* lookback;
    uint32_t n_groups;
    float x_scale;            // k_project_quantize_stream: S, a power of two (see there)
    float kappa_steps;        // ... and beside kappa, per the root of the sum over the steps (see band_of_roundings)
    PackParams pk;            // FUSED only: where the container goes
};

// FUSED: the same projection and quantizer, but the symbols of a chunk stay in LDS and the wavefront packs them
// with a code table fixed beforehand (no histogram, nothing but the container leaves the kernel).  Needs
// C = 32 NCT in {32, 64} and chunks of 4096 symbols, i.e. 4 / NCT whole pixel tiles; the grid must not exceed
// what the device holds at once (a chunk's position in the payload comes from the workgroups before it), and the
// look-back words and the control block must be clear when the kernel starts.
// WAVES wavefronts per workgroup (4, or 8 sharing one copy of a large basis); the register budget is set so that
// rows_waves_per_simd() wavefronts fit a SIMD: a wavefront spends most of a tile's time waiting for its pixels,
// and the second (third, fourth) one's arithmetic fills that time.
constexpr int rows_waves_per_simd(int nct, bool fused, int waves) {
    return fused ? 1 : (waves == 8 ? 2 : (nct == 1 ? 4 : (nct <= 3 ? 2 : 1)));
}
template <int NCT, int LAYOUT, bool VEC, bool FUSED = false, int WAVES = 4, int WPS = rows_waves_per_simd(NCT, FUSED, WAVES)>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(WPS, WPS)))
void k_project_quantize_rows(RowParams p) {
    constexpr int THREADS = WAVES * 64;
    static_assert(WAVES == 4 || (WAVES == 8 && !FUSED), "workgroup shape");
    // SEQ: contraction, then quantizer, tile by tile with one pair of accumulators (see process_tile)
    constexpr bool SEQ = WPS >= 3 || WAVES == 8;
    constexpr int NJ = NCT * 2;  // steps of 16 channels
    extern __shared__ __align__(16) uint4 basis16[];  // [NCT][NJ][2][64], then the histograms
    __shared__ __align__(16) float s_mu[NCT * 32];
    __shared__ uint32_t s_fix_list[WAVES][kFixList];
    __shared__ uint32_t s_fix_tile[WAVES][kFixList];
    __shared__ uint32_t s_red[WAVES * 256];  // per (wavefront, bin) sums of the histogram copies
    // Histogram: kHistLanes interleaved copies per wavefront (bin s of copy q at word s * kHistLanes + q), lane l
    // counts in copy l % kHistLanes.  Most symbols of a tile are the same few values: with one copy the LDS
    // would serialise up to 64 additions to one word per instruction, and the reads of the basis queue up
    // behind them.
    const int K = 1 << p.bits;
    uint32_t* whist = reinterpret_cast<uint32_t*>(basis16 + NCT * NJ * 2 * 64);  // [WAVES][K * kHistLanes]
    // FUSED: in place of the histograms, the four wavefronts' chunks of symbols (4096 bytes each, stream order)
    // and the packer's tables and images
    constexpr int TPC = FUSED ? 4 / NCT : 1;  // pixel tiles per chunk
    uint8_t* sym_tiles = reinterpret_cast<uint8_t*>(whist);
    PackShared& S = *reinterpret_cast<PackShared*>(sym_tiles + 4 * 4096);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wavefront-uniform by construction
    const int half = lane >> 5, l32 = lane & 31;
    const int C = p.C;
    // this lane's half of its pixel as loaded: xr[8j + e] = x[px][16j + 8h + e]
    float xr[NJ * 8];
    auto load_pixels = [&](int64_t tile) {
        const int64_t px = tile * 32 + l32;
        const bool px_ok = px < p.P;
        if constexpr (LAYOUT == FMTC_NHWC && VEC) {
            if (C == NCT * 32 && tile * 32 + 32 <= p.P) {  // wavefront-uniform: nothing to mask, nothing to fill
                const float4* row = reinterpret_cast<const float4*>(p.x + px * (NCT * 32)) + 2 * half;
#pragma unroll
                for (int j = 0; j < NJ; j++)
#pragma unroll
                    for (int q = 0; q < 2; q++) {
                        const float4 v = row[4 * j + q];
                        xr[8 * j + 4 * q] = v.x; xr[8 * j + 4 * q + 1] = v.y;
                        xr[8 * j + 4 * q + 2] = v.z; xr[8 * j + 4 * q + 3] = v.w;
                    }
                return;
            }
            const float4* row = reinterpret_cast<const float4*>(p.x + (px_ok ? px : 0) * C) + 2 * half;
#pragma unroll
            for (int j = 0; j < NJ; j++)
#pragma unroll
                for (int q = 0; q < 2; q++) {
                    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (px_ok && 16 * j + 8 * half + 4 * q < C) v = row[4 * j + q];
                    xr[8 * j + 4 * q] = v.x; xr[8 * j + 4 * q + 1] = v.y;
                    xr[8 * j + 4 * q + 2] = v.z; xr[8 * j + 4 * q + 3] = v.w;
                }
        } else if constexpr (LAYOUT == FMTC_NCHW && VEC && !FUSED) {
            // A multiple of 16 channels, 32-bit offsets (see k_project_quantize_stream for the addresses); rows past the
            // tensor repeat its last pixel.  With a 64-bit address and a test per value these registers spilled: 64
            // channels, N = 256, 56 x 56 95 -> 57 us; 96 channels, N = 64, 28 x 28 22 -> 14.6; 32 channels 14.4 -> 11.5.
            const uint32_t HW = (uint32_t)p.HW, P = (uint32_t)p.P, px0 = (uint32_t)tile * 32u;
            const uint32_t q = px0 + (uint32_t)l32 < P ? px0 + (uint32_t)l32 : P - 1u;
            const uint32_t n0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(px0 / HW)), n = q / HW;
            const uint32_t off = 4u * ((n - n0) * (uint32_t)C * HW + (q - n * HW) + 8u * (uint32_t)half * HW);
            const uint64_t plane_bytes = 4u * (uint64_t)HW;
            const char* image = reinterpret_cast<const char*>(p.x) + (uint64_t)n0 * (uint64_t)(uint32_t)C * plane_bytes;
#pragma unroll
            for (int j = 0; j < NJ; j++) {
                if (16 * j < C) {
#pragma unroll
                    for (int e = 0; e < 8; e++)
                        xr[8 * j + e] = *reinterpret_cast<const float*>(image + (uint64_t)(16 * j + e) * plane_bytes + off);
                } else {
#pragma unroll
                    for (int e = 0; e < 8; e++) xr[8 * j + e] = 0.f;
                }
            }
        } else {
            int64_t base = 0, stride = 1;
            if constexpr (LAYOUT == FMTC_NHWC) {
                base = (px_ok ? px : 0) * C;
            } else {
                const int64_t pp = px_ok ? px : 0;
                const int64_t n = pp / p.HW;
                base = n * (int64_t)C * p.HW + (pp - n * p.HW);
                stride = p.HW;
            }
            // (The lane's own part of the address first: what is left, (16 j + e) planes, is the same in all lanes and held in
            // scalar registers.  With a lane's channel times the plane kept in two registers for each value these were spilled: 33
            // channels, N = 674, 21 x 20, 5 bits 43 -> 29 us; 95, N = 300, 21 x 21, 6 bits 81 -> 59; 64 channels, one image of
            // 4096 x 4160, whose offsets 32 bits do not hold, 2618 -> 1265.)
            const float* at = p.x + (base + (int64_t)(8 * half) * stride);
#pragma unroll
            for (int j = 0; j < NJ; j++)
#pragma unroll
                for (int e = 0; e < 8; e++)
                    xr[8 * j + e] = (px_ok && 16 * j + 8 * half + e < C) ? at[(int64_t)(16 * j + e) * stride] : 0.f;
        }
    };
    // the first tile's pixels come from HBM: their loads go out before anything else
    int64_t tile = ((int64_t)blockIdx.x * WAVES + wave) * TPC;
    if (tile < p.n_tiles) load_pixels(tile);
    if constexpr (!FUSED) zero_coder_scratch(p.ctrl, p.lookback, p.n_groups);

    // the basis goes from global memory straight into LDS, 16 bytes per lane and instruction
    {
        const uint4* src = reinterpret_cast<const uint4*>(p.basis16);
#pragma unroll
        for (int i = 0; i < (NCT * NCT * 256 + THREADS - 1) / THREADS; i++)
            if (THREADS * i + 64 * wave < NCT * NCT * 256)  // whole wavefronts
                __builtin_amdgcn_global_load_lds(src + tid + THREADS * i, &basis16[THREADS * i + 64 * wave], 16, 0, 0);
    }
    if (tid < NCT * 32) s_mu[tid] = p.mu[tid];
    if constexpr (!FUSED) {
        for (int i = tid; i < WAVES * K * kHistLanes; i += THREADS) whist[i] = 0u;
    } else {
        S.tab[tid] = p.pk.enc_table[tid];
        if (tid == 0) {
            S.max_len = p.pk.static_max_len;
            S.payload_bits = 0ull;
        }
        if (blockIdx.x == 0) p.pk.stream[kHeaderBytes + tid] = (uint8_t)(p.pk.enc_table[tid] >> 56);  // the container's length table
        pack_clear_image(S, wave, lane);
    }

    const int zero_sym = 1 << (p.bits - 1);
    const float lo = (float)(-zero_sym), hi = (float)(zero_sym - 1), zero_f = (float)zero_sym;
    const float inv_delta = p.inv_delta;
    const float inv_delta_lo = p.inv_delta * (1.f / 2048.f);
    // Rounding, offset and conversion in one addition: for |t| < 2^22, t + (1.5 * 2^23 + 2^(b-1)) rounds (half to
    // even, the unit in the last place there being 1) to the number whose bit pattern is kMagicBits + 2^(b-1) +
    // rne(t); clamped between the patterns of symbol 0 and symbol 2^b - 1 its lowest byte is the symbol, and
    // subtracting the constant again gives rne(t) for the distance to the rounding boundary.  Larger |t| clamp the
    // same way (their distance is then meaningless and large: such a value is decided exactly, like any flagged one).
    constexpr uint32_t kMagicBits = 0x4B400000u;  // 1.5 * 2^23
    const float magic = 12582912.f + (float)zero_sym;
    const float magic_lo = 12582912.f, magic_hi = 12582912.f + (float)(2 * zero_sym - 1);
    uint32_t* wh0 = whist + wave * K * kHistLanes;          // this wavefront's histogram, copy 0
    uint32_t* wh = wh0 + (lane & (kHistLanes - 1));         // bin s of this lane's copy: wh[s * kHistLanes]
    // count of the symbol in the clamped pattern `ub` (kMagicBits + symbol): the LDS address is one shift-and-add
    // from the pattern itself (the constant is folded into the base; the arithmetic wraps)
    static_assert(kHistLanes * sizeof(uint32_t) == 64, "shift of the histogram address");
    typedef __attribute__((address_space(3))) uint32_t lds_u32;
    const uint32_t wh_magic = (uint32_t)(uintptr_t)(lds_u32*)wh - (kMagicBits << 6);
    // (one: 1, or 0 for a value that does not count -- no branch per value)
    auto hist_add = [&](uint32_t ub, uint32_t one) {
        __hip_atomic_fetch_add((lds_u32*)(uintptr_t)((ub << 6) + wh_magic), one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    uint32_t* fix_list = s_fix_list[wave];
    uint32_t* fix_tile = s_fix_tile[wave];
    uint32_t n_fix = 0;  // values listed, the same in all lanes

    // the first tile's pixels are on their way while the basis lands; every wavefront of the workgroup takes
    // part in the barrier, with or without a tile
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wavefront's part of the basis has landed in LDS
    __syncthreads();

    int64_t chunk_px0 = 0;  // FUSED: first pixel of the chunk this wavefront is working on
    // ---- exact decision where the fast pass can not be trusted (rare) ----
    // A tile notes the values that lie too close to a rounding boundary in the wavefront's list: tile, pixel
    // lane, coefficient and the symbol already stored and counted.  When the list is full, and after the
    // wavefront's last tile, the listed values are recomputed in fp64 (same arithmetic as the definition: sum of
    // T[k][c] * (x[c] - mu[c]), divided by the step), four per round, all loads of a round in flight
    // together, and the stored symbol and the histogram are patched where the decision differs.
    auto resolve_list = [&]() {
        // the symbols that get patched were stored by other lanes of this wavefront: those stores are
        // acknowledged before the patches go out (this also waits for the next tile's loads; rare)
        __builtin_amdgcn_s_waitcnt(0x0F70);
        const uint32_t n = n_fix;
        wave_sync_lds();
        for (uint32_t base = 0; base < n; base += 4) {
            const uint32_t idx = base + (uint32_t)(lane >> 4);
            const bool active = idx < n;
            const uint32_t e = active ? fix_list[idx] : 0u;
            const int k = (int)(e & 255u), pl = (int)((e >> 8) & 31u);
            const uint32_t old = e >> 13;
            const int64_t qpx = (int64_t)fix_tile[idx < (uint32_t)kFixList ? idx : 0] * 32 + pl;
            int64_t xbase, xstride;
            if constexpr (LAYOUT == FMTC_NHWC) {
                xbase = qpx * C;
                xstride = 1;
            } else {
                const int64_t n_img = qpx / p.HW;
                xbase = n_img * (int64_t)C * p.HW + (qpx - n_img * p.HW);
                xstride = p.HW;
            }
            float tv[2 * NCT], xv[2 * NCT], mv[2 * NCT];
#pragma unroll
            for (int it = 0; it < 2 * NCT; it++) {
                const int c = (lane & 15) + 16 * it;
                const bool in = active && c < C;
                tv[it] = in ? p.Trow[(size_t)k * C + c] : 0.f;
                xv[it] = in ? p.x[xbase + c * xstride] : 0.f;
                mv[it] = in ? s_mu[c] : 0.f;
            }
            double part = 0.0;
#pragma unroll
            for (int it = 0; it < 2 * NCT; it++) part += (double)tv[it] * ((double)xv[it] - (double)mv[it]);
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);  // stays inside the 16-lane group
            double qd = rint(part / (double)p.delta);
            qd = fmin(fmax(qd, (double)lo), (double)hi);
            const uint32_t sfix = (uint32_t)((int)qd + zero_sym);
            if (active && (lane & 15) == 0 && sfix != old) {
                if constexpr (FUSED) {
                    // the listed tiles are those of the chunk in this wavefront's LDS tile
                    sym_tiles[wave * 4096 + ((qpx - chunk_px0) * C + k)] = (uint8_t)sfix;
                } else {
                    atomicSub(&wh0[old * kHistLanes], 1u);
                    atomicAdd(&wh0[sfix * kHistLanes], 1u);
                    p.syms[qpx * C + k] = (uint8_t)sfix;
                }
            }
        }
        wave_sync_lds();
        n_fix = 0u;
    };
    auto process_tile = [&](const int64_t tile, const int64_t next_tile) {
        const int64_t px = tile * 32 + l32;
        const bool px_ok = px < p.P;
        // ---- mean removed, split into the two f16 parts (padding channels hold 0 - 0) ----
        halfx8 xh[NJ], xl[NJ];
        float n2 = 0.f;
        auto split = [&](bool clamp) {
            n2 = 0.f;
#pragma unroll
            for (int j = 0; j < NJ; j++)
#pragma unroll
                for (int q = 0; q < 2; q++) {
                    const float4 m = *reinterpret_cast<const float4*>(&s_mu[16 * j + 8 * half + 4 * q]);
                    const float mv[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        float v = xr[8 * j + 4 * q + i] - mv[i];
                        n2 = __builtin_fmaf(v, v, n2);
                        if (clamp) v = __builtin_amdgcn_fmed3f(v, -60000.f, 60000.f);
                        const _Float16 vh = (_Float16)v;
                        xh[j][4 * q + i] = vh;
                        // 2^11 (v - vh), exact (one multiply-add that takes the f16 operand as it is)
                        xl[j][4 * q + i] = (_Float16)__builtin_fmaf((float)vh, -2048.f, v * 2048.f);
                    }
                }
        };
        split(false);
        n2 += __shfl_xor(n2, 32, 64);  // the other half of the pixel
        // a pixel too large for f16 (or not finite) is decided exactly, every coefficient of it; its values are
        // clamped on the way into the matrix cores so that what comes out stays finite
        const bool force = !(n2 < 1.0e9f);
        if (__builtin_expect(__any(force), 0)) split(true);
        const float tau = fminf(fmaxf(p.kappa * __builtin_sqrtf(n2), p.tau_min), 0.125f);
        const float near_limit = force ? -1.f : 0.5f - tau;
        // the raw registers are free: the next tile's loads are in flight during this tile's arithmetic.  (With
        // three or more wavefronts per SIMD the others' arithmetic covers the loads, and registers held by loads in
        // flight across the whole tile are what would not fit: there the loads go out after the tile.)
        if (WPS < 3 && next_tile < p.n_tiles) load_pixels(next_tile);

        auto project_tile = [&](int kt, floatx16& am, floatx16& ac) {
            if (kt >= p.active_tiles) {  // all rows of the tile are zero (truncated basis): so are its coefficients
#pragma unroll
                for (int r = 0; r < 16; r++) { am[r] = 0.f; ac[r] = 0.f; }
                return;
            }
            // (the first step starts from the instruction's constant zero: no registers to clear)
            const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NJ; j++) {
                const uint4 th4 = basis16[((kt * NJ + j) * 2) * 64 + lane];
                const uint4 tl4 = basis16[((kt * NJ + j) * 2 + 1) * 64 + lane];
                const halfx8 th = __builtin_bit_cast(halfx8, th4), tl = __builtin_bit_cast(halfx8, tl4);
                am = __builtin_amdgcn_mfma_f32_32x32x16_f16(th, xh[j], j ? am : zero, 0, 0, 0);
                ac = __builtin_amdgcn_mfma_f32_32x32x16_f16(th, xl[j], j ? ac : zero, 0, 0, 0);
                ac = __builtin_amdgcn_mfma_f32_32x32x16_f16(tl, xh[j], ac, 0, 0, 0);
            }
        };
        // accumulator r = 4g + i of lane (pixel, h) is coefficient kt*32 + 16h + 4g + i of the pixel.
        // Quantizer, histogram and store of one tile with ragged edges (pixels past P, coefficients past C).
        auto quantize_tile = [&](const floatx16& am, const floatx16& ac, int kt, uint32_t (&word)[4]) -> float {
            const int k0 = kt * 32 + 16 * half;
            float maxd = 0.f;
#pragma unroll
            for (int g = 0; g < 4; g++) {
                word[g] = 0u;
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const float t = __builtin_fmaf(ac[4 * g + i], inv_delta_lo, am[4 * g + i] * inv_delta);
                    const float q = __builtin_rintf(t);  // round half to even
                    maxd = max_or_nan(maxd, fabsf(t - q));
                    const float qc = __builtin_amdgcn_fmed3f(q, lo, hi) + zero_f;  // clamped level, as a symbol
                    word[g] = __builtin_amdgcn_cvt_pk_u8_f32(qc, i, word[g]);
                }
            }
            if (px_ok) {
#pragma unroll
                for (int r = 0; r < 16; r++)
                    if (k0 + r < C) {
                        const uint32_t sy = (word[r >> 2] >> (8 * (r & 3))) & 255u;
                        if constexpr (FUSED) {
                            sym_tiles[wave * 4096 + ((px - chunk_px0) * C + k0 + r)] = (uint8_t)sy;
                        } else {
                            atomicAdd(&wh[sy * kHistLanes], 1u);
                            p.syms[px * C + k0 + r] = (uint8_t)sy;
                        }
                    }
            }
            return maxd;
        };
        auto note_tile = [&](const floatx16& am, const floatx16& ac, int kt, const uint32_t (&word)[4]) {
            const int k0 = kt * 32 + 16 * half;
            uint32_t near_mask = 0;
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const float t = __builtin_fmaf(ac[r], inv_delta_lo, am[r] * inv_delta);
                if (!(fabsf(t - __builtin_rintf(t)) <= near_limit) && px_ok && k0 + r < C) near_mask |= 1u << r;
            }
            // (one after the other in scalar registers: mostly it is one value)
            unsigned long long lanes = __ballot(near_mask != 0u);
#pragma unroll 1
            while (lanes) {
                const int from = __ffsll((long long)lanes) - 1;
                lanes &= lanes - 1ull;
                uint32_t mask = (uint32_t)__builtin_amdgcn_readlane((int)near_mask, from);
                uint32_t w[4];
#pragma unroll
                for (int g = 0; g < 4; g++) w[g] = (uint32_t)__builtin_amdgcn_readlane((int)word[g], from);
#pragma unroll 1
                while (mask) {
                    const int r = __ffs((int)mask) - 1;
                    mask &= mask - 1u;
                    const uint32_t of4 = r < 8 ? (r < 4 ? w[0] : w[1]) : (r < 12 ? w[2] : w[3]);
                    if (lane == 0) {
                        fix_list[n_fix] = (uint32_t)(kt * 32 + 16 * (from >> 5) + r) | ((uint32_t)(from & 31) << 8) |
                                          (((of4 >> (8 * (r & 3))) & 255u) << 13);
                        fix_tile[n_fix] = (uint32_t)tile;
                    }
                    n_fix++;
                    if (n_fix == (uint32_t)kFixList) resolve_list();
                }
            }
        };

        // whole pixel tile, and every lane's 16 coefficients of a tile all inside C or all outside (wavefront-uniform)
        const bool full = (tile * 32 + 32 <= p.P) && (C % 16 == 0);
        floatx16 am, ac;
        project_tile(0, am, ac);
        if (full && SEQ) {
            // Several wavefronts per SIMD: the others fill the shadow of this one's matrix instructions, and one
            // pair of accumulators (not two) is what lets them fit: contraction, then quantizer, tile by tile.
#pragma unroll
            for (int kt = 0; kt < NCT; kt++) {
                if (kt) project_tile(kt, am, ac);
                uint32_t word[4] = {0u, 0u, 0u, 0u};
                float maxd = 0.f;
                const bool k_ok = kt * 32 + 16 * half < C;  // false only in the upper half of a padded last tile
                uint32_t ub[16];
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    const float t = __builtin_fmaf(ac[r], inv_delta_lo, am[r] * inv_delta);
                    const float u = t + magic;  // round half to even
                    maxd = max_or_nan(maxd, fabsf(t - (u - magic)));
                    ub[r] = clamp_pattern(u, magic_lo, magic_hi);
                    if constexpr (!FUSED) hist_add(ub[r], k_ok ? 1u : 0u);
                }
#pragma unroll
                for (int g = 0; g < 4; g++)
                    word[g] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(ub[4 * g + 3], ub[4 * g + 2], 0x0c0c0400u),
                                                    __builtin_amdgcn_perm(ub[4 * g + 1], ub[4 * g], 0x0c0c0400u), 0x05040100u);
                if constexpr (FUSED) {
                    *reinterpret_cast<uint4*>(sym_tiles + wave * 4096 + ((px - chunk_px0) * C + kt * 32 + 16 * half)) =
                        make_uint4(word[0], word[1], word[2], word[3]);
                } else if (k_ok) {
                    *reinterpret_cast<uint4*>(p.syms + px * C + kt * 32 + 16 * half) =
                        make_uint4(word[0], word[1], word[2], word[3]);
                }
                if (__builtin_expect(__any(!(maxd <= near_limit) && k_ok), 0)) note_tile(am, ac, kt, word);
            }
        } else if (full) {
            // One wavefront per SIMD: nothing else fills the shadow of the matrix pipe, so the quantizer of tile
            // kt is issued between the matrix instructions of tile kt + 1 -- after each step of the contraction
            // the share of the previous tile's 16 values that keeps both in step.
#pragma unroll
            for (int kt = 0; kt < NCT; kt++) {
                floatx16 nm, nc;
#pragma unroll
                for (int r = 0; r < 16; r++) { nm[r] = 0.f; nc[r] = 0.f; }
                uint32_t word[4] = {0u, 0u, 0u, 0u};
                uint32_t ub[16];
                float maxd = 0.f;
                const bool k_ok = kt * 32 + 16 * half < C;  // false only in the upper half of a padded last tile
                auto quantize_value = [&](int r) {
                    const float t = __builtin_fmaf(ac[r], inv_delta_lo, am[r] * inv_delta);
                    const float u = t + magic;  // round half to even
                    maxd = max_or_nan(maxd, fabsf(t - (u - magic)));
                    ub[r] = clamp_pattern(u, magic_lo, magic_hi);
                    if constexpr (!FUSED) hist_add(ub[r], k_ok ? 1u : 0u);
                    if ((r & 3) == 3)
                        word[r >> 2] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(ub[r], ub[r - 1], 0x0c0c0400u),
                                                             __builtin_amdgcn_perm(ub[r - 2], ub[r - 3], 0x0c0c0400u), 0x05040100u);
                };
                if (kt + 1 < NCT) {
#pragma unroll
                    for (int j = 0; j < NJ; j++) {
                        const uint4 th4 = basis16[(((kt + 1) * NJ + j) * 2) * 64 + lane];
                        const uint4 tl4 = basis16[(((kt + 1) * NJ + j) * 2 + 1) * 64 + lane];
                        const halfx8 th = __builtin_bit_cast(halfx8, th4), tl = __builtin_bit_cast(halfx8, tl4);
                        nm = __builtin_amdgcn_mfma_f32_32x32x16_f16(th, xh[j], nm, 0, 0, 0);
                        nc = __builtin_amdgcn_mfma_f32_32x32x16_f16(th, xl[j], nc, 0, 0, 0);
                        nc = __builtin_amdgcn_mfma_f32_32x32x16_f16(tl, xh[j], nc, 0, 0, 0);
#pragma unroll
                        for (int r = 16 * j / NJ; r < 16 * (j + 1) / NJ; r++) quantize_value(r);
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < 16; r++) quantize_value(r);
                }
                // C is a multiple of 16: every lane's 16 symbols are a 16-byte aligned piece of its pixel's row
                if constexpr (FUSED) {
                    *reinterpret_cast<uint4*>(sym_tiles + wave * 4096 + ((px - chunk_px0) * C + kt * 32 + 16 * half)) =
                        make_uint4(word[0], word[1], word[2], word[3]);
                } else if (k_ok) {
                    *reinterpret_cast<uint4*>(p.syms + px * C + kt * 32 + 16 * half) =
                        make_uint4(word[0], word[1], word[2], word[3]);
                }
                if (__builtin_expect(__any(!(maxd <= near_limit) && k_ok), 0)) note_tile(am, ac, kt, word);
                am = nm;
                ac = nc;
            }
        } else if (SEQ) {
#pragma unroll
            for (int kt = 0; kt < NCT; kt++) {
                uint32_t word[4];
                if (kt) project_tile(kt, am, ac);
                const float maxd = quantize_tile(am, ac, kt, word);
                if (__builtin_expect(__any(!(maxd <= near_limit) && px_ok), 0)) note_tile(am, ac, kt, word);
            }
        } else {
#pragma unroll
            for (int kt = 0; kt < NCT; kt++) {
                floatx16 nm, nc;
                uint32_t word[4];
                if (kt + 1 < NCT) project_tile(kt + 1, nm, nc);
                const float maxd = quantize_tile(am, ac, kt, word);
                if (__builtin_expect(__any(!(maxd <= near_limit) && px_ok), 0)) note_tile(am, ac, kt, word);
                if (kt + 1 < NCT) { am = nm; ac = nc; }
            }
        }
    };
    if constexpr (FUSED) {
        // Chunk group g = the chunks 4g .. 4g + 3, one per wavefront; the workgroup takes groups blockIdx.x,
        // blockIdx.x + gridDim.x, ... in turn, so every group before one in progress is finished or in progress too.
        for (uint32_t group = blockIdx.x; group < p.pk.n_groups; group += gridDim.x) {
            const uint32_t ch = group * 4 + (uint32_t)wave;
            const int64_t tile0 = (int64_t)ch * TPC;
            const int64_t next_chunk_tile = ((int64_t)(group + gridDim.x) * 4 + wave) * TPC;  // past the end: no loads
            chunk_px0 = tile0 * 32;
            uint32_t clen = 0;
            if (ch < p.pk.n_chunks) {
                const uint64_t c0 = (uint64_t)ch * 4096u;
                clen = (uint32_t)((p.pk.V - c0 < 4096u) ? (p.pk.V - c0) : 4096u);
#pragma unroll
                for (int t = 0; t < TPC; t++) {
                    const int64_t tl = tile0 + t;
                    if (tl < p.n_tiles)  // wavefront-uniform
                        process_tile(tl, (t + 1 < TPC && tl + 1 < p.n_tiles) ? tl + 1
                                         : (group + gridDim.x < p.pk.n_groups ? next_chunk_tile : p.n_tiles));
                }
                if (n_fix) resolve_list();
            }
            wave_sync_lds();  // the symbols other lanes wrote precede the reads below
            // register q of lane l: symbols 256q + 4l .. + 3 of the chunk (C is a multiple of 32: clen one of 4)
            uint32_t w[16];
#pragma unroll
            for (int q = 0; q < 16; q++) {
                const uint32_t o = 256u * q + 4u * (uint32_t)lane;
                w[q] = (o + 4u <= clen) ? *reinterpret_cast<const uint32_t*>(sym_tiles + wave * 4096 + o) : 0u;
            }
            pack_group<kPackStatic>(S, p.pk, group, w, clen, []() {});
        }
        return;
    } else {
        for (; tile < p.n_tiles; tile += (int64_t)gridDim.x * WAVES) {
            const int64_t next_tile = tile + (int64_t)gridDim.x * WAVES;
            process_tile(tile, next_tile);
            if (WPS >= 3 && next_tile < p.n_tiles) load_pixels(next_tile);
        }
    }
    if (n_fix) resolve_list();
    __syncthreads();
    // One row of partial counts per workgroup: nothing to clear beforehand, no global atomics.  Every thread sums
    // the 16 copies of some (wavefront, bin) rows with 16-byte reads (a row is contiguous; reading one copy of
    // many bins instead would put all lanes on two banks), then the first K threads add the wavefronts.
    for (int row = tid; row < WAVES * K; row += THREADS) {
        const uint4* r4 = reinterpret_cast<const uint4*>(whist + (size_t)row * kHistLanes);
        uint32_t total = 0;
#pragma unroll
        for (int q = 0; q < kHistLanes / 4; q++) {
            const uint4 v = r4[q];
            total += (v.x + v.y) + (v.z + v.w);
        }
        s_red[row] = total;
    }
    __syncthreads();
    if (tid < K) {
        uint32_t total = 0;
#pragma unroll
        for (int q = 0; q < WAVES; q++) total += s_red[q * K + tid];
        p.hist_parts[(size_t)blockIdx.x * K + tid] = total;
    }
}

// ---------------------------------------------------------------------------
// 112 to 160 channels, a multiple of 16 of them: the same projection with the loops the other way
// round.  k_project_quantize_rows holds a whole pixel tile twice (the fp32 values of the next tile on their way in, the
// two f16 parts of this one) and one or two pairs of accumulators: 350 to 450 registers at four and five coefficient
// tiles, one wavefront per SIMD.  Here the channel steps are the outer loop: a step's eight channels per lane are
// converted when their turn comes and go into the accumulators of ALL coefficient tiles at once, and the registers they
// came in are requested again for the same step of the next tile, so that nearly a whole tile (14 to 20 KB per wavefront)
// is in flight at any time.
//
// ONE accumulator per coefficient: with v = S (x - mu), S a power of two,
//   S y = sum T_hi v_hi + sum T_hi v_lo + sum (2^11 T_lo) (2^-11 v_hi)
// where v_hi = v rounded to f16 and v_lo = v - v_hi rounded to f16, all three products at the same scale.  S follows from the
// quantizer's range and the norm of the basis' rows (see stream_scale).  Half the
// accumulator registers (80 of 160 at five coefficient tiles) are a second wavefront per SIMD, whose vector instructions
// issue while the first one's matrix instructions run (measured: a 32x32x16 product takes 32 clocks, and five independent
// vector instructions behind it none), and the quantizer takes one multiply-add where it joined two sums: u = acc g +
// magic, and the distance to the level is acc g - (u - magic) in another.  (All products being added to the large sum, its
// error is larger than that of two sums: in random data of 112 to 160 channels 2^-21.1 |x - mu|_2 against 2^-21.8 was the
// largest seen where a leading component holds most of the pixel, 2^-22.9 against 2^-23.7 where none does.  The distance
// below which a value is decided exactly follows from a bound: see band_of_roundings.)
//
// A pixel too large for f16 needs no clamp here: what its
// infinities make of the matrix product stays in its own column of outputs, all of which are decided exactly, and
// the clamp of the quantizer keeps the histogram index in range whatever the value.
// ---------------------------------------------------------------------------
// NJA: the tensor's channel count / 16 (the launcher checks it), 2 NCT - 1 or 2 NCT.
// Planar tensors: a channel's plane starts at a wavefront-uniform address (image of the tile's first pixel) and a lane's
// place in it is one 32-bit offset (the launcher checks that it fits), so the loads of 16 channels per lane and step
// take no 64-bit address each -- which is what the registers of k_project_quantize_rows go to there.
template <int NCT, int WAVES, int NJA, int LAYOUT>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(WAVES / 4, WAVES / 4)))
void k_project_quantize_stream(RowParams p) {
    constexpr int THREADS = WAVES * 64;
    constexpr int NJ = NCT * 2;        // steps of 16 channels in the basis operand (of which the first NJA hold channels)
    static_assert(NJA == NJ || NJA == NJ - 1, "channel count");
    constexpr int kSets = 4;           // histograms: wavefronts w and w + 4 share one
    extern __shared__ __align__(16) uint4 basis16[];  // [NCT][NJ][2][64], then the histograms
    __shared__ __align__(16) float s_mu[NCT * 32], s_mu_scaled[NCT * 32];  // mu, and -S mu
    __shared__ uint32_t s_fix_list[WAVES][kFixList];
    __shared__ uint32_t s_fix_tile[WAVES][kFixList];
    const int K = 1 << p.bits;
    uint32_t* whist = reinterpret_cast<uint32_t*>(basis16 + NCT * NJ * 2 * 64);  // [kSets][K * kHistLanes]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    constexpr int C = 16 * NJA;
    typedef float f4_t __attribute__((ext_vector_type(4)));

    // where a tile's pixels lie: the tile's first row, or (planar) channel 0 of the image that the tile starts in, the same
    // for all lanes, and this lane's offset from there (pixel and half); rows past the tensor repeat its last pixel, and are
    // never stored or counted
    struct Place {
        const char* base;
        uint32_t off;
    };
    auto place_of = [&](int64_t tile) __attribute__((always_inline)) {
        Place at{};
        if constexpr (LAYOUT == FMTC_NHWC) {
            const int64_t left = p.P - 1 - tile * 32;
            at.base = reinterpret_cast<const char*>(p.x) + (uint64_t)tile * (uint64_t)(32 * 4 * C);
            at.off = (uint32_t)(left < l32 ? (int)left : l32) * (uint32_t)(4 * C) + 32u * (uint32_t)half;
        } else {
            const uint32_t HW = (uint32_t)p.HW, P = (uint32_t)p.P, px0 = (uint32_t)tile * 32u;
            const uint32_t px = px0 + (uint32_t)l32 < P ? px0 + (uint32_t)l32 : P - 1u;
            const uint32_t n0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(px0 / HW)), n = px / HW;
            at.off = 4u * ((n - n0) * (uint32_t)C * HW + (px - n * HW) + 8u * (uint32_t)half * HW);
            at.base = reinterpret_cast<const char*>(p.x) + (uint64_t)n0 * (uint64_t)(4 * C) * HW;
        }
        return at;
    };
    // this lane's channels [16 j + 8 half, + 8) of its pixel
    auto load_step = [&](const Place& at, int j, f4_t (&raw)[2]) __attribute__((always_inline)) {
        if constexpr (LAYOUT == FMTC_NHWC) {
            raw[0] = *reinterpret_cast<const f4_t*>(at.base + 64 * j + at.off);
            raw[1] = *reinterpret_cast<const f4_t*>(at.base + 64 * j + 16 + at.off);
        } else {
            const uint64_t plane_bytes = 4u * (uint64_t)(uint32_t)p.HW;
            const char* plane = at.base + (uint64_t)(16 * j) * plane_bytes;
#pragma unroll
            for (int e = 0; e < 8; e++)
                raw[e >> 2][e & 3] = *reinterpret_cast<const float*>(plane + (uint64_t)e * plane_bytes + at.off);
        }
    };
    f4_t raw[NJA][2];
    const TileWalk walk(p.n_tiles, gridDim.x, WAVES, blockIdx.x, (uint32_t)wave);
    int64_t tile = walk.first;
    {
        const Place here = place_of(tile < p.n_tiles ? tile : 0);
#pragma unroll
        for (int j = 0; j < NJA; j++) load_step(here, j, raw[j]);
    }
    zero_coder_scratch(p.ctrl, p.lookback, p.n_groups);
    {
        const uint4* src = reinterpret_cast<const uint4*>(p.basis16);
#pragma unroll
        for (int i = 0; i < (NCT * NCT * 256 + THREADS - 1) / THREADS; i++)
            if (THREADS * i + 64 * wave < NCT * NCT * 256)  // whole wavefronts
                __builtin_amdgcn_global_load_lds(src + tid + THREADS * i, &basis16[THREADS * i + 64 * wave], 16, 0, 0);
    }
    const float S = p.x_scale;
    if (tid < NCT * 32) {
        const float m = p.mu[tid];
        s_mu[tid] = m;
        s_mu_scaled[tid] = -S * m;
    }
    for (int i = tid; i < kSets * K * kHistLanes; i += THREADS) whist[i] = 0u;

    const int zero_sym = 1 << (p.bits - 1);
    const float lo = (float)(-zero_sym), hi = (float)(zero_sym - 1);
    const float per_step = p.inv_delta / S;  // (exact: S is a power of two)
    float minus_one = -1.f;  // (unknown to the compiler, which then takes the multiply-add on the f16 part as it is)
    asm("" : "+s"(minus_one));
    constexpr uint32_t kMagicBits = 0x4B400000u;  // 1.5 * 2^23: see k_project_quantize_rows
    const float magic = 12582912.f + (float)zero_sym;
    const float magic_lo = 12582912.f, magic_hi = 12582912.f + (float)(2 * zero_sym - 1);
    uint32_t* wh0 = whist + (wave % kSets) * K * kHistLanes;
    uint32_t* wh = wh0 + (lane & (kHistLanes - 1));
    static_assert(kHistLanes * sizeof(uint32_t) == 64, "shift of the histogram address");
    typedef __attribute__((address_space(3))) uint32_t lds_u32;
    const uint32_t wh_magic = (uint32_t)(uintptr_t)(lds_u32*)wh - (kMagicBits << 6);
    auto hist_add = [&](uint32_t ub, uint32_t one) {
        __hip_atomic_fetch_add((lds_u32*)(uintptr_t)((ub << 6) + wh_magic), one, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    uint32_t* fix_list = s_fix_list[wave];
    uint32_t* fix_tile = s_fix_tile[wave];
    uint32_t n_fix = 0;  // values listed, the same in all lanes
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wavefront's part of the basis has landed in LDS
    __syncthreads();

    // exact decision of the listed values (as in k_project_quantize_rows)
    // LAST: after the last tile, where nothing else needs the registers.  Otherwise as many of a value's channels are in flight
    // together as fit beside the sums: all of them with one wavefront per SIMD, else a half or a third.  (Two steps at a time:
    // 144 channels, pixels of 25 times the quantizer's range, of which 1.4 % of the values are listed, 70000 pixels, 7 bits 1.44
    // times the kernel's time, 20000 pixels 1.35 times.)
    auto resolve_list = [&](auto last_c) __attribute__((always_inline)) {
        constexpr int kFlight = decltype(last_c)::value || WAVES == 4 ? NJA : (NCT == 4 ? (NJA + 1) / 2 : (NJA == 9 ? 3 : 5));
        __builtin_amdgcn_s_waitcnt(0x0F70);
        // (None of this rare path's addresses is to be kept in registers over the loop outside: where it starts from is made
        // unknown here.)
        int ln = lane;
        const float *x = p.x, *Trow = p.Trow;
        uint8_t* syms = p.syms;
        asm volatile("" : "+v"(ln), "+s"(x), "+s"(Trow), "+s"(syms));
        const uint32_t n = n_fix;
        wave_sync_lds();
        for (uint32_t base = 0; base < n; base += 4) {
            const uint32_t idx = base + (uint32_t)(ln >> 4);
            const bool active = idx < n;
            const uint32_t e = active ? fix_list[idx] : 0u;
            const int k = (int)(e & 255u), pl = (int)((e >> 8) & 31u);
            const uint32_t old = e >> 13;
            const int64_t qpx = (int64_t)fix_tile[idx < (uint32_t)kFixList ? idx : 0] * 32 + pl;
            int64_t xbase = qpx * C, xstride = 1;
            if constexpr (LAYOUT == FMTC_NCHW) {
                const int64_t n_img = active ? qpx / p.HW : 0;
                xbase = n_img * (int64_t)C * p.HW + (qpx - n_img * p.HW);
                xstride = p.HW;
            }
            double part = 0.0;
            const int k_in = active ? k : 0;
            if (!active) xbase = 0;  // (lanes without a value add up something that nobody looks at)
#pragma unroll 1
            for (int c0 = 0; c0 < NJA; c0 += kFlight) {
                float tv[kFlight], xv[kFlight];
#pragma unroll
                for (int q = 0; q < kFlight; q++) {
                    const int c = 16 * (c0 + q < NJA ? c0 + q : NJA - 1) + (ln & 15);
                    tv[q] = Trow[(size_t)k_in * C + c];
                    xv[q] = x[xbase + c * xstride];
                }
#pragma unroll
                for (int q = 0; q < kFlight; q++)
                    if (c0 + q < NJA) part += (double)tv[q] * ((double)xv[q] - (double)s_mu[16 * (c0 + q) + (ln & 15)]);
            }
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);  // stays inside the 16-lane group
            double qd = rint(part / (double)p.delta);
            qd = fmin(fmax(qd, (double)lo), (double)hi);
            const uint32_t sfix = (uint32_t)((int)qd + zero_sym);
            if (active && (ln & 15) == 0 && sfix != old) {
                atomicSub(&wh0[old * kHistLanes], 1u);
                atomicAdd(&wh0[sfix * kHistLanes], 1u);
                syms[qpx * C + k] = (uint8_t)sfix;
            }
        }
        wave_sync_lds();
        n_fix = 0u;
    };

    for (; tile < p.n_tiles; tile = walk.after(tile)) {
        const int64_t next_tile = walk.after(tile);
        const bool more = next_tile < p.n_tiles;
        const Place next = place_of(more ? next_tile : 0);
        const bool px_ok = l32 < p.P - tile * 32;
        f4_t coming[NJA][2];  // (in the registers of `raw`: see below)
        floatx16 acc[NCT];
        float n2 = 0.f, n2_steps = 0.f;  // the pixel's squares; their sums after every step added up
        const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NJA; j++) {
            // one step: this lane's eight channels converted, then into every coefficient tile's accumulators
            halfx8 vh, vl, vt;
#pragma unroll
            for (int q = 0; q < 2; q++) {
                const float4 m = *reinterpret_cast<const float4*>(&s_mu_scaled[16 * j + 8 * half + 4 * q]);
                const float mv[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const float v = __builtin_fmaf(raw[j][q][i], S, mv[i]);  // S (x - mu) as if rounded before the scaling
                    n2 = __builtin_fmaf(v, v, n2);
                    const _Float16 h = (_Float16)v;
                    vh[4 * q + i] = h;
                    vl[4 * q + i] = (_Float16)__builtin_fmaf((float)h, minus_one, v);  // v - h, exact
                }
            }
            // (converted, and their squares added up, before their registers are requested again: the compiler would rather do
            // that behind the branch, with a second set of registers for the loads)
            asm volatile("" : "+v"(vh), "+v"(vl), "+v"(n2));
            n2_steps += n2;
            if (more) load_step(next, j, coming[j]);
            vt = vh * (_Float16)(1.f / 2048.f);
#pragma unroll
            for (int kt = 0; kt < NCT; kt++) {
                // (a truncated basis' zero rows are multiplied like any others: their coefficients come out zero)
                const halfx8 th = __builtin_bit_cast(halfx8, basis16[((kt * NJ + j) * 2) * 64 + lane]);
                const halfx8 tl = __builtin_bit_cast(halfx8, basis16[((kt * NJ + j) * 2 + 1) * 64 + lane]);
                acc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(th, vl, j ? acc[kt] : zero, 0, 0, 0);
                acc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(tl, vt, acc[kt], 0, 0, 0);
                acc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(th, vh, acc[kt], 0, 0, 0);
            }
            // (The basis of two coefficient tiles is read ahead of its products, not of all five: their operands would not fit
            // the registers of two wavefronts per SIMD.  Nor would those of two steps.)
            __builtin_amdgcn_sched_group_barrier(0x100, 2 + 4, 0);  // LDS reads: the means, two coefficient tiles
#pragma unroll
            for (int kt = 0; kt < NCT; kt++) {
                __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);  // matrix products
                if (kt + 2 < NCT) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        n2 += __shfl_xor(n2, 32, 64);  // the other half of the pixel
        n2_steps += __shfl_xor(n2_steps, 32, 64);
        const bool force = !(n2 < 3.6e9f);  // too large for f16 (or not finite): every coefficient decided exactly
        // (not cut off at an eighth of a step, which pixels of 250 times the quantizer's range reach at 8 bits: the error is not
        // either)
        const float tau = fmaxf(p.kappa * __builtin_sqrtf(n2) + p.kappa_steps * __builtin_sqrtf(n2_steps), p.tau_min);
        const float near_limit = force ? -1.f : 0.5f - tau;

#pragma unroll
        for (int kt = 0; kt < NCT; kt++) {
            const bool k_ok = kt * 32 + 16 * half < C && px_ok;  // (C a multiple of 16: a lane's 16 coefficients all in or all out)
            const uint32_t one = k_ok ? 1u : 0u;  // (what does not count adds nothing: no branch per value)
            uint32_t word[4], ub[16];
            float maxd = 0.f;
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const float u = __builtin_fmaf(acc[kt][r], per_step, magic);  // round half to even
                maxd = max_or_nan(maxd, fabsf(__builtin_fmaf(acc[kt][r], per_step, magic - u)));
                ub[r] = clamp_pattern(u, magic_lo, magic_hi);
                hist_add(ub[r], one);
            }
#pragma unroll
            for (int g = 0; g < 4; g++)
                word[g] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(ub[4 * g + 3], ub[4 * g + 2], 0x0c0c0400u),
                                                __builtin_amdgcn_perm(ub[4 * g + 1], ub[4 * g], 0x0c0c0400u), 0x05040100u);
            if (k_ok)
                *reinterpret_cast<uint4*>(p.syms + (uint64_t)tile * (uint64_t)(32 * C) + kt * 32 + (uint32_t)(l32 * C + 16 * half)) =
                    make_uint4(word[0], word[1], word[2], word[3]);
            if (__builtin_expect(__any(!(maxd <= near_limit) && k_ok), 0)) {
                // the values too close to a rounding boundary go to the wavefront's list (resolved when it is full
                // and after the last tile)
                uint32_t near_mask = 0;
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    const float u = __builtin_fmaf(acc[kt][r], per_step, magic);
                    if (!(fabsf(__builtin_fmaf(acc[kt][r], per_step, magic - u)) <= near_limit) && k_ok) near_mask |= 1u << r;
                }
                // (one after the other in scalar registers: mostly it is one value.  Counted by shuffles, and placed by LDS
                // additions, they held the wavefront up for 0.7 us each time.)
                unsigned long long lanes = __ballot(near_mask != 0u);
#pragma unroll 1
                while (lanes) {
                    const int from = __ffsll((long long)lanes) - 1;
                    lanes &= lanes - 1ull;
                    uint32_t mask = (uint32_t)__builtin_amdgcn_readlane((int)near_mask, from);
                    uint32_t w[4];
#pragma unroll
                    for (int g = 0; g < 4; g++) w[g] = (uint32_t)__builtin_amdgcn_readlane((int)word[g], from);
#pragma unroll 1
                    while (mask) {
                        const int r = __ffs((int)mask) - 1;
                        mask &= mask - 1u;
                        const uint32_t of4 = r < 8 ? (r < 4 ? w[0] : w[1]) : (r < 12 ? w[2] : w[3]);
                        if (lane == 0) {
                            fix_list[n_fix] = (uint32_t)(kt * 32 + 16 * (from >> 5) + r) | ((uint32_t)(from & 31) << 8) |
                                              (((of4 >> (8 * (r & 3))) & 255u) << 13);
                            fix_tile[n_fix] = (uint32_t)tile;
                        }
                        n_fix++;
                        if (n_fix == (uint32_t)kFixList) resolve_list(std::false_type{});
                    }
                }
            }
        }
#pragma unroll
        for (int j = 0; j < NJA; j++) {
            raw[j][0] = coming[j][0];
            raw[j][1] = coming[j][1];
        }
    }
    if (n_fix) resolve_list(std::true_type{});
    __syncthreads();
    uint32_t* s_red = reinterpret_cast<uint32_t*>(basis16);  // (not read any more)
    for (int row = tid; row < kSets * K; row += THREADS) {
        const uint4* r4 = reinterpret_cast<const uint4*>(whist + (size_t)row * kHistLanes);
        uint32_t total = 0;
#pragma unroll
        for (int q = 0; q < kHistLanes / 4; q++) {
            const uint4 v = r4[q];
            total += (v.x + v.y) + (v.z + v.w);
        }
        s_red[row] = total;
    }
    __syncthreads();
    if (tid < K) {
        uint32_t total = 0;
#pragma unroll
        for (int q = 0; q < kSets; q++) total += s_red[q * K + tid];
        p.hist_parts[(size_t)blockIdx.x * K + tid] = total;
    }
}

// Planar tensors: do a lane's offsets from the start of the image that its pixel tile starts in (at most 32 pixels and
// an image further on, eight channels into it) and the pixel indices fit 32 bits?
static bool planar_offsets_fit(int C, int64_t P, int64_t HW) {
    return (uint64_t)C * ((uint64_t)HW + 32u) + 9u * (uint64_t)HW < (1ull << 30) && (uint64_t)P + 64u < (1ull << 31);
}

// Which of the narrow kernels takes a tensor.
struct RowsPlan {
    int nct, waves;
    bool stream;  // k_project_quantize_stream
    bool vec;     // k_project_quantize_rows: loads of four channels (planar: uniform plane addresses) without masks
};
static size_t rows_lds(int nct, int bits, int waves) {
    return sizeof(float) * (size_t)(32 * nct) * (32 * nct) + sizeof(uint32_t) * waves * kHistLanes * ((size_t)1 << bits);
}
static RowsPlan plan_rows(int C, int64_t P, int64_t HW, int layout, int bits) {
    RowsPlan r{};
    r.nct = (C + 31) / 32;
    const bool offsets_fit = layout == FMTC_NHWC || planar_offsets_fit(C, P, HW);
    const int64_t tiles = (P + 31) / 32;
    // Four and five coefficient tiles, a multiple of 16 channels: the streaming form, with eight wavefronts on one copy of
    // the basis where there are more tiles than SIMDs.  (Up to 1024 tiles four: 128 channels, 25088 pixels 12.7, 13.7 us with
    // eight.)  Kernel times, us, the other forms : this one, channels last, 6 bits: 128 channels, 200704 pixels 51.5 : 35.9 (8 bits
    // 67 : 42.6), 100352 33.0 : 25.1, 32992 18.1 : 14.5 (8 bits 18.9 : 18.3); 112, 32992 15.5 : 12.3.
    r.stream = r.nct >= 4 && C % 16 == 0 && offsets_fit;
    // 97 to 127 other channels, channels last: eight wavefronts on one copy of the basis, two per SIMD, each working tile by
    // tile with one pair of accumulators (two four-wavefront workgroups with a copy each would not fit a compute unit's
    // LDS).  (Planar tensors: the loads' addresses do not fit the registers; 8 bits: eight wavefronts' histograms do not
    // fit LDS beside the basis.)
    const bool eight = tiles > 1024 && (r.stream || (r.nct == 4 && layout == FMTC_NHWC && rows_lds(r.nct, bits, 8) <= 144 * 1024));
    r.waves = eight ? 8 : 4;
    // planar: vec = a multiple of 16 channels and offsets within the images of a pixel tile that fit 32 bits
    r.vec = layout == FMTC_NHWC ? C % 4 == 0 : C % 16 == 0 && offsets_fit;
    return r;
}

static hipError_t launch_rows(const BasisDevice& b, const float* d_x, int64_t P, int64_t HW, int layout, float delta,
                              int bits, uint8_t* d_syms, const CoderScratch& cs, int* n_parts, hipStream_t s) {
    RowParams p{};
    p.x = d_x;
    p.basis16 = b.fwd16;
    p.mu = b.mu;
    p.Trow = b.T;
    p.P = P;
    p.HW = HW;
    p.C = b.C;
    p.bits = bits;
    p.active_tiles = (b.active_rows + 31) / 32;
    p.inv_delta = (float)(1.0 / (double)delta);
    p.delta = delta;
    // The fast pass is off by three representation errors of 2^-22 |T[k]|_2 |x - mu|_2 each and the fp32 accumulation (2^-23 a
    // step of 16 channels and 2^-21 in all at most, mostly far less: random data are off by 2^-22 in all); values closer
    // than 2^-19 times these lengths (in steps) to a rounding boundary are decided in fp64 instead.  The floor covers the
    // rounding of the scaled value itself (magnitude up to 2^(b-1)).
    p.kappa = 1.9073486e-6f /* 2^-19 */ * b.row_norm * p.inv_delta;
    p.tau_min = 4.7683716e-7f /* 2^-21 */ * (float)(1 << (bits - 1));
    p.n_tiles = (P + 31) / 32;
    p.syms = d_syms;
    p.hist_parts = cs.hist_parts;
    p.ctrl = cs.ctrl;
    p.lookback = cs.lookback;
    p.n_groups = cs.n_groups;
    p.x_scale = stream_scale(delta, bits, b.row_norm);
    p.pk = PackParams{};
    if (!p.x || !p.basis16 || !p.mu || !p.Trow || !p.syms || !p.hist_parts || !p.ctrl || !p.lookback)
        return hipErrorInvalidValue;  // (a field left out would be a wild pointer on the device)
    const RowsPlan pl = plan_rows(b.C, P, HW, layout, bits);
    const int nct = pl.nct, waves = pl.waves;
    const bool eight = waves == 8, vec = pl.vec;
    const size_t lds = rows_lds(nct, bits, waves);
    // workgroups a compute unit holds at once: by registers (rows_waves_per_simd) and by LDS
    const size_t lds_static = (size_t)waves * (2 * kFixList + 256) * 4 + (size_t)nct * 128 + 512;
    int per_cu = eight ? 1 : rows_waves_per_simd(nct, false, 4);
    const int by_lds = (int)((160 * 1024) / (lds + lds_static));
    if (per_cu > by_lds) per_cu = by_lds < 1 ? 1 : by_lds;
    int64_t gx = (p.n_tiles + waves - 1) / waves;
    const int64_t cap = 256 * (int64_t)per_cu;
    if (gx > cap) gx = cap;
    *n_parts = (int)gx;
    hipError_t el = hipSuccess;
    if (pl.stream) {
        const double per_step = (double)b.row_norm * p.inv_delta / p.x_scale;
        p.kappa = (float)(kBandOfRest * per_step);  // (both of lengths of S (x - mu))
        p.kappa_steps = (float)(band_of_roundings(b.C / 16) * per_step);
        const bool whole = b.C == nct * 32;  // else 16 channels less
        const size_t slds = rows_lds(nct, bits, 4);  // (four histograms whatever the wavefronts)
        int64_t sgx = (p.n_tiles + waves - 1) / waves;
        if (sgx > 256) sgx = 256;  // one workgroup per compute unit (the basis takes 64 to 100 KB of its LDS)
        *n_parts = (int)sgx;
#define FMTC_STREAM_J(NCT, WV, NJA, LAY)                                                                         \
    do {                                                                                                         \
        hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_project_quantize_stream<NCT, WV, NJA, LAY>), \
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)slds);             \
        if (ea != hipSuccess) return ea;                                                                         \
        el = launch(K_PROJECT, k_project_quantize_stream<NCT, WV, NJA, LAY>, dim3((unsigned)sgx), dim3(WV * 64), slds, s, p); \
    } while (0)
#define FMTC_STREAM(NCT, WV, LAY)                                                                                \
    do {                                                                                                         \
        if (whole) FMTC_STREAM_J(NCT, WV, 2 * NCT, LAY); else FMTC_STREAM_J(NCT, WV, 2 * NCT - 1, LAY);          \
    } while (0)
#define FMTC_STREAM_W(NCT, LAY)                                                                                  \
    do {                                                                                                         \
        if (eight) FMTC_STREAM(NCT, 8, LAY); else FMTC_STREAM(NCT, 4, LAY);                                      \
    } while (0)
        if (layout == FMTC_NHWC) { if (nct == 5) FMTC_STREAM_W(5, FMTC_NHWC); else FMTC_STREAM_W(4, FMTC_NHWC); }
        else                     { if (nct == 5) FMTC_STREAM_W(5, FMTC_NCHW); else FMTC_STREAM_W(4, FMTC_NCHW); }
#undef FMTC_STREAM_W
#undef FMTC_STREAM_J
#undef FMTC_STREAM
        return el;
    }
#define FMTC_ROWS_W(NCT, LAY, VEC, WV)                                                                           \
    do {                                                                                                         \
        if (lds > 32 * 1024) {                                                                                   \
            hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_project_quantize_rows<NCT, LAY, VEC, false, WV>), \
                                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);          \
            if (ea != hipSuccess) return ea;                                                                     \
        }                                                                                                        \
        el = launch(K_PROJECT, k_project_quantize_rows<NCT, LAY, VEC, false, WV>, dim3((unsigned)gx), dim3(WV * 64), lds, s, p); \
    } while (0)
#define FMTC_ROWS(NCT, LAY, VEC) FMTC_ROWS_W(NCT, LAY, VEC, 4)
#define FMTC_ROWS_N(LAY, VEC)                                                                                    \
    do {                                                                                                         \
        if (nct == 1) FMTC_ROWS(1, LAY, VEC);                                                                    \
        else if (nct == 2) FMTC_ROWS(2, LAY, VEC);                                                               \
        else if (nct == 3) FMTC_ROWS(3, LAY, VEC);                                                               \
        else FMTC_ROWS(4, LAY, VEC);                                                                             \
    } while (0)
    if (eight) {
        if (vec) FMTC_ROWS_W(4, FMTC_NHWC, true, 8); else FMTC_ROWS_W(4, FMTC_NHWC, false, 8);
    } else if (nct == 5) {  // channels-last only (see launch_project_quantize)
        if (vec) FMTC_ROWS(5, FMTC_NHWC, true); else FMTC_ROWS(5, FMTC_NHWC, false);
    } else if (layout == FMTC_NHWC) { if (vec) FMTC_ROWS_N(FMTC_NHWC, true); else FMTC_ROWS_N(FMTC_NHWC, false); }
    else if (vec) {  // (four coefficient tiles with such offsets: the streaming form above)
        if (nct == 1) FMTC_ROWS(1, FMTC_NCHW, true); else if (nct == 2) FMTC_ROWS(2, FMTC_NCHW, true); else FMTC_ROWS(3, FMTC_NCHW, true);
    } else FMTC_ROWS_N(FMTC_NCHW, false);
#undef FMTC_ROWS_N
#undef FMTC_ROWS
#undef FMTC_ROWS_W
    return el;
}

// The fused kernel for a channel count and layout, its LDS size, and how many of its workgroups the device
// holds at once (0: shape not supported or the query failed).
static int fused_kernel_for(int C, int layout, const void** fn_out, size_t* lds_out) {
    if (!(C == 64 || (C == 32 && layout == FMTC_NHWC))) return 0;
    const int nct = C / 32;
    const size_t lds = sizeof(float) * (size_t)C * C + 4 * 4096 + sizeof(PackShared);
    const void* fn = nct == 1 ? reinterpret_cast<const void*>(&k_project_quantize_rows<1, FMTC_NHWC, true, true>)
                     : layout == FMTC_NHWC ? reinterpret_cast<const void*>(&k_project_quantize_rows<2, FMTC_NHWC, true, true>)
                                           : reinterpret_cast<const void*>(&k_project_quantize_rows<2, FMTC_NCHW, true, true>);
    *fn_out = fn;
    *lds_out = lds;
    static std::atomic<int> resident[2][2];  // (zero-initialised; every thread computes the same values)
    std::atomic<int>& slot = resident[layout == FMTC_NHWC][nct - 1];
    int cap = slot.load(std::memory_order_relaxed);
    if (!cap) {
        int dev = 0, cus = 0, per_cu = 0;
        if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
            hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, 256, lds) != hipSuccess || cus < 1 || per_cu < 1)
            return 0;
        cap = cus;  // one workgroup per compute unit, whatever more would fit
        slot.store(cap, std::memory_order_relaxed);
    }
    return cap;
}

// The one-kernel encoder is used where every chunk group gets a workgroup of its own: its workgroups work through
// their groups in lock step (project, pack, wait for the position, store), which loses to two specialised kernels for
// tensors that the device does not hold at once (135 us against 60 + 40 us at 1568 groups); below, where few groups leave most
// of the device idle while each walks its three phases, and wherever the projection is quicker in another form.  What is
// left, whole calls, one kernel against two, us: 64 channels, channels last, 4 / 6 / 8 bits 20.4 : 19.0 / 21.5 : 20.3 /
// 23.6 : 23.1 (128 groups), 20.2 : 20.6 / 21.3 : 22.1 / 23.8 : 27.2 (160), 22.0 : 22.4 / 22.8 : 23.5 / 25.1 : 28.8 (256);
// planar 24.7 : 21.9 (160, 6 bits), 27.3 : 24.0 and 27.3 : 28.4 (128 and 160, 8 bits); 32 channels, channels last, 160 groups
// 19.4 : 18.4 / 21.2 : 19.9 / 22.5 : 22.8, 256 at 8 bits 23.5 : 25.1, planar 26.4 : 25.0; 128 channels, 13 groups 24.5 :
// 16.9, 256 26.9 : 26.2, planar 28.9 : 24.7.
bool encode_static_fused_applies(int C, int layout, int bits, uint32_t chunk_syms, uint32_t n_groups) {
    const void* fn;
    size_t lds;
    if (chunk_syms != 4096u || n_groups <= 144u || (bits < 8 && !(C == 64 && layout == FMTC_NHWC))) return false;
    const int cap = fused_kernel_for(C, layout, &fn, &lds);
    return cap > 0 && n_groups <= (uint32_t)cap;
}

// Projection, quantizer and packing with a table fixed beforehand as one kernel.  Returns hipErrorNotSupported
// where encode_static_fused_applies() says no.
hipError_t launch_encode_static_fused(const BasisDevice& b, const float* d_x, int64_t N, int64_t HW, int layout,
                                      float delta, int bits, const CoderScratch& cs, const PackParams& pk,
                                      hipStream_t s) {
    const int64_t P = N * HW;
    const void* fn = nullptr;
    size_t lds = 0;
    const int cap = fused_kernel_for(b.C, layout, &fn, &lds);
    if (cap <= 0 || pk.chunk_syms != 4096u || pk.n_groups > (uint32_t)cap) return hipErrorNotSupported;
    RowParams p{};
    p.x = d_x;
    p.basis16 = b.fwd16;
    p.mu = b.mu;
    p.Trow = b.T;
    p.P = P;
    p.HW = HW;
    p.C = b.C;
    p.bits = bits;
    p.active_tiles = (b.active_rows + 31) / 32;
    p.inv_delta = (float)(1.0 / (double)delta);
    p.delta = delta;
    p.kappa = 1.9073486e-6f /* 2^-19 */ * b.row_norm * p.inv_delta;  // see launch_rows
    p.tau_min = 4.7683716e-7f /* 2^-21 */ * (float)(1 << (bits - 1));
    p.n_tiles = (P + 31) / 32;
    p.syms = nullptr;
    p.hist_parts = nullptr;
    p.ctrl = cs.ctrl;
    p.lookback = cs.lookback;
    p.n_groups = cs.n_groups;
    p.pk = pk;
    if (!p.x || !p.basis16 || !p.mu || !p.Trow || !p.ctrl || !p.lookback || !pk.enc_table || !pk.stream || !pk.lookback ||
        !pk.ctrl)
        return hipErrorInvalidValue;  // (a field left out would be a wild pointer on the device)
    const uint32_t grid = pk.n_groups < (uint32_t)cap ? pk.n_groups : (uint32_t)cap;
    void* args[] = {(void*)&p};
    hipEvent_t ev_a = nullptr, ev_b = nullptr;
    if (prof_next(K_PROJECT, &ev_a, &ev_b))
        return hipExtLaunchKernel(fn, dim3(grid), dim3(256), args, lds, s, ev_a, ev_b, 0);
    return hipLaunchKernel(fn, dim3(grid), dim3(256), args, lds, s);
}

// ---------------------------------------------------------------------------
// Wide tensors whose channel count is a multiple of 16: the projection as a tiled matrix product.
// A pixel's channels fit neither a wavefront's registers nor (for more than a few pixels) LDS, so
// the contraction index is cut instead.  A workgroup owns a tile of 128 coefficients x 128 pixels
// and walks the channels 32 at a time.  What a step needs goes from L2 / HBM straight into a ring
// of LDS slots, with no registers in between:
//   basis   16 KB in operand order;
//   pixels  16 KB of fp32: the 128 bytes of a pixel as one line.  Eight lanes fetch a line, in an
//           order that depends on the pixel (piece index XOR pixel modulo 8): its pieces then lie
//           in LDS where the operand reads of eight pixels meet all banks.
// (Steps of 16 channels, every lane fetching its own operand entry, touched 32 lines per load and
// used 32 bytes of each: the loads' passage through the cache bounded the step, whatever else was
// changed -- 0.57 us for 192 ns of matrix instructions.)
// A lane reads its sixteen values back, removes the mean and cuts them in their two f16 parts, in
// registers.  The waits count loads in flight (they complete in order), so every wavefront issues the
// same loads in the same order whatever part of its tile lies outside the tensor: addresses are
// clamped.  Quantizer, histogram, stores and exact decisions as in the narrow-tensor kernel: a lane
// ends up with 16 consecutive coefficients of its pixel.
// Each of the four wavefronts holds all 128 coefficients of its 32 pixels: twice the operand bytes of a
// 64 x 64 quarter are read from LDS, but a pixel is converted once, by the wavefront that multiplies
// it, and the conversion's round trip through LDS and its barrier go.  Two workgroups per compute unit:
// one converts while the other's matrix instructions run.  Measured against the 16-channel form, us:
// C = 256, N = 256, 14 x 14, 4 bits 44.6 -> 39.5 (planar, 8 bits 91 -> 73); C = 960, N = 256 458 -> 391;
// C = 176, N = 128, 28 x 28 62 -> 49.  At C = 960 that is 0.71 PFLOP/s of f16 products; the step's operand
// reads, conversion and matrix instructions do not overlap within a wavefront.
// ---------------------------------------------------------------------------
struct GemmParams {
    const float* x;
    const uint4* basis16;  // fwd16 packing: [ncs][NJ][2][64]
    const float* mu;       // [Cpad]
    const float* Trow;
    int64_t P, HW;
    int C, ncs, NJ, bits;
    int64_t n_pt, n_ptg;   // 32-pixel tiles, groups of four of them
    float inv_delta, delta, kappa, tau_min;
    int hist_shift;
    uint8_t* syms;
    uint32_t* hist_parts;
    CoderCtrl* ctrl;
    unsigned long long* lookback;
    uint32_t n_groups;
};

constexpr int kGemmFix = 64;  // values per wavefront waiting for their exact decision

constexpr int kGemmSlotBytes = 32 * 1024;
template <int LAYOUT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_project_quantize_gemm4(GemmParams p) {
    constexpr int WAVES = 4, THREADS = 64 * WAVES;
    constexpr int KT = 4;                              // coefficient tiles: all of the workgroup's in every wavefront
    constexpr int SLOTS = 2;
    constexpr int AL = 4;                              // a wavefront's transfers of a step's basis
    constexpr int XL = LAYOUT == FMTC_NHWC ? 4 : 16;   // ... and of its pixels
    extern __shared__ __align__(16) uint8_t dyn_lds[];
    // ring: slot = basis [coefficient tile][16-channel half][part][64], then pixels [pixel tile][256 pieces]; then the
    // mean [Cpad], then histogram copies [WAVES][K << HS]
    typedef uint4 Slot[32][64];
    Slot* ring = reinterpret_cast<Slot*>(dyn_lds);
    static_assert(sizeof(Slot) == kGemmSlotBytes, "slot size");
    float* s_mu = reinterpret_cast<float*>(dyn_lds + sizeof(Slot) * SLOTS);
    __shared__ uint32_t s_fix_a[WAVES][kGemmFix], s_fix_px[WAVES][kGemmFix], s_fix_count[WAVES];

    zero_coder_scratch(p.ctrl, p.lookback, p.n_groups);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int C = p.C, NJ = p.NJ, K = 1 << p.bits, HS = p.hist_shift, HC = 1 << HS;
    const int xpt = wave;  // this wavefront's pixel tile
    const int kt0 = blockIdx.y * 4;
    const int NS = (C + 31) / 32;                       // steps of 32 channels
    const bool odd = (C & 31) != 0;                     // (C is a multiple of 16: the last step may hold 16 only)
    uint32_t* whist = reinterpret_cast<uint32_t*>(s_mu + 16 * NJ);
    for (int i = tid; i < WAVES * K * HC; i += THREADS) whist[i] = 0u;
    for (int i = tid; i < 16 * NJ; i += THREADS) s_mu[i] = p.mu[i];
    uint32_t* wh0 = whist + wave * K * HC;
    uint32_t* wh = wh0 + (lane & (HC - 1));
    uint32_t* fix_a = s_fix_a[wave];
    uint32_t* fix_px = s_fix_px[wave];
    uint32_t* fix_count = &s_fix_count[wave];
    if (lane == 0) *fix_count = 0u;
    __builtin_amdgcn_s_waitcnt(0x0F70);  // (the loads counted below start from none in flight)
    __syncthreads();

    const int zero_sym = 1 << (p.bits - 1);
    const float lo = (float)(-zero_sym), hi = (float)(zero_sym - 1);
    const float inv_delta = p.inv_delta, inv_delta_lo = p.inv_delta * (1.f / 2048.f);
    const float magic = 12582912.f + (float)zero_sym;  // rounding, offset and conversion in one addition: see k_project_quantize_rows
    const float magic_lo = 12582912.f, magic_hi = 12582912.f + (float)(2 * zero_sym - 1);

    // exact fp64 decision of the listed values, two per round (one per half): most lists hold one or two, and what a round
    // takes is the latency of its loads, at the end of the workgroup that is last, so they should all be in flight
    // together (C = 256 at N = 256: 42.7 us with four per round and 16 lanes each, 39.4 with four and 16-byte loads, 37.7)
    auto resolve_list = [&]() {
        __builtin_amdgcn_s_waitcnt(0x0F70);  // the symbols that get patched have been stored
        const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)*fix_count);
        for (uint32_t base = 0; base < n; base += 2) {
            const uint32_t idx = base + (uint32_t)half;
            const bool active = idx < n;
            const uint32_t e = active ? fix_a[idx] : 0u;
            const int k = (int)(e & 0xffffu);
            const uint32_t old = e >> 16;
            const int64_t qpx = active ? (int64_t)fix_px[idx] : 0;
            double part = 0.0;
            if constexpr (LAYOUT == FMTC_NHWC) {
                if (active)
#pragma unroll 8
                    for (int c = 4 * l32; c < C; c += 128) {
                        const float4 t = *reinterpret_cast<const float4*>(p.Trow + (size_t)k * C + c);
                        const float4 x = *reinterpret_cast<const float4*>(p.x + qpx * C + c);
                        const float4 m = *reinterpret_cast<const float4*>(s_mu + c);
                        part += ((double)t.x * ((double)x.x - (double)m.x) + (double)t.y * ((double)x.y - (double)m.y)) +
                                ((double)t.z * ((double)x.z - (double)m.z) + (double)t.w * ((double)x.w - (double)m.w));
                    }
            } else {
                const int64_t n_img = qpx / p.HW;
                const float* xp = p.x + n_img * (int64_t)C * p.HW + (qpx - n_img * p.HW);
                if (active)
#pragma unroll 16
                    for (int c = l32; c < C; c += 32)
                        part += (double)p.Trow[(size_t)k * C + c] * ((double)xp[(int64_t)c * p.HW] - (double)s_mu[c]);
            }
#pragma unroll
            for (int o = 16; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);  // stays inside the half
            double qd = rint(part / (double)p.delta);
            qd = fmin(fmax(qd, (double)lo), (double)hi);
            const uint32_t sfix = (uint32_t)((int)qd + zero_sym);
            if (active && l32 == 0 && sfix != old) {
                atomicSub(&wh0[old << HS], 1u);
                atomicAdd(&wh0[sfix << HS], 1u);
                p.syms[qpx * C + k] = (uint8_t)sfix;
            }
        }
        wave_sync_lds();
        if (lane == 0) *fix_count = 0u;
        wave_sync_lds();
    };

    for (int64_t ptg = blockIdx.x; ptg < p.n_ptg; ptg += gridDim.x) {
        const int64_t px0 = (ptg * 4 + xpt) * 32, px = px0 + l32;  // this lane's pixel
        const bool px_ok = px < p.P;
        // Where this lane fetches pixels for the ring: channels last, instruction i takes piece `xq` of pixel 8 i + lane / 8
        // of the tile; planar, the lane's own pixel.  Past the end of the tensor the last pixel is loaded.
        const int xq = (lane & 7) ^ (lane >> 3);
        const float* xsrc[LAYOUT == FMTC_NHWC ? XL : 1];
        if constexpr (LAYOUT == FMTC_NHWC) {
#pragma unroll
            for (int i = 0; i < XL; i++) {
                int64_t q = px0 + 8 * i + (lane >> 3);
                q = q < p.P ? q : p.P - 1;
                xsrc[i] = p.x + q * C;
            }
        } else {
            const int64_t q = px_ok ? px : p.P - 1, n_img = q / p.HW;
            xsrc[0] = p.x + n_img * (int64_t)C * p.HW + (q - n_img * p.HW);
        }
        // the wavefront's share of the 16 blocks of a step's basis (one coefficient tile); a tile past the end repeats the
        // last one, its results are dropped
        int kt_ld = kt0 + wave;
        kt_ld = kt_ld < p.ncs ? kt_ld : p.ncs - 1;
        const uint4* a_src = p.basis16 + (size_t)kt_ld * NJ * 128 + lane;
        // Everything step s needs, on its way into ring slot s % SLOTS.  Steps past the end repeat the last one, so that
        // every wavefront always has the same number of loads in flight.
        auto issue = [&](int s) {
            uint4(*slot)[64] = ring[s % SLOTS];
            s = s < NS ? s : NS - 1;
#pragma unroll
            for (int q = 0; q < AL; q++) load_to_lds<16>(a_src + (size_t)s * 256 + 64 * q, &slot[wave * AL + q][0]);
            if constexpr (LAYOUT == FMTC_NHWC) {
                int c = 32 * s + 4 * xq;
                c = c < C ? c : C - 4;  // (the missing half of a last step: any channels, they are not used)
#pragma unroll
                for (int i = 0; i < XL; i++) load_to_lds<16>(xsrc[i] + c, &slot[16 + 4 * xpt + i][0]);
            } else {
#pragma unroll
                for (int i = 0; i < XL; i++) {
                    const int e = i;  // value e of the operand entries of both 16-channel halves
                    int c = 32 * s + 16 * (e >> 3) + 8 * half + (e & 7);
                    c = c < C ? c : C - 1;
                    load_to_lds<4>(xsrc[0] + (int64_t)c * p.HW, reinterpret_cast<uint32_t*>(&slot[16 + 4 * xpt][0]) + 64 * e);
                }
            }
        };
        float n2 = 0.f;
        halfx8 xh[2], xl[2];
        // this lane's sixteen channels of step s: mean removed, cut in two f16 parts
        auto convert = [&](int s) {
            const uint4(*slot)[64] = ring[s % SLOTS] + 16 + 4 * xpt;
#pragma unroll
            for (int u = 0; u < 2; u++) {
                if (u == 1 && odd && s == NS - 1) break;  // wavefront-uniform
                const int c0 = 32 * s + 16 * u + 8 * half;
                float v[8];
                if constexpr (LAYOUT == FMTC_NHWC) {
                    const uint4* row = &slot[0][0] + 8 * l32;
                    const int q = 4 * u + 2 * half;
                    const float4 a = __builtin_bit_cast(float4, row[q ^ (l32 & 7)]), b = __builtin_bit_cast(float4, row[(q + 1) ^ (l32 & 7)]);
                    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
                } else {
                    const float* raw = reinterpret_cast<const float*>(&slot[0][0]) + 512 * u + lane;
#pragma unroll
                    for (int e = 0; e < 8; e++) v[e] = raw[64 * e];
                }
                const float4 m0 = *reinterpret_cast<const float4*>(&s_mu[c0]);
                const float4 m1 = *reinterpret_cast<const float4*>(&s_mu[c0 + 4]);
                const float m[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    // (rows past the tensor repeat its last pixel: their results are dropped.  No clamp of values beyond
                    // f16: what their infinities make of the products stays in the pixel's own column of outputs, and such
                    // a pixel is decided exactly in all coefficients, see n2)
                    const float d = v[e] - m[e];
                    n2 = __builtin_fmaf(d, d, n2);
                    const _Float16 h = (_Float16)d;
                    xh[u][e] = h;
                    xl[u][e] = (_Float16)__builtin_fmaf((float)h, -2048.f, d * 2048.f);  // 2^11 (d - h), exact, one mixed multiply-add
                }
            }
        };

        floatx16 am[KT], ac[KT];
#pragma unroll
        for (int a = 0; a < KT; a++)
#pragma unroll
            for (int r = 0; r < 16; r++) { am[a][r] = 0.f; ac[a][r] = 0.f; }
        auto multiply = [&](int s) {
            const uint4(*sa)[64] = ring[s % SLOTS];
#pragma unroll
            for (int u = 0; u < 2; u++) {
                if (u == 1 && odd && s == NS - 1) break;  // wavefront-uniform
                halfx8 th[KT], tl[KT];
#pragma unroll
                for (int a = 0; a < KT; a++) {
                    th[a] = __builtin_bit_cast(halfx8, sa[4 * a + 2 * u][lane]);
                    tl[a] = __builtin_bit_cast(halfx8, sa[4 * a + 2 * u + 1][lane]);
                }
#pragma unroll
                for (int a = 0; a < KT; a++) {
                    am[a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(th[a], xh[u], am[a], 0, 0, 0);
                    ac[a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(th[a], xl[u], ac[a], 0, 0, 0);
                }
#pragma unroll
                for (int a = 0; a < KT; a++) ac[a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(tl[a], xh[u], ac[a], 0, 0, 0);
            }
        };
        // (one step ahead: the other workgroup of the compute unit works while this one waits)
        issue(0);
        for (int s = 0; s < NS; s++) {
            wait_loads<0>();  // step s has landed (this wavefront's part)
            __syncthreads();  // everybody's has, and everybody is done with the slot of step s - 1
            issue(s + 1);
            convert(s);
            multiply(s);
        }
        wait_loads<0>();  // the repeated loads of the last steps too
        __syncthreads();  // all wavefronts are done with the stages: the next group's first loads may overwrite them
        n2 += __shfl_xor(n2, 32, 64);  // the other half of the pixel

        // ---- quantizer, histogram, stores: accumulator r of lane (pixel, h) is coefficient kt*32 + 16h + r ----
        const bool force = !(n2 < 1.0e9f);  // too large for f16, or not finite: every coefficient decided exactly
        const float tau = fminf(fmaxf(p.kappa * __builtin_sqrtf(n2), p.tau_min), 0.125f);
        const float near_limit = force ? -1.f : 0.5f - tau;
#pragma unroll
        for (int a = 0; a < KT; a++) {
            const int kt = kt0 + a;
            const int k0 = kt * 32 + 16 * half;
            const bool ok = px_ok && k0 < C;  // C is a multiple of 16: all sixteen coefficients or none
            if (!__any(ok)) continue;
            uint32_t word[4], ub[16];
            float maxd = 0.f;
#pragma unroll
            for (int r = 0; r < 16; r++) {
                const float t = __builtin_fmaf(ac[a][r], inv_delta_lo, am[a][r] * inv_delta);
                const float u = t + magic;  // round half to even
                maxd = max_or_nan(maxd, fabsf(t - (u - magic)));
                ub[r] = clamp_pattern(u, magic_lo, magic_hi);  // (its lowest byte is the symbol: in range whatever u is)
                atomicAdd(&wh[(ub[r] & 255u) << HS], ok ? 1u : 0u);  // (no branch per value)
            }
#pragma unroll
            for (int g = 0; g < 4; g++)
                word[g] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(ub[4 * g + 3], ub[4 * g + 2], 0x0c0c0400u),
                                                __builtin_amdgcn_perm(ub[4 * g + 1], ub[4 * g], 0x0c0c0400u), 0x05040100u);
            if (ok) *reinterpret_cast<uint4*>(p.syms + px * C + k0) = make_uint4(word[0], word[1], word[2], word[3]);
            if (__builtin_expect(__any(!(maxd <= near_limit) && ok), 0)) {
                uint32_t near_mask = 0;
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    const float t = __builtin_fmaf(ac[a][r], inv_delta_lo, am[a][r] * inv_delta);
                    if (!(fabsf(t - __builtin_rintf(t)) <= near_limit) && ok) near_mask |= 1u << r;
                }
                // note the flagged values; the list is resolved when it could overflow and at the end
#pragma unroll 1
                for (int r = 0; r < 16; r++) {
                    const bool f = (near_mask >> r) & 1u;
                    const uint32_t incoming = (uint32_t)__popcll(__ballot(f));
                    if (incoming == 0) continue;
                    if (*fix_count + incoming > (uint32_t)kGemmFix) resolve_list();
                    if (f) {
                        const uint32_t slot = atomicAdd(fix_count, 1u);
                        fix_a[slot] = (uint32_t)(k0 + r) | (((word[r >> 2] >> (8 * (r & 3))) & 255u) << 16);
                        fix_px[slot] = (uint32_t)px;
                    }
                    wave_sync_lds();
                }
            }
        }
        if (*fix_count) resolve_list();
        __builtin_amdgcn_s_waitcnt(0x0F70);  // (nothing of this group is in flight when the next one's loads are counted)
    }
    __syncthreads();
    // one row of partial counts per workgroup (see the narrow-tensor kernel); the operand buffers are free now
    uint32_t* s_red = reinterpret_cast<uint32_t*>(dyn_lds);
    for (int row = tid; row < WAVES * K; row += THREADS) {
        uint32_t total = 0;
        for (int q = 0; q < HC; q++) total += whist[((size_t)row << HS) + q];
        s_red[row] = total;
    }
    __syncthreads();
    if (tid < K) {
        uint32_t total = 0;
#pragma unroll
        for (int q = 0; q < WAVES; q++) total += s_red[q * K + tid];
        p.hist_parts[(size_t)(blockIdx.y * gridDim.x + blockIdx.x) * K + tid] = total;
    }
}

// The same product with 8 wavefronts per 128 x 128 tile, two per SIMD, each 2 coefficient tiles x 1 pixel tile and a
// quarter of the conversion work: while one wavefront of a SIMD converts, the other's matrix instructions run.  More
// LDS operand reads per matrix instruction and one workgroup per compute unit: the faster of the two for tensors whose
// tiles all fit the device at once (few of them take the split form: see choose_projection; C = 960, N = 64, 7 x 7: 42.1 us; k_project_quantize_gemm4's steps of 32 channels
// with two wavefronts per pixel tile: 45.9, C = 1024, N = 8, 14 x 14: 46.9 and 49.2), the slower one beyond.
template <int LAYOUT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_project_quantize_gemm8(GemmParams p) {
    __shared__ __align__(16) uint4 stageA[3][8][64];     // per 16-channel step: (coefficient tile, part), operand order
    __shared__ __align__(16) uint4 stageX[3][8][64];     // per step: fp32 pixels as loaded, [wavefront][lane] (16 bytes each)
    __shared__ __align__(16) uint4 stageB[2][4][2][64];  // per step: (pixel tile, part), operand order
    __shared__ float s_n2[4][32];
    __shared__ uint32_t s_fix_a[8][kGemmFix], s_fix_px[8][kGemmFix], s_fix_count[8];
    extern __shared__ __align__(16) uint8_t dyn_lds[];    // mean [Cpad], then histogram copies [8][K << HS]
    constexpr int XL = LAYOUT == FMTC_NHWC ? 1 : 4;       // transfers of one step's pixels per wavefront
    constexpr int LD = 1 + XL;                            // ... of one step in all (basis: 1)

    zero_coder_scratch(p.ctrl, p.lookback, p.n_groups);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int C = p.C, NJ = p.NJ, K = 1 << p.bits, HS = p.hist_shift, HC = 1 << HS;
    // 8 wavefronts, two per SIMD (one converts while the other's matrix instructions run): wavefront w owns the
    // pair ktp of coefficient tiles and pixel tile xpt, and brings quarter xq of the 16 channels of xpt's pixels
    const int ktp = wave & 1, xpt = wave >> 1, xq = 2 * (wave & 1) + half;
    const int kt0 = blockIdx.y * 4;
    float* s_mu = reinterpret_cast<float*>(dyn_lds);
    uint32_t* whist = reinterpret_cast<uint32_t*>(dyn_lds) + 16 * NJ;
    for (int i = tid; i < 8 * K * HC; i += 512) whist[i] = 0u;
    for (int i = tid; i < 16 * NJ; i += 512) s_mu[i] = p.mu[i];
    uint32_t* wh0 = whist + wave * K * HC;
    uint32_t* wh = wh0 + (lane & (HC - 1));
    uint32_t* fix_a = s_fix_a[wave];
    uint32_t* fix_px = s_fix_px[wave];
    uint32_t* fix_count = &s_fix_count[wave];
    if (lane == 0) *fix_count = 0u;
    __syncthreads();

    const int zero_sym = 1 << (p.bits - 1);
    const float lo = (float)(-zero_sym), hi = (float)(zero_sym - 1), zero_f = (float)zero_sym;
    const float inv_delta = p.inv_delta, inv_delta_lo = p.inv_delta * (1.f / 2048.f);

    // exact fp64 decision of the listed values, four per round (one per 16-lane group)
    auto resolve_list = [&]() {
        __builtin_amdgcn_s_waitcnt(0x0F70);  // the symbols that get patched have been stored
        const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)*fix_count);
        for (uint32_t base = 0; base < n; base += 4) {
            const uint32_t idx = base + (uint32_t)(lane >> 4);
            const bool active = idx < n;
            const uint32_t e = active ? fix_a[idx] : 0u;
            const int k = (int)(e & 0xffffu);
            const uint32_t old = e >> 16;
            const int64_t qpx = active ? (int64_t)fix_px[idx] : 0;
            int64_t xbase, xstride;
            if constexpr (LAYOUT == FMTC_NHWC) {
                xbase = qpx * C;
                xstride = 1;
            } else {
                const int64_t n_img = qpx / p.HW;
                xbase = n_img * (int64_t)C * p.HW + (qpx - n_img * p.HW);
                xstride = p.HW;
            }
            double part = 0.0;
            if (active)
#pragma unroll 8  // independent loads of eight terms in flight together: the loop is all latency
                for (int c = lane & 15; c < C; c += 16)
                    part += (double)p.Trow[(size_t)k * C + c] * ((double)p.x[xbase + c * xstride] - (double)p.mu[c]);
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);  // stays inside the 16-lane group
            double qd = rint(part / (double)p.delta);
            qd = fmin(fmax(qd, (double)lo), (double)hi);
            const uint32_t sfix = (uint32_t)((int)qd + zero_sym);
            if (active && (lane & 15) == 0 && sfix != old) {
                atomicSub(&wh0[old << HS], 1u);
                atomicAdd(&wh0[sfix << HS], 1u);
                p.syms[qpx * C + k] = (uint8_t)sfix;
            }
        }
        wave_sync_lds();
        if (lane == 0) *fix_count = 0u;
        wave_sync_lds();
    };

    for (int64_t ptg = blockIdx.x; ptg < p.n_ptg; ptg += gridDim.x) {
        const int64_t pt0 = ptg * 4;
        floatx16 am[2], ac[2];
#pragma unroll
        for (int a = 0; a < 2; a++)
#pragma unroll
            for (int r = 0; r < 16; r++) { am[a][r] = 0.f; ac[a][r] = 0.f; }

        // this thread's pixel (of pixel tile pt0 + xpt); past the end of the tensor the last pixel is loaded
        // in its place and zeroed on conversion
        const int64_t px_raw = (pt0 + xpt) * 32 + l32;
        const bool px_ok = px_raw < p.P;
        const int64_t px_ld = px_ok ? px_raw : p.P - 1;
        int64_t xbase, xstride;
        if constexpr (LAYOUT == FMTC_NHWC) {
            xbase = px_ld * C;
            xstride = 1;
        } else {
            const int64_t n_img = px_ld / p.HW;
            xbase = n_img * (int64_t)C * p.HW + (px_ld - n_img * p.HW);
            xstride = p.HW;
        }
        int kt_ld = kt0 + (wave >> 1);
        kt_ld = kt_ld < p.ncs ? kt_ld : p.ncs - 1;  // a tile past the end repeats the last one; its results are dropped
        const uint4* a_src = p.basis16 + ((size_t)kt_ld * NJ * 2 + (wave & 1)) * 64 + lane;
        // Everything step s needs, on its way into ring slot s % 3: part wave % 2 of basis tile kt0 + wave / 2, and
        // channels [16 s + 4 xq, + 4) of this thread's pixel -- half of an operand entry.  Steps past the end
        // repeat the last one, so that every wavefront always has the same number of loads in flight.
        auto issue = [&](int s) {
            const int slot = s % 3;
            s = s < NJ ? s : NJ - 1;
            load_to_lds<16>(a_src + (size_t)s * 128, &stageA[slot][wave][0]);
            int c0 = 16 * s + 4 * xq;
            c0 = c0 < C ? c0 : 0;  // C is a multiple of 16: all four channels or none (then zeroed on conversion)
            if constexpr (LAYOUT == FMTC_NHWC) {
                load_to_lds<16>(p.x + xbase + c0, &stageX[slot][wave][0]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; e++)
                    load_to_lds<4>(p.x + xbase + (int64_t)(c0 + e) * xstride,
                                   reinterpret_cast<uint32_t*>(&stageX[slot][wave][0]) + 64 * e);
            }
        };
        float n2 = 0.f;
        // this thread's four channels of step s: mean removed, cut in two f16 parts, written into the pixel
        // operands (entry of lane (pixel, xq / 2), elements 4 (xq % 2) .. + 3)
        typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));
        auto convert = [&](int s) {
            const int c0 = 16 * s + 4 * xq;
            const bool ok = px_ok && c0 < C;
            float v[4];
            if constexpr (LAYOUT == FMTC_NHWC) {
                const float4 a = *reinterpret_cast<const float4*>(&stageX[s % 3][wave][lane]);
                v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
            } else {
                const float* raw = reinterpret_cast<const float*>(&stageX[s % 3][wave][0]) + lane;
#pragma unroll
                for (int e = 0; e < 4; e++) v[e] = raw[64 * e];
            }
            const float4 m0 = *reinterpret_cast<const float4*>(&s_mu[c0]);
            const float m[4] = {m0.x, m0.y, m0.z, m0.w};
            halfx4 vh, vl;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                float d = ok ? v[e] - m[e] : 0.f;
                n2 = __builtin_fmaf(d, d, n2);
                // (no clamp of values beyond f16: what their infinities make of the products stays in the pixel's own
                // column of outputs, and such a pixel is decided exactly in all coefficients, see n2)
                const _Float16 h = (_Float16)d;
                vh[e] = h;
                vl[e] = (_Float16)__builtin_fmaf((float)h, -2048.f, d * 2048.f);  // 2^11 (d - h), exact, one mixed multiply-add
            }
            uint2* dst = reinterpret_cast<uint2*>(&stageB[s & 1][xpt][0][l32 + 32 * (xq >> 1)]) + (xq & 1);
            dst[0] = __builtin_bit_cast(uint2, vh);
            dst[128] = __builtin_bit_cast(uint2, vl);  // part 1: 64 entries of 16 bytes further on
        };

        issue(0);
        issue(1);
        wait_loads<LD>();  // step 0 has landed (this wavefront's part)
        convert(0);
        for (int s = 0; s < NJ; s++) {
            // in flight: step s (unless s = 0) and step s + 1
            wait_loads<LD>();  // step s has landed
            __syncthreads();  // everybody's part of it, and everybody's pixel operands of step s; slot of step s - 1 is free
            if (s == 0 && tid < 128) s_n2[tid >> 5][tid & 31] = 0.f;  // everybody has left the previous group's epilogue
            issue(s + 2);
            const uint4(*sa)[64] = stageA[s % 3];
            halfx8 th[2], tl[2];
#pragma unroll
            for (int a = 0; a < 2; a++) {
                th[a] = __builtin_bit_cast(halfx8, sa[(2 * ktp + a) * 2][lane]);
                tl[a] = __builtin_bit_cast(halfx8, sa[(2 * ktp + a) * 2 + 1][lane]);
            }
            const halfx8 xh = __builtin_bit_cast(halfx8, stageB[s & 1][xpt][0][lane]);
            const halfx8 xl = __builtin_bit_cast(halfx8, stageB[s & 1][xpt][1][lane]);
#pragma unroll
            for (int a = 0; a < 2; a++) {
                am[a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(th[a], xh, am[a], 0, 0, 0);
                ac[a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(th[a], xl, ac[a], 0, 0, 0);
            }
#pragma unroll
            for (int a = 0; a < 2; a++) ac[a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(tl[a], xh, ac[a], 0, 0, 0);
            wait_loads<LD>();  // step s + 1 has landed
            if (s + 1 < NJ) convert(s + 1);  // into the operand buffer step s - 1 read, free since the barrier above
        }
        wait_loads<0>();  // the repeated loads of the last steps too
        // a pixel's sum of squares: its four quarters sit in two lanes of each of two wavefronts
        n2 += __shfl_xor(n2, 32, 64);
        if (half == 0) atomicAdd(&s_n2[xpt][l32], n2);
        __syncthreads();  // all wavefronts are done with the stages: the next group's first loads may overwrite them

        // ---- quantizer, histogram, stores: accumulator r of lane (pixel, h) is coefficient kt*32 + 16h + r ----
        {
            const int64_t pt = pt0 + xpt;
            if (pt < p.n_pt) {  // wavefront-uniform
            const int64_t px = pt * 32 + l32;
            const bool out_ok = px < p.P;
            const float pn2 = s_n2[xpt][l32];
            const bool force = !(pn2 < 1.0e9f);  // too large for f16, or not finite: every coefficient decided exactly
            const float tau = fminf(fmaxf(p.kappa * __builtin_sqrtf(pn2), p.tau_min), 0.125f);
            const float near_limit = force ? -1.f : 0.5f - tau;
#pragma unroll
            for (int a = 0; a < 2; a++) {
                const int kt = kt0 + 2 * ktp + a;
                if (kt >= p.ncs) continue;  // wavefront-uniform
                const int k0 = kt * 32 + 16 * half;
                const bool ok = out_ok && k0 < C;  // C is a multiple of 16: all sixteen coefficients or none
                uint32_t word[4] = {0u, 0u, 0u, 0u};
                uint32_t near_mask = 0;
#pragma unroll
                for (int r = 0; r < 16; r++) {
                    const float t = __builtin_fmaf(ac[a][r], inv_delta_lo, am[a][r] * inv_delta);
                    const float q = __builtin_rintf(t);  // round half to even
                    if (!(fabsf(t - q) <= near_limit)) near_mask |= 1u << r;
                    const float qc = __builtin_amdgcn_fmed3f(q, lo, hi) + zero_f;  // clamped level, as a symbol
                    word[r >> 2] = __builtin_amdgcn_cvt_pk_u8_f32(qc, r & 3, word[r >> 2]);
                    atomicAdd(&wh[((uint32_t)qc < (uint32_t)K ? (uint32_t)qc : (uint32_t)(K - 1)) << HS], ok ? 1u : 0u);  // (in range whatever qc is; no branch per value)
                }
                if (ok)
                    *reinterpret_cast<uint4*>(p.syms + px * C + k0) = make_uint4(word[0], word[1], word[2], word[3]);
                if (!ok) near_mask = 0;
                if (__builtin_expect(__any(near_mask != 0), 0)) {
                    // note the flagged values; the list is resolved when it could overflow and at the end
#pragma unroll 1
                    for (int r = 0; r < 16; r++) {
                        const bool f = (near_mask >> r) & 1u;
                        const uint32_t incoming = (uint32_t)__popcll(__ballot(f));
                        if (incoming == 0) continue;
                        if (*fix_count + incoming > (uint32_t)kGemmFix) resolve_list();
                        if (f) {
                            const uint32_t slot = atomicAdd(fix_count, 1u);
                            fix_a[slot] = (uint32_t)(k0 + r) | (((word[r >> 2] >> (8 * (r & 3))) & 255u) << 16);
                            fix_px[slot] = (uint32_t)px;
                        }
                        wave_sync_lds();
                    }
                }
            }
        }
        }
        if (*fix_count) resolve_list();  // before the next group's loads: the waits there count loads in flight
    }
    __syncthreads();
    // one row of partial counts per workgroup (see the narrow-tensor kernel); the operand buffers are free now
    uint32_t* s_red = reinterpret_cast<uint32_t*>(&stageA[0][0][0]);
    for (int row = tid; row < 8 * K; row += 512) {
        uint32_t total = 0;
        for (int q = 0; q < HC; q++) total += whist[((size_t)row << HS) + q];
        s_red[row] = total;
    }
    __syncthreads();
    if (tid < K)
        p.hist_parts[(size_t)(blockIdx.y * gridDim.x + blockIdx.x) * K + tid] =
            ((s_red[tid] + s_red[K + tid]) + (s_red[2 * K + tid] + s_red[3 * K + tid])) +
            ((s_red[4 * K + tid] + s_red[5 * K + tid]) + (s_red[6 * K + tid] + s_red[7 * K + tid]));
}

// Columns [c0, C) of the symbols [P][C] set to one value (c0 and C multiples of 16), and one row of partial
// counts that says so: what the tiled projection leaves out when the basis' last rows are all zero (a truncated
// basis: those coefficients are 0, their symbol the zero level).
__global__ __launch_bounds__(256) void k_fill_symbol_columns(uint8_t* __restrict__ syms, int64_t P, int C, int c0,
                                                             uint32_t value, int bits, uint32_t* __restrict__ hist_row) {
    const uint32_t v4 = value * 0x01010101u;
    const int64_t per_px = (C - c0) / 16;
    const int64_t n = P * per_px;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int64_t px = i / per_px, j = i - px * per_px;
        *reinterpret_cast<uint4*>(syms + (size_t)px * (size_t)C + (size_t)c0 + 16 * (size_t)j) = make_uint4(v4, v4, v4, v4);
    }
    if (blockIdx.x == 0 && (int)threadIdx.x < (1 << bits))
        hist_row[threadIdx.x] = threadIdx.x == value ? (uint32_t)(P * (int64_t)(C - c0)) : 0u;
}

// Workgroups of the tiled product over pixel groups and coefficient groups (gy_all; gy of them are computed: the others' rows
// of the basis are all zero), and whether those have eight wavefronts: while every tile has a compute unit of its own, four
// (two workgroups per compute unit) beyond.
struct GemmPlan {
    int gy, gy_all;
    bool eight;
};
static GemmPlan plan_gemm(int C, int64_t P, int active_rows) {
    GemmPlan g{};
    g.gy_all = ((C + 31) / 32 + 3) / 4;
    g.gy = ((active_rows + 31) / 32 + 3) / 4;
    g.gy = g.gy < 1 ? 1 : (g.gy > g.gy_all ? g.gy_all : g.gy);
    g.eight = ((P + 31) / 32 + 3) / 4 * g.gy <= 256;
    return g;
}

static hipError_t launch_gemm(const BasisDevice& b, const float* d_x, int64_t P, int64_t HW, int layout, float delta,
                              int bits, uint8_t* d_syms, const CoderScratch& cs, int* n_parts, hipStream_t s) {
    const int ncs = b.Cpad / 32, NJ = b.Cpad / 16;
    const int64_t n_pt = (P + 31) / 32;
    GemmParams p{};
    p.x = d_x;
    p.basis16 = reinterpret_cast<const uint4*>(b.fwd16);
    p.mu = b.mu;
    p.Trow = b.T;
    p.P = P;
    p.HW = HW;
    p.C = b.C;
    p.ncs = ncs;
    p.NJ = NJ;
    p.bits = bits;
    p.n_pt = n_pt;
    p.n_ptg = (n_pt + 3) / 4;
    p.inv_delta = (float)(1.0 / (double)delta);
    p.delta = delta;
    p.kappa = 1.9073486e-6f /* 2^-19 */ * b.row_norm * p.inv_delta;  // see launch_rows
    p.tau_min = 4.7683716e-7f /* 2^-21 */ * (float)(1 << (bits - 1));
    p.syms = d_syms;
    p.hist_parts = cs.hist_parts;
    p.ctrl = cs.ctrl;
    p.lookback = cs.lookback;
    p.n_groups = cs.n_groups;
    // every pointer the kernel follows is set (a field left out here would be a wild pointer on the device)
    if (!p.x || !p.basis16 || !p.mu || !p.Trow || !p.syms || !p.hist_parts || !p.ctrl || !p.lookback)
        return hipErrorInvalidValue;
    // groups of four coefficient tiles; those whose rows of the basis are all zero (truncation) are not computed:
    // k_fill_symbol_columns writes their symbols and counts
    const GemmPlan pl = plan_gemm(b.C, P, b.active_rows);
    const int gy_all = pl.gy_all, gy = pl.gy;
    int64_t gx = p.n_ptg;
    if (gx * gy_all > kMaxHistParts) gx = kMaxHistParts / gy_all;
    *n_parts = (int)(gx * gy) + (gy < gy_all ? 1 : 0);
    if (gy < gy_all) {
        const int c0 = gy * 128;  // < C, and C - c0 is a multiple of 16 like C
        const int64_t pieces = P * ((b.C - c0) / 16);
        int64_t blocks = (pieces + 255) / 256;
        blocks = blocks > 2048 ? 2048 : blocks;
        hipLaunchKernelGGL(k_fill_symbol_columns, dim3((unsigned)blocks), dim3(256), 0, s, d_syms, P, b.C, c0,
                           (uint32_t)(1 << (bits - 1)), bits, cs.hist_parts + (size_t)(gx * gy) * ((size_t)1 << bits));
        hipError_t ef = hipGetLastError();
        if (ef != hipSuccess) return ef;
    }
    const bool eight = pl.eight;
    const int waves = eight ? 8 : 4;
    // histogram copies per wavefront: as many as 2 KB of LDS hold, 16 at most, 2 at least
    int copies = 512 >> bits;
    copies = copies >= 16 ? 16 : (copies >= 8 ? 8 : (copies >= 4 ? 4 : 2));
    p.hist_shift = copies == 16 ? 4 : (copies == 8 ? 3 : (copies == 4 ? 2 : 1));
    const size_t lds = (eight ? 0 : 2 * (size_t)kGemmSlotBytes) + sizeof(float) * b.Cpad +
                       sizeof(uint32_t) * waves * copies * ((size_t)1 << bits);
    dim3 grid((unsigned)gx, (unsigned)gy);
    if (eight)
        return layout == FMTC_NHWC
                   ? launch(K_PROJECT, k_project_quantize_gemm8<FMTC_NHWC>, grid, dim3(512), lds, s, p)
                   : launch(K_PROJECT, k_project_quantize_gemm8<FMTC_NCHW>, grid, dim3(512), lds, s, p);
    const void* fn = layout == FMTC_NHWC ? reinterpret_cast<const void*>(&k_project_quantize_gemm4<FMTC_NHWC>)
                                         : reinterpret_cast<const void*>(&k_project_quantize_gemm4<FMTC_NCHW>);
    hipError_t ea = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (ea != hipSuccess) return ea;
    return layout == FMTC_NHWC ? launch(K_PROJECT, k_project_quantize_gemm4<FMTC_NHWC>, grid, dim3(256), lds, s, p)
                               : launch(K_PROJECT, k_project_quantize_gemm4<FMTC_NCHW>, grid, dim3(256), lds, s, p);
}

// ---------------------------------------------------------------------------
// Channel counts that are no multiple of 16, many pixels.  The contraction is the same f16 split as in the
// narrow-tensor kernel above (three v_mfma_f32_32x32x16_f16 per 16 channels, see there), but a pixel's channels do
// not fit a wavefront's registers: the workgroup (8 wavefronts) first brings a tile of 32 pixels, all channels,
// into LDS -- coalesced global reads, mean removed and split into the two f16 parts on the way, rows padded by 16
// bytes so that the 16-byte operand reads of 8 neighbouring pixels cover all banks -- then its wavefronts share out
// the coefficient tiles of the workgroup's range [kt0, kt0 + ktg) without further barriers; the basis streams from
// L2 in operand order one step ahead of its use.  Values too close to a rounding boundary are recomputed in fp64;
// the quantized tile is staged in LDS and leaves as whole rows of symbols.
// What bounds it: one workgroup per compute unit (LDS) from 480 channels on, so a tile's loads are not covered and a
// last round of few workgroups costs as much as a full one.  Its gain over the split form below: no wavefront waits for
// another one's exact decisions, and the pixels are read and converted once per 512 coefficients instead of once per 128.
// (Which of the two is used: see wide_form_is_ahead.)
// LAYOUT: FMTC_NHWC (C % 4 == 0: 16-byte loads of channels-last rows and 4-byte symbol stores are aligned) / FMTC_NCHW.
// ---------------------------------------------------------------------------
struct WideParams {
    const float* x;
    const uint16_t* basis16;  // fwd16 packing
    const float* mu;          // [Cpad]
    const float* Trow;        // [C][C] row major, for the exact decisions
    int64_t P, HW;
    int C, ncs, kt_per_group, bits;
    float inv_delta, delta, kappa, tau_min;
    int64_t px_tiles;
    uint8_t* syms;
    uint32_t* hist_parts;
    CoderCtrl* ctrl;
    unsigned long long* lookback;
    uint32_t n_groups;
};

constexpr int kWideThreads = 512, kWidePixels = 32;

// Workgroups of the kernel below for a tensor: the coefficient range is split over them only when the pixel tiles alone
// leave compute units idle, and to bound the staging rows (16 tiles).
struct WidePlan {
    int ktg, kgroups;
    int64_t px_tiles;
    size_t lds;
};
static WidePlan plan_wide(int C, int64_t P) {
    const int ncs = (C + 31) / 32;
    WidePlan w{};
    w.px_tiles = (P + kWidePixels - 1) / kWidePixels;
    w.kgroups = (int)((256 + w.px_tiles - 1) / w.px_tiles);
    w.ktg = (ncs + w.kgroups - 1) / w.kgroups;
    if (w.ktg > 16) w.ktg = 16;
    w.kgroups = (ncs + w.ktg - 1) / w.ktg;
    w.lds = sizeof(_Float16) * 2 * (size_t)kWidePixels * (32 * ncs + 8) + sizeof(uint32_t) * (size_t)kWidePixels * (w.ktg * 8 + 1);
    return w;
}

template <int LAYOUT>
__global__ __launch_bounds__(kWideThreads) void k_project_quantize_wide(WideParams p) {
    constexpr int PT = kWidePixels;
    extern __shared__ __align__(16) uint8_t dyn_lds[];
    __shared__ uint32_t lhist[256];
    __shared__ float s_n2[PT];  // |x - mu|^2 of every pixel of the tile
    zero_coder_scratch(p.ctrl, p.lookback, p.n_groups);

    const int C = p.C, ncs = p.ncs;
    const int Cpad = ncs * 32, NJ = ncs * 2;
    const int RSH = Cpad + 8;  // pixel row stride in halves
    const int kt0 = blockIdx.y * p.kt_per_group;
    const int ktg = (ncs - kt0 < p.kt_per_group) ? ncs - kt0 : p.kt_per_group;
    const int RSW = p.kt_per_group * 8 + 1;  // staging row stride in words
    _Float16* xh = reinterpret_cast<_Float16*>(dyn_lds);
    _Float16* xl = xh + (size_t)PT * RSH;
    uint32_t* st = reinterpret_cast<uint32_t*>(xl + (size_t)PT * RSH);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;

    if (tid < 256) lhist[tid] = 0u;
    const int zero_sym = 1 << (p.bits - 1);
    const float lo = (float)(-zero_sym), hi = (float)(zero_sym - 1);
    const float inv_delta = p.inv_delta, inv_delta_lo = p.inv_delta * (1.f / 2048.f);

    // the two f16 parts of one value (clamped to what f16 holds: a pixel with such a value is decided exactly)
    auto split = [](float v, _Float16& vh, _Float16& vl) {
        v = __builtin_amdgcn_fmed3f(v, -60000.f, 60000.f);
        vh = (_Float16)v;
        vl = (_Float16)((v - (float)vh) * 2048.f);
    };

    // the workgroup walks over pixel tiles; its histogram accumulates in LDS and leaves once at the end
    for (int64_t tile = blockIdx.x; tile < p.px_tiles; tile += gridDim.x) {
        const int64_t px0 = tile * PT;
        if (tid < PT) s_n2[tid] = 0.f;
        __syncthreads();  // also: the previous tile's staging rows have left

        // ---- the pixel tile, mean removed, split, as xh / xl [pixel][channel] ----
        if constexpr (LAYOUT == FMTC_NHWC) {
            const int n4 = PT * (C / 4);  // the tile is one contiguous run of PT*C floats
            const float* src = p.x + px0 * C;
            const int64_t lim = (p.P - px0) * C;  // floats of the tile that exist
            constexpr int B = 8;  // loads in flight per thread
            for (int idx0 = tid; idx0 < n4; idx0 += B * kWideThreads) {
                float4 v[B];
#pragma unroll
                for (int b = 0; b < B; b++) {
                    const int f = 4 * (idx0 + b * kWideThreads);
                    v[b] = (idx0 + b * kWideThreads < n4 && f < lim) ? *reinterpret_cast<const float4*>(src + f)
                                                                     : make_float4(0, 0, 0, 0);
                }
#pragma unroll
                for (int b = 0; b < B; b++) {
                    const int idx = idx0 + b * kWideThreads;
                    if (idx < n4) {
                        const int f = 4 * idx;
                        const int pxl = f / C, c = f - pxl * C;
                        const float4 m = *reinterpret_cast<const float4*>(p.mu + c);
                        const float d[4] = {v[b].x - m.x, v[b].y - m.y, v[b].z - m.z, v[b].w - m.w};
                        halfx4 vh, vl;
                        float n2 = 0.f;
#pragma unroll
                        for (int i = 0; i < 4; i++) {
                            _Float16 a, bb;
                            split(d[i], a, bb);
                            vh[i] = a;
                            vl[i] = bb;
                            n2 = __builtin_fmaf(d[i], d[i], n2);
                        }
                        *reinterpret_cast<halfx4*>(xh + pxl * RSH + c) = vh;
                        *reinterpret_cast<halfx4*>(xl + pxl * RSH + c) = vl;
                        atomicAdd(&s_n2[pxl], n2);
                    }
                }
            }
        } else {
            const int pxl = tid % PT;
            const int64_t px = px0 + pxl;
            const bool ok = px < p.P;
            int64_t base = 0;
            if (ok) {
                const int64_t n = px / p.HW;
                base = n * (int64_t)C * p.HW + (px - n * p.HW);
            }
            float n2 = 0.f;
            for (int c = tid / PT; c < C; c += kWideThreads / PT) {
                const float d = (ok ? p.x[base + (int64_t)c * p.HW] : 0.f) - p.mu[c];
                _Float16 a, b;
                split(d, a, b);
                xh[pxl * RSH + c] = a;
                xl[pxl * RSH + c] = b;
                n2 = __builtin_fmaf(d, d, n2);
            }
            atomicAdd(&s_n2[pxl], n2);
        }
        if (Cpad > C) {  // padding channels meet zero basis entries; they must still be finite
            const int padw = Cpad - C;
            for (int idx = tid; idx < PT * padw; idx += kWideThreads) {
                const int pxl = idx / padw, c = C + (idx - pxl * padw);
                xh[pxl * RSH + c] = (_Float16)0.f;
                xl[pxl * RSH + c] = (_Float16)0.f;
            }
        }
        __syncthreads();

        constexpr int PG = PT / 32;  // pixel groups per workgroup
        const int nunits = ktg * PG;
        for (int u = wave; u < nunits; u += kWideThreads / 64) {
            const int pg = u % PG, ktl = u / PG;
            const int kt = kt0 + ktl;
            const int pxl = pg * 32 + l32;
            const bool px_ok = px0 + pxl < p.P;
            floatx16 am, ac;
#pragma unroll
            for (int r = 0; r < 16; r++) { am[r] = 0.f; ac[r] = 0.f; }

            // (kt, j): the 64 lanes' hi parts, then their lo parts, 16 bytes per lane each; the basis comes from L2
            // (the wavefronts of a round read the same part of it), one step ahead of its use
            const uint4* asrc = reinterpret_cast<const uint4*>(p.basis16) + (size_t)kt * NJ * 2 * 64 + lane;
            uint4 th4 = asrc[0], tl4 = asrc[64];
            const _Float16* bh = xh + pxl * RSH + 8 * half;
            const _Float16* bl = xl + pxl * RSH + 8 * half;
            for (int jj = 0; jj < NJ; jj++) {
                uint4 nh4 = th4, nl4 = tl4;
                if (jj + 1 < NJ) {
                    nh4 = asrc[(size_t)(2 * jj + 2) * 64];
                    nl4 = asrc[(size_t)(2 * jj + 3) * 64];
                }
                const halfx8 th = __builtin_bit_cast(halfx8, th4), tl = __builtin_bit_cast(halfx8, tl4);
                const halfx8 xh8 = *reinterpret_cast<const halfx8*>(bh + 16 * jj);
                const halfx8 xl8 = *reinterpret_cast<const halfx8*>(bl + 16 * jj);
                am = __builtin_amdgcn_mfma_f32_32x32x16_f16(th, xh8, am, 0, 0, 0);
                ac = __builtin_amdgcn_mfma_f32_32x32x16_f16(th, xl8, ac, 0, 0, 0);
                ac = __builtin_amdgcn_mfma_f32_32x32x16_f16(tl, xh8, ac, 0, 0, 0);
                th4 = nh4;
                tl4 = nl4;
            }

            // ---- quantize ----
            // accumulator r = 4g + i of lane (pixel, h) is coefficient kt*32 + 16h + 4g + i of the pixel
            const float n2 = s_n2[pxl];
            const bool force = !(n2 < 1.0e9f);  // too large for f16, or not finite: every coefficient decided exactly
            const float tau = fminf(fmaxf(p.kappa * __builtin_sqrtf(n2), p.tau_min), 0.125f);
            const float near_limit = force ? -1.f : 0.5f - tau;
            const int k0 = kt * 32 + 16 * half;
            uint32_t words[4];
            uint32_t near_mask = 0;  // bit r: the fast value is too close to a rounding boundary to be trusted
#pragma unroll
            for (int g = 0; g < 4; g++) {
                uint32_t word = 0;
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    const float t = __builtin_fmaf(ac[4 * g + i], inv_delta_lo, am[4 * g + i] * inv_delta);
                    float q = __builtin_rintf(t);  // round half to even
                    const bool near = !(fabsf(t - q) <= near_limit);
                    q = __builtin_amdgcn_fmed3f(q, lo, hi);
                    word |= (uint32_t)((int)q + zero_sym) << (8 * i);
                    if (near && px_ok && (k0 + 4 * g + i) < C) near_mask |= 1u << (4 * g + i);
                }
                words[g] = word;
            }
            // ---- exact decision for the flagged values: fp64 recomputation, four values per round ----
            // (same arithmetic as the definition: sum of T[k][c] * (x[c] - mu[c]), divided by the step).
            // Each 16-lane group of the wavefront takes one flagged value, so the loads of four values overlap.
            unsigned long long pending = __ballot(near_mask != 0);
            while (pending) {
                int Ls[4];
                unsigned long long pm = pending;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    Ls[q] = pm ? (__ffsll((long long)pm) - 1) : -1;
                    pm &= pm - 1;
                }
                const int grp = lane >> 4;
                const int Lq = grp == 0 ? Ls[0] : (grp == 1 ? Ls[1] : (grp == 2 ? Ls[2] : Ls[3]));
                const bool active = Lq >= 0;
                const uint32_t fm = (uint32_t)__shfl((int)near_mask, active ? Lq : 0, 64);
                const int r = active ? (__ffs((int)fm) - 1) : 0;
                const int k = kt * 32 + 16 * (Lq >> 5) + r;
                const int64_t px = px0 + pg * 32 + (Lq & 31);
                double part = 0.0;
                if (active) {
                    int64_t xbase, xstride;
                    if constexpr (LAYOUT == FMTC_NHWC) {
                        xbase = px * C;
                        xstride = 1;
                    } else {
                        const int64_t n = px / p.HW;
                        xbase = n * (int64_t)C * p.HW + (px - n * p.HW);
                        xstride = p.HW;
                    }
#pragma unroll 8  // independent loads of eight terms in flight together: the loop is all latency
                    for (int c = lane & 15; c < C; c += 16)
                        part += (double)p.Trow[(size_t)k * C + c] * ((double)p.x[xbase + c * xstride] - (double)p.mu[c]);
                }
#pragma unroll
                for (int o = 8; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);  // stays inside the 16-lane group
                double qd = rint(part / (double)p.delta);
                qd = fmin(fmax(qd, (double)lo), (double)hi);
                const int sfix = (int)qd + zero_sym;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int rq = __shfl(r, 16 * q, 64);
                    const int sq = __shfl(sfix, 16 * q, 64);
                    if (lane == Ls[q]) {
#pragma unroll
                        for (int g = 0; g < 4; g++)
                            if (g == (rq >> 2))
                                words[g] = (words[g] & ~(0xffu << (8 * (rq & 3)))) | ((uint32_t)sq << (8 * (rq & 3)));
                        near_mask &= ~(1u << rq);
                    }
                }
                pending = __ballot(near_mask != 0);
            }
            // ---- count and stage ----
            // zero-level symbols (the bulk) are counted with byte arithmetic, the others with LDS atomics
            uint32_t zero_count = 0;
            const uint32_t zero4 = (uint32_t)zero_sym * 0x01010101u;
#pragma unroll
            for (int g = 0; g < 4; g++) {
                const int k = k0 + 4 * g;
                const uint32_t word = words[g];
                // 0x80 in every byte of the word that is a valid coefficient
                const int nvalid = !px_ok ? 0 : (C - k >= 4 ? 4 : (C - k > 0 ? C - k : 0));
                const uint32_t vmask = nvalid == 4 ? 0x80808080u : (0x80808080u >> (8 * (4 - nvalid))) * (nvalid != 0);
                const uint32_t xz = word ^ zero4;
                uint32_t t = (xz & 0x7f7f7f7fu) + 0x7f7f7f7fu;
                t = ~(t | xz | 0x7f7f7f7fu);  // 0x80 where the byte equals the zero level
                zero_count += (uint32_t)__popc(t & vmask);
                uint32_t nz = ~t & vmask;
                while (nz) {
                    const int bit = __ffs((int)nz) - 1;  // 8*i + 7
                    atomicAdd(&lhist[(word >> (bit - 7)) & 255u], 1u);
                    nz &= nz - 1;
                }
                st[pxl * RSW + ktl * 8 + 4 * half + g] = word;
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) zero_count += __shfl_xor(zero_count, o, 64);
            if (lane == 0 && zero_count) atomicAdd(&lhist[zero_sym], zero_count);
        }
        __syncthreads();

        // ---- symbols leave as rows of ktg*32 bytes per pixel ----
        const int kbase = kt0 * 32;
        const int row_words = ktg * 8;
        for (int idx = tid; idx < PT * row_words; idx += kWideThreads) {
            const int row = idx / row_words, col = idx - row * row_words;
            const int64_t px = px0 + row;
            const int k = kbase + 4 * col;
            if (px < p.P && k < C) {
                const uint32_t word = st[row * RSW + col];
                uint8_t* dst = p.syms + px * C + k;
                if constexpr (LAYOUT == FMTC_NHWC) {
                    *reinterpret_cast<uint32_t*>(dst) = word;
                } else {
                    for (int i = 0; i < 4 && k + i < C; i++) dst[i] = (uint8_t)(word >> (8 * i));
                }
            }
        }
    }
    __syncthreads();
    // one row of partial counts per workgroup: nothing to clear beforehand, no global atomics
    const int K = 1 << p.bits;
    if (tid < K) p.hist_parts[(size_t)(blockIdx.x + blockIdx.y * gridDim.x) * K + tid] = lhist[tid];
}

static hipError_t launch_wide(const BasisDevice& b, const float* d_x, int64_t P, int64_t HW, int layout, float delta,
                              int bits, uint8_t* d_syms, const CoderScratch& cs, int* n_parts, hipStream_t s) {
    WideParams p{};
    p.x = d_x;
    p.basis16 = b.fwd16;
    p.mu = b.mu;
    p.Trow = b.T;
    p.P = P;
    p.HW = HW;
    p.C = b.C;
    p.ncs = b.Cpad / 32;
    p.bits = bits;
    p.inv_delta = (float)(1.0 / (double)delta);
    p.delta = delta;
    // see launch_rows for the bound behind these two
    p.kappa = 1.9073486e-6f /* 2^-19 */ * b.row_norm * p.inv_delta;
    p.tau_min = 4.7683716e-7f /* 2^-21 */ * (float)(1 << (bits - 1));
    p.syms = d_syms;
    p.hist_parts = cs.hist_parts;
    p.ctrl = cs.ctrl;
    p.lookback = cs.lookback;
    p.n_groups = cs.n_groups;
    if (!p.x || !p.basis16 || !p.mu || !p.Trow || !p.syms || !p.hist_parts || !p.ctrl || !p.lookback ||
        (layout == FMTC_NHWC && b.C % 4 != 0))
        return hipErrorInvalidValue;  // (a field left out would be a wild pointer on the device)
    const WidePlan pl = plan_wide(b.C, P);
    p.kt_per_group = pl.ktg;
    p.px_tiles = pl.px_tiles;
    int64_t gx = p.px_tiles;
    if (gx * pl.kgroups > kMaxHistParts) gx = kMaxHistParts / pl.kgroups;
    const dim3 grid((unsigned)gx, (unsigned)pl.kgroups);
    *n_parts = (int)(gx * pl.kgroups);
    const void* fn = layout == FMTC_NHWC ? reinterpret_cast<const void*>(&k_project_quantize_wide<FMTC_NHWC>)
                                         : reinterpret_cast<const void*>(&k_project_quantize_wide<FMTC_NCHW>);
    hipError_t ea = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)pl.lds);
    if (ea != hipSuccess) return ea;
    return layout == FMTC_NHWC ? launch(K_PROJECT, k_project_quantize_wide<FMTC_NHWC>, grid, dim3(kWideThreads), pl.lds, s, p)
                               : launch(K_PROJECT, k_project_quantize_wide<FMTC_NCHW>, grid, dim3(kWideThreads), pl.lds, s, p);
}

// ---------------------------------------------------------------------------
// Few pixels, and channel counts that are no multiple of 16.  The kernels above walk all C / 16 dependent steps of a tile
// in one wavefront or behind barriers, and with few tiles most of the device idles meanwhile; here a tile is 32 PT pixels x 32 KT
// coefficients and its W wavefronts share out the contraction instead: each takes a run of the 16-channel steps, its
// operands straight from memory in registers one to four steps ahead (the basis in operand order, a lane's eight channels of
// its pixel as they lie), with no barrier in the loop.  The partial sums meet once in LDS, and every wavefront quantizes
// a part of the tile.  What bounds it: the latency of the loads (few tiles), then the caches' rate: a tile's operands are
// read by all tiles of its row and column.  Coefficient tiles are the fastest block index, padded to the eight dies, so
// that a die's L2 holds its share of the basis.  Measured, us (a pixel tile with all channels in LDS, the 128 x 128 tiles or the
// narrow kernel before): 314 channels, 20 x 20 25.6 -> 7.8; 768, N = 4, 7 x 6 32 -> 13.6; 1024, N = 8, 11 x 11 43 -> 29,
// planar 79 -> 31; 619, N = 20, 9 x 9 53 -> 23; 1001, N = 64, 7 x 7 186 -> 80; 169, N = 9, 80 x 80 122 -> 65; 124, N = 1,
// 20 x 20 12.9 -> 4.8; 64, 56 x 56 7.7 -> 5.3.
// ---------------------------------------------------------------------------
struct SplitParams {
    const float* x;
    const uint4* basis16;  // fwd16 packing: [ncs][NJ][2][64]
    const float* mu;       // [Cpad]
    const float* Trow;
    int64_t P, HW, n_pg;   // groups of 32 PT pixels
    int C, ncs, NJ, bits;
    int n_kg;              // groups of KT coefficient tiles
    int n_kc, n_kc_pad;    // those that are computed (the others' rows of the basis are all zero); as block indices
    uint32_t computed_blocks;  // the blocks of the others follow
    int hist_shift;
    float inv_delta, delta, kappa, tau_min;
    uint8_t* syms;
    uint32_t* hist_parts;
    CoderCtrl* ctrl;
    unsigned long long* lookback;
    uint32_t n_groups;
};

struct __attribute__((packed, aligned(4))) Float4u { float v[4]; };  // four floats at any float's address

constexpr int kSplitWaves = 4;

// PT x KT: pixel and coefficient tiles of a workgroup; D: steps that a wavefront's operands are requested ahead
template <int PT, int KT, int D, int LAYOUT>
__global__ __launch_bounds__(64 * kSplitWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_project_quantize_split(SplitParams p) {
    constexpr int W = kSplitWaves;
    constexpr int TILES = PT * KT;
    constexpr int QW = TILES * 4 / W;  // quads of accumulators that a wavefront quantizes
    static_assert(QW <= 4 && QW * W == TILES * 4, "quads of one tile per wavefront");
    extern __shared__ __align__(16) uint8_t dyn_lds[];
    // partial sums [W][TILES][4][64] (four per lane), mean [Cpad], histogram copies [K << hist_shift]
    float4* s_part = reinterpret_cast<float4*>(dyn_lds);
    float* s_mu = reinterpret_cast<float*>(s_part + W * TILES * 4 * 64);
    uint32_t* s_hist = reinterpret_cast<uint32_t*>(s_mu + 16 * p.NJ);
    __shared__ float s_n2[W][PT * 32];

    zero_coder_scratch(p.ctrl, p.lookback, p.n_groups);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int C = p.C, NJ = p.NJ, K = 1 << p.bits, HS = p.hist_shift, HC = 1 << HS;
    const bool computed = blockIdx.x < p.computed_blocks;
    const uint32_t block = computed ? blockIdx.x : blockIdx.x - p.computed_blocks;
    const uint32_t per_pg = (uint32_t)(computed ? p.n_kc_pad : p.n_kg - p.n_kc);
    const int kg = (int)(block % per_pg) + (computed ? 0 : p.n_kc);
    if (computed && kg >= p.n_kc) return;
    const int64_t pg0 = block / per_pg, pg_step = p.computed_blocks / (unsigned)p.n_kc_pad;
    const int kt0 = kg * KT;
    // this wavefront's steps (none where the basis' rows are all zero: every sum is then exactly zero)
    const int s_begin = computed ? wave * NJ / W : 0, s_end = computed ? (wave + 1) * NJ / W : 0;

    const uint4* a_src[KT];
#pragma unroll
    for (int a = 0; a < KT; a++) {
        int kt = kt0 + a;
        kt = kt < p.ncs ? kt : p.ncs - 1;  // a tile past the end repeats the last one; its results are dropped
        a_src[a] = p.basis16 + (size_t)kt * NJ * 128 + lane;
    }
    struct Step {
        uint4 th[KT], tl[KT];
        float v[PT][8];
    };
    Step buf[D];
    const float* xsrc[PT];
    auto locate = [&](int64_t pg) {  // past the end of the tensor the last pixel is loaded; its results are dropped
#pragma unroll
        for (int b = 0; b < PT; b++) {
            int64_t q = (pg * PT + b) * 32 + l32;
            q = q < p.P ? q : p.P - 1;
            if constexpr (LAYOUT == FMTC_NHWC) {
                xsrc[b] = p.x + q * C + 8 * half;
            } else {
                const int64_t n_img = q / p.HW;
                xsrc[b] = p.x + n_img * (int64_t)C * p.HW + (q - n_img * p.HW) + (int64_t)(8 * half) * p.HW;
            }
        }
    };
    auto load = [&](Step& t, int s) {
#pragma unroll
        for (int a = 0; a < KT; a++) {
            t.th[a] = a_src[a][(size_t)s * 128];
            t.tl[a] = a_src[a][(size_t)s * 128 + 64];
        }
        if (16 * s + 16 <= C) {
#pragma unroll
            for (int b = 0; b < PT; b++) {
                if constexpr (LAYOUT == FMTC_NHWC) {
                    const Float4u u0 = *reinterpret_cast<const Float4u*>(xsrc[b] + 16 * s);
                    const Float4u u1 = *reinterpret_cast<const Float4u*>(xsrc[b] + 16 * s + 4);
#pragma unroll
                    for (int e = 0; e < 4; e++) { t.v[b][e] = u0.v[e]; t.v[b][4 + e] = u1.v[e]; }
                } else {
#pragma unroll
                    for (int e = 0; e < 8; e++) t.v[b][e] = xsrc[b][(int64_t)(16 * s + e) * p.HW];
                }
            }
        } else {  // the channels that are missing from the last step meet a zero basis and a zero mean
            const int left = C - 16 * s - 8 * half;
#pragma unroll
            for (int b = 0; b < PT; b++)
#pragma unroll
                for (int e = 0; e < 8; e++)
                    t.v[b][e] = e < left ? xsrc[b][(int64_t)(16 * s + e) * (LAYOUT == FMTC_NHWC ? 1 : p.HW)] : 0.f;
        }
    };
    locate(pg0);
    if (pg0 < p.n_pg) {
#pragma unroll
        for (int d = 0; d < D; d++)
            if (s_begin + d < s_end) load(buf[d], s_begin + d);
    }
    for (int i = tid; i < 16 * NJ; i += 64 * W) s_mu[i] = p.mu[i];
    for (int i = tid; i < K << HS; i += 64 * W) s_hist[i] = 0u;
    __syncthreads();

    const int zero_sym = 1 << (p.bits - 1);
    const float lo = (float)(-zero_sym), hi = (float)(zero_sym - 1);
    const float magic = 12582912.f + (float)zero_sym;  // rounding, offset and conversion in one addition: see k_project_quantize_rows
    const float magic_lo = 12582912.f, magic_hi = 12582912.f + (float)(2 * zero_sym - 1);

    for (int64_t pg = pg0; pg < p.n_pg; pg += pg_step) {
        if (pg != pg0) {
            locate(pg);
#pragma unroll
            for (int d = 0; d < D; d++)
                if (s_begin + d < s_end) load(buf[d], s_begin + d);
        }
        floatx16 am[PT][KT], ac[PT][KT];
        float n2[PT];
#pragma unroll
        for (int b = 0; b < PT; b++) {
            n2[b] = 0.f;
#pragma unroll
            for (int a = 0; a < KT; a++)
#pragma unroll
                for (int r = 0; r < 16; r++) { am[b][a][r] = 0.f; ac[b][a][r] = 0.f; }
        }
        for (int s0 = s_begin; s0 < s_end; s0 += D) {
#pragma unroll
            for (int d = 0; d < D; d++) {
                const int s = s0 + d;
                if (s >= s_end) break;  // wavefront-uniform
                Step& t = buf[d];
                const float4 m0 = *reinterpret_cast<const float4*>(&s_mu[16 * s + 8 * half]);
                const float4 m1 = *reinterpret_cast<const float4*>(&s_mu[16 * s + 8 * half + 4]);
                const float m[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
                halfx8 xh[PT], xl[PT];
#pragma unroll
                for (int b = 0; b < PT; b++)
#pragma unroll
                    for (int e = 0; e < 8; e++) {
                        // (no clamp of values beyond f16: what their infinities make of the products stays in the pixel's own
                        // column of outputs, and such a pixel is decided exactly in all coefficients, see n2)
                        const float dv = t.v[b][e] - m[e];
                        n2[b] = __builtin_fmaf(dv, dv, n2[b]);
                        const _Float16 h = (_Float16)dv;
                        xh[b][e] = h;
                        xl[b][e] = (_Float16)__builtin_fmaf((float)h, -2048.f, dv * 2048.f);  // 2^11 (d - h), exact, one mixed multiply-add
                    }
                halfx8 th[KT], tl[KT];
#pragma unroll
                for (int a = 0; a < KT; a++) {
                    th[a] = __builtin_bit_cast(halfx8, t.th[a]);
                    tl[a] = __builtin_bit_cast(halfx8, t.tl[a]);
                }
#pragma unroll
                for (int b = 0; b < PT; b++)
#pragma unroll
                    for (int a = 0; a < KT; a++) {
                        am[b][a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(th[a], xh[b], am[b][a], 0, 0, 0);
                        ac[b][a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(th[a], xl[b], ac[b][a], 0, 0, 0);
                    }
#pragma unroll
                for (int b = 0; b < PT; b++)
#pragma unroll
                    for (int a = 0; a < KT; a++)
                        ac[b][a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(tl[a], xh[b], ac[b][a], 0, 0, 0);
                if (s + D < s_end) load(t, s + D);
            }
        }
        // ---- the partial sums meet ----
#pragma unroll
        for (int b = 0; b < PT; b++) {
            n2[b] += __shfl_xor(n2[b], 32, 64);  // the other half of the pixel
            if (half == 0) s_n2[wave][b * 32 + l32] = n2[b];
#pragma unroll
            for (int a = 0; a < KT; a++)
#pragma unroll
                for (int g = 0; g < 4; g++) {
                    float y[4];
#pragma unroll
                    for (int i = 0; i < 4; i++) y[i] = __builtin_fmaf(ac[b][a][4 * g + i], 1.f / 2048.f, am[b][a][4 * g + i]);
                    s_part[((wave * TILES + b * KT + a) * 4 + g) * 64 + lane] = make_float4(y[0], y[1], y[2], y[3]);
                }
        }
        __syncthreads();
        const int unit = wave * QW, tile = unit >> 2, q0 = unit & 3;
        const int pt = tile / KT, kt = kt0 + tile % KT;
        const int64_t px = (pg * PT + pt) * 32 + l32;
        const int k0 = kt * 32 + 16 * half + 4 * q0;
        int valid = px < p.P ? C - k0 : 0;  // coefficients of this lane that exist
        valid = valid < 0 ? 0 : (valid > 4 * QW ? 4 * QW : valid);
        float pn2 = 0.f;
#pragma unroll
        for (int w = 0; w < W; w++) pn2 += s_n2[w][pt * 32 + l32];
        const bool force = !(pn2 < 1.0e9f);  // too large for f16, or not finite: every coefficient decided exactly
        const float tau = fminf(fmaxf(p.kappa * __builtin_sqrtf(pn2), p.tau_min), 0.125f);
        const float near_limit = force ? -1.f : 0.5f - tau;
        uint32_t word[QW], near_mask = 0;
#pragma unroll
        for (int g = 0; g < QW; g++) {
            float4 y = s_part[unit * 64 + g * 64 + lane];
#pragma unroll
            for (int w = 1; w < W; w++) {
                const float4 o = s_part[(w * TILES * 4 + unit + g) * 64 + lane];
                y.x += o.x; y.y += o.y; y.z += o.z; y.w += o.w;
            }
            const float ys[4] = {y.x, y.y, y.z, y.w};
            uint32_t ub[4];
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const float t = ys[i] * p.inv_delta;
                const float u = t + magic;  // round half to even
                if (!(fabsf(t - (u - magic)) <= near_limit) && 4 * g + i < valid) near_mask |= 1u << (4 * g + i);
                ub[i] = clamp_pattern(u, magic_lo, magic_hi);  // (its lowest byte is the symbol: in range whatever u is)
            }
            word[g] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(ub[3], ub[2], 0x0c0c0400u),
                                            __builtin_amdgcn_perm(ub[1], ub[0], 0x0c0c0400u), 0x05040100u);
        }
        // ---- exact fp64 decision of the flagged values, two per round (one per half of the wavefront) ----
        unsigned long long pending = __ballot(near_mask != 0);
        while (__builtin_expect(pending != 0, 0)) {
            const int L0 = __ffsll((long long)pending) - 1;
            const unsigned long long rest = pending & (pending - 1);
            const int L1 = rest ? __ffsll((long long)rest) - 1 : -1;
            const int Lq = half ? L1 : L0;
            const bool active = Lq >= 0;
            const uint32_t fm = (uint32_t)__shfl((int)near_mask, active ? Lq : 0, 64);
            const int r = active ? __ffs((int)fm) - 1 : 0;
            double part = 0.0;
            if (active) {
                const int k = kt * 32 + 16 * (Lq >> 5) + 4 * q0 + r;
                const int64_t qpx = (pg * PT + pt) * 32 + (Lq & 31);
                int64_t xbase = qpx * C, xstride = 1;
                if constexpr (LAYOUT != FMTC_NHWC) {
                    const int64_t n_img = qpx / p.HW;
                    xbase = n_img * (int64_t)C * p.HW + (qpx - n_img * p.HW);
                    xstride = p.HW;
                }
#pragma unroll 16  // independent loads in flight together: the loop is all latency
                for (int c = l32; c < C; c += 32)
                    part += (double)p.Trow[(size_t)k * C + c] * ((double)p.x[xbase + c * xstride] - (double)s_mu[c]);
            }
#pragma unroll
            for (int o = 16; o > 0; o >>= 1) part += __shfl_xor(part, o, 64);  // stays inside the half
            double qd = rint(part / (double)p.delta);
            qd = fmin(fmax(qd, (double)lo), (double)hi);
            const int sfix = (int)qd + zero_sym;
            const int r0 = __shfl(r, 0, 64), r1 = __shfl(r, 32, 64), f0 = __shfl(sfix, 0, 64), f1 = __shfl(sfix, 32, 64);
            if (lane == L0 || lane == L1) {
                const int rq = lane == L0 ? r0 : r1;
                const uint32_t sq = (uint32_t)(lane == L0 ? f0 : f1);
#pragma unroll
                for (int g = 0; g < QW; g++)
                    if (g == (rq >> 2)) word[g] = (word[g] & ~(0xffu << (8 * (rq & 3)))) | (sq << (8 * (rq & 3)));
                near_mask &= ~(1u << rq);
            }
            pending = __ballot(near_mask != 0);
        }
        // ---- count and store ----
#pragma unroll
        for (int g = 0; g < QW; g++)
#pragma unroll
            for (int i = 0; i < 4; i++)
                if (4 * g + i < valid) atomicAdd(&s_hist[(((word[g] >> (8 * i)) & 255u) << HS) + (lane & (HC - 1))], 1u);
        uint8_t* dst = p.syms + px * C + k0;
        if ((C & 15) == 0) {  // all of a lane's coefficients or none, aligned
            if (valid) {
                if constexpr (QW == 4) *reinterpret_cast<uint4*>(dst) = make_uint4(word[0], word[1], word[2], word[3]);
                else if constexpr (QW == 2) *reinterpret_cast<uint2*>(dst) = make_uint2(word[0], word[1]);
                else *reinterpret_cast<uint32_t*>(dst) = word[0];
            }
        } else {
#pragma unroll
            for (int g = 0; g < QW; g++) {
                if ((C & 3) == 0) {
                    if (4 * g < valid) *reinterpret_cast<uint32_t*>(dst + 4 * g) = word[g];
                } else {
#pragma unroll
                    for (int i = 0; i < 4; i++)
                        if (4 * g + i < valid) dst[4 * g + i] = (uint8_t)(word[g] >> (8 * i));
                }
            }
        }
        __syncthreads();  // the partial sums have been read
    }
    // one row of partial counts per workgroup (see the narrow-tensor kernel)
    for (int row = tid; row < K; row += 64 * W) {
        uint32_t total = 0;
        for (int q = 0; q < HC; q++) total += s_hist[(row << HS) + ((q + row) & (HC - 1))];
        p.hist_parts[(size_t)(pg0 * p.n_kg + kg) * K + row] = total;
    }
}

// Workgroups per coefficient group: one row of counts each.  Up to 256 channels no more workgroups than run at once (two per
// compute unit): what adds up their rows is one workgroup (97 channels, 20800 pixels, 8 bits 20.6 us and 42.2 after it with 1024
// rows, 18.6 and 40.5 with 512).  The longer contraction of wider tensors leaves too much of a second round idle (1001
// channels, planar, 6496 pixels, 8 bits 200 us with 1024, 227 with 512).
static int64_t split_px_workgroups(int ncs, int n_kg, int64_t n_pg) {
    const int most = ncs <= 8 ? 512 : kMaxHistParts;
    return n_pg * n_kg > most ? most / n_kg : n_pg;
}

template <int PT, int KT, int D>
static hipError_t launch_split(const BasisDevice& b, const float* d_x, int64_t P, int64_t HW, int layout, float delta,
                               int bits, uint8_t* d_syms, const CoderScratch& cs, int* n_parts, hipStream_t s,
                               bool skip_zero_rows) {
    SplitParams p{};
    p.x = d_x;
    p.basis16 = reinterpret_cast<const uint4*>(b.fwd16);
    p.mu = b.mu;
    p.Trow = b.T;
    p.P = P;
    p.HW = HW;
    p.C = b.C;
    p.ncs = b.Cpad / 32;
    p.NJ = b.Cpad / 16;
    p.bits = bits;
    p.n_pg = (P + 32 * PT - 1) / (32 * PT);
    p.n_kg = (p.ncs + KT - 1) / KT;
    // Groups of four coefficient tiles whose rows of the basis are all zero (truncation) are not computed where the tiled
    // product leaves them out too.  The narrow kernels decide every coefficient of a pixel beyond f16 exactly, those of
    // zero rows too, and what a pixel that is not finite gives there must not depend on the tensor's size.
    static_assert(4 % KT == 0, "whole groups are left out");
    p.n_kc = skip_zero_rows ? (b.active_rows + 127) / 128 * (4 / KT) : p.n_kg;
    p.n_kc = p.n_kc < 4 / KT ? 4 / KT : p.n_kc;
    p.n_kc = p.n_kc > p.n_kg ? p.n_kg : p.n_kc;
    // (a block beyond the last group ends at once.  The groups that are not computed have blocks of their own behind the
    // others: in one order with them they would be whole dies' share.)
    const int padded = (p.n_kc + 7) / 8 * 8;
    p.n_kc_pad = 4 * (padded - p.n_kc) <= p.n_kc ? padded : p.n_kc;
    p.inv_delta = (float)(1.0 / (double)delta);
    p.delta = delta;
    // see launch_rows for the bound behind these two (the four partial sums and the two roundings after them add at most
    // 6 * 2^-24 |T_k|_2 |x - mu|_2 to the 2^-22 there: 2^-20.7 in all)
    p.kappa = 1.9073486e-6f /* 2^-19 */ * b.row_norm * p.inv_delta;
    p.tau_min = 4.7683716e-7f /* 2^-21 */ * (float)(1 << (bits - 1));
    p.syms = d_syms;
    p.hist_parts = cs.hist_parts;
    p.ctrl = cs.ctrl;
    p.lookback = cs.lookback;
    p.n_groups = cs.n_groups;
    // every pointer the kernel follows is set (a field left out here would be a wild pointer on the device)
    if (!p.x || !p.basis16 || !p.mu || !p.Trow || !p.syms || !p.hist_parts || !p.ctrl || !p.lookback)
        return hipErrorInvalidValue;
    const int64_t gx = split_px_workgroups(p.ncs, p.n_kg, p.n_pg);
    *n_parts = (int)(gx * p.n_kg);
    // histogram copies: 8 KB at most, so that two workgroups with 64 KB of partial sums share a compute unit
    p.hist_shift = bits <= 7 ? 4 : 3;
    const size_t lds = sizeof(float4) * kSplitWaves * PT * KT * 4 * 64 + sizeof(float) * b.Cpad + (sizeof(uint32_t) << (bits + p.hist_shift));
    const void* fn = layout == FMTC_NHWC ? reinterpret_cast<const void*>(&k_project_quantize_split<PT, KT, D, FMTC_NHWC>)
                                         : reinterpret_cast<const void*>(&k_project_quantize_split<PT, KT, D, FMTC_NCHW>);
    hipError_t ea = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (ea != hipSuccess) return ea;
    p.computed_blocks = (uint32_t)(gx * p.n_kc_pad);
    const dim3 grid(p.computed_blocks + (uint32_t)(gx * (p.n_kg - p.n_kc)));
    return layout == FMTC_NHWC ? launch(K_PROJECT, k_project_quantize_split<PT, KT, D, FMTC_NHWC>, grid, dim3(64 * kSplitWaves), lds, s, p)
                               : launch(K_PROJECT, k_project_quantize_split<PT, KT, D, FMTC_NCHW>, grid, dim3(64 * kSplitWaves), lds, s, p);
}

// Which of the forms above projects a tensor.
struct ProjectionForm {
    enum Kernel { kRows, kGemm, kWide, kSplit } kernel;
    int px_tiles, coef_tiles;  // kSplit: of a workgroup
    bool skip_zero_rows;       // kSplit
};

// Channel counts that are no multiple of 16, more than 128 channels: whether the workgroups with all channels in LDS
// (k_project_quantize_wide) are ahead of the split form.  us, theirs : split, at 4 / 6 / 8 bits:
//   - Two of them share a compute unit up to 448 channels, and 12000 to 16320 pixels are one round of 376 to 510: planar
//     185 channels, 16000 pixels 21.3 : 27.4 / 22.7 : 28.9 / 24.3 : 30.8; 265, 12800 31 : 39 / 33 : 41 / 36 : 45; channels last,
//     404, 16000 46 : 54 / 55 : 66 / 59 : 73.
//   - Beyond that one per compute unit, and a round costs the same however many are in it.  One full round: 1000 channels,
//     channels last, 4096 pixels 59 : 78 (3 bits) / 70 : 96 / 72 : 145; planar 510, 8192 31 : 53 / 38 : 60 / 44 : 76.
//   - With the bits more values are close to a rounding boundary, and in the split form three wavefronts wait while one
//     decides its own exactly, so rounds less full are worth it: channels last, 1000, 20000 (1250 workgroups in five rounds)
//     305 : 369 at 6 bits, 6496 (406 in two) 132 : 161 at 7, 14000 260 : 369 and 1024 48 : 67 at 8; but 5184 (324 in two) 125 : 115
//     at 6; 900, 5728 (358 in two) 112 : 104 at 6, 121 : 130 at 8.
//   - From 17 to 22 coefficient tiles the second workgroup of a pixel tile is given one to six of them: 580, 18496 147 : 115
//     at 6 bits, 644, 13696 132 : 151 at 7; planar, where the pixels' loads take longer, 570, 11552 113 : 94 at 6, 153 : 133 at 8.
// (Planar channel counts that are a multiple of 4 are slower there in every case: 500, 17984 150 : 115, 1000, 8992 316 : 198;
// channels last, others are: 333, 26176 145 : 78, 1001, 8992 303 : 195; 300, 28800, of a shorter contraction, 106 : 77.)
static bool wide_form_is_ahead(int C, int64_t P, int layout, int bits) {
    if ((layout == FMTC_NHWC) != (C % 4 == 0)) return false;
    const int ncs = (C + 31) / 32;
    const bool nhwc = layout == FMTC_NHWC;
    if (P > 12000 && P <= 16320 && ncs <= 16 && (ncs >= 13 || !nhwc)) return true;
    const WidePlan w = plan_wide(C, P);
    if (ncs < 15 || w.px_tiles * ncs <= (bits <= 7 ? 3500 : 640)) return false;
    if (nhwc && bits <= 6 && ncs > 16 && ncs < 23) return false;
    // percent of the rounds' workgroups (planar: of their coefficient tiles) that there are
    const int64_t slots = (w.px_tiles * w.kgroups + 255) / 256 * 256;
    const int64_t share = nhwc ? 100 * w.px_tiles * w.kgroups / slots : 100 * w.px_tiles * ncs / (slots * w.ktg);
    if (bits <= 5) return slots == 256 && share >= 97;
    return share >= (bits == 6 ? (nhwc ? 80 : 95) : bits == 7 ? (nhwc ? 75 : 85) : (nhwc ? 70 : 75));
}

static ProjectionForm choose_projection(int C, int64_t P, int64_t HW, int layout, int bits, int active_rows) {
    const int ncs = (C + 31) / 32;
    // 160 padded channels still fit the one-wavefront-per-32-pixels kernels (not at 8 bits, where the histograms find no room
    // in LDS beside the basis: 100 + 64 KB); for planar tensors only the streaming form, with 32-bit offsets and whole groups
    // of 16 channels
    const bool fits160 = ncs == 5 && bits < 8 && (layout == FMTC_NHWC || (C % 16 == 0 && planar_offsets_fit(C, P, HW)));
    const bool narrow = ncs <= 4 || fits160, whole16 = C % 16 == 0;
    const int64_t tiles = (P + 31) / 32 * ncs;  // of 32 pixels x 32 coefficients
    auto split = [&](int pt, int kt) { return ProjectionForm{ProjectionForm::kSplit, pt, kt, !narrow && whole16}; };
    const ProjectionForm rows{ProjectionForm::kRows, 0, 0, false}, gemm{ProjectionForm::kGemm, 0, 0, false};
    // Up to 32 channels the narrow kernel has no contraction to split (5.4 to 6.4 us against 6.0 at 16 and 32 channels).
    if (ncs == 1) return rows;
    // The split contraction's tile grows with their number.  One or two coefficient tiles per workgroup while that leaves
    // compute units idle otherwise (us, 1 : 2 : 4 of them: 512 channels, 64 tiles 10.5 : 11.2 : 12.8; 768 channels, 312 tiles
    // 17.3 : 14.6 : 17.2; 512 channels, 720 tiles 21.5 : 16.9 : 15.0).
    if (tiles <= 256) return split(1, 1);
    if (tiles <= 640 || (tiles <= 1024 && ncs == 2)) return split(1, 2);
    // Four of them, or two by two where the last four would be half empty (five and six coefficient tiles; us, 1 x 4 : 2 x 2:
    // 144 channels, 1300 tiles 15.5 : 11, 129, 6500 57 : 45, 161, 9000 67 : 59, 20000 133 : 109; but 200 channels, 9000 tiles
    // 54 : 60, 300 66 : 74, 500 100 : 117, 1000 182 : 198):
    const ProjectionForm large = tiles > 1200 && (ncs == 5 || ncs == 6) ? split(2, 2) : split(1, 4);
    // up to 1024 tiles instead of the narrow kernels (us, theirs first: 96 channels, 999 tiles 11.9 : 8.4; 128 10.9 : 8.5; 160
    // 13.8 : 10.4; at 144 channels and 2330 tiles 13.9 : 17.8), and of 97 to 127 channels that are no multiple of 16, which
    // those load with masks (100, 3456 tiles 19.4 : 15.9; 124, 4680 27.9 : 23.2; 97, 14000 62 : 58; of 65 to 95, channels last, 75,
    // 1998 15.7 : 17.3, 95, 9999 53 : 55, planar 19.6 : 18.0 and 60.7 : 59.4);
    if (narrow) return tiles <= (ncs == 4 && !whole16 ? 16384 : 1024) ? large : rows;
    // instead of the tiled product, whose steps are a chain of barriers: channels last up to 1536 tiles (us, theirs first: 512
    // channels, 1456 25.6 : 23.1; 256, 1600 16.9 : 12.6; 512, 2304 26.8 : 33.4), but from 544 channels on, whose exact decisions are
    // what a workgroup of the split form ends with, up to 1024 at 6 and 7 bits (1024 channels, 1024 tiles 42 : 40, 1184 42 : 50; 768,
    // 1200 33 : 35; 640, 1200 28 : 32) and up to 800 at 8 (640, 900 32 : 37; 960, 1024 46 : 51; 896, 784 42 : 38).  Planar pixels are
    // fetched four bytes at a time there: up to 4096 tiles from 512 channels on (512, 3888 64 : 50; 768, 3888 96 : 73; 1024,
    // 4096 109 : 83), up to 3840 at 256, 384 and from 448 on (256, 3800 25 : 23, 4096 24 : 27; 448, 3290 40 : 33), up to 2800
    // otherwise (192, 2598 22 : 21, 4092 25 : 29; 288, 2898 31 : 29, 3798 34 : 37; 400, 3497 35 : 37).  Both forms leave groups of
    // zero rows out, and the closer lines count the other tiles only (768 channels of which 307 are kept, channels last, 1008
    // tiles, 504 of them computed, 8 bits 37 : 25).
    const int64_t computed = tiles / ncs * (active_rows >= C ? ncs : (active_rows + 127) / 128 * 4);
    const int64_t nhwc_most = ncs <= 16 || bits <= 5 ? 1536 : (bits <= 7 ? 1024 : 800);
    const int64_t nchw_most = ncs >= 16 ? 4096 : (ncs % 4 == 0 || ncs > 13 ? 3840 : 2800);
    if (whole16)
        return (layout == FMTC_NHWC ? tiles <= 1536 && computed <= nhwc_most : tiles <= 4096 && computed <= nchw_most) ? large : gemm;
    // the tiled product needs whole groups of 16 channels.
    return tiles > 640 && wide_form_is_ahead(C, P, layout, bits) ? ProjectionForm{ProjectionForm::kWide, 0, 0, false} : large;
}

// The same in words, for tests: "rows 2 vec", "stream 5x8 half", "gemm8 fill", "split 1x4", ..., the layout, and of the split
// form the rows of counts.
int describe_projection(int C, int64_t P, int64_t HW, int layout, int bits, int active_rows, char* text, size_t size) {
    const ProjectionForm f = choose_projection(C, P, HW, layout, bits, active_rows);
    const char* lay = layout == FMTC_NHWC ? "nhwc" : "nchw";
    if (f.kernel == ProjectionForm::kRows) {
        const RowsPlan r = plan_rows(C, P, HW, layout, bits);
        if (r.stream) return snprintf(text, size, "stream %d%s%s %s", r.nct, r.waves == 8 ? "x8" : "", C == 32 * r.nct ? "" : " half", lay);
        return snprintf(text, size, "rows %d%s%s %s", r.nct, r.waves == 8 ? "x8" : "", r.vec ? " vec" : "", lay);
    }
    if (f.kernel == ProjectionForm::kGemm) {
        const GemmPlan g = plan_gemm(C, P, active_rows);
        return snprintf(text, size, "gemm%d%s %s", g.eight ? 8 : 4, g.gy < g.gy_all ? " fill" : "", lay);
    }
    if (f.kernel == ProjectionForm::kWide) return snprintf(text, size, "wide %s", lay);
    const int ncs = (C + 31) / 32, n_kg = (ncs + f.coef_tiles - 1) / f.coef_tiles;
    const int64_t px = 32 * f.px_tiles;
    return snprintf(text, size, "split %dx%d %s %d", f.px_tiles, f.coef_tiles, lay,
                    (int)(split_px_workgroups(ncs, n_kg, (P + px - 1) / px) * n_kg));
}

hipError_t launch_project_quantize(const BasisDevice& b, const float* d_x, int64_t N, int64_t HW, int layout,
                                   float delta, int bits, uint8_t* d_syms, const CoderScratch& cs, int* n_parts,
                                   hipStream_t s) {
    const int64_t P = N * HW;
    const ProjectionForm f = choose_projection(b.C, P, HW, layout, bits, b.active_rows);
    if (f.kernel == ProjectionForm::kRows) return launch_rows(b, d_x, P, HW, layout, delta, bits, d_syms, cs, n_parts, s);
    if (f.kernel == ProjectionForm::kGemm) return launch_gemm(b, d_x, P, HW, layout, delta, bits, d_syms, cs, n_parts, s);
    if (f.kernel == ProjectionForm::kWide) return launch_wide(b, d_x, P, HW, layout, delta, bits, d_syms, cs, n_parts, s);
    if (f.px_tiles == 2) return launch_split<2, 2, 1>(b, d_x, P, HW, layout, delta, bits, d_syms, cs, n_parts, s, f.skip_zero_rows);
    if (f.coef_tiles == 4) return launch_split<1, 4, 1>(b, d_x, P, HW, layout, delta, bits, d_syms, cs, n_parts, s, f.skip_zero_rows);
    if (f.coef_tiles == 2) return launch_split<1, 2, 2>(b, d_x, P, HW, layout, delta, bits, d_syms, cs, n_parts, s, f.skip_zero_rows);
    return launch_split<1, 1, 4>(b, d_x, P, HW, layout, delta, bits, d_syms, cs, n_parts, s, f.skip_zero_rows);
}

// Histogram of given symbols (staged coder entry point): one row of partial counts per workgroup.
// Values outside the alphabet are not counted.
__global__ __launch_bounds__(256) void k_histogram(const uint8_t* __restrict__ syms, uint64_t V, int bits,
                                                   uint32_t* __restrict__ hist_parts, CoderCtrl* ctrl,
                                                   unsigned long long* lookback, uint32_t n_groups) {
    __shared__ uint32_t lhist[256];
    zero_coder_scratch(ctrl, lookback, n_groups);
    lhist[threadIdx.x] = 0u;
    __syncthreads();
    const unsigned K = 1u << bits;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < V; i += (uint64_t)gridDim.x * 256) {
        unsigned sy = syms[i];
        if (sy < K) atomicAdd(&lhist[sy], 1u);
    }
    __syncthreads();
    if (threadIdx.x < K) hist_parts[(size_t)blockIdx.x * K + threadIdx.x] = lhist[threadIdx.x];
}

hipError_t launch_histogram(const uint8_t* d_syms, uint64_t V, int bits, const CoderScratch& cs, int* n_parts,
                            hipStream_t s) {
    uint64_t want = (V + 256 * 16 - 1) / (256 * 16);
    unsigned blocks = (unsigned)(want < 1 ? 1 : (want > (uint64_t)kMaxHistParts ? (uint64_t)kMaxHistParts : want));
    *n_parts = (int)blocks;
    return launch(K_HISTOGRAM, k_histogram, dim3(blocks), dim3(256), 0, s, d_syms, V, bits, cs.hist_parts, cs.ctrl,
                  cs.lookback, cs.n_groups);
}

}  // namespace fmtc
