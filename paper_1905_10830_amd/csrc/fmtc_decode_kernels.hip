// Decoder (paper section 3: variable length decoder, inverse quantizer, inverse
// transform; section 3.1 "Implementation": levels scaled back to the transform
// domain, then the inverse PCA).  One kernel per call:
//   1. every workgroup checks the header and the code length table and builds the
//      canonical decode tables and a 2^11-entry three-symbol lookup table in LDS;
//   2. one wavefront per unit (a chunk, or as many small ones as it has lanes for),
//      one lane per run of 64 symbols (bit offset = prefix sum of the stored run
//      sizes) decodes into an LDS symbol tile;
//   3. x_hat = T^T (Delta q) + mu on the f16 matrix cores
//      (v_mfma_f32_32x32x16_f16; the levels are exact in f16, the basis entries are
//      split in two f16 parts).  Narrow tensors (up to 160 channels): the wavefront
//      that decoded a unit also transforms it, the basis sits in LDS in operand
//      order and no workgroup barrier is needed after the tables.  Wide tensors: a
//      tile of several chunks per workgroup, the basis streamed from L2.
// Nothing outside [stream, stream + bytes) is read whatever the stream holds.
#include "fmtc_device.h"
#include "fmtc_internal.h"

namespace fmtc {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));

// byte address of symbol n of the tile: every run of 64 symbols is followed by 4
// pad bytes so that the 64 lanes of a decoding wavefront hit different banks
__device__ __forceinline__ uint32_t sym_addr(uint32_t n) { return n + 4u * (n >> 6); }

// Symbols n .. n + 7 of a tile (which starts on a word), four to a word.  ALIGNED4: n is a multiple of 4.  Otherwise the
// three words around them (eight byte reads instead, and their joining, took two thirds of the wide decoder's time at 293
// channels).
template <bool ALIGNED4>
__device__ __forceinline__ void read_octet(const uint8_t* tile, uint32_t n, uint32_t& w0, uint32_t& w1) {
    auto word = [&](uint32_t m) { return *reinterpret_cast<const uint32_t*>(tile + sym_addr(m)); };
    if constexpr (ALIGNED4) {
        w0 = word(n);
        w1 = word(n + 4u);
    } else {
        const uint32_t n0 = n & ~3u;
        const uint32_t a = word(n0), b = word(n0 + 4u), c = word(n0 + 8u);
        w0 = __builtin_amdgcn_alignbyte(b, a, n & 3u);
        w1 = __builtin_amdgcn_alignbyte(c, b, n & 3u);
    }
}

constexpr int kLut2Bits = 10;  // second table: codes longer than kLutBits bits

// Where the lookup table keeps the entry of the stream bits `v` (kLutBits of them, first bit lowest).  The LDS bank of
// a word is its index modulo 64; short codes are frequent, so many lanes of a wavefront look at bit patterns that
// agree in their first bits and differ in the later ones -- with the plain index these would be different words of
// one bank, read one after the other.  Folding the upper bits into the lower six spreads them over the banks
// (patterns that agree in all bits are one word, which the LDS reads once for all lanes).
__device__ __forceinline__ uint32_t lut_slot(uint32_t v) { return v ^ (v >> 6); }
// The same for the 16-bit scratch table of the construction (two entries per word: bits 1..6 choose the bank), which
// is read at values shifted left by a code length: their lower bits are zero, and the upper ones must choose the bank.
__device__ __forceinline__ uint32_t first_slot(uint32_t v) { return v ^ (v >> 5); }

// Decode tables, in LDS, built by every workgroup from the code length table of the stream.
struct DecTables {
    uint32_t cnt_len[64];     // number of codes of each length
    uint32_t rank_of_code[64];  // plus a code of the length: its rank (in (length, symbol) order), modulo 2^32
    uint64_t first_code[64];  // first canonical code of each length
    uint64_t limit[64];       // (first_code + count) << (32 - length) for length <= 32: first left-aligned 32-bit
                              // value that is NOT a code of this length or shorter
    uint32_t limit32[64];     // the same, saturated to 32 bits (exact for every length below the longest)
    uint16_t sorted_sym[256]; // symbols in (length, symbol) order
    // next kLutBits stream bits -> up to three symbols: sym0 | sym1 << 8 | sym2 << 16 | bits << 24 | n << 29,
    // n = number of whole codes found in those bits (0: the first code is longer than kLutBits), bits = their
    // total length
    uint32_t lut[1 << kLutBits];
    // Codes longer than kLutBits bits.  Canonical codes grow with their length, so left-aligned in 32 bits all of
    // them lie at or above long_base (the first value the short codes do not cover), in a range whose size is about
    // their share of the probability mass.  lut2 is indexed by (value - long_base) >> long_shift: sym | len << 8
    // where those bits decide the code (its length is at most 32 - long_shift and at most 31), 0 where they do not
    // (the decoders then search the per-length limits).  It shares its place with scratch of the construction:
    // `first` = first code in a kLutBits-bit value (first stream bit on top), sym | len << 8.
    union {
        uint16_t lut2[1 << kLut2Bits];
        uint16_t first[1 << kLutBits];
    };
    uint32_t wave_len_count[4][64];
    uint32_t lut_limit[kLutBits + 1];  // limit[] in a kLutBits-bit frame
    uint32_t n_used, ok, max_len, pad;
    uint32_t long_base, long_shift, pad0, pad1;
};

// A cold run of dependent LDS round trips and of instructions that are fetched for the first time: what counts is the number
// of barriers, of LDS operations in a row and the size of the code.  Counts by ballot instead of LDS additions, 64-bit sums
// without shuffles, the second table's limits out of one register: 6.3 -> 4.1 us at four wavefronts.
// All THREADS threads of the workgroup call this (THREADS a multiple of 256); my_len is the code length of symbol
// threadIdx.x from the stream (threads past 255: anything).  Returns false (for every thread)
// unless the lengths form a complete prefix code (Kraft sum exactly 1), or the single one-bit code of a
// one-symbol tensor.
template <int THREADS>
__device__ __forceinline__ bool build_decode_tables(DecTables& T, int my_len, int bits) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int K = 1 << bits;
    uint32_t before = 0;  // symbols of this one's length before it
    if (tid < 256) {
        const bool bad = my_len > kMaxLen || (tid >= K && my_len != 0);
        if (bad) my_len = 0;
        // the lanes of this wavefront with the same length as this one: six ballots, one per bit of the length
        unsigned long long same = ~0ull;
#pragma unroll
        for (int bit = 0; bit < 6; bit++) {
            const unsigned long long m = __ballot((my_len >> bit) & 1);
            same &= ((my_len >> bit) & 1) ? m : ~m;
        }
        before = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
        // (the wavefront's own row: cleared, then the first lane of every length leaves the length's count)
        const uint32_t n_bad = (uint32_t)__popcll(__ballot(bad)), n_used = (uint32_t)__popcll(__ballot(my_len != 0));
        T.wave_len_count[tid >> 6][lane] = 0u;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (my_len && before == 0) T.wave_len_count[tid >> 6][my_len] = (uint32_t)__popcll(same);
        if (lane == 0) T.wave_len_count[tid >> 6][0] = n_used | (n_bad << 16);  // (no code has length 0)
    }
    __syncthreads();
    if (tid < 64) {
        // running sums over the lengths: count(j) * 2^(48-j) gives the first code of each length (shifted down to
        // its own width), the Kraft sum and the "first value that is no code of this length" limits
        const bool in = tid >= 1 && tid <= kMaxLen;
        const uint32_t all = T.wave_len_count[0][tid] + T.wave_len_count[1][tid] + T.wave_len_count[2][tid] + T.wave_len_count[3][tid];
        const uint32_t c = in ? all : 0u, totals = (uint32_t)__builtin_amdgcn_readfirstlane((int)all);
        const unsigned long long w = (unsigned long long)c << (in ? kMaxLen - tid : 0);
        const unsigned long long incl = wave_inclusive_scan64(w);
        const uint32_t rank = wave_exclusive_scan(c);
        const unsigned long long kraft = __shfl(incl, 63, 64);
        const unsigned long long first = in ? ((incl - w) >> (kMaxLen - tid)) : 0ull;
        T.cnt_len[tid] = c;
        T.first_code[tid] = first;
        T.rank_of_code[tid] = in ? rank - (uint32_t)first : 0u;
        const unsigned long long lim32 = (in && tid <= 32) ? (incl >> (kMaxLen - 32)) : ~0ull;
        T.limit[tid] = lim32;
        T.limit32[tid] = lim32 > 0xffffffffull ? 0xffffffffu : (uint32_t)lim32;
        if (tid >= 1 && tid <= kLutBits) T.lut_limit[tid] = (uint32_t)(incl >> (kMaxLen - kLutBits));
        const unsigned long long used = __ballot(c != 0);
        const uint32_t n = totals & 0xffffu, c1 = (uint32_t)__builtin_amdgcn_readlane((int)c, 1);
        if (tid == 0) {
            T.n_used = n;
            T.max_len = used ? (uint32_t)(63 - __clzll((long long)used)) : 0u;
            T.ok = ((totals >> 16) == 0 && n >= 1 && (n == 1 ? c1 == 1 : kraft == (1ull << kMaxLen))) ? 1u : 0u;
        }
    }
    __syncthreads();
    if (!T.ok) return false;
    // symbols of equal length are numbered in symbol order
    if (tid < 256) {
        if (my_len) {
            for (int q = 0; q < (tid >> 6); q++) before += T.wave_len_count[q][my_len];
            T.sorted_sym[(T.rank_of_code[my_len] + (uint32_t)T.first_code[my_len] + before) & 255u] = (uint16_t)tid;
        }
        if ((uint32_t)tid >= T.n_used) T.sorted_sym[tid] = 0;  // ranks past the last code stay harmless
    }
    __syncthreads();
    {
        // Step 1: the first code in every kLutBits-bit value.  Canonical codes, left-aligned, grow with their
        // length, so the length is 1 + the number of per-length limits the value reaches.  Four values at a time: their
        // searches are independent and interleave (all of a thread's in one straight run waits for more instructions,
        // fetched for the first and only time, than it saves).
        uint32_t lim[kLutBits + 1];
#pragma unroll
        for (int l = 1; l <= kLutBits; l++) lim[l] = T.lut_limit[l];
#pragma unroll 4
        for (int it = 0; it < ((1 << kLutBits) + THREADS - 1) / THREADS; it++) {
            const uint32_t v = (uint32_t)(tid + it * THREADS);
            // (only workgroup sizes that do not divide the table need the test: without it the turns are one
            // straight run and their dependent LDS reads overlap)
            if constexpr (((1 << kLutBits) % THREADS) != 0) {
                if (v >= (1u << kLutBits)) break;
            }
            uint32_t len = 1;
#pragma unroll
            for (int l = 1; l < kLutBits; l++) len += (v >= lim[l]) ? 1u : 0u;
            const uint32_t at = (v >> (kLutBits - len)) + T.rank_of_code[len];
            const uint32_t entry = (uint32_t)T.sorted_sym[at & 255u] | (len << 8);
            T.first[first_slot(v)] = (uint16_t)(v < lim[kLutBits] ? entry : 0u);
        }
    }
    __syncthreads();
    {
        // Step 2: chain up to three codes per table entry (the index of an entry is in stream order, least
        // significant bit first).  A later code counts only if all its bits are inside the kLutBits bits.
        constexpr uint32_t kMask = (1u << kLutBits) - 1u;
#pragma unroll 4
        for (int it = 0; it < ((1 << kLutBits) + THREADS - 1) / THREADS; it++) {
            if constexpr (((1 << kLutBits) % THREADS) != 0) {
                if ((uint32_t)(tid + it * THREADS) >= (1u << kLutBits)) break;
            }
            // (neighbouring threads take neighbouring values v0: the reads of `first` below are neighbours, and the
            // entries, whose indices differ in their upper bits, go to different banks through lut_slot; taking
            // neighbouring indices instead puts every read of a wavefront on one bank)
            const uint32_t v0 = (uint32_t)(tid + it * THREADS);
            const int idx = (int)(__brev(v0) >> (32 - kLutBits));
            const uint32_t f0 = T.first[first_slot(v0)];
            const uint32_t len0 = f0 >> 8;
            const uint32_t v1 = (v0 << len0) & kMask;
            const uint32_t f1 = T.first[first_slot(v1)];
            const uint32_t len1 = f1 >> 8;
            const uint32_t v2 = (v1 << len1) & kMask;
            const uint32_t f2 = T.first[first_slot(v2)];
            const uint32_t len2 = f2 >> 8;
            const bool ok0 = len0 != 0;
            const bool ok1 = ok0 && len1 != 0 && len0 + len1 <= (uint32_t)kLutBits;
            const bool ok2 = ok1 && len2 != 0 && len0 + len1 + len2 <= (uint32_t)kLutBits;
            uint32_t e = 0;
            if (ok0) e = (f0 & 255u) | (len0 << 24) | (1u << 29);
            if (ok1) e = (f0 & 255u) | ((f1 & 255u) << 8) | ((len0 + len1) << 24) | (2u << 29);
            if (ok2) e = (f0 & 255u) | ((f1 & 255u) << 8) | ((f2 & 255u) << 16) | ((len0 + len1 + len2) << 24) | (3u << 29);
            T.lut[lut_slot((uint32_t)idx)] = e;
        }
    }
    __syncthreads();  // `first` is not read any more: the second table takes its place
    {
        // Step 3: the table of the longer codes (see DecTables).  Nothing to do where no code is longer than kLutBits.
        const uint32_t lim = T.lut_limit[kLutBits];  // kLutBits-bit values below it start with a short code
        const uint32_t max_len = T.max_len;
        const bool have_long = max_len > (uint32_t)kLutBits && lim < (1u << kLutBits);
        const uint32_t base = have_long ? lim << (32 - kLutBits) : 0xffffffffu;
        const uint64_t span = (1ull << 32) - base;  // values at or above base
        // the smallest shift that brings the span down to the table's 2^kLut2Bits entries (at most 32 - kLut2Bits),
        // in closed form: a loop over the candidates was 1.6 us of every workgroup's start
        uint32_t shift = 0;
        if (span > (1ull << kLut2Bits)) {
            const uint32_t m = 63u - (uint32_t)__clzll((long long)span);  // 2^m <= span < 2^(m+1), m > kLut2Bits - 1
            shift = m - kLut2Bits;
            if ((span >> shift) > (1ull << kLut2Bits)) shift++;
            if (shift > 32u - kLut2Bits) shift = 32u - kLut2Bits;
        }
        if (tid == 0) {
            T.long_base = base;
            T.long_shift = shift;
            T.pad0 = 0u;
            T.pad1 = 0u;
        }
        constexpr int IT = ((1 << kLut2Bits) + THREADS - 1) / THREADS;
        if (have_long) {
            // the limits of the lengths in use, out of one register (lane l holds that of length l)
            const uint32_t top = (uint32_t)__builtin_amdgcn_readfirstlane((int)(max_len < 33u ? max_len : 33u));
            const uint32_t limits = T.limit32[lane];
            uint32_t v[IT], len[IT];
#pragma unroll
            for (int it = 0; it < IT; it++) {
                v[it] = base + ((uint32_t)(tid + it * THREADS) << shift);  // (wraps past the table's last value: left out below)
                len[it] = kLutBits + 1;
            }
            for (uint32_t l = kLutBits + 1; l < top; l++) {
                const uint32_t lim_l = (uint32_t)__builtin_amdgcn_readlane((int)limits, (int)l);
#pragma unroll
                for (int it = 0; it < IT; it++) len[it] += v[it] >= lim_l ? 1u : 0u;
            }
#pragma unroll
            for (int it = 0; it < IT; it++) {
                const uint32_t idx = (uint32_t)(tid + it * THREADS), n = len[it];
                if (idx >= (1u << kLut2Bits)) break;
                uint32_t entry = 0;
                if (((uint64_t)idx << shift) < span && n <= 32u - shift && n <= 31u) {
                    const uint32_t code = v[it] >> (32 - n), off = code - (uint32_t)T.first_code[n];
                    if (off < T.cnt_len[n]) entry = (uint32_t)T.sorted_sym[(code + T.rank_of_code[n]) & 255u] | (n << 8);
                }
                T.lut2[idx] = (uint16_t)entry;
            }
        } else {
            // no entry of the first table sends a valid stream here; a corrupt one finds "undecided" and is caught
            // by the search
            for (uint32_t idx = (uint32_t)tid; idx < (1u << kLut2Bits); idx += THREADS) T.lut2[idx] = 0;
        }
    }
    __syncthreads();
    return true;
}

// Decode tables made once for a code table that is fixed beforehand, in global memory: what build_decode_tables
// leaves in LDS, and the code lengths they were made from.
struct PrebuiltTables {
    DecTables T;
    uint8_t len[256];
};
static_assert(sizeof(DecTables) % 16 == 0, "copied 16 bytes at a time");

// The prebuilt tables into LDS in place of building them -- after checking that the stream carries the very
// lengths they were made from (my_len: the stream's length of symbol threadIdx.x, threads past 255: anything).
// All THREADS threads call it; returns false for every thread on a mismatch.
template <int THREADS>
__device__ __forceinline__ bool load_decode_tables(DecTables& T, int my_len, const PrebuiltTables* pre) {
    const int tid = threadIdx.x;
    const uint4* src = reinterpret_cast<const uint4*>(&pre->T);
    uint4* dst = reinterpret_cast<uint4*>(&T);
    for (int i = tid; i < (int)(sizeof(DecTables) / 16); i += THREADS) dst[i] = src[i];
    const int mismatch = (tid < 256 && my_len != (int)pre->len[tid]) ? 1 : 0;
    return __syncthreads_or(mismatch) == 0;  // (also the barrier behind the copy)
}

__global__ __launch_bounds__(256) void k_build_decode_tables(const uint8_t* __restrict__ len_table, int bits,
                                                             PrebuiltTables* __restrict__ out, uint32_t* __restrict__ ok) {
    __shared__ __align__(16) DecTables T;
    const int tid = threadIdx.x;
    const bool good = build_decode_tables<256>(T, (int)len_table[tid], bits);
    if (tid == 0) *ok = good ? 1u : 0u;
    if (!good) return;
    const uint4* src = reinterpret_cast<const uint4*>(&T);
    uint4* dst = reinterpret_cast<uint4*>(&out->T);
    for (int i = tid; i < (int)(sizeof(DecTables) / 16); i += 256) dst[i] = src[i];
    out->len[tid] = len_table[tid];
}

hipError_t launch_build_decode_tables(const uint8_t* d_len_table, int bits, void* d_prebuilt, uint32_t* d_ok, hipStream_t s) {
    return launch(K_TABLE, k_build_decode_tables, dim3(1), dim3(256), 0, s, d_len_table, bits,
                  static_cast<PrebuiltTables*>(d_prebuilt), d_ok);
}
size_t prebuilt_decode_tables_bytes() { return sizeof(PrebuiltTables); }

// Decodes the `cnt` symbols of one run (one lane) starting at bit `start` of a chunk too large for the LDS copy of the
// payload into the symbol tile: its `nwords` words are read from global memory (`gw`), zero past their end.  Returns
// false if bits matched no code word.
// State: lo/hi are payload words widx and widx+1, sh the bit offset in lo, nxt word widx+2 (read ahead),
// so 32 valid bits are at hand for every table lookup and a step crosses at most one word boundary.
//
// Output of a run: symbol n of the tile at sym_addr(n).
struct ByteOut {
    uint8_t* tile;
    uint32_t a0, o, i;
    __device__ __forceinline__ ByteOut(uint8_t* t, uint32_t nbase) : tile(t), a0(nbase + 4u * (nbase >> 6)), o(nbase & 63u), i(0) {}
    __device__ __forceinline__ void put(uint32_t sym) {  // sym_addr(nbase + i) = a0 + i + 4 * ((o + i) >> 6)
        tile[a0 + i + (((o + i) >> 6) << 2)] = (uint8_t)sym;
        i++;
    }
};
template <typename Out>
__device__ __forceinline__ bool decode_run(const uint32_t* __restrict__ gw, uint32_t nwords, uint32_t start, uint32_t cnt,
                                           const DecTables& T, Out out) {
    auto fetch = [&](uint32_t rel) -> uint32_t { return (rel < nwords) ? gw[rel] : 0u; };
    // word index can not wrap: start <= 64 runs * 65535 bits
    uint32_t widx = start >> 5, sh = start & 31;
    uint32_t lo = fetch(widx), hi = fetch(widx + 1), nxt = fetch(widx + 2);
    bool ok = true;
    uint32_t i = 0;
    while (i < cnt) {
        const uint32_t w = __builtin_amdgcn_alignbit(hi, lo, sh);
        uint32_t e = T.lut[lut_slot(w & ((1u << kLutBits) - 1))];
        uint32_t n = e >> 29, sym0 = e & 255u, len0 = (e >> 24) & 31u;
        if (n == 0) {  // a code longer than the table: the second table decides most of them
            const uint32_t e2 = T.lut2[((__brev(w) - T.long_base) >> T.long_shift) & ((1u << kLut2Bits) - 1)];
            if (e2) {
                sym0 = e2 & 255u;
                len0 = e2 >> 8;
                n = 1;
            }
        }
        if (__builtin_expect(n == 0, 0)) {
            // Canonical codes, left-aligned, grow with their length, so the
            // length is kLutBits + 1 + the number of longer-length limits the next 32 bits reach.
            const uint32_t v = __brev(w);  // first stream bit on top
            uint32_t len = kLutBits + 1;
#pragma unroll
            for (int l = kLutBits + 1; l <= 32; l++) len += ((uint64_t)v >= T.limit[l]) ? 1u : 0u;
            if (len <= 32) {
                const uint32_t off = (v >> (32 - len)) - (uint32_t)T.first_code[len];
                if (off >= T.cnt_len[len]) ok = false;
                sym0 = T.sorted_sym[((v >> (32 - len)) + T.rank_of_code[len]) & 255u];
                len0 = len;
                n = 1;
            } else {
                // longer than 32 bits (needs a histogram as skewed as the Fibonacci numbers): bit by bit
                uint32_t bp = widx * 32 + sh;
                uint64_t code = 0;
                uint32_t sym = 0, l = 1;
                bool found = false;
                for (; l <= (uint32_t)kMaxLen; l++) {
                    code = (code << 1) | ((fetch(bp >> 5) >> (bp & 31)) & 1u);
                    bp++;
                    const uint64_t f = T.first_code[l];
                    const uint32_t c = T.cnt_len[l];
                    if (c && code >= f && code - f < c) {
                        sym = T.sorted_sym[((uint32_t)code + T.rank_of_code[l]) & 255u];
                        found = true;
                        break;
                    }
                }
                if (!found) ok = false;
                out.put(sym);
                i++;
                widx = bp >> 5;
                sh = bp & 31;
                lo = fetch(widx);
                hi = fetch(widx + 1);
                nxt = fetch(widx + 2);
                continue;
            }
        }
        // all symbols of the entry are consumed; those past the end of the run (they belong to the next run,
        // or are pad bits) are dropped, and where the cursor ends up after the run does not matter
        out.put(sym0);
        if (n >= 2 && i + 1 < cnt) out.put((e >> 8) & 255u);
        if (n >= 3 && i + 2 < cnt) out.put((e >> 16) & 255u);
        i += n;
        sh += len0;  // total length of the entry; at most 31 + 32: one word boundary at most
        const bool cross = sh >= 32;
        lo = cross ? hi : lo;
        hi = cross ? nxt : hi;
        widx += cross ? 1u : 0u;
        sh &= 31u;
        nxt = fetch(widx + 2);
    }
    return ok;
}

// The same for a chunk staged in LDS whose run goes to 64 consecutive bytes `out`, which 4 pad bytes of the tile
// follow.  One turn of the loop reads the 64 stream bits around the cursor once (two words, at least 33 of them
// ahead of the cursor) and looks three table entries up in them, one after the other (up to 11 bits each, so the
// third still finds its 11 bits): up to nine symbols for one read of the stream and three of the table.  An
// entry's three symbol bytes go to the current position with byte stores (one unaligned 32-bit store instead
// stalls the LDS: its counters showed 70 % of its busy time in such stalls); the next entry overwrites what was not a
// symbol, and stores past the end of the run go to the pad bytes.  An entry of no symbols (a code longer than the table) leaves the cursor where it is, so the
// entries after it in the same turn are the same one: the wavefront looks at the last entry only, and branches (as
// a whole) when one of its lanes has met such a code inside its run.
// `pw` holds the chunk's nwords words and at least kPayOverrun words of any content behind them: a run of a corrupt
// stream may read that far (every symbol moves the cursor by at most 48 bits, and a run ends after 64 symbols and
// at most two more table entries), never further.
constexpr int kPayOverrun = 104;
__device__ __forceinline__ bool decode_run_bytes(const uint32_t* pw, uint32_t nwords, uint32_t start, uint32_t cnt,
                                                 const DecTables& T, uint8_t* out) {
    constexpr uint32_t kMask = (1u << kLutBits) - 1u;
    uint32_t bit = start < 32u * nwords ? start : 32u * nwords;  // (side information of a corrupt stream)
    uint32_t bad = 0u, i = 0u;
    // An entry's symbols, at the current position; the next entry is requested before they are stored (the LDS serves a
    // wavefront in order: behind the three stores the chain of entries waits for them too).
    auto put = [&](uint32_t e, uint32_t at) {
        out[at] = (uint8_t)e;
        out[at + 1] = (uint8_t)(e >> 8);
        out[at + 2] = (uint8_t)(e >> 16);
    };
    uint32_t lo = pw[bit >> 5], hi = pw[(bit >> 5) + 1u];
    while (i < cnt) {
        const unsigned long long win = ((unsigned long long)hi << 32) | lo;
        uint32_t sh = bit & 31u;
        const uint32_t e0 = T.lut[lut_slot(__builtin_amdgcn_alignbit(hi, lo, sh) & kMask)];
        const uint32_t l0 = (e0 >> 24) & 31u;
        sh += l0;
        const uint32_t e1 = T.lut[lut_slot((uint32_t)(win >> sh) & kMask)];
        put(e0, i);  // i < 64: the store stays inside the run's 64 + 4 bytes
        i += e0 >> 29;
        const uint32_t l1 = (e1 >> 24) & 31u;
        sh += l1;
        const uint32_t e2 = T.lut[lut_slot((uint32_t)(win >> sh) & kMask)];
        put(e1, i < 64u ? i : 64u);
        i += e1 >> 29;
        bit += l0 + l1 + ((e2 >> 24) & 31u);
        lo = pw[bit >> 5];
        hi = pw[(bit >> 5) + 1u];
        put(e2, i < 64u ? i : 64u);
        i += e2 >> 29;
        const bool is_long = (e2 >> 29) == 0 && i < cnt;
        if (__builtin_expect(__any(is_long), 0)) {
            if (is_long) {
                // A code longer than the table starts at the cursor.  The next 32 bits, first stream bit on top:
                const uint32_t* qq = pw + (bit >> 5);
                const uint32_t v = __brev(__builtin_amdgcn_alignbit(qq[1], qq[0], bit & 31u));
                uint32_t sym = 0, len = 0;
                // the second table decides most of them
                const uint32_t e2 = T.lut2[((v - T.long_base) >> T.long_shift) & ((1u << kLut2Bits) - 1)];
                if (e2) {
                    sym = e2 & 255u;
                    len = e2 >> 8;
                } else {
                    // Canonical codes, left-aligned, grow with their length, so the length is kLutBits + 1 + the
                    // number of longer-length limits the 32 bits reach (limits of the lengths below the longest one
                    // are below 2^32; the longest needs no test).  One limit at a time: this is rare, and registers
                    // it would hold for all limits at once would be the whole loop's.
                    const uint32_t top = T.max_len < 33u ? T.max_len : 33u;
                    len = kLutBits + 1;
#pragma unroll 1
                    for (uint32_t q = kLutBits + 1; q < top; q++) {
                        if (v < T.limit32[q]) break;
                        len++;
                    }
                    if (len <= 32) {
                        const uint32_t off = (v >> (32 - len)) - (uint32_t)T.first_code[len];
                        if (off >= T.cnt_len[len]) bad = 1u;
                        sym = T.sorted_sym[((v >> (32 - len)) + T.rank_of_code[len]) & 255u];
                    } else {
                        // longer than 32 bits (needs a histogram as skewed as the Fibonacci numbers): bit by bit
                        unsigned long long code = 0;
                        bool found = false;
                        uint32_t bp = bit;
#pragma unroll 1
                        for (len = 1; len <= (uint32_t)kMaxLen; len++) {
                            code = (code << 1) | ((pw[bp >> 5] >> (bp & 31)) & 1u);
                            bp++;
                            const unsigned long long f = T.first_code[len];
                            const uint32_t c = T.cnt_len[len];
                            if (c && code >= f && code - f < c) {
                                sym = T.sorted_sym[((uint32_t)code + T.rank_of_code[len]) & 255u];
                                found = true;
                                break;
                            }
                        }
                        if (!found) {
                            bad = 1u;
                            len = kMaxLen;
                        }
                    }
                }
                out[i] = (uint8_t)sym;
                i++;
                bit += len;
                lo = pw[bit >> 5];
                hi = pw[(bit >> 5) + 1u];
            }
        }
    }
    return bad == 0u;
}

struct DecodeParams {
    const uint8_t* stream;
    size_t bytes;
    int64_t P;
    int64_t HW;
    int C;
    int bits;
    int tile_px;       // pixels of a workgroup tile (k_decode_tiles; its chunks follow from the stream's header)
    uint32_t tile_bytes;  // ... and the LDS for its symbols
    int ncs;           // Cpad / 32
    const uint16_t* Bp16;  // inverse operand (T^T), f16 split, in operand order
    const float* mu;   // [Cpad]
    float* xhat;       // NULL in symbols-only mode
    uint8_t* syms_out; // non-NULL in symbols-only mode
    uint32_t* err;
    // where the side information and the payload start if the stream was made with the nominal chunk size
    size_t g_off_chunk_off, g_off_sub_bits, g_off_payload;
    uint32_t g_n_chunks, g_spc, g_tile_chunks;
    const void* prebuilt;  // PrebuiltTables of a code table fixed beforehand, or NULL: build them from the stream
    // chunk decoder: bytes of the basis operand at the start of its dynamic LDS, and the words of payload the LDS
    // copy of a chunk holds (larger chunks are read in place); a multiple of 64
    uint32_t lds_basis_bytes, pay_words;
    int active_steps;      // contraction steps of 16 coefficients up to the basis' last row that is not all zero
    // 8-bit reconstruction in the chunk decoder (k_decode_chunks<..., U8 = true>): the transposed 8-bit basis in
    // the operand order of the integer matrix instruction [ncs][ceil(C / 16)][64], its column sums and the mean
    // in activation units (both padded to ncs * 32), h / 256 = s_T Delta / s_x, and the output bytes
    const unsigned long long* op8;
    const int* col_sum;
    const double* mean_d;
    double factor8;
    uint8_t* out8;
};

// Header checks.  Returns false unless the header matches the arguments and the
// buffer holds every section it announces.
struct StreamView {
    uint32_t n_chunks, spc, chunk_syms, payload_words;
    uint64_t ppc;
    const uint32_t* chunk_off;
    const uint16_t* sub_bits;
    const uint32_t* payload;
    float delta;
};
// (requested before anything else of the stream: see the kernels)
__device__ __forceinline__ Header load_header(const DecodeParams& p) {
    return p.bytes < (size_t)(kHeaderBytes + kLenTableBytes) ? Header{} : *reinterpret_cast<const Header*>(p.stream);
}
__device__ __forceinline__ bool open_stream(const DecodeParams& p, const Header& hd, StreamView* v) {
    if (p.bytes < (size_t)(kHeaderBytes + kLenTableBytes)) return false;
    const uint64_t ppc = hd.px_per_chunk;
    const uint64_t chunk_syms64 = ppc * (uint64_t)p.C;
    bool ok = hd.magic == kMagic && hd.version == 1 && hd.bits == p.bits && hd.C == (uint32_t)p.C &&
              hd.P == (uint64_t)p.P && hd.sub_syms == (uint32_t)kSubSyms && ppc >= 1 &&
              (chunk_syms64 <= 4096 || ppc == 1) && hd.delta > 0.f;
    if (!ok) return false;
    const uint64_t nch = ((uint64_t)p.P + ppc - 1) / ppc;
    const uint32_t spc = (uint32_t)((chunk_syms64 + kSubSyms - 1) / kSubSyms);
    if (nch != hd.n_chunks || spc != hd.subs_per_chunk) return false;
    const size_t off_co = kHeaderBytes + kLenTableBytes;
    const size_t off_sub = (off_co + 4 * ((size_t)nch + 1) + 15) & ~(size_t)15;
    const size_t off_pay = (off_sub + 2 * (size_t)nch * spc + 15) & ~(size_t)15;
    if (!(p.bytes >= off_pay && (p.bytes - off_pay) / 4 >= hd.payload_words && hd.payload_words <= 0xffffffffull))
        return false;
    v->n_chunks = (uint32_t)nch;
    v->spc = spc;
    v->chunk_syms = (uint32_t)chunk_syms64;
    v->payload_words = (uint32_t)hd.payload_words;
    v->ppc = ppc;
    v->chunk_off = reinterpret_cast<const uint32_t*>(p.stream + off_co);
    v->sub_bits = reinterpret_cast<const uint16_t*>(p.stream + off_sub);
    v->payload = reinterpret_cast<const uint32_t*>(p.stream + off_pay);
    v->delta = hd.delta;
    return true;
}

// A unit: the neighbouring chunks that one wavefront decodes together, as many as leave a lane for each of their runs (one
// where a chunk has more than 32 runs).  Lane l takes run l of them (their run sizes lie one behind the other in the
// stream, and so do their words), whose symbols go to slot l of the unit's tile (see sym_addr).
// (One chunk per wavefront and turn leaves three quarters of the lanes idle where chunks have 1024 symbols, pays every
// chunk's latencies by itself, and made a wide tensor's tiles as many pixels smaller as its chunks are.  Kernel times, us:
// 128 channels, 21 x 24, chunks of 1024 52 -> 20; 100 channels, N = 33, 27 x 31, chunks of 2048 35 -> 29; 384 channels,
// N = 71, 11 x 11, 1024 106 -> 30; 1024 channels, 25 x 25, 1024 86 -> 31.)
struct Unit {
    uint32_t m, n_units;
    uint32_t lane_ch, lane_run;  // this lane's chunk of the unit and run of the chunk
    __device__ __forceinline__ Unit(const StreamView& v, int lane)
        : m(1u), n_units(v.n_chunks), lane_ch((uint32_t)lane < v.spc ? 0u : 1u), lane_run((uint32_t)lane) {
        if (v.spc <= 32u) {  // (no divisions before the first chunk otherwise)
            m = 64u / v.spc;
            n_units = (v.n_chunks + m - 1u) / m;
            lane_ch = (uint32_t)lane / v.spc;
            lane_run = (uint32_t)lane - lane_ch * v.spc;
        }
    }
};
// What the stream says about a unit of `count` chunks from chunk c0 on, requested ahead of its use.
struct UnitInfo {
    uint32_t off;  // first payload word of this lane's chunk (lane 0: of the unit; lanes without a chunk: anything)
    uint32_t end;  // the unit's end
    uint32_t run;  // bits of this lane's run
    __device__ __forceinline__ void load(const StreamView& v, const Unit& un, uint32_t c0, uint32_t count, int lane) {
        const bool in = un.lane_ch < count;
        off = v.chunk_off[c0 + (in ? un.lane_ch : 0u)];
        end = v.chunk_off[c0 + count];
        run = in ? v.sub_bits[(size_t)c0 * v.spc + (uint32_t)lane] : 0u;
    }
};
// The same checked, for the wavefront that is about to decode it.
struct UnitBits {
    uint32_t w0, n_words;  // the unit's words of the payload
    uint32_t rel;          // ... of which this many come before this lane's chunk
    uint32_t start;        // first bit of this lane's run in its chunk
    uint32_t cnt;          // its symbols
    bool bad;              // offsets out of order or past the payload: nothing of the unit is read
};
__device__ __forceinline__ UnitBits open_unit(const StreamView& v, const Unit& un, const UnitInfo& in, uint32_t c0, uint32_t count,
                                              uint32_t last_syms, int lane) {
    UnitBits b;
    b.w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)in.off);
    const uint32_t w1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)in.end);
    b.bad = b.w0 > w1 || w1 > v.payload_words;
    const bool mine = un.lane_ch < count;
    b.start = wave_exclusive_scan(in.run);
    b.rel = 0u;
    if (count > 1u) {  // wavefront-uniform
        const uint32_t next = (uint32_t)__shfl((int)in.off, lane + (int)v.spc, 64);
        b.bad = b.bad || __any(mine && in.off > (un.lane_ch + 1u < count ? next : w1)) != 0;
        b.start -= (uint32_t)__shfl((int)b.start, lane - (int)un.lane_run, 64);
        b.rel = mine && !b.bad ? in.off - b.w0 : 0u;
    }
    b.n_words = b.bad ? 0u : w1 - b.w0;
    if (b.bad) b.w0 = 0u;
    const uint32_t syms = c0 + un.lane_ch == v.n_chunks - 1u ? last_syms : v.chunk_syms, r0 = un.lane_run * (uint32_t)kSubSyms;
    b.cnt = mine && r0 < syms ? (syms - r0 < (uint32_t)kSubSyms ? syms - r0 : (uint32_t)kSubSyms) : 0u;
    return b;
}

// Wide tensors and the symbols-only mode: a tile of G chunks per workgroup is decoded into an LDS tile of symbol
// bytes, one unit per wavefront and round; the inverse transform of the tile's pixels then runs on the f16 matrix
// cores with the arithmetic of the narrow-tensor kernel below (levels exact in f16, basis entries split in two f16
// parts, two matrix instructions per 16 coefficients), shared out over the wavefronts (see the loop).
// MT: pixel tiles of 32 per workgroup; KS: wavefronts that share a channel tile's contraction (MT = 1).
template <int MT, int KS, int LAYOUT, bool ALIGNED4>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(MT == 1 ? 4 : 2, MT == 1 ? 4 : 2))) void k_decode_tiles(DecodeParams p) {
    static_assert(KS == 1 || MT == 1, "the partial sums of one pixel tile fit the payload buffers");
    __shared__ __align__(16) DecTables T;
    constexpr int CTW = 8 / KS;  // channel tiles of a workgroup: a wavefront (or KS of them) each
    // dynamic LDS: the chunks' payload words (a buffer per wavefront: the unit's words and the room a corrupt stream's
    // cursor may run into) while decoding, the partial sums [KS][CTW][4][64] afterwards (the two uses are a workgroup
    // barrier apart), then the symbol tile
    extern __shared__ __align__(16) uint8_t dyn_lds[];
    float4* s_part = reinterpret_cast<float4*>(dyn_lds);
    uint8_t* symtile = dyn_lds + p.lds_basis_bytes;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wavefront-uniform by construction
    const int half = lane >> 5, l32 = lane & 31;
    const int C = p.C;

    // What does not depend on the header goes out first: the code lengths, and (see the chunk decoder) offsets, run sizes
    // and payload of the wavefront's first chunk, where the nominal chunk size puts them.  The guess is checked against the
    // header below.  Nothing outside [stream, stream + bytes) is touched either way.
    const Header hd = load_header(p);
    const int my_len = tid < 256 && p.bytes >= (size_t)(kHeaderBytes + kLenTableBytes) ? (int)p.stream[kHeaderBytes + tid] : 0;
    uint32_t* pw = reinterpret_cast<uint32_t*>(dyn_lds) + (size_t)wave * (p.pay_words + (uint32_t)kPayOverrun);
    const uint32_t ch_first = blockIdx.y * p.g_tile_chunks + (uint32_t)wave;
    const bool guess = p.g_off_payload <= p.bytes && (uint32_t)wave < p.g_tile_chunks && ch_first < p.g_n_chunks && p.g_spc > 32u;  // (a chunk is a unit)
    UnitInfo first{0u, 0u, 0u};
    uint32_t first_w0 = 0u, first_w1 = 0u;
    bool first_in_lds = false;
    if (guess) {
        const uint32_t* co = reinterpret_cast<const uint32_t*>(p.stream + p.g_off_chunk_off);
        const uint16_t* sb = reinterpret_cast<const uint16_t*>(p.stream + p.g_off_sub_bits);
        first.off = co[ch_first];
        first.end = co[ch_first + 1];
        first.run = ((uint32_t)lane < p.g_spc) ? sb[(size_t)ch_first * p.g_spc + lane] : 0u;
        const size_t cap_words = (p.bytes - p.g_off_payload) / 4;
        first_w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)first.off);
        first_w1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)first.end);
        first_in_lds = first_w0 <= first_w1 && (size_t)first_w1 <= cap_words && first_w1 - first_w0 <= p.pay_words;
        if (first_in_lds) {
            const uint32_t* src = reinterpret_cast<const uint32_t*>(p.stream + p.g_off_payload) + first_w0;
            for (uint32_t k = 0; 64u * k < first_w1 - first_w0; k++) {  // wavefront-uniform trip count
                const uint32_t i = (uint32_t)lane + 64u * k;
                if (i < first_w1 - first_w0) load_to_lds<4>(src + i, pw + 64u * k);
            }
        }
    }
    StreamView sv;
    if (!open_stream(p, hd, &sv)) {
        if (tid == 0) atomicOr(p.err, FMTC_ERR_HEADER);
        return;
    }
    const uint32_t n_chunks = sv.n_chunks, spc = sv.spc, chunk_syms = sv.chunk_syms, ppc = (uint32_t)sv.ppc;
    const uint32_t slot_bytes = 68u * spc;  // of a chunk in the symbol tile: every run has its place (see sym_addr)
    const uint64_t V = (uint64_t)p.P * (uint64_t)C;
    const uint32_t last_syms = (uint32_t)(V - (uint64_t)(n_chunks - 1u) * chunk_syms);
    const Unit un(sv, lane);
    const float delta = sv.delta;
    // Chunks of a tile: what the stream's chunk size makes of the tile's pixels (symbols only: of a unit per wavefront), and
    // what its LDS holds.
    uint32_t G = p.syms_out ? 8u * un.m : (uint32_t)p.tile_px / ppc;
    const uint32_t fits = p.tile_bytes / slot_bytes;
    G = G < 1u ? 1u : (G > fits ? fits : G);
    bool guessed = guess && sv.n_chunks == p.g_n_chunks && sv.spc == p.g_spc && G == p.g_tile_chunks;  // of the first unit
    const uint32_t n_tiles = (n_chunks + G - 1) / G;
    if (blockIdx.y >= n_tiles) {  // (the grid is made for any chunk size)
        wait_loads<0>();  // (nothing is on its way into LDS any more)
        return;
    }
    if (!(p.prebuilt ? load_decode_tables<512>(T, my_len, static_cast<const PrebuiltTables*>(p.prebuilt))
                     : build_decode_tables<512>(T, my_len, p.bits))) {
        if (tid == 0) atomicOr(p.err, FMTC_ERR_TABLE);
        return;
    }
    __syncthreads();

    // 0x6400 | s is the f16 number 1024 + s: the level s - 2^(b-1) is that minus (1024 + 2^(b-1)), exactly
    const _Float16 level_off = (_Float16)(float)(1024 + (1 << (p.bits - 1)));
    const halfx2 level_off2 = {level_off, level_off};
    const int NJ = p.ncs * 2;  // steps of 16 coefficients
    // ... of which the first NJA meet basis rows that are not all zero (fewer than NJ for a truncated basis)
    const int NJA = p.active_steps < 1 ? 1 : (p.active_steps > NJ ? NJ : p.active_steps);

    // x_hat = Delta (sum q T_hi + 2^-11 sum q T_lo) + mu for quads g0 .. g0 + NQ - 1 of one 32 x 32 tile (channel tile ct, pixel
    // tile pt of a workgroup tile of TP pixels starting at pixel px_tile0), y the sums.  Element 4 g + i of lane l is element
    // (8 g + 4*(l/32) + i, l%32) of the tile: rows = pixels for NHWC, channels for NCHW.  Whole tiles are
    // stored without per-element predicates (one straight run of stores).
    auto store_quads = [&](int ct, int pt, int TP, int64_t px_tile0, auto& y, int g0) {
        constexpr int NR = sizeof(y) / sizeof(float);
        if constexpr (LAYOUT == FMTC_NHWC) {
            const int c = ct * 32 + l32;
            if (c < C) {
                const float m_c = p.mu[c];
                const int px_first = pt * 32 + 8 * g0;
                float* dst = p.xhat + (px_tile0 + px_first + 4 * half) * C + c;
                if (pt * 32 + 32 <= TP) {
#pragma unroll
                    for (int r = 0; r < NR; r++) dst[(size_t)(8 * (r >> 2) + (r & 3)) * C] = y[r] * delta + m_c;
                } else {
#pragma unroll
                    for (int r = 0; r < NR; r++) {
                        int pxl = px_first + 8 * (r >> 2) + 4 * half + (r & 3);
                        if (pxl < TP) dst[(size_t)(8 * (r >> 2) + (r & 3)) * C] = y[r] * delta + m_c;
                    }
                }
            }
        } else {
            float m_r[NR];
            const int cb = ct * 32 + 8 * g0 + 4 * half;
#pragma unroll
            for (int r = 0; r < NR; r++) m_r[r] = p.mu[cb + 8 * (r >> 2) + (r & 3)];  // mu is padded to a multiple of 32
            const int pxl = pt * 32 + l32;
            if (pxl < TP) {
                const int64_t px = px_tile0 + pxl;
                const int64_t n = px / p.HW, hw = px - n * p.HW;
                float* dst = p.xhat + (n * (int64_t)C + cb) * p.HW + hw;
                if (ct * 32 + 32 <= C) {
#pragma unroll
                    for (int r = 0; r < NR; r++) dst[(int64_t)(8 * (r >> 2) + (r & 3)) * p.HW] = y[r] * delta + m_r[r];
                } else {
#pragma unroll
                    for (int r = 0; r < NR; r++) {
                        int c = cb + 8 * (r >> 2) + (r & 3);
                        if (c < C) dst[(int64_t)(8 * (r >> 2) + (r & 3)) * p.HW] = y[r] * delta + m_r[r];
                    }
                }
            }
        }
    };

    for (uint32_t tile = blockIdx.y; tile < n_tiles; tile += gridDim.y) {
        const uint32_t first_ch = tile * G;
        const uint32_t tile_chunks = n_chunks - first_ch < G ? n_chunks - first_ch : G;
        // ---- variable length decoding into the LDS tile, a unit per wavefront and round ----
        for (uint32_t k0 = (uint32_t)wave * un.m; k0 < tile_chunks; k0 += 8u * un.m) {
            const uint32_t count = tile_chunks - k0 < un.m ? tile_chunks - k0 : un.m;
            UnitInfo info = first;
            if (!guessed) info.load(sv, un, first_ch + k0, count, lane);
            const UnitBits ub = open_unit(sv, un, info, first_ch + k0, count, last_syms, lane);
            if (ub.bad && lane == 0) atomicOr(p.err, FMTC_ERR_OFFSETS);
            uint8_t* slots = symtile + slot_bytes * k0;
            bool ok_run = true;
            if (ub.n_words <= p.pay_words) {
                // the unit's payload goes to LDS with full-width loads (what lies behind it there is never taken for a
                // symbol of a run)
                if (guessed && first_in_lds && ub.w0 == first_w0 && ub.w0 + ub.n_words == first_w1) {
                    wait_loads<0>();
                } else {
                    wait_loads<0>();  // (a guess that was wrong must not land later)
                    const uint32_t* src = sv.payload + ub.w0;
                    for (uint32_t i = lane; i < ub.n_words; i += 64) pw[i] = src[i];
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
                if (ub.cnt) ok_run = decode_run_bytes(pw, ub.n_words, ub.start + 32u * ub.rel, ub.cnt, T, slots + 68u * (uint32_t)lane);
                // the next unit of this wavefront overwrites the copy: all lanes are done reading here
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            } else if (ub.cnt) {
                // a unit too large for the LDS copy is read in place
                ok_run = decode_run(sv.payload + ub.w0 + ub.rel, ub.n_words - ub.rel, ub.start, ub.cnt, T, ByteOut(slots, 64u * (uint32_t)lane));
            }
            if (!ok_run) atomicOr(p.err, FMTC_ERR_CODE);
            guessed = false;
        }
        guessed = false;
        wait_loads<0>();  // (of a wavefront without a unit: the room is used again below)
        __syncthreads();

        if (p.syms_out) {
            // (a chunk per wavefront and round)
            for (uint32_t k = (uint32_t)wave; k < tile_chunks; k += 8u) {
                const uint32_t syms = first_ch + k == n_chunks - 1u ? last_syms : chunk_syms;
                const uint8_t* src = symtile + slot_bytes * k;
                uint8_t* dst = p.syms_out + (uint64_t)(first_ch + k) * chunk_syms;
                if constexpr (ALIGNED4) {
                    for (uint32_t n = 4u * (uint32_t)lane; n < syms; n += 256u)
                        *reinterpret_cast<uint32_t*>(dst + n) = *reinterpret_cast<const uint32_t*>(src + sym_addr(n));
                } else {
                    for (uint32_t n = (uint32_t)lane; n < syms; n += 64u) dst[n] = src[sym_addr(n)];
                }
            }
        } else {
            // ---- inverse quantizer + inverse transform: a tiled matrix product over the workgroup's pixels ----
            // A wavefront takes one channel tile for all MT pixel tiles (KS of them share its contraction).  The basis (both
            // f16 parts, 16 bytes per lane each, operand order) comes straight into registers D steps ahead, every block
            // once per workgroup; no barrier until the sums are made.  The other operand is read from the symbol tile: lane
            // (pixel, h) takes the eight symbols 16 ks + 8 h .. + 7 of its pixel and turns them into f16 levels with two
            // byte permutes each.
            const int64_t px_tile0 = (int64_t)first_ch * (int64_t)ppc;
            int TP = p.P - px_tile0 < (int64_t)(tile_chunks * ppc) ? (int)(p.P - px_tile0) : (int)(tile_chunks * ppc);  // pixels in this tile
            if (TP > MT * 32) TP = MT * 32;  // (not so: a chunk of a wide tensor has fewer pixels than a tile)
            const int n_cg = (p.ncs + CTW - 1) / CTW;
            const int slice = wave / CTW;
            const int s_begin = slice * NJA / KS, s_end = (slice + 1) * NJA / KS;
            uint32_t rowbase[MT];       // this lane's first symbol of a pixel in its chunk ...
            const uint8_t* rows[MT];    // ... which starts here
#pragma unroll
            for (int b = 0; b < MT; b++) {
                int pxl = b * 32 + l32;
                if (pxl > TP - 1) pxl = TP - 1;  // rows past the tile repeat the last pixel; never stored
                if (pxl < 0) pxl = 0;
                const uint32_t k = (uint32_t)pxl / ppc;
                rows[b] = symtile + slot_bytes * k;
                rowbase[b] = ((uint32_t)pxl - k * ppc) * (uint32_t)C + 8u * half;
            }
            constexpr int D = MT == 4 ? 2 : 3;
            for (int cg = blockIdx.x; cg < n_cg; cg += gridDim.x) {
                const int ct = cg * CTW + wave % CTW;
                const bool mine = ct < p.ncs;  // wavefront-uniform
                floatx16 acc[MT], acl[MT];
#pragma unroll
                for (int b = 0; b < MT; b++)
#pragma unroll
                    for (int r = 0; r < 16; r++) { acc[b][r] = 0.f; acl[b][r] = 0.f; }
                if (mine) {
                    const uint4* src = reinterpret_cast<const uint4*>(p.Bp16) + (size_t)ct * NJ * 128 + lane;
                    uint4 bufh[D], bufl[D];
#pragma unroll
                    for (int d = 0; d < D; d++)
                        if (s_begin + d < s_end) {
                            bufh[d] = src[(size_t)(s_begin + d) * 128];
                            bufl[d] = src[(size_t)(s_begin + d) * 128 + 64];
                        }
                    for (int k0 = s_begin; k0 < s_end; k0 += D) {
#pragma unroll
                        for (int d = 0; d < D; d++) {
                            const int ks = k0 + d;
                            if (ks >= s_end) break;  // wavefront-uniform
                            halfx8 q[MT];
#pragma unroll
                            for (int b = 0; b < MT; b++) {
                                // (coefficients past C meet zero basis entries; whatever level the tile's bytes give there
                                // does not count)
                                const uint32_t n = rowbase[b] + 16u * (uint32_t)ks;
                                uint32_t w0, w1;
                                read_octet<ALIGNED4>(rows[b], n, w0, w1);
                                const halfx2 q01 = __builtin_bit_cast(halfx2, __builtin_amdgcn_perm(0x64646464u, w0, 0x05010400u)) - level_off2;
                                const halfx2 q23 = __builtin_bit_cast(halfx2, __builtin_amdgcn_perm(0x64646464u, w0, 0x07030602u)) - level_off2;
                                const halfx2 q45 = __builtin_bit_cast(halfx2, __builtin_amdgcn_perm(0x64646464u, w1, 0x05010400u)) - level_off2;
                                const halfx2 q67 = __builtin_bit_cast(halfx2, __builtin_amdgcn_perm(0x64646464u, w1, 0x07030602u)) - level_off2;
                                q[b] = halfx8{q01[0], q01[1], q23[0], q23[1], q45[0], q45[1], q67[0], q67[1]};
                            }
                            const halfx8 bh = __builtin_bit_cast(halfx8, bufh[d]), bl = __builtin_bit_cast(halfx8, bufl[d]);
#pragma unroll
                            for (int b = 0; b < MT; b++) {
                                if constexpr (LAYOUT == FMTC_NHWC) {
                                    acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(q[b], bh, acc[b], 0, 0, 0);
                                    acl[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(q[b], bl, acl[b], 0, 0, 0);
                                } else {
                                    acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bh, q[b], acc[b], 0, 0, 0);
                                    acl[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bl, q[b], acl[b], 0, 0, 0);
                                }
                            }
                            if (ks + D < s_end) {
                                bufh[d] = src[(size_t)(ks + D) * 128];
                                bufl[d] = src[(size_t)(ks + D) * 128 + 64];
                            }
                        }
                    }
                }
                if constexpr (KS == 1) {
                    if (mine) {
#pragma unroll
                        for (int b = 0; b < MT; b++) {
                            if (b * 32 >= TP) break;  // wavefront-uniform
                            float y[16];
#pragma unroll
                            for (int r = 0; r < 16; r++) y[r] = __builtin_fmaf(acl[b][r], 1.f / 2048.f, acc[b][r]);
                            store_quads(ct, b, TP, px_tile0, y, 0);
                        }
                    }
                } else {
                    // the partial sums meet; each of the KS wavefronts finishes its share of the tile
                    __syncthreads();  // the payload (the previous group's sums) has been read
#pragma unroll
                    for (int g = 0; g < 4; g++) {
                        float y[4];
#pragma unroll
                        for (int i = 0; i < 4; i++) y[i] = __builtin_fmaf(acl[0][4 * g + i], 1.f / 2048.f, acc[0][4 * g + i]);
                        s_part[(wave * 4 + g) * 64 + lane] = make_float4(y[0], y[1], y[2], y[3]);
                    }
                    __syncthreads();
                    if (mine) {
                        constexpr int NQ = 4 / KS;
                        float y[4 * NQ];
#pragma unroll
                        for (int g = 0; g < NQ; g++) {
                            float4 t = s_part[((wave % CTW) * 4 + slice * NQ + g) * 64 + lane];
#pragma unroll
                            for (int w = 1; w < KS; w++) {
                                const float4 o = s_part[((wave % CTW + w * CTW) * 4 + slice * NQ + g) * 64 + lane];
                                t.x += o.x; t.y += o.y; t.z += o.z; t.w += o.w;
                            }
                            y[4 * g] = t.x; y[4 * g + 1] = t.y; y[4 * g + 2] = t.z; y[4 * g + 3] = t.w;
                        }
                        store_quads(ct, 0, TP, px_tile0, y, slice * NQ);
                    }
                }
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Narrow tensors (at most 160 channels after padding to 32): a chunk holds at least 25
// pixels, so the wavefront that decoded it has whole matrix tiles of its own.  The inverse
// transform runs on the f16 matrix cores (v_mfma_f32_32x32x16_f16): the levels s - 2^(b-1)
// are small integers, exact in f16, and every basis entry is split in two f16 parts,
// T = hi + lo / 2^11 (22 significant bits; see pack_operand16 on the host), so
//   x_hat = Delta (sum q T_hi + 2^-11 sum q T_lo) + mu
// with exact products and fp32 accumulation: two instructions per 16 coefficients where the
// fp32 instruction needs eight four times as long.  The basis is copied once per workgroup
// into LDS in operand order; lane (row, half) of the other operand reads the eight symbols
// 16j + 8*half + e of its pixel (the contraction index may be walked in any order as long as
// both operands agree on it).  Delta and mu are applied in the epilogue.
// ---------------------------------------------------------------------------
typedef int intx16 __attribute__((ext_vector_type(16)));
constexpr int kChunkTileBytes = 4096 + 4096 / 16 + 64;  // symbols, 4 pad bytes per run, slack for padded reads

// WAVES wavefronts per workgroup: two per SIMD (the second hides the latencies of the first; the workgroup holds one copy of
// the basis), up to four where registers and LDS allow, one for five channel tiles of a count left open (see launch_decode).
// U8: the tile's symbols go through the 8-bit basis on the integer matrix cores instead (v_mfma_i32_32x32x16_i8;
// exact sums, one fused fp64 multiply-add and one rounding per value, 8-bit activations out); the 8-bit basis
// takes the f16 basis' place in LDS.
// CFIX: the tensor's channel count if the kernel is built for one (the launcher checks it; 0: any), which makes every
// row stride a constant.
// LOG: only the upper f16 parts of the basis are kept in LDS; the lower parts, whose products are the small
// correction, are read from global memory (the cache serves them: every wavefront of the device reads the same few
// tens of KB) while the matrix instructions of the upper parts run.  Half the LDS per workgroup buys a third
// wavefront per SIMD for 128 to 160 channels.
template <int NCT, int LAYOUT, bool ALIGNED4, int WAVES, bool U8 = false, int CFIX = 0, bool LOG = false, int NLO = 0>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(WAVES / 4, WAVES / 4))) void k_decode_chunks(DecodeParams p) {
    constexpr int THREADS = WAVES * 64;
    __shared__ __align__(16) DecTables T;
    __shared__ __align__(16) uint8_t symtile[WAVES][kChunkTileBytes];
    __shared__ float s_mu[NCT * 32];
    // 8-bit variant: column sums and means of the channels (read for every value of the epilogue)
    __shared__ int s_col_sum[U8 ? NCT * 32 : 1];
    __shared__ double s_mean_d[U8 ? NCT * 32 : 1];
    // the basis operand [NCT][NJ][2][64], then per wavefront the chunk's payload words and room for a corrupt
    // stream's overrun
    extern __shared__ __align__(16) uint4 basis16[];
    constexpr int NJ = NCT * 2;  // steps of 16 coefficients
    const uint32_t pay_cap = p.pay_words;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wavefront-uniform by construction
    const int half = lane >> 5, l32 = lane & 31;
    const int C = CFIX ? CFIX : p.C;
    static_assert(!(LOG && U8), "the 8-bit basis has one part");
    // The variants for many chunks (tens of MB of output and more) store the activations with the streaming hint:
    // written through the 256 MB memory-side cache, a large tensor leaves its write-back to whatever kernel runs
    // next.  (Measured on the 205 MB tensor: the decoder, which has memory bandwidth to spare, takes 7 us longer, and
    // the projection after it, which no longer shares the memory with that write-back, 14 us less.)
    constexpr bool kStreamOut = !U8 && (WAVES >= 12 || LOG);

    // the header, and the loads that do not depend on it, go out first: the code length table and the basis
    const Header hd = load_header(p);
    int my_len = 0;
    if (tid < 256 && p.bytes >= (size_t)(kHeaderBytes + kLenTableBytes)) my_len = p.stream[kHeaderBytes + tid];
    // the basis goes from global memory straight into LDS (no registers in between), 16 bytes per lane and
    // instruction: lane l of a wavefront lands at the wavefront's LDS base + 16 l
    constexpr int kBasisPieces = NCT * NJ * 2 * 64;  // 16-byte pieces of the basis, a multiple of 64
    if constexpr (U8) {
        // the 8-bit basis operand, [NCT][NS][64] entries of 8 bytes, goes into the same dynamic LDS
        const int n16 = NCT * ((C + 15) / 16) * 32;  // 16-byte pieces
        const uint4* src = reinterpret_cast<const uint4*>(p.op8);
        for (int i = tid; i < n16; i += THREADS) basis16[i] = src[i];
    }
    if constexpr (!U8 && !LOG) {
        const uint4* src = reinterpret_cast<const uint4*>(p.Bp16);
#pragma unroll
        for (int i = 0; i < (kBasisPieces + THREADS - 1) / THREADS; i++)
            if (THREADS * i + 64 * wave < kBasisPieces)  // whole wavefronts
                __builtin_amdgcn_global_load_lds(src + tid + THREADS * i, &basis16[THREADS * i + 64 * wave], 16, 0, 0);
    }
    if constexpr (LOG) {
        // block g = (channel tile, step) of the upper parts: 64 pieces at [g][0][64] of the operand, to [g][64] in LDS
        const uint4* src = reinterpret_cast<const uint4*>(p.Bp16);
        for (int g = wave; g < NCT * NJ; g += WAVES)
            __builtin_amdgcn_global_load_lds(src + (size_t)g * 128 + lane, &basis16[g * 64], 16, 0, 0);
        // ... and the lower parts of the first NLO channel tiles behind them
        for (int g = wave; g < NLO * NJ; g += WAVES)
            __builtin_amdgcn_global_load_lds(src + (size_t)g * 128 + 64 + lane, &basis16[(NCT * NJ + g) * 64], 16, 0, 0);
    }
    // The first chunk's offsets, run sizes and payload are requested before the header has arrived, at the places
    // the nominal chunk size puts them: three dependent memory round trips (header, offsets, payload) become
    // two that overlap with the table build.  The guess is checked against the header below; a stream made with
    // another chunk size loads them again.  Nothing outside [stream, stream + bytes) is touched either way.
    // (chunk c goes to workgroup c mod gridDim.x: a last, partly filled round of chunks is spread over all compute
    // units, one wavefront each, instead of filling a few of them)
    const uint32_t ch_first = (uint32_t)wave * gridDim.x + blockIdx.x;
    // this wavefront's LDS copy of a chunk's payload: pay_cap words and the overrun room
    uint32_t* pw = reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(basis16) + p.lds_basis_bytes) +
                   (size_t)wave * (pay_cap + (uint32_t)kPayOverrun);
    // Words [w0, w0 + n) of the payload go from global memory straight into that copy, 4 bytes per lane and
    // instruction, no registers in between; lanes past the chunk's end load nothing (what lies behind the chunk in
    // LDS is whatever was there: the decoder never takes a symbol of its run from it).  Asynchronous: wait_loads<0>()
    // before the copy is read.
    auto request_payload = [&](const uint32_t* payload, uint32_t w0, uint32_t n) {
        const uint32_t* src = payload + w0;
        for (uint32_t k = 0; 64u * k < n; k++) {  // wavefront-uniform trip count
            const uint32_t i = (uint32_t)lane + 64u * k;
            if (i < n) load_to_lds<4>(src + i, pw + 64u * k);
        }
    };
    const bool guess = p.g_off_payload <= p.bytes && ch_first < p.g_n_chunks && p.g_spc > 32u;  // (a chunk is a unit)
    UnitInfo cur{0u, 0u, 0u};
    bool pay_pre = false;
    if (guess) {
        const uint32_t* co = reinterpret_cast<const uint32_t*>(p.stream + p.g_off_chunk_off);
        const uint16_t* sb = reinterpret_cast<const uint16_t*>(p.stream + p.g_off_sub_bits);
        cur.off = co[ch_first];
        cur.end = co[ch_first + 1];
        cur.run = ((uint32_t)lane < p.g_spc) ? sb[(size_t)ch_first * p.g_spc + lane] : 0u;
        const size_t cap_words = (p.bytes - p.g_off_payload) / 4;
        const uint32_t gw0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)cur.off);
        const uint32_t gw1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)cur.end);
        pay_pre = gw0 <= gw1 && (size_t)gw1 <= cap_words && gw1 - gw0 <= pay_cap;
        if (pay_pre) request_payload(reinterpret_cast<const uint32_t*>(p.stream + p.g_off_payload), gw0, gw1 - gw0);
    }
    StreamView sv;
    if (!open_stream(p, hd, &sv)) {
        if (tid == 0 && blockIdx.x == 0) atomicOr(p.err, FMTC_ERR_HEADER);
        return;
    }
    const bool guess_valid = guess && sv.n_chunks == p.g_n_chunks && sv.spc == p.g_spc;  // same section offsets
    const uint32_t guess_w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)cur.off);
    const uint32_t guess_w1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)cur.end);
    const Unit un(sv, lane);
    if (blockIdx.x >= un.n_units) {  // (the grid is made for any chunk size)
        wait_loads<0>();  // (nothing is on its way into LDS any more)
        return;
    }
    auto chunks_of = [&](uint32_t u) { return sv.n_chunks - u * un.m < un.m ? sv.n_chunks - u * un.m : un.m; };
    if (!guess_valid && ch_first < un.n_units) cur.load(sv, un, ch_first * un.m, chunks_of(ch_first), lane);
    if constexpr (!U8) {
        if (tid < NCT * 32) s_mu[tid] = p.mu[tid];
    } else {
        if (tid < NCT * 32) {  // (both arrays are padded to NCT * 32 entries)
            s_col_sum[tid] = p.col_sum[tid];
            s_mean_d[tid] = p.mean_d[tid];
        }
    }
    if (!(p.prebuilt ? load_decode_tables<THREADS>(T, my_len, static_cast<const PrebuiltTables*>(p.prebuilt))
                     : build_decode_tables<THREADS>(T, my_len, p.bits))) {
        if (tid == 0 && blockIdx.x == 0) atomicOr(p.err, FMTC_ERR_TABLE);
        return;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wavefront's part of the basis has landed in LDS
    __syncthreads();
    const uint32_t payload_words = sv.payload_words;
    const uint32_t last_syms = (uint32_t)((uint64_t)p.P * (uint64_t)C - (uint64_t)(sv.n_chunks - 1u) * sv.chunk_syms);
    const float delta = sv.delta;
    // contraction steps that meet a non-zero row of the basis (all of them unless the basis is truncated)
    const int NJA = p.active_steps < 1 ? 1 : (p.active_steps > NJ ? NJ : p.active_steps);
    // 0x6400 | s is the f16 number 1024 + s: the level s - 2^(b-1) is that minus (1024 + 2^(b-1)), exactly
    const _Float16 level_off = (_Float16)(float)(1024 + (1 << (p.bits - 1)));
    const halfx2 level_off2 = {level_off, level_off};
    uint8_t* tile = symtile[wave];

    // Side information and payload of a unit are requested one unit ahead: its payload words right after the
    // variable length decoding of the unit before it (the LDS copy is free then; they arrive during the inverse
    // transform), offsets and run sizes of the unit after it once those words have landed (they arrive during the
    // variable length decoding) -- a unit would otherwise start with two dependent memory round trips.  cur:
    // what is at hand for the unit of this turn; pay_*: the offsets the words in the LDS copy were requested for.
    bool pay_ok = guess_valid && pay_pre;
    uint32_t pay_w0 = guess_w0, pay_w1 = guess_w1;
    const uint32_t u_step = gridDim.x * WAVES;
    // The wavefronts with a unit more than the others are the last to end: theirs go first.  (64 channels, 12544 chunks: 256 of
    // 4096 wavefronts have a fourth; they ended 9 us after the others, of 51.)
    if (ch_first < un.n_units % u_step && un.n_units > u_step) __builtin_amdgcn_s_setprio(2);
    for (uint32_t u = ch_first; u < un.n_units; u += u_step) {
        // ---- variable length decoding of the unit into the wavefront's tile ----
        const UnitBits ub = open_unit(sv, un, cur, u * un.m, chunks_of(u), last_syms, lane);
        if (ub.bad && lane == 0) atomicOr(p.err, FMTC_ERR_OFFSETS);
        const bool staged = ub.n_words <= pay_cap;
        // (whatever was requested for the LDS copy has landed before it is read or requested again; this also waits
        // for the stores of the unit before)
        wait_loads<0>();
        if (staged && !(pay_ok && ub.w0 == pay_w0 && ub.w0 + ub.n_words == pay_w1)) {
            request_payload(sv.payload, ub.w0, ub.n_words);
            wait_loads<0>();
        }
        const uint32_t nu = u + u_step;
        const bool have_next = nu < un.n_units && nu > u;  // wavefront-uniform
        if (have_next) cur.load(sv, un, nu * un.m, chunks_of(nu), lane);
        bool ok_run = true;
        if (staged) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // run `lane` goes to bytes [68 * lane, 68 * lane + 64) of the tile (sym_addr), 4 pad bytes behind it
            if (ub.cnt) ok_run = decode_run_bytes(pw, ub.n_words, ub.start + 32u * ub.rel, ub.cnt, T, tile + 68u * (uint32_t)lane);
        } else if (ub.cnt) {
            ok_run = decode_run(sv.payload + ub.w0 + ub.rel, ub.n_words - ub.rel, ub.start, ub.cnt, T, ByteOut(tile, 64u * (uint32_t)lane));
        }
        // the next unit's payload words: in flight during this unit's inverse transform (every lane is done with
        // the LDS copy: the reads of a wavefront complete in order, and each lane has used its last one)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        pay_ok = false;
        if (have_next) {
            pay_w0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)cur.off);
            pay_w1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)cur.end);
            pay_ok = pay_w0 <= pay_w1 && pay_w1 <= payload_words && pay_w1 - pay_w0 <= pay_cap;
            if (pay_ok) request_payload(sv.payload, pay_w0, pay_w1 - pay_w0);
        }
        if (!ok_run) atomicOr(p.err, FMTC_ERR_CODE);
        // the symbols of all lanes are in place before any lane reads them: one wavefront, LDS in order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();

        // ---- inverse quantizer + inverse transform of the unit's pixels ----
        const int64_t px_chunk0 = (int64_t)u * (int64_t)(un.m * (uint32_t)sv.ppc);
        const int TP = p.P - px_chunk0 < (int64_t)(un.m * (uint32_t)sv.ppc) ? (int)(p.P - px_chunk0) : (int)(un.m * (uint32_t)sv.ppc);
        for (int pt = 0; pt * 32 < TP; pt++) {
            int pxl = pt * 32 + l32;
            if (pxl > TP - 1) pxl = TP - 1;  // rows past the unit repeat its last pixel; never stored
            // (chunks of whole runs lie in the tile as one chunk would; others each start a slot of their own)
            const uint8_t* tile = symtile[wave];
            if ((CFIX == 0 || CFIX % 64 != 0) && un.m > 1u && (sv.chunk_syms & 63u)) {  // wavefront-uniform
                const uint32_t j = (uint32_t)pxl / (uint32_t)sv.ppc;
                tile += 68u * sv.spc * j;
                pxl -= (int)(j * (uint32_t)sv.ppc);
            }
            const uint32_t rowbase = (uint32_t)pxl * (uint32_t)C + 8u * (uint32_t)half;
            if constexpr (U8) {
                // Operands: lane (l32, half) holds the 8 symbols 16j + 8*half .. + 7 of its pixel as (s - 128),
                // and of the basis the same 8 coefficients of channel row perm(l32) of tile ct (rows permuted so
                // that a lane ends up with channels ct*32 + 16*half .. + 15 of its pixel).  Symbols past C meet
                // zero basis bytes.
                const int NS = (C + 15) / 16;  // <= NJ
                const unsigned long long* op8_lds = reinterpret_cast<const unsigned long long*>(basis16);
                const int hk = 1 << (p.bits - 1);
                long b[NJ];
#pragma unroll
                for (int j = 0; j < NJ; j++) {
                    const uint32_t n = rowbase + 16u * (uint32_t)j;
                    uint32_t w0 = 0, w1 = 0;
                    if (j < NS) read_octet<ALIGNED4>(tile, n, w0, w1);
                    b[j] = (long)((((unsigned long long)w1 << 32) | w0) ^ 0x8080808080808080ull);
                }
                const int my_px = pt * 32 + l32;
                const int64_t px = px_chunk0 + my_px;
#pragma unroll
                for (int ct = 0; ct < NCT; ct++) {
                    intx16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                    for (int j = 0; j < NJ; j++)
                        if (j < NS)
                            acc = __builtin_amdgcn_mfma_i32_32x32x16_i8((long)op8_lds[(ct * NS + j) * 64 + lane], b[j], acc, 0, 0, 0);
                    const int r0 = ct * 32 + 16 * half;
                    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                    for (int v = 0; v < 16; v++) {
                        const int r = r0 + v;  // < NCT * 32: the per-channel arrays are padded to that
                        const int m = acc[v] + (128 - hk) * s_col_sum[r];
                        const double t = fmin(fmax(rint(fma((double)m, p.factor8, s_mean_d[r])), 0.0), 255.0);
                        w[v >> 2] |= (uint32_t)(int)t << (8 * (v & 3));
                    }
                    if (my_px < TP && r0 < C) {
                        if constexpr (LAYOUT == FMTC_NHWC) {
                            uint8_t* q = p.out8 + (size_t)px * (size_t)C + (size_t)r0;
                            if ((C % 16) == 0) {
                                *reinterpret_cast<uint4*>(q) = make_uint4(w[0], w[1], w[2], w[3]);
                            } else {
#pragma unroll
                                for (int v = 0; v < 16; v++)
                                    if (r0 + v < C) q[v] = (uint8_t)(w[v >> 2] >> (8 * (v & 3)));
                            }
                        } else {
                            const int64_t n = px / p.HW, hw = px - n * p.HW;
#pragma unroll
                            for (int v = 0; v < 16; v++)
                                if (r0 + v < C)
                                    p.out8[((size_t)n * (size_t)C + (size_t)(r0 + v)) * (size_t)p.HW + (size_t)hw] =
                                        (uint8_t)(w[v >> 2] >> (8 * (v & 3)));
                        }
                    }
                    // (one channel tile at a time: interleaved by the compiler, the tiles' accumulators and plane addresses
                    // spill; 128 channels, N = 64, 28 x 28, 8 bits 53 -> 28 us)
                    if constexpr (LAYOUT == FMTC_NCHW) __builtin_amdgcn_sched_barrier(0);
                }
                continue;
            }
            // planar, built for one channel count: the image the chunk starts in, the bytes of a plane, and this lane's
            // pixel (and its half's four channels) as a 32-bit offset from channel 0 of that image
            const int my_pxl = pt * 32 + l32;
            uint32_t plane_bytes = 0, px_off = 0;
            char* plane0 = nullptr;
            if constexpr (LAYOUT == FMTC_NCHW && CFIX != 0 && !U8) {
                const uint32_t HW = (uint32_t)p.HW, px = (uint32_t)px_chunk0 + (uint32_t)my_pxl;
                const uint32_t n0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)px_chunk0 / HW));
                const uint32_t n = px / HW;
                plane_bytes = 4u * HW;
                px_off = 4u * ((n - n0) * (uint32_t)CFIX * HW + (px - n * HW) + 4u * (uint32_t)half * HW);
                plane0 = reinterpret_cast<char*>(p.xhat) + (uint64_t)n0 * (uint64_t)CFIX * plane_bytes;
            }
            // the levels of this lane's pixel as f16 operands, all contraction steps (coefficients past C meet zero
            // basis entries; whatever finite level the tile's bytes give there does not count)
            halfx8 q[NJ];
#pragma unroll
            for (int j = 0; j < NJ; j++) {
                const uint32_t n = rowbase + 16u * (uint32_t)j;
                uint32_t w0, w1;
                read_octet<ALIGNED4>(tile, n, w0, w1);
                const halfx2 q01 = __builtin_bit_cast(halfx2, __builtin_amdgcn_perm(0x64646464u, w0, 0x05010400u)) - level_off2;
                const halfx2 q23 = __builtin_bit_cast(halfx2, __builtin_amdgcn_perm(0x64646464u, w0, 0x07030602u)) - level_off2;
                const halfx2 q45 = __builtin_bit_cast(halfx2, __builtin_amdgcn_perm(0x64646464u, w1, 0x05010400u)) - level_off2;
                const halfx2 q67 = __builtin_bit_cast(halfx2, __builtin_amdgcn_perm(0x64646464u, w1, 0x07030602u)) - level_off2;
                q[j] = halfx8{q01[0], q01[1], q23[0], q23[1], q45[0], q45[1], q67[0], q67[1]};
            }
            // One channel tile at a time: one pair of accumulators, the contraction, the epilogue, the stores (all
            // tiles at once would hold 2 NCT accumulators: the registers of a third wavefront per SIMD).
            // LOG: the lower parts of the first NLO channel tiles sit in LDS behind the upper parts (as many as fit
            // beside the wavefronts' buffers), those of the others come from global memory.  The tiles with everything in
            // LDS go first, and the others' lower parts are requested before them: a round trip to the cache takes 1 to
            // 1.5 us under this kernel's load, a channel tile's arithmetic a third of that.  At most two wavefronts per
            // SIMD have the registers to request all of them at the top; three request one tile's, and the next tile's
            // when that one's matrix instructions have issued.
            constexpr int NG = LOG ? NCT - NLO : 0;
            constexpr bool kLoAll = LOG && WAVES <= 8 && NG <= 2;
            uint4 lo_g[kLoAll ? (NG > 0 ? NG : 1) : 1][LOG ? NJ : 1];
            auto request_lo = [&](int ct, uint4 (&dst)[LOG ? NJ : 1]) __attribute__((always_inline)) {
                if constexpr (LOG) {
                    const uint4* lo_src = reinterpret_cast<const uint4*>(p.Bp16) + ((size_t)(ct * NJ) * 2 + 1) * 64 + lane;
#pragma unroll
                    for (int j = 0; j < NJ; j++)
                        if (j < NJA) dst[j] = lo_src[(size_t)j * 128];
                }
            };
            if constexpr (LOG && NG > 0) {
                request_lo(NLO, lo_g[0]);
                if constexpr (kLoAll) {
#pragma unroll
                    for (int g = 1; g < NG; g++) request_lo(NLO + g, lo_g[g]);
                }
            }
#pragma unroll
            for (int ct = 0; ct < NCT; ct++) {
                floatx16 acc, acl;
#pragma unroll
                for (int r = 0; r < 16; r++) { acc[r] = 0.f; acl[r] = 0.f; }
                if constexpr (LOG) {
#pragma unroll
                    for (int j = 0; j < NJ; j++) {
                        if (j >= NJA) continue;  // wavefront-uniform (truncation, and padding rows of the last tile)
                        const halfx8 bh = __builtin_bit_cast(halfx8, basis16[(ct * NJ + j) * 64 + lane]);
                        if constexpr (LAYOUT == FMTC_NHWC) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(q[j], bh, acc, 0, 0, 0);
                        else acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(bh, q[j], acc, 0, 0, 0);
                    }
#pragma unroll
                    for (int j = 0; j < NJ; j++) {
                        if (j >= NJA) continue;
                        halfx8 bl;
                        if (ct < NLO) bl = __builtin_bit_cast(halfx8, basis16[((NCT + ct) * NJ + j) * 64 + lane]);
                        else bl = __builtin_bit_cast(halfx8, lo_g[kLoAll ? ct - NLO : 0][j]);
                        if constexpr (LAYOUT == FMTC_NHWC) acl = __builtin_amdgcn_mfma_f32_32x32x16_f16(q[j], bl, acl, 0, 0, 0);
                        else acl = __builtin_amdgcn_mfma_f32_32x32x16_f16(bl, q[j], acl, 0, 0, 0);
                    }
                    if constexpr (!kLoAll) {
                        if (ct >= NLO && ct + 1 < NCT) request_lo(ct + 1, lo_g[0]);
                    }
                } else {
#pragma unroll
                for (int j = 0; j < NJ; j++) {
                    if (j >= NJA) continue;  // wavefront-uniform: steps past the basis' last non-zero row (truncation)
                    const halfx8 bh = __builtin_bit_cast(halfx8, basis16[((ct * NJ + j) * 2) * 64 + lane]);
                    const halfx8 bl = __builtin_bit_cast(halfx8, basis16[((ct * NJ + j) * 2 + 1) * 64 + lane]);
                    if constexpr (LAYOUT == FMTC_NHWC) {
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(q[j], bh, acc, 0, 0, 0);
                        acl = __builtin_amdgcn_mfma_f32_32x32x16_f16(q[j], bl, acl, 0, 0, 0);
                    } else {
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(bh, q[j], acc, 0, 0, 0);
                        acl = __builtin_amdgcn_mfma_f32_32x32x16_f16(bl, q[j], acl, 0, 0, 0);
                    }
                }
                }
#pragma unroll
                for (int r = 0; r < 16; r++) acc[r] = __builtin_fmaf(acl[r], 1.f / 2048.f, acc[r]);
                // accumulator r of lane l is element (8*(r/4) + 4*(l/32) + r%4, l%32) of the 32x32 tile
                if constexpr (LAYOUT == FMTC_NHWC) {
                    const int c = ct * 32 + l32;
                    if (c < C) {
                        const float m_c = s_mu[c];
                        float* dst = p.xhat + (px_chunk0 + pt * 32 + 4 * half) * C + c;
                        if (pt * 32 + 32 <= TP && C == NCT * 32) {
                            // (the usual case, with the row stride a constant: the stores' offsets are immediates
                            // instead of sixteen 64-bit values in registers)
                            if constexpr (kStreamOut) {
#pragma unroll
                                for (int r = 0; r < 16; r++)
                                    __builtin_nontemporal_store(__builtin_fmaf(acc[r], delta, m_c),
                                                                &dst[(size_t)(8 * (r >> 2) + (r & 3)) * (NCT * 32)]);
                            } else {
#pragma unroll
                                for (int r = 0; r < 16; r++)
                                    dst[(size_t)(8 * (r >> 2) + (r & 3)) * (NCT * 32)] = __builtin_fmaf(acc[r], delta, m_c);
                            }
                        } else if (CFIX != 0 && CFIX != NCT * 32) {
                            // (a channel count known at build time that is no multiple of 32: the same, with the
                            // rows past the chunk's last pixel left out)
                            // (a whole chunk of such a tensor ends inside the last eight rows of the tile: the rows before
                            // them need no test -- wavefront-uniform -- and the stores go out in one run)
                            const bool first24 = pt * 32 + 24 <= TP;
#pragma unroll
                            for (int r = 0; r < 16; r++)
                                if ((r < 12 && first24) || pt * 32 + 8 * (r >> 2) + 4 * half + (r & 3) < TP) {
                                    float* at = &dst[(size_t)(8 * (r >> 2) + (r & 3)) * (CFIX ? CFIX : 1)];
                                    if constexpr (kStreamOut) __builtin_nontemporal_store(__builtin_fmaf(acc[r], delta, m_c), at);
                                    else *at = __builtin_fmaf(acc[r], delta, m_c);
                                }
                        } else if (pt * 32 + 32 <= TP) {
#pragma unroll
                            for (int r = 0; r < 16; r++)
                                dst[(size_t)(8 * (r >> 2) + (r & 3)) * C] = __builtin_fmaf(acc[r], delta, m_c);
                        } else {
#pragma unroll
                            for (int r = 0; r < 16; r++)
                                if (pt * 32 + 8 * (r >> 2) + 4 * half + (r & 3) < TP)
                                    dst[(size_t)(8 * (r >> 2) + (r & 3)) * C] = __builtin_fmaf(acc[r], delta, m_c);
                        }
                    }
                } else if constexpr (CFIX != 0) {
                    // A channel's plane starts at a wavefront-uniform address, the lane's place in it is a 32-bit offset
                    // (the launcher has checked that both fit): no 64-bit address per value and lane.
                    // (Without the streaming hint: a chunk's part of a plane mostly starts and ends inside a line, and
                    // the cache joins it with the neighbouring chunk's; with the hint 14 x 14 images of 128 channels
                    // take 94 us instead of 56, 55 x 55 of 64 channels 176 instead of 67, 28 x 28 of 128 44 instead of 49.)
                    const float* const mu_t = &s_mu[ct * 32 + 4 * half];
                    char* const plane = plane0 + (uint64_t)(ct * 32) * plane_bytes;
                    if (my_pxl < TP) {
#pragma unroll
                        for (int g = 0; g < 4; g++) {
                            if (ct * 32 + 8 * g >= CFIX) break;  // (known at build time: the last tile's padding)
                            const float4 m = *reinterpret_cast<const float4*>(mu_t + 8 * g);
                            const float mv[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
                            for (int e = 0; e < 4; e++)
                                *reinterpret_cast<float*>(plane + (uint64_t)(8 * g + e) * plane_bytes + px_off) =
                                    __builtin_fmaf(acc[4 * g + e], delta, mv[e]);
                        }
                    }
                } else {
                    const int my_px = pt * 32 + l32;
                    if (my_px < TP) {
                        const int64_t px = px_chunk0 + my_px;
                        const int64_t n = px / p.HW, hw = px - n * p.HW;
                        const int cb = ct * 32 + 4 * half;
                        float* dst = p.xhat + (n * (int64_t)C + cb) * p.HW + hw;
#pragma unroll
                        for (int r = 0; r < 16; r++) {
                            const int co = 8 * (r >> 2) + (r & 3);
                            if (cb + co < C) dst[(int64_t)co * p.HW] = __builtin_fmaf(acc[r], delta, s_mu[cb + co]);
                        }
                    }
                }
            }
        }
        // the next chunk of this wavefront overwrites the tile and pay[]: all lanes are done reading here
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

hipError_t launch_decode(const BasisDevice* b, const uint8_t* d_stream, size_t bytes, const Geometry& g, int bits,
                         int64_t HW, int layout, float* d_xhat, uint8_t* d_syms, uint32_t* d_err, const void* d_prebuilt,
                         hipStream_t s) {
    const int C = g.C;
    const int ncs = (C + 31) / 32;
    DecodeParams p{};
    p.stream = d_stream;
    p.bytes = bytes;
    p.P = g.P;
    p.HW = HW;
    p.C = C;
    p.bits = bits;
    p.ncs = ncs;
    p.Bp16 = b ? b->inv16 : nullptr;
    p.active_steps = b ? (b->active_rows + 15) / 16 : 0;
    p.mu = b ? b->mu : nullptr;
    p.xhat = d_xhat;
    p.syms_out = d_syms;
    p.err = d_err;
    p.prebuilt = d_prebuilt;
    p.g_off_chunk_off = g.off_chunk_off;
    p.g_off_sub_bits = g.off_sub_bits;
    p.g_off_payload = g.off_payload;
    p.g_n_chunks = g.n_chunks;
    p.g_spc = g.subs_per_chunk;
    const bool al = (C % 4) == 0;
    hipError_t el = hipSuccess;
    // (five channel tiles: channels-last only, the planar stores take more registers than are left)
    // Planar tensors of 32, 64, 128 and 144 channels have the variants built for one channel count too, whose stores take
    // 32-bit offsets: within the images that a chunk touches (an image and 4096 values) and of pixels.  (With the
    // channel count left open and with it fixed, us: 128 channels, N = 256, 28 x 28, 6 bits 66 and 49; 64 channels,
    // N = 256, 56 x 56 79 and 52; 144 channels, N = 64, 56 x 56, 5 bits, whose tiles of several chunks the kernel below
    // took, 125 and 61.)
    const bool planar32 = layout == FMTC_NCHW && (uint64_t)C * (uint64_t)HW + 4096u + 5u * (uint64_t)HW < (1ull << 30) &&
                          (uint64_t)g.P + 64u < (1ull << 31);
    const bool fixed_ok = layout == FMTC_NHWC || planar32;
    if (!d_syms && (ncs <= 4 || (ncs == 5 && (layout == FMTC_NHWC || (C == 144 && planar32 && g.n_chunks > 2048))))) {
        // ---- one wavefront per chunk ----
        const size_t lds_basis = sizeof(float) * (size_t)ncs * 32 * ncs * 32;
        // The LDS copy of a chunk's payload holds what a chunk takes at the fixed-length rate of `bits` per symbol
        // (which the code of the whole tensor never exceeds on average) and a little more; a chunk beyond that is
        // read in place.
        p.lds_basis_bytes = (uint32_t)lds_basis;
        p.pay_words = 128u * (uint32_t)bits + 64u;
        auto lds_dyn = [&](int wv) { return lds_basis + (size_t)wv * (p.pay_words + kPayOverrun) * 4; };
        auto lds_all = [&](int wv) { return lds_dyn(wv) + sizeof(DecTables) + (size_t)wv * kChunkTileBytes + (size_t)ncs * 128 + 64; };
        // Two or four wavefronts per SIMD: the variable length decoding is a chain of dependent LDS reads, and the other
        // wavefronts' work fills its waits; where there are fewer units than wavefronts they still build the tables in half
        // the time.  (Four wavefronts per workgroup up to 1024 chunks before, us: 64 channels, 3136 pixels, 8 bits 17.4 -> 15.8;
        // 128, 25088 pixels, 6 bits 19.7 -> 17.1; 100, 27621, 7 bits 26.7 -> 23.7; 30, 5000 14.0 -> 12.4.  Five channel tiles
        // need more LDS than two wavefronts per SIMD leave; four per SIMD fit up to two channel tiles.)
        int waves = ncs == 5 ? 4 : 8;
        if (g.n_chunks > 3072 && ncs <= 2 && C == ncs * 32 && fixed_ok && lds_all(16) <= 160 * 1024) waves = 16;
        // 128 to 160 channels: three wavefronts per SIMD with the lower parts of the basis left in global memory
        // (k_decode_chunks<..., LOG>); built for the channel counts 128 and 144, channels last (with a channel count
        // left open the kernel does not fit the registers of three wavefronts)
        // (144 channels: two wavefronts per SIMD, the registers of a third do not fit)
        // (the lower parts of the first `nlo` channel tiles go to LDS all the same if the bit depth's payload buffers
        // leave the room: 2 of 4 tiles at 128 channels, 3 of 5 at 144)
        const int log_waves = C == 128 ? 12 : 8;
        const int nlo_want = C == 128 ? 2 : 3;
        const size_t lo_tile = lds_basis / 2 / (size_t)ncs;  // bytes of one channel tile's lower parts
        auto lds_basis_for = [&](int nlo) { return lds_basis / 2 + (size_t)nlo * lo_tile; };
        const bool fits_lo = lds_all(log_waves) - lds_basis + lds_basis_for(nlo_want) <= 160 * 1024;
        const int nlo = fits_lo ? nlo_want : 0;
        const size_t lds_basis_log = lds_basis_for(nlo);
        const bool log12 = (C == 128 || C == 144) && fixed_ok && g.n_chunks > 2048 &&
                           lds_all(log_waves) - lds_basis + lds_basis_log <= 160 * 1024;
        if (log12) {
            waves = log_waves;
            p.lds_basis_bytes = (uint32_t)lds_basis_log;
        }
        const size_t lds = log12 ? lds_dyn(waves) - lds_basis + lds_basis_log : lds_dyn(waves);
        // A unit of chunks of another size than the nominal may hold half its symbols: workgroups for twice the chunks.  The
        // units are dealt to the workgroups first and to their wavefronts then, so a small tensor's have a compute unit
        // each; a workgroup without one ends when it has read the header.
        // (As many wavefronts as nominal chunks before: chunks of 2210 symbols, 24 channels, 6510 pixels 18.0 -> 11.2 us; of
        // 1024, 80 channels, 2187 pixels, planar 34 -> 21.)
        // (One workgroup per compute unit: the registers allow no second.)
        const unsigned gx = g.n_chunks < 128u ? 2u * g.n_chunks : 256u;
#define FMTC_DECC_L(NCT, LAY, AL, WV, CF, LG, NL)                                                                \
    do {                                                                                                         \
        if (lds > 16 * 1024) {                                                                                   \
            hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_decode_chunks<NCT, LAY, AL, WV, false, CF, LG, NL>), \
                                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);          \
            if (ea != hipSuccess) return ea;                                                                     \
        }                                                                                                        \
        el = launch(K_DECODE, k_decode_chunks<NCT, LAY, AL, WV, false, CF, LG, NL>, dim3(gx), dim3(WV * 64), lds, s, p); \
    } while (0)
#define FMTC_DECC_F(NCT, LAY, AL, WV, CF, LG) FMTC_DECC_L(NCT, LAY, AL, WV, CF, LG, 0)
#define FMTC_DECC(NCT, LAY, AL, WV) FMTC_DECC_F(NCT, LAY, AL, WV, 0, false)
#define FMTC_DECC_N(LAY, AL)                                                                                     \
    do {                                                                                                         \
        if (ncs == 1) FMTC_DECC(1, LAY, AL, 8);                                                                  \
        else if (ncs == 2) FMTC_DECC(2, LAY, AL, 8);                                                             \
        else if (ncs == 3) FMTC_DECC(3, LAY, AL, 8);                                                             \
        else FMTC_DECC(4, LAY, AL, 8);                                                                           \
    } while (0)
#define FMTC_DECC_FIXED(LAY)                                                                                     \
    do {                                                                                                         \
        if (waves == 16) { if (ncs == 1) FMTC_DECC_F(1, LAY, true, 16, 32, false); else FMTC_DECC_F(2, LAY, true, 16, 64, false); } \
        else if (C == 128) { if (nlo) FMTC_DECC_L(4, LAY, true, 12, 128, true, 2); else FMTC_DECC_L(4, LAY, true, 12, 128, true, 0); } \
        else { if (nlo) FMTC_DECC_L(5, LAY, true, 8, 144, true, 3); else FMTC_DECC_L(5, LAY, true, 8, 144, true, 0); } \
    } while (0)
        if (waves == 16 || log12) { if (layout == FMTC_NHWC) FMTC_DECC_FIXED(FMTC_NHWC); else FMTC_DECC_FIXED(FMTC_NCHW); }
        else if (ncs == 5 && layout != FMTC_NHWC) return hipErrorInvalidValue;  // (planar 144 without LDS room: no bit depth gets here)
        else if (ncs == 5) { if (al) FMTC_DECC(5, FMTC_NHWC, true, 4); else FMTC_DECC(5, FMTC_NHWC, false, 4); }
        else if (layout == FMTC_NHWC) { if (al) FMTC_DECC_N(FMTC_NHWC, true); else FMTC_DECC_N(FMTC_NHWC, false); }
        else                          { if (al) FMTC_DECC_N(FMTC_NCHW, true); else FMTC_DECC_N(FMTC_NCHW, false); }
#undef FMTC_DECC_FIXED
#undef FMTC_DECC_N
#undef FMTC_DECC
#undef FMTC_DECC_F
#undef FMTC_DECC_L
        return el;
    }

    // ---- tiles of several chunks per workgroup ----
    // the LDS copy of a unit's payload: see above
    p.pay_words = 128u * (uint32_t)bits + 64u;
    const uint32_t pay_bytes = 8u * 4u * (p.pay_words + (uint32_t)kPayOverrun);
    const uint32_t slot_bytes = d_syms ? 4352u : 68u * g.subs_per_chunk;  // of a chunk in the symbol tile
    const int max_chunks = (int)((159u * 1024u - sizeof(DecTables) - pay_bytes - 128u) / slot_bytes);
    // The tile: 32, 64 or 128 pixels (as many chunks as give them at the nominal chunk size), 32 of them with one, two or four
    // wavefronts per channel tile.  The channel groups (256 channels, fewer where wavefronts share a tile) of a tile go to
    // workgroups of their own (each decodes the tile's symbols again) while that still fills the device; otherwise a
    // workgroup walks them in turn.
    int mt = 0, ks = 0, G = 0, n_cg = 0;
    uint32_t n_tiles = 0;
    uint64_t blocks = 0;
    auto choose = [&](int m, int k) {
        mt = m;
        ks = k;
        G = (int)(32 * m / (int64_t)g.px_per_chunk);
        G = G < 1 ? 1 : (G > max_chunks ? max_chunks : G);
        if (d_syms) G = 8;  // symbols only: no projection to feed, one chunk per wavefront and as many workgroups as that gives
        n_tiles = (g.n_chunks + G - 1) / G;
        n_cg = (ncs * k + 7) / 8;
        return blocks = (uint64_t)n_tiles * (uint64_t)n_cg;
    };
    // The finest split whose workgroups run at the same time: one per compute unit (two of 32 pixels and one wavefront per
    // channel tile: 128 registers, and LDS for two at up to 512 channels).  Beyond that the largest tile, and from 513
    // channels, whose symbols take the LDS, the smallest.  Kernel times, us, for 1 x 4 : 1 x 2 : 1 x 1 : 2 x 1 : 4 x 1 (32-pixel
    // tiles x wavefronts per channel tile): 512 channels, 121 pixels 15 : 17 : 20 : 24 : 37; 1024, 968 35 : 24 : 30 : 50 : 50; 512,
    // 3146 35 : 22 : 21 : 25 : 38; 384, 5670 34 : 33 : 23 : 27 : 38; 304, 7220 34 : 35 : 34 : 36 : 31; 256, 50176 64 : 58 : 53 :
    // 56 : 45; 640, 11760 68 : 63 : 62 : 92 : 87; 960, 12544 158 : 156 : 101 : 150 : 132.
    if (d_syms) choose(1, 1);
    else if (choose(1, 4) > 256u && choose(1, 2) > 256u && choose(1, 1) > 256u) {
        // (up to 256 channels: 64 pixels while those workgroups have a compute unit each; 256, 9792 pixels 19.8 : 18.9)
        if (C > 256 || choose(2, 1) > 256u)
            if (choose(1, 1) > 512u && C <= 512) choose(4, 1);
    }
    // the grid is sized from the nominal geometry; the kernel takes the real one from the header
    int groups = 1;
    if (!d_syms) {
        groups = (int)(1024 / (n_tiles < 1024u ? n_tiles : 1024u));
        if (groups > n_cg) groups = n_cg;
        if (groups < 1) groups = 1;
        // (a test can make every workgroup walk all channel groups of its tile, as it does for tensors with more
        // tiles than the device holds)
        if (test_option(kTestDecodeOneRow)) groups = 1;
    }
    // More tiles than run at the same time are walked by the workgroups that do, which build their tables once (256
    // channels, 392 tiles 51 -> 45 us; 169, 470 tiles 49 -> 43).
    const uint32_t most = d_syms || blocks <= 512u ? 512u : 256u;
    // (Chunks of another size than the nominal may give a tile fewer pixels: workgroups for twice the tiles where they run at
    // the same time; one without a tile ends when it has read the header.)
    const uint32_t resident = 256u / (uint32_t)groups;
    uint32_t gx = 2u * n_tiles < resident ? 2u * n_tiles : resident;
    if (gx < n_tiles) gx = n_tiles < most ? n_tiles : most;
    dim3 grid((unsigned)groups, gx);  // (a tile's channel groups side by side, spread over the dies; workgroups without a tile last)
    p.g_tile_chunks = (uint32_t)G;
    // (chunks of another size than the nominal may take more room for the same pixels: their tiles get smaller)
    p.tile_px = 32 * mt;
    uint32_t tile_bytes = (uint32_t)G * slot_bytes;
    const uint32_t singly = 32u * (uint32_t)mt * 68u * (uint32_t)((C + kSubSyms - 1) / kSubSyms);  // every pixel a chunk of its own
    if (!d_syms && tile_bytes < singly && (mt == 1 || C <= 512)) tile_bytes = singly;
    p.tile_bytes = tile_bytes < 4352u ? 4352u : tile_bytes;  // (any chunk fits)
    p.lds_basis_bytes = ks > 1 && pay_bytes < 32u * 1024u ? 32u * 1024u : pay_bytes;
    const size_t lds = (size_t)p.lds_basis_bytes + p.tile_bytes + 128;
    // more than 64 KB of dynamic LDS has to be requested per kernel (the CU has 160 KB)
#define FMTC_DEC_L(MT, KS, LAY, AL)                                                                          \
    do {                                                                                                     \
        if (lds > 8 * 1024) {                                                                                \
            hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_decode_tiles<MT, KS, LAY, AL>), \
                                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);      \
            if (ea != hipSuccess) return ea;                                                                 \
        }                                                                                                    \
        el = launch(K_DECODE, k_decode_tiles<MT, KS, LAY, AL>, grid, dim3(512), lds, s, p);                  \
    } while (0)
#define FMTC_DEC(MT, KS)                                                                                     \
    do {                                                                                                     \
        if (layout == FMTC_NHWC) { if (al) FMTC_DEC_L(MT, KS, FMTC_NHWC, true); else FMTC_DEC_L(MT, KS, FMTC_NHWC, false); } \
        else                     { if (al) FMTC_DEC_L(MT, KS, FMTC_NCHW, true); else FMTC_DEC_L(MT, KS, FMTC_NCHW, false); } \
    } while (0)
    if (mt == 4) FMTC_DEC(4, 1);
    else if (mt == 2) FMTC_DEC(2, 1);
    else if (ks == 1) FMTC_DEC(1, 1);
    else if (ks == 2) FMTC_DEC(1, 2);
    else FMTC_DEC(1, 4);
#undef FMTC_DEC_L
#undef FMTC_DEC
    return el;
}

// Whole decoder of the 8-bit path in one kernel: the chunk decoder with the integer reconstruction in place of the
// f16 one.  *applies = false (and nothing launched) for tensors of more than 128 channels, which the caller then
// decodes to symbols and reconstructs with the tile kernel.
hipError_t launch_decode_u8(const Basis8Device& b, const uint8_t* d_stream, size_t bytes, const Geometry& g, int bits,
                            int64_t HW, int layout, double h, uint8_t* d_xq_hat, uint32_t* d_err, bool* applies,
                            hipStream_t s) {
    const int C = g.C;
    const int ncs = (C + 31) / 32;
    *applies = ncs <= 4;
    if (!*applies) return hipSuccess;
    if (!d_stream || !d_xq_hat || !d_err || !b.inv8 || !b.col_sum || !b.mean_d || b.C != C) return hipErrorInvalidValue;
    DecodeParams p{};
    p.stream = d_stream;
    p.bytes = bytes;
    p.P = g.P;
    p.HW = HW;
    p.C = C;
    p.bits = bits;
    p.ncs = ncs;
    p.Bp16 = nullptr;
    p.mu = nullptr;
    p.xhat = nullptr;
    p.syms_out = nullptr;
    p.err = d_err;
    p.prebuilt = nullptr;
    p.g_off_chunk_off = g.off_chunk_off;
    p.g_off_sub_bits = g.off_sub_bits;
    p.g_off_payload = g.off_payload;
    p.g_n_chunks = g.n_chunks;
    p.g_spc = g.subs_per_chunk;
    p.active_steps = ncs * 2;  // (not used by the 8-bit variant)
    p.op8 = b.inv8;
    p.col_sum = b.col_sum;
    p.mean_d = b.mean_d;
    p.factor8 = h;
    p.out8 = d_xq_hat;
    const bool al = (C % 4) == 0;
    const size_t lds_basis = (size_t)ncs * ((C + 15) / 16) * 64 * 8;  // the basis operand
    p.lds_basis_bytes = (uint32_t)lds_basis;
    p.pay_words = 128u * (uint32_t)bits + 64u;
    auto lds_dyn = [&](int wv) { return lds_basis + (size_t)wv * (p.pay_words + kPayOverrun) * 4; };
    // four wavefronts per SIMD under the conditions of the fp32 decoder (see launch_decode)
    const bool sixteen = g.n_chunks > 3072 && ncs <= 2 && C == ncs * 32 && layout == FMTC_NHWC &&
                         lds_dyn(16) + sizeof(DecTables) + 16 * (size_t)kChunkTileBytes + 64 <= 160 * 1024;
    const int waves = sixteen ? 16 : 8;
    const size_t lds = lds_dyn(waves);
    const unsigned gx = g.n_chunks < 128u ? 2u * g.n_chunks : 256u;  // see launch_decode
    hipError_t el = hipSuccess;
#define FMTC_DECU_F(NCT, LAY, AL, WV, CF) \
    do {                                                                                                         \
        hipError_t ea = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_decode_chunks<NCT, LAY, AL, WV, true, CF>), \
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);              \
        if (ea != hipSuccess) return ea;                                                                         \
        el = launch(K_DECODE, k_decode_chunks<NCT, LAY, AL, WV, true, CF>, dim3(gx), dim3(WV * 64), lds, s, p);  \
    } while (0)
#define FMTC_DECU(NCT, LAY, AL, WV) FMTC_DECU_F(NCT, LAY, AL, WV, 0)
#define FMTC_DECU_N(LAY, AL)                                                                                     \
    do {                                                                                                         \
        if (ncs == 1) FMTC_DECU(1, LAY, AL, 8);                                                                  \
        else if (ncs == 2) FMTC_DECU(2, LAY, AL, 8);                                                             \
        else if (ncs == 3) FMTC_DECU(3, LAY, AL, 8);                                                             \
        else FMTC_DECU(4, LAY, AL, 8);                                                                           \
    } while (0)
    if (sixteen) { if (ncs == 1) FMTC_DECU_F(1, FMTC_NHWC, true, 16, 32); else FMTC_DECU_F(2, FMTC_NHWC, true, 16, 64); }
    else if (layout == FMTC_NHWC) { if (al) FMTC_DECU_N(FMTC_NHWC, true); else FMTC_DECU_N(FMTC_NHWC, false); }
    else                     { if (al) FMTC_DECU_N(FMTC_NCHW, true); else FMTC_DECU_N(FMTC_NCHW, false); }
#undef FMTC_DECU_N
#undef FMTC_DECU
#undef FMTC_DECU_F
    return el;
}

}  // namespace fmtc
