// Variable length coder (paper section 3.1 "Variable length coding"; appendix
// "Huffman encoder as VLC"): Huffman code lengths from the symbol histogram,
// canonical code words, per-run bit counts, chunk offsets and the packed stream.
// All integer work; results are unique, so they are bit-exact by construction.
//
// Two kernels at most:
//   k_huffman_table  one workgroup: sums the partial histograms and builds the code
//                    (large tensors; small ones build it inside the pack kernel, every
//                    workgroup for itself, which saves a launch on the critical path);
//   k_pack           one wavefront per chunk: run sizes, the chunk's place in the payload
//                    (a running sum over the chunk groups handed from workgroup to
//                    workgroup), then the code bits;
//   k_pack_stream    the same for large tensors, a range of chunks per workgroup.
#include <atomic>
#include <type_traits>

#include "fmtc_device.h"
#include "fmtc_internal.h"
#include "fmtc_pack_device.h"
#include "fmtc_pack_ranges.h"

namespace fmtc {

constexpr uint32_t kInf = 0xffffffffu;

// ---------------------------------------------------------------------------
// Code table.  Lengths follow the classic construction: leaves ordered by
// (count, symbol), the two lightest nodes merged until one is left; a leaf wins
// over an internal node of equal weight, internal nodes leave in the order they
// were made.  Codes are canonical in (length, symbol) order.
// ---------------------------------------------------------------------------
struct TableLds {
    __attribute__((aligned(16))) uint32_t h[256];
    uint32_t weight[320];       // leaf weights in (count, symbol) order (64 spare entries: windows that reach past the end)
    uint32_t children[64];      // small alphabets, per merge: node ids of the two children (leaf i: i, internal j: 256 + j)
    uint16_t leaf_parent[256];  // merge that consumed each sorted leaf
    uint32_t node[256];         // internal nodes in creation order: parent | 1 << 16, then ancestor | distance << 16
    uint8_t len_sorted[256];    // code length of the sorted leaves
    uint32_t rank[320];         // position of every used symbol in (count, symbol) order; then the internal nodes' weights
};

// LDS traffic of one wavefront completes in order; this keeps the compiler from moving it across the point
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// More than 64 used symbols: the merges in rounds.  With t the sum of the two lightest nodes, every node of weight at
// most t is gone before any node made from now on (those weigh at least t, and leaves as well as older internal nodes
// win ties; the internal nodes at hand all weigh at most t), so these nodes, in (weight, leaf first, age) order, pair
// off all at once; the last one stays if their number is odd.  A round takes the first 62 of them, one per lane (a
// shorter run of that order is just as good).  Which places of the order internal nodes hold is a 64-bit mask in
// scalar registers: node k of the queue stands behind k others and the leaves not heavier than it.  A lane then finds
// its node by counting mask bits below it, and a pair's sum is its neighbour's weight away.
// 15 to 25 rounds for the 130 to 250 symbols of 7 and 8 bits, where one merge after the other in one lane took
// 0.11 us each: 168 symbols 19.4 -> 8 us, bound by one wavefront's issue and LDS latencies (11.2 us where the waiting
// internal nodes' places were found one node at a time, up to 30 of them a round).  (Up to
// 64 symbols the loop below stays: 70 ns a merge, and the small alphabets' steep counts need as many rounds.)
// Leaves parents in leaf_parent and node (see TableLds).  Internal node weights go where the ranks were (the caller
// holds those in registers by now).  One wavefront.
__device__ __forceinline__ void huffman_merge_rounds(TableLds& L, int lane, int n) {
    uint32_t* iw = L.rank;
    for (int i = lane; i < 320; i += 64) {
        iw[i] = kInf;
        if (i >= n) L.weight[i] = kInf;
    }
    wave_sync();
    int nl = 0, ni = 0, made = 0;
    while (made < n - 1) {  // a round makes at least one node
        const uint32_t lw = L.weight[nl + lane], iv = iw[ni + lane];  // (nl and ni at most 256: both arrays have 320 entries)
        // the two lightest nodes: two leaves, one of each, or two internal nodes
        auto add = [](uint32_t a, uint32_t b) { const uint32_t c = a + b; return c < a ? kInf : c; };
        const uint32_t l0 = (uint32_t)__builtin_amdgcn_readlane((int)lw, 0), l1 = (uint32_t)__builtin_amdgcn_readlane((int)lw, 1);
        const uint32_t i0 = (uint32_t)__builtin_amdgcn_readlane((int)iv, 0), i1 = (uint32_t)__builtin_amdgcn_readlane((int)iv, 1);
        const uint32_t s0 = add(l0, l1), s1 = add(l0, i0), s2 = add(i0, i1);
        const uint32_t t01 = s0 < s1 ? s0 : s1, t = t01 < s2 ? t01 : s2;
        const int wait = made - ni;
        // Places of internal nodes among the first 62 of the order (a place past them sets bit 63, which nobody looks at).
        unsigned long long places = 0;
        if (wait <= 4) {
            // their chains side by side; past the queue's end the weight is infinite, the place too
            int at[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)iv, u);
                at[u] = u + __popcll(__ballot(lw <= w));  // (leaves not heavier than an internal node: at most t)
            }
#pragma unroll
            for (int u = 0; u < 4; u++) places |= 1ull << (at[u] < 63 ? at[u] : 63);
        } else {
            // a node per lane: the block of eight leaves that its weight falls into, by the blocks' last leaves in scalar
            // registers, and its place in the block, by the others, fetched all at once
            uint32_t block = 0;
#pragma unroll
            for (int q = 0; q < 7; q++) block += (uint32_t)__builtin_amdgcn_readlane((int)lw, 8 * q + 7) <= iv ? 1u : 0u;
            uint32_t leaf[7];
#pragma unroll
            for (int q = 0; q < 7; q++) leaf[q] = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(32u * block + 4u * q), (int)lw);
            uint32_t at = (uint32_t)lane + 8u * block;
#pragma unroll
            for (int q = 0; q < 7; q++) at += leaf[q] <= iv ? 1u : 0u;
            at = lane < wait && at < 63u ? at : 63u;
            // (a lane that nobody writes to receives 0)
            places = __ballot(__builtin_amdgcn_ds_permute((int)(4u * at), at < 63u ? 1 : 0) != 0);
        }
        const int all = __popcll(__ballot(lw <= t && nl + lane < n)) + wait;
        const int count = all < 62 ? all & ~1 : 62;
        const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(places >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)places, 0u));
        const bool internal = (places >> lane) & 1ull;
        const uint32_t at = internal ? (uint32_t)ni + before : (uint32_t)(nl + lane) - before;
        const uint32_t up = (uint32_t)made + ((uint32_t)lane >> 1);
        if (lane < count) {
            const uint32_t w = (internal ? iw : L.weight)[at];
            if (internal) L.node[at] = up | (1u << 16);
            else L.leaf_parent[at] = (uint16_t)up;
            const uint32_t sum = w + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xf, 0xf, false);  // lane ^ 1
            if (!(lane & 1)) iw[up] = sum;
        }
        wave_sync();
        const int used = __popcll(places & ((1ull << count) - 1ull));
        ni += used;
        nl += count - used;
        made += count >> 1;
    }
}

// The same loop for at most 64 used symbols (one register per queue), written out by hand: the compiler's
// version moves the wavefront-uniform flags through vector registers, which puts several vector-to-scalar
// round trips into every step of a loop that is one long dependency chain.  Registers only; the trip count is
// n - 1.  Lane m of the result holds the number of leaves consumed before merge m, which fixes the two
// children of every merge: merges take the queues' heads, and 2m nodes are gone before merge m.
__device__ __forceinline__ void huffman_merge_small(TableLds& L, int lane, int n) {
    const uint32_t lw = (lane < n) ? L.weight[lane] : kInf;
    uint32_t iw = kInf, rec = 0;
    const uint32_t n1 = (uint32_t)__builtin_amdgcn_readfirstlane(n - 1);
    const uint32_t nn = (uint32_t)__builtin_amdgcn_readfirstlane(n);
    uint32_t nl, ni, made, t0, t1, l0, l1, i0, i1, x, y, wa, wb, k, w, m0save;
    asm volatile(
        "s_mov_b32 %[m0save], m0\n\t"
        "s_mov_b32 %[nl], 0\n\t"
        "s_mov_b32 %[ni], 0\n\t"
        "s_mov_b32 %[made], 0\n"
        "1:\n\t"
        "s_mov_b32 m0, %[made]\n\t"
        "s_add_u32 %[t0], %[nl], 1\n\t"
        "s_add_u32 %[t1], %[ni], 1\n\t"
        "v_readlane_b32 %[l0], %[lw], %[nl]\n\t"
        "v_readlane_b32 %[i0], %[iw], %[ni]\n\t"
        "v_readlane_b32 %[l1], %[lw], %[t0]\n\t"
        "v_readlane_b32 %[i1], %[iw], %[t1]\n\t"
        "s_nop 3\n\t"
        "s_cmp_lt_u32 %[nl], %[n]\n\t"           // a queue that has run out shows "infinity"
        "s_cselect_b32 %[l0], %[l0], -1\n\t"
        "s_cmp_lt_u32 %[t0], %[n]\n\t"
        "s_cselect_b32 %[l1], %[l1], -1\n\t"
        "s_cmp_le_u32 %[l0], %[i0]\n\t"          // first pick: a leaf wins a tie
        "s_cselect_b32 %[x], %[l1], %[l0]\n\t"   // heads after the first pick
        "s_cselect_b32 %[y], %[i0], %[i1]\n\t"
        "s_cselect_b32 %[wa], %[l0], %[i0]\n\t"
        "s_cselect_b32 %[k], 1, 0\n\t"
        "s_cmp_le_u32 %[x], %[y]\n\t"            // second pick
        "s_cselect_b32 %[wb], %[x], %[y]\n\t"
        "s_addc_u32 %[k], %[k], 0\n\t"           // leaves taken by this merge
        "v_writelane_b32 %[rec], %[nl], m0\n\t"
        "s_add_u32 %[w], %[wa], %[wb]\n\t"
        "s_sub_u32 %[t0], 2, %[k]\n\t"
        "v_writelane_b32 %[iw], %[w], m0\n\t"
        "s_add_u32 %[nl], %[nl], %[k]\n\t"
        "s_add_u32 %[ni], %[ni], %[t0]\n\t"
        "s_add_u32 %[made], %[made], 1\n\t"
        "s_cmp_lt_u32 %[made], %[n1]\n\t"
        "s_cbranch_scc1 1b\n\t"
        "s_mov_b32 m0, %[m0save]\n\t"
        : [rec] "+v"(rec), [iw] "+v"(iw), [nl] "=&s"(nl), [ni] "=&s"(ni), [made] "=&s"(made), [t0] "=&s"(t0),
          [t1] "=&s"(t1), [l0] "=&s"(l0), [l1] "=&s"(l1), [i0] "=&s"(i0), [i1] "=&s"(i1), [x] "=&s"(x),
          [y] "=&s"(y), [wa] "=&s"(wa), [wb] "=&s"(wb), [k] "=&s"(k), [w] "=&s"(w), [m0save] "=&s"(m0save)
        : [lw] "v"(lw), [n1] "s"(n1), [n] "s"(nn)
        : "scc");
    // children of merge m (lane m): leaves [nlb, nla), internal nodes [2m - nlb, 2(m+1) - nla)
    const uint32_t nlb = rec;
    uint32_t nla = __shfl_down(rec, 1, 64);
    if (lane >= n - 2) nla = (uint32_t)n;  // the last merge leaves no leaf behind
    const uint32_t kk = nla - nlb, nib = 2u * (uint32_t)lane - nlb;
    const uint32_t ida = kk >= 1 ? nlb : 256u + nib;
    const uint32_t idb = kk == 2 ? nlb + 1u : (kk == 1 ? 256u + nib : 256u + nib + 1u);
    L.children[lane] = ida | (idb << 16);
}

// Sum of the partial histograms into L.h.  All THREADS threads of the workgroup call it; ends with a barrier.
// Workgroups that do this side by side start at rows of their own (`who`): reading the same rows at the same time they
// would queue up at one part of the cache after the other.
template <int THREADS>
__device__ __forceinline__ void sum_partials(TableLds& L, const uint32_t* __restrict__ hist_parts, int n_parts,
                                             int bits, uint32_t who = 0u) {
    const int tid = threadIdx.x;
    const int K = 1 << bits;
    if (tid < 256) {
        L.h[tid] = 0u;
        L.rank[tid] = 0u;
    }
    __syncthreads();
    // a thread owns four neighbouring bins of every rstep-th row; sixteen independent 16-byte loads in flight
    const int tpr = K / 4, col = tid % tpr, row0 = tid / tpr, rstep = THREADS / tpr;
    const uint4* rows = reinterpret_cast<const uint4*>(hist_parts);
    const int turn_by = (int)((who * 37u) % (uint32_t)n_parts);
    auto row = [&](int q) { q += turn_by; return (size_t)(q < n_parts ? q : q - n_parts) * tpr + col; };
    uint4 acc = make_uint4(0, 0, 0, 0);
    int q = row0;
    for (; q + 15 * rstep < n_parts; q += 16 * rstep) {
        uint4 v[16];
#pragma unroll
        for (int j = 0; j < 16; j++) v[j] = rows[row(q + j * rstep)];
#pragma unroll
        for (int j = 0; j < 16; j++) {
            acc.x += v[j].x; acc.y += v[j].y; acc.z += v[j].z; acc.w += v[j].w;
        }
    }
    if (q < n_parts) {  // the rest, still all in flight together
        uint4 v[15];
#pragma unroll
        for (int j = 0; j < 15; j++)
            v[j] = (q + j * rstep < n_parts) ? rows[row(q + j * rstep)] : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < 15; j++) {
            acc.x += v[j].x; acc.y += v[j].y; acc.z += v[j].z; acc.w += v[j].w;
        }
    }
    if (acc.x) atomicAdd(&L.h[4 * col], acc.x);
    if (acc.y) atomicAdd(&L.h[4 * col + 1], acc.y);
    if (acc.z) atomicAdd(&L.h[4 * col + 2], acc.z);
    if (acc.w) atomicAdd(&L.h[4 * col + 3], acc.w);
    __syncthreads();
}

// Position of every used symbol in (count, symbol) order, into L.rank (zero on entry).  A wavefront takes one block of
// 64 symbols (a symbol per lane) and one slice of the symbols to compare against, read four at a time as broadcasts:
// symbols of a block before the lane's own count when they are not larger, of a block behind it when they are smaller,
// and only inside the own block does the order of the symbols need a test per comparison.  Unused symbols compare as
// the smallest of all and are taken off at the end.  256 symbols, 256 threads: 12.1 us with a test of everything in
// every comparison, 4.3 us this way (issue-bound: two instructions per comparison).
// All THREADS threads call it, after sum_partials; ends with a barrier.
template <int THREADS>
__device__ __forceinline__ void rank_symbols(TableLds& L, int bits) {
    constexpr int NW = THREADS / 64;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int K = 1 << bits;
    const int nb = (K + 63) >> 6, slices = NW / nb;  // (K at most 256, so at most as many blocks as wavefronts)
    const int blk = wave % nb, slice = wave / nb;
    const int s = 64 * blk + lane;
    const int quads = K / 4, per = (quads + slices - 1) / slices;
    const int q0 = slice * per, q1 = (q0 + per < quads) ? q0 + per : quads;
    const uint32_t cnt = s < K ? L.h[s] : 0u;
    const uint4* h4 = reinterpret_cast<const uint4*>(L.h);
    uint32_t r = 0;
    auto count = [&](int a, int b, auto less) {
#pragma unroll 8  // the reads of many steps in flight together: a step is one LDS round trip otherwise
        for (int q = a; q < b; q++) {
            const uint4 o = h4[q];
            r += (less(o.x, 4 * q) ? 1u : 0u) + (less(o.y, 4 * q + 1) ? 1u : 0u);
            r += (less(o.z, 4 * q + 2) ? 1u : 0u) + (less(o.w, 4 * q + 3) ? 1u : 0u);
        }
    };
    auto within = [&](int q) { return q < q0 ? q0 : (q > q1 ? q1 : q); };
    const int own0 = within(16 * blk), own1 = within(16 * blk + 16);
    count(q0, own0, [&](uint32_t o, int) { return o <= cnt; });
    count(own0, own1, [&](uint32_t o, int t) { return o < cnt || (o == cnt && t < s); });
    count(own1, q1, [&](uint32_t o, int) { return o < cnt; });
    if (slice == 0) {
        uint32_t unused = 0;
        for (int j = 0; j < nb; j++) unused += (uint32_t)__popcll(__ballot(64 * j + lane < K && L.h[64 * j + lane] == 0u));
        r -= unused;  // (the sum over the slices is what counts: it may pass through negative values)
    }
    if (r && cnt) atomicAdd(&L.rank[s], r);
    __syncthreads();
}

// What the table build leaves for its caller.
struct TableOut {
    unsigned long long* entry;  // [256] (LDS): bit-reversed code | length << 56
    uint32_t max_len;
    unsigned long long payload_bits;
};

// Canonical codes from code lengths (len[j] of symbol 64 j + lane, 0 = unused; max_len the longest, the same in
// every lane): codes of one length are numbered in symbol order, shorter codes first.  One wavefront; entry[] (256
// words, LDS or global) is written whole.
// scratch: 64 NVS words of LDS the wavefront may use (or NULL).
template <int NVS>
__device__ __forceinline__ void canonical_entries(const uint32_t (&len)[NVS], int lane, uint32_t max_len,
                                                  unsigned long long* entry_out, uint32_t* scratch = nullptr) {
    uint32_t before[NVS];
#pragma unroll
    for (int j = 0; j < NVS; j++) before[j] = 0;
    // lane q ends up with the number of codes of length q
    uint32_t my_count = 0;
    if (scratch) {
        // The lanes of equal length found with six ballots (one per bit of the length) instead of a loop over the
        // lengths; the first lane of every length leaves the group's size in the scratch row of its block of 64
        // symbols, and the rows before give the place of the block's codes among those of their length.
        // (Lengths are at most kMaxLen < 64.)
#pragma unroll
        for (int j = 0; j < NVS; j++) scratch[64 * j + lane] = 0u;
        wave_sync();
#pragma unroll
        for (int j = 0; j < NVS; j++) {
            unsigned long long same = ~0ull;
#pragma unroll
            for (int bit = 0; bit < 6; bit++) {
                const unsigned long long m = __ballot((len[j] >> bit) & 1u);
                same &= ((len[j] >> bit) & 1u) ? m : ~m;
            }
            before[j] = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
            if (len[j] && before[j] == 0) scratch[64 * j + (int)len[j]] = (uint32_t)__popcll(same);
        }
        wave_sync();
#pragma unroll
        for (int j = 0; j < NVS; j++) {
#pragma unroll
            for (int q = 0; q < j; q++) before[j] += scratch[64 * q + (int)len[j]];
            my_count += scratch[64 * j + lane];
        }
    } else {
        for (uint32_t q = 1; q <= max_len; q++) {
            uint32_t total = 0;
#pragma unroll
            for (int j = 0; j < NVS; j++) {
                const unsigned long long m = __ballot(len[j] == q);
                if (len[j] == q) before[j] = total + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                total += (uint32_t)__popcll(m);
            }
            if ((uint32_t)lane == q) my_count = total;
        }
    }
    // first canonical code of every length: code(l) = sum_{j<l} count(j) << (l-j), i.e. the running sum of
    // count(j) * 2^(48-j) shifted down to l bits
    const bool in = lane >= 1 && lane <= kMaxLen;
    const unsigned long long w = (unsigned long long)my_count << (in ? kMaxLen - lane : 0);
    const unsigned long long incl = wave_inclusive_scan64(w);
    const unsigned long long first_code = in ? ((incl - w) >> (kMaxLen - lane)) : 0ull;
#pragma unroll
    for (int j = 0; j < NVS; j++) {
        const unsigned long long fc = __shfl(first_code, (int)len[j], 64);
        unsigned long long entry = 0;
        if (len[j]) {
            const unsigned long long code = fc + (unsigned long long)before[j];
            const unsigned long long rev = __brevll(code) >> (64 - len[j]);  // stream order: least significant bit first
            entry = rev | ((unsigned long long)len[j] << 56);
        }
        entry_out[64 * j + lane] = entry;
    }
    if (NVS < 4)
        for (int s = 64 * NVS + lane; s < 256; s += 64) entry_out[s] = 0ull;
}

// Code table from the histogram L.h.  Runs in ONE wavefront (64 lanes, `lane`), no workgroup barrier inside;
// lane l owns symbols l, l + 64, ... (NVS = alphabet size / 64, at least 1).  Every lane returns the same
// max_len and payload_bits; entry[] is complete when the function returns (for this wavefront).
template <int NVS>
__device__ __forceinline__ void table_from_hist(TableLds& L, int lane, int K, TableOut& out) {
    uint32_t cnt[NVS], rank[NVS];
#pragma unroll
    for (int j = 0; j < NVS; j++) {
        cnt[j] = (64 * j + lane < K) ? L.h[64 * j + lane] : 0u;
        rank[j] = (64 * j + lane < K) ? L.rank[64 * j + lane] : 0u;  // made by rank_symbols
    }
    int n = 0;
#pragma unroll
    for (int j = 0; j < NVS; j++) {
        n += __popcll(__ballot(cnt[j] != 0));
        if (cnt[j]) L.weight[rank[j]] = cnt[j];
    }
    n = __builtin_amdgcn_readfirstlane(n);
    wave_sync();
    if (n >= 2) {
        const uint32_t root = (uint32_t)n - 2u;
        if (n <= 64) {
            huffman_merge_small(L, lane, n);
            wave_sync();
            if (lane < n - 1) {
                const uint32_t c = L.children[lane];
                const uint32_t a = c & 0xffffu, b = c >> 16, up = (uint32_t)lane | (1u << 16);
                if (a < 256u) L.leaf_parent[a] = (uint16_t)lane; else L.node[a - 256u] = up;
                if (b < 256u) L.leaf_parent[b] = (uint16_t)lane; else L.node[b - 256u] = up;
            }
        } else {
            huffman_merge_rounds(L, lane, n);
        }
        if (lane == 0) L.node[root] = root;
        wave_sync();
        // depth of every internal node: distance to an ancestor, doubled until that is the root for all of them
        {
            constexpr int NM = NVS == 1 ? 1 : 4;  // (an alphabet of up to 64 symbols makes up to 63 nodes)
            uint32_t v[NM];
#pragma unroll
            for (int j = 0; j < NM; j++) v[j] = 64 * j + lane < n - 1 ? L.node[64 * j + lane] : root;
            for (;;) {
                bool up = false;
#pragma unroll
                for (int j = 0; j < NM; j++) up |= (v[j] & 0xffffu) != root;
                if (!__any(up)) break;
                uint32_t w[NM];
#pragma unroll
                for (int j = 0; j < NM; j++) w[j] = L.node[v[j] & 0xffffu];
                wave_sync();
#pragma unroll
                for (int j = 0; j < NM; j++) {
                    v[j] = (v[j] & 0xffff0000u) + w[j];  // (distances add up, the ancestor's ancestor takes its place)
                    if (64 * j + lane < n - 1) L.node[64 * j + lane] = v[j];
                }
                wave_sync();
            }
        }
        for (int i = lane; i < n; i += 64) {
            uint32_t l = (L.node[L.leaf_parent[i]] >> 16) + 1u;
            // more than kMaxLen is unreachable for V < 2^32 (depth d needs a total count >= Fibonacci(d+2))
            L.len_sorted[i] = (uint8_t)(l > (uint32_t)kMaxLen ? (uint32_t)kMaxLen : l);
        }
    } else if (lane == 0) {
        L.len_sorted[0] = 1;  // a single used symbol gets the one-bit code 0
    }
    wave_sync();
    uint32_t len[NVS];
    uint32_t max_len = 0;
    unsigned long long pbits = 0;
#pragma unroll
    for (int j = 0; j < NVS; j++) {
        len[j] = cnt[j] ? (uint32_t)L.len_sorted[rank[j]] : 0u;
        max_len = len[j] > max_len ? len[j] : max_len;
        pbits += (unsigned long long)cnt[j] * len[j];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t t = __shfl_xor(max_len, o, 64);
        max_len = t > max_len ? t : max_len;
        pbits += __shfl_xor(pbits, o, 64);
    }
    max_len = (uint32_t)__builtin_amdgcn_readfirstlane((int)max_len);
    canonical_entries<NVS>(len, lane, max_len, out.entry, L.rank);  // (the ranks are in registers by now)
    out.max_len = max_len;
    out.payload_bits = pbits;
    wave_sync();
}

__device__ __forceinline__ void table_from_hist_any(TableLds& L, int lane, int bits, TableOut& out) {
    if (bits <= 6) table_from_hist<1>(L, lane, 1 << bits, out);
    else if (bits == 7) table_from_hist<2>(L, lane, 128, out);
    else table_from_hist<4>(L, lane, 256, out);
}

__global__ __launch_bounds__(1024) void k_huffman_table(const uint32_t* __restrict__ hist_parts, int n_parts,
                                                        int bits, uint32_t* __restrict__ hist_out,
                                                        uint64_t* __restrict__ enc_table,
                                                        uint8_t* __restrict__ len_table,
                                                        CoderCtrl* __restrict__ ctrl, uint32_t add_each) {
    __shared__ TableLds L;
    __shared__ unsigned long long entry[256];
    sum_partials<1024>(L, hist_parts, n_parts, bits);
    if (add_each) {  // a table for tensors to come: every symbol of the alphabet gets a code
        if ((int)threadIdx.x < (1 << bits)) L.h[threadIdx.x] += add_each;
        __syncthreads();
    }
    rank_symbols<1024>(L, bits);
    const int tid = threadIdx.x;
    if (tid < 64) {
        TableOut out;
        out.entry = entry;
        table_from_hist_any(L, tid, bits, out);
        if (tid == 0 && ctrl) {
            ctrl->max_len = out.max_len;
            ctrl->payload_bits = out.payload_bits;
        }
    }
    __syncthreads();
    if (tid < 256) {
        if (hist_out) hist_out[tid] = L.h[tid];
        if (enc_table) enc_table[tid] = entry[tid];
        if (len_table) len_table[tid] = (uint8_t)(entry[tid] >> 56);
    }
}

// Code table of given lengths (a complete prefix code over the 2^bits symbols; the host has checked that).
__global__ __launch_bounds__(64) void k_table_from_lengths(const uint8_t* __restrict__ len_table, int bits,
                                                           uint64_t* __restrict__ enc_table) {
    const int lane = threadIdx.x, K = 1 << bits;
    uint32_t len[4], max_len = 0;
#pragma unroll
    for (int j = 0; j < 4; j++) {
        len[j] = (64 * j + lane < K) ? (uint32_t)len_table[64 * j + lane] : 0u;
        max_len = len[j] > max_len ? len[j] : max_len;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t t = __shfl_xor(max_len, o, 64);
        max_len = t > max_len ? t : max_len;
    }
    max_len = (uint32_t)__builtin_amdgcn_readfirstlane((int)max_len);
    canonical_entries<4>(len, lane, max_len, reinterpret_cast<unsigned long long*>(enc_table));
}

hipError_t launch_table_from_lengths(const uint8_t* d_len_table, int bits, uint64_t* d_enc_table, hipStream_t s) {
    return launch(K_TABLE, k_table_from_lengths, dim3(1), dim3(64), 0, s, d_len_table, bits, d_enc_table);
}

// Table of the summed partial histograms with `add_each` added to every symbol's count.
hipError_t launch_table_from_hist(const uint32_t* d_hist_parts, int n_parts, int bits, uint32_t add_each,
                                  uint64_t* d_enc_table, uint8_t* d_len_table, hipStream_t s) {
    return launch(K_TABLE, k_huffman_table, dim3(1), dim3(1024), 0, s, d_hist_parts, n_parts, bits,
                  (uint32_t*)nullptr, d_enc_table, d_len_table, (CoderCtrl*)nullptr, add_each);
}

// Sum of the partial histograms only.
__global__ __launch_bounds__(256) void k_histogram_sum(const uint32_t* __restrict__ hist_parts, int n_parts,
                                                       int bits, uint32_t* __restrict__ hist_out) {
    const int K = 1 << bits, s = threadIdx.x;
    uint32_t acc = 0;
    if (s < K)
        for (int q = 0; q < n_parts; q++) acc += hist_parts[(size_t)q * K + s];
    hist_out[s] = acc;
}

hipError_t launch_histogram_sum(const uint32_t* d_hist_parts, int n_parts, int bits, uint32_t* d_hist,
                                hipStream_t s) {
    return launch(K_TABLE, k_histogram_sum, dim3(1), dim3(256), 0, s, d_hist_parts, n_parts, bits, d_hist);
}

// ---------------------------------------------------------------------------
// Packing kernel: the table (made here, by k_huffman_table, or given), then the chunk groups
// in turn (see fmtc_pack_device.h).
// ---------------------------------------------------------------------------
// kPackWaves chunks per group: one wavefront per chunk.
template <int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_pack(PackParams p) {
    static_assert(kPackWaves == 4, "one chunk per wavefront of the 256-thread workgroup");
    __shared__ PackShared S;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wavefront-uniform by construction
    const bool aligned4 = (p.chunk_syms & 3u) == 0;  // every chunk starts on a 4-byte boundary of the symbols

    // Which groups a workgroup packs.  A group's position in the payload comes from the groups before it, so
    // whoever waits for one must know that its owner gets to run.  This kernel is only launched with no more
    // groups than the device holds workgroups of it, and workgroup g takes group g: within a part of the chip
    // workgroups start in index order, so the lowest unfinished group is either running or next in line for a
    // place that only other kernels' workgroups (which finish) or this kernel's finished ones can hold.  Larger
    // tensors take the kernel below, whose workgroups claim their groups.
    uint32_t w[16];
    const uint32_t group = blockIdx.x;  // the grid never has more workgroups than groups
    load_chunk_symbols(p, group * kPackWaves + (uint32_t)wave, lane, aligned4, w);  // in flight while the table is made

    TableLds& L = *reinterpret_cast<TableLds*>(&S.stage[0][0]);  // shares LDS with the chunk images, not in use yet
    static_assert(sizeof(TableLds) <= sizeof(S.stage), "table scratch must fit the chunk images");
    if constexpr (MODE == kPackBuild) {
        sum_partials<256>(L, p.hist_parts, p.n_parts, p.bits);
        rank_symbols<256>(L, p.bits);
        if (wave == 0) {
            TableOut out;
            out.entry = S.tab;
            table_from_hist_any(L, lane, p.bits, out);
            if (lane == 0) {
                S.max_len = out.max_len;
                S.payload_bits = out.payload_bits;
            }
        }
        __syncthreads();
        if (blockIdx.x == 0) p.stream[kHeaderBytes + tid] = (uint8_t)(S.tab[tid] >> 56);  // the container's length table
    } else {
        S.tab[tid] = p.enc_table[tid];
        if (tid == 0) {
            // a static table does not know this tensor's bit count: it comes out of the look-back
            S.max_len = MODE == kPackStatic ? p.static_max_len : p.ctrl->max_len;
            S.payload_bits = MODE == kPackStatic ? 0ull : p.ctrl->payload_bits;
        }
        __syncthreads();
        if (MODE == kPackStatic && blockIdx.x == 0) p.stream[kHeaderBytes + tid] = (uint8_t)(S.tab[tid] >> 56);
    }
    // nobody reads the table scratch any more: the images start out clear
    pack_clear_image(S, wave, lane);
    pack_group<MODE>(S, p, group, w, chunk_len_of(p, group * kPackWaves + (uint32_t)wave), []() {});
}

// ---------------------------------------------------------------------------
// Large tensors (more chunk groups than the device holds pack workgroups): one pass over the symbols.
// One workgroup of 16 wavefronts per compute unit takes a range of neighbouring chunks, as many as its LDS holds packed
// images of: all its wavefronts pack, one publishes the range's size, adds up the sizes of the ranges before it, and all
// of them store.  A tensor with more chunks than that is packed in rounds, a range per workgroup and round, all ranges
// of one size, so that every workgroup has the same number of chunks.  Ranges are claimed from a counter, so those before
// a range have all been claimed by workgroups that run, and their sizes are published without waiting for any later one:
// whatever shares the device, the lowest range without a size can always go on.  The wait is bounded all the same and
// ends in an invalid stream.
// Every workgroup builds the code table for itself (the range's ticket and the first symbols arrive meanwhile).
// Chunks go to the wavefronts in a fixed order: dealt by a counter, the older wavefronts of a SIMD, which issue first, took
// four each and the others two, which then had nobody to share the SIMD with (12544 chunks of 4096 symbols at 6 bits, whole
// encoder 99.8 us, 97.9 this way).
// (Before: 15 chunks at a time, claimed in turn, packed by 15 wavefronts while the 16th saw to places that one wavefront of
// the device added up.  Of its 45 us for those chunks the packing took 8: the wavefronts spent 7 us waiting for their last
// places, some compute units having four turns and others three, 4.6 on dealing chunks that must not get stuck, 4 on what a
// turn leaves for its server.)
// What bounds it, at 33.8 us for those chunks: 13 us before the first one (partial counts 4.3, table 7.4, pair table 1), 16 of packing,
// two thirds of whose clocks issue vector instructions, 3 from the last size published to the places, 2 of stores.
// A lane takes eight neighbouring symbols per step, and up to 6 bits the table holds the joined code words of symbol
// pairs: four lookups, one prefix sum over the lanes and two or three ORs into the image per 512 symbols.
// ---------------------------------------------------------------------------
constexpr uint32_t kStreamWaves = 16;
constexpr uint32_t kStreamRoom = kStreamWaves * 2064;  // words for the images, each with 4 spare ones (see PackShared)
constexpr uint32_t kMaxImages = 64;     // an image per lane of the wavefront that adds up
constexpr uint32_t kShortCode = 26;     // a table entry holds up to 26 code bits below 6 bits of length ...
constexpr uint32_t kNoCode = 63u << kShortCode;  // ... or says that the code word is longer: any eight symbols with
                                        // such an entry come to more than 64 bits (less than eight: see octet_of)
// Marks a range's published size: its payload words; with a fixed table also its code bits, from bit 32 on.  (Added up in
// memory before the size was published, a round trip per turn: 25088 chunks of 1024 symbols 55.5 -> 43.5 us without, the
// N = 256, C = 64 tensor at 6 bits 47.4 -> 42.5.)
constexpr unsigned long long kKnown = 1ull << 62;

struct StreamShared {
    unsigned long long tab[256];                 // bit-reversed code | length << 56
    __align__(16) uint32_t image[kStreamRoom];
    uint16_t runs[kStreamWaves][64];
    uint32_t past[72];                           // what lies past the images' ends: a word and up to four behind it per lane
    // of the chunks of the range: payload words, code bits, where the second window starts (see pack_window)
    uint32_t words[kMaxImages], bits[kMaxImages], from[kMaxImages];
    uint32_t range, next_range;
    uint32_t images, image_words;
    uint32_t gone;                               // the wait ran out
    unsigned long long before;                   // payload words of the ranges before
    unsigned long long payload_bits;
};
// In front of it: code | length << 26 of symbol pairs, or of single ones.  (At the start of the LDS, where an entry's
// address needs no base.)
template <bool PAIRS>
constexpr uint32_t kStreamCodes = PAIRS ? 4096u : 256u;
// Eight symbols from any address (the compiler makes one 8-byte load of it: global memory takes them unaligned).
__device__ __forceinline__ uint2 load_octet(const uint8_t* at) {
    uint2 v;
    __builtin_memcpy(&v, at, 8);
    return v;
}
// The symbols of a chunk: register q of lane l holds symbols 512q + 8l .. + 7.  Past the chunk's end there is anything
// (octet_of takes none of it into account), so no load is masked: one address instruction each.  Nothing outside the tensor is read: where a piece would reach
// past its end, the tensor's last eight symbols are loaded (more than eight there are, in a tensor of this kernel), and
// align_last_octet shifts them into place.
// (Chunks that are no multiple of 8 symbols, fetched byte by byte and their last piece coded symbol by symbol: 8000 chunks
// of 4092 symbols 68.8 us for the kernel, 25.5 this way; 100000 chunks of 66 474.8 and 104.)
__device__ __forceinline__ void load_chunk_octets(const PackParams& p, uint32_t ch, int lane, uint2 (&w)[8]) {
    const uint32_t clen = chunk_len_of(p, ch);
    const uint64_t at = (uint64_t)ch * p.chunk_syms;
    const uint8_t* src = p.syms + at - 8;  // (the last chunk may have less than eight symbols)
    const uint64_t room = p.V - at;
    const uint32_t last = room < 4104u ? (uint32_t)room : 4104u;
#pragma unroll
    for (int q = 0; q < 8; q++) {
        const uint32_t o = 512u * q + 8u * (uint32_t)lane + 8u;
        if (512u * q < clen) w[q] = load_octet(src + (o < last ? o : last));  // wavefront-uniform
    }
}
// Octet `o` as loaded (at `last`, if that is before it).
__device__ __forceinline__ uint2 align_last_octet(uint2 v, int o, int last) {
    const uint32_t past = o > last && o - last < 8 ? (uint32_t)(o - last) : 0u;
    const unsigned long long e = (((unsigned long long)v.y << 32) | v.x) >> (8u * past);
    return make_uint2((uint32_t)e, (uint32_t)(e >> 32));
}
// ... all of a chunk's, before it is packed.
__device__ __forceinline__ void align_chunk_octets(const PackParams& p, uint32_t ch, int lane, uint2 (&w)[8]) {
    const uint32_t clen = chunk_len_of(p, ch);
    const uint64_t at = (uint64_t)ch * p.chunk_syms;
    if (at + ((clen + 7u) & ~7u) <= p.V) return;  // wavefront-uniform: all but the tensor's last chunk or two
    const int last = (int)((int64_t)(p.V - at) - 8);
#pragma unroll
    for (int q = 0; q < 8; q++) w[q] = align_last_octet(w[q], 512 * q + 8 * lane, last);
}

// How many images the room is divided into, and their words: as many as hold a chunk of the average size and a
// third more.  (A larger chunk is finished window by window from its symbols in memory.)
struct StreamImages {
    uint32_t count, words;
};
__device__ __forceinline__ StreamImages images_for(unsigned long long payload_bits, uint32_t n_chunks) {
    const unsigned long long need = payload_bits / 24u;  // words, and a third more
    if (need <= 512ull * n_chunks) return {64u, 512u};
    if (need <= 684ull * n_chunks) return {48u, 684u};
    return {32u, 1024u};
}
// The entropy of the symbol counts (`h`, 2^bits of them) and a little more, in bits, for images_for: the table's own bit
// count is known only when the first symbols should already be on their way.  The same in every workgroup, which all
// cut the tensor into the same ranges with it.  One wavefront.
__device__ __forceinline__ unsigned long long bits_from_counts(const uint32_t* h, int bits, uint64_t V, int lane) {
    const float log_v = __builtin_amdgcn_logf((float)V);
    float sum = 0.f;
    for (int s = lane; s < (1 << bits); s += 64) {
        const uint32_t n = h[s];
        const float l = log_v - __builtin_amdgcn_logf((float)(n ? n : 1u));  // (base 2)
        sum += (float)n * (l > 1.f ? l : 1.f);  // (a code word has a bit at least)
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    return (unsigned long long)(uint32_t)(sum * (1.f / 64.f)) * 66ull;
}

// ORs the up to 64 bits of `c` into the image at bit `pos` of the chunk (the last ones, if they start in its `words`, into its
// spare words).  What starts past them goes to a place of the lane's own that nobody reads, `past`: with one such word for
// all lanes the LDS took them one after the other, and where the chunks of a workgroup are larger than their images it
// served nothing else (see pack_window).
__device__ __forceinline__ void place_octet(unsigned long long c, uint32_t len, uint32_t pos, uint32_t* img, uint32_t words, uint32_t* past) {
    const uint32_t sh = pos & 31u;
    uint32_t* at = pos < words * 32u ? img + (pos >> 5) : past;
    const unsigned long long t0 = c << sh;
    atomicOr(at, (uint32_t)t0);
    atomicOr(at + 1, (uint32_t)(t0 >> 32));
    if (__any(len + sh > 64u)) atomicOr(at + 2, sh ? (uint32_t)((c >> 32) >> (32u - sh)) : 0u);
}

// The same for the usual step, without a test per lane.  Counted from the end of the word that the bits start in: k of them
// (0 to 31) go there, 32 into the next word, the rest behind that; with k the shift of all three pieces, none of them needs
// a case of its own for bits that start on a word (k = 0: nothing goes into the word before, which is there in any case).
// The rest is left to the caller (none where past is not positive).
// INSIDE: all lanes' bits start in the image.
struct Placed {
    uint32_t* next;
    uint32_t rest;
    int past;
};
template <bool INSIDE>
__device__ __forceinline__ Placed place_plain(unsigned long long c, uint32_t len, uint32_t pos, uint32_t* img, uint32_t words, uint32_t* past) {
    const uint32_t k = (0u - pos) & 31u;
    uint32_t* at = INSIDE || pos < words * 32u ? img + ((pos + 31u) >> 5) : past + 1;
    const uint32_t lo = (uint32_t)c, hi = (uint32_t)(c >> 32);
    atomicOr(at - 1, __builtin_amdgcn_alignbit(lo, 0u, k));
    atomicOr(at, __builtin_amdgcn_alignbit(hi, lo, k));
    return {at + 1, hi >> k, (int)(len - 32u - k)};
}

// A table entry of one symbol (see kShortCode).
__device__ __forceinline__ uint32_t short_entry(unsigned long long e) {
    const uint32_t len = (uint32_t)(e >> 56);
    return len <= kShortCode ? (uint32_t)e | (len << kShortCode) : kNoCode;
}

// Where the table of pairs keeps the entry of symbols s0, s1.  The LDS bank of a word is its index modulo 64: with the plain
// index s0 | s1 << 6 that is s0, the same few values for most lanes, whose pairs then wait for each other.
__device__ __forceinline__ uint32_t pair_slot(uint32_t s0, uint32_t s1) { return (s0 ^ s1) | (s1 << 6); }

// The code words of a lane's eight symbols, on their way into one value.
constexpr uint32_t kCodeBits = (1u << kShortCode) - 1u;
// N table entries joined, the first one lowest (at most 64 bits; of an entry without its code word: anything).
template <int N>
__device__ __forceinline__ unsigned long long join(const uint32_t* e) {
    unsigned long long c = e[N - 1] & kCodeBits;
#pragma unroll
    for (int i = N - 2; i >= 0; i--) c = (c << ((e[i] >> kShortCode) & 63u)) | (e[i] & kCodeBits);
    return c;
}
// The two halves of an octet.
struct Halves {
    unsigned long long lo, hi;
    uint32_t l_lo;  // bits of the first
};
// len: all its bits (more than 64 where an entry is without its code word).
// Of pairs the entries are kept, of which the usual octet, of up to 64 bits, is joined in one run; eight single ones would
// be the registers of the kernel's third and fourth wavefront.
template <bool PAIRS>
struct Octet;
template <>
struct Octet<true> {
    uint32_t e[4], len;
    __device__ __forceinline__ unsigned long long whole() const { return join<4>(e); }
    __device__ __forceinline__ Halves halves() const {
        Halves h;
        h.lo = join<2>(e);
        h.hi = join<2>(e + 2);
        h.l_lo = (e[0] >> kShortCode) + (e[1] >> kShortCode);
        if (len - (e[2] >> kShortCode) - (e[3] >> kShortCode) != h.l_lo) h.l_lo = 127u;  // (without a code word, at a chunk's end)
        return h;
    }
};
template <>
struct Octet<false> {
    Halves h;
    uint32_t len;
    __device__ __forceinline__ unsigned long long whole() const { return h.lo | (h.hi << (h.l_lo & 63u)); }  // (64 bits in `lo` leave none in `hi`)
    __device__ __forceinline__ Halves halves() const { return h; }
};

// Table entries of eight symbols, in stream order.
// PAIRS: the codes at the start of the LDS are the joined code words of symbol pairs (at pair_slot), else of single symbols.
template <bool PAIRS>
__device__ __forceinline__ void look_up(uint32_t x, uint32_t y, uint32_t (&e)[PAIRS ? 4 : 8]) {
    // (an entry's offset is its address)
    typedef const __attribute__((address_space(3))) uint32_t* lds_word;
    if constexpr (PAIRS) {
        // The byte address of a pair's entry is 4 (s0 ^ s1) | s1 << 8 (see pair_slot): with symbols of six bits the lower
        // byte is one of (x << 2) ^ (x >> 6), and one byte permute takes the two from their places.  (Six bits whatever
        // lies past a chunk's end.)
        const uint32_t x1 = x & 0x3f3f3f3fu, y1 = y & 0x3f3f3f3fu;
        const uint32_t x4 = (x1 << 2) ^ (x1 >> 6), y4 = (y1 << 2) ^ (y1 >> 6);
        e[0] = *(lds_word)__builtin_amdgcn_perm(x1, x4, 0x0c0c0500u);
        e[1] = *(lds_word)__builtin_amdgcn_perm(x1, x4, 0x0c0c0702u);
        e[2] = *(lds_word)__builtin_amdgcn_perm(y1, y4, 0x0c0c0500u);
        e[3] = *(lds_word)__builtin_amdgcn_perm(y1, y4, 0x0c0c0702u);
    } else {
        const uint32_t at[8] = {x << 2, x >> 6, x >> 14, x >> 22, y << 2, y >> 6, y >> 14, y >> 22};
#pragma unroll
        for (int i = 0; i < 8; i++) e[i] = *(lds_word)(at[i] & 0x3fcu);
    }
}
// ... made an octet.
// LAST: `left` is the number of the chunk's symbols from this lane's first one on (0 or less: none); those past the end
// count no bits.
template <bool PAIRS, bool LAST>
__device__ __forceinline__ Octet<PAIRS> octet_of(uint32_t (&e)[PAIRS ? 4 : 8], uint32_t x, uint32_t y, int left, const unsigned long long* tab) {
    Octet<PAIRS> o;
    o.len = 0u;
    bool none = false;
    if constexpr (PAIRS) {
        if constexpr (LAST) {
            // (a pair of which the chunk has only the first symbol: that one's own code word)
            auto first_only = [&](uint32_t v) { return short_entry(tab[v & 255u]); };
            if (__any(left > 0 && left < 8 && (left & 1))) {
                if (left == 1) e[0] = first_only(x);
                if (left == 3) e[1] = first_only(x >> 16);
                if (left == 5) e[2] = first_only(y);
                if (left == 7) e[3] = first_only(y >> 16);
            }
        }
#pragma unroll
        for (int i = 0; i < 4; i++) {
            if constexpr (LAST) {
                e[i] = left > 2 * i ? e[i] : 0u;
                none |= e[i] >= kNoCode;
            }
            o.e[i] = e[i];
            o.len += e[i] >> kShortCode;
        }
    } else {
        o.h.l_lo = 0u;
#pragma unroll
        for (int i = 0; i < 8; i++) {
            if constexpr (LAST) {
                e[i] = i < left ? e[i] : 0u;
                none |= e[i] >= kNoCode;
            }
            o.len += e[i] >> kShortCode;
            if (i == 3) o.h.l_lo = o.len;
        }
        o.h.lo = join<4>(e);
        o.h.hi = join<4>(e + 4);
        if constexpr (LAST)
            if (none) o.h.l_lo = 127u;
    }
    if constexpr (LAST)
        if (none) o.len = 127u;
    return o;
}

// An octet that 64 bits do not hold in at least one lane: its two halves as one 128-bit value, or (a code word that does
// not fit its entry, halves of more than 63 bits) every symbol by itself.
// octet_length: the lane's bits (`len` where no entry is without its code word), with the top bit set where it has to be
// symbol by symbol.
__device__ __forceinline__ uint32_t octet_length(uint32_t x, uint32_t y, uint32_t first, uint32_t l_lo, uint32_t len,
                                                 uint32_t clen, const unsigned long long* tab) {
    // (an entry without its code word says 63 bits, and any other symbol at least one; at the end of a chunk see octet_of)
    if (!__any(l_lo > 63u || len - l_lo > 63u)) return len;
    uint32_t n = 0u;
#pragma unroll 1
    for (uint32_t i = 0; i < 8u; i++) {
        const uint32_t sym = ((i < 4u ? x : y) >> (8u * (i & 3u))) & 255u;
        n += first + i < clen ? (uint32_t)(tab[sym] >> 56) : 0u;
    }
    return n | 0x80000000u;
}
__device__ __forceinline__ void place_long_octet(uint32_t x, uint32_t y, uint32_t first, unsigned long long lo,
                                                 unsigned long long hi, uint32_t l_lo, uint32_t len, bool single,
                                                 uint32_t clen, const unsigned long long* tab, uint32_t pos,
                                                 uint32_t* img, uint32_t words, uint32_t* past) {
    if (!single) {
        // (both halves as one value of up to 126 bits: the leading components of a pixel need 9 to 11 bits a symbol at 8 bits,
        // so most steps of such a tensor come here: the halves one after the other took 67 % more of the kernel's time at
        // chunks of 256 symbols, 301.8 us for 138660 of them, 204.7 this way)
        const uint32_t sh = pos & 31u, reach = len + sh;
        uint32_t* at = pos < words * 32u ? img + (pos >> 5) : past;
        const unsigned long long c0 = lo | (hi << l_lo), c1 = l_lo ? hi >> (64u - l_lo) : 0ull;
        const unsigned long long t0 = c0 << sh, t1 = (c1 << sh) | (sh ? c0 >> (64u - sh) : 0ull);
        atomicOr(at, (uint32_t)t0);
        atomicOr(at + 1, (uint32_t)(t0 >> 32));
        if (__any(reach > 64u)) atomicOr(at + 2, (uint32_t)t1);
        if (__any(reach > 96u)) {  // (behind the image's end there are four spare words)
            atomicOr(at + 3, (uint32_t)(t1 >> 32));
            atomicOr(at + 4, sh ? (uint32_t)(c1 >> (64u - sh)) : 0u);
        }
        return;
    }
#pragma unroll 1
    for (uint32_t i = 0; i < 8u; i++) {
        const uint32_t sym = ((i < 4u ? x : y) >> (8u * (i & 3u))) & 255u;
        const unsigned long long e = first + i < clen ? tab[sym] : 0ull;
        place_octet(e & 0x00ffffffffffffffull, (uint32_t)(e >> 56), pos, img, words, past);
        pos += (uint32_t)(e >> 56);
    }
}

// One chunk (`clen` symbols in w, see load_chunk_octets) into the first `words` words of its image.  Returns the chunk's
// code bits and leaves the bit counts of its runs of 64 symbols (eight lanes; 64 of them, zeros past the end) in run_bits.
// last_from: the last step that starts inside the image (see pack_window).
// Two octets per lane and turn, 512 symbols apart: their chains run side by side, and one prefix sum over the lanes
// serves both (16 bits each: a chunk has at most 64 x 8 x 48 bits in 512 symbols).
template <bool PAIRS>
__device__ __forceinline__ uint32_t pack_octets(const uint2 (&w)[8], uint32_t clen, const unsigned long long* tab,
                                                uint32_t* img, uint32_t words, uint32_t* past, int lane, uint16_t* run_bits, uint32_t& last_from) {
    uint32_t base = 0;
    auto step = [&](uint32_t q, uint32_t x0, uint32_t y0, uint32_t x1, uint32_t y1, auto some_c) __attribute__((always_inline)) -> uint32_t {
        constexpr bool some = decltype(some_c)::value;
        const uint32_t f0 = 512u * q + 8u * (uint32_t)lane, f1 = f0 + 512u;
        last_from = base < words * 32u ? (512u * q) | (base << 12) : last_from;
        // (Wavefront-uniform.  Chunks of up to 512 symbols are one such octet per lane; with an empty second one 138660
        // chunks of 256 symbols took 266.7 us at 6 bits, 207.7 without, 249 in three kernels.)
        const bool two = !some || 512u * q + 512u < clen;
        uint32_t ea[PAIRS ? 4 : 8], eb[PAIRS ? 4 : 8];
        look_up<PAIRS>(x0, y0, ea);
        if (two) look_up<PAIRS>(x1, y1, eb);
        if constexpr (!some) __builtin_amdgcn_sched_barrier(0);  // (all of them on their way before the first is waited for)
        const Octet<PAIRS> a = octet_of<PAIRS, some>(ea, x0, y0, (int)(clen - f0), tab);
        Octet<PAIRS> b{};
        if (two) b = octet_of<PAIRS, some>(eb, x1, y1, (int)(clen - f1), tab);
        // inclusive prefix sum over the lanes (see wave_inclusive_scan_rows; lanes 7 and 15 of a row of 16 hold
        // their eight lanes' sum after three steps: a run of 64 symbols)
        uint32_t run = 0u, pos_a = 0u, pos_b = 0u;
        auto add_up = [&](uint32_t len_a, uint32_t len_b) __attribute__((always_inline)) {
            uint32_t v = len_a | (len_b << 16);
            v = dpp_add<0x111, 0xf>(v);
            v = dpp_add<0x112, 0xf>(v);
            v = dpp_add<0x114, 0xf>(v);
            run = v;
            v = dpp_add<0x118, 0xf>(v);
            v = dpp_add<0x142, 0xa>(v);
            v = dpp_add<0x143, 0xc>(v);
            const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
            pos_a = base + (v & 0xffffu) - len_a;
            pos_b = base + (total & 0xffffu) + (v >> 16) - len_b;
            base += (total & 0xffffu) + (total >> 16);
        };
        const uint32_t longer = a.len > b.len ? a.len : b.len;
        if (__builtin_expect(!__any(longer > 64u), 1)) {
            // (one straight run: what is joined fills the waits of the prefix sum)
            add_up(a.len, b.len);
            auto place = [&](auto inside_c) __attribute__((always_inline)) {
                constexpr bool inside = decltype(inside_c)::value;
                const Placed at_a = place_plain<inside>(a.whole(), a.len, pos_a, img, words, past);
                Placed at_b{at_a.next, 0u, 0};
                if (two) at_b = place_plain<inside>(b.whole(), b.len, pos_b, img, words, past);
                if (__any((int)(at_a.past > at_b.past ? at_a.past : at_b.past) > 0)) {
                    atomicOr(at_a.next, at_a.rest);
                    atomicOr(at_b.next, at_b.rest);
                }
            };
            if (__builtin_expect(base <= words * 32u, 1)) place(std::true_type{});
            else place(std::false_type{});
        } else {
            const Halves ha = a.halves(), hb = b.halves();
            uint32_t len_a = octet_length(x0, y0, f0, ha.l_lo, a.len, clen, tab);
            uint32_t len_b = octet_length(x1, y1, f1, hb.l_lo, b.len, clen, tab);
            const bool single_a = __any(len_a >> 31) != 0, single_b = __any(len_b >> 31) != 0;
            len_a &= 0x7fffffffu;
            len_b &= 0x7fffffffu;
            add_up(len_a, len_b);
            place_long_octet(x0, y0, f0, ha.lo, ha.hi, ha.l_lo, len_a, single_a, clen, tab, pos_a, img, words, past);
            if (two) place_long_octet(x1, y1, f1, hb.lo, hb.hi, hb.l_lo, len_b, single_b, clen, tab, pos_b, img, words, past);
        }
        return run;
    };
    const uint32_t n_whole = clen >> 10;
    uint32_t run[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int q = 0; q < 4; q++)
        if ((uint32_t)q < n_whole)  // wavefront-uniform
            run[q] = step(2u * q, w[2 * q].x, w[2 * q].y, w[2 * q + 1].x, w[2 * q + 1].y, std::false_type{});
    if (clen & 1023u) {
        uint32_t x0 = w[0].x, y0 = w[0].y, x1 = w[1].x, y1 = w[1].y;
#pragma unroll
        for (int q = 1; q < 4; q++) {
            x0 = (uint32_t)q == n_whole ? w[2 * q].x : x0;
            y0 = (uint32_t)q == n_whole ? w[2 * q].y : y0;
            x1 = (uint32_t)q == n_whole ? w[2 * q + 1].x : x1;
            y1 = (uint32_t)q == n_whole ? w[2 * q + 1].y : y1;
        }
        const uint32_t last = step(2u * n_whole, x0, y0, x1, y1, std::true_type{});
#pragma unroll
        for (int q = 0; q < 4; q++)
            if ((uint32_t)q == n_whole) run[q] = last;
    }
    if ((lane & 7) == 7) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            run_bits[16 * q + (lane >> 3)] = (uint16_t)run[q];
            run_bits[16 * q + 8 + (lane >> 3)] = (uint16_t)(run[q] >> 16);
        }
    }
    return base;
}

// A later window [win, win + words) of a chunk too large for its image, once more from the symbols in memory: an octet per
// lane and step, the next step's symbols on their way meanwhile, from the step in which the window starts (from: its first
// symbol | code bits before it << 12; afterwards the next window's) to the one that ends behind it.  Words outside the
// window go to `past`.  (Chunks of flat and of busy regions differ several times in size, so a tensor
// can have many such chunks, and side by side in one workgroup.  12544 chunks of 4096 symbols at 6 bits, a tenth of them
// large, us: every tenth 39, the first tenth 57; with one word for all that lies outside, which all wavefronts of such a
// workgroup then wait for, 45 and 137.)
template <bool PAIRS>
__device__ __forceinline__ void pack_window(const PackParams& p, uint32_t ch, const unsigned long long* tab,
                                            uint32_t* img, uint32_t words, uint32_t* past, uint32_t win, int lane, uint32_t& from) {
    const uint32_t clen = chunk_len_of(p, ch);
    const uint64_t at = (uint64_t)ch * p.chunk_syms;
    const uint8_t* src = p.syms + at;
    const int64_t room = (int64_t)(p.V - at) - 8;
    const int last = room < 4096 ? (int)room : 4096;
    auto load = [&](uint32_t o) {  // (see load_chunk_octets)
        return o < clen ? load_octet(src + ((int)o < last ? (int)o : last)) : make_uint2(0u, 0u);
    };
    auto put = [&](unsigned long long c, uint32_t pos) {
        const uint32_t sh = pos & 31u, rel = (pos >> 5) - win;
        const unsigned long long t0 = c << sh;
        // (each word by itself: the first may lie before the window and the next ones inside)
        atomicOr(rel < words ? img + rel : past, (uint32_t)t0);
        atomicOr(rel + 1u < words ? img + (rel + 1u) : past, (uint32_t)(t0 >> 32));
        atomicOr(rel + 2u < words ? img + (rel + 2u) : past, sh ? (uint32_t)((c >> 32) >> (32u - sh)) : 0u);
    };
    const uint32_t end = 32u * (win + words);
    uint32_t base = from >> 12, s0 = from & 0xfffu;
    uint2 next = load(s0 + 8u * (uint32_t)lane);
#pragma unroll 1
    for (; s0 < clen && base < end; s0 += 512u) {
        from = s0 | (base << 12);
        const uint32_t first = s0 + 8u * (uint32_t)lane;
        const uint2 xy = align_last_octet(next, (int)first, last);
        const uint32_t x = xy.x, y = xy.y;
        next = load(first + 512u);
        uint32_t e[PAIRS ? 4 : 8];
        look_up<PAIRS>(x, y, e);
        const Octet<PAIRS> o = octet_of<PAIRS, true>(e, x, y, (int)(clen - first), tab);
        const bool plain = !__any(o.len > 64u);
        uint32_t len = o.len;
        Halves h{};
        if (__builtin_expect(!plain, 0)) {
            h = o.halves();
            len = octet_length(x, y, first, h.l_lo, o.len, clen, tab);
        }
        const bool single = __any(len >> 31) != 0;
        len &= 0x7fffffffu;
        uint32_t row, half;
        const uint32_t incl = wave_inclusive_scan_rows(len, row, half);
        uint32_t pos = base + incl - len;
        base += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        if (__builtin_expect(plain, 1)) {
            put(o.whole(), pos);
        } else if (!single) {
            put(h.lo, pos);
            put(h.hi, pos + h.l_lo);
        } else {
#pragma unroll 1
            for (uint32_t i = 0; i < 8u; i++) {
                const uint32_t sym = ((i < 4u ? x : y) >> (8u * (i & 3u))) & 255u;
                const unsigned long long e = first + i < clen ? tab[sym] : 0ull;
                put(e & 0x00ffffffffffffffull, pos);
                pos += (uint32_t)(e >> 56);
            }
        }
    }
}

// STATIC: the table is a fixed one, and the code bits of the tensor are added up on the way; otherwise every workgroup
// builds the table from the partial histograms.
template <bool STATIC, bool PAIRS>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_pack_stream(PackParams p) {
    extern __shared__ __align__(16) uint8_t dyn_lds[];
    uint32_t* const codes = reinterpret_cast<uint32_t*>(dyn_lds);
    StreamShared& S = *reinterpret_cast<StreamShared*>(dyn_lds + 4u * kStreamCodes<PAIRS>);
    const int tid = threadIdx.x, lane = tid & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr uint32_t kLast = kStreamWaves - 1u;  // the wavefront that draws the tickets
    auto claim = [&]() -> uint32_t {
        return __hip_atomic_fetch_add(&p.ctrl->ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto sync_wave = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    uint32_t ticket = 0;  // (on its way while the counts are added up)
    if (wave == kLast && lane == 0) ticket = claim();
    TableLds& L = *reinterpret_cast<TableLds*>(&S.image[0]);  // shares LDS with the first images
    static_assert(sizeof(TableLds) <= 4u * kStreamRoom / kStreamWaves && kStreamRoom / kStreamWaves / 4u <= 1024u, "table scratch must fit the first wavefront's part of the images");
    if constexpr (!STATIC) {
        sum_partials<1024>(L, p.hist_parts, p.n_parts, p.bits, blockIdx.x);
        if (wave == kLast && lane == 0) S.range = ticket;  // (a barrier follows)
        rank_symbols<1024>(L, p.bits);
    } else {
        if (tid < 256) S.tab[tid] = p.enc_table[tid];
        if (wave == kLast && lane == 0) S.range = ticket;
        __syncthreads();
    }
    // While the first wavefront builds the table, the others clear the images and request their first symbols.
    uint32_t images = 0, words = 0, c0 = 0, count = 0;
    Ranges ranges{0u, 0u};
    auto take_range = [&](uint32_t range) {
        const ChunkSpan span = range_chunks(ranges, range, p.n_chunks);
        c0 = span.first;
        count = span.count;
    };
    uint2 w[8];
    if (STATIC || wave != 0u) {
        // (a fixed table says nothing of the tensor: room for 6 bits a symbol)
        const StreamImages im = images_for(STATIC ? 6ull * p.V : bits_from_counts(L.h, p.bits, p.V, lane), p.n_chunks);
        images = (uint32_t)__builtin_amdgcn_readfirstlane((int)im.count);
        words = (uint32_t)__builtin_amdgcn_readfirstlane((int)im.words);
        if (tid == 64 * (int)kLast) {
            S.images = images;
            S.image_words = words;
            S.gone = 0u;
        }
        ranges = cut_ranges(p.n_chunks, gridDim.x, images);
        take_range((uint32_t)__builtin_amdgcn_readfirstlane((int)S.range));
        if (wave < count) load_chunk_octets(p, c0 + wave, lane, w);
    } else {
        TableOut out;
        out.entry = S.tab;
        table_from_hist_any(L, lane, p.bits, out);
        if (lane == 0) S.payload_bits = out.payload_bits;
    }
    constexpr uint32_t kPart = kStreamRoom / kStreamWaves;
    if (wave != 0u)  // (the first wavefront's part holds the counts and the table's scratch)
        for (uint32_t i = wave * kPart + 4u * (uint32_t)lane; i < (wave + 1u) * kPart; i += 256u)
            *reinterpret_cast<uint4*>(&S.image[i]) = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    if (tid < (int)kPart / 4) *reinterpret_cast<uint4*>(&S.image[4 * tid]) = make_uint4(0u, 0u, 0u, 0u);
    if (!STATIC && wave == 0u) {
        images = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.images);
        words = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.image_words);
        ranges = cut_ranges(p.n_chunks, gridDim.x, images);
        take_range((uint32_t)__builtin_amdgcn_readfirstlane((int)S.range));
        if (wave < count) load_chunk_octets(p, c0 + wave, lane, w);
    }
    uint32_t range = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.range);
    if (blockIdx.x == 0 && tid < 256) p.stream[kHeaderBytes + tid] = (uint8_t)(S.tab[tid] >> 56);  // the container's length table
    for (int i = tid; i < (int)kStreamCodes<PAIRS>; i += 1024) {
        const unsigned long long e0 = S.tab[PAIRS ? i & 63 : i], e1 = PAIRS ? S.tab[i >> 6] : 0ull;
        const uint32_t l0 = (uint32_t)(e0 >> 56), l1 = (uint32_t)(e1 >> 56);
        const bool fits = l0 + l1 <= kShortCode;
        codes[PAIRS ? pair_slot((uint32_t)i & 63u, (uint32_t)i >> 6) : (uint32_t)i] = fits ? (uint32_t)e0 | ((uint32_t)e1 << (l0 & 31u)) | ((l0 + l1) << kShortCode) : kNoCode;
    }
    // (look_up reads them by their place in the LDS, which starts with them: no other shared memory in this kernel)
    asm volatile("" : : "s"((uint32_t)(uintptr_t)(lds_void_t*)dyn_lds) : "memory");
    __syncthreads();
    uint32_t* chunk_off = reinterpret_cast<uint32_t*>(p.stream + kHeaderBytes + kLenTableBytes);
    uint16_t* sub_bits = reinterpret_cast<uint16_t*>(p.stream + p.off_sub_bits);
    uint32_t* payload = reinterpret_cast<uint32_t*>(p.stream + p.off_payload);
    const uint32_t n_runs = p.subs_per_chunk;  // at most 64
    // First wavefront: what ranges [0, added) come to (bits: of the sizes this lane has read).
    uint32_t added = 0;
    unsigned long long added_words = 0, my_bits = 0;

    while (range < ranges.count) {
        const bool more = claims_another(ranges, gridDim.x);
        if (more && wave == kLast && lane == 0) ticket = claim();
        // ---- the chunks of the range into their images ----
        uint32_t slot = wave;
        while (slot < count) {
            const uint32_t next = slot + kStreamWaves;
            uint2 wn[8];
            if (next < count) load_chunk_octets(p, c0 + next, lane, wn);  // they arrive while this chunk is packed
            const uint32_t ch = c0 + slot;
            uint32_t from = 0;
            align_chunk_octets(p, ch, lane, w);
            const uint32_t bits = pack_octets<PAIRS>(w, chunk_len_of(p, ch), S.tab, S.image + slot * (words + 4u), words, S.past + lane, lane, S.runs[wave], from);
            if (lane == 0) {
                S.words[slot] = (bits + 31u) >> 5;
                if constexpr (STATIC) S.bits[slot] = bits;
                S.from[slot] = from;
            }
            sync_wave();
            if ((uint32_t)lane < n_runs) (sub_bits + (size_t)ch * n_runs)[lane] = S.runs[wave][lane];
            sync_wave();
            slot = next;
#pragma unroll
            for (int q = 0; q < 8; q++) w[q] = wn[q];
        }
        if (wave == kLast && lane == 0) S.next_range = more ? ticket : ranges.count;
        __syncthreads();
        // ---- the range's place: its size is published, and the sizes before it are added up ----
        const uint32_t first_ch = c0, n_here = count, next_range = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.next_range);
        const uint32_t my_words = (uint32_t)lane < n_here ? S.words[lane] : 0u;
        const uint32_t my_end = wave_exclusive_scan(my_words) + my_words;  // (of the range's first lane + 1 chunks)
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)my_end, 63);
        if (wave == 0u) {
            unsigned long long size = total;
            if constexpr (STATIC) size |= (unsigned long long)wave_sum((uint32_t)lane < n_here ? S.bits[lane] : 0u) << 32;
            if (lane == 0) publish64(&p.lookback[range], kKnown | size);  // (at most 64 x 6144 words and 64 x 196608 bits)
            // 256 sizes at a time, all loads in flight together; only those still missing are looked at again
            bool gone = false;
            for (; added < range && !gone; added += 256u) {
                unsigned long long e[4] = {0ull, 0ull, 0ull, 0ull};
                uint32_t tries = 0;
                for (;;) {
                    bool missing = false;
                    if (tries < p.spin_limit) {
#pragma unroll
                        for (int j = 0; j < 4; j++) {
                            const uint32_t i = added + 64u * (uint32_t)j + (uint32_t)lane;
                            if (i < range && e[j] == 0ull) e[j] = peek64(&p.lookback[i]);
                        }
                    }
#pragma unroll
                    for (int j = 0; j < 4; j++) missing |= added + 64u * (uint32_t)j + (uint32_t)lane < range && e[j] == 0ull;
                    if (!__any(missing)) break;
                    gone = ++tries > p.spin_limit;  // (seconds: never reached)
                    if (gone) break;
                    __builtin_amdgcn_s_sleep(1);
                }
                uint32_t sum = 0;
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    sum += (uint32_t)e[j];
                    if constexpr (STATIC) my_bits += (e[j] & (kKnown - 1ull)) >> 32;
                }
                added_words += wave_sum(sum);
            }
            if (gone && lane == 0) {
                const uint32_t was = __hip_atomic_fetch_or(&p.ctrl->error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                asm volatile("" : : "v"(was) : "memory");  // (the returned value is waited for)
                publish32(reinterpret_cast<uint32_t*>(p.stream), 0u);  // the header's magic
                S.gone = 1u;
            }
            if (lane == 0) S.before = added_words;
            added = range + 1u;
            added_words += total;
            if (STATIC && lane == 0) my_bits += size >> 32;
        }
        range = next_range;
        take_range(range);
        if (wave < count) load_chunk_octets(p, c0 + wave, lane, w);
        __syncthreads();
        if (S.gone) return;
        // ---- the images leave ----
        const unsigned long long before = S.before;
        if (wave == 0u && (uint32_t)lane < n_here) chunk_off[first_ch + (uint32_t)lane] = (uint32_t)before + my_end - my_words;
        for (slot = wave; slot < n_here; slot += kStreamWaves) {
            const uint32_t n_words = (uint32_t)__builtin_amdgcn_readlane((int)my_words, (int)slot);
            const unsigned long long word0 = before + ((uint32_t)__builtin_amdgcn_readlane((int)my_end, (int)slot) - n_words);
            uint32_t* img = S.image + slot * (words + 4u);
            uint32_t from = (uint32_t)__builtin_amdgcn_readfirstlane((int)S.from[slot]);
            const bool fits = word0 + n_words <= p.cap_words;  // (else the header is left invalid)
            for (uint32_t win = 0; win < n_words; win += words) {
                const uint32_t win_words = n_words - win < words ? n_words - win : words;
                if (win) {
                    pack_window<PAIRS>(p, first_ch + slot, S.tab, img, words, S.past + lane, win, lane, from);
                    sync_wave();
                }
                // four words per lane, to any word of the payload (images start on 16 bytes); then the last one to three
                uint32_t* out = payload + (size_t)word0 + win;
                for (uint32_t i = 4u * (uint32_t)lane; i + 4u <= win_words; i += 256u) {
                    const uint4 v = *reinterpret_cast<const uint4*>(img + i);
                    *reinterpret_cast<uint4*>(img + i) = make_uint4(0u, 0u, 0u, 0u);
                    if (fits) __builtin_memcpy(out + i, &v, 16);
                }
                const uint32_t i = (win_words & ~3u) + (uint32_t)lane;
                if (i < win_words) {
                    if (fits) out[i] = img[i];
                    img[i] = 0u;
                }
                sync_wave();  // the image is read and clear before the next window or chunk writes it
            }
        }
        if (wave == 0u && added == ranges.count) {  // the last range: the header
            if constexpr (STATIC) {
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) my_bits += __shfl_xor(my_bits, o, 64);
            }
            if (lane == 0) {
                chunk_off[p.n_chunks] = (uint32_t)added_words;
                // (word by word: a copy of the header on the stack is one that every lane of the kernel would write)
                Header* hdr = reinterpret_cast<Header*>(p.stream);
                hdr->version = p.hdr.version;
                hdr->bits = p.hdr.bits;
                hdr->reserved0 = p.hdr.reserved0;
                hdr->C = p.hdr.C;
                hdr->px_per_chunk = p.hdr.px_per_chunk;
                hdr->P = p.hdr.P;
                hdr->n_chunks = p.hdr.n_chunks;
                hdr->sub_syms = p.hdr.sub_syms;
                hdr->delta = p.hdr.delta;
                hdr->subs_per_chunk = p.hdr.subs_per_chunk;
                hdr->payload_words = added_words;
                hdr->payload_bits = STATIC ? my_bits : S.payload_bits;
                hdr->reserved1 = p.hdr.reserved1;
                // The magic last, past this part of the chip's cache: somebody who gives up waiting says so first and then
                // clears the magic the same way, so one of the two sees it.
                const bool fits = added_words <= p.cap_words && added_words <= 0xffffffffull;
                publish32(&hdr->magic, fits ? p.hdr.magic : 0u);
                __builtin_amdgcn_s_waitcnt(0);
                if (__hip_atomic_load(&p.ctrl->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) publish32(&hdr->magic, 0u);
                if (p.out_bytes) *p.out_bytes = (uint64_t)p.off_payload + 4 * added_words;
                // alignment gaps between the sections are part of the stream: keep them zero
                for (size_t o = kHeaderBytes + kLenTableBytes + 4 * ((size_t)p.n_chunks + 1); o < p.off_sub_bits; o++) p.stream[o] = 0;
                for (size_t o = p.off_sub_bits + 2 * (size_t)p.n_chunks * n_runs; o < p.off_payload; o++) p.stream[o] = 0;
            }
        }
        if (more) __syncthreads();  // the images are clear, and what the range left in LDS has been read
    }
}

// Number of workgroups of the pack kernel the device holds at once (queried once per kernel variant).
template <int MODE>
static int pack_resident_groups() {
    static std::atomic<int> cached{0};  // (every thread computes the same value)
    if (int c = cached.load(std::memory_order_relaxed)) return c;
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_pack<MODE>, 256, 0) != hipSuccess || cus < 1 ||
        per_cu < 1)
        return 64;  // conservative: any device this library runs on holds 64 workgroups
    if (per_cu > 4) per_cu = 4;
    cached.store(cus * per_cu, std::memory_order_relaxed);
    return cus * per_cu;
}

// Table (a kernel of its own only where every pack workgroup building it would cost more than the launch)
// and packing.
PackParams pack_params(const uint8_t* d_syms, const Geometry& g, int bits, float delta, const CoderScratch& cs,
                       int n_parts, const uint64_t* d_enc_table, uint8_t* d_stream, uint64_t cap_words,
                       uint64_t* d_out_bytes) {
    PackParams p{};
    p.cap_words = cap_words;
    p.syms = d_syms;
    p.V = (uint64_t)g.P * (uint64_t)g.C;
    p.n_chunks = g.n_chunks;
    p.chunk_syms = g.chunk_syms;
    p.subs_per_chunk = g.subs_per_chunk;
    p.n_groups = cs.n_groups;
    p.bits = bits;
    p.hist_parts = cs.hist_parts;
    p.n_parts = n_parts;
    p.enc_table = d_enc_table;
    p.ctrl = cs.ctrl;
    p.lookback = cs.lookback;
    p.hdr = Header{};
    p.hdr.magic = kMagic;
    p.hdr.version = 1;
    p.hdr.bits = (uint8_t)bits;
    p.hdr.C = (uint32_t)g.C;
    p.hdr.px_per_chunk = g.px_per_chunk;
    p.hdr.P = (uint64_t)g.P;
    p.hdr.n_chunks = g.n_chunks;
    p.hdr.sub_syms = kSubSyms;
    p.hdr.delta = delta;
    p.hdr.subs_per_chunk = g.subs_per_chunk;
    p.off_sub_bits = g.off_sub_bits;
    p.off_payload = g.off_payload;
    p.stream = d_stream;
    p.out_bytes = d_out_bytes;
    p.static_max_len = 0;
    p.spin_limit = test_option(kTestShortWaits) ? 0u : kSpinLimit;
    return p;
}

// Packing of a tensor with more chunk groups than the device holds pack workgroups.
template <bool STATIC>
static hipError_t launch_pack_large(const PackParams& p, hipStream_t s) {
    // One workgroup per compute unit: its images take most of the LDS.  Ranges have four chunks at least, so their sizes
    // fit the look-back words.
    if (p.n_groups < pack_groups(p.n_chunks)) return hipErrorInvalidValue;
    const unsigned grid = p.n_groups < 256u ? p.n_groups : 256u;
    // (7 and 8 bits: a table of pairs would not fit beside the images)
    const bool pairs = p.bits <= 6;
    const size_t lds = sizeof(StreamShared) + sizeof(uint32_t) * (pairs ? kStreamCodes<true> : kStreamCodes<false>);
    const void* fn = pairs ? reinterpret_cast<const void*>(&k_pack_stream<STATIC, true>)
                           : reinterpret_cast<const void*>(&k_pack_stream<STATIC, false>);
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    if (pairs) return launch(K_PACK, k_pack_stream<STATIC, true>, dim3(grid), dim3(1024), lds, s, p);
    return launch(K_PACK, k_pack_stream<STATIC, false>, dim3(grid), dim3(1024), lds, s, p);
}

hipError_t launch_coder(const uint8_t* d_syms, const Geometry& g, int bits, float delta, const CoderScratch& cs,
                        int n_parts, uint64_t* d_enc_table, uint8_t* d_stream, uint64_t cap_words,
                        uint64_t* d_out_bytes, hipStream_t s) {
    PackParams p = pack_params(d_syms, g, bits, delta, cs, n_parts, d_enc_table, d_stream, cap_words, d_out_bytes);
    const uint32_t resident = (uint32_t)pack_resident_groups<kPackTable>();
    if (cs.n_groups > resident) return launch_pack_large<false>(p, s);
    // every pack workgroup sums the partial histograms itself while that is at most 64 KB to read
    const bool build_in_pack = ((size_t)n_parts << bits) * 4 <= 64 * 1024;
    if (!build_in_pack) {
        hipError_t e = launch(K_TABLE, k_huffman_table, dim3(1), dim3(1024), 0, s, (const uint32_t*)cs.hist_parts,
                              n_parts, bits, (uint32_t*)nullptr, d_enc_table, d_stream + kHeaderBytes, cs.ctrl, 0u);
        if (e != hipSuccess) return e;
        return launch(K_PACK, k_pack<kPackTable>, dim3(cs.n_groups), dim3(256), 0, s, p);
    }
    const uint32_t cap = (uint32_t)pack_resident_groups<kPackBuild>();
    if (cs.n_groups > cap) return hipErrorInvalidValue;  // (not reachable: the two variants hold the same number)
    return launch(K_PACK, k_pack<kPackBuild>, dim3(cs.n_groups), dim3(256), 0, s, p);
}

// Packing with a table fixed beforehand (one code for every symbol of the alphabet): no histogram, no table build.
// The coder's counters must be clear (the kernel that made the symbols clears them).
hipError_t launch_coder_static(const uint8_t* d_syms, const Geometry& g, int bits, float delta, const CoderScratch& cs,
                               const uint64_t* d_enc_table, uint32_t max_len, uint8_t* d_stream, uint64_t cap_words,
                               uint64_t* d_out_bytes, hipStream_t s) {
    PackParams p = pack_params(d_syms, g, bits, delta, cs, 0, d_enc_table, d_stream, cap_words, d_out_bytes);
    p.static_max_len = max_len;
    const uint32_t cap = (uint32_t)pack_resident_groups<kPackStatic>();
    if (cs.n_groups > cap) return launch_pack_large<true>(p, s);
    return launch(K_PACK, k_pack<kPackStatic>, dim3(cs.n_groups), dim3(256), 0, s, p);
}

}  // namespace fmtc
