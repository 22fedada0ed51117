// How the packer of large tensors (k_pack_stream) cuts a tensor into ranges of chunks, and when a workgroup claims its next
// one: the rules that decide whether every wait of a workgroup ends.  Plain C++, so that a model of the protocol on the CPU
// runs the same rules.
//
// A workgroup claims a range by a ticket from a counter, packs it, publishes its size, waits for the sizes of all ranges
// before it and stores.  A range's number is its ticket, so the ranges before it are claimed by workgroups that run, and a
// size waits for nothing but its workgroup's range before: the lowest range without a size can always go on, however few of
// the grid's workgroups run at a time and in whatever order they start.
#pragma once
#include <stdint.h>

namespace fmtc {

struct Ranges {
    uint32_t chunks, count;  // chunks of a range (the last one: the rest), and how many ranges there are
};
// All ranges of one size, as few rounds of them per workgroup as its images allow.
constexpr Ranges cut_ranges(uint32_t n_chunks, uint32_t grid, uint32_t images) {
    const uint32_t rounds = (n_chunks + grid * images - 1u) / (grid * images);
    const uint32_t chunks = (n_chunks + grid * rounds - 1u) / (grid * rounds);
    return {chunks, (n_chunks + chunks - 1u) / chunks};
}
struct ChunkSpan {
    uint32_t first, count;
};
// (past the last range: no chunks)
constexpr ChunkSpan range_chunks(Ranges r, uint32_t range, uint32_t n_chunks) {
    const uint32_t first = range < r.count ? range * r.chunks : n_chunks;
    return {first, n_chunks - first < r.chunks ? n_chunks - first : r.chunks};
}
// Does a workgroup that has a range claim another one?  (Where there are no more ranges than workgroups each has one at most.)
constexpr bool claims_another(Ranges r, uint32_t grid) { return r.count > grid; }

}  // namespace fmtc
