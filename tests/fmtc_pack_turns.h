// Who packs what, and who waits for whom, in a packer whose workgroups take turns: the rules that decide whether every wait of
// a workgroup ends.  Plain C++, for the model of the protocol on the CPU (pack_turns_model.cpp).  k_pack_stream followed these
// rules until its workgroups took whole ranges of chunks, with workgroup barriers in place of these waits.
//
// A workgroup's turns are the groups of chunks that it claims, one after the other.  Packers keep images of packed chunks
// until the place of the chunk's turn is known.  A turn's size is published when all its chunks are packed, and its place
// follows some time after that.  So a packer may wait for the place of a turn only if it holds no unpacked chunk of it:
// of a turn that is not packed whole a packer takes at most as many chunks as it has images (`most`), and with every
// image in use and one more chunk in hand the oldest image is then of an earlier turn than that chunk.
#pragma once
#include <stdint.h>

namespace fmtc {

constexpr uint32_t kStreamWaves = 15;        // packing wavefronts per workgroup = chunks per group
constexpr uint32_t kSlots = 16;              // what a turn leaves in LDS is kept by turn modulo kSlots
constexpr uint32_t kTurnsAhead = 2;          // turns published that may be waiting for their places when one more is
constexpr uint32_t kGone = 0xffffffffu;      // in place of a number of turns: a wait ran out, all packers leave

// The next chunk to be taken, in one word: the lowest turn with chunks left << 8 | chunks taken of the turn after it << 4 |
// chunks taken of it.  (A workgroup has fewer than 2^24 turns: a chunk holds at least 33 symbols, a tensor less than 2^32.)
struct Dealt {
    uint32_t state, n;  // the word afterwards; the chunk's number in the workgroup, turn * waves + place
};
// A packer that has taken `own` chunks of its latest turn `own_turn` takes the next one: of the lowest turn with chunks
// left, or of the turn after that once it has had its share.  It never finds its share of both used up, since none of
// these chunks has been stored yet: it would hold 2 * most of them, and it has `most` images (at least two) and at most
// one chunk in hand when it takes the next.  Nor does the later turn run out before the lower one: the packers that have
// had their share of the lower one are fewer than waves / most.  (Should it come to that, the chunk of the lower turn is
// taken after all.)
constexpr Dealt deal(uint32_t state, uint32_t own_turn, uint32_t own, uint32_t most, uint32_t waves = kStreamWaves) {
    const uint32_t turn = state >> 8, later = (state >> 4) & 15u, now = state & 15u;
    const bool had_share = own_turn > turn || (own_turn == turn && own >= most);
    const bool had_next = own_turn == turn + 1u && own >= most;
    if (had_share && !had_next && later < waves) return {state + 16u, (turn + 1u) * waves + later};
    const uint32_t n = turn * waves + now;
    if (now + 1u < waves) return {state + 1u, n};
    if (later < waves) return {((turn + 1u) << 8) | later, n};
    return {(turn + 2u) << 8, n};
}

// Does a packer with `waiting` images, the oldest of turn `oldest`, store one before it packs the next chunk?  (`placed`:
// turns whose place is known.  With all images in use it waits for that place.)
constexpr bool stores_first(uint32_t waiting, uint32_t images, uint32_t placed, uint32_t oldest) {
    return waiting != 0u && (waiting >= images || placed > oldest);
}

// May the size of turn `published` be published, its chunks being packed?  (Not so many turns ahead of the places that a
// slot would be used again while a packer still needs it.)
constexpr bool may_publish(uint32_t published, uint32_t placed) { return published - placed <= kTurnsAhead; }

}  // namespace fmtc
