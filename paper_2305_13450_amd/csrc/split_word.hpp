// The word the parts of a tile split along K meet on, where every part finishes a slice of the tile's rows (see the
// exchange in gemm_tile.hpp): what one thread of each part does with it, in order.  Templates over the memory, so that
// the host can run the same code against a model of it (tests/split_word_check.cpp).
//
// The word is zero between chains.  Parts that have published in bits 0-7, slices left behind in bits 8-15 (bit 8 + z: part
// z's), parts that have left in bits 16-23, parts that have started in bits 24-31; up to 8 parts.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define DS_SPLIT_FN __host__ __device__ __forceinline__
#else
#define DS_SPLIT_FN inline
#endif

namespace depsync {

constexpr uint32_t SPLIT_PUBLISHED = 1u, SPLIT_BEHIND = 1u << 8, SPLIT_LEFT = 1u << 16, SPLIT_STARTED = 1u << 24;
constexpr uint32_t SPLIT_AGAIN = 1u << 8;   // instead of a list of slices (bits 0-7)

DS_SPLIT_FN uint32_t split_published(uint32_t word) { return word & 0xffu; }
DS_SPLIT_FN bool split_all_started(uint32_t word, uint32_t S) { return (word >> 24) == S; }

// Part z's partials but for its own slice are in memory.  The slices it finishes now, or SPLIT_AGAIN: it must not wait for the
// others, so it leaves its own slice in memory as well and calls split_publish_whole.
// has_slice: part z has rows to finish.  all_started: every part was seen to have been started.
template <class Mem>
DS_SPLIT_FN uint32_t split_publish(Mem& m, uint32_t S, uint32_t z, bool has_slice, bool all_started) {
    if (has_slice && !all_started) return SPLIT_AGAIN;
    const uint32_t old = m.add(SPLIT_PUBLISHED);
    const bool last = split_published(old) == S - 1;
    uint32_t todo = 0;
    if (has_slice && (last || m.wait_published(S))) todo = 1u << z;
    if (last) todo |= (old >> 8) & 0xffu;
    return todo;
}

// All of part z's partials are in memory.
template <class Mem>
DS_SPLIT_FN uint32_t split_publish_whole(Mem& m, uint32_t S, uint32_t z) {
    const uint32_t old = m.add(SPLIT_PUBLISHED + (SPLIT_BEHIND << z));
    return split_published(old) == S - 1 ? ((old >> 8) & 0xffu) | (1u << z) : 0u;
}

// Part z's slices are in memory.  The last part to leave clears the word and posts the tile.
// outlives: the post lets the chain end, and a later chain begin, while this launch is still running (side launches are
// not joined back).  The clear must then be in memory before the post: it would wipe out what the later chain's parts have counted.
// Everywhere else the end of the launch stands between, and the post does not wait for the clear's round trip.
template <class Mem, class Post>
DS_SPLIT_FN void split_leave(Mem& m, uint32_t S, bool outlives, Post post) {
    if (((m.add(SPLIT_LEFT) >> 16) & 0xffu) != S - 1) return;
    m.clear();
    if (outlives) m.drain();
    post();
}

}  // namespace depsync
