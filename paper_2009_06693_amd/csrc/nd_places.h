// Where things go, as plain arithmetic that kernels and host code share (constexpr functions are both).
#pragma once

#include <stdint.h>

namespace nd {

// The bit of a vertex in the 65,536-bit map of a sample's vertices (nd_edges.hip): word 0-2047 and the bit in it, counted
// from the top.  Every bit of the id reaches both, as ids have structure in any of theirs: of 2,048 vertices of a
// graph, others pass with a chance of 0.03 when they are spread, and of 0.37 (multiples of 64) to 1 (64 communities
// 2^16 apart, 256 vertices each) when word and bit are bits of the id.  One 24-bit multiplication and addition, at the
// full rate; of 120 odd factors the one with nearly the least chance over strides and blocks of ids (0.06).
constexpr uint32_t edge_map_hash(int32_t v) { return ((uint32_t)v & 0xFFFFFFu) * 0x77C9A9u + (uint32_t)v; }
constexpr uint32_t edge_map_word(uint32_t hash) { return (hash >> 15) & 2047u; }
constexpr uint32_t edge_map_bit(uint32_t hash) { return (hash >> 26) & 31u; }

}  // namespace nd
