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

// Lane-per-draw sampling (nd_sample.hip): 256-lane groups, four to a workgroup, take blocks of the sorted pairs in turn.
// Workgroups go to the eight XCDs in turn, so that by themselves neighbouring groups are on different ones, each of which
// reads the rows at a block's end as well.  With the groups of an XCD next to each other the pairs of a transit meet its
// row in one L2, as a rule even in one L1; but a round that does not fill the grid then leaves whole XCDs idle, and
// at few draws per pair the pairs and their rows weigh more than the draws.  Grid in turn over the other order, by
// draws per pair and rounds of the grid, 2 M vertices of mean degree 30 and 233 K of 257:
//   1 draw, 0.5 rounds 0.88, 1.25 0.91, 3 0.90, 10 0.98; by weights 0.69, 0.78, 0.99, 1.00;
//   3 draws 0.86, 0.90, 1.02, 1.02;  5 draws 0.84, 0.91, 1.06, 1.03, 6 rounds 0.99;
//   10 draws 0.87, 0.94, 1.08, 1.00;  25 draws 0.94, 0.96, 1.07, 1.07;  300 draws 1.00, 1.02, 1.04, 1.10.
// 5.8 M pairs of 10 draws, mean degree 487 (57 rounds): 317 us in turn, 297 like this.
constexpr uint32_t kNeighbourRounds = 3, kNeighbourDraws = 5;
// The number of pairs from which a launch has its groups next to each other; draws_per_round: of all its groups.
constexpr uint32_t pairs_of_neighbours(uint32_t per_pair, uint32_t workgroups, uint32_t draws_per_round) {
    return workgroups % 8u == 0u && per_pair >= kNeighbourDraws ? (kNeighbourRounds * draws_per_round + per_pair - 1u) / per_pair
                                                                : 0xFFFFFFFFu;
}
// Which block of the first round group `group` (0-3) of workgroup `workgroup` takes.
constexpr uint32_t first_block(uint32_t workgroup, uint32_t group, uint32_t workgroups, bool next_to_each_other) {
    return next_to_each_other ? (workgroup % 8u) * (workgroups / 8u * 4u) + workgroup / 8u * 4u + group
                              : group * workgroups + workgroup;
}

}  // namespace nd
