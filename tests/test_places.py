"""The arithmetic of nd_places.h, which kernels share with the host, compiled for the CPU."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SOURCE = r"""
#include "nd_places.h"
extern "C" void edge_bits(const int32_t* v, int64_t n, int32_t* bit) {
    for (int64_t i = 0; i < n; ++i) {
        const uint32_t h = nd::edge_map_hash(v[i]);
        bit[i] = (int32_t)(nd::edge_map_word(h) * 32u + nd::edge_map_bit(h));
    }
}
extern "C" int blocks_of_groups(uint32_t pairs, uint32_t per_pair, uint32_t workgroups, uint32_t per_round, uint32_t* block) {
    const bool next = pairs >= nd::pairs_of_neighbours(per_pair, workgroups, per_round);
    for (uint32_t w = 0; w < workgroups; ++w)
        for (uint32_t g = 0; g < 4; ++g) block[w * 4 + g] = nd::first_block(w, g, workgroups, next);
    return next;
}
"""


@pytest.fixture(scope="module")
def places(tmp_path_factory):
    d = tmp_path_factory.mktemp("places")
    (d / "places.cpp").write_text(SOURCE)
    csrc = os.path.join(os.path.dirname(HERE), "paper_2009_06693_amd", "csrc")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-shared", "-fPIC", "-I", csrc, str(d / "places.cpp"),
                    "-o", str(d / "places.so")], check=True)
    return ctypes.CDLL(str(d / "places.so"))


def _bits(places, v):
    v = np.ascontiguousarray(v, dtype=np.int32)
    out = np.empty_like(v)
    places.edge_bits(v.ctypes.data_as(ctypes.c_void_p), ctypes.c_int64(v.size), out.ctypes.data_as(ctypes.c_void_p))
    return out


def _blocks(n, low_bits, high_bit):
    """n blocks of 2^low_bits consecutive ids, 2^high_bit apart."""
    return ((np.arange(n, dtype=np.int64)[:, None] << high_bit) + np.arange(1 << low_bits)).ravel()


@pytest.mark.parametrize("ids", [
    pytest.param(np.arange(0, 1 << 22, stride) + first, id=f"{first} and every {stride}th")
    for stride, first in ((1, 0), (2, 1), (8, 0), (8, 3), (64, 0), (256, 0), (1000, 0), (4096, 5))
] + [pytest.param(np.arange(0, (1 << 31) - 1, s), id=f"every {s}th of all") for s in (4096, 65536)
] + [pytest.param(_blocks(n, low, high), id=f"{n} blocks of 2^{low} at 2^{high}")
     for n, low, high in ((64, 8, 14), (64, 8, 16), (64, 10, 18), (64, 12, 24), (1000, 8, 20), (1000, 5, 11))])
def test_few_vertices_share_a_bit_of_the_edge_map_whatever_the_ids_structure(places, ids):
    """2,048 vertices set at most 2,048 of 65,536 bits: a chance of 0.031 that a vertex of no slot passes when ids are
    spread.  Three times that is allowed for: entries that pass are looked up, which takes a multiple of the test
    (multiples of 64 with a map of id bits: 0.37 passed, and the passes took twice as long)."""
    rng = np.random.default_rng(11)
    bits = _bits(places, ids)
    assert bits.min() >= 0 and bits.max() < 65536
    rates = []
    for _ in range(4):
        order = rng.permutation(ids.size)
        held, others = order[:min(2048, ids.size // 4)], order[min(2048, ids.size // 4):][:50_000]
        in_map = np.zeros(65536, dtype=bool)
        in_map[bits[held]] = True
        rates.append(in_map[bits[others]].mean())
    assert np.mean(rates) < 3 * 2048 / 65536


@pytest.mark.parametrize("workgroups", [1, 7, 8, 100, 504, 512])
@pytest.mark.parametrize("per_pair,in_flight", [(1, 1), (1, 2), (2, 2), (3, 2), (5, 2), (10, 2), (25, 2), (100, 1), (300, 2),
                                                (250_000, 2)])
def test_groups_of_lanes_take_each_block_once_and_few_rounds_use_every_xcd(places, workgroups, per_pair, in_flight):
    """A block of pairs per group and round, workgroup w on XCD w % 8: no XCD has much more than the mean, at any number
    of draws (half a round on four of the eight: 1.25 to 1.45 times the time of the draws, one per pair by weights).  A
    round that is nearly empty weighs a third where there are three before it, and all there is where it is alone."""
    groups = 4 * workgroups
    whole = 256 // per_pair
    per_group = whole * in_flight if whole * per_pair >= 231 else 256 / per_pair  # pairs per round
    block = np.empty(groups, dtype=np.uint32)
    orders = set()
    for rounds in (0.3, 0.5, 0.75, 1.0, 1.25, 1.5, 2.1, 2.98, 3.0, 3.2, 5.5, 20.0, 40.0):
        pairs = max(1, int(rounds * groups * per_group))
        orders.add(places.blocks_of_groups(pairs, per_pair, workgroups, round(groups * per_group * per_pair),
                                           block.ctypes.data_as(ctypes.c_void_p)))
        assert np.array_equal(np.sort(block), np.arange(groups))
        blocks = int(-(-pairs // per_group))                           # block b, b + groups, b + 2 groups, ... are a group's
        load = np.zeros(8)
        np.add.at(load, (np.arange(groups) // 4) % 8, np.maximum(0, -(-(blocks - block.astype(np.int64)) // groups)))
        if workgroups % 8 == 0 and blocks >= 8 * 4:
            assert load.max() <= (1.34 if rounds > 3 else 1.13) * load.mean(), (rounds, load)
    allowed = workgroups % 8 == 0 and per_pair >= 5
    whole_pairs_are_many_rounds = per_pair >= 3 * groups * 256
    assert orders == ({1} if allowed and whole_pairs_are_many_rounds else {0, 1} if allowed else {0})
