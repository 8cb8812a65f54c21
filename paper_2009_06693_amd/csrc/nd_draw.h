// What one lane draws (Section 4.2 of the paper: the `next` functions of the
// applications), shared by every sampling kernel: uniform neighbour (DeepWalk,
// PPR, k-hop), weight-proportional neighbour by inverse transform, node2vec by
// rejection sampling.  One Philox call per (sample, slot, step, attempt).
#pragma once

#include "nd_common.h"
#include "nd_philox.h"
#include "nd_sample.h"

namespace nd {

constexpr uint32_t kOneQ16 = 65536u;

// ---------------------------------------------------------------- one draw
// adj / cum / wq point at the transit's row (global memory or its LDS copy).

template <typename OffT>
__device__ __forceinline__ bool row_contains(const GraphView<OffT>& g, uint64_t rs, uint32_t deg,
                                             int32_t u) {
    uint32_t lo = 0, hi = deg;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        const int32_t c = g.col[rs + mid];
        if (c < u) lo = mid + 1;
        else hi = mid;
    }
    return lo < deg && g.col[rs + lo] == u;
}

// Uniform neighbour (DeepWalk, PPR, k-hop): index = high word of R0 * degree.
__device__ __forceinline__ int32_t draw_uniform(const DrawArgs& a, uint32_t deg, uint32_t sid,
                                                uint32_t slot, const int32_t* adj) {
    const Rand4 r = draw4(a.seed, sid, slot, a.step, 0u);
    if (a.ppr_thr != 0 && (uint64_t)r.r3 < a.ppr_thr) return ND_NULL_VERTEX;
    return adj[mulhi32(r.r0, deg)];
}

// Weight-proportional neighbour: inverse transform on the row's running sums.
__device__ __forceinline__ int32_t draw_weighted(const DrawArgs& a, uint32_t deg, uint32_t sid,
                                                 uint32_t slot, const int32_t* adj,
                                                 const uint64_t* cum) {
    const Rand4 r = draw4(a.seed, sid, slot, a.step, 0u);
    if (a.ppr_thr != 0 && (uint64_t)r.r3 < a.ppr_thr) return ND_NULL_VERTEX;
    const uint64_t x = mulhi64(cat64(r.r0, r.r1), cum[deg - 1]);
    uint32_t lo = 0, hi = deg - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (cum[mid] > x) hi = mid;
        else lo = mid + 1;
    }
    return adj[lo];
}

// The same draw over the row's WeightLinks (deg >= 1): the link of the first entry whose threshold exceeds the
// draw's 64-bit word.  The guide of the word's cell names an entry at or before it, about one entry before on
// average; a look is at two entries and their links (as compiled one entry after the other, the last word of
// each after its threshold).  A cell holds as many entries as are light
// beside the row's heavy ones, up to nearly the whole row, so after two looks what is left of the cell, which
// ends at the next cell's guide, is searched by halves: 65,536 walks of 8 steps between a hub of 20,000 entries,
// one of which outweighs the others together, and its leaves took 2.4 ms where the walk went on entry by entry,
// 0.013 like this; 64 samples of one transit and 4,096 draws from rows whose weights span five decades 22.4 us with
// four looks and the rest of the row by halves, 16.6 like this, 17.6 with a search of the row's running sums.
__device__ __forceinline__ Link drawn_link(const Link* row, uint32_t deg, uint64_t word) {
    const WeightLink* weights = reinterpret_cast<const WeightLink*>(row);
    const uint32_t cell = mulhi32((uint32_t)(word >> 32), deg);
    uint32_t j = deg > 1u ? weights[2ull * cell + 1u].guide : 0u;
    for (int look = 0; look < 2; ++look) {
        const uint32_t j1 = j + 1u < deg ? j + 1u : j;
        const WeightLink w0 = weights[2ull * j + 1u], w1 = weights[2ull * j1 + 1u];
        const Link l0 = row[2ull * j], l1 = row[2ull * j1];
        if (word < w0.thr || w0.always() || j1 == j) return l0;
        if (word < w1.thr || w1.always() || j1 + 1u == deg) return l1;
        j = j1 + 1u;
    }
    uint32_t lo = j, hi = cell + 1u < deg ? weights[2ull * (cell + 1u) + 1u].guide : deg - 1u;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        const WeightLink w = weights[2ull * mid + 1u];
        if (word < w.thr || w.always()) hi = mid;
        else lo = mid + 1u;
    }
    return row[2ull * lo];
}

// The same draw through the row's WeightCells: one scattered fetch, where the guide and then the entries are two or
// three.  100 steps of PPR at 0.01, weights in [1, 5): 57 K walks on 1.6 M entries 174 us by the links and 85 by the
// cells, 64 walks (16 lanes each) 54 and 31, 600 K walks on 39 M entries 1,465 and 1,001; symmetric weights 2^14 / (deg
// deg), where a draw ends behind its cell's four entries more often, 216 and 146 for the 57 K.  Not used by layer
// sampling: over the 115 M entries of 2.9 M vertices, 7 GB of cells, 257 samples of [512, 512] took 42.8 us, 30.5 by
// the links.  In two halves so that other work can go between them: the cell's fetch,
// and the choice.  The assembler statement keeps the four loads whole and together: the compiler otherwise leaves loads of
// the words that are selected until it knows which, a second and a third wait.
typedef uint32_t Words4 __attribute__((ext_vector_type(4)));
struct CellWords {
    Words4 thr, a, b, c;
};
__device__ __forceinline__ void fetch_cell(CellWords& x, const WeightCell* cells, uint32_t rs, uint32_t deg, uint32_t hi) {
    const Words4* piece = reinterpret_cast<const Words4*>(cells + (uint64_t)(rs + mulhi32(hi, deg)));
    x.thr = piece[0];
    x.a = piece[1];
    x.b = piece[2];
    x.c = piece[3];
}
__device__ __forceinline__ uint32_t either(bool which, uint32_t x, uint32_t y) { return which ? x : y; }
// draws: this lane has fetched a cell (others' answers mean nothing).
__device__ __forceinline__ Link pick_link(CellWords& x, const Link* links, uint32_t rs, uint32_t deg, uint64_t word,
                                          bool draws) {
    asm volatile("" : "+v"(x.thr), "+v"(x.a), "+v"(x.b), "+v"(x.c));
    const uint32_t hi = (uint32_t)(word >> 32);
    const bool b0 = hi >= x.thr.x, b1 = hi >= x.thr.y, b2 = hi >= x.thr.z;
    Link l;
    // one selection after the other (nested, they become branches)
    l.v = (int32_t)either(b2, x.c.y, either(b1, x.b.z, either(b0, x.a.w, x.a.x)));
    l.rs = either(b2, x.c.z, either(b1, x.b.w, either(b0, x.b.x, x.a.y)));
    l.deg = either(b2, x.c.w, either(b1, x.c.x, either(b0, x.b.y, x.a.z)));
    l.wq = 0;
    const bool unsure = hi >= x.thr.w || hi == x.thr.x || hi == x.thr.y || hi == x.thr.z;
    if (draws && unsure) l = drawn_link(links + (uint64_t)rs * 2u, deg, word);
    return l;
}

// node2vec (Section 4.2): rejection sampling under the envelope
// maxEdgeWeight(v) * largest bias; the bias of candidate u depends on its
// relation to t, the transit of the previous step.  The membership search in
// t's row is skipped when both possible biases give the same verdict.
template <typename OffT>
__device__ __forceinline__ uint32_t n2v_bias(const GraphView<OffT>& g, const DrawArgs& a, int32_t t,
                                             uint64_t rs_t, uint32_t deg_t, int32_t u) {
    if (!a.has_prev) return kOneQ16;
    if (u == t) return a.b_ret;
    // values, not a choice between two members: the latter is a choice between two addresses and
    // keeps the whole structure in memory
    const uint32_t b_com = a.b_com, b_far = a.b_far;
    return row_contains(g, rs_t, deg_t, u) ? b_com : b_far;
}

// t: the transit of the previous step (read only when a.has_prev).
template <typename OffT>
__device__ __forceinline__ int32_t draw_node2vec(const GraphView<OffT>& g, const DrawArgs& a,
                                                 int32_t v, uint32_t deg, uint32_t sid,
                                                 int32_t t_prev, const int32_t* adj,
                                                 const uint32_t* wq) {
    const uint32_t maxw = a.use_weights ? g.maxwq[v] : kOneQ16;
    const uint64_t envelope = (uint64_t)maxw * (a.has_prev ? a.b_max : kOneQ16);
    int32_t t = ND_NULL_VERTEX;
    uint64_t rs_t = 0;
    uint32_t deg_t = 0;
    if (a.has_prev) {
        t = t_prev;
        rs_t = (uint64_t)g.off[t];
        deg_t = row_length(g, t, rs_t);
    }
    const uint32_t b_com = a.b_com, b_far = a.b_far;  // values: see n2v_bias
    const uint32_t b_lo = b_com < b_far ? b_com : b_far;
    const uint32_t b_hi = b_com < b_far ? b_far : b_com;
    for (int32_t att = 0; att < a.max_attempts; ++att) {
        const Rand4 r = draw4(a.seed, sid, 0u, a.step, (uint32_t)att);
        const uint32_t e = mulhi32(r.r0, deg);
        const int32_t u = adj[e];
        const uint64_t y = mulhi64(cat64(r.r1, r.r2), envelope);
        const uint64_t w = a.use_weights ? wq[e] : kOneQ16;
        if (!a.has_prev) {
            if (y < w * kOneQ16) return u;
        } else if (u == t) {
            if (y < w * a.b_ret) return u;
        } else if (y < w * b_lo) {
            return u;
        } else if (y < w * b_hi) {
            const uint32_t bias = row_contains(g, rs_t, deg_t, u) ? b_com : b_far;
            if (y < w * bias) return u;
        }
    }
    // exact fallback: inverse transform over all biased weights of the row
    const Rand4 r = draw4(a.seed, sid, 0u, a.step, (uint32_t)a.max_attempts);
    uint64_t Z = 0;
    for (uint32_t e = 0; e < deg; ++e) {
        const uint64_t w = a.use_weights ? wq[e] : kOneQ16;
        Z += w * n2v_bias(g, a, t, rs_t, deg_t, adj[e]);
    }
    const uint64_t x = mulhi64(cat64(r.r0, r.r1), Z);
    uint64_t run = 0;
    for (uint32_t e = 0; e < deg; ++e) {
        const uint64_t w = a.use_weights ? wq[e] : kOneQ16;
        run += w * n2v_bias(g, a, t, rs_t, deg_t, adj[e]);
        if (run > x) return adj[e];
    }
    return adj[deg - 1];  // not reached: x < Z
}

}  // namespace nd
