// Random walks whose lanes run free: the default route of the walks.
//
// A walk step is a chain - generator, edge, the row of the vertex it leads to - and its output must
// not depend on how samples are grouped.  Grouping by transit (Section 6.1.2 of the paper, GPU-wide
// or in the windows of nd_walk.hip) costs barriers and LDS traffic at every step to save scattered
// reads that the caches mostly serve already; what a walk is bound by is the chain itself (few walks)
// or the rate of scattered fetches (many).  Both are cut by the graph's Links: the edge that is drawn
// carries the row of its end vertex, so a step is one fetch instead of two dependent ones, and a lane
// keeps its walk in registers from the first step to the last, with no barrier in between.
#include <utility>

#include "nd_common.h"
#include "nd_philox.h"
#include "nd_wave.h"
#include "nd_sample.h"
#include "nd_draw.h"

namespace nd {

namespace {

constexpr int kFreeChunk = 128;  // steps per launch: their output pointers are kernel arguments
constexpr int kDrawCells = 3;    // kDrawWeighted through the WeightCells
constexpr int kAttemptLanes = 4;  // few walks of node2vec: attempts at once
constexpr int kFewThreads = 256, kFewLanes = 16;  // few walks: threads per workgroup, lanes per walk

struct FreeArgs {
    const Link* links;
    uint64_t seed;
    uint64_t ppr_thr;
    uint32_t sample_base;
    uint32_t S;
    uint32_t s_first;          // the launch's first sample: a call of very many samples takes several launches
    uint32_t first_step, n_steps;
    int32_t V;
    const int32_t* src;        // the roots, or the output of step first_step - 1 (multi-dimensional walk: its roots)
    const int32_t* prev_src;   // node2vec, first_step > 0: the output of step first_step - 2
    const int32_t* rowset;     // node2vec: membership tables, may be null
    const WeightCell* cells;   // weighted draws: may be null
    uint32_t b_ret, b_com, b_far, b_max;
    int32_t max_attempts, use_weights;
    uint32_t R;                // multi-dimensional walk: roots per sample
    const uint64_t* filled;    // ... a bit per vertex, whether its row has entries (FILLED)
    int32_t* state;            // ... and where they go when more steps follow, else null
    WsHeader* hdr;
    uint32_t* flags;           // per workgroup: a root was outside [0, V) (launches of the first steps)
    uint32_t* parts;           // [workgroup][step of the call]: live walks
                               // launches after the call's first samples add to both
    uint32_t total_steps;
    uint64_t o_flags, o_parts;
    int32_t* out[kFreeChunk];
};

// Live pairs of every step, from what each lane knows at the end: its walk had a transit at the first
// `lived` steps of this launch.  One histogram entry per lane, then sums from the top.
template <int THREADS>
__device__ __forceinline__ void publish_live(uint32_t lived, const FreeArgs& a, uint32_t* hist) {
    const uint32_t n_steps = a.n_steps;
    uint32_t* parts = a.parts + (uint64_t)blockIdx.x * a.total_steps + a.first_step;
    for (uint32_t i = threadIdx.x; i <= (uint32_t)kFreeChunk; i += THREADS) hist[i] = 0;
    __syncthreads();
    if (lived > 0) atomicAdd(&hist[lived], 1u);
    __syncthreads();
    if (threadIdx.x < 64) {  // one wavefront: two positions per lane, from the last step down
        const int lane = lane_id();
        uint32_t carry = 0;
        for (int half = 1; half >= 0; --half) {
            const uint32_t step = (uint32_t)(half * 64 + 63 - lane);  // a live length above `step` counts
            const uint32_t mine = step < n_steps ? hist[step + 1u] : 0u;
            const uint32_t incl = wave_inclusive_scan(mine, lane);
            if (step < n_steps) parts[step] = (a.s_first > 0 ? parts[step] : 0u) + carry + incl;
            carry += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        }
    }
}

// One lane per workgroup: what its roots looked like, and the header.
__device__ __forceinline__ void publish_root_check(const FreeArgs& a, int any_bad) {
    a.flags[blockIdx.x] = (a.s_first > 0 ? a.flags[blockIdx.x] : 0u) | (any_bad ? 1u : 0u);
    if (blockIdx.x == 0 && a.s_first == 0) write_header(a.hdr, a.total_steps, gridDim.x, a.o_flags, a.o_parts);
}

// The walk's first transit and, in the first launch, what the host may ask for afterwards.
template <int THREADS>
__device__ __forceinline__ int32_t first_transit(const FreeArgs& a, uint32_t s) {
    int32_t v = s < a.S ? a.src[s] : ND_NULL_VERTEX;
    if (a.first_step == 0) {
        const bool bad = v >= a.V || v < ND_NULL_VERTEX;
        if (bad) v = ND_NULL_VERTEX;
        const int any = __syncthreads_or(bad ? 1 : 0);
        if (threadIdx.x == 0) publish_root_check(a, any);
    }
    return v;
}

// DeepWalk and PPR.  Many walks: bound by the scattered 128-byte fetches of the links (one per draw;
// the chip serves 5.5e10 of them per second whatever the array's size, once it exceeds L2).  Fewer: by the chain of a
// step, 0.27 us from L2 (0.18 with 16 lanes per walk).  While a link is on its way, the vertex of the step before is stored and the words of the
// next step are made; the assembler statement keeps the compiler (ROCm 7.2) from moving their making behind the wait for
// the link, where it and the acknowledged store were part of the chain (32,768 walks of 100 steps over 1.5 MB of
// links 37 us, like this 29; over 1.1 GB 72 and 60).
template <int DRAW, int STRIDE, typename OffT, int THREADS>
__global__ __launch_bounds__(THREADS) void walk_free_kernel(GraphView<OffT> g, FreeArgs a) {
    __shared__ uint32_t s_hist[kFreeChunk + 1];
    const uint32_t at = a.s_first + blockIdx.x * (uint32_t)THREADS + threadIdx.x;
    const uint32_t s = at < a.S ? at : a.S - 1u;  // lanes past the last sample walk and write with it
    int32_t v = first_transit<THREADS>(a, s);
    uint32_t rs = 0, deg = 0;
    if (v >= 0) {
        const uint64_t r = (uint64_t)g.off[v];
        rs = (uint32_t)r;
        deg = row_length(g, v, r);
    }
    const uint32_t sid = a.sample_base + s;
    uint32_t lived = 0;
    Rand4 r = draw4(a.seed, sid, 0u, a.first_step, 0u);
    CellWords cell{};
    for (uint32_t si = 0; si < a.n_steps; ++si) {
        lived += v >= 0 ? 1u : 0u;
        const bool draws = deg > 0u && !(a.ppr_thr != 0 && (uint64_t)r.r3 < a.ppr_thr);
        Link l;
        l.v = ND_NULL_VERTEX;
        l.rs = 0;
        l.deg = 0;
        if (draws) {
            if (DRAW == kDrawUniform) l = a.links[(uint64_t)(rs + mulhi32(r.r0, deg)) * STRIDE];
            else if (DRAW == kDrawCells) fetch_cell(cell, a.cells, rs, deg, r.r0);
            else l = drawn_link(a.links + (uint64_t)rs * 2u, deg, cat64(r.r0, r.r1));
        }
        const uint64_t word = cat64(r.r0, r.r1);
        if (si > 0) {  // after the load, which the next wait is for
            // Past the caches where walks are many.  Through them and past them, us: 4.2 M walks of 100 steps on R-MAT 22
            // 4,921 and 4,855, 300 K of 40 143 and 140; on R-MAT 16 300 K of 100 355 and 353.  Records read the steps
            // next, and find those of few outputs in the last-level cache: with them 600 K walks of 10 steps on R-MAT 16
            // 83.5 and 86.5, of 100 steps 815 and 811, on R-MAT 22 93.8 and 95.4, 860 and 847.  (A line by the volume of
            // the outputs gives up to 4 % to short walks with records and takes up to 2.5 % from walks without.)
            if (THREADS > 64) __builtin_nontemporal_store(v, &a.out[si - 1u][s]);
            else a.out[si - 1u][s] = v;
        }
        r = draw4(a.seed, sid, 0u, a.first_step + si + 1u, 0u);
        asm volatile("" : "+v"(r.r0), "+v"(r.r1), "+v"(r.r3));
        if (DRAW == kDrawCells) {
            const Link c = pick_link(cell, a.links, rs, deg, word, draws);
            l.v = draws ? c.v : ND_NULL_VERTEX;
            l.rs = c.rs;
            l.deg = draws ? c.deg : 0u;
        }
        v = l.v;
        rs = l.rs;
        deg = l.deg;
    }
    a.out[a.n_steps - 1u][s] = v;
    publish_live<THREADS>(at < a.S ? lived : 0u, a, s_hist);
}

// The value that lane I of every row of 16 lanes holds, in all of them.
template <int I>
__device__ __forceinline__ uint32_t from_lane(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x150 + I, 0xf, 0xf, true);  // row_newbcast
}

template <int... I, typename F>
__device__ __forceinline__ void unrolled(std::integer_sequence<int, I...>, F& f) {
    (f(std::integral_constant<int, I>{}), ...);
}

// DeepWalk and PPR where walks are few, so that the time is that of one walk: 16 lanes per walk.  The words of a
// step depend on nothing that the walk does, so each lane makes those of one step in 16, and all 16 lanes
// take the walk's step with them (same link, one fetch); what is left of a step's chain is the multiplication, the
// link's fetch and three selections: 0.18 us a step where L2 holds the links, 0.36 where the last-level cache does (26 MB of
// links), 0.51 over 1.1 GB (64 to 4,096 walks, another seed each call).  The words of the next 16 steps and
// the vertices of the last 16 leave while a link is on its way.  4,096 walks of 100 steps over 1.5 MB of links: 36.5 us
// with a lane per walk that made its words between two links, 18.3 like this.
template <int DRAW, int STRIDE, typename OffT>
__global__ __launch_bounds__(kFewThreads) void walk_free_few_kernel(GraphView<OffT> g, FreeArgs a) {
    __shared__ uint32_t s_hist[kFreeChunk + 1];
    constexpr int L = kFewLanes;
    static_assert(L == 16, "from_lane");
    const uint32_t k = threadIdx.x & (uint32_t)(L - 1);
    const uint32_t at = a.s_first + blockIdx.x * (uint32_t)(kFewThreads / L) + threadIdx.x / (uint32_t)L;
    const uint32_t s = at < a.S ? at : a.S - 1u;  // lanes past the last sample walk and write with it
    int32_t v = first_transit<kFewThreads>(a, s);
    uint32_t rs = 0, deg = 0;
    if (v >= 0) {
        const uint64_t r = (uint64_t)g.off[v];
        deg = row_length(g, v, r);
        rs = deg > 0u ? (uint32_t)r : 0u;  // a place inside the links, as a link has it
    }
    const uint32_t sid = a.sample_base + s;
    uint32_t lived = 0;
    int32_t mine = ND_NULL_VERTEX;                              // the vertex of step base + k
    Rand4 next = draw4(a.seed, sid, 0u, a.first_step + k, 0u);  // the words of step base + k
    CellWords cell{};
    uint32_t base = 0;
    for (;; base += (uint32_t)L) {
        const Rand4 r = next;
        uint32_t last = (uint32_t)L;                            // the walk stops before step base + last
        if (a.ppr_thr != 0) {
            const uint64_t stops = __ballot((uint64_t)r.r3 < a.ppr_thr) >> (threadIdx.x & 63u & ~(uint32_t)(L - 1));
            last = (uint32_t)__builtin_ctz((uint32_t)stops | (1u << L));
        }
        int32_t* const before = base > 0 ? a.out[base - (uint32_t)L + k] : nullptr;
        auto step = [&](auto index) {
            constexpr int I = decltype(index)::value;
            if (base + (uint32_t)I >= a.n_steps) return;  // the same for the whole launch
            lived += v >= 0 ? 1u : 0u;
            const bool draws = deg > 0u && (uint32_t)I < last;
            const uint32_t r0 = from_lane<I>(r.r0), r1 = DRAW == kDrawUniform ? 0u : from_lane<I>(r.r1);
            Link l;
            if (DRAW == kDrawUniform) {
                // a walk that has ended looks again where it stood: no branch on the way to the load
                l = a.links[(uint64_t)(rs + mulhi32(r0, deg)) * STRIDE];
            } else if (DRAW == kDrawCells) {
                if (draws) fetch_cell(cell, a.cells, rs, deg, r0);
            } else {
                l.v = ND_NULL_VERTEX;
                l.rs = l.deg = 0;
                if (draws) l = drawn_link(a.links + (uint64_t)rs * 2u, deg, cat64(r0, r1));
            }
            if (I == 0) {
                if (base > 0) before[s] = mine;
                next = draw4(a.seed, sid, 0u, a.first_step + base + (uint32_t)L + k, 0u);
                asm volatile("" : "+v"(next.r0), "+v"(next.r1), "+v"(next.r3));
            }
            if (DRAW == kDrawCells) l = pick_link(cell, a.links, rs, deg, cat64(r0, r1), draws);
            v = draws ? l.v : ND_NULL_VERTEX;
            rs = draws ? l.rs : rs;
            deg = draws ? l.deg : 0u;
            mine = k == (uint32_t)I ? v : mine;
        };
        unrolled(std::make_integer_sequence<int, L>{}, step);
        if (base + (uint32_t)L >= a.n_steps) break;
    }
    if (base + k < a.n_steps) a.out[base + k][s] = mine;
    publish_live<kFewThreads>(k == 0 && at < a.S ? lived : 0u, a, s_hist);
}

// ---------------------------------------------------------------- node2vec
// Is u in the row of t?  (rs, deg: where that row lies.)  One 16-byte fetch of the row's table as a rule.
template <typename OffT>
__device__ __forceinline__ bool row_has(const GraphView<OffT>& g, const int32_t* rowset, int32_t t, uint32_t rs,
                                        uint32_t deg, int32_t u) {
    if (rowset == nullptr) return row_contains(g, rs, deg, u);
    const int4* set = reinterpret_cast<const int4*>(rowset) + RowSet::first_group(t, rs);
    const uint32_t ng = RowSet::groups(rs, deg);
    uint32_t grp = mulhi32(RowSet::hash(u), ng);
    bool found = false, on = true;
    for (uint32_t probe = 0; on && probe < ng; ++probe) {
        const int4 x = set[grp];
        found = x.x == u || x.y == u || x.z == u || x.w == u;
        on = !found && x.w >= 0;  // a group fills from the front: if its last place is free, that was all
        grp = grp + 1u < ng ? grp + 1u : 0u;
    }
    return found;
}

// The exact draw after the last rejected attempt: inverse transform over the row's biased weights.  `exact`:
// this lane's walk needs one; returns the entry's place in the row.  All lanes of the wavefront call it.
// Rare where the biases are alike; where they are far apart (p = 0.05, q = 20) it is most of the time.  Lanes at their own pace come here one or two at a time, and a lane that goes through its row by
// itself keeps 63 others waiting, so the wavefront goes through one lane's row after the other, 256 entries
// at a time; what it has added up tells the stretch in which the draw ends, so only that is gone through
// again.  Where many lanes come at once and the longest of their rows has fewer entries than that takes
// steps, each lane does its own, and so does it in rows of up to four entries.  The sums are whole numbers: their
// order does not matter.  A row per lane, in windows, and like this: 57 K weighted walks of 20 steps, p = 0.05,
// q = 20, 87, 42 and 5.7 ms; 4 M walks of 5 steps, p = 0.25, q = 4, over the scale-22 R-MAT graph 101, 310 and
// 6.7 ms; 64 walks of 4 steps through a hub of a million entries one of which outweighs the rest 7.2, 1.0, 0.78 s.
__device__ __forceinline__ uint64_t lane_value(uint64_t x, int lane) {
    return cat64((uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), lane),
                 (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, lane));
}
__device__ __forceinline__ uint64_t wave_sum(uint64_t x) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
    return x;
}
template <typename OffT>
__device__ __forceinline__ uint32_t n2v_exact(const OffT* off, const int32_t* col, const uint32_t* wq, const int32_t* rowset,
                                           bool exact, uint64_t R, uint32_t b_ret, uint32_t b_com, uint32_t b_far,
                                           int32_t t, uint32_t rs_t, uint32_t deg_t, uint32_t rs, uint32_t deg) {
    constexpr uint32_t kPieces = 4u, kBlock = kPieces * 64u;  // entries per lane and step, entries per step
    uint32_t e = 0;
    const GraphView<OffT> g{off, col, nullptr, nullptr, nullptr, 0};
    auto bias = [&](int32_t u, int32_t prev, uint32_t prev_rs, uint32_t prev_deg) -> uint64_t {
        if (prev < 0) return kOneQ16;
        return u == prev ? b_ret : row_has(g, rowset, prev, prev_rs, prev_deg, u) ? b_com : b_far;
    };
    const int lane = lane_id();
    bool alone = __ballot(exact && deg > 4u) == 0ull;
    if (!alone) {
        uint32_t longest = exact ? deg : 0u;
        uint32_t steps = exact ? (deg >> 8) + 2u : 0u;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            const uint32_t o = (uint32_t)__shfl_xor((int)longest, d, 64);
            longest = o > longest ? o : longest;
            steps += (uint32_t)__shfl_xor((int)steps, d, 64);
        }
        alone = steps > longest;
    }
    if (alone) {
        if (exact) {
            auto biased = [&](uint32_t i) {
                const uint64_t at = (uint64_t)rs + i;
                return (wq != nullptr ? wq[at] : (uint64_t)kOneQ16) * bias(col[at], t, rs_t, deg_t);
            };
            uint64_t Z = 0, run = 0;
            for (uint32_t i = 0; i < deg; ++i) Z += biased(i);
            const uint64_t x = mulhi64(R, Z);
            for (e = 0; e + 1u < deg; ++e) {
                run += biased(e);
                if (run > x) break;
            }
        }
        return e;
    }
    for (uint64_t need = __ballot(exact); need != 0ull; need &= need - 1ull) {
        const int who = __builtin_ctzll(need);
        const int32_t p_t = __builtin_amdgcn_readlane(t, who);
        const uint32_t p_rs_t = (uint32_t)__builtin_amdgcn_readlane((int)rs_t, who);
        const uint32_t p_deg_t = (uint32_t)__builtin_amdgcn_readlane((int)deg_t, who);
        const uint32_t p_rs = (uint32_t)__builtin_amdgcn_readlane((int)rs, who);
        const uint32_t p_deg = (uint32_t)__builtin_amdgcn_readlane((int)deg, who);
        uint64_t w[kPieces];
        auto take_block = [&](uint32_t base) {  // my entries of a block: base + 64 p + lane
            int32_t u[kPieces];
#pragma unroll
            for (uint32_t p = 0; p < kPieces; ++p) {
                const uint32_t i = base + p * 64u + (uint32_t)lane;
                u[p] = ND_NULL_VERTEX;
                w[p] = 0;
                if (i < p_deg) {
                    const uint64_t at = (uint64_t)p_rs + i;
                    u[p] = col[at];
                    w[p] = wq != nullptr ? wq[at] : kOneQ16;
                }
            }
#pragma unroll
            for (uint32_t p = 0; p < kPieces; ++p)
                if (u[p] >= 0) w[p] *= bias(u[p], p_t, p_rs_t, p_deg_t);
        };
        // 64 stretches of whole blocks; lane k keeps the sum of stretch k
        const uint32_t blocks = (p_deg + kBlock - 1u) / kBlock;
        const uint32_t stretch = (blocks + 63u) / 64u * kBlock;
        uint64_t mine = 0;
        int k = 0;
        for (uint32_t lo = 0; lo < p_deg; ++k) {
            const uint32_t hi = p_deg - lo > stretch ? lo + stretch : p_deg;
            uint64_t sum = 0;
            for (; lo < hi; lo += kBlock) {
                take_block(lo);
                sum += w[0] + w[1] + w[2] + w[3];
            }
            sum = wave_sum(sum);
            if (lane == k) mine = sum;
        }
        const uint64_t through = wave_inclusive_scan(mine, lane);
        const uint64_t x = mulhi64(lane_value(R, who), lane_value(through, 63));
        const uint64_t past = __ballot(through > x);
        uint32_t found = p_deg - 1u;  // where no weight is left, as for a row that a lane goes through
        if (past != 0ull) {
            const int in = __builtin_ctzll(past);
            uint64_t run = lane_value(through, in) - lane_value(mine, in);
            bool more = true;
            for (uint32_t lo = (uint32_t)in * stretch; more; lo += kBlock) {  // ends: the stretch's sum exceeds x
                if (blocks > 1u) {  // one block: still in registers
                    take_block(lo);
                    const uint64_t all = wave_sum(w[0] + w[1] + w[2] + w[3]);
                    if (run + all <= x) {
                        run += all;
                        continue;
                    }
                }
                more = false;
                bool open = true;
#pragma unroll
                for (uint32_t p = 0; p < kPieces; ++p) {
                    const uint64_t incl = run + wave_inclusive_scan(w[p], lane);
                    const uint64_t hit = __ballot(incl > x);
                    if (open && hit != 0ull) {
                        found = lo + p * 64u + (uint32_t)__builtin_ctzll(hit);
                        open = false;
                    }
                    run = lane_value(incl, 63);
                }
            }
        }
        if (lane == who) e = found;
    }
    return e;
}

// Out of line for workgroups of one wavefront (at most 65,536 walks, of which a SIMD has one wavefront or two), inlined
// for many walks (61 to 63 registers, 86 to 94 out of line: 7 wavefronts per SIMD instead of 5).  100 weighted steps,
// out of line and inlined, us: p = 2, q = 0.5, 57 K walks on 1.6 M entries 262 and 262, on 38 M 338 and 337; p = 0.25, q = 4,
// whose attempts are often used up, 4,439 and 4,361, 10,133 and 9,994.  Many walks, out of line
// and inlined: a million of 10 steps on 38 M entries 549 and 554, of 20 steps without weights 511 and 515.
template <typename OffT>
__device__ __noinline__ uint32_t n2v_exact_call(const OffT* off, const int32_t* col, const uint32_t* wq,
                                                const int32_t* rowset, bool exact, uint64_t R, uint32_t b_ret,
                                                uint32_t b_com, uint32_t b_far, int32_t t, uint32_t rs_t, uint32_t deg_t,
                                                uint32_t rs, uint32_t deg) {
    return n2v_exact(off, col, wq, rowset, exact, R, b_ret, b_com, b_far, t, rs_t, deg_t, rs, deg);
}

// Every walk goes through its attempts at its own pace: a wavefront whose lanes wait for each other at every step
// pays for the slowest of 64 geometrically distributed attempt counts (7 rounds per step where the mean is 1.9).
// A round is one fetch: of the candidate's link or, where the two biases differ in their verdict on the candidate before,
// of a group of the previous vertex's table; both are 16 bytes, and a lane that looks into a table does not keep the
// others from their links.  While it is on its way, the generator makes the words of both possible next attempts and the
// vertex that was taken last is stored; the assembler statements keep the compiler (ROCm 7.2) from making the words
// after the wait.  100 steps, p = 2, q = 0.5, weights in [1, 5): 57 K walks on 1.6 M entries 417 us with the table asked in
// the attempt's own round and everything after the wait, 327 with rounds of one fetch, 264 with the words made
// meanwhile (rounds of about 1.1 us, one wavefront per SIMD; 13 M fetches would take 0.2 ms at the rate of
// scattered fetches); 57 K walks on 39 M entries 644 and 347.
// LANES lanes per walk make as many attempts at once, of which the first that is not refused counts (walks are few, and a
// step is as long as its attempts; the rule stands at attempt_lanes).
typedef __attribute__((address_space(1))) int32_t GlobalInt;  // what lies behind a pointer that was read from LDS
template <int STRIDE, typename OffT, int THREADS, int LANES>
__global__ __launch_bounds__(THREADS) void walk_free_n2v_kernel(GraphView<OffT> g, FreeArgs a) {
    __shared__ uint32_t s_hist[kFreeChunk + 1];
    __shared__ int32_t* s_out[kFreeChunk];
    constexpr uint32_t kWalks = (uint32_t)(THREADS / LANES);
    const uint32_t k = threadIdx.x % (uint32_t)LANES;
    const int walk = (int)(threadIdx.x & 63u) - (int)k;  // the wavefront's lane that is my walk's first
    const uint32_t s = a.s_first + blockIdx.x * kWalks + threadIdx.x / (uint32_t)LANES;
    for (uint32_t i = threadIdx.x; i < a.n_steps; i += THREADS) s_out[i] = a.out[i];
    int32_t v = first_transit<THREADS>(a, s);
    __syncthreads();
    uint32_t rs = 0, deg = 0, maxw = kOneQ16;
    int32_t t = ND_NULL_VERTEX;        // the transit before v: none at the first step
    uint32_t rs_t = 0, deg_t = 0;
    if (v >= 0) {
        const uint64_t r = (uint64_t)g.off[v];
        rs = (uint32_t)r;
        deg = row_length(g, v, r);
        if (a.use_weights) maxw = g.maxwq[v];
        if (a.first_step > 0) {
            t = a.prev_src[s];
            const uint64_t rt = (uint64_t)g.off[t];
            rs_t = (uint32_t)rt;
            deg_t = row_length(g, t, rt);
        }
    }
    const uint32_t sid = a.sample_base + s;
    const uint32_t b_lo = a.b_com < a.b_far ? a.b_com : a.b_far, b_hi = a.b_com < a.b_far ? a.b_far : a.b_com;
    const bool common_high = a.b_com > a.b_far;
    uint32_t si = 0;
    int32_t att = 0;                   // the attempt of my walk's first lane
    Rand4 r = draw4(a.seed, sid, 0u, a.first_step, k);
    enum : uint32_t { kTry, kAsk, kTake, kNo };
    uint32_t what = kTry;              // my attempt: to be made; its verdict needs the table; accepted; refused
    Link cand{};
    uint32_t cand_top = kOneQ16, grp = 0, probe = 0;
    uint32_t stores = 0;               // a vertex taken, not stored yet
    GlobalInt* store_at = nullptr;
    int32_t store_v = 0;
    for (;;) {
        while (si < a.n_steps && deg > 0u) {  // deg is 0 for a walk that has ended
            if (__ballot(att >= a.max_attempts) != 0ull) break;  // the wavefront leaves: a walk's attempts are used up
            const uint32_t ng = RowSet::groups(rs_t, deg_t);
            const Words4* link_at = reinterpret_cast<const Words4*>(a.links + (uint64_t)(rs + mulhi32(r.r0, deg)) * STRIDE);
            const Words4* set_at = reinterpret_cast<const Words4*>(a.rowset) + (RowSet::first_group(t, rs_t) + grp);
            const Words4* at = what == kAsk ? set_at : link_at;
            Words4 got = *at;
            uint32_t top = 0;
            if (STRIDE == 2) top = reinterpret_cast<const uint32_t*>(at)[what == kAsk ? 0 : 7];
            if (stores != 0u) *store_at = store_v;
            Rand4 onward = draw4(a.seed, sid, 0u, a.first_step + si + 1u, k);
            Rand4 again = r;
            if (LANES == 1) again = draw4(a.seed, sid, 0u, a.first_step + si, (uint32_t)att + 1u);
            const bool start = t < 0;
            uint64_t y = mulhi64(cat64(r.r1, r.r2), (uint64_t)maxw * (start ? kOneQ16 : a.b_max));
            store_at = (GlobalInt*)s_out[si] + s;
            asm volatile("" : "+v"(onward.r0), "+v"(onward.r1), "+v"(onward.r2), "+v"(y));
            if (LANES == 1) asm volatile("" : "+v"(again.r0), "+v"(again.r1), "+v"(again.r2));
            asm volatile("" : "+v"(got), "+v"(top));
            const int4 x = make_int4((int)got.x, (int)got.y, (int)got.z, (int)got.w);
            // The verdict and the move to the next vertex are selections, not branches.  From a nest of branches that
            // said the same, the compiler (ROCm 7.2, -O3) made code in which the registers of the link's row and length
            // took the weight and the envelope; compiled for the CPU, under sanitizers, both forms gave the oracle's walks.
            const bool back = x.x == t;
            const uint64_t w = a.use_weights ? (uint32_t)x.w : kOneQ16;
            // a row of one entry has one outcome, whatever its attempts say
            const bool low = deg == 1u || y < w * (start ? kOneQ16 : back ? a.b_ret : b_lo);
            const bool high = !start && !back && y < w * b_hi;  // between the biases: accepted if it has the higher one
            // a table's group: found, or not to be found, or in the next group (a group fills from the front)
            const bool found = x.x == cand.v || x.y == cand.v || x.z == cand.v || x.w == cand.v;
            const bool more = !found && x.w >= 0 && probe + 1u < ng;
            const bool tries = what == kTry;
            cand.v = tries ? x.x : cand.v;
            cand.rs = tries ? (uint32_t)x.y : cand.rs;
            cand.deg = tries ? (uint32_t)x.z : cand.deg;
            if (STRIDE == 2) cand_top = tries ? (a.use_weights ? top & 0x7FFFFFFFu : kOneQ16) : cand_top;
            const uint32_t first = LANES > 1 && att + (int32_t)k >= a.max_attempts ? kNo : low ? kTake : high ? kAsk : kNo;
            const uint32_t then = more ? kAsk : found == common_high ? kTake : kNo;
            grp = tries ? mulhi32(RowSet::hash(cand.v), ng) : grp + 1u < ng ? grp + 1u : 0u;
            probe = tries ? 0u : probe + 1u;
            what = tries ? first : what == kAsk ? then : what;
            if (a.rowset == nullptr && what == kAsk)
                what = row_contains(g, rs_t, deg_t, cand.v) == common_high ? kTake : kNo;
            bool moves = what == kTake, refused = what == kNo;
            Link to = cand;
            uint32_t to_top = cand_top;
            if (LANES > 1) {  // the first lane that has not been refused speaks for the walk, once it knows
                constexpr uint32_t kAll = (1u << LANES) - 1u;
                const uint32_t open = (uint32_t)(__ballot(what != kNo) >> walk) & kAll;
                const uint32_t taken = (uint32_t)(__ballot(what == kTake) >> walk) & kAll;
                const int from = walk + (int)__builtin_ctz(open | (1u << LANES));  // none: not used
                refused = open == 0u;
                moves = (open & (0u - open) & taken) != 0u;
                to.v = __shfl(cand.v, from, 64);
                to.rs = (uint32_t)__shfl((int)cand.rs, from, 64);
                to.deg = (uint32_t)__shfl((int)cand.deg, from, 64);
                if (STRIDE == 2) to_top = (uint32_t)__shfl((int)cand_top, from, 64);
                if (refused) again = draw4(a.seed, sid, 0u, a.first_step + si, (uint32_t)att + (uint32_t)LANES + k);
            }
            store_v = to.v;
            stores = moves && k == 0u ? 1u : 0u;
            t = moves ? v : t;
            rs_t = moves ? rs : rs_t;
            deg_t = moves ? deg : deg_t;
            v = moves ? to.v : v;
            rs = moves ? to.rs : rs;
            deg = moves ? to.deg : deg;
            maxw = moves ? to_top : maxw;
            si += moves ? 1u : 0u;
            att = moves ? 0 : refused ? att + LANES : att;
            r.r0 = moves ? onward.r0 : refused ? again.r0 : r.r0;
            r.r1 = moves ? onward.r1 : refused ? again.r1 : r.r1;
            r.r2 = moves ? onward.r2 : refused ? again.r2 : r.r2;
            what = moves || refused ? (uint32_t)kTry : what;
        }
        if (stores != 0u) *store_at = store_v;
        stores = 0;
        const bool ends = si < a.n_steps && deg > 0u && att >= a.max_attempts, exact = ends && k == 0u;
        if (__ballot(ends) == 0ull) break;  // every walk of the wavefront is done
        if (LANES > 1 && ends) r = draw4(a.seed, sid, 0u, a.first_step + si, (uint32_t)a.max_attempts);
        const uint32_t* wq = a.use_weights ? g.wq : nullptr;
        const uint64_t word = cat64(r.r0, r.r1);
        uint32_t e = THREADS == 64 ? n2v_exact_call(g.off, g.col, wq, a.rowset, exact, word, a.b_ret, a.b_com,
                                                          a.b_far, t, rs_t, deg_t, rs, deg)
                                         : n2v_exact(g.off, g.col, wq, a.rowset, exact, word, a.b_ret, a.b_com, a.b_far,
                                                     t, rs_t, deg_t, rs, deg);
        if (LANES > 1) e = (uint32_t)__shfl((int)e, walk, 64);
        if (ends) {
            const Link* at = a.links + (uint64_t)(rs + e) * STRIDE;
            const Link l = *at;
            if (STRIDE == 2 && a.use_weights) maxw = reinterpret_cast<const WeightLink*>(at)[1].top & 0x7FFFFFFFu;
            if (k == 0u) s_out[si][s] = l.v;
            t = v;
            rs_t = rs;
            deg_t = deg;
            v = l.v;
            rs = l.rs;
            deg = l.deg;
            ++si;
            att = 0;
            r = draw4(a.seed, sid, 0u, a.first_step + si, k);
        }
    }
    // a walk that stands on a vertex without out-edges had a transit at this step still
    const uint32_t lived = si + (si < a.n_steps && v >= 0 ? 1u : 0u);
    if (s < a.S)
        for (si += k; si < a.n_steps; si += (uint32_t)LANES) s_out[si][s] = ND_NULL_VERTEX;
    publish_live<THREADS>(k == 0u ? lived : 0u, a, s_hist);
}

// ---------------------------------------------------------------- multi-dimensional walk
// A sample's steps depend on each other only through the root they pick, and which root a step picks
// comes from the generator alone.  So a wavefront takes a sample and 64 of its steps at a time, one per
// lane: a step that picks a root no earlier one of the 64 picked reads it from the sample's roots
// in LDS, the others wait for the last earlier step with the same root - two to four rounds for 64 steps
// and 100 roots, where step after step is 64 chains of three dependent fetches.
// Many samples are bound by the rate of scattered requests to memory (41,943 samples of 100 roots and steps on R-MAT 22:
// 5.6 M of them in 116 us, two in three for the offsets of a root's row).  KEEP: later steps find the rows of roots that
// earlier ones moved in LDS (108 us).  FILLED: a bit per vertex, which the L2s hold, says which rows are empty (97 us).
// All 100 steps at once, two per lane, took 110: more instructions per round.
template <int STRIDE, typename OffT, int WAVES, bool KEEP, bool FILLED = false>
__global__ __launch_bounds__(WAVES * 64) void mrw_free_kernel(GraphView<OffT> g, FreeArgs a) {
    extern __shared__ uint32_t s_dyn[];
    constexpr uint32_t T = WAVES * 64;
    __shared__ int32_t s_tile[64][WAVES + 1];
    __shared__ uint32_t s_live[kFreeChunk];
    const uint32_t R = a.R;
    const uint32_t wave = wave_uniform((uint32_t)wave_id());
    const int lane = lane_id();
    int32_t* state = (int32_t*)s_dyn + wave * R * (KEEP ? 5u : 3u);  // the roots of my sample
    uint32_t* picked = (uint32_t*)state + R;           // per root: which of the 64 steps pick it (two words)
    uint32_t* rows = picked + 2u * R;                  // KEEP: the root's row, its length kUnknown until a step has looked
    constexpr uint32_t kUnknown = 0xFFFFFFFFu;         // a row has fewer than 2^31 entries
    const uint32_t s0 = a.s_first + blockIdx.x * WAVES, s = s0 + wave;
    const bool mine = s < a.S;
    bool bad = false;
    for (uint32_t i = (uint32_t)lane; i < R; i += 64u) {
        int32_t v = ND_NULL_VERTEX;
        if (mine) {
            v = a.src[(uint64_t)s * R + i];
            if (v >= a.V || v < ND_NULL_VERTEX) {
                bad = true;
                v = ND_NULL_VERTEX;
            }
        }
        state[i] = v;
        picked[2u * i] = 0u;
        picked[2u * i + 1u] = 0u;
        if (KEEP) rows[2u * i + 1u] = kUnknown;
    }
    for (uint32_t i = threadIdx.x; i < (uint32_t)kFreeChunk; i += T) s_live[i] = 0;
    const int any_bad = __syncthreads_or(bad ? 1 : 0);
    if (threadIdx.x == 0 && a.first_step == 0) publish_root_check(a, any_bad);
    for (uint32_t base = 0; base < a.n_steps; base += 64u) {
        const uint32_t si = base + (uint32_t)lane;
        const bool step = mine && si < a.n_steps;
        const Rand4 r = draw4(a.seed, a.sample_base + s, 0u, a.first_step + si, 0u);
        const uint32_t pick = mulhi32(r.r2, R);
        if (step) atomicOr(&picked[2u * pick + ((uint32_t)lane >> 5)], 1u << (lane & 31));
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const uint64_t same = step ? cat64(picked[2u * pick + 1u], picked[2u * pick]) : 0ull;
        const uint64_t before = same & lanes_below(lane);
        const int pred = before ? 63 - __clzll((long long)before) : -1;
        // the root as I leave it (vertex, row); the first step of a root starts from the sample's
        int32_t av = ND_NULL_VERTEX, added = ND_NULL_VERTEX;
        uint32_t ars = 0, adeg = 0;
        if (step && pred < 0) {
            av = state[pick];
            adeg = KEEP ? rows[2u * pick + 1u] : kUnknown;
            if (adeg != kUnknown) {
                ars = rows[2u * pick];
            } else {
                adeg = 0u;
                if (av >= 0 && (!FILLED || ((a.filled[(uint32_t)av >> 6] >> (av & 63)) & 1ull) != 0ull)) {
                    const uint64_t rs = (uint64_t)g.off[av];
                    ars = (uint32_t)rs;
                    adeg = row_length(g, av, rs);
                }
            }
        }
        bool had = false;
        bool done = !step;
        for (uint64_t all_done = __ballot(done); all_done != ~0ull; all_done = __ballot(done)) {
            const bool go = !done && (pred < 0 || ((all_done >> (pred & 63)) & 1ull) != 0ull);
            const int from = pred < 0 ? lane : pred;
            const int32_t pv = __shfl(av, from, 64);
            const uint32_t prs = (uint32_t)__shfl((int)ars, from, 64), pdeg = (uint32_t)__shfl((int)adeg, from, 64);
            if (go) {
                had = pv >= 0;
                av = pv;
                ars = prs;
                adeg = pdeg;
                if (adeg > 0u) {
                    const Link l = a.links[(uint64_t)(ars + mulhi32(r.r0, adeg)) * STRIDE];
                    added = av = l.v;
                    ars = l.rs;
                    adeg = l.deg;
                }
                done = true;
            }
        }
        if (step) {
            if ((same >> lane) == 1ull) {  // the last of the 64 steps that picked this root
                state[pick] = av;
                if (KEEP) {
                    rows[2u * pick] = ars;
                    rows[2u * pick + 1u] = adeg;
                }
            }
            picked[2u * pick] = 0u;
            picked[2u * pick + 1u] = 0u;
            if (had) atomicAdd(&s_live[si], 1u);
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        s_tile[lane][wave] = added;
        __syncthreads();
        // the samples of the workgroup are neighbours in every step's output
        for (uint32_t i = threadIdx.x; i < 64u * WAVES; i += T) {
            const uint32_t row = i / WAVES, w = i % WAVES;
            if (base + row < a.n_steps && s0 + w < a.S) a.out[base + row][s0 + w] = s_tile[row][w];
        }
        __syncthreads();
    }
    uint32_t* parts = a.parts + (uint64_t)blockIdx.x * a.total_steps + a.first_step;
    for (uint32_t i = threadIdx.x; i < a.n_steps; i += T) parts[i] = (a.s_first > 0 ? parts[i] : 0u) + s_live[i];
    if (a.state != nullptr && mine)  // more steps follow in another launch
        for (uint32_t i = (uint32_t)lane; i < R; i += 64u) a.state[(uint64_t)s * R + i] = state[i];
}

// Samples (wavefronts) per workgroup: sixteen, whose outputs then leave in runs of 64 bytes, as long as
// their roots fit 48 KB of LDS (two workgroups per compute unit and room for a third).  20,000 samples of 100 steps
// with one, four and sixteen: 75, 60 and 59 us with 100 roots each, 80, 67 and 63 with 256; up to 5,000 samples
// they are alike.
int mrw_waves(uint32_t R) { return R <= 256u ? 16 : R <= 1024u ? 4 : 1; }

// Later steps of a launch find rows in LDS that earlier ones left: a second round of 64 steps, and LDS for the rows, no
// more than the roots alone may take (154 to 256 roots per sample pass that; rows in more LDS have not been timed).
constexpr size_t kMrwLds = 48 << 10;
size_t mrw_keep_lds(int waves, uint32_t R) { return (size_t)waves * R * 20; }
bool mrw_may_keep_rows(int32_t n_steps, uint32_t R) { return n_steps > 64 && mrw_keep_lds(mrw_waves(R), R) <= kMrwLds; }

int64_t offsets_bytes(const Graph& gr) { return gr.V * (gr.off64 ? 8 : 4); }

// ... and is the faster for it where the offsets are what an L2 holds or more, and the second round is half full.  Time
// without over time with kept rows, 100 roots, 16 to 41,943 samples: 70 steps 0.97 to 1.00 on seven graphs of 0.2 to 33 MB
// of offsets, 80 steps 0.97 to 1.02, 96 0.98 to 1.05, 100 0.97 to 1.08, 128 1.00 to 1.09 (from 8,192 samples and 4 MB on
// 96 1.01 to 1.05, 100 1.02 to 1.08); offsets of 0.2 and 1 MB 0.97 to 0.99 at 30 and 100 roots and any number of steps
// (4 roots 1.00 to 1.02), of 2 MB 0.98 to 1.02.
bool mrw_keeps_rows(const Graph& gr, int32_t n_steps, uint32_t R) {
    return mrw_may_keep_rows(n_steps, R) && n_steps >= 96 && offsets_bytes(gr) >= (4 << 20);
}

template <int WAVES, typename OffT>
void launch_mrw(const Graph& gr, const FreeArgs& a, uint32_t groups, hipStream_t stream) {
    const dim3 grid(groups), block(WAVES * 64);
    const size_t lds = (size_t)WAVES * a.R * 12;  // within kMrwLds
    const bool filled = a.filled != nullptr && mrw_may_keep_rows((int32_t)a.n_steps, a.R);
    const bool keep = filled || mrw_keeps_rows(gr, (int32_t)a.n_steps, a.R);
    const GraphView<OffT> g = view_of<OffT>(gr);
#define ND_MRW_LAUNCH(STRIDE)                                                                             \
    do {                                                                                                  \
        auto* kernel = filled ? &mrw_free_kernel<STRIDE, OffT, WAVES, true, true>                         \
                       : keep ? &mrw_free_kernel<STRIDE, OffT, WAVES, true>                               \
                              : &mrw_free_kernel<STRIDE, OffT, WAVES, false>;                             \
        hipLaunchKernelGGL(kernel, grid, block, keep ? mrw_keep_lds(WAVES, a.R) : lds, stream, g, a);       \
    } while (0)
    if (gr.wq) ND_MRW_LAUNCH(2);
    else ND_MRW_LAUNCH(1);
#undef ND_MRW_LAUNCH
}

template <typename OffT>
void launch_few(const Graph& gr, int draw, const FreeArgs& a, uint32_t groups, hipStream_t stream) {
    const dim3 grid(groups), block(kFewThreads);
    const GraphView<OffT> g = view_of<OffT>(gr);
    if (draw == kDrawWeighted && a.cells)
        hipLaunchKernelGGL((walk_free_few_kernel<kDrawCells, 2, OffT>), grid, block, 0, stream, g, a);
    else if (draw == kDrawWeighted)
        hipLaunchKernelGGL((walk_free_few_kernel<kDrawWeighted, 2, OffT>), grid, block, 0, stream, g, a);
    else if (gr.wq)
        hipLaunchKernelGGL((walk_free_few_kernel<kDrawUniform, 2, OffT>), grid, block, 0, stream, g, a);
    else
        hipLaunchKernelGGL((walk_free_few_kernel<kDrawUniform, 1, OffT>), grid, block, 0, stream, g, a);
}

template <int THREADS, int LANES, typename OffT>
void launch_n2v_shape(const Graph& gr, const FreeArgs& a, uint32_t groups, hipStream_t stream) {
    const dim3 grid(groups), block(THREADS);
    const GraphView<OffT> g = view_of<OffT>(gr);
    if (gr.wq) hipLaunchKernelGGL((walk_free_n2v_kernel<2, OffT, THREADS, LANES>), grid, block, 0, stream, g, a);
    else hipLaunchKernelGGL((walk_free_n2v_kernel<1, OffT, THREADS, LANES>), grid, block, 0, stream, g, a);
}
template <typename OffT>
void launch_n2v(const Graph& gr, const FreeArgs& a, int lanes, int64_t walks_per_group, uint32_t groups,
                hipStream_t stream) {
    if (lanes > 1) launch_n2v_shape<64, kAttemptLanes, OffT>(gr, a, groups, stream);
    else if (walks_per_group == 64) launch_n2v_shape<64, 1, OffT>(gr, a, groups, stream);
    else launch_n2v_shape<256, 1, OffT>(gr, a, groups, stream);
}

template <int THREADS, typename OffT>
void launch_free(const Graph& gr, int draw, const FreeArgs& a, uint32_t groups, hipStream_t stream) {
    const dim3 grid(groups), block(THREADS);
    const GraphView<OffT> g = view_of<OffT>(gr);
    if (draw == kDrawWeighted && a.cells)
        hipLaunchKernelGGL((walk_free_kernel<kDrawCells, 2, OffT, THREADS>), grid, block, 0, stream, g, a);
    else if (draw == kDrawWeighted)
        hipLaunchKernelGGL((walk_free_kernel<kDrawWeighted, 2, OffT, THREADS>), grid, block, 0, stream, g, a);
    else if (gr.wq)
        hipLaunchKernelGGL((walk_free_kernel<kDrawUniform, 2, OffT, THREADS>), grid, block, 0, stream, g, a);
    else
        hipLaunchKernelGGL((walk_free_kernel<kDrawUniform, 1, OffT, THREADS>), grid, block, 0, stream, g, a);
}

}  // namespace

// One walk per lane, and a workgroup of one wavefront as long as that gives every compute unit at
// most a few of them: a workgroup of four starts and ends later than its wavefronts would.  20 steps on R-MAT 22, one
// wavefront and four, us: 16,384 walks of DeepWalk 10.3 and 11.5, of node2vec 33.8 and 35.4; 65,536 17.3 and 17.1, 38.9 and
// 38.4.  More walks take workgroups of four, which have fewer headers and counters to write: a million of DeepWalk 261 and
// 254, of PPR 239 and 232 (node2vec 506 and 515).
static int free_threads(int64_t S) { return S <= 65536 ? 64 : 256; }

// DeepWalk and PPR up to this many walks: sixteen lanes per walk (walk_free_few_kernel).  100 steps, sixteen lanes and
// one, us: over links that L2 holds (1.5 MB) 18.6 and 28.1 for 4,096 walks, 20.8 and 28.4 for 8,192, 25.6 and 28.9 for
// 16,384, 39 and 29 for 32,768; over 1.1 GB 18.3 and 27.4 for 1,024, 34 and 39 for 4,096, 38.1 and 39.5 for 8,192,
// 42.6 and 40.8 for 16,384 (calls repeated with one seed, whose links the caches then hold).  Over weights, PPR at 0.01 by the cells: 1.6 M entries, weights in [1, 5), 30.5 and 37.8 for
// 1,024, 51.8 and 54.3 for 8,192, 57.0 and 55.2 for 16,384, 123 and 63 for 32,768; symmetric weights, whose draws search
// more often, 64.6 and 86.2 for 8,192, 71 and 86 for 16,384, 139 and 103 for 32,768.
constexpr int64_t kFewWalks = 8192;

// Whether weighted walks draw from the cells.  One fetch of 64 bytes per entry stands against two of 32, so a graph's
// cells pass sooner what the chip translates addresses of at once: from 4 GB on the scattered fetches of many walks
// come at 2e10 a second instead of 4e10, and the two fetches of a draw over the links, which lie in one row, are
// faster.  100 steps of DeepWalk, weights in [1, 5), links and cells, us: 600 K walks on 52 M entries 1.26 times as fast by
// the cells, on 66 M 1.01, on 82 M 0.94, on 117 M (7.5 GB) 2,692 and 2,941; 20 steps of PPR over symmetric weights 1.04,
// 0.89, 0.87 and 0.75 (445 and 590).  Walks of which most have ended (100 steps of PPR at 0.01) gain longer: 1.35 on 66 M
// and 1.16 on 117 M over weights in [1, 5), 1.24 and 0.92 over symmetric ones.  Up to 32,768 walks a call is a chain of
// fetches, and shorter by the cells at every size up to 412 M entries (26 GB): 8,192 walks 137 and 57 us, 32,768 on 102 M
// entries 1.05 to 2.07 times as fast; 57,000 0.86 to 1.6.
constexpr uint64_t kCellsReach = 7ull << 29;
constexpr int64_t kCellsWalks = 32768;
bool walk_uses_cells(const Graph& gr, int64_t S) {
    return S <= kCellsWalks || (uint64_t)gr.E * sizeof(WeightCell) <= kCellsReach;
}

// Attempts at once (lanes per walk) of a node2vec call: several where walks are few and an attempt is refused more often
// than one time in four, estimated as if every neighbour were far and weighed 0.6 of its row's heaviest.  100 steps,
// four lanes and one, us, weights in [1, 5), p = 2, q = 0.5: 57 K vertices 110 and 154 for 64 walks, 154 and 184 for
// 8,192, 160 and 187 for 16,384, 261 and 206 for 32,768; 1 M vertices 195 and 220 for 8,192, 222 and 244 for 16,384, 346
// and 280 for 32,768.  Without weights (one refused in fifty) 134 and 115 for 1,024, 149 and 127 for 16,384.
// Eight lanes: 150 for 8,192 walks, 201 for 16,384.
constexpr int64_t kFewAttemptWalks = 16384;
static int attempt_lanes(int64_t S, const DrawArgs& d) {
    const double accepted = (double)d.b_far / (double)d.b_max * (d.use_weights ? 0.6 : 1.0);
    return S <= kFewAttemptWalks && accepted < 0.75 ? kAttemptLanes : 1;
}

// Whether rows are looked up in the bits first: each empty row then costs no fetch, each other one a look more.  The more
// roots a sample has the more of its looks go past the kept rows, and the fewer empty rows it takes.  Time without
// over time with bits, 100 steps, 8, 16 and 32 MB of offsets, 8,192, 12,000 and 41,943 samples:
//   empty rows   30 %          35 %          40 %          45 %          50 %          70 %
//   16 roots     0.98 to 1.01  0.99 to 1.01  0.99 to 1.01  0.99 to 1.02  0.99 to 1.02  1.00 to 1.04
//   30 roots     0.98 to 1.00  0.99 to 1.01  0.99 to 1.02  1.00 to 1.02  1.00 to 1.03  1.04 to 1.10
//   60 roots     0.98 to 1.02  0.99 to 1.03  1.00 to 1.04  1.02 to 1.07  1.04 to 1.08  1.09 to 1.16
//   100 roots    0.99 to 1.03  1.00 to 1.05  1.01 to 1.07  1.03 to 1.08  1.05 to 1.10  1.12 to 1.21
//   150 roots    0.99 to 1.05  1.01 to 1.07  1.02 to 1.09  1.04 to 1.12  1.06 to 1.13  1.15 to 1.25
// R-MAT 22 (47 %), 100 roots: 8,192 samples 1.13, 41,943 1.12 (70 steps, against none kept, 1.10 and 1.08), 4,000 1.03, 1,000
// 0.96.  Half of the rows empty, 4 MB 1.02 to 1.10, 2 MB 0.98 to 1.09.
bool mrw_reads_filled(const Graph& gr, int64_t S, int32_t num_steps, uint32_t R) {
    return R >= 30u && mrw_may_keep_rows(num_steps, R) && S >= 8192 && offsets_bytes(gr) >= (8 << 20) &&
           700 * gr.empty_rows >= (int64_t)(345u - (R < 150u ? R : 150u)) * gr.V;
}

// Walks per workgroup; lanes: attempts at once of a node2vec call, 0 for the others.
static int64_t samples_per_group(int64_t S, int lanes, uint32_t mrw_R) {
    if (mrw_R > 0) return mrw_waves(mrw_R);
    if (lanes > 1) return 64 / lanes;
    return lanes == 0 && S <= kFewWalks ? kFewThreads / kFewLanes : free_threads(S);
}

// Bytes of the workspace that hold a multi-dimensional walk's roots between two launches.
int64_t walk_free_state_bytes(int64_t S, int32_t num_steps, uint32_t mrw_R) {
    return num_steps > kFreeChunk ? S * (int64_t)mrw_R * 4 : 0;
}

// Workgroups per launch, at most (node2vec may take fewer: its scratch does not depend on its biases).  Each owns a
// flag and a counter per step of the call in the workspace; samples
// beyond what these workgroups take go to further launches.  24 MB of counters are 62,000 workgroups (15.9 M
// walks) of 100 steps, or 1,535 of the 4,096 steps that a call may have.  No call may need more of the
// static scratch array than walks whose scratch is a control block (64 bytes) per step, the roots and a
// transit per sample of the multi-dimensional walk, so beside many roots the counters take what those took.
int64_t walk_free_groups(int64_t S, int32_t num_steps, bool node2vec, uint32_t mrw_R) {
    const int lanes = !node2vec ? 0 : S <= kFewAttemptWalks ? kAttemptLanes : 1;
    const int64_t per = samples_per_group(S, lanes, mrw_R), k = num_steps;
    int64_t room = (24ll << 20) - walk_free_state_bytes(S, num_steps, mrw_R);
    const int64_t least = 64 * k + (mrw_R > 0 ? 4 * S : 0);
    if (room < least) room = least;
    const int64_t most = room / (4 + 4 * k);  // at least 8 (one step)
    const int64_t groups = (S + per - 1) / per;
    return groups < most ? groups : most;
}

int walk_free(const Graph& gr, int draw, const DrawArgs& d, int64_t S, int32_t num_steps, const int32_t* roots,
              int32_t* const* step_out, char* ws, uint64_t o_flags, uint64_t o_parts, uint32_t mrw_R, int32_t* mrw_state,
              hipStream_t stream) {
    FreeArgs a{};
    a.links = gr.links;
    a.seed = d.seed;
    a.ppr_thr = d.ppr_thr;
    a.sample_base = d.sample_base;
    a.S = (uint32_t)S;
    a.V = (int32_t)gr.V;
    a.rowset = gr.rowset.load(std::memory_order_acquire);
    a.cells = walk_uses_cells(gr, S) ? gr.cells.load(std::memory_order_acquire) : nullptr;
    a.b_ret = d.b_ret;
    a.b_com = d.b_com;
    a.b_far = d.b_far;
    a.b_max = d.b_max;
    a.max_attempts = d.max_attempts;
    a.use_weights = d.use_weights;
    a.R = mrw_R;
    a.filled = mrw_R > 0 && mrw_reads_filled(gr, S, num_steps, mrw_R) ? gr.filled.load(std::memory_order_acquire) : nullptr;
    a.hdr = (WsHeader*)ws;
    a.flags = (uint32_t*)(ws + o_flags);
    a.parts = (uint32_t*)(ws + o_parts);
    a.total_steps = (uint32_t)num_steps;
    a.o_flags = o_flags;
    a.o_parts = o_parts;
    const bool node2vec = draw == kDrawNode2vec;
    const int lanes = node2vec ? attempt_lanes(S, d) : 0;
    const int64_t per = samples_per_group(S, lanes, mrw_R);
    const int64_t most = walk_free_groups(S, num_steps, node2vec, mrw_R);  // S >= 1
    for (int64_t s = 0; s < S; s += most * per) {
        const int64_t left = (S - s + per - 1) / per;
        const uint32_t groups = (uint32_t)(left < most ? left : most);
        a.s_first = (uint32_t)s;
        for (int32_t first = 0; first < num_steps; first += kFreeChunk) {
            const int32_t n = num_steps - first < kFreeChunk ? num_steps - first : kFreeChunk;
            a.first_step = (uint32_t)first;
            a.n_steps = (uint32_t)n;
            a.src = first > 0 ? step_out[first - 1] : roots;
            a.prev_src = first > 0 ? step_out[first - 2] : nullptr;  // kFreeChunk is at least two
            for (int32_t i = 0; i < kFreeChunk; ++i) a.out[i] = i < n ? step_out[first + i] : nullptr;
            mark_phase(ND_PHASE_WALK_WINDOW, stream);
            if (mrw_R > 0) {
                a.src = first > 0 ? mrw_state : roots;
                a.state = first + n < num_steps ? mrw_state : nullptr;
                const int waves = mrw_waves(mrw_R);
                if (gr.off64) {
                    if (waves == 16) launch_mrw<16, int64_t>(gr, a, groups, stream);
                    else if (waves == 4) launch_mrw<4, int64_t>(gr, a, groups, stream);
                    else launch_mrw<1, int64_t>(gr, a, groups, stream);
                } else {
                    if (waves == 16) launch_mrw<16, int32_t>(gr, a, groups, stream);
                    else if (waves == 4) launch_mrw<4, int32_t>(gr, a, groups, stream);
                    else launch_mrw<1, int32_t>(gr, a, groups, stream);
                }
            } else if (node2vec) {
                if (gr.off64) launch_n2v<int64_t>(gr, a, lanes, per, groups, stream);
                else launch_n2v<int32_t>(gr, a, lanes, per, groups, stream);
            } else if (S <= kFewWalks) {
                if (gr.off64) launch_few<int64_t>(gr, draw, a, groups, stream);
                else launch_few<int32_t>(gr, draw, a, groups, stream);
            } else if (gr.off64) {
                if (free_threads(S) == 64) launch_free<64, int64_t>(gr, draw, a, groups, stream);
                else launch_free<256, int64_t>(gr, draw, a, groups, stream);
            } else {
                if (free_threads(S) == 64) launch_free<64, int32_t>(gr, draw, a, groups, stream);
                else launch_free<256, int32_t>(gr, draw, a, groups, stream);
            }
            ND_HIP_CHECK(hipGetLastError());
        }
    }
    return ND_OK;
}

}  // namespace nd
