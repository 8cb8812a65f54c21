// k-hop sampling (Section 3 and Section 6.1 of the paper: `stepSize(i)` uniform neighbours of every
// transit) in one launch: every workgroup carries a few samples through all hops.  What a hop draws is
// a Link, which holds the row of the drawn vertex, so the next hop finds its rows in LDS; nothing is
// read back from the outputs and nothing is sorted.  Grouping by transit (nd_sort.hip, nd_sched.hip,
// nd_sample.hip) remains for calls whose draws meet often enough in a line of the graph.
#include "nd_common.h"
#include "nd_philox.h"
#include "nd_wave.h"
#include "nd_sample.h"
#include "nd_draw.h"
#include "nd_group.h"

#include <type_traits>

namespace nd {

namespace {

constexpr int kFusedThreads = 256;

struct FusedArgs {
    const Link* links;
    PackedCols packed;
    uint64_t seed;
    uint32_t sample_base;
    uint32_t S, G, splits;      // samples; per workgroup; workgroups that share the last hop of a group
    int32_t V;
    int32_t k;
    uint32_t m[ND_MAX_FANOUT_STEPS], W[ND_MAX_FANOUT_STEPS];  // draws per parent, slots per sample
    FastDiv div_m[ND_MAX_FANOUT_STEPS], div_w[ND_MAX_FANOUT_STEPS];
    uint32_t lds_half;          // entries of the first of the two row buffers
    const int32_t* roots;
    int32_t* out[ND_MAX_FANOUT_STEPS];
    WsHeader* hdr;
    uint32_t* flags;
    uint32_t* parts;
    uint64_t o_flags, o_parts;
    uint32_t* status_out;       // may be null
};

// R consecutive entries (R = 2: eight bytes, aligned).  PAST: past the caches.
template <int R, bool PAST>
__device__ __forceinline__ void store_run(int32_t* p, const int32_t* v) {
    typedef int32_t Int2 __attribute__((ext_vector_type(2)));
    if (PAST) {
        if (R == 2) __builtin_nontemporal_store(Int2{v[0], v[1]}, reinterpret_cast<Int2*>(p));
        else __builtin_nontemporal_store(v[0], p);
    } else {
        if (R == 2) *reinterpret_cast<Int2*>(p) = Int2{v[0], v[1]};
        else *p = v[0];
    }
}

// A place in a buffer of rows: where the row of a slot's vertex lies.
__device__ __forceinline__ uint2 row_of_link(const Link& l) { return make_uint2(l.rs, l.deg); }

// Bound by latency (small calls: a hop is generator, link, row; 37 roots of three hops take one launch
// instead of 26) or by the rate of scattered fetches (large ones).
// R: draws per lane of the last hop, a divisor of its fanout.  PAST: outputs go past the caches.  PACKED: the last hop
// reads the packed columns (R-MAT 22, every vertex, [25,10]: 22 bits instead of 32, 3,075 us and 2,860 like this).
template <int STRIDE, int R, bool PAST, bool PACKED, typename OffT>
__global__ __launch_bounds__(kFusedThreads) void khop_fused_kernel(GraphView<OffT> g, FusedArgs a) {
    extern __shared__ uint2 s_rows[];  // rows of the parents of this hop, of the next, in turn
    __shared__ uint32_t s_live[ND_MAX_FANOUT_STEPS];
    constexpr uint32_t T = kFusedThreads;
    const uint32_t tid = threadIdx.x;
    const uint32_t group = blockIdx.x / a.splits, part = blockIdx.x - group * a.splits;
    const uint32_t s0 = group * a.G;
    const uint32_t ns = a.S - s0 < a.G ? a.S - s0 : a.G;
    if (tid < ND_MAX_FANOUT_STEPS) s_live[tid] = 0;
    bool bad = false;
    uint32_t live = 0;
    for (uint32_t i = tid; i < ns; i += T) {
        int32_t v = a.roots[s0 + i];
        if (v >= a.V || v < ND_NULL_VERTEX) {
            bad = true;
            v = ND_NULL_VERTEX;
        }
        uint2 row = make_uint2(0u, 0u);
        if (v >= 0) {
            const uint64_t rs = (uint64_t)g.off[v];
            row = make_uint2((uint32_t)rs, row_length(g, v, rs));
        }
        live += (uint32_t)__popcll(__ballot(v >= 0));
        s_rows[i] = row;
    }
    const int any_bad = __syncthreads_or(bad ? 1 : 0);
    if (lane_id() == 0 && live) atomicAdd(&s_live[0], live);
    for (int hop = 0; hop < a.k; ++hop) {
        const bool last = hop == a.k - 1;
        const uint2* rows = s_rows + ((hop & 1) ? a.lds_half : 0u);
        uint2* next = s_rows + ((hop & 1) ? 0u : a.lds_half);
        const uint32_t W = a.W[hop], total = ns * W;
        int32_t* out = a.out[hop] + (uint64_t)s0 * W;
        if (!last) {
            live = 0;
            for (uint32_t d = tid; d < total; d += T) {
                const uint32_t s = fastdiv(d, a.div_w[hop]);
                const uint2 row = rows[fastdiv(d, a.div_m[hop])];
                Link l;
                l.v = ND_NULL_VERTEX;
                l.rs = 0;
                l.deg = 0;
                if (row.y > 0u) {
                    const Rand4 r = draw4(a.seed, a.sample_base + s0 + s, d - s * W, (uint32_t)hop, 0u);
                    l = a.links[(uint64_t)(row.x + mulhi32(r.r0, row.y)) * STRIDE];
                }
                live += (uint32_t)__popcll(__ballot(row.y > 0u));
                next[d] = row_of_link(l);
                if (part == 0) store_run<1, PAST>(out + d, &l.v);
            }
            if (lane_id() == 0 && live) atomicAdd(&s_live[hop + 1], live);
        } else {
            // kInFlight independent pieces per lane and round, of R consecutive draws of one parent each
            constexpr uint32_t kInFlight = 4 / R;
            const uint32_t pieces = total / R;
            const uint32_t share = ((pieces + a.splits - 1u) / a.splits + T - 1u) / T * T;
            const uint32_t begin = part * share;
            const uint32_t end = begin + share < pieces ? begin + share : pieces;
            for (uint32_t d0 = begin + tid; d0 < end; d0 += kInFlight * T) {
                uint2 row[kInFlight];
                uint32_t e[kInFlight][R];
                int32_t v[kInFlight][R];
#pragma unroll
                for (uint32_t u = 0; u < kInFlight; ++u) {
                    const uint32_t d = (d0 + u * T) * R;
                    row[u] = d0 + u * T < end ? rows[fastdiv(d, a.div_m[hop])] : make_uint2(0u, 0u);
                    if (PACKED)
                        for (uint32_t i = 0; i < R; ++i) e[u][i] = 0u;
                    // the draws of a sample without live parents are neighbours: whole wavefronts skip this
                    if (row[u].y > 0u) {
                        const uint32_t s = fastdiv(d, a.div_w[hop]);
#pragma unroll
                        for (uint32_t i = 0; i < R; ++i) {
                            const Rand4 r = draw4(a.seed, a.sample_base + s0 + s, d - s * W + i, (uint32_t)hop, 0u);
                            e[u][i] = row[u].x + mulhi32(r.r0, row[u].y);
                        }
                    }
                }
#pragma unroll
                for (uint32_t u = 0; u < kInFlight; ++u)
#pragma unroll
                    for (uint32_t i = 0; i < R; ++i) {
                        v[u][i] = ND_NULL_VERTEX;
                        if (row[u].y > 0u) v[u][i] = PACKED ? (int32_t)packed_word(a.packed, e[u][i], &e[u][i]) : g.col[e[u][i]];
                    }
#pragma unroll
                for (uint32_t u = 0; u < kInFlight; ++u) {
                    if (PACKED)
                        for (uint32_t i = 0; i < R; ++i)
                            v[u][i] = row[u].y > 0u ? packed_vertex(a.packed, (uint32_t)v[u][i], e[u][i]) : ND_NULL_VERTEX;
                    if (d0 + u * T < end) store_run<R, PAST>(out + (d0 + u * T) * R, v[u]);
                }
            }
        }
        __syncthreads();
    }
    if (tid < (uint32_t)a.k) a.parts[(uint64_t)blockIdx.x * (uint32_t)a.k + tid] = part == 0 ? s_live[tid] : 0u;
    if (tid == 0) {
        a.flags[blockIdx.x] = any_bad ? 1u : 0u;
        if (blockIdx.x == 0) write_header(a.hdr, (uint32_t)a.k, gridDim.x, a.o_flags, a.o_parts);
    }
    if (a.status_out != nullptr && blockIdx.x == gridDim.x - 1u) {  // few roots: this workgroup looks at them all
        bad = false;
        for (uint32_t i = tid; i < a.S; i += T) {
            const int32_t v = a.roots[i];
            bad |= v >= a.V || v < ND_NULL_VERTEX;
        }
        const int any = __syncthreads_or(bad ? 1 : 0);
        if (tid == 0) *a.status_out = any ? 1u : 0u;
    }
}

// The first hop of a call that groups its later ones: roots as a rule differ, so that grouping them by transit finds
// nothing to share, and their draws leave in order.  Bound by the lines of the rows.  233 K roots of 25 draws, mean
// degree 487: 66 us over packed columns, 71 with the gap to the next launch and 87 so over plain ones; 133 with the grouping
// (a sort, four kernels of groups and classes, 74 for the draws over plain columns).
template <bool PACKED, typename OffT>
__global__ __launch_bounds__(kFusedThreads) void khop_first_kernel(GraphView<OffT> g, PackedCols packed, uint64_t seed, uint32_t sample_base,
                                                                   const int32_t* __restrict__ roots, uint32_t n,
                                                                   FastDiv div_m, int32_t* __restrict__ out, StepCtl* ctl,
                                                                   uint32_t* status) {
    __shared__ uint32_t s_live;
    if (threadIdx.x == 0) s_live = 0;
    bool bad = false;
    uint32_t live = 0;
    constexpr uint32_t kInFlight = 4;
    for (uint64_t d0 = (uint64_t)blockIdx.x * kFusedThreads * kInFlight + threadIdx.x; d0 < n;
         d0 += (uint64_t)gridDim.x * kFusedThreads * kInFlight) {
        uint64_t rs[kInFlight];
        uint32_t deg[kInFlight];
        int32_t v[kInFlight];
#pragma unroll
        for (uint32_t u = 0; u < kInFlight; ++u) {
            const uint64_t d = d0 + u * kFusedThreads;
            v[u] = ND_NULL_VERTEX;
            if (d < n) v[u] = roots[fastdiv((uint32_t)d, div_m)];
        }
#pragma unroll
        for (uint32_t u = 0; u < kInFlight; ++u) {
            if (v[u] >= g.V || v[u] < ND_NULL_VERTEX) {
                bad = true;
                v[u] = ND_NULL_VERTEX;
            }
            rs[u] = 0;
            deg[u] = 0;
            if (v[u] >= 0) {
                rs[u] = (uint64_t)g.off[v[u]];
                deg[u] = row_length(g, v[u], rs[u]);
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < kInFlight; ++u) {
            const uint32_t d = (uint32_t)d0 + u * kFusedThreads, q = fastdiv(d, div_m), j = d - q * div_m.d;
            live += (uint32_t)__popcll(__ballot(v[u] >= 0 && j == 0u));
            v[u] = ND_NULL_VERTEX;
            if (deg[u] > 0u) {
                const uint64_t e = rs[u] + mulhi32(draw4(seed, sample_base + q, j, 0u, 0u).r0, deg[u]);
                v[u] = PACKED ? packed_entry(packed, (uint32_t)e) : g.col[e];
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < kInFlight; ++u)
            if (d0 + u * kFusedThreads < n) out[d0 + u * kFusedThreads] = v[u];
    }
    __syncthreads();
    if (lane_id() == 0 && live) atomicAdd(&s_live, live);  // lane 0 has been through every round of its wavefront
    const int any = __syncthreads_or(bad ? 1 : 0);
    if (threadIdx.x == 0) {
        if (s_live) atomicAdd(&ctl->P, s_live);
        if (any) atomicOr(status, 1u);
    }
}

// ---------------------------------------------------------------- unique neighbours (Section 6.3)
// All hops of a sample whose slots must hold different vertices, by one group of lanes.  The rules are
// those of unique_kernel (nd_sample.hip): among the slots of a hop that propose the same vertex the
// lowest keeps it, a slot that lost draws again with the next attempt, up to `rounds` draws, and a slot
// whose parent's slots hold as many distinct vertices as the parent's row has entries ends empty.  Here
// the first draws come straight from the parents' rows in LDS into the hash table, the later rounds find
// the rows there too, and the outputs are written once, in order.
//
// Bound by instruction issue (vector and scalar alike), then by the fabric's lines; measured on the scale-22
// R-MAT graph, every vertex, [25,10], 4 draws: 7.26 ms with the ordinary kernels first, all slots read back
// and patched; 6.1 ms with one pass of the generator per round; 5.35 ms when lanes without a slot draw the
// next attempts AND the registers are held to 64, so that a SIMD keeps 8 wavefronts (5.8 ms at 7, 6.4 at 5);
// 5.2 ms with workgroups of one wavefront, which leave when their own samples are done; 5.0 ms with the
// narrow hops' first round treated as one of the later ones.
struct UniqueFusedArgs {
    const Link* links;
    uint64_t seed;
    uint32_t sample_base;
    uint32_t S;
    int32_t V;
    int32_t k, rounds;
    uint32_t W[ND_MAX_FANOUT_STEPS];
    FastDiv div_m[ND_MAX_FANOUT_STEPS];
    uint32_t slots;             // widest hop, rounded up to what the lanes take: entries per LDS array
    uint32_t rows;              // rows of the widest hop with children (or the root's)
    const int32_t* roots;
    int32_t* out[ND_MAX_FANOUT_STEPS];
    WsHeader* hdr;
    uint32_t* flags;
    uint32_t* parts;
    uint64_t o_flags, o_parts;
};

// Bytes of LDS per group: a multiple of 16, so that the hash table of a workgroup's second group lies as the
// first one's does (it is cleared 16 bytes at a time; an even number of rows lies before it).
__host__ __device__ inline uint32_t unique_group_bytes(uint32_t slots, uint32_t rows) {
    const uint32_t bytes = 2u * slots * 4u      // hash table: a slot per bucket, two buckets per slot
                           + slots * 4u         // the hop's vertices
                           + slots * 4u         // two queues of open slots, 16 bits per entry
                           + rows * 4u          // per parent: distinct vertices its slots hold
                           + 2u * rows * 8u;    // rows of this hop's parents and of the next hop's
    return (bytes + 15u) & ~15u;
}

// PAST: outputs go past the caches.
template <int STRIDE, typename OffT, int THREADS, int PER, bool PAST = false>
__global__ __launch_bounds__(THREADS <= 64 ? 64 : THREADS, THREADS <= 64 ? 8 : 4)
void khop_unique_kernel(GraphView<OffT> g, UniqueFusedArgs a) {
    extern __shared__ __align__(16) unsigned char s_raw[];
    constexpr uint32_t SUBS = THREADS <= 64 ? 64 / THREADS : 1;  // groups (samples in flight) per workgroup
    constexpr int kLanes = THREADS <= 64 ? THREADS : 64;         // lanes of a group within one wavefront
    // Who holds a vertex is found in passes (see settle) by whole wavefronts.  Half a one's 32 slots rarely share a bucket,
    // and its compare-and-swap loops are shorter than two passes (every vertex of R-MAT 22, [25]: 1,152 us, 1,203 with
    // passes); several wavefronts would need two barriers for each.
    constexpr bool kPasses = THREADS == 64;
    __shared__ uint32_t s_live[ND_MAX_FANOUT_STEPS];
    __shared__ uint32_t q_fill[2];            // queue lengths of a group of several wavefronts
    const uint32_t sub = threadIdx.x / (uint32_t)THREADS;
    const uint32_t tix = threadIdx.x % (uint32_t)THREADS;  // my place in the group
    const uint64_t group_lanes = THREADS == 32 ? 0xFFFFFFFFull << (threadIdx.x & 32u) : ~0ull;
    unsigned char* mem = s_raw + (size_t)sub * unique_group_bytes(a.slots, a.rows);
    uint2* rows_a = (uint2*)mem;
    uint2* rows_b = rows_a + a.rows;
    // A bucket names the slot whose vertex it stands for.  By compare and swap: j = slot j holds the vertex, kOpen + j = slot j
    // is the lowest that proposes it so far.  (Keys and claims apart took twice the LDS, and with it a
    // quarter of the wavefronts a compute unit can hold.)
    constexpr uint32_t kOpen = 4096u, kFree = 0xFFFFFFFFu;
    uint32_t* table = (uint32_t*)(rows_b + a.rows);
    int32_t* s_res = (int32_t*)(table + 2u * a.slots);  // vertex that slot j holds or proposes
    uint32_t* p_held = (uint32_t*)(s_res + a.slots);
    uint16_t* queue[2] = {(uint16_t*)(p_held + a.rows), (uint16_t*)(p_held + a.rows) + a.slots};
    if (threadIdx.x < ND_MAX_FANOUT_STEPS) s_live[threadIdx.x] = 0;
    __syncthreads();
    bool bad = false;
    // live slots per hop of all my samples, counted where lane 0 of the group can add them up
    for (uint32_t at = blockIdx.x * SUBS + sub; at < a.S; at += gridDim.x * SUBS) {  // the same in the whole group
        // a wavefront's sample is a scalar, and with it the generator's first rounds (sample and step only)
        const uint32_t s = THREADS >= 64 ? wave_uniform(at) : at;
        int32_t root = a.roots[s];
        if (root >= a.V || root < ND_NULL_VERTEX) {
            bad = true;
            root = ND_NULL_VERTEX;
        }
        uint2 first = make_uint2(0u, 0u);
        if (root >= 0) {
            const uint64_t rs = (uint64_t)g.off[root];
            first = make_uint2((uint32_t)rs, row_length(g, root, rs));
            if (tix == 0) atomicAdd(&s_live[0], 1u);
        }
        if (tix == 0) rows_a[0] = first;
        bool any = first.y > 0u;   // some parent of this hop has a row
        group_sync<THREADS>();
        for (int hop = 0; hop < a.k; ++hop) {
            const uint32_t W = a.W[hop], parents = hop > 0 ? a.W[hop - 1] : 1u;
            const bool last = hop == a.k - 1;
            const uint2* rows = (hop & 1) ? rows_b : rows_a;
            uint2* next = (hop & 1) ? rows_a : rows_b;
            int32_t* out_row = a.out[hop] + (uint64_t)s * W;
            if (!any) {  // uniform: nothing to draw in this hop and those after it
                const int32_t none = ND_NULL_VERTEX;
                for (uint32_t j = tix; j < W; j += (uint32_t)THREADS) store_run<1, PAST>(out_row + j, &none);
                continue;
            }
            uint32_t buckets = 64;                  // power of two, at least 2 W
            while (buckets < 2u * W) buckets <<= 1;
            const uint32_t mask = buckets - 1u;
            // In passes: a bucket holds the lowest key of those who came to it, a key being the pass and the slot, so that who
            // came in an earlier pass stays.  Whoever finds itself in its bucket holds its vertex, whoever finds a slot of the
            // same vertex has lost, and who finds another vertex goes on to its next bucket in the next pass (the
            // sequence depends on the vertex only, so that equal vertices meet).  Nothing is marked afterwards, a pass is
            // an LDS minimum without a result and two reads, and the few that the first pass leaves are packed before the
            // second (R-MAT 22, every vertex, [25,10], 4 draws: 4,685 us with compare and swap, 4,460 like this; 1,024
            // vertices of 57 K 19.1 and 15.8).
            uint32_t pass = 0;
            auto bucket_of = [&](int32_t c) -> uint32_t { return ((uint32_t)c * 2654435761u >> 15) & mask; };
            // a pass has put its keys: 1 slot j holds c, 2 it has lost, 0 neither
            auto verdict = [&](uint32_t b, int32_t c, uint32_t j) -> uint32_t {
                const uint32_t w = table[b] & (kOpen - 1u);
                return w == j ? 1u : s_res[w] == c ? 2u : 0u;
            };
            // up to `n` slots per lane that come together; open[i] tells who does, won[i] receives who holds its vertex.
            // `step` buckets of the sequences have been looked at, b[i] is the next.
            auto settle = [&](auto count, uint32_t limit, const uint32_t* j, const int32_t* c, uint32_t* b, bool* open, bool* won,
                              uint32_t step) {
                constexpr int N = decltype(count)::value;
                bool more;
                do {
                    ++pass;
                    ++step;
#pragma unroll
                    for (int i = 0; i < N; ++i) {
                        if ((uint32_t)i * (uint32_t)THREADS >= limit) break;
                        if (open[i]) atomicMin(&table[b[i]], (pass << 12) + j[i]);  // at most 64 rounds of 512 passes
                    }
                    group_sync<THREADS>();
                    more = false;
#pragma unroll
                    for (int i = 0; i < N; ++i) {
                        if ((uint32_t)i * (uint32_t)THREADS >= limit) break;
                        if (open[i]) {
                            const uint32_t v = verdict(b[i], c[i], j[i]);
                            won[i] = v == 1u;
                            open[i] = v == 0u;
                            b[i] = (b[i] + step) & mask;
                        }
                        more |= open[i];
                    }
                    group_sync<THREADS>();
                } while (group_any<kLanes>(more, group_lanes));  // ends: there are more buckets than vertices
            };
            // By compare and swap:
            // proposes vertex c for slot j (s_res[j] is c already, for every proposer); returns the bucket of
            // c.  The table never holds more than W distinct vertices in at least 2 W buckets, so a free or
            // matching bucket is found long before the probe bound.
            auto propose = [&](int32_t c, uint32_t j) -> uint32_t {
                uint32_t b = bucket_of(c);
                for (uint32_t probe = 0; probe < buckets; ++probe) {
                    const uint32_t old = atomicCAS(&table[b], kFree, kOpen + j);
                    if (old == kFree) break;
                    if (s_res[old & (kOpen - 1u)] == c) {
                        atomicMin(&table[b], kOpen + j);
                        break;
                    }
                    b = (b + 1u) & mask;
                }
                return b;
            };
            for (uint32_t b = tix; b < buckets / 4u; b += (uint32_t)THREADS)  // four free buckets per store
                reinterpret_cast<int4*>(table)[b] = make_int4(-1, -1, -1, -1);
            for (uint32_t pj = tix; pj < parents; pj += (uint32_t)THREADS) p_held[pj] = 0;
            if (THREADS > 64 && tix == 0) q_fill[0] = 0;
            // what a slot draws: an entry of the parent's row (its link where the hop has children)
            auto fetch = [&](uint2 row, uint32_t j, uint32_t attempt, uint2* row_out) -> int32_t {
                // Joined exclusive ors make a call of few samples, by four wavefronts each, longer: 56 of [15,10,5] with 8
                // draws 30.6 us and 31.9 with them, 200 with 4 draws 22.2 and 22.6; two wavefronts gain (100,000 on
                // R-MAT 22 692 and 684).
                const Rand4 r = draw4<THREADS != 256>(a.seed, a.sample_base + s, j, (uint32_t)hop, attempt);
                const uint64_t e = (uint64_t)row.x + mulhi32(r.r0, row.y);
                *row_out = make_uint2(0u, 0u);
                if (last) return g.col[e];
                const Link l = a.links[e * STRIDE];
                *row_out = make_uint2(l.rs, l.deg);
                return l.v;
            };
            int32_t cand[PER];
            uint32_t where[PER];                // bucket, and from bit 16 the parent
            bool won[PER];
            uint32_t cur = 0;                   // the queue being read
            uint32_t fill = 0;                  // entries in the queue being written (group inside one wavefront)
            int32_t r = 0;
            if (THREADS <= 64 && 2u * W <= (uint32_t)THREADS) {
                // every slot is open, and the first round is one of those below
                if (tix < W) {
                    s_res[tix] = ND_NULL_VERTEX;
                    if (!last) next[tix] = make_uint2(0u, 0u);
                    queue[0][tix] = (uint16_t)tix;
                }
                fill = W;
            } else {
                r = 1;
                // The kernel pays for vector instructions first, so the unrolled loops end where the hop or the
                // queue does: a test of scalars (W, L), the same in the whole group.
#pragma unroll
                for (int t = 0; t < PER; ++t) {   // all fetches are on their way before the first is looked at
                    const uint32_t j = tix + (uint32_t)t * (uint32_t)THREADS;
                    cand[t] = ND_NULL_VERTEX;
                    where[t] = 0;
                    if ((uint32_t)t * (uint32_t)THREADS < W && j < W) {
                        const uint32_t pj = fastdiv(j, a.div_m[hop]);
                        const uint2 row = rows[pj];
                        where[t] = pj << 16;
                        uint2 crow = make_uint2(0u, 0u);
                        if (row.y > 0u) cand[t] = fetch(row, j, 0u, &crow);
                        if (!last) next[j] = crow;
                    }
                }
#pragma unroll
                for (int t = 0; t < PER; ++t) {
                    const uint32_t j = tix + (uint32_t)t * (uint32_t)THREADS;
                    if ((uint32_t)t * (uint32_t)THREADS < W && j < W) s_res[j] = cand[t];
                }
                group_sync<THREADS>();
                if constexpr (kPasses) {
#pragma unroll
                    for (int t = 0; t < PER; ++t) {   // the first pass, all slots at once
                        if ((uint32_t)t * (uint32_t)THREADS >= W) break;
                        if (cand[t] >= 0) {
                            where[t] |= bucket_of(cand[t]);
                            atomicMin(&table[where[t] & 0xFFFFu], tix + (uint32_t)t * (uint32_t)THREADS);
                        }
                    }
                    group_sync<THREADS>();
                    uint32_t undecided = 0;   // packed in the other queue, ascending
#pragma unroll
                    for (int t = 0; t < PER; ++t) {
                        if ((uint32_t)t * (uint32_t)THREADS >= W) break;
                        const uint32_t j = tix + (uint32_t)t * (uint32_t)THREADS;
                        uint32_t v = 2u;
                        if (cand[t] >= 0) v = verdict(where[t] & 0xFFFFu, cand[t], j);
                        if (v == 1u) atomicAdd(&p_held[where[t] >> 16], 1u);
                        const uint32_t later = group_reserve<THREADS>(v == 0u, group_lanes, &undecided, nullptr);
                        if (v == 0u) queue[1][later] = (uint16_t)j;
                        const bool lost = v == 2u && cand[t] >= 0;
                        const uint32_t at = group_reserve<THREADS>(lost, group_lanes, &fill, nullptr);
                        if (lost) queue[0][at] = (uint16_t)j;
                        if (v == 2u && j < W) {
                            s_res[j] = ND_NULL_VERTEX;
                            if (!last) next[j] = make_uint2(0u, 0u);
                        }
                    }
                    group_sync<THREADS>();
                    if (THREADS >= 64) undecided = wave_uniform(undecided);
                    for (uint32_t e0 = 0; e0 < undecided; e0 += (uint32_t)THREADS) {  // a fifth where W fills half the table
                        bool open = e0 + tix < undecided, held = false;
                        const bool mine = open;
                        const uint32_t j = mine ? queue[1][e0 + tix] : 0u;
                        const int32_t c = mine ? s_res[j] : ND_NULL_VERTEX;
                        uint32_t b = (bucket_of(c) + 1u) & mask;
                        settle(std::integral_constant<int, 1>{}, 1u, &j, &c, &b, &open, &held, 1u);
                        if (held) atomicAdd(&p_held[fastdiv(j, a.div_m[hop])], 1u);
                        const bool lost = mine && !held;
                        const uint32_t at = group_reserve<THREADS>(lost, group_lanes, &fill, nullptr);
                        if (lost) {
                            queue[0][at] = (uint16_t)j;
                            s_res[j] = ND_NULL_VERTEX;
                            if (!last) next[j] = make_uint2(0u, 0u);
                        }
                    }
                } else {
#pragma unroll
                    for (int t = 0; t < PER; ++t) {
                        if ((uint32_t)t * (uint32_t)THREADS >= W) break;
                        if (cand[t] >= 0) where[t] |= propose(cand[t], tix + (uint32_t)t * (uint32_t)THREADS);
                    }
                    group_sync<THREADS>();
#pragma unroll
                    for (int t = 0; t < PER; ++t) {
                        won[t] = false;
                        if ((uint32_t)t * (uint32_t)THREADS >= W) continue;
                        won[t] = cand[t] >= 0 && table[where[t] & 0xFFFFu] == kOpen + tix + (uint32_t)t * (uint32_t)THREADS;
                    }
                    group_sync<THREADS>();              // every claim has been read
                    // a winner marks its bucket as held: whoever proposes that vertex later loses; a loser queues
#pragma unroll
                    for (int t = 0; t < PER; ++t) {
                        if ((uint32_t)t * (uint32_t)THREADS >= W) break;
                        const uint32_t j = tix + (uint32_t)t * (uint32_t)THREADS;
                        if (won[t]) {
                            table[where[t] & 0xFFFFu] = j;
                            atomicAdd(&p_held[where[t] >> 16], 1u);
                        } else if (j < W) {
                            s_res[j] = ND_NULL_VERTEX;
                            if (!last) next[j] = make_uint2(0u, 0u);
                        }
                        const bool open = cand[t] >= 0 && !won[t];
                        const uint32_t at = group_reserve<THREADS>(open, group_lanes, &fill, &q_fill[0]);
                        if (open) queue[0][at] = (uint16_t)j;
                    }
                }
            }
            if (THREADS > 64 && tix == 0) q_fill[1] = 0;
            group_sync<THREADS>();
            uint32_t L = THREADS > 64 ? q_fill[0] : fill;  // slots still open (uniform in the group)
            if (THREADS >= 64) L = wave_uniform(L);

            // ---- rounds.  The generator's quarter-rate multiplies are what a round pays for most, and it costs
            // a wavefront the same for one open slot as for 64.  So when at most half the lanes have a slot, the
            // others draw the same slots' next attempts: one pass of the generator and one fetch serve two, four
            // or eight rounds, which then only take their candidates from the lanes that hold them.  A group of
            // several wavefronts leaves its last 64 open slots to the first one, whose rounds need no barriers: slots
            // that cannot win (two neighbours, one held elsewhere) stay open for all rounds, and with four barriers
            // of 256 lanes each, 64 rounds of [10,10,10] from 30,000 vertices of a ring took 3.5 ms, 2.3 in a kernel
            // per hop whose narrow hops run in one wavefront, 1.9 like this (1.5 with 128 lanes).
            while (r < a.rounds && L > 0) {
                if (THREADS > 64 ? L <= (uint32_t)kLanes : L <= (uint32_t)kLanes / 2u && r + 1 < a.rounds) {
                    if (THREADS <= 64 || tix < (uint32_t)kLanes) {
                        do {
                            const uint32_t lg = L <= (uint32_t)kLanes / 8u   ? 3u
                                                : L <= (uint32_t)kLanes / 4u ? 2u
                                                : L <= (uint32_t)kLanes / 2u ? 1u
                                                                             : 0u;
                            const uint32_t span = (uint32_t)kLanes >> lg;  // lanes per attempt
                            const uint32_t e = tix & (span - 1u);
                            const int32_t mine = r + (int32_t)(tix / span);
                            uint32_t j = 0, pj = 0;
                            uint2 row = make_uint2(0u, 0u), vrow = make_uint2(0u, 0u);
                            int32_t v = ND_NULL_VERTEX;
                            if (e < L && mine < a.rounds) {
                                j = queue[cur][e];
                                pj = fastdiv(j, a.div_m[hop]);
                                row = rows[pj];
                                if (p_held[pj] < row.y) v = fetch(row, j, (uint32_t)mine, &vrow);
                            }
                            bool open = tix < span && v >= 0;  // lane e speaks for slot e
                            for (uint32_t i = 0; i < (1u << lg) && r < a.rounds; ++i, ++r) {
                                const int from = (int)((threadIdx.x & 63u) - tix + i * span + e);
                                const int32_t c = __shfl(v, from, 64);
                                const uint2 cr = make_uint2((uint32_t)__shfl((int)vrow.x, from, 64),
                                                            (uint32_t)__shfl((int)vrow.y, from, 64));
                                // as many distinct vertices as the parent's row has entries: nothing left to draw
                                open = open && p_held[pj] < row.y;
                                if (!group_any<kLanes>(open, group_lanes)) {
                                    r = a.rounds;
                                    break;
                                }
                                if (open) s_res[j] = c;
                                group_sync<kLanes>();
                                bool win = false;
                                uint32_t at = 0;
                                if constexpr (kPasses) {
                                    bool come = open;
                                    at = bucket_of(c);
                                    settle(std::integral_constant<int, 1>{}, 1u, &j, &c, &at, &come, &win, 0u);
                                } else {
                                    if (open) at = propose(c, j);
                                    group_sync<kLanes>();
                                    win = open && table[at] == kOpen + j;
                                    group_sync<kLanes>();          // every claim has been read
                                    if (win) table[at] = j;
                                }
                                if (win) {
                                    if (!last) next[j] = cr;
                                    atomicAdd(&p_held[pj], 1u);
                                } else if (open) {
                                    s_res[j] = ND_NULL_VERTEX;
                                }
                                open = open && !win;
                                group_sync<kLanes>();
                            }
                            fill = 0;
                            const uint32_t at = group_reserve<kLanes>(open, group_lanes, &fill, nullptr);
                            if (open) queue[cur ^ 1u][at] = (uint16_t)j;
                            group_sync<kLanes>();
                            cur ^= 1u;
                            L = fill;
                            if (THREADS >= 64) L = wave_uniform(L);
                        } while (THREADS > 64 && r < a.rounds && L > 0);
                    }
                    if (THREADS <= 64) continue;
                    group_sync<THREADS>();
                    break;  // the other wavefronts' L and r are those of the first one's start
                }
                uint32_t jq[PER];
#pragma unroll
                for (int p = 0; p < PER; ++p) {
                    const uint32_t e = tix + (uint32_t)p * (uint32_t)THREADS;
                    cand[p] = ND_NULL_VERTEX;
                    where[p] = 0;
                    jq[p] = 0;
                    if ((uint32_t)p * (uint32_t)THREADS >= L || e >= L) continue;
                    const uint32_t j = queue[cur][e];
                    const uint32_t pj = fastdiv(j, a.div_m[hop]);
                    const uint2 row = rows[pj];
                    // the parent's slots already hold as many distinct vertices as its row has entries:
                    // whatever this slot draws is held, now and in every later round
                    if (p_held[pj] >= row.y) continue;
                    uint2 crow;
                    cand[p] = fetch(row, j, (uint32_t)r, &crow);
                    jq[p] = j;
                    where[p] = pj << 16;
                    s_res[j] = cand[p];
                    if (!last) next[j] = crow;
                }
                group_sync<THREADS>();
                if constexpr (kPasses) {
                    uint32_t b[PER];
                    bool come[PER];
#pragma unroll
                    for (int p = 0; p < PER; ++p) {
                        won[p] = false;
                        come[p] = cand[p] >= 0;
                        b[p] = bucket_of(cand[p]);
                    }
                    settle(std::integral_constant<int, PER>{}, L, jq, cand, b, come, won, 0u);
                } else {
#pragma unroll
                    for (int p = 0; p < PER; ++p) {
                        if ((uint32_t)p * (uint32_t)THREADS >= L) break;
                        if (cand[p] >= 0) where[p] |= propose(cand[p], jq[p]);
                    }
                    group_sync<THREADS>();
#pragma unroll
                    for (int p = 0; p < PER; ++p) {
                        won[p] = false;
                        if ((uint32_t)p * (uint32_t)THREADS >= L) continue;
                        won[p] = cand[p] >= 0 && table[where[p] & 0xFFFFu] == kOpen + jq[p];
                    }
                    group_sync<THREADS>();          // every claim has been read
                }
                fill = 0;
#pragma unroll
                for (int p = 0; p < PER; ++p) {
                    if ((uint32_t)p * (uint32_t)THREADS >= L) break;
                    if (won[p]) {
                        if (!kPasses) table[where[p] & 0xFFFFu] = jq[p];
                        atomicAdd(&p_held[where[p] >> 16], 1u);
                    }
                    const bool open = cand[p] >= 0 && !won[p];
                    if (open) {
                        s_res[jq[p]] = ND_NULL_VERTEX;
                        if (!last) next[jq[p]] = make_uint2(0u, 0u);
                    }
                    const uint32_t at = group_reserve<THREADS>(open, group_lanes, &fill, &q_fill[cur ^ 1u]);
                    if (open) queue[cur ^ 1u][at] = (uint16_t)jq[p];
                }
                if (THREADS > 64 && tix == 0) q_fill[cur] = 0;  // everybody read it two barriers ago
                group_sync<THREADS>();
                cur ^= 1u;
                L = THREADS > 64 ? q_fill[cur] : fill;
                if (THREADS >= 64) L = wave_uniform(L);
                ++r;
            }
            // ---- a slot that never won a vertex of its own stays empty; the hop leaves in order
            int alive = 0;
            uint32_t got = 0;
            for (uint32_t j = tix; j < W; j += (uint32_t)THREADS) {
                const int32_t v = s_res[j];
                store_run<1, PAST>(out_row + j, &v);
                got += (uint32_t)__popcll(__ballot(v >= 0) & group_lanes);
                if (!last) alive |= next[j].y > 0u ? 1 : 0;
            }
            if (!last) {
                if (tix % 64u == 0u && got) atomicAdd(&s_live[hop + 1], got);
                any = group_or<THREADS>(alive, group_lanes) != 0;
            }
            group_sync<THREADS>();  // table, queues and rows are rebuilt for the next hop or sample
        }
    }
    const int any_bad = __syncthreads_or(bad ? 1 : 0);
    if (threadIdx.x < (uint32_t)a.k)
        a.parts[(uint64_t)blockIdx.x * (uint32_t)a.k + threadIdx.x] = s_live[threadIdx.x];
    if (threadIdx.x == 0) {
        a.flags[blockIdx.x] = any_bad ? 1u : 0u;
        if (blockIdx.x == 0) write_header(a.hdr, (uint32_t)a.k, gridDim.x, a.o_flags, a.o_parts);
    }
}

constexpr int64_t kFusedRows = 4096;  // rows per workgroup (32 KB of LDS) of the widest hop that has children

struct FusedShape {
    uint32_t G = 1, splits = 1, half = 1;
    size_t lds = 0;
    int64_t groups = 0;
};

// Samples per workgroup: enough draws in the last hop for a few rounds of its lanes when there are
// plenty of samples; one sample, its last hop shared by several workgroups, when there are few.
FusedShape fused_shape(const Graph& gr, int32_t k, const int64_t* W, int64_t S) {
    FusedShape f;
    int64_t widest[2] = {1, 1};  // per sample: rows kept in each of the two buffers (the roots, hop 1, ... in turn)
    for (int i = 0; i + 1 < k; ++i) {
        int64_t& w = widest[(i + 1) & 1];
        if (W[i] > w) w = W[i];
    }
    const int64_t rows = widest[0] + widest[1], last = W[k - 1];
    const int64_t want = (int64_t)gr.num_cus * 8;   // workgroups that fill the chip
    int64_t G = 2048 / last;
    if (G > kFusedRows / rows) G = kFusedRows / rows;
    if (G > S / want) G = S / want;
    if (G < 1) G = 1;
    f.G = (uint32_t)G;
    const int64_t groups = S > 0 ? (S + G - 1) / G : 1;
    int64_t splits = 1;
    if (groups < want) {
        splits = want / groups;
        const int64_t rounds = (last * G + kFusedThreads - 1) / kFusedThreads;
        if (splits > rounds) splits = rounds;
    }
    f.splits = (uint32_t)splits;
    f.half = (uint32_t)(widest[0] * G);
    f.lds = (size_t)(rows * G) * sizeof(uint2);
    f.groups = groups * splits;
    return f;
}

// Two draws per lane where the fanout is even and the output aligned: what a lane looks up about its
// pair (slot, row) and works out about its place then serves two draws, and they leave in one store.
bool khop_in_pairs(uint32_t m, const int32_t* out) { return m % 2u == 0u && ((uintptr_t)out & 7u) == 0; }

void slots_per_sample(const int32_t* fanout, int32_t k, int64_t* W) {
    int64_t w = 1;
    for (int32_t i = 0; i < k; ++i) W[i] = w = w * fanout[i];
}

}  // namespace

// Whether the fused kernel takes the call.  Its limits are the rows in LDS and the links.  Its cost is one
// scattered fetch per line a pair's draws touch, whatever other pairs touch; grouping by transit fetches a
// line once for all its draws and pays for it with the sort and with scattered stores.  Measured from
// all, a tenth and a fiftieth of the vertices of twelve graphs with fanouts [25,10], [10,10], [10,25], [20],
// [15,10,5], [7,13], [8,8,4] and [5,5]: grouping wins, by up to 1.7x, on dense graphs (rows that ten draws
// rarely share a line of) with many pairs per vertex and enough draws to pay for its launches; elsewhere it
// loses, by up to 6x from 1 M draws on.  Near the lines, over links and grouped: mean degree 152, 10 pairs per vertex, 23 M
// draws 255 and 173 us, 58 M 402 and 319; degree 211, 25 pairs, 14 M 127 and 120, 10 pairs, 14 M 88 and 104; degree 98,
// 10 pairs, 26 M 228 and 197, 25 pairs, 66 M 471 and 481; degree 84, 25 pairs, 66 M 433 and 469; degree 1059, 25 pairs,
// 5 M 78 and 78; degree 487, 15 pairs, 17 M 343 and 341, 7 pairs, 21 M 301 and 217; degree 61, 25 pairs, 58 M 342 and 418; degree
// 58, 10 pairs, 100 M 933 and 767.  The lines were drawn on times of earlier kernels of both routes; they now leave up to
// 39 % (7 pairs per vertex, mean degrees of 152 and 487) and 22 % (the last one).
bool khop_fused_fits(const Graph& gr, const int32_t* fanout, int32_t k, int64_t S) {
    if (!gr.links) return false;
    int64_t pairs = S;
    for (int32_t i = 0; i + 1 < k; ++i) pairs *= fanout[i];  // below 2^31 by the call's plan
    const int64_t draws = pairs * fanout[k - 1];
    if ((draws >= 20000000 && gr.E >= 120 * gr.V && pairs >= 8 * gr.V) ||
        (draws >= 14000000 && gr.E >= 80 * gr.V && pairs >= 16 * gr.V))
        return false;
    int64_t w = 1, prev = 1;
    for (int32_t i = 0; i + 1 < k; ++i) {
        prev = w;
        w *= fanout[i];
        if (w + prev > kFusedRows) return false;
    }
    return w * fanout[k - 1] < (1ll << 31);
}

// Whether a call is faster over the packed columns: where its draws fetch a line each or two and are many.  The m draws of
// a short row share its lines anyway, and then only the instructions of the unpacking are felt.  Measured with
// [25,10], [10,10], [10,25], [20], [15,10,5], [7,13], [8,8,4] and [5,5] on twelve graphs, plain time over packed time: where the rule
// reads them 1.01 ([8,8,4] on the dense graph) to 1.45 ([10,25], 57 K vertices of mean degree 211); elsewhere 0.94
// ([10,25] at a mean degree of 29) to 1.26 (6 M draws of [10,25], mean degree 61).
bool khop_reads_packed(const Graph& gr, const int32_t* fanout, int32_t k, int64_t S) {
    if (!gr.links) return false;
    int64_t draws = S;
    for (int32_t i = 0; i < k; ++i) draws *= fanout[i];  // below 2^31 by the call's plan
    return (draws >= 6000000 && 5 * gr.E >= 6 * (int64_t)fanout[k - 1] * gr.V) ||
           (draws >= 200000 && gr.E >= 128 * gr.V);
}

// Draws of the last hop from which a call's outputs leave past the caches, which then hold more of the graph: every
// vertex of R-MAT 22, [25,10], 1.05 G draws, 3,220 us and 3,058 like this; 400 M draws of [25,10] on R-MAT 18 979 and 891,
// over weights on 57 K vertices 1,070 and 1,041, on 2 M alike.  A batch that L2 holds (1,024 roots) is faster through it
// (8.6 and 8.8).  Outputs that leave one by one (odd fanouts) go past the
// caches only where the L2s, of 4 MB each, hold the entries between them: 400 M draws on 57 K vertices (6 MB of
// entries) [7,13] 1,258 and 1,221, [15,10,5] 2,390 and 2,352, on R-MAT 18 (16 MB) 1,156 and 1,186, 2,114 and 2,096; not
// on R-MAT 22 (275 MB) with 1,520 and 1,581 for [7,13], 2,637 and 2,719 for [5,5], 2,703 and 2,727 for [15,10,5], nor on 2 M
// vertices (128 MB): 1,985 and 2,022, 3,883 and 3,983, 3,122 and 3,141.
//
// In pairs and after a hop that reads links, and where neighbours are unique, they do so from 24 M draws on (96 MB) where the
// last-level cache, of 256 MB, does not hold them together with the entries.  Who reads them next has to be counted in:
// the call alone is faster past the caches from 6 M draws on (up to 6 %), but outputs that the last-level cache would
// have held then come from memory.  Time through the caches over time past them, the call alone and with a copy of
// the last hop, a maximum per sample, the gathered records and a look-up per vertex behind it:
//   57 K vertices, 2 M entries, [25,10]: 48 MB 1.02, with those 0.95, 0.97, 0.86, 1.00; 128 MB 1.02, 1.00, 0.97, 0.93, 1.00;
//     200 MB 1.03, 1.07, 0.97, 1.03, 0.94; 256 MB 1.05, 1.03, 1.04, 1.04, 1.01
//   R-MAT 20, 30 M entries, 48 MB 1.02, 0.94, 0.99, 0.90, 0.99; 128 MB 1.03, 1.06, 0.99, 1.01, 0.98; 200 MB 1.02, 1.02, 1.02,
//     1.02, 0.99
//   R-MAT 22, 69 M entries, 48 MB 1.02, 0.94, 0.96, 0.89, 1.00; 80 MB 1.03, 1.05, 0.98, 0.94, 0.99; 100 MB 1.08, 1.06, 1.00, 1.00,
//     0.99; 128 MB 1.14, 1.04, 1.02, 1.04, 1.00; 256 MB 1.19, 1.05, 1.04, 1.05, 1.04
// and [10,10], [15,10,4] and unique neighbours alike ([25,10], 57 K vertices, 80 MB 1.00, 0.97, 0.99, 0.92, 0.99; R-MAT 22, 48 MB
// 1.03, 0.97, 0.99, 0.91, 1.00, 128 MB 1.04, 1.02, 0.99, 1.00, 0.99).
constexpr int64_t kPastCaches = 64 << 20;
constexpr int64_t kPastCachesPairs = 24000000;
constexpr int64_t kPastCachesOneByOne = 8 << 20;  // entries: 32 MB
bool last_level_is_passed(const Graph& gr, int64_t draws) { return draws >= kPastCachesPairs && draws + gr.E >= (64 << 20); }

int64_t khop_fused_groups(const Graph& gr, const int32_t* fanout, int32_t k, int64_t S) {
    int64_t W[ND_MAX_FANOUT_STEPS];
    slots_per_sample(fanout, k, W);
    return fused_shape(gr, k, W, S).groups;
}

int khop_fused(const Graph& gr, const DrawArgs& d, const int32_t* fanout, int32_t k, int64_t S, const int32_t* roots,
               int32_t* const* step_out, char* ws, uint64_t o_flags, uint64_t o_parts, uint32_t* status_out,
               hipStream_t stream) {
    int64_t W[ND_MAX_FANOUT_STEPS];
    slots_per_sample(fanout, k, W);
    const FusedShape f = fused_shape(gr, k, W, S);
    FusedArgs a{};
    a.links = gr.links;
    a.packed = d.packed;
    a.seed = d.seed;
    a.sample_base = d.sample_base;
    a.S = (uint32_t)S;
    a.G = f.G;
    a.splits = f.splits;
    a.V = (int32_t)gr.V;
    a.k = k;
    for (int32_t i = 0; i < k; ++i) {
        a.m[i] = (uint32_t)fanout[i];
        a.W[i] = (uint32_t)W[i];
        a.div_m[i] = make_fastdiv(a.m[i]);
        a.div_w[i] = make_fastdiv(a.W[i]);
        a.out[i] = step_out[i];
    }
    a.lds_half = f.half;
    a.roots = roots;
    a.hdr = (WsHeader*)ws;
    a.flags = (uint32_t*)(ws + o_flags);
    a.parts = (uint32_t*)(ws + o_parts);
    a.o_flags = o_flags;
    a.o_parts = o_parts;
    a.status_out = status_out;
    mark_phase(ND_PHASE_SAMPLE_SUB, stream);
    const dim3 grid((unsigned)f.groups), block(kFusedThreads);
    const bool pairs = khop_in_pairs(a.m[k - 1], step_out[k - 1]);
    const int64_t draws = S * W[k - 1];
    const bool past = pairs ? draws >= kPastCaches || (k > 1 && last_level_is_passed(gr, draws))
                            : draws >= kPastCaches && gr.E <= kPastCachesOneByOne;
#define ND_FUSED_LAUNCH_R(STRIDE, R, PAST, OFFT)                                                                  \
    do {                                                                                                          \
        auto* kernel = a.packed.bytes ? &khop_fused_kernel<STRIDE, R, PAST, true, OFFT>                           \
                                      : &khop_fused_kernel<STRIDE, R, PAST, false, OFFT>;                         \
        hipLaunchKernelGGL(kernel, grid, block, f.lds, stream, view_of<OFFT>(gr), a);                             \
    } while (0)
#define ND_FUSED_LAUNCH(STRIDE, OFFT)                           \
    do {                                                        \
        if (pairs && past) ND_FUSED_LAUNCH_R(STRIDE, 2, true, OFFT);       \
        else if (pairs) ND_FUSED_LAUNCH_R(STRIDE, 2, false, OFFT);         \
        else if (past) ND_FUSED_LAUNCH_R(STRIDE, 1, true, OFFT);           \
        else ND_FUSED_LAUNCH_R(STRIDE, 1, false, OFFT);                    \
    } while (0)
    if (gr.off64) {
        if (gr.wq) ND_FUSED_LAUNCH(2, int64_t);
        else ND_FUSED_LAUNCH(1, int64_t);
    } else {
        if (gr.wq) ND_FUSED_LAUNCH(2, int32_t);
        else ND_FUSED_LAUNCH(1, int32_t);
    }
#undef ND_FUSED_LAUNCH
#undef ND_FUSED_LAUNCH_R
    ND_HIP_CHECK(hipGetLastError());
    return ND_OK;
}

int khop_first(const Graph& gr, const DrawArgs& d, int32_t m, int64_t S, const int32_t* roots, int32_t* out, StepCtl* ctl,
               uint32_t* status, hipStream_t stream) {
    const uint32_t n = (uint32_t)(S * m);  // below 2^31
    const int64_t per = kFusedThreads * 4;
    int64_t groups = (n + per - 1) / per;
    // Half of what a unit holds: each group adds to the counter of live pairs, and 233 K roots of 25 draws leave
    // after 5.6 rounds (the whole call 497 us, 502 to 507 with 2, 8 or 16 per unit).
    if (groups > (int64_t)gr.num_cus * 4) groups = (int64_t)gr.num_cus * 4;
    const FastDiv div_m = make_fastdiv((uint32_t)m);
    mark_phase(ND_PHASE_SAMPLE_SP, stream);
#define ND_FIRST_LAUNCH(PACKED, OFFT)                                                                              \
    hipLaunchKernelGGL((khop_first_kernel<PACKED, OFFT>), dim3((unsigned)groups), dim3(kFusedThreads), 0, stream,  \
                       view_of<OFFT>(gr), d.packed, d.seed, d.sample_base, roots, n, div_m, out, ctl, status)
    if (gr.off64) {
        if (d.packed.bytes) ND_FIRST_LAUNCH(true, int64_t);
        else ND_FIRST_LAUNCH(false, int64_t);
    } else {
        if (d.packed.bytes) ND_FIRST_LAUNCH(true, int32_t);
        else ND_FIRST_LAUNCH(false, int32_t);
    }
#undef ND_FIRST_LAUNCH
    ND_HIP_CHECK(hipGetLastError());
    return ND_OK;
}

// ---------------------------------------------------------------- unique neighbours
namespace {
struct UniqueShape {
    uint32_t slots, rows, threads;
    int64_t groups;   // workgroups
    size_t lds;
};
UniqueShape unique_shape(const Graph& gr, const int32_t* fanout, int32_t k, int64_t S) {
    int64_t W[ND_MAX_FANOUT_STEPS];
    slots_per_sample(fanout, k, W);
    int64_t widest = 1, rows = 1;
    for (int32_t i = 0; i < k; ++i) {
        if (W[i] > widest) widest = W[i];
        if (i + 1 < k && W[i] > rows) rows = W[i];
    }
    UniqueShape u;
    // Half a wavefront per sample up to 32 slots, a whole one up to 256.  Above, four where samples are few and
    // the time is that of one, two where they are many and what counts is how long lanes wait at barriers:
    // [25,20] of 1,000 vertices of a 57 K-vertex graph take 21.7 us with four and 25.1 with two, 3,000 44 and 34,
    // 20,000 220 and 150 (145 with one); [30,30] of 3,000 54 and 59, of 10,000 144 and 139, of 20,000 271 and 253.
    // Above 1,024 slots two would keep 16 slots per lane in registers.
    const bool many = S >= (int64_t)gr.num_cus * (widest <= 512 ? 8 : 32);
    u.threads = widest <= 32 ? 32 : widest <= 256 ? 64 : widest <= 1024 && many ? 128 : 256;
    u.slots = 32;
    while (u.slots < widest) u.slots <<= 1;
    u.rows = (uint32_t)(rows + 1) / 2 * 2;
    const int64_t subs = u.threads <= 64 ? 64 / u.threads : 1;
    u.lds = (size_t)subs * unique_group_bytes(u.slots, u.rows);
    u.groups = (S + subs - 1) / subs;
    if (u.groups > (int64_t)gr.num_cus * 128) u.groups = (int64_t)gr.num_cus * 128;  // groups walk over samples with a stride
    if (u.groups < 1) u.groups = 1;
    return u;
}
constexpr size_t kUniqueLdsMost = 128 << 10;
}  // namespace

// At most ND_MAX_UNIQUE_SLOTS slots per sample and hop (the call's plan has checked).
bool khop_unique_fits(const Graph& gr, const int32_t* fanout, int32_t k) {
    return gr.links && unique_shape(gr, fanout, k, 1).lds <= kUniqueLdsMost;
}

int64_t khop_unique_groups(const Graph& gr, const int32_t* fanout, int32_t k, int64_t S) {
    return unique_shape(gr, fanout, k, S).groups;
}

int khop_unique(const Graph& gr, const DrawArgs& d, const int32_t* fanout, int32_t k, int32_t rounds, int64_t S,
                const int32_t* roots, int32_t* const* step_out, char* ws, uint64_t o_flags, uint64_t o_parts,
                hipStream_t stream) {
    int64_t W[ND_MAX_FANOUT_STEPS];
    slots_per_sample(fanout, k, W);
    const UniqueShape u = unique_shape(gr, fanout, k, S);
    UniqueFusedArgs a{};
    a.links = gr.links;
    a.seed = d.seed;
    a.sample_base = d.sample_base;
    a.S = (uint32_t)S;
    a.V = (int32_t)gr.V;
    a.k = k;
    a.rounds = rounds;
    for (int32_t i = 0; i < k; ++i) {
        a.W[i] = (uint32_t)W[i];
        a.div_m[i] = make_fastdiv((uint32_t)fanout[i]);
        a.out[i] = step_out[i];
    }
    a.slots = u.slots;
    a.rows = u.rows;
    a.roots = roots;
    a.hdr = (WsHeader*)ws;
    a.flags = (uint32_t*)(ws + o_flags);
    a.parts = (uint32_t*)(ws + o_parts);
    a.o_flags = o_flags;
    a.o_parts = o_parts;
    mark_phase(ND_PHASE_UNIQUE, stream);
    // outputs of groups inside a wavefront: every vertex of R-MAT 22, [25,10], 4,460 us and 4,340, one draw per slot 3,550 and 3,390,
    // [25] 1,152 and 1,127, 1 M vertices of [60] 400 and 380
    const bool past = last_level_is_passed(gr, S * W[k - 1]);
#define ND_UNIQUE_ONE(STRIDE, OFFT, THREADS, PER)                                                                  \
    do {                                                                                                           \
        auto* kernel = past ? &khop_unique_kernel<STRIDE, OFFT, THREADS, PER, true> : &khop_unique_kernel<STRIDE, OFFT, THREADS, PER>; \
        hipLaunchKernelGGL(kernel, dim3((unsigned)u.groups), dim3(64), u.lds, stream, view_of<OFFT>(gr), a);       \
    } while (0)
#define ND_UNIQUE_GO(STRIDE, OFFT, THREADS, PER)                                                                   \
    hipLaunchKernelGGL((khop_unique_kernel<STRIDE, OFFT, THREADS, PER>), dim3((unsigned)u.groups), dim3(THREADS), u.lds, \
                       stream, view_of<OFFT>(gr), a)
#define ND_UNIQUE_SIZE(STRIDE, OFFT)                                    \
    do {                                                                \
        if (u.slots <= 32) ND_UNIQUE_ONE(STRIDE, OFFT, 32, 1);          \
        else if (u.slots <= 64) ND_UNIQUE_ONE(STRIDE, OFFT, 64, 1);     \
        else if (u.slots <= 128) ND_UNIQUE_ONE(STRIDE, OFFT, 64, 2);    \
        else if (u.slots <= 256) ND_UNIQUE_ONE(STRIDE, OFFT, 64, 4);    \
        else if (u.threads == 128 && u.slots <= 512) ND_UNIQUE_GO(STRIDE, OFFT, 128, 4); \
        else if (u.threads == 128) ND_UNIQUE_GO(STRIDE, OFFT, 128, 8);  \
        else if (u.slots <= 512) ND_UNIQUE_GO(STRIDE, OFFT, 256, 2);    \
        else if (u.slots <= 1024) ND_UNIQUE_GO(STRIDE, OFFT, 256, 4);   \
        else ND_UNIQUE_GO(STRIDE, OFFT, 256, 8);                        \
    } while (0)
    if (gr.off64) {
        if (gr.wq) ND_UNIQUE_SIZE(2, int64_t);
        else ND_UNIQUE_SIZE(1, int64_t);
    } else {
        if (gr.wq) ND_UNIQUE_SIZE(2, int32_t);
        else ND_UNIQUE_SIZE(1, int32_t);
    }
    ND_HIP_CHECK(hipGetLastError());
    return ND_OK;
}

// Dynamic LDS above the 64 KB default has to be allowed once per kernel (samples of 1,025 to 2,048 slots
// use more); done when a graph is created, so that the call itself only launches.
int khop_prepare() {
#define ND_UNIQUE_ALLOW(STRIDE, OFFT)                                                                             \
    ND_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(&khop_unique_kernel<STRIDE, OFFT, 256, 8>),    \
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kUniqueLdsMost))
    ND_UNIQUE_ALLOW(1, int64_t);
    ND_UNIQUE_ALLOW(2, int64_t);
    ND_UNIQUE_ALLOW(1, int32_t);
    ND_UNIQUE_ALLOW(2, int32_t);
#undef ND_UNIQUE_ALLOW
    return ND_OK;
}

}  // namespace nd
