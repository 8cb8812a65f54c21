// Edges between consecutive layers (Section 4.2 of the paper, "Importance
// Sampling": in FastGCN / LADIES style sampling every sample carries the
// adjacency matrix between the transits of a step and the vertices the step
// added; the paper's `next` adds an edge between the new vertex and every
// transit that has it as a neighbour).
//
// The paper's kernel tests each new vertex against each transit.  Here one
// workgroup per sample puts the sample's new vertices into an LDS hash table
// once and then streams the adjacency lists of the sample's transits through
// it, 64 consecutive (coalesced) entries per wavefront load, so the cost is
// per adjacency entry instead of a binary search per (transit, new vertex) pair.
//
// Output is one CSR over the rows (sample, transit slot).  A row lists the new
// slots j whose vertex is a neighbour of the row's transit, ordered by (vertex
// id, j) - the order a walk down the ascending adjacency list meets them - so
// the result is unique.  A hash table maps a vertex to its slots, which lie together and ascending.
//
// Nine adjacency entries in ten are of no sample vertex, and the kernel is bound by instruction issue
// (scalar instructions as much as vector ones) before the 4 bytes per entry it streams.  So an entry first tests one
// bit of a 65,536-bit map of the sample's vertices (no loop, no divergence); the few that pass are packed, in order,
// into a queue of the wavefront in LDS, and the table is probed by a full wavefront of queued entries at a time.
// The map's bits are hashed from the whole id: 512 samples of 2,048 transits and vertices on a graph whose ids are
// multiples of 64, where bits of the id let 39 % of the entries pass, count in 674 us (2,070) and fill in 866 (2,200), with
// ids in 64 blocks 2^16 apart 705 (2,720) and 894 (3,480); on relabelled ids both are as fast.
// Whether there are as many is asked once for two or four loads of 64 entries, whose looks at the map then wait for LDS
// together, and full steps have code of their own, without a test of where the list ends.  Counting pass of 4,096
// samples of 2,048 transits and vertices (10 GB of lists): 2.12 ms with one load at a time and the lists' places fetched
// one after the other, 1.46 like this (6.9 TB/s; the loads alone, without the test, 1.44; loads of 16 bytes per lane
// 1.47).  L2 serves one look in eight, and vector instructions issue in 0.89 of the cycles.  The filling pass is at 2.02
// (3.08 so), of which its stores are 0.65.
//
// The sample's transit slots are grouped by vertex as well: a vertex that several slots hold (layer
// samples hold well-connected vertices many times over) is streamed once, and what is found goes to
// the row of each of those slots.  The wavefronts take the distinct transits from a counter.
//
// Two passes share the kernel: counting (row sizes, then a device-wide
// exclusive scan into 64-bit row pointers) and filling.
#include <type_traits>

#include "nd_common.h"
#include "nd_edges.h"
#include "nd_places.h"
#include "nd_wave.h"

namespace nd {

namespace {

constexpr int kEdgeThreads = 1024;  // two workgroups (77 KB of LDS each) fill a CU's 32 wave slots
constexpr int kBitWords = 2048;     // the vertex map: 65,536 bits
constexpr int kMaxSlots = 2048;     // new vertices per sample (ND_MAX_EDGE_SLOTS)
constexpr int kTable = 2 * kMaxSlots;
constexpr int kChunk = 2048;        // transit slots of a sample that are grouped together
constexpr uint32_t kRun = 64;       // slots of a vertex up to which each of them looks at all the others
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;

struct EdgeArgs {
    const int32_t* transits;  // [S][n_prev]
    const int32_t* sampled;   // [S][m]
    uint32_t n_prev, m;
    uint32_t table;           // places of the vertices' table: a power of two, at least 2 m
    uint32_t shift;           // 32 - log2(table)
    int32_t* counts;          // count pass: [S * n_prev]
    const int64_t* row_ptr;   // fill pass
    int32_t* edge_slot;
    int64_t capacity;
    uint32_t* status;
};

// What a workgroup keeps in LDS.  PIECES: wavefront loads of 64 entries between two looks at the queue's fill.
template <bool FILL>
struct EdgeLds {
    static constexpr int kPieces = FILL ? 2 : 4;
    static constexpr uint32_t kQueue = 64 + 64 * kPieces;  // fewer than 64 left over, the entries of the pieces, a spare place
    static constexpr uint32_t kOut = 64 + 64;              // filling pass: edges of the current item not yet written
    uint32_t bits[kBitWords];       // bit set: a vertex of the sample may be there
    uint32_t keys[kTable];          // the sample's vertices, hashed; kNoKey = free
    uint16_t first[kTable + 8];     // slots of the vertices in the places before (while they are counted: in this place)
    union {
        uint32_t t_keys[2 * kChunk];                        // the chunk's transits, hashed; then, per distinct transit:
        struct { uint32_t rs[kChunk], deg[kChunk]; } item;  // its list: low word of the start, length
    };
    uint16_t t_first[kChunk];       // its first place in t_slot, and from bit 11 on the start's bits from 32 on
    uint16_t t_slot[kChunk];        // the chunk's live slots, those of one transit together
    uint16_t slot[FILL ? kMaxSlots : 2];                    // the sample's slots, those of one vertex together and ascending
    uint16_t out[FILL ? (kEdgeThreads / 64) * kOut : 2];    // per wavefront: edges waiting to be written
    union {
        uint32_t queue[(kEdgeThreads / 64) * kQueue];       // per wavefront: entries that passed the bit test
        uint16_t t_count[2 * kChunk];                       // while transits are grouped: slots, then the item, per place
    };
    uint64_t scan[kEdgeThreads / 64 + 1];
    uint32_t items, live;           // distinct transits and live slots of the chunk
    uint32_t next;                  // next item to hand out
    uint32_t long_runs;             // filling pass: a vertex of the sample is held by more than kRun slots
};
static_assert(sizeof(EdgeLds<true>) <= 80 * 1024 && sizeof(EdgeLds<false>) <= 80 * 1024, "two workgroups per compute unit");

constexpr uint32_t kNoKey = 0xFFFFFFFFu;
__device__ __forceinline__ uint32_t hash_vertex(int32_t v) { return (uint32_t)v * 0x9E3779B1u; }

// one wavefront: its LDS operations complete in order; keeps the compiler from moving them
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Puts v (>= 0) into a table of at least twice as many places as vertices and adds one to its 16-bit count; the place
// in the low half of the result, in the high half how many came before.
__device__ __forceinline__ uint32_t count_key(uint32_t* keys, uint16_t* counts, uint32_t mask, uint32_t shift, int32_t v) {
    uint32_t pos = hash_vertex(v) >> shift;
    for (;;) {  // ends: the table is never full
        const uint32_t old = atomicCAS(&keys[pos], kNoKey, (uint32_t)v);
        if (old == kNoKey || old == (uint32_t)v) break;
        pos = (pos + 1u) & mask;
    }
    const uint32_t half = (pos & 1u) * 16u;  // at most 2,048 per count: no carry into the other half
    const uint32_t before = atomicAdd((uint32_t*)counts + (pos >> 1), 1u << half) >> half;
    return pos | (before << 16);
}

// Two workgroups of 1,024 threads per compute unit are eight wavefronts per SIMD.  That takes at most
// 64 vector registers and, on this register file (800 scalar registers per SIMD), at most 96 scalar
// registers per wavefront: left to itself the compiler uses more scalar registers than that, which
// silently halves the occupancy, so the bound is stated (the surplus goes to lanes of a vector register; of the set-up's
// vector registers 2 and, in the filling pass, 12 go to memory, none of the loop's).
template <typename OffT, bool FILL>
__global__ __launch_bounds__(kEdgeThreads) __attribute__((amdgpu_waves_per_eu(8, 8)))
void edges_kernel(GraphView<OffT> g, EdgeArgs a) {
    using Lds = EdgeLds<FILL>;
    __shared__ Lds s;
    constexpr uint32_t T = (uint32_t)kEdgeThreads;
    constexpr int kPieces = Lds::kPieces;
    // Adjacency loads in flight per lane and step
    constexpr int kEdgeUnroll = 8;
    constexpr uint32_t kBatch = 64 * kEdgeUnroll;  // adjacency entries a wavefront takes per step
    const uint32_t b = blockIdx.x;
    const uint32_t tid = threadIdx.x;
    const int lane = lane_id();
    const uint32_t wave = wave_uniform((uint32_t)wave_id());
    const uint32_t mask = a.table - 1u;
    const uint64_t row0 = (uint64_t)b * a.n_prev;
    bool bad = false;
    auto checked = [&](int32_t v) -> int32_t {  // NULL instead of what is no vertex
        const bool out = v >= g.V || v < ND_NULL_VERTEX;
        bad |= out;
        return out ? ND_NULL_VERTEX : v;
    };
    uint32_t* queue = s.queue + wave * Lds::kQueue;
    uint16_t* obuf = s.out + (FILL ? wave * Lds::kOut : 0u);

    for (uint32_t chunk0 = 0; chunk0 < a.n_prev; chunk0 += (uint32_t)kChunk) {
        // ---- The sample's vertices (once) and kChunk transit slots at a time are grouped by a hash table each: layer
        // samples hold well-connected vertices many times over (569 distinct among the 2,048 transits of the
        // benchmark's second step), and a vertex's adjacency list is streamed once for all the slots that hold it.
        // Groups need no order among each other, so this takes a table's insertions and one scan of its places where a
        // sort by vertex took three passes (4,096 samples of 64 transits and 2,048 vertices, 2,400 entries to stream:
        // the counting pass 245 us with sorts, 135 like this).
        const bool first = chunk0 == 0;
        const uint32_t n_chunk = a.n_prev - chunk0 < (uint32_t)kChunk ? a.n_prev - chunk0 : (uint32_t)kChunk;
        uint32_t t_table = 128, t_shift = 25;
        while (t_table < 2u * n_chunk) {
            t_table <<= 1;
            --t_shift;
        }
        int32_t v[2], t[2];
#pragma unroll
        for (uint32_t e = 0; e < 2u; ++e) {
            const uint32_t i = tid + e * T;
            v[e] = t[e] = ND_NULL_VERTEX;
            if (first && i < a.m) v[e] = checked(a.sampled[(uint64_t)b * a.m + i]);
            if (i < n_chunk) t[e] = checked(a.transits[row0 + chunk0 + i]);
            if (!FILL && i < n_chunk && t[e] < 0) a.counts[row0 + chunk0 + i] = 0;  // a slot without a transit has no edges
        }
        bool edges[2] = {true, true};  // filling pass: the counting pass found edges for this slot
        if (FILL) {
#pragma unroll
            for (uint32_t e = 0; e < 2u; ++e)
                if (t[e] >= 0) {
                    const int64_t* r = a.row_ptr + row0 + chunk0 + tid + e * T;
                    edges[e] = r[0] != r[1];
                }
        }
        const uint4 none = make_uint4(kNoKey, kNoKey, kNoKey, kNoKey);
        if (first) {
            for (uint32_t i = tid; i < a.table / 4u; i += T) {
                reinterpret_cast<uint4*>(s.keys)[i] = none;
                reinterpret_cast<uint2*>(s.first)[i] = make_uint2(0u, 0u);
            }
            for (uint32_t i = tid; i < (uint32_t)kBitWords; i += T) s.bits[i] = 0u;
            if (FILL && tid == 0) s.long_runs = 0u;
        }
        for (uint32_t i = tid; i < t_table / 4u; i += T) {
            reinterpret_cast<uint4*>(s.t_keys)[i] = none;
            reinterpret_cast<uint2*>(s.t_count)[i] = make_uint2(0u, 0u);
        }
        __syncthreads();
        uint32_t vp[2] = {0u, 0u}, tp[2] = {0u, 0u};  // place, and how many of the vertex came before
#pragma unroll
        for (uint32_t e = 0; e < 2u; ++e) {
            if (v[e] >= 0) vp[e] = count_key(s.keys, s.first, mask, a.shift, v[e]);
            if (t[e] >= 0) tp[e] = count_key(s.t_keys, s.t_count, t_table - 1u, t_shift, t[e]);
        }
        __syncthreads();
        {   // four places of each table per thread
            uint4 vk = none, tk = none;
            uint2 vc = make_uint2(0u, 0u), tc = make_uint2(0u, 0u);
            if (first && tid < a.table / 4u) {
                vk = reinterpret_cast<const uint4*>(s.keys)[tid];
                vc = reinterpret_cast<const uint2*>(s.first)[tid];
            }
            if (tid < t_table / 4u) {
                tk = reinterpret_cast<const uint4*>(s.t_keys)[tid];
                tc = reinterpret_cast<const uint2*>(s.t_count)[tid];
            }
            const uint32_t vkey[4] = {vk.x, vk.y, vk.z, vk.w}, tkey[4] = {tk.x, tk.y, tk.z, tk.w};
            const uint32_t vcnt[4] = {vc.x & 0xFFFFu, vc.x >> 16, vc.y & 0xFFFFu, vc.y >> 16};
            const uint32_t tcnt[4] = {tc.x & 0xFFFFu, tc.x >> 16, tc.y & 0xFFFFu, tc.y >> 16};
            // one scan for the three sums (each at most 2,048): the sample's slots, the chunk's live slots and its items
            uint64_t mine = 0, total;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                mine += (uint64_t)vcnt[j] | ((uint64_t)tcnt[j] << 16) | ((uint64_t)(tcnt[j] > 0u ? 1u : 0u) << 32);
            const uint64_t ex = block_exclusive_scan<uint64_t, kEdgeThreads>(mine, s.scan, &total);
            if (first && tid < a.table / 4u) {
                uint32_t at = (uint32_t)ex & 0xFFFFu;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    s.first[tid * 4u + (uint32_t)j] = (uint16_t)at;
                    at += vcnt[j];
                    if (FILL && vcnt[j] > kRun) s.long_runs = 1u;
                    if (vkey[j] != kNoKey) {
                        const uint32_t h = edge_map_hash((int32_t)vkey[j]);
                        atomicOr(&s.bits[edge_map_word(h)], 0x80000000u >> edge_map_bit(h));
                    }
                }
                if (tid == a.table / 4u - 1u) s.first[a.table] = (uint16_t)at;
            }
            if (tid < t_table / 4u) {
                uint32_t at = (uint32_t)(ex >> 16) & 0xFFFFu, it = (uint32_t)(ex >> 32);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (tcnt[j] == 0u) continue;
                    const uint64_t rs = (uint64_t)g.off[tkey[j]];
                    s.item.rs[it] = (uint32_t)rs;
                    s.item.deg[it] = row_length(g, (int32_t)tkey[j], rs);
                    // a device holds fewer than 2^37 columns (512 GiB)
                    s.t_first[it] = (uint16_t)(at | ((uint32_t)(rs >> 32) << 11));
                    s.t_count[tid * 4u + (uint32_t)j] = (uint16_t)it;
                    at += tcnt[j];
                    ++it;
                }
            }
            if (tid == 0) {
                s.live = (uint32_t)(total >> 16) & 0xFFFFu;
                s.items = (uint32_t)(total >> 32);
                s.next = 0;
            }
        }
        __syncthreads();
#pragma unroll
        for (uint32_t e = 0; e < 2u; ++e) {
            if (t[e] >= 0) {
                const uint32_t it = s.t_count[tp[e] & 0xFFFFu], before = tp[e] >> 16;
                s.t_slot[(s.t_first[it] & 0x7FFu) + before] = (uint16_t)(tid + e * T);
                if (FILL && before == 0u && !edges[e]) s.item.deg[it] = 0u;  // nothing to look for
            }
            if (FILL && v[e] >= 0) s.slot[s.first[vp[e] & 0xFFFFu] + (vp[e] >> 16)] = (uint16_t)(tid + e * T);
        }
        if (FILL && first) {  // the slots of a vertex, in any order yet: each counts the lower ones
            // Of more than kRun slots in a bitmap of theirs, 2,048 bits in the queues' LDS: every such run has a multiple of kRun
            // among its places, and the first one names its bitmap (512 samples of 64 transits and 2,048 slots that all hold
            // one vertex, no edges: 167 us when each slot looks at every other, 32 like this, 20 with different vertices).
            constexpr uint32_t kWords = kMaxSlots / 32;
            static_assert(kMaxSlots / kRun * kWords * 4 <= sizeof(s.queue), "a bitmap for every multiple");
            __syncthreads();
            const bool long_runs = wave_uniform(s.long_runs) != 0u;
            if (long_runs) {
                for (uint32_t i = tid; i < kMaxSlots / kRun * kWords; i += T) s.queue[i] = 0u;
                __syncthreads();
#pragma unroll
                for (uint32_t e = 0; e < 2u; ++e)
                    if (v[e] >= 0) {
                        const uint32_t k = s.first[vp[e] & 0xFFFFu], end = s.first[(vp[e] & 0xFFFFu) + 1u];
                        if (end - k > kRun) atomicOr(&s.queue[(k + kRun - 1u) / kRun * kWords + ((tid + e * T) >> 5)], 1u << (tid & 31u));
                    }
                __syncthreads();
            }
            uint32_t at[2] = {0u, 0u};
#pragma unroll
            for (uint32_t e = 0; e < 2u; ++e)
                if (v[e] >= 0) {
                    const uint32_t k = s.first[vp[e] & 0xFFFFu], end = s.first[(vp[e] & 0xFFFFu) + 1u], slot = tid + e * T;
                    at[e] = k;
                    if (long_runs && end - k > kRun) {
                        const uint32_t* map = s.queue + (k + kRun - 1u) / kRun * kWords;
                        for (uint32_t w = 0; w < slot >> 5; ++w) at[e] += (uint32_t)__popc(map[w]);
                        at[e] += (uint32_t)__popc(map[slot >> 5] & ((1u << (slot & 31u)) - 1u));
                    } else {
                        for (uint32_t i = k; end - k > 1u && i < end; ++i) at[e] += s.slot[i] < slot ? 1u : 0u;
                    }
                }
            __syncthreads();
#pragma unroll
            for (uint32_t e = 0; e < 2u; ++e)
                if (v[e] >= 0) s.slot[at[e]] = (uint16_t)(tid + e * T);
        }
        __syncthreads();
        const uint32_t n_items = wave_uniform(s.items);
        const uint32_t n_live = wave_uniform(s.live);  // the live slots are the first n_live of t_slot
        const uint64_t row1 = row0 + chunk0;

        // ---- The wavefronts take the items from a counter: lists differ in length by orders of magnitude, and a fixed
        // share per wavefront leaves most of them waiting for the slowest.  Everything about an item is the same in all
        // lanes of its wavefront and is kept in scalar registers.  The loop runs over steps of up to kBatch entries of a
        // list; the entries of the next step (the same item's or the next item's) are requested before the current
        // step is worked on.
        auto claim = [&]() -> uint32_t {
            uint32_t i = 0;
            if (lane == 0) i = atomicAdd(&s.next, 1u);
            return wave_uniform(i);
        };
        uint32_t item = claim();
        uint32_t item_next = claim();
        uint32_t p0 = 0, p1 = 0;    // positions [p0, p1) of t_slot hold the slots of the item being requested
        uint64_t rs = 0;            // where its list starts
        uint32_t deg = 0;           // how long it is (0: nothing to stream); a list has fewer than 2^31 entries
        uint32_t e0 = 0;            // the next entry of it to request
        // Filling pass: the chunk's rows lie together, in at most 16 MB, so that a place among them is a 32-bit offset (in
        // bytes), and a store beyond them or the capacity is one that the buffer drops.
        int64_t base = 0;
        uint32_t bytes = 0;
        if constexpr (FILL) {
            base = a.row_ptr[row1];
            const int64_t end = a.row_ptr[row1 + n_chunk] < a.capacity ? a.row_ptr[row1 + n_chunk] : a.capacity;
            const int64_t room = end > base ? (end - base) * 4 : 0;
            bytes = room < 0x7FFFFFFCll ? (uint32_t)room : 0x7FFFFFFCu;
        }
        const auto rows = __builtin_amdgcn_make_buffer_rsrc(a.edge_slot + (bytes > 0u ? base : 0), 0, (int)bytes, 0x00027000);
        uint32_t my_row = 0, row_next = 0;  // filling pass: where the row of the item's slot number `lane` starts
        auto adopt = [&]() {        // `item` becomes the item being requested
            e0 = 0;
            deg = 0;
            if (item < n_items) {
                const uint32_t f = wave_uniform((uint32_t)s.t_first[item]);
                rs = ((uint64_t)(f >> 11) << 32) | wave_uniform(s.item.rs[item]);
                deg = wave_uniform(s.item.deg[item]);
                p0 = f & 0x7FFu;
                p1 = item + 1u < n_items ? wave_uniform((uint32_t)s.t_first[item + 1u]) & 0x7FFu : n_live;
                if (FILL && deg > 0u && p0 + (uint32_t)lane < p1) row_next = (uint32_t)(a.row_ptr[row1 + s.t_slot[p0 + (uint32_t)lane]] - base) * 4u;
            }
        };
        // an item without entries to stream: its slots' counts are 0 (counting pass), nothing else
        auto next_item = [&]() {
            do {
                item = item_next;
                item_next = claim();
                adopt();
                if (!FILL && item < n_items && deg == 0u)
                    for (uint32_t d = p0 + (uint32_t)lane; d < p1; d += 64u) a.counts[row1 + s.t_slot[d]] = 0;
            } while (item < n_items && deg == 0u);
        };
        auto request_entries = [&](int32_t (&u)[kEdgeUnroll]) {
            const int32_t* p = g.col + rs + e0;
            const uint32_t left = deg - e0;
            if (left >= kBatch) {  // a full step, the common case: nothing to test
#pragma unroll
                for (int r = 0; r < kEdgeUnroll; ++r) u[r] = p[r * 64 + lane];
                return;
            }
#pragma unroll
            for (int r = 0; r < kEdgeUnroll; ++r) {
                // the test is the same in all lanes; inside the last 64 entries a lane past the end
                // reads the last entry again instead of branching (and drops it when it looks at it:
                // looking at it here would wait for each load in turn)
                if ((uint32_t)r * 64u < left) {
                    const uint32_t e = (uint32_t)r * 64u + (uint32_t)lane;
                    u[r] = p[e < left ? e : left - 1u];
                }
            }
        };

        adopt();
        if (item < n_items && deg == 0u) {
            if (!FILL)
                for (uint32_t d = p0 + (uint32_t)lane; d < p1; d += 64u) a.counts[row1 + s.t_slot[d]] = 0;
            next_item();
        }
        int32_t u_next[kEdgeUnroll];
#pragma unroll
        for (int r = 0; r < kEdgeUnroll; ++r) u_next[r] = 0;
        if (item < n_items) request_entries(u_next);
        my_row = row_next;

        uint32_t queued = 0;  // entries in the queue (the same in all lanes)
        uint32_t count = 0;   // counting pass: my share of the item's edges
        uint32_t done = 0;    // filling pass: edges of the item written so far (to each of its slots' rows)
        uint32_t ofill = 0;   // filling pass: edges of the item waiting in obuf
        while (item < n_items) {
            // ---- the step whose entries have been requested
            int32_t u[kEdgeUnroll];
#pragma unroll
            for (int r = 0; r < kEdgeUnroll; ++r) {
                u[r] = u_next[r];
                // taken here, before the requests below are issued: loads return in order, and a wait
                // for these entries placed after those requests would wait for them as well
                asm volatile("" : "+v"(u[r]));
            }
            const uint32_t cnt = deg - e0;
            const bool row_ends = cnt <= kBatch;
            const uint32_t q0 = p0, q1 = p1;  // the slots of the item being worked on
            // ---- request the next step's entries before working on this one
            if (row_ends) next_item();
            else e0 += kBatch;
            if (item < n_items) request_entries(u_next);

            // ---- entries that pass the bit test join the queue, in order; the table is probed by 64 queued entries at a
            // time (by what is left when the item ends).
            // Filling pass: the edges found are collected in obuf, in order, and leave 64 at a time, one
            // coalesced store per slot that holds the item's transit.
            // The first nf (at most 64) entries of obuf, to every row of the item: a store per row whose place is one scalar
            // (4,096 samples of 2,048 transits and vertices: 2.35 ms with 64-bit places and their bounds per lane, 2.16 like this;
            // two to eight short rows per store 2.18, and stores held back until after the next wait 2.5).
            auto write_out = [&](uint32_t nf) {
                const int32_t val = (uint32_t)lane < nf ? (int32_t)obuf[lane] : 0;
                for (uint32_t d0 = q0; d0 < q1; d0 += 64u) {
                    // the rows of up to 64 slots at a time: their starts come by one load, a lane per slot
                    const uint32_t nd = q1 - d0 < 64u ? q1 - d0 : 64u;
                    uint32_t row = my_row;
                    if (d0 > q0 && (uint32_t)lane < nd) row = (uint32_t)(a.row_ptr[row1 + s.t_slot[d0 + (uint32_t)lane]] - base) * 4u;
                    row += done * 4u;
                    if (__ballot((uint32_t)lane < nd && row + nf * 4u > bytes) == 0ull) {
                        if ((uint32_t)lane < nf)
                            for (uint32_t dd = 0; dd < nd; ++dd)
                                __builtin_amdgcn_raw_buffer_store_b32(val, rows, lane * 4, __builtin_amdgcn_readlane((int)row, (int)dd), 0);
                    } else {  // the capacity ends in or before one of these rows
                        for (uint32_t dd = 0; dd < nd; ++dd) {
                            const uint32_t to = (uint32_t)__builtin_amdgcn_readlane((int)row, (int)dd) + (uint32_t)lane * 4u;
                            if ((uint32_t)lane < nf && to < bytes) __builtin_amdgcn_raw_buffer_store_b32(val, rows, (int)to, 0, 0);
                        }
                    }
                }
                done += nf;
            };
            auto leave = [&]() {  // a full wavefront of edges leaves, the rest moves to the front
                wave_lds_order();
                if (ofill >= 64u) {
                    write_out(64u);
                    const uint16_t moved = (uint32_t)lane < ofill - 64u ? obuf[64 + lane] : (uint16_t)0;
                    wave_lds_order();
                    if ((uint32_t)lane < ofill - 64u) obuf[lane] = moved;
                    ofill -= 64u;
                    wave_lds_order();
                }
            };
            auto probe = [&](uint32_t from, uint32_t n) {  // n (at most 64) queued entries
                const int32_t w = (uint32_t)lane < n ? (int32_t)queue[from + (uint32_t)lane] : ND_NULL_VERTEX;
                uint32_t c = 0, k = 0;
                if (w >= 0) {
                    uint32_t pos = hash_vertex(w) >> a.shift, key;
                    while ((key = s.keys[pos]) != (uint32_t)w && key != kNoKey) pos = (pos + 1u) & mask;  // never full
                    if (key == (uint32_t)w) {
                        k = s.first[pos];
                        c = s.first[pos + 1u] - k;
                    }
                }
                if constexpr (FILL) {
                    // the lanes hold runs (k, c); their entries go to obuf in lane order, 64 positions
                    // at a time: a lane with a short run writes it itself, a long run (a vertex held by
                    // many slots) is spread by a search over the running sums
                    const uint32_t incl = wave_inclusive_scan(c, lane);
                    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                    const uint32_t ex = incl - c;
                    if (total <= 64u && __ballot(c > 8u) == 0ull) {
                        for (uint32_t i = 0; __ballot(i < c) != 0ull; ++i)
                            if (i < c) obuf[ofill + ex + i] = s.slot[k + i];
                        ofill += total;
                        leave();
                    } else {
                        for (uint32_t base = 0; base < total; base += 64u) {
                            const uint32_t p = base + lane;
                            uint32_t owner = 0;
#pragma unroll
                            for (uint32_t step = 32; step > 0; step >>= 1)
                                if (__shfl(incl, (int)(owner + step - 1), 64) <= p) owner += step;
                            owner &= 63u;
                            const uint32_t ok = __shfl(k, (int)owner, 64);
                            const uint32_t oex = __shfl(ex, (int)owner, 64);
                            const uint32_t nb = total - base < 64u ? total - base : 64u;
                            if (p < total) obuf[ofill + lane] = s.slot[ok + (p - oex)];
                            ofill += nb;
                            leave();
                        }
                    }
                } else {
                    count += c;
                }
            };
            auto pieces = [&](auto full) {
                constexpr bool FULL = decltype(full)::value;
#pragma unroll
                for (int r0 = 0; r0 < kEdgeUnroll; r0 += kPieces) {
                    if (!FULL && (uint32_t)r0 * 64u >= cnt) break;  // the same for the whole wavefront
                    uint32_t word[kPieces];
#pragma unroll
                    for (int r = 0; r < kPieces; ++r) word[r] = s.bits[edge_map_word(edge_map_hash(u[r0 + r]))];
#pragma unroll
                    for (int r = 0; r < kPieces; ++r) {
                        const bool pass = (int32_t)(word[r] << edge_map_bit(edge_map_hash(u[r0 + r]))) < 0;
                        uint64_t votes = __ballot(pass);
                        if (!FULL) {
                            // The lanes past the list's end are struck from the votes and not from `pass`: such a lane that
                            // passes writes to the place after the last live entry (at most the spare one), which
                            // nothing reads.
                            const uint32_t at = (uint32_t)(r0 + r) * 64u, live = cnt > at ? cnt - at : 0u;
                            votes &= live >= 64u ? ~0ull : (1ull << live) - 1ull;
                        }
                        const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(votes >> 32),
                                                                      __builtin_amdgcn_mbcnt_lo((uint32_t)votes, queued));
                        // no branch: a lane that does not pass writes to the queue's spare last place
                        queue[pass ? at : Lds::kQueue - 1u] = (uint32_t)u[r0 + r];
                        queued += (uint32_t)__popcll(votes);
                    }
                    if (queued >= 64u) {
                        wave_lds_order();
                        uint32_t from = 0;
                        do {
                            probe(from, 64u);
                            from += 64u;
                        } while (queued - from >= 64u);
                        // what is left of the queue moves to the front
                        queued -= from;
                        const uint32_t moved = (uint32_t)lane < queued ? queue[from + (uint32_t)lane] : 0u;
                        wave_lds_order();
                        if ((uint32_t)lane < queued) queue[lane] = moved;
                        wave_lds_order();
                    }
                }
            };
            if (cnt >= kBatch) pieces(std::true_type{});
            else pieces(std::false_type{});
            if (row_ends) {  // the item ends
                if (queued > 0u) {
                    wave_lds_order();
                    probe(0u, queued);
                    queued = 0;
                }
                if constexpr (!FILL) {
                    const uint32_t incl = wave_inclusive_scan(count, lane);
                    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                    for (uint32_t d = q0 + (uint32_t)lane; d < q1; d += 64u) a.counts[row1 + s.t_slot[d]] = (int32_t)total;
                    count = 0;
                } else {
                    if (ofill > 0u) {
                        wave_lds_order();
                        write_out(ofill);
                    }
                    ofill = 0;
                    done = 0;
                    my_row = row_next;
                }
                wave_lds_order();
            }
        }
        __syncthreads();  // the chunk's transits and the queues' LDS are replaced by the next chunk's
    }
    if (bad && a.status) atomicOr(a.status, 1u);
}

__global__ void edges_clear_status_kernel(uint32_t* status) { *status = 0u; }

// ---- exclusive scan of n int32 counts into n + 1 int64 row pointers (reduce, scan the tile
// sums in one workgroup, scan again with the tile's base)
__global__ __launch_bounds__(kScanThreads) void scan_sums_kernel(const int32_t* counts, int64_t n,
                                                                 int64_t* sums) {
    __shared__ int64_t tmp[kScanThreads / 64 + 1];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    int64_t s = 0;
    for (int i = 0; i < kScanItems; ++i) {
        const int64_t p = base + (int64_t)i * kScanThreads + threadIdx.x;
        if (p < n) s += counts[p];
    }
    int64_t total;
    block_exclusive_scan<int64_t, kScanThreads>(s, tmp, &total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanThreads) void scan_top_kernel(int64_t* sums, int64_t tiles) {
    __shared__ int64_t tmp[kScanThreads / 64 + 1];
    int64_t carry = 0;
    for (int64_t base = 0; base < tiles; base += kScanThreads) {
        const int64_t p = base + threadIdx.x;
        const int64_t x = p < tiles ? sums[p] : 0;
        int64_t total;
        const int64_t ex = block_exclusive_scan<int64_t, kScanThreads>(x, tmp, &total);
        if (p < tiles) sums[p] = carry + ex;
        carry += total;
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[tiles] = carry;
}

// Four consecutive counts per thread and round, so that 32 bytes per lane leave next to each other (8.4 M rows: 57 us
// with 16 consecutive counts per thread, 20 like this).
__global__ __launch_bounds__(kScanThreads) void scan_write_kernel(const int32_t* counts, int64_t n,
                                                                 const int64_t* sums, int64_t tiles,
                                                                 int64_t* row_ptr) {
    typedef int64_t Pair __attribute__((ext_vector_type(2), aligned(8)));
    __shared__ int64_t tmp[kScanThreads / 64 + 1];
    int64_t carry = sums[blockIdx.x];
    for (int i = 0; i < kScanItems; i += 4) {
        const int64_t at = (int64_t)blockIdx.x * kScanTile + (int64_t)i * kScanThreads + (int64_t)threadIdx.x * 4;
        int4 c = make_int4(0, 0, 0, 0);
        if (at + 4 <= n) {
            c = *reinterpret_cast<const int4*>(counts + at);
        } else {
            if (at < n) c.x = counts[at];
            if (at + 1 < n) c.y = counts[at + 1];
            if (at + 2 < n) c.z = counts[at + 2];
        }
        int64_t total;
        const int64_t run = carry + block_exclusive_scan<int64_t, kScanThreads>((int64_t)c.x + c.y + c.z + c.w, tmp, &total);
        const Pair a = {run, run + c.x}, b = {run + c.x + c.y, run + c.x + c.y + c.z};
        if (at + 4 <= n) {
            *reinterpret_cast<Pair*>(row_ptr + at) = a;
            *reinterpret_cast<Pair*>(row_ptr + at + 2) = b;
        } else {
            if (at < n) row_ptr[at] = a.x;
            if (at + 1 < n) row_ptr[at + 1] = a.y;
            if (at + 2 < n) row_ptr[at + 2] = b.x;
        }
        carry += total;
        __syncthreads();  // tmp is written again
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) row_ptr[n] = sums[tiles];
}

inline int64_t scan_tiles(int64_t n) { return (n + kScanTile - 1) / kScanTile; }

inline EdgeArgs make_args(const int32_t* transits, int32_t n_prev, const int32_t* sampled,
                          int32_t m) {
    EdgeArgs a{};
    a.transits = transits;
    a.sampled = sampled;
    a.n_prev = (uint32_t)n_prev;
    a.m = (uint32_t)m;
    a.table = 128;
    a.shift = 25;
    while (a.table < 2u * (uint32_t)m) {
        a.table <<= 1;
        --a.shift;
    }
    return a;
}

}  // namespace

size_t edges_workspace_bytes(int64_t num_samples, int32_t n_prev) {
    const int64_t rows = num_samples * (int64_t)n_prev;
    const size_t counts = ((size_t)(rows > 0 ? rows : 1) * 4 + 255) / 256 * 256;
    return 256 + counts + (size_t)(scan_tiles(rows) + 1) * 8 + 256;
}

int edges_count(const Graph& gr, const int32_t* transits, int32_t n_prev, const int32_t* sampled,
                int32_t m, int64_t num_samples, int64_t* row_ptr, void* workspace, hipStream_t stream) {
    const int64_t rows = num_samples * (int64_t)n_prev;
    char* ws = (char*)workspace;
    uint32_t* status = (uint32_t*)ws;
    int32_t* counts = (int32_t*)(ws + 256);
    const size_t counts_bytes = ((size_t)(rows > 0 ? rows : 1) * 4 + 255) / 256 * 256;
    int64_t* sums = (int64_t*)(ws + 256 + counts_bytes);
    const int64_t tiles = scan_tiles(rows);
    hipLaunchKernelGGL(edges_clear_status_kernel, dim3(1), dim3(1), 0, stream, status);
    if (num_samples > 0) {
        EdgeArgs a = make_args(transits, n_prev, sampled, m);
        a.counts = counts;
        a.status = status;
        if (gr.off64)
            hipLaunchKernelGGL((edges_kernel<int64_t, false>), dim3((unsigned)num_samples),
                               dim3(kEdgeThreads), 0, stream, view_of<int64_t>(gr), a);
        else
            hipLaunchKernelGGL((edges_kernel<int32_t, false>), dim3((unsigned)num_samples),
                               dim3(kEdgeThreads), 0, stream, view_of<int32_t>(gr), a);
        hipLaunchKernelGGL(scan_sums_kernel, dim3((unsigned)tiles), dim3(kScanThreads), 0, stream, counts,
                           rows, sums);
    }
    hipLaunchKernelGGL(scan_top_kernel, dim3(1), dim3(kScanThreads), 0, stream, sums, tiles);
    hipLaunchKernelGGL(scan_write_kernel, dim3((unsigned)(tiles > 0 ? tiles : 1)), dim3(kScanThreads), 0,
                       stream, counts, rows, sums, tiles, row_ptr);
    ND_HIP_CHECK(hipGetLastError());
    return ND_OK;
}

int edges_fill(const Graph& gr, const int32_t* transits, int32_t n_prev, const int32_t* sampled,
               int32_t m, int64_t num_samples, const int64_t* row_ptr, int32_t* edge_slot,
               int64_t capacity, hipStream_t stream) {
    if (num_samples == 0) return ND_OK;
    EdgeArgs a = make_args(transits, n_prev, sampled, m);
    a.row_ptr = row_ptr;
    a.edge_slot = edge_slot;
    a.capacity = capacity;
    a.status = nullptr;
    if (gr.off64)
        hipLaunchKernelGGL((edges_kernel<int64_t, true>), dim3((unsigned)num_samples), dim3(kEdgeThreads),
                           0, stream, view_of<int64_t>(gr), a);
    else
        hipLaunchKernelGGL((edges_kernel<int32_t, true>), dim3((unsigned)num_samples), dim3(kEdgeThreads),
                           0, stream, view_of<int32_t>(gr), a);
    ND_HIP_CHECK(hipGetLastError());
    return ND_OK;
}

}  // namespace nd
