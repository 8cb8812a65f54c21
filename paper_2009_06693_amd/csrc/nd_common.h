// Internal declarations shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include <atomic>
#include <mutex>

#include "../../include/nd.h"

namespace nd {

constexpr int kWave = 64;

// ---------------------------------------------------------------- errors
void set_error(const char* fmt, ...);
#define ND_HIP_CHECK(expr)                                                              \
    do {                                                                                \
        hipError_t e_ = (expr);                                                         \
        if (e_ != hipSuccess) {                                                         \
            nd::set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, __LINE__); \
            return ND_ERR_HIP;                                                          \
        }                                                                               \
    } while (0)

// ---------------------------------------------------------------- phase timing (measurement only)
// When enabled on the calling thread, every call of mark_phase records a HIP
// event on the stream; the time between two marks is charged to the phase of
// the first.  ND_PHASE_NONE closes the current interval.
void mark_phase(int phase, hipStream_t stream);

// ---------------------------------------------------------------- graph
// What a walk needs of the edge it draws, in one aligned 16-byte piece: the vertex at its end and
// where that vertex's row lies, so that a step is one scattered fetch instead of two dependent ones
// (row offsets, then the entry).  The quantised weight sits in the fourth word.
struct Link {
    int32_t v;
    uint32_t rs, deg;   // the row of v: first entry (0 for an empty row) and length
    uint32_t wq;        // quantised weight of this edge (0 on an unweighted graph)
};
static_assert(sizeof(Link) == 16, "one 16-byte load");
// On a weighted graph every Link is followed by what the inverse transform needs (32 bytes per edge).
// Entry j of a row with running sums cum and total T is drawn when mulhi64(R, T) < cum[j] for the
// first time, R being the draw's 64-bit word, and that is R < ceil(cum[j] * 2^64 / T): `thr`, so the
// total is not looked up and nothing is multiplied.  The words with mulhi32(high word, deg) == i
// start the search at entry `guide` of cell i (Chen and Asau's guide table: on average about one
// entry is looked at, whatever the row's length).
struct WeightLink {
    uint64_t thr;
    uint32_t guide;
    uint32_t top;       // bits 0-30: largest quantised weight in the row of the link's vertex (node2vec's
                        // envelope); bit 31: thr would be 2^64 (only zero weights follow)
    __host__ __device__ bool always() const { return (top >> 31) != 0u; }
};
static_assert(sizeof(WeightLink) == 16, "one 16-byte load");

// What a step of a weighted walk looks up, in one aligned 64-byte piece (half a line: the scattered fetch of a line is
// what a draw costs, whatever is read of it).  Cell i of a row belongs to the words whose guide-table cell is i,
// and holds the four entries from the guide on: the high words of their thresholds, all ones where the threshold would
// be 2^64, and their links without the weight.  A draw that ends behind them, or whose high word equals a threshold's,
// is made from the WeightLinks.
struct WeightCell {
    uint32_t thr[4];
    uint32_t link[4][3];  // v, rs, deg
};
static_assert(sizeof(WeightCell) == 64, "four 16-byte loads");

// The columns in as many bits as a vertex takes, one after the other, for the draws of k-hop, which are bound by the
// lines they touch: a row has fewer of them.  Entry e starts at bit e * bits; the four bytes from that bit's byte on
// hold the whole entry while bits <= 25, so that a draw stays one load, of any alignment.  Less than 4 GB, so that the
// place is a 32-bit offset.
struct PackedCols {
    const uint8_t* bytes;   // null: not there
    uint32_t bits;
    static constexpr uint32_t kMostBits = 25;
};
// The load and what is made of it are apart, so that a kernel can have several loads under way: where a branch around the
// load held both, each of a lane's four waited for the one before (300 K vertices of 3 M, [8,8,4], 1,202 us, 1,158 like this).
__device__ __forceinline__ uint32_t packed_word(const PackedCols& p, uint32_t e, uint32_t* shift) {
    const uint64_t bit = (uint64_t)e * p.bits;
    uint32_t word;
    __builtin_memcpy(&word, p.bytes + (uint32_t)(bit >> 3), 4);
    *shift = (uint32_t)bit & 7u;
    return word;
}
__device__ __forceinline__ int32_t packed_vertex(const PackedCols& p, uint32_t word, uint32_t shift) {
    return (int32_t)__builtin_amdgcn_ubfe(word, shift, p.bits);
}
__device__ __forceinline__ int32_t packed_entry(const PackedCols& p, uint32_t e) {
    uint32_t shift;
    const uint32_t word = packed_word(p, e, &shift);
    return packed_vertex(p, word, shift);
}
inline uint32_t packed_bits(int64_t V) {
    uint32_t bits = 1;
    while ((1ll << bits) < V) ++bits;
    return bits;
}

struct Graph {
    int64_t V = 0, E = 0;
    int off64 = 0;              // width of row offsets as stored
    void* off = nullptr;        // V+1 int32 or int64 (device)
    int32_t* col = nullptr;     // E (device)
    uint32_t* wq = nullptr;     // E quantised weights (device) or null
    uint64_t* cumq = nullptr;   // E inclusive running sums of wq per row (device) or null
    uint32_t* maxwq = nullptr;  // V largest wq per row (device) or null
    int device = 0;
    int num_cus = 256;
    int64_t max_degree = 0;
    int64_t empty_rows = 0;
    // E links, each followed by its WeightLink on a weighted graph; null when E >= 2^31 or when the
    // device had no room for them (walks then take the window kernel)
    Link* links = nullptr;
    // Membership table of every row (see RowSet): built when the sizes of a node2vec call are first asked for
    mutable std::atomic<int32_t*> rowset{nullptr};
    // E cells: built when the sizes of a call that draws from them (walk_uses_cells) are first asked for
    mutable std::atomic<WeightCell*> cells{nullptr};
    // V sums of the rows' weights: built when the sizes of a layer call over edge weights are first asked for
    mutable std::atomic<uint64_t*> totals{nullptr};
    // E columns in packed_bits(V) bits: built when the sizes of a k-hop call that reads them are first asked for
    mutable std::atomic<uint8_t*> packed{nullptr};
    // A bit per vertex, whether its row has entries: built when the sizes of a multi-dimensional walk that looks
    // (mrw_reads_filled) are first asked for
    mutable std::atomic<uint64_t*> filled{nullptr};
    mutable std::mutex extra_mutex;
};
void graph_need_rowset(const Graph& g);
void graph_need_totals(const Graph& g);
void graph_need_cells(const Graph& g);
void graph_need_packed(const Graph& g);
void graph_need_filled(const Graph& g);

// Is u in the row of v?  Every row owns a hash table of at least 2 deg + 1 places in groups of four
// (16 bytes), open addressing by groups, empty places -1: one fetch answers most questions where a
// search down the row takes log2(deg) dependent ones.  Row v's groups start at rs / 2 + v.
struct RowSet {
    const int32_t* table;
    __host__ __device__ static uint64_t first_group(int64_t v, uint64_t rs) { return rs / 2 + (uint64_t)v; }
    __host__ __device__ static uint32_t groups(uint64_t rs, uint32_t deg) {
        return (uint32_t)((rs + deg) / 2 - rs / 2) + 1u;
    }
    __host__ __device__ static uint32_t hash(int32_t u) {
        const uint32_t x = (uint32_t)u * 0x9E3779B1u;
        return x ^ (x >> 15);
    }
};

// Device-side view passed to kernels by value.
template <typename OffT>
struct GraphView {
    const OffT* off;
    const int32_t* col;
    const uint32_t* wq;
    const uint64_t* cumq;
    const uint32_t* maxwq;
    int32_t V;
};

template <typename OffT>
inline GraphView<OffT> view_of(const Graph& g) {
    return GraphView<OffT>{(const OffT*)g.off, g.col, g.wq, g.cumq, g.maxwq, (int32_t)g.V};
}

// Length of row v, given where it starts.  A row is shorter than 2^32, so the low words of the two
// offsets suffice, and with 64-bit offsets the high word of the second one is not fetched: a
// register that a load in flight is about to fill and nobody reads is reused at once, and that use
// waits for the load (in the k-hop loop this cost a tenth of the kernel's time).
template <typename OffT>
__device__ __forceinline__ uint32_t row_length(const GraphView<OffT>& g, int32_t v, uint64_t row_start) {
    return reinterpret_cast<const uint32_t*>(g.off + v + 1)[0] - (uint32_t)row_start;
}

int graph_create(Graph** out, int64_t V, int64_t E, const void* off, int off64, const int32_t* col,
                 const float* w, int src_is_device, hipStream_t stream);
void graph_destroy(Graph* g);

// ---------------------------------------------------------------- division by a runtime constant
// Exact floor(n / d) for 0 <= n < 2^31 and 1 <= d < 2^31:
// q = mulhi32(n, magic) >> shift with magic = ceil(2^(32+shift) / d) (Granlund-Montgomery,
// valid because n < 2^31 leaves one bit of headroom).
struct FastDiv {
    uint32_t d, magic, shift;
};
inline FastDiv make_fastdiv(uint32_t d) {
    FastDiv f;
    f.d = d;
    if (d == 1) {
        f.magic = 0;
        f.shift = 0;
        return f;
    }
    uint32_t s = 0;
    while ((1ull << s) < d) ++s;  // s = ceil(log2 d)
    f.shift = s - 1;
    f.magic = (uint32_t)(((1ull << (32 + s - 1)) + d - 1) / d);
    return f;
}

// ---------------------------------------------------------------- per-step control block (device)
// Written by the grouping kernels, read by the kernels that follow on the same
// stream; the host never reads it inside nd_sample.
struct StepCtl {
    uint32_t P;             // live pairs of the step
    uint32_t U;             // distinct transits
    uint32_t n_wg;          // transits in the workgroup class
    uint32_t n_grid;        // transits in the grid class
    uint32_t n_chunks;      // grid chunks
    uint32_t reserved0;
    uint32_t n_staged;      // workgroup/grid work items that staged their list in LDS
    uint32_t wg_cursor;     // next workgroup-class item to hand out
    uint32_t reserved1;
    uint32_t heavy_draws;   // draws of the workgroup- and grid-class transits
    uint32_t pad[6];
};
static_assert(sizeof(StepCtl) == 64, "one control block per 64 bytes");

struct WsHeader {
    uint32_t status;        // bit 0: a root was out of range
    uint32_t num_steps;
    // Routes that need no kernel to clear counters: every workgroup writes what it found to places of
    // its own, and whoever asks (nd_sample_status, nd_sample_stats) adds up.  0 groups: not that route.
    uint32_t n_groups;
    uint32_t mark;          // kGroupsMark where the four fields beside it are this library's: a workspace that no
                            // call has written to holds whatever it held
    uint64_t o_flags;       // n_groups words: a root was out of range
    uint64_t o_parts;       // [n_groups][num_steps] words: live pairs
    uint32_t pad[56];
};
static_assert(sizeof(WsHeader) == 256, "header is one 256-byte block");
constexpr uint32_t kGroupsMark = 0x6E645753u;
__device__ __forceinline__ void write_header(WsHeader* h, uint32_t num_steps, uint32_t n_groups, uint64_t o_flags,
                                             uint64_t o_parts) {
    h->status = 0;
    h->num_steps = num_steps;
    h->n_groups = n_groups;
    h->mark = kGroupsMark;
    h->o_flags = o_flags;
    h->o_parts = o_parts;
}

// ---------------------------------------------------------------- radix sort plan
constexpr int kSortThreads = 512;       // large inputs: 8,192 keys per tile
constexpr int kSortItems = 16;
constexpr int kSmallSortThreads = 256;  // small inputs: 2,048 keys per tile
constexpr int kSmallSortItems = 8;
constexpr int64_t kSmallSortLimit = 1 << 23;
constexpr int kMaxRadixBits = 8;

struct SortPlan {
    int passes;
    int bits[4];
    int shift[4];
    int tile;               // keys per tile
    int64_t max_tiles;      // tiles of the slot array (pass 0); later passes never need more
};
// group_bits > 0: sort on the top group_bits bits of the key only.
SortPlan make_sort_plan(int64_t n_slots, int64_t V, int group_bits = 0);
size_t sort_hist_bytes(const SortPlan& p);

// Pass 0 reads `src` (n_slots transits, negative = no transit, implicit value = index)
// and, if fill_out is given, writes ND_NULL_VERTEX into the m children of every dead slot.
// The sorted pairs end in (keys_out, vals_out) which is one of the two buffer pairs.
int sort_pairs(const int32_t* src, int64_t n_slots, int32_t V, const SortPlan& plan,
               int32_t* keysA, int32_t* valsA, int32_t* keysB, int32_t* valsB, uint32_t* hist,
               StepCtl* ctl, int32_t* fill_out, int32_t m, uint32_t* status_word,
               int32_t** keys_out, int32_t** vals_out, hipStream_t stream);

// ---------------------------------------------------------------- scheduling index
constexpr int kSegThreads = 256;
constexpr int kSegItems = 16;
constexpr int kSegTile = kSegThreads * kSegItems;
size_t seg_scratch_bytes(int64_t n_slots);
// heavy_bits (may be null): the per-vertex marks of the previous step are cleared on the way.
int build_groups(const int32_t* sorted_keys, int64_t max_pairs, StepCtl* ctl, int32_t* g_key,
                 int32_t* g_start, uint32_t* tile_counts, uint32_t* heavy_bits, int64_t bit_words,
                 hipStream_t stream);

struct SchedParams {
    int32_t m;              // draws per pair
    int32_t sub_max;        // draws <= sub_max: sub-wavefront class
    int32_t wg_max;         // draws <= wg_max: workgroup class; chunk size of the grid class
    int32_t force_class;    // nd_sched_class
};
// Scheduling class of a transit that must produce `draws` neighbours
// (Section 6.1.2, Table "Types of kernels", with wave64 thresholds).
__host__ __device__ inline int class_of(uint32_t draws, const SchedParams& sp) {
    if (sp.force_class != ND_CLASS_AUTO) return sp.force_class;
    if (draws <= (uint32_t)sp.sub_max) return ND_CLASS_SUBWAVE;
    if (draws <= (uint32_t)sp.wg_max) return ND_CLASS_WORKGROUP;
    return ND_CLASS_GRID;
}
// Fills the workgroup list and the grid chunk list and marks their transits in heavy_bits
// (one bit per vertex; may be null when a class is forced).
int classify_groups(const int32_t* g_key, const int32_t* g_start, int64_t max_groups, StepCtl* ctl,
                    const SchedParams& sp, int32_t* list_wg, int32_t* chunk_gid, int32_t* chunk_idx,
                    int64_t max_chunks, uint32_t* heavy_bits, hipStream_t stream);

}  // namespace nd
