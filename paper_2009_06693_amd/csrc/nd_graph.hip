// CSR loader: copies the graph to device memory, validates it there and builds
// the per-vertex weight data the paper's Vertex class offers (Section 4.1:
// degree, largest edge weight, running sums of the edge weights).
#include <cmath>
#include <cstdio>
#include <new>

#include "nd_common.h"
#include "nd_philox.h"
#include "nd_wave.h"

namespace nd {

namespace {

enum : uint32_t {
    kBadFirst = 1u,      // offsets[0] != 0
    kBadMonotone = 2u,   // offsets decrease somewhere or leave [0, E]
    kBadLast = 4u,       // offsets[V] != E
    kBadColumn = 8u,     // a column outside [0, V)
    kBadOrder = 16u,     // a row not strictly ascending
    kBadWeight = 32u,    // weight not finite, <= 0 or >= 2^15
    kBadRowTotal = 64u   // a row's quantised weights sum to 2^39 or more
};

// Checks the offsets, and finds the longest row and how many rows are empty.
// found: [0] flags, [2..3] the longest row, [4..5] the empty rows.  One atomic per workgroup and word: atomics on one word
// take 12 ns each (4.2 M rows: 102 us with one per wavefront, 39 like this).
template <typename OffT>
__global__ __launch_bounds__(256) void check_offsets_kernel(const OffT* __restrict__ off, int64_t V, int64_t E,
                                                            uint32_t* __restrict__ found) {
    __shared__ unsigned long long s_max;
    __shared__ uint32_t s_empty, s_bad;
    if (threadIdx.x == 0) {
        s_max = 0;
        s_empty = s_bad = 0;
    }
    __syncthreads();
    uint32_t bad = 0, empty = 0;
    unsigned long long mx = 0;
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < V; v += (int64_t)gridDim.x * 256) {
        if (v == 0 && off[0] != 0) bad |= kBadFirst;
        if (v == 0 && (int64_t)off[V] != E) bad |= kBadLast;
        const int64_t a = (int64_t)off[v], b = (int64_t)off[v + 1];
        if (a > b || a < 0 || b > E) bad |= kBadMonotone;
        else if ((unsigned long long)(b - a) > mx) mx = (unsigned long long)(b - a);
        empty += a == b ? 1u : 0u;
    }
    for (int d = 32; d >= 1; d >>= 1) {
        const unsigned long long o = __shfl_xor(mx, d, 64);
        mx = o > mx ? o : mx;
        empty += (uint32_t)__shfl_xor((int)empty, d, 64);
    }
    if (lane_id() == 0) {
        atomicMax(&s_max, mx);
        atomicAdd(&s_empty, empty);
    }
    if (bad) atomicOr(&s_bad, bad);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (s_max > 0) atomicMax((unsigned long long*)(found + 2), s_max);
        if (s_empty > 0) atomicAdd((unsigned long long*)(found + 4), (unsigned long long)s_empty);
        if (s_bad) atomicOr(found, s_bad);
    }
}

// One wavefront per row, 64 entries at a time: columns in range and strictly
// ascending; with weights, quantise (w_q = floor(w * 2^16 + 0.5), evaluated in
// double), accumulate the running sums (a wave scan per 64 entries plus the sum
// carried from the entries before) and the row maximum.  Rows are dealt to the
// wavefronts round robin, so a row of any length costs its wavefront
// ceil(deg / 64) rounds and the long rows of a skewed graph do not serialise.
template <typename OffT>
__global__ __launch_bounds__(256) void check_rows_kernel(const OffT* __restrict__ off, const int32_t* __restrict__ col,
                                                         const float* __restrict__ w, int64_t V,
                                                         uint32_t* __restrict__ wq, uint64_t* __restrict__ cumq,
                                                         uint32_t* __restrict__ maxwq, uint32_t* __restrict__ flags) {
    const int lane = lane_id();
    const int64_t wave0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6;
    const int64_t n_waves = ((int64_t)gridDim.x * 256) >> 6;
    uint32_t bad = 0;
    for (int64_t v = wave0; v < V; v += n_waves) {  // the same v on every lane of the wave
        const int64_t lo = (int64_t)off[v], hi = (int64_t)off[v + 1];
        unsigned long long run = 0;
        uint32_t mx = 0;
        for (int64_t base = lo; base < hi; base += 64) {
            const int64_t e = base + lane;
            const bool in = e < hi;
            const int32_t c = in ? col[e] : 0;
            int32_t before = __shfl_up(c, 1, 64);
            if (lane == 0) before = e > lo ? col[e - 1] : -1;
            if (in && (c < 0 || (int64_t)c >= V)) bad |= kBadColumn;
            if (in && c <= before) bad |= kBadOrder;
            if (w) {
                uint32_t q = 0;
                if (in) {
                    const float x = w[e];
                    q = 1;
                    if (!(x > 0.0f) || !(x < 32768.0f)) bad |= kBadWeight;
                    else q = (uint32_t)floor((double)x * 65536.0 + 0.5);
                    wq[e] = q;
                    if (q > mx) mx = q;
                }
                const unsigned long long incl = wave_inclusive_scan((unsigned long long)q, lane);
                if (in) cumq[e] = run + incl;
                run += __shfl(incl, 63, 64);
            }
        }
        if (w) {
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) {
                const uint32_t o = __shfl_xor(mx, d, 64);
                mx = o > mx ? o : mx;
            }
            if (lane == 0) maxwq[v] = mx;
            if (run >= (1ull << 39)) bad |= kBadRowTotal;
        }
    }
    if (bad) atomicOr(flags, bad);
}

// The row that holds entry e: the last one that starts at or before it, among rows [lo, hi].
template <typename OffT>
__device__ __forceinline__ int64_t row_of(const OffT* __restrict__ off, int64_t e, int64_t lo, int64_t hi) {
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if ((int64_t)off[mid] <= e) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Links and WeightLinks, one entry per thread whatever row it belongs to (a wavefront per row leaves
// most lanes of a skewed graph idle behind chains of dependent look-ups).  Bound by the scattered
// look-ups of the neighbours' offsets.  On an unweighted graph it checks the rows as well (otherwise
// check_rows_kernel has).  Where a row starts matters only there and for the weights.
constexpr int kLinkTile = 256;
template <typename OffT>
__global__ __launch_bounds__(256) void build_links_kernel(const OffT* __restrict__ off, const int32_t* __restrict__ col,
                                                          const uint32_t* __restrict__ wq,
                                                          const uint64_t* __restrict__ cumq,
                                                          const uint32_t* __restrict__ maxwq, int64_t V, int64_t E,
                                                          Link* __restrict__ links, uint32_t* __restrict__ flags) {
    const int64_t first = (int64_t)blockIdx.x * kLinkTile;
    const int64_t last = first + kLinkTile < E ? first + kLinkTile - 1 : E - 1;
    const int64_t row_lo = row_of(off, first, 0, V - 1), row_hi = row_of(off, last, row_lo, V - 1);
    uint32_t bad = 0;
    for (int64_t e = first + threadIdx.x; e <= last; e += 256) {
        const int64_t v = row_of(off, e, row_lo, row_hi);
        const uint64_t lo = (uint64_t)off[v];
        const uint32_t deg = (uint32_t)((uint64_t)off[v + 1] - lo);
        const int32_t u = col[e];
        if (wq == nullptr) {
            if (u < 0 || (int64_t)u >= V) {
                bad |= kBadColumn;
                continue;
            }
            if ((uint64_t)e > lo && u <= col[e - 1]) bad |= kBadOrder;
        }
        Link l;
        l.v = u;
        l.rs = (uint32_t)off[u];
        l.deg = (uint32_t)off[u + 1] - l.rs;
        l.rs = l.deg > 0u ? l.rs : 0u;  // a place inside the links whatever the row
        l.wq = wq != nullptr ? wq[e] : 0u;
        if (wq == nullptr) {
            links[e] = l;
        } else {
            const uint64_t T = cumq[lo + deg - 1u], c = cumq[e];
            WeightLink w;
            w.top = maxwq[u] | (c == T && T > 0 ? 0x80000000u : 0u);
            w.thr = c == T ? 0u : scaled_threshold(c, T);
            // first entry whose running sum exceeds the smallest value that a word of cell i gives
            const uint32_t i = (uint32_t)((uint64_t)e - lo);
            const uint64_t r0 = (((uint64_t)i << 32) + deg - 1u) / deg;
            const uint64_t x = mulhi64(r0 << 32, T);
            uint32_t a = 0, b = deg - 1u;
            while (a < b) {
                const uint32_t mid = (a + b) >> 1;
                if (cumq[lo + mid] > x) b = mid;
                else a = mid + 1u;
            }
            w.guide = a;
            links[2 * e] = l;
            reinterpret_cast<WeightLink*>(links)[2 * e + 1] = w;
        }
    }
    if (bad) atomicOr(flags, bad);
}

// The rows' membership tables, one entry per thread.
template <typename OffT>
__global__ __launch_bounds__(256) void build_rowset_kernel(const OffT* __restrict__ off, const int32_t* __restrict__ col,
                                                           int64_t V, int64_t E, int32_t* rowset) {
    const int64_t first = (int64_t)blockIdx.x * kLinkTile;
    const int64_t last = first + kLinkTile < E ? first + kLinkTile - 1 : E - 1;
    const int64_t row_lo = row_of(off, first, 0, V - 1), row_hi = row_of(off, last, row_lo, V - 1);
    const int64_t e = first + threadIdx.x;
    if (e > last) return;
    const int64_t v = row_of(off, e, row_lo, row_hi);
    const uint64_t lo = (uint64_t)off[v];
    const uint32_t ng = RowSet::groups(lo, (uint32_t)((uint64_t)off[v + 1] - lo));
    int32_t* set = rowset + RowSet::first_group(v, lo) * 4;
    const int32_t u = col[e];
    uint32_t grp = mulhi32(RowSet::hash(u), ng);
    for (bool placed = false; !placed;) {  // more places than entries: the loop ends
        for (uint32_t k = 0; k < 4u && !placed; ++k)
            placed = atomicCAS(&set[grp * 4u + k], ND_NULL_VERTEX, u) == ND_NULL_VERTEX;
        grp = grp + 1u < ng ? grp + 1u : 0u;
    }
}

// The WeightCells, one entry per thread: 64 bytes stored for each at 1.5 to 1.9 TB/s (1.6 M entries 55 us, beside 0.28 ms
// for the memory and the stream; 39 M 1.7 ms, 117 M 4.4, 412 M 14.5 with those), once per graph.
template <typename OffT>
__global__ __launch_bounds__(256) void build_cells_kernel(const OffT* __restrict__ off, const Link* __restrict__ links,
                                                          int64_t V, int64_t E, WeightCell* __restrict__ cells) {
    const int64_t first = (int64_t)blockIdx.x * kLinkTile;
    const int64_t last = first + kLinkTile < E ? first + kLinkTile - 1 : E - 1;
    const int64_t row_lo = row_of(off, first, 0, V - 1), row_hi = row_of(off, last, row_lo, V - 1);
    const int64_t e = first + threadIdx.x;
    if (e > last) return;
    const WeightLink* weights = reinterpret_cast<const WeightLink*>(links);
    const int64_t v = row_of(off, e, row_lo, row_hi);
    const uint64_t lo = (uint64_t)off[v];
    const uint32_t deg = (uint32_t)((uint64_t)off[v + 1] - lo);
    const uint32_t guide = weights[2 * e + 1].guide;
    WeightCell c;
#pragma unroll
    for (uint32_t k = 0; k < 4u; ++k) {
        const uint32_t j = guide + k < deg ? guide + k : deg - 1u;
        const WeightLink w = weights[2ull * (lo + j) + 1u];
        const Link l = links[2ull * (lo + j)];
        c.thr[k] = w.always() ? 0xFFFFFFFFu : (uint32_t)(w.thr >> 32);
        c.link[k][0] = (uint32_t)l.v;
        c.link[k][1] = l.rs;
        c.link[k][2] = l.deg;
    }
    cells[e] = c;
}

template <typename OffT>
__global__ __launch_bounds__(256) void build_totals_kernel(const OffT* __restrict__ off, const uint64_t* __restrict__ cumq,
                                                           int64_t V, uint64_t* __restrict__ totals) {
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < V; v += (int64_t)gridDim.x * 256) {
        const int64_t a = (int64_t)off[v], b = (int64_t)off[v + 1];
        totals[v] = b > a ? cumq[b - 1] : 0ull;
    }
}

// A bit per vertex, whether its row has entries.
template <typename OffT>
__global__ __launch_bounds__(256) void build_filled_kernel(const OffT* __restrict__ off, int64_t V, uint64_t* __restrict__ filled) {
    for (int64_t v0 = (int64_t)blockIdx.x * 256; v0 < V; v0 += (int64_t)gridDim.x * 256) {
        const int64_t v = v0 + threadIdx.x;
        const uint64_t votes = __ballot(v < V && off[v + 1] > off[v]);
        if (lane_id() == 0 && v < V) filled[v >> 6] = votes;
    }
}

// The packed columns, a 32-bit word per thread: the entries that have a bit in it, two to four where bits >= 11.  Reads
// come from the caches, which neighbouring words share.
__global__ __launch_bounds__(256) void build_packed_kernel(const int32_t* __restrict__ col, int64_t E, uint32_t bits,
                                                           uint32_t words, uint32_t* __restrict__ packed) {
    for (uint32_t w = blockIdx.x * 256u + threadIdx.x; w < words; w += gridDim.x * 256u) {  // words < 2^30
        const uint32_t group = w / bits;                        // 32 entries fill `bits` whole words
        const uint32_t first_bit = (w - group * bits) * 32u;
        uint32_t k = first_bit / bits, word = 0;
        int32_t at = (int32_t)(k * bits) - (int32_t)first_bit;  // where entry k starts in the word, from -(bits - 1) on
        for (; at < 32; ++k, at += (int32_t)bits) {
            const int64_t e = (int64_t)group * 32 + k;
            const uint32_t v = e < E ? (uint32_t)col[e] : 0u;
            word |= at < 0 ? v >> -at : v << at;
        }
        packed[w] = word;
    }
}

__global__ __launch_bounds__(256) void fill_empty_kernel(int4* p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        p[i] = make_int4(-1, -1, -1, -1);
}

// What only makes calls faster may take a quarter of the device memory that is free when it is made; the rest
// stays for the caller's outputs and workspaces.  (E = 2^31 weighted entries: 64 GB of links, which an empty
// device of 288 GB grants.  The question takes 4 to 30 us.)
bool spare_room(size_t bytes) {
    size_t avail = 0, total = 0;
    if (hipMemGetInfo(&avail, &total) == hipSuccess) return bytes <= avail / 4;
    (void)hipGetLastError();
    return false;
}

// Room for the links.  Optional: without them walks and k-hop take longer.
void allocate_links(Graph* g, bool weighted) {
    if (g->E < 1 || g->E >= (1ll << 31)) return;
    const size_t bytes = (size_t)g->E * sizeof(Link) * (weighted ? 2 : 1);
    if (spare_room(bytes) && hipMalloc((void**)&g->links, bytes) != hipSuccess) {
        (void)hipGetLastError();
        g->links = nullptr;
    }
}

void free_graph(Graph* g) {
    if (!g) return;
    (void)hipFree(g->off);
    (void)hipFree(g->col);
    (void)hipFree(g->wq);
    (void)hipFree(g->cumq);
    (void)hipFree(g->maxwq);
    (void)hipFree(g->links);
    (void)hipFree(g->rowset.load());
    (void)hipFree(g->cells.load());
    (void)hipFree(g->totals.load());
    (void)hipFree(g->packed.load());
    (void)hipFree(g->filled.load());
    delete g;
}

template <typename OffT>
int validate_and_build(Graph* g, const float* w_dev, uint32_t* flags_dev, hipStream_t stream) {
    const int threads = 256;
    int64_t blocks = (g->V + threads - 1) / threads;
    if (blocks > (int64_t)g->num_cus * 4) blocks = (int64_t)g->num_cus * 4;
    hipLaunchKernelGGL(check_offsets_kernel<OffT>, dim3((unsigned)blocks), dim3(threads), 0, stream,
                       (const OffT*)g->off, g->V, g->E, flags_dev);
    ND_HIP_CHECK(hipGetLastError());
    struct {
        uint32_t flags, unused;
        uint64_t max_degree, empty;
    } found;
    ND_HIP_CHECK(hipMemcpyAsync(&found, flags_dev, sizeof(found), hipMemcpyDeviceToHost, stream));
    ND_HIP_CHECK(hipStreamSynchronize(stream));
    uint32_t flags = found.flags;
    g->max_degree = (int64_t)found.max_degree;
    g->empty_rows = (int64_t)found.empty;
    if (flags) {
        set_error("bad CSR offsets:%s%s%s", (flags & kBadFirst) ? " offsets[0] != 0;" : "",
                  (flags & kBadMonotone) ? " offsets not monotone within [0, E];" : "",
                  (flags & kBadLast) ? " offsets[V] != E;" : "");
        return ND_ERR_BAD_GRAPH;
    }
    // rows may only be walked once the offsets are known to be sane
    if (w_dev || !g->links) {  // one wavefront per row; enough workgroups to fill the chip several times, never more than rows / 4
        int64_t row_blocks = (g->V + 3) / 4;
        const int64_t cap = (int64_t)g->num_cus * 16;
        if (row_blocks > cap) row_blocks = cap;
        hipLaunchKernelGGL(check_rows_kernel<OffT>, dim3((unsigned)row_blocks), dim3(256), 0, stream,
                           (const OffT*)g->off, g->col, w_dev, g->V, g->wq, g->cumq, g->maxwq, flags_dev);
        ND_HIP_CHECK(hipGetLastError());
        if (g->links) {  // the links look columns up: these have to be in range
            ND_HIP_CHECK(hipMemcpyAsync(&flags, flags_dev, sizeof(flags), hipMemcpyDeviceToHost, stream));
            ND_HIP_CHECK(hipStreamSynchronize(stream));
        }
    }
    if (g->links && !flags) {
        hipLaunchKernelGGL(build_links_kernel<OffT>, dim3((unsigned)((g->E + kLinkTile - 1) / kLinkTile)), dim3(256), 0,
                           stream, (const OffT*)g->off, g->col, g->wq, g->cumq, g->maxwq, g->V, g->E, g->links, flags_dev);
        ND_HIP_CHECK(hipGetLastError());
    }
    ND_HIP_CHECK(hipMemcpyAsync(&flags, flags_dev, sizeof(flags), hipMemcpyDeviceToHost, stream));
    ND_HIP_CHECK(hipStreamSynchronize(stream));
    if (flags & (kBadColumn | kBadOrder)) {
        set_error("bad CSR rows:%s%s", (flags & kBadColumn) ? " a column is outside [0, V);" : "",
                  (flags & kBadOrder) ? " a row is not strictly ascending (unsorted or duplicate);" : "");
        return ND_ERR_BAD_GRAPH;
    }
    if (flags & (kBadWeight | kBadRowTotal)) {
        set_error("bad weights:%s%s",
                  (flags & kBadWeight) ? " a weight is not finite, <= 0 or >= 2^15;" : "",
                  (flags & kBadRowTotal) ? " a row's quantised weights sum to 2^39 or more;" : "");
        return ND_ERR_BAD_WEIGHT;
    }
    return ND_OK;
}

}  // namespace

int graph_create(Graph** out, int64_t V, int64_t E, const void* off, int off64, const int32_t* col,
                 const float* w, int src_is_device, hipStream_t stream) {
    Graph* g = new (std::nothrow) Graph;
    if (!g) {
        set_error("out of host memory");
        return ND_ERR_HIP;
    }
    g->V = V;
    g->E = E;
    g->off64 = off64;
    float* w_dev = nullptr;
    uint32_t* flags_dev = nullptr;
    int rc = ND_OK;
    auto body = [&]() -> int {
        ND_HIP_CHECK(hipGetDevice(&g->device));
        ND_HIP_CHECK(hipDeviceGetAttribute(&g->num_cus, hipDeviceAttributeMultiprocessorCount, g->device));
        if (g->num_cus < 1) g->num_cus = 1;
        const size_t off_bytes = (size_t)(V + 1) * (off64 ? 8 : 4);
        const size_t e_alloc = (size_t)(E > 0 ? E : 1);
        const hipMemcpyKind kind = src_is_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
        ND_HIP_CHECK(hipMalloc(&g->off, off_bytes));
        ND_HIP_CHECK(hipMalloc((void**)&g->col, e_alloc * 4));
        ND_HIP_CHECK(hipMalloc((void**)&flags_dev, 256));
        ND_HIP_CHECK(hipMemsetAsync(flags_dev, 0, 256, stream));
        ND_HIP_CHECK(hipMemcpyAsync(g->off, off, off_bytes, kind, stream));
        if (E > 0) ND_HIP_CHECK(hipMemcpyAsync(g->col, col, (size_t)E * 4, kind, stream));
        if (w) {
            ND_HIP_CHECK(hipMalloc((void**)&w_dev, e_alloc * 4));
            ND_HIP_CHECK(hipMalloc((void**)&g->wq, e_alloc * 4));
            ND_HIP_CHECK(hipMalloc((void**)&g->cumq, e_alloc * 8));
            ND_HIP_CHECK(hipMalloc((void**)&g->maxwq, (size_t)V * 4));
            if (E > 0) ND_HIP_CHECK(hipMemcpyAsync(w_dev, w, (size_t)E * 4, kind, stream));
        }
        allocate_links(g, w != nullptr);
        return off64 ? validate_and_build<int64_t>(g, w_dev, flags_dev, stream)
                     : validate_and_build<int32_t>(g, w_dev, flags_dev, stream);
    };
    rc = body();
    (void)hipStreamSynchronize(stream);
    (void)hipFree(w_dev);
    (void)hipFree(flags_dev);
    if (rc != ND_OK) {
        free_graph(g);
        *out = nullptr;
        return rc;
    }
    *out = g;
    return ND_OK;
}

void graph_destroy(Graph* g) { free_graph(g); }

// What is built on a graph after its creation: on the graph's device and a stream of its own, so that it neither waits
// for the caller's work nor joins a stream capture, and from a quarter of the free memory.  Without it calls are
// slower; whoever asks next tries again.  launch(memory, stream) enqueues the kernels that fill the memory.
template <typename T, typename F>
static void need_extra(const Graph& g, std::atomic<T*>& extra, size_t bytes, F launch) {
    if (!g.links || extra.load(std::memory_order_acquire)) return;
    std::lock_guard<std::mutex> lock(g.extra_mutex);
    if (extra.load(std::memory_order_acquire)) return;
    hipStreamCaptureMode capture = hipStreamCaptureModeRelaxed;
    (void)hipThreadExchangeStreamCaptureMode(&capture);
    int here = -1;
    if (hipGetDevice(&here) == hipSuccess && (here == g.device || hipSetDevice(g.device) == hipSuccess)) {
        T* memory = nullptr;
        hipStream_t stream = nullptr;
        bool ok = spare_room(bytes) && hipMalloc((void**)&memory, bytes) == hipSuccess &&
                  hipStreamCreateWithFlags(&stream, hipStreamNonBlocking) == hipSuccess;
        if (ok) {
            launch(memory, stream);
            ok = hipGetLastError() == hipSuccess && hipStreamSynchronize(stream) == hipSuccess;
        }
        if (stream) (void)hipStreamDestroy(stream);
        if (ok) {
            extra.store(memory, std::memory_order_release);
        } else {
            (void)hipGetLastError();
            (void)hipFree(memory);
        }
        if (here != g.device) (void)hipSetDevice(here);
    }
    (void)hipThreadExchangeStreamCaptureMode(&capture);
}

// The rows' membership tables: 8 bytes per entry and 16 per vertex.  Without them node2vec searches the rows.
void graph_need_rowset(const Graph& g) {
    const int64_t n = g.E / 2 + g.V + 1;
    const dim3 grid((unsigned)((g.E + kLinkTile - 1) / kLinkTile));
    need_extra(g, g.rowset, (size_t)n * 16, [&](int32_t* set, hipStream_t stream) {
        hipLaunchKernelGGL(fill_empty_kernel, dim3((unsigned)g.num_cus * 32u), dim3(256), 0, stream, (int4*)set, n);
        if (g.off64)
            hipLaunchKernelGGL(build_rowset_kernel<int64_t>, grid, dim3(256), 0, stream, (const int64_t*)g.off, g.col,
                               g.V, g.E, set);
        else
            hipLaunchKernelGGL(build_rowset_kernel<int32_t>, grid, dim3(256), 0, stream, (const int32_t*)g.off, g.col,
                               g.V, g.E, set);
    });
}

// The rows' sums of weights: 8 bytes per vertex.  Without them layer sampling reads the last running sum of a row.
void graph_need_totals(const Graph& g) {
    if (!g.wq) return;
    const dim3 grid((unsigned)g.num_cus * 8u);
    need_extra(g, g.totals, (size_t)g.V * 8, [&](uint64_t* totals, hipStream_t stream) {
        if (g.off64)
            hipLaunchKernelGGL(build_totals_kernel<int64_t>, grid, dim3(256), 0, stream, (const int64_t*)g.off, g.cumq,
                               g.V, totals);
        else
            hipLaunchKernelGGL(build_totals_kernel<int32_t>, grid, dim3(256), 0, stream, (const int32_t*)g.off, g.cumq,
                               g.V, totals);
    });
}

// Which rows have entries: a bit per vertex.
void graph_need_filled(const Graph& g) {
    const dim3 grid((unsigned)g.num_cus * 8u);
    need_extra(g, g.filled, ((size_t)g.V + 63) / 64 * 8, [&](uint64_t* filled, hipStream_t stream) {
        if (g.off64)
            hipLaunchKernelGGL(build_filled_kernel<int64_t>, grid, dim3(256), 0, stream, (const int64_t*)g.off, g.V, filled);
        else
            hipLaunchKernelGGL(build_filled_kernel<int32_t>, grid, dim3(256), 0, stream, (const int32_t*)g.off, g.V, filled);
    });
}

// The packed columns: packed_bits(V) bits per entry and up to three bytes that the last entry's load takes with it.
void graph_need_packed(const Graph& g) {
    const uint32_t bits = packed_bits(g.V);
    if (bits > PackedCols::kMostBits) return;
    const int64_t words = ((g.E + 31) / 32) * bits;
    if (words * 4 + 4 >= (1ll << 32)) return;
    need_extra(g, g.packed, (size_t)words * 4 + 4, [&](uint8_t* packed, hipStream_t stream) {
        hipLaunchKernelGGL(build_packed_kernel, dim3((unsigned)g.num_cus * 16u), dim3(256), 0, stream, g.col, g.E, bits,
                           (uint32_t)words, (uint32_t*)packed);
    });
}

// The cells of weighted draws: 64 bytes per entry.  Without them a draw looks its guide up first.
void graph_need_cells(const Graph& g) {
    if (!g.wq) return;
    const dim3 grid((unsigned)((g.E + kLinkTile - 1) / kLinkTile));
    need_extra(g, g.cells, (size_t)g.E * sizeof(WeightCell), [&](WeightCell* cells, hipStream_t stream) {
        if (g.off64)
            hipLaunchKernelGGL(build_cells_kernel<int64_t>, grid, dim3(256), 0, stream, (const int64_t*)g.off, g.links,
                               g.V, g.E, cells);
        else
            hipLaunchKernelGGL(build_cells_kernel<int32_t>, grid, dim3(256), 0, stream, (const int32_t*)g.off, g.links,
                               g.V, g.E, cells);
    });
}

}  // namespace nd
