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

namespace nd {

namespace {

constexpr int kFusedThreads = 256;

struct FusedArgs {
    const Link* links;
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

// R consecutive entries (R = 2: eight bytes, aligned).
template <int R>
__device__ __forceinline__ void store_run(int32_t* p, const int32_t* v) {
    if (R == 2) *reinterpret_cast<int2*>(p) = make_int2(v[0], v[1]);
    else *p = v[0];
}

// A place in a buffer of rows: where the row of a slot's vertex lies.
__device__ __forceinline__ uint2 row_of_link(const Link& l) { return make_uint2(l.rs, l.deg); }

// Bound by latency (small calls: a hop is generator, link, row; 37 roots of three hops take one launch
// instead of 26) or by the rate of scattered fetches (large ones).
// R: draws per lane of the last hop, a divisor of its fanout.
template <int STRIDE, int R, typename OffT>
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
            ++live;
        }
        s_rows[i] = row;
    }
    const int any_bad = __syncthreads_or(bad ? 1 : 0);
    if (live) atomicAdd(&s_live[0], live);
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
                    ++live;
                }
                next[d] = row_of_link(l);
                if (part == 0) out[d] = l.v;
            }
            if (live) atomicAdd(&s_live[hop + 1], live);
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
                        if (row[u].y > 0u) v[u][i] = g.col[e[u][i]];
                    }
#pragma unroll
                for (uint32_t u = 0; u < kInFlight; ++u)
                    if (d0 + u * T < end) store_run<R>(out + (d0 + u * T) * R, v[u]);
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
// all, a tenth and a fiftieth of the vertices of ten graphs with fanouts [25,10], [10,10], [10,25], [20] and
// [15,10,5]: grouping wins, by up to 1.4x, on dense graphs (rows that ten draws rarely share a line of)
// with many pairs per vertex and enough draws to pay for its 26 launches; elsewhere it loses, by up to 9x.
bool khop_fused_fits(const Graph& gr, const int32_t* fanout, int32_t k, int64_t S) {
    if (!gr.links) return false;
    int64_t pairs = S;
    for (int32_t i = 0; i + 1 < k; ++i) pairs *= fanout[i];  // below 2^31 by the call's plan
    if (pairs * fanout[k - 1] >= 20000000 &&
        ((gr.E >= 300 * gr.V && pairs >= 8 * gr.V) || (gr.E >= 80 * gr.V && pairs >= 16 * gr.V)))
        return false;
    int64_t w = 1, prev = 1;
    for (int32_t i = 0; i + 1 < k; ++i) {
        prev = w;
        w *= fanout[i];
        if (w + prev > kFusedRows) return false;
    }
    return w * fanout[k - 1] < (1ll << 31);
}

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
#define ND_FUSED_LAUNCH(STRIDE, OFFT)                                                                              \
    do {                                                                                                           \
        if (pairs)                                                                                                 \
            hipLaunchKernelGGL((khop_fused_kernel<STRIDE, 2, OFFT>), grid, block, f.lds, stream, view_of<OFFT>(gr), a); \
        else                                                                                                       \
            hipLaunchKernelGGL((khop_fused_kernel<STRIDE, 1, OFFT>), grid, block, f.lds, stream, view_of<OFFT>(gr), a); \
    } while (0)
    if (gr.off64) {
        if (gr.wq) ND_FUSED_LAUNCH(2, int64_t);
        else ND_FUSED_LAUNCH(1, int64_t);
    } else {
        if (gr.wq) ND_FUSED_LAUNCH(2, int32_t);
        else ND_FUSED_LAUNCH(1, int32_t);
    }
#undef ND_FUSED_LAUNCH
    ND_HIP_CHECK(hipGetLastError());
    return ND_OK;
}

}  // namespace nd
