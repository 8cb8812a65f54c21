// k-hop sampling (Section 3 and Section 6.1 of the paper: `stepSize(i)` uniform neighbours of every
// transit) by two routes that need no exact grouping by transit:
//
//   fused    every workgroup carries a few samples through all hops: what a hop draws is a Link, which
//            holds the row of the drawn vertex, so the next hop finds its rows in LDS.  One launch,
//            nothing read back from the outputs, no sort.  For calls that draw too little of the
//            graph for two draws to meet in a cache line.
//   grouped  a step with many draws per line of the graph: its (transit, slot) pairs are brought into
//            256 buckets of neighbouring transits by one stable radix pass, drawn bucket by bucket while
//            the bucket's rows sit in L2, written in that order, and put back into slot order by a pass
//            that reads 256 rising streams and writes whole lines (NULL included).
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

// A place in a buffer of rows: where the row of a slot's vertex lies.
__device__ __forceinline__ uint2 row_of_link(const Link& l) { return make_uint2(l.rs, l.deg); }

// Bound by latency (small calls: a hop is generator, link, row; 37 roots of three hops take one launch
// instead of 26) or by the rate of scattered fetches (large ones).
template <int STRIDE, typename OffT>
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
                const Rand4 r = draw4(a.seed, a.sample_base + s0 + s, d - s * W, (uint32_t)hop, 0u);
                Link l;
                l.v = ND_NULL_VERTEX;
                l.rs = 0;
                l.deg = 0;
                if (row.y > 0u) {
                    l = a.links[(uint64_t)(row.x + mulhi32(r.r0, row.y)) * STRIDE];
                    ++live;
                }
                next[d] = row_of_link(l);
                if (part == 0) out[d] = l.v;
            }
            if (live) atomicAdd(&s_live[hop + 1], live);
        } else {
            // four independent draws per lane and round
            const uint32_t share = ((total + a.splits - 1u) / a.splits + T - 1u) / T * T;
            const uint32_t begin = part * share;
            const uint32_t end = begin + share < total ? begin + share : total;
            for (uint32_t d0 = begin + tid; d0 < end; d0 += 4u * T) {
                uint2 row[4];
                uint32_t e[4];
                int32_t v[4];
#pragma unroll
                for (uint32_t u = 0; u < 4u; ++u) {
                    const uint32_t d = d0 + u * T < end ? d0 + u * T : d0;
                    row[u] = rows[fastdiv(d, a.div_m[hop])];
                    const uint32_t s = fastdiv(d, a.div_w[hop]);
                    e[u] = 0;
                    if (u == 0 || d != d0) {
                        const Rand4 r = draw4(a.seed, a.sample_base + s0 + s, d - s * W, (uint32_t)hop, 0u);
                        e[u] = row[u].x + mulhi32(r.r0, row[u].y);
                    }
                }
#pragma unroll
                for (uint32_t u = 0; u < 4u; ++u) {
                    v[u] = ND_NULL_VERTEX;
                    if (row[u].y > 0u && d0 + u * T < end) v[u] = g.col[e[u]];
                }
#pragma unroll
                for (uint32_t u = 0; u < 4u; ++u)
                    if (d0 + u * T < end) out[d0 + u * T] = v[u];
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

void slots_per_sample(const int32_t* fanout, int32_t k, int64_t* W) {
    int64_t w = 1;
    for (int32_t i = 0; i < k; ++i) W[i] = w = w * fanout[i];
}

}  // namespace

bool khop_fused_fits(const Graph& gr, const int32_t* fanout, int32_t k) {
    if (!gr.links) return false;
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
#define ND_FUSED_LAUNCH(STRIDE, OFFT) \
    hipLaunchKernelGGL((khop_fused_kernel<STRIDE, OFFT>), grid, block, f.lds, stream, view_of<OFFT>(gr), a)
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
