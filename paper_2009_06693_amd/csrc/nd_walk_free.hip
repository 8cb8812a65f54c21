// Random walks whose lanes run free: the default route of the walks.
//
// A walk step is a chain - generator, edge, the row of the vertex it leads to - and its output must
// not depend on how samples are grouped.  Grouping by transit (Section 6.1.2 of the paper, GPU-wide
// or in the windows of nd_walk.hip) costs barriers and LDS traffic at every step to save scattered
// reads that the caches mostly serve already; what a walk is bound by is the chain itself (few walks)
// or the rate of scattered fetches (many).  Both are cut by the graph's Links: the edge that is drawn
// carries the row of its end vertex, so a step is one fetch instead of two dependent ones, and a lane
// keeps its walk in registers from the first step to the last, with no barrier in between.
#include "nd_common.h"
#include "nd_philox.h"
#include "nd_wave.h"
#include "nd_sample.h"
#include "nd_draw.h"

namespace nd {

namespace {

constexpr int kFreeChunk = 128;  // steps per launch: their output pointers are kernel arguments

struct FreeArgs {
    const Link* links;
    uint64_t seed;
    uint64_t ppr_thr;
    uint32_t sample_base;
    uint32_t S;
    uint32_t first_step, n_steps;
    int32_t V;
    const int32_t* src;        // the roots, or the output of step first_step - 1
    WsHeader* hdr;
    uint32_t* flags;           // per workgroup: a root was outside [0, V) (first launch)
    uint32_t* parts;           // [workgroup][step of the call]: live walks
    uint32_t total_steps;
    uint64_t o_flags, o_parts;
    int32_t* out[kFreeChunk];
};

// Live pairs of every step, from what each lane knows at the end: its walk had a transit at the first
// `lived` steps of this launch.  One histogram entry per lane, then sums from the top.
template <int THREADS>
__device__ __forceinline__ void publish_live(uint32_t lived, uint32_t n_steps, uint32_t* hist, uint32_t* parts) {
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
            if (step < n_steps) parts[step] = carry + incl;
            carry += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        }
    }
}

// The walk's first transit and, in the first launch, what the host may ask for afterwards.
template <int THREADS>
__device__ __forceinline__ int32_t first_transit(const FreeArgs& a, uint32_t s) {
    int32_t v = s < a.S ? a.src[s] : ND_NULL_VERTEX;
    if (a.first_step == 0) {
        const bool bad = v >= a.V || v < ND_NULL_VERTEX;
        if (bad) v = ND_NULL_VERTEX;
        const int any = __syncthreads_or(bad ? 1 : 0);
        if (threadIdx.x == 0) {
            a.flags[blockIdx.x] = any ? 1u : 0u;
            if (blockIdx.x == 0) write_header(a.hdr, a.total_steps, gridDim.x, a.o_flags, a.o_parts);
        }
    }
    return v;
}

// DeepWalk and PPR.  Many walks: bound by the scattered 128-byte fetches of the links (one per draw;
// the chip serves 5.5e10 of them per second whatever the array's size).  Few walks: by one fetch per
// step, the generator runs while it is under way.
template <int DRAW, int STRIDE, typename OffT, int THREADS>
__global__ __launch_bounds__(THREADS) void walk_free_kernel(GraphView<OffT> g, FreeArgs a) {
    __shared__ uint32_t s_hist[kFreeChunk + 1];
    const uint32_t s = blockIdx.x * (uint32_t)THREADS + threadIdx.x;
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
    for (uint32_t si = 0; si < a.n_steps; ++si) {
        lived += v >= 0 ? 1u : 0u;
        const bool draws = deg > 0u && !(a.ppr_thr != 0 && (uint64_t)r.r3 < a.ppr_thr);
        Link l;
        l.v = ND_NULL_VERTEX;
        l.rs = 0;
        l.deg = 0;
        if (draws) {
            const uint32_t i = mulhi32(r.r0, deg);
            if (DRAW == kDrawUniform) {
                l = a.links[(uint64_t)(rs + i) * STRIDE];
            } else {
                const Link* row = a.links + (uint64_t)rs * 2u;
                const uint64_t R = cat64(r.r0, r.r1);
                uint32_t j = reinterpret_cast<const WeightLink*>(row)[2u * i + 1u].guide;
                for (;; ++j) {  // ends at the row's last entry; two entries are on their way at a time
                    const uint32_t j1 = j + 1u < deg ? j + 1u : j;
                    const WeightLink w0 = reinterpret_cast<const WeightLink*>(row)[2u * j + 1u];
                    const WeightLink w1 = reinterpret_cast<const WeightLink*>(row)[2u * j1 + 1u];
                    const Link l0 = row[2u * j], l1 = row[2u * j1];
                    if (R < w0.thr || w0.always || j == j1) {
                        l = l0;
                        break;
                    }
                    if (R < w1.thr || w1.always || j1 + 1u == deg) {
                        l = l1;
                        break;
                    }
                    j = j1;
                }
            }
        }
        // the next step's word does not wait for the link
        r = draw4(a.seed, sid, 0u, a.first_step + si + 1u, 0u);
        v = l.v;
        rs = l.rs;
        deg = l.deg;
        if (s < a.S) a.out[si][s] = v;
    }
    publish_live<THREADS>(lived, a.n_steps, s_hist, a.parts + (uint64_t)blockIdx.x * a.total_steps + a.first_step);
}

template <int THREADS, typename OffT>
void launch_free(const Graph& gr, int draw, const FreeArgs& a, hipStream_t stream) {
    const dim3 grid((a.S + THREADS - 1u) / THREADS), block(THREADS);
    const GraphView<OffT> g = view_of<OffT>(gr);
    if (draw == kDrawWeighted)
        hipLaunchKernelGGL((walk_free_kernel<kDrawWeighted, 2, OffT, THREADS>), grid, block, 0, stream, g, a);
    else if (gr.wq)
        hipLaunchKernelGGL((walk_free_kernel<kDrawUniform, 2, OffT, THREADS>), grid, block, 0, stream, g, a);
    else
        hipLaunchKernelGGL((walk_free_kernel<kDrawUniform, 1, OffT, THREADS>), grid, block, 0, stream, g, a);
}

}  // namespace

// One walk per lane, and a workgroup of one wavefront as long as that gives every compute unit at
// most a few of them (a step then waits for nobody else); more walks take workgroups of four, which
// have fewer headers and counters to write.
static int free_threads(int64_t S) { return S <= 65536 ? 64 : 256; }

int64_t walk_free_groups(int64_t S) { return (S + free_threads(S) - 1) / free_threads(S); }

int walk_free(const Graph& gr, int draw, const DrawArgs& d, int64_t S, int32_t num_steps, const int32_t* roots,
              int32_t* const* step_out, char* ws, uint64_t o_flags, uint64_t o_parts, hipStream_t stream) {
    FreeArgs a{};
    a.links = gr.links;
    a.seed = d.seed;
    a.ppr_thr = d.ppr_thr;
    a.sample_base = d.sample_base;
    a.S = (uint32_t)S;
    a.V = (int32_t)gr.V;
    a.hdr = (WsHeader*)ws;
    a.flags = (uint32_t*)(ws + o_flags);
    a.parts = (uint32_t*)(ws + o_parts);
    a.total_steps = (uint32_t)num_steps;
    a.o_flags = o_flags;
    a.o_parts = o_parts;
    for (int32_t first = 0; first < num_steps; first += kFreeChunk) {
        const int32_t n = num_steps - first < kFreeChunk ? num_steps - first : kFreeChunk;
        a.first_step = (uint32_t)first;
        a.n_steps = (uint32_t)n;
        a.src = first > 0 ? step_out[first - 1] : roots;
        for (int32_t i = 0; i < kFreeChunk; ++i) a.out[i] = i < n ? step_out[first + i] : nullptr;
        mark_phase(ND_PHASE_WALK_WINDOW, stream);
        if (gr.off64) {
            if (free_threads(S) == 64) launch_free<64, int64_t>(gr, draw, a, stream);
            else launch_free<256, int64_t>(gr, draw, a, stream);
        } else {
            if (free_threads(S) == 64) launch_free<64, int32_t>(gr, draw, a, stream);
            else launch_free<256, int32_t>(gr, draw, a, stream);
        }
        ND_HIP_CHECK(hipGetLastError());
    }
    return ND_OK;
}

}  // namespace nd
