// Collective transit sampling (Section 6.2 of the paper; layer sampling with
// LADIES-style importance weights, Section 4.2 "Importance Sampling").
//
// The paper materialises every sample's combined neighbourhood in global
// memory (transit-parallel copy of whole adjacency lists) and then draws from
// it sample-parallel.  On this GPU the copy is the dominant traffic, so the
// combined neighbourhood stays implicit: it is the concatenation, in slot
// order, of the transits' adjacency lists, described by a running sum of
// per-transit masses deg(v) * c(v) kept in LDS; a draw picks a position in the
// concatenation by inverse transform (binary search over the running sums,
// then an integer division by c(v) inside the chosen list) and reads that one
// neighbour.  One workgroup per sample, as in the paper's sample-parallel draw.
// A transit's degree and row start are fetched once per (sample, transit slot).
//
// c(v) = floor(2^48 / deg(v)^2) is the fixed-point squared entry of the
// row-normalised adjacency matrix, so a vertex is drawn with probability
// proportional to its squared column norm restricted to the transit rows.
#include "nd_common.h"
#include "nd_philox.h"
#include "nd_sample.h"
#include "nd_draw.h"
#include "nd_wave.h"

namespace nd {

namespace {

// 512 lanes per sample: the transits' 24 bytes each of LDS allow three workgroups per CU, and the
// draws are chains of dependent reads, so the wider workgroup (24 waves per CU) hides more latency
constexpr int kLayerThreads = 512;

// Exact floor(num / c) for num < 2^24 * c: the quotient is estimated in double precision
// (relative error 2^-52, so off by at most one for a quotient below 2^24) and corrected with
// integer arithmetic.
__device__ __forceinline__ uint64_t div_small_quotient(uint64_t num, uint64_t c) {
    uint64_t q = (uint64_t)((double)num / (double)c);
    int64_t r = (int64_t)(num - q * c);
    if (r < 0) {
        --q;
        r += (int64_t)c;
    }
    if (r >= (int64_t)c) ++q;
    return q;
}

// Dynamic LDS: per transit slot the running sum of masses, the weight c(v) and the first
// adjacency entry of the transit (24 bytes), so a draw touches global memory once.
// WEIGHTED: an entry from transit v to u weighs the graph's quantised edge weight w_q(v,u); the
// mass of a transit is its row's weight sum and the place inside the row is found by a search
// over the row's running sums (global memory).
template <typename OffT, bool WEIGHTED>
__global__ __launch_bounds__(kLayerThreads) void layer_kernel(GraphView<OffT> g, LayerArgs a) {
    extern __shared__ uint64_t lds[];
    uint64_t* s_incl = lds;
    uint64_t* s_c = lds + a.n_prev;
    uint64_t* s_rs = lds + 2 * (size_t)a.n_prev;
    __shared__ uint64_t scan_tmp[kLayerThreads / 64 + 1];
    const uint32_t b = blockIdx.x;
    const int32_t* transits = a.transits + (uint64_t)b * a.n_prev;

    uint64_t carry = 0;
    bool bad = false;
    for (uint32_t base = 0; base < a.n_prev; base += kLayerThreads) {
        const uint32_t t = base + threadIdx.x;
        uint64_t mass = 0, c = 0, rs = 0;
        if (t < a.n_prev) {
            int32_t v = transits[t];
            if (v >= g.V || v < ND_NULL_VERTEX) {
                bad = true;
                v = ND_NULL_VERTEX;
            }
            if (v >= 0) {
                rs = (uint64_t)g.off[v];
                const uint64_t deg = (uint64_t)g.off[v + 1] - rs;
                if (deg > 0) {
                    if (WEIGHTED) {
                        c = deg;  // the row length takes the weight's place
                        mass = g.cumq[rs + deg - 1];
                    } else {
                        c = (1ull << 48) / (deg * deg);
                        mass = deg * c;
                    }
                }
            }
        }
        uint64_t total;
        const uint64_t ex = block_exclusive_scan<uint64_t, kLayerThreads>(mass, scan_tmp, &total);
        if (t < a.n_prev) {
            s_incl[t] = carry + ex + mass;
            s_c[t] = c;
            s_rs[t] = rs;
        }
        carry += total;
        __syncthreads();
    }
    if (a.check_roots && bad) atomicOr(a.status, 1u);
    const uint64_t total = carry;

    for (uint32_t j = threadIdx.x; j < a.m; j += kLayerThreads) {
        int32_t res = ND_NULL_VERTEX;
        if (total > 0) {
            const Rand4 r = draw4(a.seed, a.sample_base + b, j, a.step, 0u);
            const uint64_t x = mulhi64(cat64(r.r0, r.r1), total);
            uint32_t lo = 0, hi = a.n_prev - 1;
            while (lo < hi) {  // first transit whose running sum exceeds x
                const uint32_t mid = (lo + hi) >> 1;
                if (s_incl[mid] > x) hi = mid;
                else lo = mid + 1;
            }
            const uint64_t before = lo ? s_incl[lo - 1] : 0ull;
            uint64_t idx;
            if (WEIGHTED) {  // first entry of the row whose running sum exceeds what is left of x
                const uint64_t* cum = g.cumq + s_rs[lo];
                const uint64_t rest = x - before;
                uint64_t l = 0, h = s_c[lo] - 1;
                while (l < h) {
                    const uint64_t mid = (l + h) >> 1;
                    if (cum[mid] > rest) h = mid;
                    else l = mid + 1;
                }
                idx = l;
            } else {
                idx = div_small_quotient(x - before, s_c[lo]);
            }
            res = g.col[s_rs[lo] + idx];
        }
        a.out[(uint64_t)b * a.m + j] = res;
    }
}

// ---------------------------------------------------------------- all steps of a sample in one launch
// A sample's steps depend on nothing but the sample, so its workgroup does them one after the other: the
// rows of a step's transits come with the links of the entries that were drawn (off, then off + 1, are
// only looked up for the roots) and stay in LDS.  One scattered line per draw is what a large call is bound
// by; a call with a few samples is a chain of dependent fetches, and what counts there is their number.
// Inside a weighted row the guide table (WeightLink) starts the search, where a binary search over the
// running sums is one fetch per level: 257 samples of [512, 512] over 2.9 M vertices, symmetric weights,
// took 37 us with a launch per step and the binary search, 30.9 us like this, and 29.6 with the rows' weight sums in an
// array of their own: 24 MB of it instead of places all over 0.9 GB of running sums, and for a root known before its
// row is (a draw's fetches take 5 of the 12 us of a step, over 4 GB of links).
struct LayerFusedArgs {
    const Link* links;
    uint64_t seed;
    uint32_t sample_base;
    uint32_t S;
    int32_t k;
    uint32_t n[ND_MAX_FANOUT_STEPS];    // transits of a step (roots_per_sample, then the fanouts)
    uint32_t m[ND_MAX_FANOUT_STEPS];    // draws of a step
    uint32_t o_rows_b, o_incl;          // in LDS, in bytes: the second rows buffer, the running sums
    uint32_t o_v;                       // ... and, where totals are, the rows' vertices
    const uint64_t* totals;             // weighted: sum of every vertex's row, may be null
    const int32_t* roots;
    int32_t* out[ND_MAX_FANOUT_STEPS];
    WsHeader* hdr;
    uint32_t* flags;
    uint64_t o_flags;
};

// c(v) = floor(2^48 / deg^2).  In double precision: deg^2 < 2^48 is exact, and the quotient lies at least
// 2^-48 of its value below the next whole number, which rounding to 2^-53 does not bridge.
__device__ __forceinline__ uint64_t column_weight(uint32_t deg) {
    return (uint64_t)(281474976710656.0 / ((double)deg * (double)deg));
}

// The link of the first entry of a row whose running sum exceeds rest < total.  ceil(rest * 2^64 / total) is a
// word that a draw over this row alone would turn into `rest`, so the row's own thresholds answer in its place:
// thr rises with the running sum (2^64 / total exceeds 2^25, so different sums have different thresholds).  It
// looks at nothing but the row's links: over the running sums, four at a time, and the link or column after
// them, a draw was three dependent fetches and a third array: 257 samples of [512, 512] over 2.9 M vertices took
// 31.4 us, 97 on a graph not looked at before; now 30.9 and 76.
__device__ __forceinline__ Link guided_search(const Link* row, uint32_t deg, uint64_t rest, uint64_t total) {
    if (deg == 1u) return row[0];
    return drawn_link(row, deg, scaled_threshold(rest, total));
}

template <typename OffT, bool WEIGHTED, int STRIDE, int THREADS>
__global__ __launch_bounds__(THREADS) void layer_fused_kernel(GraphView<OffT> g, LayerFusedArgs a) {
    extern __shared__ uint64_t lds[];
    char* mem = (char*)lds;
    uint2* buf_a = (uint2*)mem;
    uint2* buf_b = (uint2*)(mem + a.o_rows_b);
    uint64_t* s_incl = (uint64_t*)(mem + a.o_incl);
    int32_t* s_v = (int32_t*)(mem + a.o_v);
    __shared__ uint64_t scan_tmp[THREADS / 64 + 1];
    bool bad = false;
    for (uint32_t b = blockIdx.x; b < a.S; b += gridDim.x) {
        for (uint32_t t = threadIdx.x; t < a.n[0]; t += THREADS) {
            const int32_t v = a.roots[(uint64_t)b * a.n[0] + t];
            uint2 row = make_uint2(0u, 0u);
            if (v >= g.V || v < ND_NULL_VERTEX) bad = true;
            else if (v >= 0) {
                const uint64_t rs = (uint64_t)g.off[v];
                row = make_uint2((uint32_t)rs, row_length(g, v, rs));
                if (WEIGHTED && a.totals) s_v[t] = v;
            }
            buf_a[t] = row;
        }
        __syncthreads();
        for (int step = 0; step < a.k; ++step) {
            const uint2* rows = (step & 1) ? buf_b : buf_a;
            uint2* next = (step & 1) ? buf_a : buf_b;
            const uint32_t n = a.n[step], m = a.m[step];
            const bool last = step == a.k - 1;
            // running sums of the transits' masses: every thread a stretch of its own, one scan
            const uint32_t per = (n + THREADS - 1) / THREADS;
            const uint32_t t0 = threadIdx.x * per, t1 = t0 + per < n ? t0 + per : n;
            uint64_t sum = 0;
            for (uint32_t t = t0; t < t1; ++t) {
                const uint2 row = rows[t];
                if (row.y > 0u) {
                    if (WEIGHTED) sum += a.totals ? a.totals[s_v[t]] : g.cumq[(uint64_t)row.x + row.y - 1u];
                    else sum += row.y * column_weight(row.y);
                }
                s_incl[t] = sum;
            }
            uint64_t total;
            const uint64_t before_me = block_exclusive_scan<uint64_t, THREADS>(sum, scan_tmp, &total);
            for (uint32_t t = t0; t < t1; ++t) s_incl[t] += before_me;
            __syncthreads();
            int32_t* out = a.out[step] + (uint64_t)b * m;
            for (uint32_t j = threadIdx.x; j < m; j += THREADS) {
                int32_t res = ND_NULL_VERTEX;
                uint2 row_out = make_uint2(0u, 0u);
                if (total > 0) {
                    const Rand4 r = draw4(a.seed, a.sample_base + b, j, (uint32_t)step, 0u);
                    const uint64_t x = mulhi64(cat64(r.r0, r.r1), total);
                    uint32_t lo = 0, hi = n - 1u;
                    while (lo < hi) {  // first transit whose running sum exceeds x
                        const uint32_t mid = (lo + hi) >> 1;
                        if (s_incl[mid] > x) hi = mid;
                        else lo = mid + 1u;
                    }
                    const uint64_t before = lo ? s_incl[lo - 1u] : 0ull;
                    const uint2 row = rows[lo];
                    if (WEIGHTED) {
                        const Link l = guided_search(a.links + 2ull * row.x, row.y, x - before, s_incl[lo] - before);
                        res = l.v;
                        row_out = make_uint2(l.rs, l.deg);
                    } else {
                        const uint64_t e = row.x + div_small_quotient(x - before, column_weight(row.y));
                        if (last) {
                            res = g.col[e];
                        } else {
                            const Link l = a.links[e * STRIDE];
                            res = l.v;
                            row_out = make_uint2(l.rs, l.deg);
                        }
                    }
                }
                out[j] = res;
                if (!last) {
                    next[j] = row_out;
                    if (WEIGHTED && a.totals) s_v[j] = res;  // this step's have been read
                }
            }
            __syncthreads();  // the next step reads the rows and rewrites the sums
        }
    }
    const int any = __syncthreads_or(bad ? 1 : 0);
    if (threadIdx.x == 0) {
        a.flags[blockIdx.x] = any ? 1u : 0u;
        if (blockIdx.x == 0) write_header(a.hdr, (uint32_t)a.k, gridDim.x, a.o_flags, 0);
    }
}

}  // namespace

// Dynamic LDS above the 64 KB default has to be allowed once per kernel; done when a graph is
// created so that layer_step itself only launches.
int layer_prepare() {
#define ND_LAYER_ALLOW(OFFT, W)                                                                 \
    ND_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(&layer_kernel<OFFT, W>),     \
                                     hipFuncAttributeMaxDynamicSharedMemorySize,                \
                                     ND_MAX_LAYER_TRANSITS * 24))
    ND_LAYER_ALLOW(int64_t, true);
    ND_LAYER_ALLOW(int64_t, false);
    ND_LAYER_ALLOW(int32_t, true);
    ND_LAYER_ALLOW(int32_t, false);
#undef ND_LAYER_ALLOW
#define ND_LAYER_ALLOW_T(OFFT, W, STRIDE, T)                                                               \
    ND_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(&layer_fused_kernel<OFFT, W, STRIDE, T>), \
                                     hipFuncAttributeMaxDynamicSharedMemorySize,                           \
                                     ND_MAX_LAYER_TRANSITS * 28))
#define ND_LAYER_ALLOW(OFFT, W, STRIDE)       \
    ND_LAYER_ALLOW_T(OFFT, W, STRIDE, 64);    \
    ND_LAYER_ALLOW_T(OFFT, W, STRIDE, 128);   \
    ND_LAYER_ALLOW_T(OFFT, W, STRIDE, 256);   \
    ND_LAYER_ALLOW_T(OFFT, W, STRIDE, 512);   \
    ND_LAYER_ALLOW_T(OFFT, W, STRIDE, 1024)
    ND_LAYER_ALLOW(int64_t, true, 2);
    ND_LAYER_ALLOW(int64_t, false, 2);
    ND_LAYER_ALLOW(int64_t, false, 1);
    ND_LAYER_ALLOW(int32_t, true, 2);
    ND_LAYER_ALLOW(int32_t, false, 2);
    ND_LAYER_ALLOW(int32_t, false, 1);
#undef ND_LAYER_ALLOW_T
#undef ND_LAYER_ALLOW
    return ND_OK;
}

constexpr size_t kLdsPerUnit = 160 << 10;
constexpr size_t kLdsPiece = 1280;                            // LDS is given out in pieces of this size
constexpr size_t kLayerStaticLds = 256 + (512 / 64 + 1) * 8;  // the kernel's votes and its scan, with 512 lanes

// Samples of 512 lanes that a compute unit has at a time: by their LDS, and by registers at most three.
int64_t layer_samples_per_unit(size_t lds_bytes) {
    const size_t each = (lds_bytes + kLayerStaticLds + kLdsPiece - 1) / kLdsPiece * kLdsPiece;
    const int64_t n = (int64_t)(kLdsPerUnit / each);
    return n < 3 ? n : 3;
}

int64_t layer_fused_groups(const Graph& gr, int64_t S) {
    const int64_t most = (int64_t)gr.num_cus * 64;  // bounds the flags; the workgroups stride over the samples
    return S < most ? S : most;
}

int layer_fused(const Graph& gr, uint64_t seed, uint32_t sample_base, bool weighted, int32_t roots_per_sample,
                const int32_t* fanout, int32_t k, int64_t S, const int32_t* roots, int32_t* const* step_out, char* ws,
                uint64_t o_flags, hipStream_t stream) {
    LayerFusedArgs a{};
    a.links = gr.links;
    a.seed = seed;
    a.sample_base = sample_base;
    a.S = (uint32_t)S;
    a.k = k;
    uint32_t rows[2] = {0, 0}, widest = 0, most_draws = 0;
    for (int32_t i = 0; i < k; ++i) {
        a.n[i] = (uint32_t)(i == 0 ? roots_per_sample : fanout[i - 1]);
        a.m[i] = (uint32_t)fanout[i];
        a.out[i] = step_out[i];
        if (a.m[i] > most_draws) most_draws = a.m[i];
        if (a.n[i] > rows[i & 1]) rows[i & 1] = a.n[i];
        if (a.n[i] > widest) widest = a.n[i];
    }
    a.o_rows_b = rows[0] * 8u;
    a.o_incl = a.o_rows_b + rows[1] * 8u;
    a.o_v = a.o_incl + widest * 8u;
    // At most 24 bytes per transit, 28 with totals; without them where a call's samples then run at once and would not
    // with them.  Without and with, us: 512 samples of [2920,2920] over 1.6 M entries 110 and 132 (two per unit and
    // one), 700 of [2100,2100] 110 and 132 (three and two), 257 of [3200,3200] 93 and 108; more samples take more rounds
    // either way, and the totals make up for it (4,096 of [3200,3200] 951 and 924; over 115 M entries 1,630 and 1,549).
    const size_t with = (size_t)a.o_v + (size_t)widest * 4u;
    const bool waits = S > (int64_t)gr.num_cus * layer_samples_per_unit(with) &&
                       S <= (int64_t)gr.num_cus * layer_samples_per_unit(a.o_v);
    a.totals = weighted && !waits ? gr.totals.load(std::memory_order_acquire) : nullptr;
    const size_t lds_bytes = a.totals ? with : (size_t)a.o_v;
    a.roots = roots;
    a.hdr = (WsHeader*)ws;
    a.flags = (uint32_t*)(ws + o_flags);
    a.o_flags = o_flags;
    mark_phase(ND_PHASE_LAYER, stream);
    // A lane per transit and draw up to 512, so that a compute unit holds as many small samples as it can: 50,000
    // samples of 4 transits and 7 draws over 1.6 M entries take 31 us with 64 lanes, 55, 91 and 179 with 128, 256
    // and 512; 3,000 of [100,100,100] 17 with 64 or 128, 42 with 512; 2,000 of [512,512] 25 with 128 or 256, 28
    // with 512, but 257 of them 29 with 64 and 10.5 with 512.  1,024 lanes where a unit has one sample at a time,
    // because there are no more (200 of [2048]: 9.5 us, 10.4 with 512; 300: 16.4 and 13.2) or because two
    // do not fit its LDS (600 of [4096,4096]: 108 and 137).
    const uint32_t lanes = widest > most_draws ? widest : most_draws;
    const bool one_each = S <= (int64_t)gr.num_cus || layer_samples_per_unit(lds_bytes) == 1;
    const int threads = lanes <= 64u ? 64 : lanes <= 128u ? 128 : lanes <= 256u ? 256
                        : lanes > 512u && one_each ? 1024 : 512;
#define ND_LAYER_LAUNCH_T(OFFT, W, STRIDE, T)                                                               \
    hipLaunchKernelGGL((layer_fused_kernel<OFFT, W, STRIDE, T>), dim3((unsigned)layer_fused_groups(gr, S)), \
                       dim3(T), lds_bytes, stream, view_of<OFFT>(gr), a)
#define ND_LAYER_LAUNCH(OFFT, W, STRIDE)                       \
    do {                                                       \
        if (threads == 64) ND_LAYER_LAUNCH_T(OFFT, W, STRIDE, 64);        \
        else if (threads == 128) ND_LAYER_LAUNCH_T(OFFT, W, STRIDE, 128); \
        else if (threads == 256) ND_LAYER_LAUNCH_T(OFFT, W, STRIDE, 256); \
        else if (threads == 512) ND_LAYER_LAUNCH_T(OFFT, W, STRIDE, 512); \
        else ND_LAYER_LAUNCH_T(OFFT, W, STRIDE, 1024);                    \
    } while (0)
    if (gr.off64) {
        if (weighted) ND_LAYER_LAUNCH(int64_t, true, 2);
        else if (gr.wq) ND_LAYER_LAUNCH(int64_t, false, 2);
        else ND_LAYER_LAUNCH(int64_t, false, 1);
    } else {
        if (weighted) ND_LAYER_LAUNCH(int32_t, true, 2);
        else if (gr.wq) ND_LAYER_LAUNCH(int32_t, false, 2);
        else ND_LAYER_LAUNCH(int32_t, false, 1);
    }
#undef ND_LAYER_LAUNCH_T
#undef ND_LAYER_LAUNCH
    ND_HIP_CHECK(hipGetLastError());
    return ND_OK;
}

// One step with the rows looked up per transit: graphs without links.
int layer_step(const Graph& gr, const LayerArgs& a, int64_t num_samples, hipStream_t stream) {
    if (num_samples == 0) return ND_OK;
    const size_t lds_bytes = (size_t)a.n_prev * 24;  // at most 96 KB of the 160 KB per CU
#define ND_LAYER_LAUNCH(OFFT, W)                                                                    \
    hipLaunchKernelGGL((layer_kernel<OFFT, W>), dim3((unsigned)num_samples), dim3(kLayerThreads),  \
                       lds_bytes, stream, view_of<OFFT>(gr), a)
    if (gr.off64) {
        if (a.use_weights) ND_LAYER_LAUNCH(int64_t, true);
        else ND_LAYER_LAUNCH(int64_t, false);
    } else {
        if (a.use_weights) ND_LAYER_LAUNCH(int32_t, true);
        else ND_LAYER_LAUNCH(int32_t, false);
    }
#undef ND_LAYER_LAUNCH
    ND_HIP_CHECK(hipGetLastError());
    return ND_OK;
}

}  // namespace nd
