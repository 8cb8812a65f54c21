// Output format 1 of the paper (Section 4.1, "Output format"): one record per
// sample that holds everything the sample gained at all steps, which is what
// consumers of random walks and layer samples read.  The sampling steps write
// one array per step (format 2); this file gathers them into records:
//
//     samples[s][off_i + j] = step_out[i][s * w_i + j],  off_i = w_0 + ... + w_{i-1}
//
// A step with several slots per sample moves runs of w_i ints, which coalesce on
// both sides.  Walk steps (w_i = 1) are a transpose of [steps][samples]: a workgroup takes 32 or 64
// samples and up to 128 steps through LDS, so that it reads rows of 128 or 256 bytes of the step arrays, all of
// them requested before the first is stored, and writes its samples' records as one stretch of memory.
// (Tiles of 32 steps cut a 100-step record into pieces that end inside a 128-byte line, and a line
// written in two pieces is read in between: 2.0 ms for 4.2 M walks of 100 steps.)
#include "nd_common.h"
#include "nd_pack.h"
#include "nd_philox.h"

namespace nd {

namespace {

constexpr int kTileSteps = 128;
// Up to here 32 samples per workgroup: 16,384 walks of 100 steps 5.7 us, 6.2 with 64; 57,000 11.0 and 9.6.
constexpr int64_t kFewSamples = 16384;

struct WalkChunk {
    const int32_t* step[kTileSteps];  // step arrays of this chunk (w = 1)
    int32_t n_steps;                  // used entries
    int32_t first_col;                // record position of the chunk's first step
    FastDiv div_steps;                // by n_steps
};

// Four neighbouring samples of a step per load and four entries of the stretch per store, wherever they lie: the memory
// takes 16 bytes at any multiple of four.  Bound by memory: 4.2 M walks of 100 steps 1,073 us with an entry per load and
// store, 626 like this (5.4 TB/s, a large copy 5.1), 1 M walks of 80 steps that start anywhere 222 and 140; 4,096 walks 8.9 and 5.2, with 32 samples per workgroup, which are
// then as many workgroups as the chip has compute units and more loads at once per sample (64: 7.0).
typedef int32_t Int4 __attribute__((ext_vector_type(4), aligned(4)));
template <int SAMPLES>
__global__ __launch_bounds__(256) void pack_walk_kernel(WalkChunk c, int64_t S, int64_t rec_len,
                                                        int32_t* __restrict__ samples) {
    extern __shared__ int32_t tile[];  // [n_steps][SAMPLES + 1]: a column is free of bank conflicts
    constexpr uint32_t kPitch = SAMPLES + 1, kLanes = SAMPLES / 4, kRows = 256 / kLanes;  // lanes per row, rows at a time
    const int64_t s0 = (int64_t)blockIdx.x * SAMPLES;
    const uint32_t n_here = S - s0 < SAMPLES ? (uint32_t)(S - s0) : (uint32_t)SAMPLES;
    const uint32_t s_mine = threadIdx.x % kLanes * 4u, row = threadIdx.x / kLanes;
    const uint32_t n = (uint32_t)c.n_steps;
    const uint32_t left = s_mine < n_here ? n_here - s_mine : 0u;
    for (uint32_t i0 = row; i0 < n; i0 += 8u * kRows) {
        Int4 x[8];
#pragma unroll
        for (uint32_t r = 0; r < 8u; ++r)
            if (i0 + r * kRows < n) {
                const int32_t* from = c.step[i0 + r * kRows] + s0 + s_mine;
                if (left >= 4u) {
                    x[r] = *reinterpret_cast<const Int4*>(from);
                } else {
                    x[r].x = left > 0u ? from[0] : 0;
                    x[r].y = left > 1u ? from[1] : 0;
                    x[r].z = left > 2u ? from[2] : 0;
                }
            }
#pragma unroll
        for (uint32_t r = 0; r < 8u; ++r)
            if (i0 + r * kRows < n) {
                int32_t* to = tile + (i0 + r * kRows) * kPitch + s_mine;
                to[0] = x[r].x;
                to[1] = x[r].y;
                to[2] = x[r].z;
                to[3] = x[r].w;
            }
    }
    __syncthreads();
    const uint32_t total = n_here * n;
    // where records are longer than this chunk, four entries lie together only inside one of its pieces
    const bool together = n % 4u == 0u || rec_len == (int64_t)n;
    for (uint32_t e = threadIdx.x * 4u; e < total; e += 1024u) {
        uint32_t r = fastdiv(e, c.div_steps), col = e - r * n;
        int32_t* to = samples + (s0 + r) * rec_len + c.first_col + col;
        int32_t y[4];
#pragma unroll
        for (uint32_t k = 0; k < 4u; ++k) {
            if (e + k < total) {
                y[k] = tile[col * kPitch + r];
                if (!together) samples[(s0 + r) * rec_len + c.first_col + col] = y[k];
            }
            ++col;
            if (col == n) {
                col = 0;
                ++r;
            }
        }
        if (!together) continue;
        if (e + 4u <= total) {
            *reinterpret_cast<Int4*>(to) = Int4{y[0], y[1], y[2], y[3]};
        } else {
            to[0] = y[0];
            if (e + 1u < total) to[1] = y[1];
            if (e + 2u < total) to[2] = y[2];
        }
    }
}

__global__ __launch_bounds__(256) void pack_wide_kernel(const int32_t* __restrict__ src, int64_t n,
                                                        FastDiv div_w, int64_t rec_len, int32_t first_col,
                                                        int32_t* __restrict__ samples) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= n) return;
    const uint32_t s = fastdiv((uint32_t)e, div_w);
    const uint32_t j = (uint32_t)e - s * div_w.d;
    samples[(int64_t)s * rec_len + first_col + j] = src[e];
}

// Measurement only: n_runs runs of run_len ints, one lane per int, run r at run position
// mix(r) (a bijection of [0, n_runs) for a power of two: odd multiplications and xor-shifts) or at r.
__device__ __forceinline__ uint32_t probe_mix(uint32_t x, uint32_t mask, int half) {
    x = (x * 0x9E3779B1u) & mask;
    x ^= x >> half;
    x = (x * 0x85EBCA6Bu) & mask;
    x ^= x >> half;
    x = (x * 0xC2B2AE35u) & mask;
    x ^= x >> half;
    return x;
}

__global__ __launch_bounds__(256) void probe_store_runs_kernel(int32_t* __restrict__ out, uint32_t n_runs,
                                                               FastDiv div_len, int scattered, int half) {
    // a 256-lane round covers 256 / run_len whole runs; a lane keeps its place j inside the run
    const uint32_t len = div_len.d;
    const uint32_t r_local = fastdiv(threadIdx.x, div_len), j = threadIdx.x - r_local * len;
    const uint32_t per_round = 256u / len;
    if (r_local >= per_round) return;
    for (uint64_t r = (uint64_t)blockIdx.x * per_round + r_local; r < n_runs; r += (uint64_t)gridDim.x * per_round) {
        const uint32_t dst = scattered ? probe_mix((uint32_t)r, n_runs - 1u, half) : (uint32_t)r;
        out[(uint64_t)dst * len + j] = (int32_t)r;
    }
}

}  // namespace

int probe_store_runs(int32_t* out, int64_t n_runs, int32_t run_len, int scattered, hipStream_t stream) {
    if (n_runs == 0) return ND_OK;
    int bits = 0;
    while ((1ll << bits) < n_runs) ++bits;
    hipLaunchKernelGGL(probe_store_runs_kernel, dim3(2048), dim3(256), 0, stream, out, (uint32_t)n_runs,
                       make_fastdiv((uint32_t)run_len), scattered, bits / 2 + 1);
    ND_HIP_CHECK(hipGetLastError());
    return ND_OK;
}

int pack_samples(const int32_t* const* step_out, int32_t num_steps, const int64_t* step_len, int64_t S,
                 int32_t* samples, hipStream_t stream) {
    if (S == 0) return ND_OK;
    int64_t rec_len = 0;
    for (int32_t i = 0; i < num_steps; ++i) rec_len += step_len[i] / S;
    int64_t col = 0;
    int32_t i = 0;
    while (i < num_steps) {
        const int64_t w = step_len[i] / S;
        if (w == 1) {
            WalkChunk c{};
            c.first_col = (int32_t)col;
            while (i < num_steps && step_len[i] / S == 1 && c.n_steps < kTileSteps) {
                c.step[c.n_steps++] = step_out[i];
                ++i;
            }
            col += c.n_steps;
            c.div_steps = make_fastdiv((uint32_t)c.n_steps);
            const int per = S <= kFewSamples ? 32 : 64;
            const dim3 grid((unsigned)((S + per - 1) / per)), block(256);
            const size_t lds = (size_t)c.n_steps * (per + 1) * 4;  // at most 33 KB
            if (per == 32)
                hipLaunchKernelGGL(pack_walk_kernel<32>, grid, block, lds, stream, c, S, rec_len, samples);
            else
                hipLaunchKernelGGL(pack_walk_kernel<64>, grid, block, lds, stream, c, S, rec_len, samples);
        } else {
            const int64_t n = step_len[i];
            const int64_t blocks = (n + 255) / 256;
            hipLaunchKernelGGL(pack_wide_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, step_out[i], n,
                               make_fastdiv((uint32_t)w), rec_len, (int32_t)col, samples);
            col += w;
            ++i;
        }
    }
    ND_HIP_CHECK(hipGetLastError());
    return ND_OK;
}

}  // namespace nd
