// Arguments of the sampling kernels and their host-side launchers.
#pragma once

#include "nd_common.h"

namespace nd {

enum : int { kDrawUniform = 0, kDrawWeighted = 1, kDrawNode2vec = 2 };

// Everything a lane needs to make the draws of one step; passed by value.
struct DrawArgs {
    uint64_t seed;
    uint64_t ppr_thr;             // walk ends when R3 < ppr_thr; 0 = never
    uint32_t sample_base;         // id of the call's first sample
    uint32_t step;
    uint32_t m;                   // draws per (transit, sample) pair
    FastDiv div_m;                // by m
    FastDiv div_wprev;            // by the number of transit slots per sample
    uint32_t b_ret, b_com, b_far, b_max;  // node2vec biases, Q16
    int32_t max_attempts;
    int32_t has_prev;             // node2vec: a previous transit exists (step > 0)
    int32_t use_weights;
    int32_t lds_policy;
    const int32_t* prev_transit;  // node2vec: previous transit of every sample
    int32_t* out;                 // this step's output array
    PackedCols packed;            // k-hop: what the sub-wavefront class and the fused kernel read, where it is there
};

// Device arrays and launch bounds of one transit-parallel step.
struct TpStep {
    StepCtl* ctl;
    const int32_t* keys;       // pairs sorted by transit: transit ...
    const int32_t* vals;       // ... and slot in the previous step's array
    const int32_t* g_key;      // distinct transits
    const int32_t* g_start;    // first pair of each transit's group (+ sentinel)
    const int32_t* list_wg;    // workgroup-class transits
    const int32_t* chunk_gid;  // grid-class chunks: transit ...
    const int32_t* chunk_idx;  // ... and chunk number
    uint32_t* heavy_bits;      // one bit per vertex: set for workgroup / grid class transits
    int64_t max_draws;         // host-known upper bounds that size the launches
    int64_t max_wg, max_chunks;
    int64_t cap_wg, cap_chunks;
};

int sample_step_tp(const Graph& gr, int draw, const DrawArgs& a, const SchedParams& sp,
                   const TpStep& t, hipStream_t stream);

int sample_step_sp(const Graph& gr, int draw, const DrawArgs& a, const int32_t* src, int64_t n_slots,
                   int check_roots, uint32_t* status, hipStream_t stream);

// Multi-dimensional walk (Section 3): the sample's root set lives in `state` (S * R vertices).
// init copies the roots (out-of-range ones become NULL and are reported), select writes the
// step's transit of every sample (the root picked with R2 of the step's generator call) and
// update puts the vertex the step added in the picked root's place.
int multirw_init(const Graph& gr, const int32_t* roots, int64_t n, int32_t* state, uint32_t* status,
                 hipStream_t stream);
int multirw_select(const int32_t* state, int64_t S, uint32_t R, uint64_t seed, uint32_t sample_base,
                   uint32_t step, int32_t* transits, hipStream_t stream);
int multirw_update(int32_t* state, int64_t S, uint32_t R, uint64_t seed, uint32_t sample_base,
                   uint32_t step, const int32_t* added, hipStream_t stream);

// Random walks grouped per window of samples (nd_walk.hip): all num_steps steps of DeepWalk, PPR,
// node2vec or the multi-dimensional walk, one launch per 128 steps.  d carries the draw's
// constants (seed, sample_base, PPR threshold, node2vec biases, LDS policy); window is 256, 1024 or
// 2048; heavy_min the number of pairs of one transit inside a window from which the whole
// workgroup serves it; ctl (may be null) receives per-step counters.
int walk_window_auto(int64_t S);
int walk_windows(const Graph& gr, int draw, bool multirw, const DrawArgs& d, int64_t S, int32_t num_steps,
                 int window, uint32_t heavy_min, int force_class, const int32_t* roots, int check_roots,
                 int32_t* const* step_out, uint32_t* status, StepCtl* ctl, int32_t* mrw_state, uint32_t R,
                 hipStream_t stream);

// Random walks over the graph's links (nd_walk_free.hip): DeepWalk, PPR, node2vec and (mrw_R > 0) the
// multi-dimensional walk, whose roots pass through mrw_state where the call takes several launches.  The
// call's header, one flag per workgroup (o_flags) and the live walks per workgroup and step (o_parts)
// go to the workspace.
bool mrw_reads_filled(const Graph& gr, int64_t S, int32_t num_steps, uint32_t R);
int64_t walk_free_groups(int64_t S, int32_t num_steps, bool node2vec, uint32_t mrw_R);
bool walk_uses_cells(const Graph& gr, int64_t S);  // DeepWalk and PPR over edge weights, where the cells are there
int64_t walk_free_state_bytes(int64_t S, int32_t num_steps, uint32_t mrw_R);
int walk_free(const Graph& gr, int draw, const DrawArgs& d, int64_t S, int32_t num_steps, const int32_t* roots,
              int32_t* const* step_out, char* ws, uint64_t o_flags, uint64_t o_parts, uint32_t mrw_R, int32_t* mrw_state,
              hipStream_t stream);

// All hops of a k-hop call in one launch (nd_khop.hip).  fits: the graph has links, the rows of a
// sample's widest hop with children fit LDS, and grouping by transit would not be faster; reads_packed: the call, grouped
// or not, is faster over the packed columns; groups: workgroups, hence flags and rows of live counts.
// status_out (may be null): receives the status word when the roots are few enough for one
// workgroup to look at (kKhopStatusRoots).
constexpr int64_t kKhopStatusRoots = 8192;
bool khop_fused_fits(const Graph& gr, const int32_t* fanout, int32_t k, int64_t S);
bool khop_reads_packed(const Graph& gr, const int32_t* fanout, int32_t k, int64_t S);
int64_t khop_fused_groups(const Graph& gr, const int32_t* fanout, int32_t k, int64_t S);
int khop_fused(const Graph& gr, const DrawArgs& d, const int32_t* fanout, int32_t k, int64_t S, const int32_t* roots,
               int32_t* const* step_out, char* ws, uint64_t o_flags, uint64_t o_parts, uint32_t* status_out,
               hipStream_t stream);

// The first hop without grouping, for calls whose later hops are grouped: at most a root per vertex (ctl, status: the
// step's live pairs and the call's bad roots are counted there).
int khop_first(const Graph& gr, const DrawArgs& d, int32_t m, int64_t S, const int32_t* roots, int32_t* out, StepCtl* ctl,
               uint32_t* status, hipStream_t stream);

// All hops with unique neighbours (Section 6.3), one group of lanes per sample.
bool khop_unique_fits(const Graph& gr, const int32_t* fanout, int32_t k);
int64_t khop_unique_groups(const Graph& gr, const int32_t* fanout, int32_t k, int64_t S);
int khop_unique(const Graph& gr, const DrawArgs& d, const int32_t* fanout, int32_t k, int32_t rounds, int64_t S,
                const int32_t* roots, int32_t* const* step_out, char* ws, uint64_t o_flags, uint64_t o_parts,
                hipStream_t stream);
// Once per device before the first call (nd_graph_create does it).
int khop_prepare();

// Unique neighbours (Section 6.3) for one k-hop step whose first draw round has already been
// written to `out`: per sample, duplicates are removed (the lowest slot keeps the vertex) and
// the slots that lost draw again, sample-parallel, for rounds - 1 further attempts.
struct UniqueArgs {
    uint64_t seed;
    uint32_t sample_base;
    uint32_t step;
    uint32_t W;               // slots per sample at this step (at most ND_MAX_UNIQUE_SLOTS)
    uint32_t W_prev;          // slots per sample of the previous step (1 at step 0)
    FastDiv div_m;            // slot j descends from slot j / m of the previous step
    int32_t rounds;
    const int32_t* parents;   // roots (step 0) or the previous step's output
    int32_t* out;
};
int unique_step(const Graph& gr, const UniqueArgs& a, int64_t num_samples, hipStream_t stream);

// Layer (collective) sampling: one step for all samples.
struct LayerArgs {
    uint64_t seed;
    uint32_t sample_base;
    uint32_t step;
    uint32_t n_prev;              // transit slots per sample at this step
    uint32_t m;                   // draws per sample
    const int32_t* transits;      // num_samples * n_prev (roots or the previous layer)
    int32_t* out;                 // num_samples * m
    int32_t check_roots;
    int32_t use_weights;          // entries weigh w_q(v,u) instead of c(v)
    uint32_t* status;
};
// All steps of a call in one launch (graphs with links): workgroups, for the flags, and the launch.
int64_t layer_fused_groups(const Graph& gr, int64_t S);
int layer_fused(const Graph& gr, uint64_t seed, uint32_t sample_base, bool weighted, int32_t roots_per_sample,
                const int32_t* fanout, int32_t k, int64_t S, const int32_t* roots, int32_t* const* step_out, char* ws,
                uint64_t o_flags, hipStream_t stream);
int layer_step(const Graph& gr, const LayerArgs& a, int64_t num_samples, hipStream_t stream);
// Once per device before the first layer_step (nd_graph_create does it): lifts the kernels' LDS limit.
int layer_prepare();

}  // namespace nd
