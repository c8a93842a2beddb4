// Per-property networks with their constant neurons folded away.
//
// Inside one property's domain most hidden neurons cannot change: their
// potential stays below zero or above the requantiser's window whatever the
// (at most k) perturbed pixels do.  Interval bounds over the domain find the
// neurons that can change (the live ones); the constant ones go into the next
// layer's bias, and the enumeration runs a smaller network per property whose
// logits are the original ones, point by point.
#pragma once

#include "kernels_q8.h"

namespace ibmc {

constexpr int kFoldWidths[] = {32, 48, 64, 96, 128, 256};   // compiled first-layer widths (live units, padded)
__host__ __device__ constexpr int fold_blocks(int kw) { return kw <= 64 ? 1 : kw <= 128 ? 2 : 4; }
__host__ __device__ constexpr int fold_units_per_block(int kw) { return kw / (4 * fold_blocks(kw)); }
constexpr int kFoldMaxWidth = 256;
constexpr int kFoldGroup = 8;                       // segments per group at most
constexpr int kFoldMaxLevels = 4096;                // levels of all folded properties of a call at most
constexpr const char *kFoldVariantName = "fold";    // forces folding whatever the workload's size
constexpr int kFoldMaxStage = 96 * 1024;            // bytes of staged weights per workgroup at most

// What the scan reads per property.
struct FoldProp {
    int32_t pid;           // property (index into PropDev, u0_store)
    int32_t net;           // index into the call's network table
    int32_t k;             // largest level checked
    int32_t dlo, dhi;      // smallest and largest delta, widened to contain 0
    int32_t joint;         // layers 1 and 2 hold no weight of -128 (the joint bound's absolute values fit int8)
    int32_t *ws;           // see FoldWs
    int32_t *counts;       // [4]: live units of layer 1; of layer 2 | uncapped pairs of tiles << 16; whether output
                           // differences need two bytes (1) or don't fit two (2); clean label
};

// Layout of a property's scan results (words).
struct FoldWs {
    int ub, lb, iv1, list1, iv2, list2, b2, rs2, bo, rso, done, total;
};
__host__ __device__ inline FoldWs fold_ws(int H1, int H2) {
    FoldWs w;
    w.ub = 0;                      // [H1] largest single-pixel increase of the potential, sigma order
    w.lb = w.ub + H1;              // [H1] smallest (<= 0)
    w.iv1 = w.lb + H1;             // [H1] activations lowest | highest << 8 | clean << 16, natural order
    w.list1 = w.iv1 + H1;          // live units of layer 1 as sigma positions
    w.iv2 = w.list1 + H1;          // [H2] activations lowest | highest << 8 | form << 16 of layer 2
    w.list2 = w.iv2 + H2;          // live units of layer 2 (natural index), in the order of their forms
    w.b2 = w.list2 + H2;           // [H2] layer-2 bias plus the constant units' contribution
    w.rs2 = w.b2 + H2;             // [H2] sum of the row's weights over the live units
    w.bo = w.rs2 + H2;             // [16] output bias plus the constant units' contribution
    w.rso = w.bo + 16;             // [16] sum of the row's weights over the live units times their offsets
    w.done = w.rso + 16;           // row groups of layer 2 finished
    w.total = w.done + 1;
    return w;
}

// Forms of a live layer-2 unit under the saturating epilogue (see
// enum_fold_impl.h): never below 0; never above 127; both ends in reach.
enum FoldForm : int { FOLD_UPPER = 0, FOLD_LOWER = 1, FOLD_BOTH = 2 };

// A folded property as the enumeration reads it.
struct FoldRun {
    const int16_t *W1;     // [n][KW] f * W1 of the live units, f = 2^(8 - shift - halvings)
    const int32_t *v0;     // [KW] f * u0 - 2^(14 - halvings)
    const int16_t *etab;   // [n * m] effective deltas clamp(x + d) - x, candidate order
    const int8_t *stage;   // weights and inits of the later layers, staged in LDS as they are:
                           // [W2 tiles][layer-2 init][output tiles][their second bytes][output init]
    int32_t stage_bytes;
    int32_t npair;         // pairs of 16-row tiles of layer 2
    int32_t free_pairs;    // of them, the leading ones that need no cap (saturating epilogue)
    int32_t two;           // output differences need a second byte
    int32_t s2;            // requantiser shift of layer 2 (general epilogue; inputs are doubled)
    int32_t halvings;      // see W1
    int32_t vlo, vhi;      // clamp of the segment base
    int32_t label, nc;
};

// What the gather builds a FoldRun from.
struct FoldBuild {
    int32_t pid, net, kw, live1, live2;
    int32_t epi, f;
    const int32_t *ws;
    FoldRun run;
};

struct FoldParams {
    const EnumJob *jobs;               // chunk ranges start at multiples of 4 * batch
    int32_t n_jobs;
    int32_t batch;                     // chunks of one wave per ticket
    int64_t total_chunks;
    const PropDev *props;
    const FoldRun *runs;               // by property
    int32_t stage_max;                 // largest stage_bytes of the launch's properties
    int32_t pad_;
    unsigned long long *queue;
    unsigned long long *rec_count;
    int64_t rec_cap;
    DevRec *recs;
    unsigned long long *slot_cex;
    unsigned long long *slot_ties;
    volatile int32_t *abort_host;
};

struct FoldVariant {
    int L, kw, wide, epi, nt, wave_bytes;
    const void *fn;
};
const FoldVariant *fold_variants(int *count);
const FoldVariant *fold_variants_l2a(int *count);
const FoldVariant *fold_variants_l2b(int *count);
const FoldVariant *fold_variants_l2c(int *count);
const FoldVariant *fold_variants_l3fa(int *count);
const FoldVariant *fold_variants_l3fb(int *count);
const FoldVariant *fold_variants_l3fc(int *count);
const FoldVariant *fold_variants_l3ga(int *count);
const FoldVariant *fold_variants_l3gb(int *count);
const FoldVariant *fold_variants_l3gc(int *count);

// Bytes of LDS of a launch whose largest staged block is stage_max.
int64_t fold_lds_bytes(const FoldVariant &v, int stage_max);
// Bytes of the staged block, and of the whole gathered property.
int fold_stage_bytes(int L, int kw, int npair, int two);

// First-layer potentials, clean label, live units and folded biases of the
// listed properties (block_map: property index << 8 | 64-unit slice), then
// those of the second hidden layer (row_map: property index << 8 | group of
// 64 rows, three-layer nets only).
hipError_t launch_fold_bound(const QNetDev *nets, const FoldProp *fps, const PropDev *props, const int32_t *row_map,
                             int n_blocks, hipStream_t s);
hipError_t launch_fold_scan(const QNetDev *nets, const FoldProp *fps, PropDev *props, const int32_t *block_map,
                            int n_blocks, int32_t *u0_store, int64_t u0_stride, hipStream_t s);
// The reduced networks of n builds; runs[pid] receives each build's run.
hipError_t launch_fold_gather(const QNetDev *nets, const FoldBuild *builds, int n, int parts, const PropDev *props,
                              const int32_t *u0_store, int64_t u0_stride, FoldRun *runs, hipStream_t s);
hipError_t launch_enum_fold(const FoldVariant &v, int grid, const FoldParams &P, hipStream_t s);

}  // namespace ibmc
