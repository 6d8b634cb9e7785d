// Grouped launches over the snapshots (and pairs) of a sequence: one launch
// of a kernel family covers the tiles of every snapshot, found through a
// prefix table of per-snapshot workgroup counts; snapshots whose solve has
// converged (a device-side flag) skip their workgroups.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cdl {

// Everything the grouped chain and solve kernels need of one snapshot.
struct BatchSnap {
    int64_t n, ld;
    const double *W, *deg;
    char *levels;              // chain levels (level l at levels + l * level_bytes)
    int64_t level_bytes;
    const double *dm;          // chain's (cD)^{-1/2}
    double *fro;               // squaring's per-tile norm partials
    float inv_scale;           // 1 / storage scale of the levels
    double *Yt, *Xt, *Rt, *V64;
    void *Vlo[2];              // rounded operand ping-pong
    float *Pap;                // split-K partials of the application
    double *Pres;              // split-K partials of the residual product
    double *npart, *mpart, *scal;
    int ap_splits, res_splits;
};

struct SelectState;

// Everything the grouped graph build (padding, distance Gram, median
// selection, weights, degrees, statistics) and the level-0 chain of one
// snapshot need.
struct GraphSnap {
    const double *X;           // series, n x T, row pitch ldx
    int64_t n, T, ldx, Tp, ld;
    double *Xp, *sqn;          // padded series (ld x Tp) and squared row norms
    int *flags;                // non-finite input flag
    double *W, *deg, *stats;   // distances, then weights in place; degrees; statistics
    SelectState *sel;
    unsigned long long *buf;   // bracket buffer of the selection
    int64_t cap;               // its capacity (keys)
    int bracket;               // the selection starts with a sampled bracket
    double *dpart;             // degree partials
    // level 0 of the chain
    double *dmn, *dm, *u;
    void *level0;
    double *fro, *fro64;
    double scale;              // storage scale of the level
};

// Prefix tables of the grouped graph build (one per workgroup count):
enum GraphTable {
    kGtRows,      // padded rows, four per workgroup: ld / 4
    kGtOne,       // one workgroup per snapshot
    kGtGram,      // upper-triangle tiles of the group's shape
    kGtSample,    // 64 per snapshot whose selection starts with a sampled bracket (keys, ranks)
    kGtPass,      // workgroups of a selection's pass over the snapshot
    kGtSym,       // upper 64 x 64 tiles
    kGtNodes64,   // ceil(n / 64)
    kGtPrep,      // ceil(ld / 256)
    kGraphTables
};
// Workgroup counts of table `tb` for a snapshot (bracket: its selection
// starts with the sampled bracket).
int graph_table_count(int tb, int64_t n, int64_t ld, bool bracket, int gram_shape);
// Tile shape of the group's distance Gram.
int graph_gram_shape(int P, const int64_t *ld, const int64_t *T);
// Whether the stored selection of n keys' matrix starts with a sampled
// bracket (the bracket must fit the buffer).
bool select_uses_bracket(int64_t n, bool allowed);

// The graph of every snapshot: padding, Gram (with the key bounds when
// selecting), the exact lower median (sigma <= 0) or the given sigma,
// weights, degrees and statistics.  tables: kGraphTables x (P + 1) prefix
// tables in device memory; totals: their last entries (host); nmax: the
// largest snapshot's nodes.
hipError_t launch_graph_grouped(const GraphSnap *snaps, const int *tables, const int *totals,
                                int P, int64_t nmax, double sigma, int gram_shape, hipStream_t s);
// Level 0 of every snapshot's chain: (cD)^{-1/2}, u and the normalised,
// deflated, rounded level with its norm partials.
hipError_t launch_chain_level0_grouped(int prec, const GraphSnap *snaps, const int *tables,
                                       const int *totals, int P, hipStream_t s);

// One pair of consecutive snapshots for the grouped score kernels.
struct BatchPair {
    int64_t m, mpad;
    const double *Z0, *Z1;
    const int32_t *map0, *map1;
    const double *stats0, *stats1;
    const double *W0, *W1;     // weighted mode only
    int64_t ld0, ld1;
    double *Zh, *sq, *part;
    double *F;
    int32_t *top;              // min(top_k, m) best nodes (NULL: not asked for)
    int shape;                 // tile shape of its score Gram
};

// Problem index of workgroup b: prefix[p] <= b < prefix[p + 1] (P problems).
__device__ inline int group_find(const int *prefix, int P, int b) {
    int p = 0;
    while (p + 1 < P && b >= prefix[p + 1]) ++p;
    return p;
}

// ---- host launchers (grouped kernels; every pointer table in device memory) --

// One squaring of level `level` into level + 1 for every snapshot; prefix over
// each snapshot's upper-tile count (square_tiles of `tile`).  Stream-ordered.
hipError_t launch_square_grouped(int prec, int tile, const BatchSnap *snaps, const int *prefix, int P,
                                 int total, int level, hipStream_t s);
// The chain application of one level for every unconverged snapshot: the
// split-K product (prefix over mt * nt * ap_splits) then the update of
// V64 / Vlo[out] / X (prefix over the reduction's workgroups, last level
// when `last`).
hipError_t launch_apply_grouped(int prec, int shape, const BatchSnap *snaps, const int *prefix_gemm,
                                int total_gemm, const int *prefix_red, int total_red, int P, int64_t k,
                                int64_t kpad, int level, int in, int accumulate, int last,
                                const int *done, hipStream_t s);
// Workgroups of one snapshot's share of the application's update (also the
// FP16 operand preparation's), at most `cap`; the kernels stride over them.
int apply_reduce_blocks(int64_t ld, int64_t kpad, int cap = 2048);
// Tile shape of the applications' products of P snapshots in one launch, a
// snapshot's workgroups in it, and its 256-node tiles, by which split counts go.
int apply_shape(int prec, int P, const int64_t *n, const int64_t *ld, const int *nsplit, int64_t k,
                int64_t kpad);
int apply_gemm_tiles(int shape, int64_t ld, int64_t k, int64_t kpad, int nsplit);
int apply_base_tiles(int64_t ld, int64_t kpad);
// Workgroups of a snapshot's residual product with tile shape `shape`.
int residual_gemm_tiles(int shape, int64_t ld, int64_t k, int64_t kpad, int S);
// Tile shape (returned) and per-snapshot split counts of the grouped residual
// product; cap: the most splits a snapshot's workspace holds; fixed: counts
// given by the caller (nullptr: chosen here).
int residual_group_plan(int P, const int64_t *n, const int64_t *ld, int64_t k, int64_t kpad,
                        const int *cap, const int *fixed, int *splits);
// Split-K count S clamped to what a snapshot of n nodes allows (a grouped
// launch picks one S for all snapshots from the tiles of the whole group).
int apply_splits_fixed(int prec, int64_t n, int S);
// R = Y - deg X + W X, V = dm R (rounded copy into Vlo[0]) and the norm
// partials, for every unconverged snapshot; skip_gemm: R = Y (initial).
hipError_t launch_residual_grouped(int prec, const BatchSnap *snaps, int shape, const int *prefix_gemm,
                                   int total_gemm, const int *prefix_red, int total_red, int P,
                                   int64_t kpad, int64_t k, int skip_gemm, const int *done,
                                   hipStream_t s);
// Column norms (and the FP16 operand scale) of every unconverged snapshot,
// then per snapshot: rel = max_r ||R_r|| / ||Y_r|| (ynorm: P x kpad), and
// done[p] = rel <= tol (tol > 0), iters[p] += 1 when it was not done before.
// init: ynorm = the norms (no convergence test).
hipError_t launch_norms_grouped(const BatchSnap *snaps, int P, int64_t kpad, int64_t k,
                                int scaled, double tol, int init, double *ynorm,
                                double *rel_out, int *done, int *iters, hipStream_t s);
// FP16 operand: V = scale * dm R and its rounded copy, unconverged snapshots.
hipError_t launch_prep_grouped(int prec, const BatchSnap *snaps, const int *prefix, int total,
                               int P, int64_t kpad, const int *done, hipStream_t s);
// Scores of every pair: signature embeddings, the FP64 Gram tiles over the upper
// triangles (kScoreShapes prefix tables, `pitch` entries apart, and totals: the
// pairs of each shape) and the row sums.
hipError_t launch_score_grouped(const BatchPair *pairs, const int *prefix_zhat,
                                int total_zhat, const int *prefix_score, int pitch,
                                const int *total_score, const int *prefix_red, int total_red, int P,
                                int64_t k, int weighted, hipStream_t s);
// The min(top_k, m[p]) best nodes of every pair (m: host copy), after the
// scores.
hipError_t launch_topk_grouped(const BatchPair *pairs, const int64_t *m, int P, int top_k,
                               hipStream_t s);

}  // namespace cdl
