// Batched-lane engine: argument blocks, workspace layouts and launchers
// shared by gx_batch.hip and the serving scheduler.
#pragma once

#include "gx_device.h"
#include "gx_internal.h"
#include "gx_limits.h"

namespace gx {

constexpr int BS_MIN_TILE = 1024;  // smallest SSSP work tile among the variants
constexpr int BP_TILE = 256;       // tile the PPR tunings name (the graph fixes the tiles)

// Counters of four consecutive supersteps, slot k & 3; superstep k clears the
// next one's.
struct BsCtl {
    unsigned long long list[4];     // (entries << 32) | units
    unsigned long long changed[4];  // (vertex, lane) activations
    uint32_t steps;                 // supersteps up to and including the first that changed nothing (0: none yet)
    uint32_t pad[3];
    uint32_t inv_low[4][256];       // pull: ~(smallest active distance) of every lane, 0: none active
};

struct BsArgs {
    const int32_t *rp;
    const uint2 *adj;
    // pull (in_adj NULL: push only)
    const uint2 *in_adj;
    const uint4 *segs, *packs;
    const int32_t *slot;
    int64_t nsegs, npacks;
    uint32_t pull_units;  // a superstep with at least this many units pulls
    int64_t V;
    uint32_t B, l0, G;  // lane stride, first lane of the pass, 32-lane groups in the pass
    uint32_t *D;
    uint32_t *M[2];
    uint4 *list;
    uint4 *S;           // every row's distances at the superstep's start, by slot
    uint32_t *tile_start;
    BsCtl *ctl;
    uint32_t *lane_cnt;   // optional [supersteps x B], 0 before: nonzero where a lane changed in a superstep
};

struct BsWork {
    uint32_t *M[2];
    uint4 *list;
    uint4 *S;
    uint32_t *tile_start;
    BsCtl *ctl;
    int32_t *src;
};

struct BsVariant {
    uint32_t block, vt;
    const void *fn;  // k_bs_relax of that shape
};

struct BpArgs {
    const int32_t *src;  // slot of every in-edge's source
    const int2 *nz;
    const int32_t *nz_slot, *slot;
    const uint64_t *row_last;
    const int32_t *tile_nz;
    const int4 *cross;
    const int32_t *dang;
    const int32_t *in_rp, *outdeg;
    int64_t n_nz, ntiles, E, n_dang;
    int32_t tile, dtile, ndtiles, n_cross, n_cross_long, n_cross_wide;
    uint32_t B;   // lane stride of the tiles
    uint32_t Bw;  // lanes processed (0..Bw-1); the rest keep their values untouched
    float d;
    const int32_t *seed;  // per lane; -1 = free lane
    const int32_t *end;   // per lane: first superstep it no longer runs (NULL: every lane's is `last`)
    uint32_t last;
    float *x;             // ranks, written in a lane's last superstep
    float *c[2];          // contributions x / out-degree (x itself where that is 0) by slot, c[k & 1] read by superstep k
    double *head, *tailp, *dpart, *seed_acc;
};

struct BpWork {
    float *c[2];
    double *head, *tailp, *dpart, *seed_acc;
    int32_t *seed, *end;
};

const BsVariant *bs_variants(int *n);
BsArgs bs_args_for(const DevGraph &d, const BsWork &w, uint32_t *D, uint32_t B, uint32_t l0, uint32_t G);
void bs_layout(const DevGraph &d, uint32_t B, Carver &c, BsWork *w);
void bp_layout(const DevGraph &d, uint32_t B, Carver &c, BpWork *w);
gx_tune default_tune(uint32_t B);

// Superstep k (lane_cnt row `it`); grid: workgroups of the push, 0 = as many as are resident.
hipError_t bs_launch_superstep(const BsArgs &a, uint32_t k, uint32_t it, const BsVariant &v, int grid, int cus,
                               hipStream_t s);
hipError_t bp_launch_superstep(const BpArgs &a, uint32_t k, int grid, hipStream_t s);
// Lane `lane` restarts from `src` at superstep k.
hipError_t bs_lane_reset(const BsArgs &a, uint32_t k, uint32_t lane, int32_t src, hipStream_t s);
BpArgs bp_args_for(const DevGraph &d, const BpWork &w, float *x, uint32_t B, float damping);
// Lane `lane` restarts from `seed` at superstep k; `old`: its previous seed (-1: none).
hipError_t bp_lane_reset(const BpArgs &a, uint32_t k, int64_t V, uint32_t lane, int32_t seed, int32_t old, hipStream_t s);
hipError_t lane_extract(const uint32_t *tile, int64_t V, uint32_t B, uint32_t lane, uint32_t *out, hipStream_t s);

}  // namespace gx
