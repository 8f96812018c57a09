// Assignment for the unprotected path: a scan on the 16-bit matrix instructions names each point's
// nearest centroid, further passes settle it exactly (see ftk_scan.hip).
#pragma once

#include "ftk_internal.h"

namespace ftk {

struct ScanPlan {
    bool ok;
    int form;           // layout of a block (ScanForm)
    bool stream;        // rows beyond 128 features: both operands streamed through LDS
    int nb;             // blocks of 16 features in the centroid image (and of the compiled variant)
    int tiles, tiles_pad;  // tiles of 32 centroids, and those the image holds (whole chunks)
    int tpc, nch;       // tiles per staged chunk, chunks
    int splits, cps;    // workgroups sharing a block of points, chunks each of them sweeps
    int ct;             // stream: centroid tiles per wave
    int64_t pblocks;    // blocks of 256 points
    int64_t batch;      // points of a launch: the rest of this is cut for those
    int64_t rec_reserve;  // records to reserve
    bool half;          // a scan on fp16 pieces is prepared too, and runs instead where a sample of the rows says so
    int half_nb, half_tiles;  // blocks and tiles of its image
    bool either;        // part of a problem that may take either form, so that neither must show in the distances
    bool resolve;       // listed points are settled by the scan's own third pass (else refine_kernel)
};

// what the scan leaves of a point: its best score and centroid, the second-best score
struct ScanRecord {
    float m1, m2;
    int32_t j1;
    int32_t unused;
};
// a point to resolve, and the score a centroid needs to be a candidate (not a number: every centroid is one)
struct ScanListed {
    int32_t point;
    float thr;
};

struct ScanBuffers {
    uint4 *image;       // [tiles_pad][nb][2][64] centroid pieces in fragment order
    float *start;       // [tiles_pad][32] accumulator start values -||c||^2/2 - r.c (c less the reference r, scaled), raised, fragment order
    float *norm;        // [tiles_pad][32] ||c|| (scaled)
    float4 *tile_stat;  // [tiles_pad] largest ||c||^2 (scaled), ||c1||^2 / ||c||^2, ||r_c||^2 / ||c||^2 of a tile
    double *scale;      // [2] the power of two both operands are multiplied by; length of the (scaled) reference
    void *ref;          // [D] the reference, zero where none is taken
    float4 *sample;     // [tiles][rows] scores of the rows that choose the form
    ScanRecord *rec;    // [splits][N]
    ScanListed *list;   // points to resolve: lists of equal capacity ...
    int32_t *list_count;  // ... and a counter each (then the counters of `rest`, and which form was chosen)
    int32_t *tickets;   // [N/32 + 1] workgroups done with a group of listed points
    uint4 *half_image;  // [half_tiles][half_nb][64] fp16 pieces, and the start values that go with them
    float *half_start;
    ScanListed *rest;   // listed points that go on from the fp16 scan's own third pass
    size_t bytes;
};

// the rule: which problems take this path, and how they are cut up
ScanPlan plan_scan(ftk_dtype dtype, int64_t N, int D, int K);
// the cut alone, for part of a problem that takes this path
ScanPlan cut_scan(ftk_dtype dtype, int64_t N, int D, int K);
// the same for n points of a problem that is cut as `whole`
ScanPlan cut_part(const ScanPlan &whole, ftk_dtype dtype, int64_t n, int D, int K);
// rows that the preparation writes for the points or for any batch of them, and those its images are reserved for
void scan_padded_rows(ftk_dtype dtype, int64_t N, int D, int K, int64_t *planned, int64_t *reserved);
// buffers for the whole problem and for any batch of it
ScanBuffers carve_scan(void *base, const ScanPlan &whole, int64_t N, int D);
// whole: the problem that c is a part of, whose rows choose the form
ftk_status launch_scan_assign(const AssignCall &c, const ScanPlan &p, const ScanBuffers &b, const Workspace &w,
                              const AssignCall &whole, hipStream_t st);

}  // namespace ftk
