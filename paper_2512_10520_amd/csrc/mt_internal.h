// Private structures shared by the host API (mt_api.hip) and the kernels
// (mt_kernels.hip).  Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mt.h"

namespace mt {

constexpr int kWave = 64;
constexpr int kLdsBytes = 160 * 1024;      // LDS of a CU
constexpr int kCkptEvery = 16;             // RK4 state checkpoint interval
constexpr double kKappa = 0.299792458;     // GeV / (c T m)
constexpr int kBlockRec = 20;              // doubles per convex block record
constexpr int kGridCells = 1024;           // cells of the block grid (LDS-resident)

// Histogram tables on the device.  cdf[h][c] is the inclusive cumulative
// count of cell c of histogram h = material * n_pbin + bin; guide[h][g]
// brackets the answer of the inverse-CDF search for every word whose top
// gbits bits equal g: x = first candidate cell lo (low 16 bits) and last
// candidate hi (high 16 bits), y = cdf[h][lo], so that any bucket spanning
// at most two cells resolves without a probe of cdf.
struct DevHist {
    const uint32_t *cdf;
    const uint2 *guide;          // [h][2^gbits]
    const uint2 *alias;          // [h][c] alias method: (24-bit threshold split, alias cell)
    int32_t n_mat, n_pbin, n_loss, n_scat, n_cells, gbits;
    float nscat_f, nscat_inv;    // n_scat, 1 / n_scat
    float loss_lo, loss_w, scat_lo, scat_w;   // log10 units on a logarithmic axis
    int32_t log_loss, log_scat;  // axis binned uniformly in log10 of the value
};

// Band of a momentum bin: the floats f for which float(|p|^2) = f proves that
// |p|^2 lies in the bin (and, once a run has raised it, above its momentum
// threshold).  Rounding to float is monotone, so f > float(a) gives |p|^2 > a
// and f < float(b) gives |p|^2 < b; a lane whose f is on a rounded bound itself
// decides in FP64.  Positive floats order as their bit patterns: a band is
// (first pattern, number of patterns), and one subtraction and one unsigned
// compare replace three FP64 compares.  Values below kBandLow, infinities and
// NaN lie outside every band.  The band after the last histogram's is that of
// a step outside every material.
constexpr float kBandLow = 1e-30f;

// Region of a box (x and y) and of a slab (z): centre and 1 / half width, the
// half widths shrunk by more than a lane's FP32 tracking can be off (see the
// kernels' struct Lane).  An axis without a usable region has a centre so far
// away that no position is inside.
struct BoxRegion {
    double xc, yc;
    float ix, iy;
};

struct SlabRegion {
    double zc;
    float iz, pad;
};

// A convex block in FP32 about the centre of its bounding box, for points that
// are clear of its faces.  S_i formed in FP32 is off by less than err: a point
// with sigma S_i < -err for some i is outside; one with the slack of edge i =
// sigma S_i - tau > 0 for every i (tau >= err) is inside the block and in none
// of lower index (see mt_load_blocks), and stays so while it moves by at most
// cxl_i slack_i to the left, cxh_i slack_i to the right, cyl_i, cyh_i down and
// up, and cz_i slack_i in z, for every i.
struct BlockRegion {
    double xc, yc;               // centre; vertices below are relative to it
    float bx[4], by[4];          // at z_lo
    float dx[4], dy[4];          // change from z_lo to z_hi
    float cxl[4], cxh[4], cyl[4], cyh[4], cz[4];
    float sigma;                 // vertex order +-1
    float err, tau;              // tau = infinity: the block has no clear points
    float ext;                   // largest lateral extent: |x - xc|, |y - yc| must be below it
    float xlo, xhi, ylo, yhi;    // lateral bounding box, rounded outwards
};

// The sides of a block as planes about its centre (xc, yc, zc): a position
// (x, y, z) relative to it with f_i = side[i].x x + side[i].y y + side[i].z z +
// side[i].w > 0 for every i and |z| < hz is clear of the block's faces, as
// classify_block's clear points are; one with f_i < -2 err for some i is
// outside.  A block whose sides are not plane (end quads with edges that are
// not parallel), one that is not clear of those before it and one that reaches
// out of the world have none (hz = -1).  One more record, the unit box, serves
// positions tracked in a region (see the kernels' Lane).
struct BlockPlanes {
    float4 side[4];
    float hz, err, pad[2];
    double xc, yc, zc, pad1;
};

// Geometry (its tables are in the staged image): boxes split into z-slabs.  Slab s covers [slab_z[s], slab_z[s+1])
// with slab_z[0] = -inf and slab_z[n_slab] = +inf; slab_mask[s] has bit b set
// when box b spans the whole slab in z, so inside the slab only the x and y
// ranges of those boxes need testing, lowest index first.
struct DevGeom {
    int32_t n_box, n_slab, n_mag;    // n_box: volumes (boxes or blocks)
    int32_t n_poly;              // > 0: the volumes are convex blocks
    int32_t gx, gy, gz;
    double g0[3], g1[3], ginv[3];   // grid origin, end and cells per metre
    int32_t vertical;            // every volume's field has bx = bz = 0
    int32_t disjoint;            // no two boxes overlap: a box that holds a point is its box
    double x_max, y_max, z_max;
};

struct DevField {
    const float4 *map;           // cell-major [nz-1][ny-1][nx-1][8] (bx, by, bz, 0): the cell's
                                 // trilinear interpolant as coefficients of 1, fx, fy, fz, fx fy,
                                 // fx fz, fy fz, fx fy fz; nullptr = no map
    const float4 *nodes;         // node-major [nz][ny][nx] (bx, by, bz, 0), for the nearest node
    int32_t vertical;            // every node has bx = bz = 0; then also:
    const float4 *mapv;          // cell-major [..][2]: the 8 coefficients of by
    const float *nodesv;         // node-major by
    int32_t nx, ny, nz;
    double lo[3];
    double inv_d[3];             // (n - 1) / (hi - lo)
    double umax[3];              // n - 1: the largest grid coordinate inside the map
    double off[3];               // -lo (n - 1) / (hi - lo): u = x inv_d + off
};

// Byte offsets of the tables every block stages in LDS: squared momentum
// edges, the bands and totals of the histograms, and the geometry; in the wide
// layout (AllTables) the ends of the momentum bins' bands (at off_band), the totals
// and the geometry.
struct LdsLayout {
    int32_t off_e2, off_band, off_tot, off_box4, off_mat, off_bf, off_mag, off_slabz, off_slabm, off_breg, off_sreg;
    int32_t off_blk, off_grid, off_preg, off_planes;
    int32_t bytes;
};

struct DevRun {
    double h;                    // step length
    int32_t sampler;             // MT_SAMPLER_*
    int32_t interp;              // MT_INTERP_*
    int32_t stage_field;         // 0: field held from the step start, 1: at every RK4 stage
    int32_t share_shift;         // variant-wave form: log2 of the lanes sharing a random stream
    int32_t room;                // few waves in the launch (see kRoom)
    int32_t ahead;               // variant-wave form: form the next step's draw ahead
    int32_t solo;                // variant-wave form: one of those lanes carries a muon
    int32_t wide;                // the kernels for large tables run (see AllTables)
    double pmin2;
    int32_t max_steps;
    uint32_t key0, key1;
    int64_t n;                   // input muons
    int64_t lanes;               // n_variants * n
    const float *scales;         // [n_variants][n_mag] or nullptr
    double *ckpt;                // [n_ckpt][6][lanes] or nullptr
    float *tape;                 // [max_steps][lanes][3] or nullptr
    int32_t *trace;
    int64_t n_trace;
    int32_t trace_steps;
};

struct DevIO {
    const double *x, *y, *z, *px, *py, *pz;
    const int8_t *q;
    double *ox, *oy, *oz, *opx, *opy, *opz;
    int32_t *status, *n_steps, *volume;
};

struct Tables {
    const uint4 *image;          // the staged tables as one block of lds.bytes (a multiple of 16),
                                 // followed by the block records that are not staged
    DevHist hist;
    DevGeom geom;
    DevField field;
    LdsLayout lds;
};

// Host side: the tables with both layouts of their image.
//
// Every block of a launch stages its own copy, so a large copy takes waves off a
// CU (160 KB of LDS).  And with narrow momentum bins a step takes muons over several
// of them, past the next lower one that the common step looks at.  The wide kernels,
// for such tables, stage one band end of 4 bytes per momentum bin instead of a band
// of 8 per histogram, keep the edges in memory and walk down the bins; they have the
// general field only.  10^6 muons through 40 boxes: 4 materials of 1024 bins 12.75 ->
// 5.03 ms, 3 of 600 6.89 -> 4.83, 43 of 95 7.77 -> 4.57; but 3 of 95 bins 3.84 -> 4.55.
struct AllTables : Tables {
    int32_t narrow;              // many draws cross more than one momentum bin
    LdsLayout wide_lds;
    const uint4 *wide_image;
};

// One pass of the compacting form: the items (the launch's lanes, or the
// output slots listed by the previous pass) step from k_begin up to the
// DevRun::max_steps of the launch;
// every muon is stored in its output slot, and the slots of those still
// running there are appended to `out` for the next pass.
struct PassArgs {
    int32_t k_begin;             // first step of the pass (its last is DevRun::max_steps)
    int32_t max_steps;           // the real step cap
    const unsigned long long *n_in;   // slots listed by the previous pass, or nullptr: all lanes
    const int64_t *in;           // [*n_in] output slots to resume
    unsigned long long *n_out;   // slots appended by this pass (zeroed beforehand)
    int64_t *out;                // [lanes] at most
};

// The one argument of every transport kernel (the pass fields are used by the
// compacting form only).
struct KArgs {
    Tables T;
    DevRun R;
    DevIO io;
    PassArgs P;
    uint32_t pbin_magic;         // floor((2^32 - 1) / n_pbin): h / n_pbin = umulhi(h + 1, it),
                                 // exact for h < 2^16
};

// Launchers implemented in mt_kernels.hip.
hipError_t launch_plain(const AllTables &T, const DevRun &R, const DevIO &io, int block,
                        hipStream_t s);
// One pass of the compacting form (see PassArgs).
hipError_t launch_pass(const AllTables &T, const DevRun &R, const DevIO &io, int block,
                       const PassArgs &P, hipStream_t s);
// Variant-wave form: groups of 2^R.share_shift lanes hold variants of one muon.
hipError_t launch_variant_waves(const AllTables &T, const DevRun &R, const DevIO &io, int block,
                               hipStream_t s);
// Field map tables (device pointers; nodesv and mapv may be nullptr): the node
// tables of n node values, and from them the cells'.
hipError_t launch_map_nodes(const float *b, int64_t n, float4 *nodes, float *nodesv,
                            hipStream_t s);
hipError_t launch_map_cells(const float4 *nodes, int nx, int ny, int nz, float4 *map, float4 *mapv,
                            hipStream_t s);
hipError_t launch_queue_reset(unsigned long long *queue, double *zero, int64_t n_zero,
                              hipStream_t s);
hipError_t launch_adjoint(const AllTables &T, const DevRun &R, const DevIO &io,
                          const double *g_out, double *g_in, double *gs_lane, void *scratch,
                          int block, bool lds_history, hipStream_t s);
// Deterministic per-variant sums.  tally: (zmax count, hit count, sigmoid sum);
// column sums: out[v][c] = sum over lanes of variant v of vals[c][lane].
hipError_t launch_tally(const DevIO &io, int64_t n, int32_t n_variants, double z_det,
                        double r_ap, double r_scale, double *partial, int32_t n_part_blocks,
                        double *out, hipStream_t s);
hipError_t launch_column_sums(const double *vals, int32_t n_cols, int64_t n, int32_t n_variants,
                              double *partial, int32_t n_part_blocks, double *out, hipStream_t s);
int64_t adjoint_scratch_bytes(const Tables &T, int64_t lanes);

}  // namespace mt
