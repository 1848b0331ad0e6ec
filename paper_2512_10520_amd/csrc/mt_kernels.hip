// HIP kernels of the histogram-sampling muon transport for gfx950 (MI355X).
//
// One lane carries one muon through the transport loop of Algorithm 1
// (Section "Simulation").  Muon state (r, p) lives in FP64 registers for the
// whole trajectory; the per-step arithmetic (kick, rotation, RK4 stages) is
// FP32 and its increments are accumulated into the FP64 state.  Every
// discrete decision (break test, box, momentum bin) is an FP64 compare, and
// the histogram cell is drawn by an exact integer inverse CDF, so decisions
// agree with a double-precision reference except at stated boundary ties.
//
// Build with -ffp-contract=off: every fused multiply-add is written out as
// fmaf(), so the same source yields the same bits in every kernel that
// inlines it (plain, persistent and the adjoint's re-forward).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdlib.h>

#include <array>
#include <utility>

#include "mt_internal.h"

namespace mt {
namespace {

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds, each forming
// the 64-bit products of counter words 0 and 2 with the two multipliers,
// the high halves xored with words 1 and 3 and the round key, the key then
// advanced by the two Weyl increments.  The key is the same for every lane.
//
// The counter is (j mod 2^32, j / 2^32, step, 0) for muon j.  Everything in
// rounds 1 and 2 that does not depend on the step is the same for all steps
// of a muon, so it is formed once per muon (philox_prefix) and each step
// starts from it (philox_step): one product in each of the first two rounds
// instead of two.
// ---------------------------------------------------------------------------
constexpr uint32_t kMulA = 0xD2511F53u, kMulB = 0xCD9E8D57u;
constexpr uint32_t kWeylA = 0x9E3779B9u, kWeylB = 0xBB67AE85u;

struct PhiloxPrefix {
    uint32_t c1;   // round 1: j_hi ^ key0
    uint32_t c4;   // round 2: hi(kMulB * n2_1) ^ (key0 + kWeylA)
    uint32_t c5;   // round 2: lo(kMulB * n2_1)
    uint32_t c6;   // round 2: n3_1 ^ (key1 + kWeylB)
};

__device__ __forceinline__ PhiloxPrefix philox_prefix(uint32_t jlo, uint32_t jhi, uint32_t k0,
                                                      uint32_t k1) {
    const uint64_t pa1 = (uint64_t)kMulA * jlo;
    const uint32_t n2_1 = (uint32_t)(pa1 >> 32) ^ k1;   // round 1, word 2 (counter word 3 is 0)
    const uint32_t n3_1 = (uint32_t)pa1;
    const uint64_t pb2 = (uint64_t)kMulB * n2_1;
    PhiloxPrefix P;
    P.c1 = jhi ^ k0;
    P.c4 = (uint32_t)(pb2 >> 32) ^ (k0 + kWeylA);
    P.c5 = (uint32_t)pb2;
    P.c6 = n3_1 ^ (k1 + kWeylB);
    return P;
}

// a ^ b ^ c in one v_bitop3_b32 (truth table 0x96), a gfx950 instruction
// the compiler does not form from two xors by itself.
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ uint4 philox_step(const PhiloxPrefix &P, uint32_t step, uint32_t k0,
                                             uint32_t k1) {
    // The round keys k + r (Weyl increment) are formed here, by scalar adds,
    // at every call: hoisted out of a step loop they would be 16 more
    // long-lived scalar registers, which the step loops do not have (they
    // were spilled to vector-register lanes and read back with v_readlane,
    // a vector instruction, plus a wait, for every round of every step).
    __asm__ volatile("" : "+s"(k0), "+s"(k1));
    // round 1: only the product with the step word varies
    const uint64_t pb1 = (uint64_t)kMulB * step;
    const uint32_t n0_1 = (uint32_t)(pb1 >> 32) ^ P.c1;
    const uint32_t n1_1 = (uint32_t)pb1;
    // round 2
    const uint64_t pa2 = (uint64_t)kMulA * n0_1;
    uint32_t c0 = n1_1 ^ P.c4;
    uint32_t c1 = P.c5;
    uint32_t c2 = (uint32_t)(pa2 >> 32) ^ P.c6;
    uint32_t c3 = (uint32_t)pa2;
    k0 += 2u * kWeylA;
    k1 += 2u * kWeylB;
#pragma unroll
    for (int r = 2; r < 10; ++r) {
        const uint64_t pa = (uint64_t)kMulA * c0;
        const uint64_t pb = (uint64_t)kMulB * c2;
        const uint32_t n0 = xor3((uint32_t)(pb >> 32), c1, k0);
        const uint32_t n2 = xor3((uint32_t)(pa >> 32), c3, k1);
        c1 = (uint32_t)pb;
        c3 = (uint32_t)pa;
        c0 = n0;
        c2 = n2;
        k0 += kWeylA;
        k1 += kWeylB;
    }
    return make_uint4(c0, c1, c2, c3);
}

// ---------------------------------------------------------------------------
// Kernel arguments read where they are used.  A step loop that keeps every
// argument in scalar registers needs more than the 102 a wave has; the
// compiler then parks them in vector-register lanes and reads each back with a
// v_readlane (a vector instruction) on every step.  What only the cold paths
// of a step need is therefore loaded there, from the kernel's argument segment
// through a pointer the compiler cannot see through (cold): a scalar load of a
// few cached words.  The argument of every transport kernel is one KArgs.
// ---------------------------------------------------------------------------
using ArgPtr = const __attribute__((address_space(4))) KArgs *;

__device__ __forceinline__ ArgPtr kernel_args() {
    return (ArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
}

__device__ __forceinline__ ArgPtr cold(ArgPtr p) {
    __asm__ volatile("" : "+s"(p));
    return p;
}

// ---------------------------------------------------------------------------
// Tables staged in LDS by every block.
// ---------------------------------------------------------------------------
struct Lds {
    const double *e2;           // squared momentum edges (kWide: not staged)
    const uint2 *band;          // [n_hist + 1]: band of |p|^2 of every histogram, see kBandLow
    const uint32_t *edge;       // kWide, instead: [n_pbin + 1] ends of the momentum bins' bands
    const uint32_t *tot;
    const double *box4;
    const int32_t *mat;
    const float4 *bf;
    const int32_t *mag;
    const double *slabz;
    const uint64_t *slabm;
    const BoxRegion *breg;
    const SlabRegion *sreg;
    const double *blk;          // convex blocks [n_poly][kBlockRec], not staged
    const BlockRegion *preg;    // [n_poly], not staged
    const BlockPlanes *planes;
    const uint64_t *grid;       // block grid candidate masks
};

__device__ __forceinline__ char *lds_base() {
    extern __shared__ __align__(16) char smem[];
    return smem;
}

// The staged tables of a layout.
template <bool WIDE, class TT>
__device__ __forceinline__ Lds lds_view(const TT &T) {
    const auto &L = T.lds;
    char *smem = lds_base();
    const char *image = reinterpret_cast<const char *>(T.image);
    return Lds{reinterpret_cast<const double *>(WIDE ? image + L.off_e2 : smem + L.off_e2),
               reinterpret_cast<uint2 *>(smem + L.off_band),
               reinterpret_cast<uint32_t *>(smem + L.off_band),
               reinterpret_cast<uint32_t *>(smem + L.off_tot),
               reinterpret_cast<double *>(smem + L.off_box4),
               reinterpret_cast<int32_t *>(smem + L.off_mat),
               reinterpret_cast<float4 *>(smem + L.off_bf),
               reinterpret_cast<int32_t *>(smem + L.off_mag),
               reinterpret_cast<double *>(smem + L.off_slabz),
               reinterpret_cast<uint64_t *>(smem + L.off_slabm),
               reinterpret_cast<BoxRegion *>(smem + L.off_breg),
               reinterpret_cast<SlabRegion *>(smem + L.off_sreg),
               reinterpret_cast<const double *>(image + L.off_blk),
               reinterpret_cast<const BlockRegion *>(image + L.off_preg),
               reinterpret_cast<BlockPlanes *>(smem + L.off_planes),
               reinterpret_cast<uint64_t *>(smem + L.off_grid)};
}

// Copies the image of the tables (one coalesced 16-byte load per thread and
// trip, all in flight together) and raises the bands to the momentum threshold
// of the run.
template <bool WIDE>
__device__ __forceinline__ void stage_tables(const Tables &T, double pmin2) {
    uint4 *dst = reinterpret_cast<uint4 *>(lds_base());
    const int tid = threadIdx.x, nt = blockDim.x, n16 = T.lds.bytes / 16;
    for (int i = tid; i < n16; i += nt) dst[i] = T.image[i];
    __syncthreads();
    if constexpr (WIDE) {
        uint32_t *edge = reinterpret_cast<uint32_t *>(lds_base() + T.lds.off_band);
        const uint32_t threshold = __float_as_uint((float)pmin2);
        for (int i = tid; i < T.hist.n_pbin; i += nt) edge[i] = max(edge[i], threshold);
        __syncthreads();
        return;
    }
    uint2 *band = reinterpret_cast<uint2 *>(lds_base() + T.lds.off_band);
    const uint32_t above = __float_as_uint((float)pmin2) + 1u;
    for (int i = tid; i <= T.hist.n_mat * T.hist.n_pbin; i += nt) {
        const uint2 b = band[i];
        const uint32_t lo = max(b.x, above), hi = b.x + b.y;
        band[i] = make_uint2(lo, hi > lo ? hi - lo : 0u);
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Lane state.  Besides the muon, a lane keeps what rarely changes from one
// step to the next: the volume, its field, its histogram and the momentum
// band of the bin, and how far it may still travel before any of the FP64
// tests of the loop could come out differently:
//   xr, yr, zr  position relative to the centre of a box (the region), in
//               units of its half widths, ix, iy, iz being 1 / half width:
//               while max(|xr|, |yr|, |zr|) < 1 the position is inside the
//               same volume and the world.
// A step whose position is inside the region skips the volume lookup and the
// break test; otherwise it repeats them in FP64 (locate_region) and forms the
// region again, as every lane does at each step that is a multiple of
// kRegionSteps.  The region is smaller than the true one by more than xr, yr,
// zr can be off after that many FP32 sums, so a skipped test is one whose
// outcome is known: results do not change.  Why: a step is bound by VALU issue,
// an FP64 compare issues in 4.4 cycles against 2.4 of an FP32 operation, and the
// FP64 tests of every step were some 160 of its 950 (block, 10^6 muons, 1718 ->
// 1413 us; 2000, 381 -> 298 us; design scan 9.79 -> 8.87 ms).
//
// With convex blocks the box test is a test of four planes and |zr| (record
// rec in LDS): for a lane in a block with plane sides the block's, with xr, yr,
// zr in metres about the block's centre (ix = iy = iz = 1); for the others the
// unit box.
// ---------------------------------------------------------------------------
constexpr int kRegionSteps = 128;              // steps a region is used for at most
constexpr float kRegionHalf = 16.0f;           // its largest half width (m)
constexpr double kRegionCoord = 1048576.0;     // |x|, |y|, |z| (m) up to which regions are used

struct Lane {
    double x, y, z, px, py, pz;
    float kq;             // kappa q
    float xr, yr, zr, ix, iy, iz;
    uint32_t rec;         // LDS byte offset of the BlockPlanes record (convex blocks)
    uint32_t plo, pspan;  // band of float(|p|^2), see kBandLow
    uint32_t hoff;        // the histogram's row in the sampler's table (see row_of), or kVacuum
    uint32_t tot;         // the histogram's total (inverse CDF)
    float bx, by, bz;     // scaled field of the volume (times kq in kernels without a map)
    bool bent;            // that field is not zero
    int32_t steps, status, slab, vol;
    PhiloxPrefix ph;
    uint4 w;              // random words of the next step and the entry of the sampler's table
    uint2 e;              // they select in row eh (kVacuum: neither), see advance
    uint32_t eh;
    float ci, cj, ck;     // field-map cell (or node) whose values are in mc; NaN: none
    float mc[24];         // its coefficients (bx, by, bz) x 8 (or the node's value)
};

// y and p_y of a lane.  A field that is not finite makes a muon NaN; the vertical
// forms leave out the products that would carry the NaN to y, so it is taken
// from x and p_x there, where the value counts (outputs and checkpoints).
template <bool V>
__device__ __forceinline__ double lane_y(const Lane &L) {
    return V && L.x != L.x ? L.x : L.y;
}

template <bool V>
__device__ __forceinline__ double lane_py(const Lane &L) {
    return V && L.px != L.px ? L.px : L.py;
}

constexpr uint32_t kVacuum = 0xFFFFFFFFu;      // hoff outside every material

// LDS byte offset of the unit box, the BlockPlanes record behind the blocks'.
template <class TT>
__device__ __forceinline__ uint32_t unit_box(const TT &T) {
    return (uint32_t)T.lds.off_planes +
           (uint32_t)sizeof(BlockPlanes) * (uint32_t)T.geom.n_poly;
}

// A lane that knows nothing yet: outside its region, at whatever step it starts
// (position 2 on every axis is outside the boxes' region and the unit box).
template <class TT>
__device__ __forceinline__ void reset_lane_caches(Lane &L, const TT &T) {
    L.xr = L.yr = L.zr = 2.0f;
    L.ix = L.iy = L.iz = 0.0f;
    L.rec = unit_box(T);
    L.plo = L.pspan = 0u;
    L.hoff = kVacuum;
    L.eh = kVacuum;
    L.tot = 0u;
    L.slab = -1;
    L.vol = -2;
    L.bx = L.by = L.bz = 0.0f;
    L.bent = false;
    L.ci = L.cj = L.ck = __builtin_nanf("");
}

// Lane state of input muon j.
__device__ __forceinline__ void load_lane_at(Lane &L, int64_t j, const KArgs &A) {
    const DevIO &io = A.io;
    const DevRun &R = A.R;
    L.x = io.x[j];
    L.y = io.y[j];
    L.z = io.z[j];
    L.px = io.px[j];
    L.py = io.py[j];
    L.pz = io.pz[j];
    const int qi = io.q[j];
    L.kq = (float)kKappa * (float)qi;
    L.ph = philox_prefix((uint32_t)j, (uint32_t)((uint64_t)j >> 32), R.key0, R.key1);
    L.steps = 0;
    reset_lane_caches(L, A.T);
    L.status = MT_ST_RUNNING;
    const double p2 = L.px * L.px + L.py * L.py + L.pz * L.pz;
    const bool ok = isfinite(L.x) && isfinite(L.y) && isfinite(L.z) && isfinite(p2) &&
                    p2 > 0.0 && (qi == 1 || qi == -1);
    if (!ok) L.status = MT_ST_INVALID;
}

// Variant of output slot g = var * n + j.  Formed where it is needed (a new
// volume's scaled field) rather than kept in a register.
template <class RR>
__device__ __forceinline__ int64_t variant_of(int64_t g, const RR &R) {
    if (R.lanes == R.n) return 0;
    return R.lanes <= 0xFFFFFFFFll ? (int64_t)((uint32_t)g / (uint32_t)R.n) : g / R.n;
}

__device__ __forceinline__ void load_lane(Lane &L, int64_t g, const KArgs &A) {
    load_lane_at(L, g - variant_of(g, A.R) * A.R.n, A);
}

// ---------------------------------------------------------------------------
// Geometry: z-slab, then the slab's candidate boxes in index order.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int find_slab(const Lds &S, int n_slab, double z, int s) {
    if (s < 0) {                       // largest s with slabz[s] <= z (slabz[0] = -inf)
        int lo = 0, hi = n_slab - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (S.slabz[mid] <= z) lo = mid; else hi = mid - 1;
        }
        return lo;
    }
    while (s > 0 && z < S.slabz[s]) --s;
    while (s < n_slab - 1 && z >= S.slabz[s + 1]) ++s;
    return s;
}

// Branch-free: the four bounds come in two 16-byte LDS reads and the four
// compares are combined with bitwise ands (short-circuit && would turn every
// compare into a branch with its own dependent LDS read).
__device__ __forceinline__ bool in_box_xy(const Lds &S, int b, double x, double y) {
    const double2 *bx = reinterpret_cast<const double2 *>(S.box4 + 4 * b);
    const double2 xr = bx[0], yr = bx[1];
    return (xr.x <= x) & (x < xr.y) & (yr.x <= y) & (y < yr.y);
}

__device__ __forceinline__ int find_box(const Lds &S, int s, double x, double y) {
    uint64_t m = S.slabm[s];
    while (m) {
        const int b = __builtin_ctzll(m);
        if (in_box_xy(S, b, x, y)) return b;
        m &= m - 1;
    }
    return -1;
}

// Distances from the position to both ends of a region on every axis.  In
// FP32 (the lookups around them are FP64): set_region takes off more than that
// rounds.
struct Region {
    float xl, xh, yl, yh, zl, zh;
};

// Box containing the lane's position (lowest index).
template <class TT>
__device__ __forceinline__ int locate_box(Lane &L, const TT &T, const Lds &S) {
    L.slab = find_slab(S, T.geom.n_slab, L.z, L.slab);
    return find_box(S, L.slab, L.x, L.y);
}

// Region of the position from the tables: the loader keeps one of every slab
// and, for geometries without overlapping boxes, of every box (within the
// world).  Returns whether the position is inside it.
template <class TT>
__device__ __forceinline__ bool table_region(Lane &L, int vol, const TT &T, const Lds &S) {
    if (vol < 0 || !T.geom.disjoint) return false;
    const BoxRegion b = S.breg[vol];
    const SlabRegion z = S.sreg[L.slab];
    L.ix = b.ix;
    L.iy = b.iy;
    L.iz = z.iz;
    L.xr = (float)(L.x - b.xc) * b.ix;
    L.yr = (float)(L.y - b.yc) * b.iy;
    L.zr = (float)(L.z - z.zc) * z.iz;
    return fmaxf(fmaxf(fabsf(L.xr), fabsf(L.yr)), fabsf(L.zr)) < 1.0f;
}

// Region of a position in empty space, in overlapping boxes or beside a face:
// in z the slab; laterally the box, no nearer than any candidate of lower
// index (all of them in empty space).
__device__ __forceinline__ Region box_region(const Lane &L, int vol, const Lds &S) {
    Region r;
    float gap = kRegionHalf;    // largest violated bound of the nearest candidate passed over
    uint64_t c = S.slabm[L.slab];
    while (c) {
        const int b = __builtin_ctzll(c);
        if (b == vol) break;
        const double *bx = S.box4 + 4 * b;
        gap = fminf(gap, fmaxf(fmaxf((float)(bx[0] - L.x), (float)(L.x - bx[1])),
                               fmaxf((float)(bx[2] - L.y), (float)(L.y - bx[3]))));
        c &= c - 1;
    }
    r.xl = r.xh = r.yl = r.yh = gap;
    if (vol >= 0) {
        const double *bx = S.box4 + 4 * vol;
        r.xl = fminf(gap, (float)(L.x - bx[0]));
        r.xh = fminf(gap, (float)(bx[1] - L.x));
        r.yl = fminf(gap, (float)(L.y - bx[2]));
        r.yh = fminf(gap, (float)(bx[3] - L.y));
    }
    r.zl = fminf(kRegionHalf, (float)(L.z - S.slabz[L.slab]));
    r.zh = fminf(kRegionHalf, (float)(S.slabz[L.slab + 1] - L.z));
    return r;
}

// One axis of the region: relative position and 1 / half width.  The 2^-14
// and the 1e-7 m pay for the rounding of the distances, of at most
// kRegionSteps FP32 sums and of FP64 positions below kRegionCoord; a region
// narrower than that is none (relative position 2).
__device__ __forceinline__ void set_axis(float lo, float hi, bool use, float &rel, float &inv) {
    const float half = fmaf(0.5f * (lo + hi), 1.0f - 0x1p-14f, -1e-7f);
    const bool ok = use & (half > 1e-6f);
    inv = ok ? __builtin_amdgcn_rcpf(half) : 0.0f;
    rel = ok ? 0.5f * (lo - hi) * inv : 2.0f;
}

template <class GG>
__device__ __forceinline__ void set_region(Lane &L, Region r, const GG &G) {
    r.xl = fminf(r.xl, (float)(G.x_max + L.x));
    r.xh = fminf(r.xh, (float)(G.x_max - L.x));
    r.yl = fminf(r.yl, (float)(G.y_max + L.y));
    r.yh = fminf(r.yh, (float)(G.y_max - L.y));
    r.zh = fminf(r.zh, (float)(G.z_max - L.z));
    const bool use = (fabs(L.x) <= kRegionCoord) & (fabs(L.y) <= kRegionCoord) &
                     (fabs(L.z) <= kRegionCoord);
    set_axis(r.xl, r.xh, use, L.xr, L.ix);
    set_axis(r.yl, r.yh, use, L.yr, L.iy);
    set_axis(r.zl, r.zh, use, L.zr, L.iz);
}

__device__ __forceinline__ bool outside_region(const Lane &L, int k) {
    return (k % kRegionSteps == 0) |
           !(fmaxf(fmaxf(fabsf(L.xr), fabsf(L.yr)), fabsf(L.zr)) < 1.0f);
}

// Least of the plane functions and hz - |zr|: positive inside.
__device__ __forceinline__ float plane_slack(const BlockPlanes &b, float x, float y, float z) {
    float f[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float4 p = b.side[i];
        f[i] = fmaf(p.x, x, fmaf(p.y, y, fmaf(p.z, z, p.w)));
    }
    return fminf(fminf(fminf(f[0], f[1]), f[2]), fminf(f[3], b.hz - fabsf(z)));
}

__device__ __forceinline__ bool outside_planes(const Lane &L, int k) {
    const BlockPlanes &b = *reinterpret_cast<const BlockPlanes *>(lds_base() + L.rec);
    return (k % kRegionSteps == 0) | !(plane_slack(b, L.xr, L.yr, L.zr) > 0.0f);
}

__device__ __forceinline__ void move_in_region(Lane &L, float dx, float dy, float dz) {
    L.xr = fmaf(dx, L.ix, L.xr);
    L.yr = fmaf(dy, L.iy, L.yr);
    L.zr = fmaf(dz, L.iz, L.zr);
}

// Convex block b holds (x, y, z): z_lo <= z < z_hi and the edge cross
// products of the slice at z (Eq. (1)) all >= 0 or all <= 0.  Needed only
// beside a face, so it is a loop over the edges with few registers.
__device__ __forceinline__ bool in_block(const Lds &S, int b, double x, double y, double z) {
    const double *r = S.blk + kBlockRec * b;
    if (!(r[0] <= z && z < r[1])) return false;
    const double t = (z - r[0]) * r[2];
    bool pos = true, neg = true;
#pragma unroll 1
    for (int i = 0; i < 4; ++i) {
        const int j = (i + 1) & 3;
        const double vxi = fma(t, r[12 + 2 * i], r[4 + 2 * i]);
        const double vyi = fma(t, r[13 + 2 * i], r[5 + 2 * i]);
        const double vxj = fma(t, r[12 + 2 * j], r[4 + 2 * j]);
        const double vyj = fma(t, r[13 + 2 * j], r[5 + 2 * j]);
        const double si = (vxj - vxi) * (y - vyi) - (vyj - vyi) * (x - vxi);
        pos = pos && si >= 0.0;
        neg = neg && si <= 0.0;
    }
    return pos || neg;
}

// Where the position lies with respect to block b, decided in FP32 with a
// margin for its rounding (see BlockRegion): 1 inside and clear of the faces
// (then no block of lower index holds it, and r is the region in which that
// stays so), -1 outside, 0 too close to a face to say.
__device__ __forceinline__ int classify_block(const Lds &S, int b, const Lane &L, Region &r) {
    const BlockRegion &c = S.preg[b];
    const double *q = S.blk + kBlockRec * b;
    if (!(q[0] <= L.z && L.z < q[1])) return -1;
    const float x = (float)(L.x - c.xc), y = (float)(L.y - c.yc);
    const float zl = (float)(L.z - q[0]), zh = (float)(q[1] - L.z);
    if (!(fmaxf(fabsf(x), fabsf(y)) < c.ext)) return -1;
    const float t = zl * (float)q[2];
    r = Region{kRegionHalf, kRegionHalf, kRegionHalf, kRegionHalf, zl, zh};
    const float vx0 = fmaf(t, c.dx[0], c.bx[0]), vy0 = fmaf(t, c.dy[0], c.by[0]);
    float vx = vx0, vy = vy0, least = INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float wx = i == 3 ? vx0 : fmaf(t, c.dx[(i + 1) & 3], c.bx[(i + 1) & 3]);
        const float wy = i == 3 ? vy0 : fmaf(t, c.dy[(i + 1) & 3], c.by[(i + 1) & 3]);
        const float s = fmaf(wx - vx, y - vy, -((wy - vy) * (x - vx)));
        const float side = c.sigma * s, slack = side - c.tau;
        least = fminf(least, side);
        r.xl = fminf(r.xl, slack * c.cxl[i]);
        r.xh = fminf(r.xh, slack * c.cxh[i]);
        r.yl = fminf(r.yl, slack * c.cyl[i]);
        r.yh = fminf(r.yh, slack * c.cyh[i]);
        r.zl = fminf(r.zl, slack * c.cz[i]);
        r.zh = fminf(r.zh, slack * c.cz[i]);
        vx = wx;
        vy = wy;
    }
    return least > c.tau ? 1 : (least < -c.err ? -1 : 0);
}

// Cuts r laterally so that it stays out of a rectangle, on the axis on which the
// position is farther from it; leaves it no width if that is not outside.
__device__ __forceinline__ void cut_region(Region &r, const Lane &L, double xlo, double xhi,
                                           double ylo, double yhi) {
    const float ax = (float)(xlo - L.x), bx = (float)(L.x - xhi);
    const float ay = (float)(ylo - L.y), by = (float)(L.y - yhi);
    const float gx = fmaxf(ax, bx), gy = fmaxf(ay, by);
    if (gx > 0.0f && gx >= gy) {
        if (ax > bx) r.xh = fminf(r.xh, gx); else r.xl = fminf(r.xl, gx);
    } else if (gy > 0.0f) {
        if (ay > by) r.yh = fminf(r.yh, gy); else r.yl = fminf(r.yl, gy);
    } else {
        r.yl = r.yh = 0.0f;
    }
}

// Lowest-index block holding the lane's position.  In turn the block found last
// and the candidates (those of the grid cell that span the z-slab) are
// classified in FP32, by their planes where they have any; a clear one is the
// answer.  Only if none is and some cannot be told apart the exact sign test
// decides, lowest index first.  known: the answer is a block whose planes track
// the lane from here (the position is inside the world too).  Otherwise r: a
// region in which the answer stays, or one of no width (beside a face).  In
// empty space that is the slab, laterally without limit where no block spans
// it, else the grid cell (or the space beside the grid) without the bounding
// boxes of the candidates.
template <class TT>
__device__ __forceinline__ int locate_block(Lane &L, const TT &T, const Lds &S, Region &r,
                                            bool &known) {
    const auto &G = T.geom;
    const int sl = find_slab(S, G.n_slab, L.z, L.slab);
    L.slab = sl;
    const uint64_t in_slab = S.slabm[sl];
    const double u = (L.x - G.g0[0]) * G.ginv[0];
    const double v = (L.y - G.g0[1]) * G.ginv[1];
    const double w = (L.z - G.g0[2]) * G.ginv[2];
    const bool in_grid = u >= 0.0 && v >= 0.0 && w >= 0.0 && u < (double)G.gx &&
                         v < (double)G.gy && w < (double)G.gz;
    const int cu = (int)u, cv = (int)v, cw = (int)w;
    uint64_t mask = 0;
    if (in_grid && in_slab != 0) mask = S.grid[(cw * G.gy + cv) * G.gx + cu] & in_slab;
    bool unsure = false;
    uint64_t m = mask;
    int b = L.vol >= 0 && ((in_slab >> L.vol) & 1) ? L.vol : -1;
    for (;;) {
        if (b >= 0) {
            const BlockPlanes &P = S.planes[b];
            const float x = (float)(L.x - P.xc), y = (float)(L.y - P.yc), z = (float)(L.z - P.zc);
            const float slack = plane_slack(P, x, y, z);
            if (slack > 0.0f) {
                L.rec = (uint32_t)T.lds.off_planes + (uint32_t)sizeof(BlockPlanes) * (uint32_t)b;
                L.ix = L.iy = L.iz = 1.0f;
                L.xr = x;
                L.yr = y;
                L.zr = z;
                known = true;
                return b;
            }
            // (a block of the slab spans z: a point outside is beside a plane)
            if (P.hz < 0.0f || !(slack < -2.0f * P.err)) {
                const int side = classify_block(S, b, L, r);
                if (side > 0) return b;
                unsure |= side == 0;
            }
        }
        if (m == 0) break;
        b = __builtin_ctzll(m);
        m &= m - 1;
    }
    if (unsure) {
        r = Region{0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (m = mask; m; m &= m - 1) {
            b = __builtin_ctzll(m);
            if (in_block(S, b, L.x, L.y, L.z)) return b;
        }
        return -1;
    }
    r = Region{kRegionHalf, kRegionHalf, kRegionHalf, kRegionHalf,
               fminf(kRegionHalf, (float)(L.z - S.slabz[sl])),
               fminf(kRegionHalf, (float)(S.slabz[sl + 1] - L.z))};
    if (in_slab == 0) return -1;
    if (!in_grid) {
        cut_region(r, L, G.g0[0], G.g1[0], G.g0[1], G.g1[1]);
        return -1;
    }
    const float fx = (float)(u - (double)cu), fy = (float)(v - (double)cv);
    const float cx = __builtin_amdgcn_rcpf((float)G.ginv[0]);
    const float cy = __builtin_amdgcn_rcpf((float)G.ginv[1]);
    const float cz = __builtin_amdgcn_rcpf((float)G.ginv[2]), fz = (float)(w - (double)cw);
    r = Region{fx * cx, (1.0f - fx) * cx, fy * cy, (1.0f - fy) * cy,
               fminf(r.zl, fz * cz), fminf(r.zh, (1.0f - fz) * cz)};
    for (m = mask; m; m &= m - 1) {
        const BlockRegion &c = S.preg[__builtin_ctzll(m)];
        cut_region(r, L, (double)c.xlo, (double)c.xhi, (double)c.ylo, (double)c.yhi);
    }
    return -1;
}

// Momentum bin i with e_i^2 <= |p|^2 < e_{i+1}^2, clamped to [0, P-1]; the
// previous step's bin is the starting guess.
__device__ __forceinline__ int find_bin(const Lds &S, int P, double p2, int i) {
    if (i <= 0) {
        int lo = 0, hi = P - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (S.e2[mid] <= p2) lo = mid; else hi = mid - 1;
        }
        return lo;
    }
    while (i > 0 && p2 < S.e2[i]) --i;
    while (i < P - 1 && p2 >= S.e2[i + 1]) ++i;
    return i;
}

// The same with large tables, by pb, the bits of float(|p|^2), and the ends of the
// bands, which decide as |p|^2 would (a raised end is no larger than pb, |p|^2
// being at least the threshold) unless pb is on one of them or outside every band:
// then the edges in memory decide.
__device__ __forceinline__ int find_bin_wide(const Lds &S, int P, double p2, uint32_t pb, int i) {
    if (p2 != p2) return max(i, 0);
    if (i <= 0) {
        int lo = 0, hi = P - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (S.edge[mid] <= pb) lo = mid; else hi = mid - 1;
        }
        i = lo;
    } else {
        while (i > 0 && pb < S.edge[i]) --i;
        while (i < P - 1 && pb >= S.edge[i + 1]) ++i;
    }
    if (pb <= S.edge[i] || pb >= 0x7f800000u) {
        while (i > 0 && p2 < S.e2[i]) --i;
        while (i < P - 1 && p2 >= S.e2[i + 1]) ++i;
    }
    return i;
}

// The band between two ends: first pattern and number of patterns.
__device__ __forceinline__ uint2 band_between(uint32_t lo, uint32_t hi) {
    return make_uint2(lo + 1u, __builtin_elementwise_sub_sat(hi, lo + 1u));
}

// Exact inverse CDF: t = floor(w * T / 2^32), cell = smallest c with C[c] > t.
// The guide entry of the word's top bits brackets c in [lo, hi] and carries
// C[lo]: t < C[lo] gives lo at once, a bracket of two cells gives hi, and only
// wider brackets probe C.
__device__ __forceinline__ uint2 guide_entry(const DevHist &H, uint32_t hoff, uint32_t w0) {
    // hoff = 8 h << gbits < 2^31 (h < 2^12, gbits <= 16): the entry's byte
    // offset is a 32-bit number
    const uint32_t at = hoff | ((w0 >> (29 - H.gbits)) & ~7u);
    return *reinterpret_cast<const uint2 *>(reinterpret_cast<const char *>(H.guide) + at);
}

__device__ __forceinline__ int sample_cell(const DevHist &H, uint2 e, uint32_t hoff, uint32_t T,
                                           uint32_t w0) {
    const uint32_t t = __umulhi(w0, T);
    int lo = (int)(e.x & 0xFFFFu);
    int hi = (int)(e.x >> 16);
    if (t < e.y) return lo;
    ++lo;
    // h K < 2^28 (4 h K < 2^30 bytes): 32-bit offsets from the table's base
    const uint32_t row = (hoff >> (H.gbits + 3)) * (uint32_t)H.n_cells;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (H.cdf[row + (uint32_t)mid] > t) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// Alias method: column j = floor(w0 K / 2^32); the 24-bit threshold word x
// (low bytes of w1, w2, w3, which the jitters and the azimuth leave unused)
// keeps cell j when x is below the column's split, else gives its alias.
// One 8-byte load per draw, its byte offset 8 (h K + j) < 2^31.
__device__ __forceinline__ uint2 alias_entry(const DevHist &H, uint32_t h, uint32_t w0) {
    const uint32_t j = __umulhi(w0, (uint32_t)H.n_cells);
    return *reinterpret_cast<const uint2 *>(
        reinterpret_cast<const char *>(H.alias) + 8u * (__umul24(h, (uint32_t)H.n_cells) + j));
}

__device__ __forceinline__ int alias_cell(const DevHist &H, uint2 e, uint4 w) {
    const uint32_t j = __umulhi(w.x, (uint32_t)H.n_cells);
    const uint32_t x = (w.y & 0xFFu) | ((w.z & 0xFFu) << 8) | ((w.w & 0xFFu) << 16);
    return (int)(x < e.x ? j : e.y);
}

// ---------------------------------------------------------------------------
// Kick: p <- p + R(p_hat) (|p| u), u = (tau cos phi, tau sin phi, -f).  The
// rotation maps the local z axis onto p_hat, so the loss part is exactly
// -f p and is applied in FP64 (it is what accumulates over a trajectory);
// the transverse part uses the division-free Rodrigues form
// R v = c v + a x v + (a.v) a / (1 + c), a = z x p_hat = (-ny, nx, 0),
// c = nz (equal to Eq. (2) with k = a/|a|), in FP32.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void kick(Lane &L, float p2f, float ux, float uy, float uz) {
    const float rinv = __builtin_amdgcn_rsqf(p2f);
    const float pm = p2f * rinv;
    const float nx = (float)L.px * rinv, ny = (float)L.py * rinv, nz = (float)L.pz * rinv;
    const float dx = pm * ux, dy = pm * uy;
    const float opc = 1.0f + nz;
    float tx, ty, tz;
    if (opc > 0.0f) {
        const float coef = fmaf(nx, dy, -ny * dx) * __builtin_amdgcn_rcpf(opc);
        tx = fmaf(nz, dx, -coef * ny);
        ty = fmaf(nz, dy, coef * nx);
        tz = -fmaf(nx, dx, ny * dy);
    } else {                           // exactly backwards: rotation by pi about x
        tx = dx;
        ty = -dy;
        tz = 0.0f;
    }
    const double keep = 1.0 + (double)uz;       // 1 - f, exact
    L.px = fma(L.px, keep, (double)tx);
    L.py = fma(L.py, keep, (double)ty);
    L.pz = fma(L.pz, keep, (double)tz);
}

// ---------------------------------------------------------------------------
// Field at the start of the step: scaled per-box field + trilinear map.
// ---------------------------------------------------------------------------
// The trilinear interpolant of a map cell as a polynomial in the point's
// fractional coordinates (fx, fy, fz) in the cell:
//   B = k0 + k1 fx + k2 fy + k3 fz + k4 fx fy + k5 fx fz + k6 fy fz + k7 fx fy fz,
// the coefficients formed by the loader in FP64 from the cell's 8 corner
// values (k0 = B000, k1 = B100 - B000, ..., k7 the alternating sum of all
// eight) and stored as the cell's 128-byte record.  It equals the nested
// linear interpolation of the corners (the oracle's form) up to rounding,
// and takes 7 FMAs per component instead of 14 operations.
struct CellPoly {
    float4 k[8];
    float fx, fy, fz;
};

// Grid coordinates of a point: u = (x - lo) / d as one FMA, x (n - 1)/(hi -
// lo) - lo (n - 1)/(hi - lo), with both factors formed on the host.  Every
// map lookup (forward, replay, stage points) uses this, so the forward and
// the adjoint's replay see the same cells and weights.
__device__ __forceinline__ void map_coords(const DevField &F, double x, double y, double z,
                                           double &u, double &v, double &w) {
    u = fma(x, F.inv_d[0], F.off[0]);
    v = fma(y, F.inv_d[1], F.off[1]);
    w = fma(z, F.inv_d[2], F.off[2]);
}

// Inside the map's node range on all three axes (closed): six compares
// combined without branches, against the node counts as doubles.
template <class FF>
__device__ __forceinline__ bool in_map(const FF &F, double u, double v, double w) {
    return (u >= 0.0) & (u <= F.umax[0]) & (v >= 0.0) & (v <= F.umax[1]) & (w >= 0.0) &
           (w <= F.umax[2]);
}

__device__ __forceinline__ bool map_cell(const DevField &F, double x, double y, double z,
                                         CellPoly &c) {
    double u, v, w;
    map_coords(F, x, y, z, u, v, w);
    if (!in_map(F, u, v, w))
        return false;
    const int i = min((int)u, F.nx - 2), j = min((int)v, F.ny - 2), k = min((int)w, F.nz - 2);
    c.fx = (float)(u - (double)i);
    c.fy = (float)(v - (double)j);
    c.fz = (float)(w - (double)k);
    const float4 *b = F.map + (((size_t)k * (F.ny - 1) + j) * (F.nx - 1) + i) * 8;
#pragma unroll
    for (int q = 0; q < 8; ++q) c.k[q] = b[q];
    return true;
}

// One component of the cell polynomial, grouped as
// k0 + fz k3 + fy (k2 + fz k6) + fx (k1 + fy (k4 + fz k7) + fz k5).
__device__ __forceinline__ float cell_poly1(float k0, float k1, float k2, float k3, float k4,
                                            float k5, float k6, float k7, float fx, float fy,
                                            float fz) {
    const float a = fmaf(fz, k5, fmaf(fy, fmaf(fz, k7, k4), k1));
    const float b = fmaf(fy, fmaf(fz, k6, k2), fmaf(fz, k3, k0));
    return fmaf(fx, a, b);
}

__device__ __forceinline__ float3 cell_field(const CellPoly &c) {
    float3 r;
    r.x = cell_poly1(c.k[0].x, c.k[1].x, c.k[2].x, c.k[3].x, c.k[4].x, c.k[5].x, c.k[6].x,
                     c.k[7].x, c.fx, c.fy, c.fz);
    r.y = cell_poly1(c.k[0].y, c.k[1].y, c.k[2].y, c.k[3].y, c.k[4].y, c.k[5].y, c.k[6].y,
                     c.k[7].y, c.fx, c.fy, c.fz);
    r.z = cell_poly1(c.k[0].z, c.k[1].z, c.k[2].z, c.k[3].z, c.k[4].z, c.k[5].z, c.k[6].z,
                     c.k[7].z, c.fx, c.fy, c.fz);
    return r;
}

// V: the field is vertical and only its y component is read; a scale that is not
// finite, which makes a general field NaN on every axis (0 times it is NaN),
// makes this one NaN too.
template <bool V, class TT, class RR>
__device__ __forceinline__ float3 box_field(const TT &T, const Lds &S, const RR &R, int vol,
                                            int var) {
    float3 B = make_float3(0.f, 0.f, 0.f);
    if (vol >= 0) {
        const float4 b = S.bf[vol];
        const int m = S.mag[vol];
        const float s = (m >= 0 && R.scales != nullptr) ? R.scales[var * T.geom.n_mag + m] : 1.0f;
        if (V) B.y = fmaf(-0.0f, fabsf(s), b.y * s);     // + -0 or NaN
        else B = make_float3(b.x * s, b.y * s, b.z * s);
    }
    return B;
}

template <bool MAP>
__device__ __forceinline__ float3 add_map(const Tables &T, float3 B, double x, double y, double z) {
    if (MAP) {
        CellPoly c;
        if (map_cell(T.field, x, y, z, c)) {
            const float3 m = cell_field(c);
            B.x += m.x;
            B.y += m.y;
            B.z += m.z;
        }
    }
    return B;
}

// Trilinear map at a point (the lane's position, or an RK4 stage point near
// it) with the lane's current cell's coefficients kept in registers:
// consecutive 2 cm steps and their stage points mostly stay in one cell, so
// the 128-byte record is loaded only when the point lies in another cell
// (which then becomes the lane's cell).  The point is in the lane's cell, and
// so inside the map, when its fractional coordinates in that cell lie in
// [0, 1): as bit patterns, one unsigned maximum and one compare; negative, NaN
// and rounded-up values fail it and take the exact lookup.  Same values and
// arithmetic as map_cell + cell_field.  Outside the map the cell is empty
// (all coefficients zero, no cell remembered).
template <bool V>
__device__ __forceinline__ float3 add_map_cached(Lane &L, const DevField &H, ArgPtr args, float3 B,
                                                 double x, double y, double z) {
    double u, v, w;
    map_coords(H, x, y, z, u, v, w);
    CellPoly c;
    c.fx = (float)(u - (double)L.ci);      // cell indices are below 2^24: exact floats
    c.fy = (float)(v - (double)L.cj);
    c.fz = (float)(w - (double)L.ck);
    if (max(max(__float_as_uint(c.fx), __float_as_uint(c.fy)), __float_as_uint(c.fz)) >=
        0x3f800000u) {
        const auto &F = cold(args)->T.field;
        if (in_map(F, u, v, w)) {
            const int i = min((int)u, F.nx - 2), j = min((int)v, F.ny - 2),
                      k = min((int)w, F.nz - 2);
            // 24-bit products: the loader keeps nx and ny nz below 2^24
            const int cell = (int)__umul24(__umul24((uint32_t)k, (uint32_t)(F.ny - 1)) +
                                               (uint32_t)j, (uint32_t)(F.nx - 1)) + i;
            if constexpr (V) {
                const float4 *b = F.mapv + (size_t)cell * 2;
                const float4 p = b[0], r = b[1];
                L.mc[0] = p.x;
                L.mc[1] = p.y;
                L.mc[2] = p.z;
                L.mc[3] = p.w;
                L.mc[4] = r.x;
                L.mc[5] = r.y;
                L.mc[6] = r.z;
                L.mc[7] = r.w;
            } else {
                const float4 *b = F.map + (size_t)cell * 8;
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const float4 r = b[q];
                    L.mc[3 * q] = r.x;
                    L.mc[3 * q + 1] = r.y;
                    L.mc[3 * q + 2] = r.z;
                }
            }
            L.ci = (float)i;
            L.cj = (float)j;
            L.ck = (float)k;
            c.fx = (float)(u - (double)i);
            c.fy = (float)(v - (double)j);
            c.fz = (float)(w - (double)k);
        } else {
#pragma unroll
            for (int q = 0; q < (V ? 8 : 24); ++q) L.mc[q] = 0.0f;
            L.ci = __builtin_nanf("");
            c.fx = c.fy = c.fz = 0.0f;
        }
    }
    if constexpr (V) {
        const float by = cell_poly1(L.mc[0], L.mc[1], L.mc[2], L.mc[3], L.mc[4], L.mc[5], L.mc[6],
                                    L.mc[7], c.fx, c.fy, c.fz);
        return make_float3(0.0f, B.y + by, 0.0f);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q)
        c.k[q] = make_float4(L.mc[3 * q], L.mc[3 * q + 1], L.mc[3 * q + 2], 0.f);
    const float3 m = cell_field(c);
    return make_float3(B.x + m.x, B.y + m.y, B.z + m.z);
}

// Nearest-node lookup of the map: the node closest to (x, y, z) on every axis
// (half-way points take the higher node), zero outside the grid; one 16-byte
// load from the node-major copy of the map.  The last node's value is kept in
// registers (mc[0..2]) and used while the point is less than half a spacing
// from it on every axis; nodes on the map's border are not remembered, since
// near them that test does not say whether the point is inside the map.
template <bool V>
__device__ __forceinline__ float3 add_nearest_cached(Lane &L, const DevField &H, ArgPtr args,
                                                     float3 B, double x, double y, double z) {
    double u, v, w;
    map_coords(H, x, y, z, u, v, w);
    const float du = (float)(u - (double)L.ci), dv = (float)(v - (double)L.cj),
                dw = (float)(w - (double)L.ck);
    if (!((fabsf(du) < 0.5f) & (fabsf(dv) < 0.5f) & (fabsf(dw) < 0.5f))) {
        L.ci = __builtin_nanf("");
        float4 q = make_float4(0.f, 0.f, 0.f, 0.f);
        const auto &F = cold(args)->T.field;
        if (in_map(F, u, v, w)) {
            const int i = min((int)(u + 0.5), F.nx - 1), j = min((int)(v + 0.5), F.ny - 1),
                      k = min((int)(w + 0.5), F.nz - 1);
            const int node = (int)__umul24(__umul24((uint32_t)k, (uint32_t)F.ny) + (uint32_t)j,
                                           (uint32_t)F.nx) + i;
            if constexpr (V) q.y = F.nodesv[node];
            else q = F.nodes[node];
            if ((i > 0) & (i < F.nx - 1) & (j > 0) & (j < F.ny - 1) & (k > 0) & (k < F.nz - 1)) {
                L.ci = (float)i;
                L.cj = (float)j;
                L.ck = (float)k;
            }
        }
        L.mc[0] = q.x;
        L.mc[1] = q.y;
        L.mc[2] = q.z;
    }
    return make_float3(B.x + L.mc[0], B.y + L.mc[1], B.z + L.mc[2]);
}

// ---------------------------------------------------------------------------
// RK4 over arc length with B frozen: dr/ds = p/|p|, dp/ds = kappa q (p/|p|) x B.
// FP32 stages, increments added to the FP64 state.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float3 cross3(float3 a, float3 b) {
    return make_float3(fmaf(a.y, b.z, -a.z * b.y), fmaf(a.z, b.x, -a.x * b.z),
                       fmaf(a.x, b.y, -a.y * b.x));
}

__device__ __forceinline__ float norm2(float3 a) { return fmaf(a.x, a.x, fmaf(a.y, a.y, a.z * a.z)); }

__device__ __forceinline__ float3 axpy(float a, float3 x, float3 y) {
    return make_float3(fmaf(a, x.x, y.x), fmaf(a, x.y, y.y), fmaf(a, x.z, y.z));
}

__device__ __forceinline__ float3 scale3(float a, float3 x) {
    return make_float3(a * x.x, a * x.y, a * x.z);
}

__device__ __forceinline__ float3 add3(float3 a, float3 b) {
    return make_float3(a.x + b.x, a.y + b.y, a.z + b.z);
}

// n x b and a h + k where the field may be known to be vertical (V: b.x = b.z =
// 0, so the product has no y component): the general forms' values without
// their multiplications by zero.
template <bool V>
__device__ __forceinline__ float3 cross_field(float3 n, float3 b) {
    if constexpr (V) return make_float3(-n.z * b.y, 0.0f, n.x * b.y);
    else return cross3(n, b);
}

template <bool V>
__device__ __forceinline__ float3 axpy_field(float h, float3 k, float3 a) {
    if constexpr (V) return make_float3(fmaf(h, k.x, a.x), a.y, fmaf(h, k.z, a.z));
    else return axpy(h, k, a);
}

template <bool V>
__device__ __forceinline__ float3 scale_field(float s, float3 b) {
    if constexpr (V) return make_float3(0.0f, s * b.y, 0.0f);
    else return scale3(s, b);
}

struct StepConst {
    float h, h2, h6, h3;   // d, d/2, d/6, d/3
};

__device__ __forceinline__ float3 stage0(const Lane &L) {
    return make_float3((float)L.px, (float)L.py, (float)L.pz);
}

// Is any component of b non-zero?  One or of the three bit patterns and one
// compare (the or is +-0 exactly when all three are).
template <bool V>
__device__ __forceinline__ bool non_zero(float3 b) {
    if constexpr (V) return b.y != 0.0f;
    return __uint_as_float(__float_as_uint(b.x) | __float_as_uint(b.y) | __float_as_uint(b.z)) !=
           0.0f;
}

// a0 must be stage0(L) (the FP32 momentum the stages start from), cb = kq B
// and bent = (B is not zero).
template <bool V>
__device__ __forceinline__ void rk4_from(Lane &L, float3 a0, float3 cb, bool bent,
                                         const StepConst &c) {
    const float r0 = __builtin_amdgcn_rsqf(norm2(a0));
    const float3 n0 = scale3(r0, a0);
    float drx, dry, drz;
    if (!bent) {
        drx = c.h * n0.x;
        dry = c.h * n0.y;
        drz = c.h * n0.z;
    } else {
        const float3 k1 = cross_field<V>(n0, cb);
        const float3 a1 = axpy_field<V>(c.h2, k1, a0);
        const float3 n1 = scale3(__builtin_amdgcn_rsqf(norm2(a1)), a1);
        const float3 k2 = cross_field<V>(n1, cb);
        const float3 a2 = axpy_field<V>(c.h2, k2, a0);
        const float3 n2 = scale3(__builtin_amdgcn_rsqf(norm2(a2)), a2);
        const float3 k3 = cross_field<V>(n2, cb);
        const float3 a3 = axpy_field<V>(c.h, k3, a0);
        const float3 n3 = scale3(__builtin_amdgcn_rsqf(norm2(a3)), a3);
        const float3 k4 = cross_field<V>(n3, cb);
        // h/6 (v1 + 2 v2 + 2 v3 + v4)
        drx = c.h6 * (fmaf(2.0f, n1.x + n2.x, n0.x) + n3.x);
        dry = c.h6 * (fmaf(2.0f, n1.y + n2.y, n0.y) + n3.y);
        drz = c.h6 * (fmaf(2.0f, n1.z + n2.z, n0.z) + n3.z);
        const float dpx = c.h6 * (fmaf(2.0f, k2.x + k3.x, k1.x) + k4.x);
        const float dpz = c.h6 * (fmaf(2.0f, k2.z + k3.z, k1.z) + k4.z);
        L.px += (double)dpx;
        if constexpr (!V) {
            const float dpy = c.h6 * (fmaf(2.0f, k2.y + k3.y, k1.y) + k4.y);
            L.py += (double)dpy;
        }
        L.pz += (double)dpz;
    }
    // the position update is shared by both branches (keeps every Lane field
    // in registers: no store through a selected address)
    move_in_region(L, drx, dry, drz);
    L.x += (double)drx;
    L.y += (double)dry;
    L.z += (double)drz;
}

// Compile-time features of a transport kernel (bit mask).
enum : unsigned {
    kMap = 1u,       // a field map is loaded
    kTape = 2u,      // write checkpoints and the kick tape (differentiable form)
    kWide = 4u,      // large histogram tables (see AllTables), and per-step traces
    kAlias = 8u,     // alias-method sampler instead of the inverse CDF
    kNearest = 16u,  // nearest-node map lookup instead of trilinear (with kMap)
    kStages = 32u,   // field evaluated at every RK4 stage position
    kPoly = 64u,     // convex-block geometry instead of boxes
    kLog = 128u,     // a histogram axis is binned in log10
    kVert = 256u,    // every field (boxes, blocks and map) is vertical: B = (0, By, 0)
    kFeatures = 512u,// number of masks
    kPasses = 512u,  // the kernel runs passes (not a mask bit)
    kNow = 1024u,    // the step's draw is not formed ahead (not a mask bit)
    kRoom = 2048u    // few waves: registers before occupancy (not a mask bit)
};

// Masks that have a kernel: the tape belongs to the differentiable form,
// whose adjoint holds the trilinear field over each step, and the
// nearest-node lookup needs a map; large tables and traces run the general field.
constexpr bool valid_mask(unsigned F) {
    return !((F & kTape) && (F & (kNearest | kStages))) && !((F & kNearest) && !(F & kMap)) &&
           !((F & kPoly) && (F & (kTape | kStages))) && !((F & kVert) && (F & kWide));
}

// The map part of the field, added to the volume's, through the lane's cell.
template <unsigned F>
__device__ __forceinline__ float3 with_map(Lane &L, const KArgs &A, ArgPtr args, float3 B, double x,
                                           double y, double z) {
    if constexpr ((F & kNearest) != 0) return add_nearest_cached<(F & kVert) != 0>(L, A.T.field, args, B, x, y, z);
    else if constexpr ((F & kMap) != 0) return add_map_cached<(F & kVert) != 0>(L, A.T.field, args, B, x, y, z);
    else return B;
}

// Field at a stage point: scaled field of the box holding it plus the map.
// `inside`: the lane's region proves that the point is in the lane's volume.
template <unsigned F, typename V>
__device__ __forceinline__ float3 field_at_point(const KArgs &A, ArgPtr args, Lane &L, bool inside,
                                                 V &&var, double x, double y, double z) {
    float3 B = make_float3(L.bx, L.by, L.bz);
    if (!inside) {
        const ArgPtr c = cold(args);
        const Lds S = lds_view<(F & kWide) != 0>(c->T);
        const int vol = find_box(S, find_slab(S, c->T.geom.n_slab, z, L.slab), x, y);
        if (vol != L.vol) B = box_field<(F & kVert) != 0>(c->T, S, c->R, vol, var());
    }
    return with_map<F>(L, A, args, B, x, y, z);
}

// RK4 with the field evaluated afresh at each stage position (stage s sits
// at r + c_s h v_{s-1}, c = 1/2, 1/2, 1); B1 is the step-start field.
// The stage points lie within one step length of the step start, so they are
// in its volume when the region reaches that far.
template <unsigned F, typename V>
__device__ __forceinline__ void rk4_stages(Lane &L, V &&var, float3 B1, const KArgs &A, ArgPtr args,
                                           const StepConst &c) {
    constexpr bool VERT = (F & kVert) != 0;
    const float kq = L.kq;
    const float reach = 1.001f * c.h;
    const bool inside = fmaxf(fmaxf(fmaf(reach, L.ix, fabsf(L.xr)), fmaf(reach, L.iy, fabsf(L.yr))),
                              fmaf(reach, L.iz, fabsf(L.zr))) < 1.0f;
    const float3 a0 = stage0(L);
    const float3 n0 = scale3(__builtin_amdgcn_rsqf(norm2(a0)), a0);
    const float3 k1 = cross_field<VERT>(n0, scale_field<VERT>(kq, B1));
    float3 n = n0, kk = k1;                     // direction and slope of the last stage
    float3 n12 = make_float3(0.f, 0.f, 0.f), k12 = n12;
    // one copy of the stage (its field lookup holds two cold paths)
#pragma unroll 1
    for (int st = 1; st <= 3; ++st) {
        const float cs = st == 3 ? c.h : c.h2;
        const float3 B = field_at_point<F>(A, args, L, inside, var, L.x + (double)(cs * n.x),
                                           L.y + (double)(cs * n.y), L.z + (double)(cs * n.z));
        const float3 a = axpy_field<VERT>(cs, kk, a0);
        n = scale3(__builtin_amdgcn_rsqf(norm2(a)), a);
        kk = cross_field<VERT>(n, scale_field<VERT>(kq, B));
        if (st == 1) {
            n12 = n;
            k12 = kk;
        } else if (st == 2) {
            n12 = add3(n12, n);
            k12 = add3(k12, kk);
        }
    }
    const float drx = c.h6 * (fmaf(2.0f, n12.x, n0.x) + n.x);
    const float dry = c.h6 * (fmaf(2.0f, n12.y, n0.y) + n.y);
    L.px += (double)(c.h6 * (fmaf(2.0f, k12.x, k1.x) + kk.x));
    if constexpr (!VERT) L.py += (double)(c.h6 * (fmaf(2.0f, k12.y, k1.y) + kk.y));
    L.pz += (double)(c.h6 * (fmaf(2.0f, k12.z, k1.z) + kk.z));
    const float drz = c.h6 * (fmaf(2.0f, n12.z, n0.z) + n.z);
    move_in_region(L, drx, dry, drz);
    L.x += (double)drx;
    L.y += (double)dry;
    L.z += (double)drz;
}

// ---------------------------------------------------------------------------
// One iteration of the transport loop at step k (the same for all running
// lanes of a wavefront, so it stays in a scalar register).  Returns false
// (with L.status and L.steps set) when a break condition holds at the top of
// the iteration.
//
// What bounds it: VALU issue.  On gfx950 an FP32 add / mul / fma or a bitwise
// operation on vector registers takes 2 cycles per 64-lane instruction, an
// FP64, compare, conversion or integer product 4, rsq / rcp / sin / cos 8, and
// an FP32 instruction with a scalar-register operand 4 (measured with all
// SIMDs full).  So the common step carries no FP64 compare: it is decided by
// the region and the momentum band of the lane (struct Lane), four cheap
// tests, and everything about the volume and its histogram that does not
// change with the step is in registers.
// ---------------------------------------------------------------------------
template <unsigned F>
constexpr bool kScaledField = !(F & (kMap | kStages));   // L.b* holds kq B

// Step of hoff from one histogram to the next: bytes of a guide row, or (alias
// tables, whose rows are no power of two) one.
template <unsigned F>
__device__ __forceinline__ uint32_t row_of(int gbits) {
    return (F & kAlias) ? 1u : 8u << gbits;
}

template <unsigned F>
__device__ __forceinline__ uint32_t hist_of(const Lane &L, int gbits) {
    return (F & kAlias) ? L.hoff : L.hoff >> (gbits + 3);
}

// Words and table entry of the next step formed ahead, during this one (see
// advance): hides the load's latency where few waves share a SIMD (2000 block
// muons 284 -> 252 us, 123 457 with aliases 322 -> 298, 10^6 1350 -> 1302, 250
// 007 shield muons in the plain form 3.30 -> 3.17 ms).  Not where the seven
// registers it takes cost more: with a general map (trilinear, compiled for 5
// waves, 250 007 muons 3.80 -> 4.39 ms; nearest node, 10^6, 9.20 -> 9.48), the
// field at every stage (7.30 -> 7.41 ms) and the passes over a map, whose waves
// hide it anyway (10^7 muons 77.7 -> 78.0 ms).
// With a general map and at most 4 waves a SIMD to run (DevRun::room), the
// occupancy that plain_min_waves keeps is of no use: the plain form then has
// kernels of its own (kRoom), which take the registers they want and do form
// draws ahead (100 000 muons in the fringe field 3.03 -> 2.79 ms, 250 007 3.81
// -> 3.69, nearest node 3.33 -> 3.19).  A compacting call of one pass that small
// takes the plain form too (200 000: 3.80 -> 3.66; vertical map, 100 000: 2.68
// -> 2.47).
// Past 4 waves a SIMD the fifth wave hides more than the draw formed ahead.
// The variant-wave form has kernels with and without (DevRun::ahead): 12
// variants of 20 011 muons 427 -> 417 us, but 64 of 131 072, which fill the chip,
// 7.72 -> 8.05 ms with it.
template <unsigned F>
constexpr bool kAhead = !(F & (kStages | kNow)) &&
                        (!(F & kMap) || ((F & kVert) && !(F & kPasses)) || (F & kRoom));

// The exact tests of a step that the lane's region or momentum band does not
// decide.
template <unsigned F, typename V>
__device__ __forceinline__ bool locate_region(Lane &L, V &&var, int k, double p2, float p2f,
                                              bool outside, ArgPtr args) {
    const ArgPtr c = cold(args);
    const auto &T = c->T;
    const auto &R = c->R;
    const Lds S = lds_view<(F & kWide) != 0>(T);
    const int P = T.hist.n_pbin, gbits = T.hist.gbits;
    if (outside) {
        int vol;
        bool known = false;
        Region r{};
        if constexpr ((F & kPoly) != 0) {
            vol = locate_block(L, T, S, r, known);
            known = known & (k < R.max_steps);
        } else {
            vol = locate_box(L, T, S);
            known = table_region(L, vol, T, S) & (k < R.max_steps);
        }
        const int old = L.vol;
        L.vol = vol;
        if (!known) {
            // Break test in the order p_min, z_max, x_max, y_max, step cap (the
            // first that holds decides the status; vol is the final volume).
            const bool c_pmin = p2 < R.pmin2, c_z = L.z >= T.geom.z_max;
            // (0 x: a muon made NaN by its field has no y, see lane_y)
            const double y = (F & kVert) ? fma(0.0, L.x, L.y) : L.y;
            const bool c_x = fabs(L.x) >= T.geom.x_max, c_y = fabs(y) >= T.geom.y_max;
            const bool c_k = k >= R.max_steps;
            if (c_pmin | c_z | c_x | c_y | c_k) {
                L.status = c_pmin ? MT_ST_PMIN
                         : c_z    ? MT_ST_ZMAX
                         : c_x    ? MT_ST_XMAX
                         : c_y    ? MT_ST_YMAX
                                  : MT_ST_MAXSTEPS;
                L.steps = k;
                return false;
            }
            if constexpr ((F & kPoly) == 0) {
                r = box_region(L, vol, S);
            } else {
                L.rec = unit_box(T);
            }
            set_region(L, r, T.geom);
        }
        if (vol != old) {
            const float3 b = box_field<(F & kVert) != 0>(T, S, R, vol, var());
            L.bent = non_zero<(F & kVert) != 0>(b);
            const float s = kScaledField<F> ? L.kq : 1.0f;
            L.bx = s * b.x;
            L.by = s * b.y;
            L.bz = s * b.z;
            // another material: the same momentum bin of its histograms; into
            // or out of empty space: the band is looked up below
            const int mat = vol >= 0 ? S.mat[vol] : -1, mat_old = old >= 0 ? S.mat[old] : -1;
            if (mat != mat_old) {
                if ((mat >= 0) & (mat_old >= 0)) {
                    const uint32_t h = hist_of<F>(L, gbits) + (uint32_t)((mat - mat_old) * P);
                    L.hoff = h * row_of<F>(gbits);
                    if constexpr ((F & kAlias) == 0) L.tot = S.tot[h];
                } else {
                    L.hoff = mat >= 0 ? (uint32_t)(mat * P) * row_of<F>(gbits) : kVacuum;
                    L.plo = L.pspan = 0u;
                }
            }
        }
    }
    if (__float_as_uint(p2f) - L.plo >= L.pspan) {
        if (p2 < R.pmin2) {
            L.status = MT_ST_PMIN;
            L.steps = k;
            return false;
        }
        uint2 r;
        if constexpr ((F & kWide) != 0) r = band_between(S.edge[0], S.edge[P]);
        else r = S.band[T.hist.n_mat * P];
        if (L.hoff != kVacuum) {
            const int h0 = S.mat[L.vol] * P, guess = (int)hist_of<F>(L, gbits) - h0;
            uint32_t h;
            if constexpr ((F & kWide) != 0) {
                const int i = find_bin_wide(S, P, p2, __float_as_uint(p2f), guess);
                h = (uint32_t)(h0 + i);
                r = band_between(S.edge[i], S.edge[i + 1]);
            } else {
                h = (uint32_t)(h0 + find_bin(S, P, p2, guess));
                r = S.band[h];
            }
            L.hoff = h * row_of<F>(gbits);
            if constexpr ((F & kAlias) == 0) L.tot = S.tot[h];
        }
        L.plo = r.x;
        L.pspan = r.y;
    }
    return true;
}

// Large tables: a muon that went into a lower bin of the same volume, one or several
// below its own, walks down the ends of the bands (those at the threshold or below
// are one and the same: a muon that stops does not walk them).  The bin is the
// histogram's index modulo n_pbin, an exact division by multiplication.
template <unsigned F>
__device__ __forceinline__ void lower_bin(Lane &L, uint32_t pb, const KArgs &A) {
    const char *lds = lds_base();
    const uint32_t *edge = reinterpret_cast<const uint32_t *>(lds + A.T.lds.off_band);
    if ((pb < L.plo) & (L.hoff != kVacuum) & (pb > edge[0])) {
        const uint32_t h = hist_of<F>(L, A.T.hist.gbits);
        const uint32_t bin =
            h - __umulhi(h + 1u, A.pbin_magic) * (uint32_t)A.T.hist.n_pbin;
        uint32_t i = max(bin, 1u) - 1u, lo = edge[i], hi = edge[i + 1u];
        while ((pb <= lo) & (i > 0u)) {
            hi = lo;
            lo = edge[--i];
        }
        const uint2 r = band_between(lo, hi);
        if (pb - r.x < r.y) {
            L.hoff -= (bin - i) * row_of<F>(A.T.hist.gbits);
            if constexpr ((F & kAlias) == 0)
                L.tot = reinterpret_cast<const uint32_t *>(lds + A.T.lds.off_tot)[h - (bin - i)];
            L.plo = r.x;
            L.pspan = r.y;
        }
    }
}

// A muon that went into the next lower bin of the same volume (3-4 % of steps,
// so some lane of a wavefront in most of them): the histogram before its own,
// whose band is above the threshold.  A momentum below a material's bin 0 is
// below that row's band too.
template <unsigned F>
__device__ __forceinline__ void next_lower_bin(Lane &L, uint32_t pb, const KArgs &A) {
    if constexpr ((F & kWide) != 0) return lower_bin<F>(L, pb, A);
    if ((pb < L.plo) & (L.hoff != kVacuum)) {
        const uint32_t h = max(hist_of<F>(L, A.T.hist.gbits), 1u) - 1u;
        const char *lds = lds_base();
        const uint2 r = reinterpret_cast<const uint2 *>(lds + A.T.lds.off_band)[h];
        if (pb - r.x < r.y) {
            L.hoff -= row_of<F>(A.T.hist.gbits);
            if constexpr ((F & kAlias) == 0)
                L.tot = reinterpret_cast<const uint32_t *>(lds + A.T.lds.off_tot)[h];
            L.plo = r.x;
            L.pspan = r.y;
        }
    }
}

template <unsigned F>
__device__ __forceinline__ uint2 sampler_entry(const DevHist &H, uint32_t hoff, uint32_t w0) {
    if constexpr ((F & kAlias) != 0) return alias_entry(H, hoff, w0);
    else return guide_entry(H, hoff, w0);
}

// var() gives the lane's variant, words(k) the Philox words of step k.
template <unsigned F, typename V, typename W>
__device__ __forceinline__ bool advance(Lane &L, int64_t g, V &&var, W &&words, int k,
                                        const KArgs &A, ArgPtr args, const StepConst &sc) {
    constexpr bool TAPE = (F & kTape) != 0, TRACE = (F & kWide) != 0, VERT = (F & kVert) != 0;
    const DevHist &H = A.T.hist;
    const DevRun &R = A.R;
    const double p2 = L.px * L.px + L.py * L.py + L.pz * L.pz;
    const float p2f = (float)p2;
    bool outside;
    if constexpr ((F & kPoly) != 0) outside = outside_planes(L, k);
    else outside = outside_region(L, k);
    outside |= k >= R.max_steps;
    const uint32_t pb = __float_as_uint(p2f);
    if (outside | (pb - L.plo >= L.pspan)) {
        // |p| so small or large that the step's FP32 arithmetic may give positions
        // that are not finite: everything in FP64
        outside |= !((p2f >= kBandLow) & (p2f < INFINITY));
        if (!outside) next_lower_bin<F>(L, pb, A);
        if (outside | (pb - L.plo >= L.pspan)) {
            if (!locate_region<F>(L, var, k, p2, p2f, outside, args)) return false;
        }
    }
    float ux = 0.0f, uy = 0.0f, uz = 0.0f;
    int cell = -1, bin = -1;
    if (TRACE && L.hoff != kVacuum) bin = (int)(hist_of<F>(L, H.gbits) % (uint32_t)H.n_pbin);
    if (L.hoff != kVacuum) {
        uint4 w;
        uint2 e;
        if constexpr (!kAhead<F>) {
            w = words(k);
            e = sampler_entry<F>(H, L.hoff, w.x);
        } else {
            if (L.eh != L.hoff) {        // a new volume, or a bin not foreseen
                if (L.eh == kVacuum) L.w = words(k);
                L.e = sampler_entry<F>(H, L.hoff, L.w.x);
            }
            w = L.w;
            e = L.e;
        }
        if constexpr ((F & kAlias) != 0) cell = alias_cell(H, e, w);
        else cell = sample_cell(H, e, L.hoff, L.tot, w.x);
        // loss index = floor(cell / n_scat) = floor((cell + 1/2) / n_scat) in
        // FP32: exact for cell < 2^16 and every n_scat (the quotient is at
        // least 1 / (2 n_scat) from an integer, its error below 2^-6 / n_scat)
        const float cf = (float)cell;
        const float il = floorf(fmaf(cf, H.nscat_inv, 0.5f * H.nscat_inv));
        const float is = fmaf(-il, H.nscat_f, cf);
        // index + jitter: the product with 2^-24 is exact, one rounding
        const float v1 = fmaf((float)(w.y >> 8), 0x1p-24f, il);
        const float v2 = fmaf((float)(w.z >> 8), 0x1p-24f, is);
        const float v3 = (float)(w.w >> 8) * 0x1p-24f;
        float f = fmaf(v1, H.loss_w, H.loss_lo);
        float tau = fmaf(v2, H.scat_w, H.scat_lo);
        if constexpr ((F & kLog) != 0) {      // jitter uniform in log10 of the value
            // 10^u = 2^(u log2 10) on the hardware exp2 (relative error ~1e-6
            // for |u| <= 7, far inside the FP32 kick arithmetic around it)
            constexpr float kLog2Of10 = 3.32192809488736f;
            if (H.log_loss) f = __builtin_amdgcn_exp2f(f * kLog2Of10);
            if (H.log_scat) tau = __builtin_amdgcn_exp2f(tau * kLog2Of10);
        }
        // v_sin_f32 / v_cos_f32 take their argument in revolutions: sin(2 pi v3).
        const float sn = __builtin_amdgcn_sinf(v3);
        const float cs = __builtin_amdgcn_cosf(v3);
        ux = tau * cs;
        uy = tau * sn;
        uz = -f;
        kick(L, p2f, ux, uy, uz);
        if constexpr (kAhead<F>) {
            // The next step's words, and its table entry on its way while this
            // step's Runge-Kutta stages run: they turn the momentum and keep
            // its size, so the bin of the kicked momentum is the next step's
            // but for rounding (and a new volume), which the next step checks.
            const uint32_t q = __float_as_uint(norm2(stage0(L)));
            if (q - L.plo >= L.pspan) next_lower_bin<F>(L, q, A);
            L.w = words(k + 1);
            L.e = sampler_entry<F>(H, L.hoff, L.w.x);
            L.eh = L.hoff;
        }
    } else {
        L.eh = kVacuum;
    }
    if constexpr (TAPE) {   // the local kick; the replay finds the volume again from the state
        float *t = R.tape + ((size_t)k * R.lanes + g) * 3;
        t[0] = ux;
        t[1] = uy;
        t[2] = uz;
    }
    if (TRACE && R.n_trace > 0 && g < R.n_trace && k < R.trace_steps) {
        int32_t *tr = R.trace + ((size_t)g * R.trace_steps + k) * 3;
        tr[0] = L.vol;
        tr[1] = bin;
        tr[2] = cell;
    }
    const float3 b = make_float3(L.bx, L.by, L.bz);
    if constexpr (kScaledField<F>) {
        rk4_from<VERT>(L, stage0(L), b, L.bent, sc);
    } else {
        const float3 B = with_map<F>(L, A, args, b, L.x, L.y, L.z);
        if constexpr ((F & kStages) != 0) rk4_stages<F>(L, var, B, A, args, sc);
        else rk4_from<VERT>(L, stage0(L), scale_field<VERT>(L.kq, B), non_zero<VERT>(B), sc);
    }
    return true;
}

__device__ __forceinline__ StepConst step_const(const DevRun &R) {
    StepConst c;
    c.h = (float)R.h;
    c.h2 = (float)(0.5 * R.h);
    c.h6 = (float)(R.h / 6.0);
    c.h3 = (float)(R.h / 3.0);
    return c;
}

template <bool V, class IO>
__device__ __forceinline__ void store_lane(const Lane &L, int64_t g, const IO &io) {
    io.ox[g] = L.x;
    io.oy[g] = lane_y<V>(L);
    io.oz[g] = L.z;
    io.opx[g] = L.px;
    io.opy[g] = lane_py<V>(L);
    io.opz[g] = L.pz;
    io.status[g] = L.status;
    io.n_steps[g] = L.steps;
    io.volume[g] = L.status == MT_ST_INVALID ? -1 : L.vol;
}

template <bool V>
__device__ __forceinline__ void write_ckpt(const Lane &L, int64_t g, int k, const DevRun &R) {
    double *c = R.ckpt + (size_t)(k / kCkptEvery) * 6 * R.lanes + g;
    c[0] = L.x;
    c[R.lanes] = lane_y<V>(L);
    c[2 * R.lanes] = L.z;
    c[3 * R.lanes] = L.px;
    c[4 * R.lanes] = lane_py<V>(L);
    c[5 * R.lanes] = L.pz;
}

// ---------------------------------------------------------------------------
// Plain form: one lane per (variant, muon) until it stops.
//
// With a general trilinear map held over the step, the lane's 24 cached
// interpolation values leave the kernel near the 96 registers that 5 waves/SIMD
// allow; where more than 4 waves a SIMD run, 5 waves took 11 % less time than 4
// on the shield (140 -> 124 ms before the vertical kernels, which need 72).
// With fewer to run the registers serve better (kRoom).
//
// Convex blocks without a map take 116 registers by themselves; held to 96 (5
// waves) they keep a few values of the cold lookup in scratch.  That pays where
// the fifth wave saves a dispatch round (300 000 muons 4.79 -> 3.78 ms) and past 8
// waves a SIMD, where blocks end at many times (530 000 7.01 -> 6.45, 655 361 7.75 ->
// 7.14, 780 000 8.68 -> 8.51, 10^6 11.15 -> 10.91, 3 10^6 29.5 -> 27.9; of 15 sizes
// only 700 000 lost, 8.08 -> 8.21), not with at most 4 waves a SIMD to run (250 000
// 3.20 -> 3.36, 100 000 2.49 -> 2.66) or 5 to 8 (400 000 5.83 -> 5.97, 500 000 6.69 ->
// 6.74): those run the kernels of kRoom.  Nor with aliases (10^6 10.29 -> 10.52).
// ---------------------------------------------------------------------------
constexpr bool blocks_alone(unsigned F) { return (F & kPoly) && !(F & (kMap | kAlias)); }

constexpr int plain_min_waves(unsigned F) {
    if (F & kRoom) return 1;
    return blocks_alone(F) || ((F & kMap) && !(F & (kStages | kNearest | kTape))) ? 5 : 1;
}

template <unsigned F>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(plain_min_waves(F))))
k_plain(KArgs A) {
    constexpr bool CKPT = (F & kTape) != 0;
    const ArgPtr args = kernel_args();
    const DevRun &R = A.R;
    stage_tables<(F & kWide) != 0>(A.T, R.pmin2);
    const StepConst sc = step_const(R);
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= R.lanes) return;
    Lane L;
    load_lane(L, g, A);
    if (L.status == MT_ST_RUNNING) {
        auto var = [&] { return (int)variant_of(g, cold(args)->R); };
        auto words = [&](int step) { return philox_step(L.ph, (uint32_t)step, R.key0, R.key1); };
        for (int k = 0;; ++k) {
            if (CKPT && (k % kCkptEvery) == 0 && k < R.max_steps) write_ckpt<(F & kVert) != 0>(L, g, k, R);
            if (!advance<F>(L, g, var, words, k, A, args, sc)) break;
        }
    }
    store_lane<(F & kVert) != 0>(L, g, cold(args)->io);
}

// ---------------------------------------------------------------------------
// Compacting form: step-synchronised passes.
//
// The whole batch advances in passes of S steps: pass p takes every muon
// still in flight from step p S to step (p + 1) S (the last pass runs to the
// step cap), and the muons still running there are compacted into the list
// the next pass runs on, so every wave of a pass starts full.
// Muons in flight at any time are within S steps of each other, i.e. at
// about the same depth in z, so the part of a field map they read is a slab
// of the map, not the whole map: its lines stay in the caches instead of
// streaming from HBM.  A wave of a pass runs at most S steps, so lanes
// whose muon stops early idle for at most S steps.
//
// One lane per item as in the plain form (item i of the pass: lane i of the
// launch in the first pass, entry i of the previous pass's list after it).
// Every lane stores its muon in its output slot as the plain form does; a
// muon still running at the pass's end is stored there too (status running, its step
// count, its state) and its slot is appended to the list, with one atomic
// add per wavefront (ballot, then each lane at the wave's base + the
// survivors of lower lanes) and no block barrier, so a wave that is done
// leaves at once.  The next pass resumes the muon from its output slot.
// Results are bit-identical to the plain form: the random stream is keyed by
// (muon, step), the state moves exactly, and the lookup caches are rebuilt
// when a muon is resumed.
// ---------------------------------------------------------------------------

// Lane state of the muon of output slot g resumed from that slot.
__device__ __forceinline__ void resume_lane(Lane &L, int64_t g, const KArgs &A) {
    const DevIO &io = A.io;
    load_lane(L, g, A);                     // charge, Philox prefix, caches reset
    L.x = io.ox[g];
    L.y = io.oy[g];
    L.z = io.oz[g];
    L.px = io.opx[g];
    L.py = io.opy[g];
    L.pz = io.opz[g];
    L.status = MT_ST_RUNNING;
}

template <unsigned F>     // F never holds kTape
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(plain_min_waves(F))))
k_pass(KArgs A) {
    const ArgPtr args = kernel_args();
    const DevRun &R = A.R;
    const PassArgs &P = A.P;
    // items of this pass: the launch's lanes (first pass) or the survivors
    // of the previous pass, whose count that pass left in memory
    const int64_t items = P.n_in ? (int64_t)*P.n_in : R.lanes;
    if ((int64_t)blockIdx.x * blockDim.x >= items) return;     // the whole block
    stage_tables<(F & kWide) != 0>(A.T, R.pmin2);
    const StepConst sc = step_const(R);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    bool parked = false;        // still running at the pass's end: goes on in the next pass
    int64_t slot = 0;           // its output slot
    if (i < items) {
        Lane L;
        if (P.n_in) resume_lane(L, P.in[i], A);
        else load_lane(L, i, A);
        // The pass ends where R.max_steps says (the host sets it to the
        // pass's last step, or to the step cap in the last pass), so the
        // step loop is the plain form's: a muon that meets no other break
        // condition at the pass's end stops with the step-cap status, and
        // is parked here if the real cap lies beyond.  The break test it
        // passed there is the one the next pass repeats at the same step.
        if (L.status == MT_ST_RUNNING) {
            // the output slot, which only traces need in the loop
            const int64_t g = (F & kWide) && P.n_in ? P.in[i] : i;
            auto var = [&] {
                const ArgPtr c = cold(args);
                return (int)variant_of(c->P.n_in ? c->P.in[i] : i, c->R);
            };
            auto words = [&](int step) {
                return philox_step(L.ph, (uint32_t)step, R.key0, R.key1);
            };
            for (int k = P.k_begin;; ++k) {
                if (!advance<F | kPasses>(L, g, var, words, k, A, args, sc)) break;
            }
        }
        const ArgPtr c = cold(args);
        if (L.status == MT_ST_MAXSTEPS && L.steps < c->P.max_steps) {
            parked = true;
            L.status = MT_ST_RUNNING;
        }
        // the slot is read again rather than kept in registers over the loop
        slot = c->P.n_in ? c->P.in[i] : i;
        store_lane<(F & kVert) != 0>(L, slot, c->io);         // status running if parked
    }
    // wave-aggregated append of the survivors' slots (no block barrier: a
    // wave that is done leaves at once and frees its registers for the next)
    const uint64_t m = __ballot(parked);
    if (m) {
        const ArgPtr c = cold(args);
        unsigned long long base = 0;
        if ((threadIdx.x & (kWave - 1)) == 0)
            base = atomicAdd(c->P.n_out, (unsigned long long)__popcll(m));
        base = __builtin_amdgcn_readfirstlane((uint32_t)base) |
               ((unsigned long long)__builtin_amdgcn_readfirstlane((uint32_t)(base >> 32)) << 32);
        if (parked) {
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
                (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            c->P.out[base + rank] = slot;
        }
    }
}

// ---------------------------------------------------------------------------
// Variant-wave form (field variants of the same muons).  All variants of
// muon j draw the same random words at step k, so G lanes that hold G
// variants of one muon need one Philox block per step, not G.  G is the
// largest power of two that divides the variant count, at most 64 (the
// design scan's 64 variants give G = 64: a whole wavefront per muon).  Every
// G steps lane l forms the block of step k + (l mod G) for its group's muon
// into the wavefront's 1 KB of LDS, and at step k every lane reads its
// group's entry k mod G (one address per group, which the LDS broadcasts;
// the wavefront's own LDS writes and reads are executed in order, so only
// the compiler's ordering needs a wave barrier).  The lanes of a wavefront step in lockstep (all start at step 0,
// and each pass of the loop is one step for every lane still running), which
// is what makes the shared block the right one; a lane whose muon has
// stopped still forms its block for the others.  Wavefront w takes the
// 64 / G consecutive (muon, group of G variants) units from w 64 / G on.
// Results are bit-identical to the other forms (same words, same arithmetic,
// same output slots).
//
// Lone muons (DevRun::solo, small launches of the other forms): a group of G
// lanes belongs to one muon that its first lane carries; the others only form
// its random words, one step of G each.
// ---------------------------------------------------------------------------
//
// Convex blocks without a map: the kernel that forms draws ahead runs few waves (lone
// muons, and launches of at most 5 waves a SIMD) and takes the registers it wants;
// the other is held to 5 waves, as the plain form is (8 variants of 50 000 muons 3.60 ->
// 3.48 ms, 16 of 50 000 5.52 -> 5.02, 64 of 100 000 28.4 -> 24.6; 16 of 22 000, 5.4 waves
// a SIMD, 2.90 and 2.91).
constexpr int waves_min_waves(unsigned F, bool ahead) {
    if ((F & kPoly) && !(F & kMap)) return ahead ? 1 : 5;
    return (F & (kMap | kStages)) ? plain_min_waves(F) : (F & kVert) && !ahead ? 7 : 6;
}

template <unsigned F, bool AHEAD>     // kTape for lone muons only
__global__ void __launch_bounds__(1024)
    __attribute__((amdgpu_waves_per_eu(waves_min_waves(F, AHEAD))))
k_variant_waves(KArgs A) {
    const ArgPtr args = kernel_args();
    const DevRun &R = A.R;
    stage_tables<(F & kWide) != 0>(A.T, R.pmin2);
    const StepConst sc = step_const(R);
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int gs = R.share_shift, gm = (1 << gs) - 1;   // G = 2^gs lanes per muon
    const int64_t n = R.n;
    const int64_t vgroups = R.solo ? 1 : (R.lanes / n) >> gs;    // groups of G variants per muon
    const int64_t units = R.solo ? R.lanes : n * vgroups;
    // the first unit of the wavefront is the same for all its lanes
    const int64_t first = ((int64_t)blockIdx.x * (blockDim.x / kWave) +
                           __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave))) *
                          (kWave >> gs);
    if (first >= units) return;
    const int64_t unit = first + (lane >> gs);
    const bool in_range = unit < units;                // the last wavefront may be ragged
    int64_t j = 0, var = 0;
    if (in_range) {
        if (R.solo) {
            var = variant_of(unit, R);
            j = unit - var * n;
        } else {
            j = unit / vgroups;
            var = (unit - j * vgroups) * (gm + 1) + (lane & gm);
        }
    }
    const bool valid = in_range && (!R.solo || (lane & gm) == 0);
    Lane L;
    bool running = false;
    if (valid) {
        load_lane_at(L, j, A);
        running = L.status == MT_ST_RUNNING;
    }
    const PhiloxPrefix P =
        philox_prefix((uint32_t)j, (uint32_t)((uint64_t)j >> 32), R.key0, R.key1);
    // the wavefront's Philox blocks: lane l holds its group's block of step
    // k0 + (l mod G), 1 KB of LDS per wavefront; two groups of steps where a
    // step also asks for the next one's words
    uint4 *wblk = reinterpret_cast<uint4 *>(lds_base() + A.T.lds.bytes) +
                  (AHEAD ? 2 : 1) * (threadIdx.x & ~(unsigned)(kWave - 1));
    const int base = lane & ~gm;
    const int64_t g = var * n + j;
    auto var_of = [&] { return (int)var; };
    auto words = [&](int step) {                   // one address per group: a broadcast
        return wblk[(AHEAD ? ((step >> gs) & 1) * kWave : 0) + base + (step & gm)];
    };
    // the wavefront's LDS accesses are executed in order; the wave barriers
    // keep the compiler from moving reads of the group of steps that a write
    // replaces below it, or reads of the new one above it
    auto fill = [&](int k0) {
        __builtin_amdgcn_wave_barrier();
        wblk[(AHEAD ? ((k0 >> gs) & 1) * kWave : 0) + lane] =
            philox_step(P, (uint32_t)(k0 + (lane & gm)), R.key0, R.key1);
        __builtin_amdgcn_wave_barrier();
    };
    if (AHEAD) fill(0);
    for (int k = 0; __ballot(running) != 0; ++k) {
        if ((k & gm) == (AHEAD ? gm : 0)) fill(k + (AHEAD ? 1 : 0));
        if (running) {
            if ((F & kTape) && (k % kCkptEvery) == 0 && k < R.max_steps) write_ckpt<(F & kVert) != 0>(L, g, k, R);
            running = advance<AHEAD ? F : F | kNow>(L, g, var_of, words, k, A, args, sc);
        }
    }
    if (valid) {
        store_lane<(F & kVert) != 0>(L, var * n + j, cold(args)->io);
    }
}

__global__ void k_queue_reset(unsigned long long *queue, double *zero, int64_t n_zero) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *queue = 0ull;
    if (i < n_zero) zero[i] = 0.0;
}

// ---------------------------------------------------------------------------
// Adjoint (pathwise; sampled kicks, decisions and step count held fixed).
//
// Forward step, in the order of the plain kernel:
//   a0 = p + |p| R(p_hat) u                          (kick, if in material)
//   k_i = c n_i x B, n_i = a_i/|a_i|, c = kappa q     (RK4 stages)
//   a1 = a0 + h/2 k1, a2 = a0 + h/2 k2, a3 = a0 + h k3
//   r' = r + h/6 (n0 + 2 n1 + 2 n2 + n3),  p' = a0 + h/6 (k1 + 2 k2 + 2 k3 + k4)
// The reverse sweep maps (lr', lp') to (lr, lp) and accumulates lB . dB/ds
// into the magnet's scale gradient.  The identity part of every Jacobian is
// applied in FP64; the O(h) and O(f, tau) corrections are formed in FP32.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float3 unit_jt(float3 n, float rinv, float3 l) {
    // (I - n n^T) l / |a|
    const float d = fmaf(n.x, l.x, fmaf(n.y, l.y, n.z * l.z));
    return make_float3(rinv * fmaf(-d, n.x, l.x), rinv * fmaf(-d, n.y, l.y),
                       rinv * fmaf(-d, n.z, l.z));
}

__device__ __forceinline__ float dot3(float3 a, float3 b) {
    return fmaf(a.x, b.x, fmaf(a.y, b.y, a.z * b.z));
}

// Gradient of l . g_u(p) with g_u(p) = p_z u + A x u + (A.u) A / (|p| + p_z),
// A = (-p_y, p_x, 0): the kick is p -> p + g_u(p).
__device__ __forceinline__ float3 kick_adjoint_corr(float3 p, float3 u, float3 l) {
    // hardware reciprocal square root and reciprocal: these are FP32
    // corrections to an FP64 adjoint, where 1-ulp accuracy is ample
    const float p2 = norm2(p);
    const float invP = __builtin_amdgcn_rsqf(p2);
    const float P = p2 * invP;
    const float D = P + p.z;
    const float alpha = fmaf(-p.y, u.x, p.x * u.y);
    const float beta = fmaf(-p.y, l.x, p.x * l.y);
    const float3 v = cross3(u, l);
    const float invD = __builtin_amdgcn_rcpf(D);
    const float Q = alpha * beta * invD;
    float3 g;
    g.x = v.y + (beta * u.y + alpha * l.y) * invD - Q * invD * (p.x * invP);
    g.y = -v.x + (-beta * u.x - alpha * l.x) * invD - Q * invD * (p.y * invP);
    g.z = dot3(l, u) - Q * invD * (p.z * invP + 1.0f);
    return g;
}

// d(trilinear)/dr contracted with lB.
template <bool V>
__device__ __forceinline__ float3 map_grad_t(const DevField &F, const CellPoly &c, float3 lB) {
    // lB . k_q for the seven non-constant coefficients, then the partial
    // derivatives of the cell polynomial in fx, fy, fz
    auto dot4 = [&](float4 a) {
        if constexpr (V) return lB.y * a.y;
        else return fmaf(lB.x, a.x, fmaf(lB.y, a.y, lB.z * a.z));
    };
    const float v1 = dot4(c.k[1]), v2 = dot4(c.k[2]), v3 = dot4(c.k[3]), v4 = dot4(c.k[4]);
    const float v5 = dot4(c.k[5]), v6 = dot4(c.k[6]), v7 = dot4(c.k[7]);
    const float dx = fmaf(c.fy, fmaf(c.fz, v7, v4), fmaf(c.fz, v5, v1));
    const float dy = fmaf(c.fx, fmaf(c.fz, v7, v4), fmaf(c.fz, v6, v2));
    const float dz = fmaf(c.fx, fmaf(c.fy, v7, v5), fmaf(c.fy, v6, v3));
    return make_float3(dx * (float)F.inv_d[0], dy * (float)F.inv_d[1], dz * (float)F.inv_d[2]);
}

// Products of the reverse sweep with a field that may be vertical: b x l, and
// l x n where only its y component will count.
template <bool V>
__device__ __forceinline__ float3 field_cross(float3 b, float3 l) {
    if constexpr (V) return make_float3(b.y * l.z, 0.0f, -b.y * l.x);
    else return cross3(b, l);
}

template <bool V>
__device__ __forceinline__ float3 field_grad(float3 l, float3 n) {
    if constexpr (V) return make_float3(0.0f, fmaf(l.z, n.x, -l.x * n.z), 0.0f);
    else return cross3(l, n);
}

template <bool V>
__device__ __forceinline__ float3 add_field_grad(float3 a, float3 b) {
    if constexpr (V) return make_float3(0.0f, a.y + b.y, 0.0f);
    else return add3(a, b);
}

// One reverse step: (lr, lp) of the state after step k -> before step k, and
// the step's contribution to the scale gradient of its magnet.  p0 is the
// momentum at the start of the step (FP32 is enough for Jacobians), (rx, ry,
// rz) its position (used only with a field map).
// V: every field is vertical (b.x = b.z = 0), so of lB, the gradient of the
// field, only the y component counts, and the products with the field have no
// y component: the general form's values without the multiplications by zero
// (10^6-muon design step: adjoint kernel 3.39 -> 2.95 ms, near the 2.6 ms its
// 51 bytes a step take at copy bandwidth).
template <bool MAP, bool V>
__device__ __forceinline__ void reverse_step(const Tables &T, const Lds &S, const DevRun &R,
                                             const StepConst &sc, float kq, float3 p0, float3 a0,
                                             double rx, double ry, double rz, int vol, float3 u,
                                             float3 Bbox, double lr[3], double lp[3], int &mag_out,
                                             double &dsg) {
    const int mat = vol >= 0 ? S.mat[vol] : -1;
    const float3 B = add_map<MAP>(T, Bbox, rx, ry, rz);
    const float3 Lr = make_float3((float)lr[0], (float)lr[1], (float)lr[2]);
    const float3 Lp = make_float3((float)lp[0], (float)lp[1], (float)lp[2]);
    // RK4 stages of the step (the straight-line shortcut of the forward pass
    // equals them at B = 0, so one form serves both).
    const float3 cb = scale_field<V>(kq, B);
    const float r0 = __builtin_amdgcn_rsqf(norm2(a0));
    const float3 n0 = scale3(r0, a0);
    const float3 k1v = cross_field<V>(n0, cb);
    const float3 a1 = axpy_field<V>(sc.h2, k1v, a0);
    const float r1 = __builtin_amdgcn_rsqf(norm2(a1));
    const float3 n1 = scale3(r1, a1);
    const float3 k2v = cross_field<V>(n1, cb);
    const float3 a2 = axpy_field<V>(sc.h2, k2v, a0);
    const float r2 = __builtin_amdgcn_rsqf(norm2(a2));
    const float3 n2 = scale3(r2, a2);
    const float3 k3v = cross_field<V>(n2, cb);
    const float3 a3 = axpy_field<V>(sc.h, k3v, a0);
    const float r3 = __builtin_amdgcn_rsqf(norm2(a3));
    const float3 n3 = scale3(r3, a3);
    // Reverse through k4 = c n3 x B, a3 = a0 + h k3, ..., k1 = c n0 x B.
    float3 lk3 = scale3(sc.h3, Lp);
    float3 lk2 = scale3(sc.h3, Lp);
    float3 lk1 = scale3(sc.h6, Lp);
    const float3 lk4 = scale3(sc.h6, Lp);
    float3 lBc = field_grad<V>(lk4, n3);
    float3 la = unit_jt(n3, r3, axpy(sc.h6, Lr, field_cross<V>(cb, lk4)));
    float3 corr = la;
    lk3 = axpy(sc.h, la, lk3);
    lBc = add_field_grad<V>(lBc, field_grad<V>(lk3, n2));
    la = unit_jt(n2, r2, axpy(sc.h3, Lr, field_cross<V>(cb, lk3)));
    corr = add3(corr, la);
    lk2 = axpy(sc.h2, la, lk2);
    lBc = add_field_grad<V>(lBc, field_grad<V>(lk2, n1));
    la = unit_jt(n1, r1, axpy(sc.h3, Lr, field_cross<V>(cb, lk2)));
    corr = add3(corr, la);
    lk1 = axpy(sc.h2, la, lk1);
    lBc = add_field_grad<V>(lBc, field_grad<V>(lk1, n0));
    la = unit_jt(n0, r0, axpy(sc.h6, Lr, field_cross<V>(cb, lk1)));
    corr = add3(corr, la);
    const float3 lB = scale_field<V>(kq, lBc);
    // lambda of a0 (post-kick momentum), then through the kick
    double la0[3] = {lp[0] + (double)corr.x, lp[1] + (double)corr.y, lp[2] + (double)corr.z};
    if (mat >= 0) {
        const float3 l = make_float3((float)la0[0], (float)la0[1], (float)la0[2]);
        const float3 kc = kick_adjoint_corr(p0, u, l);
        la0[0] += (double)kc.x;
        la0[1] += (double)kc.y;
        la0[2] += (double)kc.z;
    }
    lp[0] = la0[0];
    lp[1] = la0[1];
    lp[2] = la0[2];
    mag_out = -1;
    dsg = 0.0;
    if (vol >= 0) {
        const int m = S.mag[vol];
        if (m >= 0) {
            const float4 b = S.bf[vol];
            mag_out = m;
            dsg = V ? (double)(lB.y * b.y)
                    : (double)fmaf(lB.x, b.x, fmaf(lB.y, b.y, lB.z * b.z));
        }
    }
    if (MAP) {
        CellPoly cc;
        if (map_cell(T.field, rx, ry, rz, cc)) {
            const float3 gr = map_grad_t<V>(T.field, cc, lB);
            lr[0] += (double)gr.x;
            lr[1] += (double)gr.y;
            lr[2] += (double)gr.z;
        }
    }
}

// One FP32 momentum of the adjoint's segment history (12 bytes, so a
// wavefront's records of a step are one contiguous 768-byte run).
struct Float3r {
    float x, y, z;
};

// The stage-0 momentum of a step formed again from its FP32 pre-kick
// momentum: the forward's kick arithmetic on (double)p0 instead of the FP64
// state it was rounded from.  It agrees with the forward's a0 to the last bit
// or, rarely, one unit in the last place (the FP64 state and its FP32
// rounding differ by ~1e-8 relative), which is what the FP32 Jacobians
// built from it need.
__device__ __forceinline__ float3 kick_again(float3 p0, float3 u) {
    Lane K;
    K.px = (double)p0.x;
    K.py = (double)p0.y;
    K.pz = (double)p0.z;
    const double p2 = K.px * K.px + K.py * K.py + K.pz * K.pz;
    kick(K, (float)p2, u.x, u.y, u.z);
    return stage0(K);
}

// Re-run one step of a segment with its recorded kick (the arithmetic of
// advance(), so the same bits).  The volume is looked up again from the
// state, which is the forward's to the bit, so it is the forward's volume.
// Returns the volume.
template <bool MAP, bool V>
__device__ __forceinline__ int replay_step(Lane &L, int k, const Tables &T, const Lds &S,
                                           const DevRun &R, const StepConst &sc, int var,
                                           float3 u) {
    if (outside_region(L, k)) {
        const int vol = locate_box(L, T, S);
        if (!table_region(L, vol, T, S)) set_region(L, box_region(L, vol, S), T.geom);
        if (vol != L.vol) {
            L.vol = vol;
            const float3 b = box_field<V>(T, S, R, vol, var);
            L.bent = non_zero<V>(b);
            const float s = MAP ? 1.0f : L.kq;
            L.bx = s * b.x;
            L.by = s * b.y;
            L.bz = s * b.z;
            L.hoff = vol >= 0 && S.mat[vol] >= 0 ? 0u : kVacuum;
        }
    }
    if (L.hoff != kVacuum) {
        const double p2 = L.px * L.px + L.py * L.py + L.pz * L.pz;
        kick(L, (float)p2, u.x, u.y, u.z);
    }
    const float3 b = make_float3(L.bx, L.by, L.bz);
    if (MAP) {
        const float3 B = add_map<MAP>(T, b, L.x, L.y, L.z);
        rk4_from<V>(L, stage0(L), scale_field<V>(L.kq, B), non_zero<V>(B), sc);
    } else {
        rk4_from<V>(L, stage0(L), b, L.bent, sc);
    }
    return L.vol;
}

// The segment's start momenta are kept either in LDS (LDSH) or in a per-lane
// scratch area in device memory; with a field map the start positions are
// needed too and always go to the scratch area.
// Without a map the kernel takes 89 VGPRs for vertical fields and 96 for general
// ones: 5 waves/SIMD, which the bound keeps (when the kernel took 103, 5 waves with a
// few values in scratch were 3 % faster than 4; now it gives the same time with the
// bound and without: design step of 10^6 muons 3.00 ms in the adjoint, 200 000 in
// general fields 1.34 ms with the forward).
template <bool MAP, bool LDSH, bool V>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MAP ? 1 : 5)))
k_adjoint(Tables T, DevRun R, DevIO io, const double *g_out,
                                                 double *g_in, double *gs_lane, char *scratch) {
    stage_tables<true>(T, R.pmin2);
    const Lds S = lds_view<true>(T);
    char *smem = lds_base();
    const StepConst sc = step_const(R);
    const int bd = blockDim.x;
    const int n_mag = T.geom.n_mag;
    double *sgs = reinterpret_cast<double *>(smem + ((T.lds.bytes + 15) & ~15)) + threadIdx.x;
    float *hist = reinterpret_cast<float *>(smem + ((T.lds.bytes + 15) & ~15) +
                                            (size_t)n_mag * bd * sizeof(double)) + threadIdx.x;
    // volume of every step of the segment, found again by the replay and
    // read back by the reverse sweep: [step][thread], one byte each
    int8_t *vh = reinterpret_cast<int8_t *>(smem + ((T.lds.bytes + 15) & ~15) +
                                           (size_t)n_mag * bd * sizeof(double) +
                                           (LDSH ? (size_t)kCkptEvery * 3 * bd * sizeof(float) : 0)) +
                 threadIdx.x;
    const int64_t g0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = g0 < R.lanes;
    const int64_t g = live ? g0 : R.lanes - 1;   // lanes past the end idle below
    const int64_t lanes = R.lanes;
    for (int m = 0; m < n_mag; ++m) sgs[m * bd] = 0.0;
    double lr[3], lp[3];
    for (int a = 0; a < 3; ++a) {
        lr[a] = g_out[a * lanes + g];
        lp[a] = g_out[(3 + a) * lanes + g];
    }
    const int ns = io.n_steps[g];
    const int status = io.status[g];
    int var = 0;
    if (R.lanes != R.n) var = (int)(g / R.n);
    const float q = (float)io.q[g - (int64_t)var * R.n];
    const float kq = (float)kKappa * q;

    // The lanes of a wavefront walk the checkpoint segments together, from
    // the wavefront's last one down: a lane whose own last segment is lower
    // waits until the walk reaches it.  Lanes then read the same tape and
    // checkpoint rows at the same time (one cache line per 8 lanes), where
    // each lane starting at its own last segment would split a wavefront's
    // reads over several rows.  Every lane's arithmetic and its order are
    // unchanged.
    const int top = (live && status != MT_ST_INVALID && ns > 0) ? (ns - 1) / kCkptEvery : -1;
    int wtop = top;
    for (int o = kWave / 2; o > 0; o >>= 1) wtop = max(wtop, __shfl_xor(wtop, o));
    wtop = __builtin_amdgcn_readfirstlane(wtop);

    {
        for (int seg = wtop; seg >= 0; --seg) {
            if (seg > top) continue;
            const int k0 = seg * kCkptEvery;
            const int k1 = min(k0 + kCkptEvery, ns);
            Lane L;
            const double *c = R.ckpt + (size_t)seg * 6 * lanes + g;
            L.x = c[0];
            L.y = c[lanes];
            L.z = c[2 * lanes];
            L.px = c[3 * lanes];
            L.py = c[4 * lanes];
            L.pz = c[5 * lanes];
            L.kq = kq;
            // kick records of the segment: three floats per (step, lane)
            const float *rec = R.tape + ((size_t)k0 * lanes + g) * 3;
            reset_lane_caches(L, T);     // lookup caches start empty
            // history of the segment: the pre-kick momentum p0 of every step
            // (FP32), [step][3][thread] in LDS (LDSH) or one 12-byte record per
            // (step, lane) in device memory.  The stage-0 momentum a0 is formed
            // again from p0 in the reverse sweep (kick_again), which halves the
            // history traffic the adjoint is bound by.
            float *hp;
            int64_t hs;
            if (LDSH) {
                hp = hist;
                hs = bd;
            } else {
                hp = nullptr;
                hs = 0;
            }
            Float3r *h3 = reinterpret_cast<Float3r *>(scratch) + g;
            double *hr = reinterpret_cast<double *>(
                scratch + (size_t)kCkptEvery * sizeof(Float3r) * lanes) + g;
            // running pointers (one 64-bit add per array and step) rather
            // than (k - k0) * lanes products
            const size_t rs = (size_t)lanes * 3;     // record stride between steps
            const float *rp = rec;
            Float3r *h3p = h3;
            double *hrp = hr;
            float3 next = make_float3(rp[0], rp[1], rp[2]);
            for (int k = k0; k < k1; ++k) {
                const float3 cur = next;
                rp += rs;
                if (k + 1 < k1) next = make_float3(rp[0], rp[1], rp[2]);
                const float p0x = (float)L.px, p0y = (float)L.py, p0z = (float)L.pz;
                if (MAP) {
                    hrp[0] = L.x;
                    hrp[lanes] = L.y;
                    hrp[2 * lanes] = L.z;
                    hrp += 3 * lanes;
                }
                vh[(k - k0) * bd] = (int8_t)replay_step<MAP, V>(L, k, T, S, R, sc, var, cur);
                if (LDSH) {
                    float *h = hp + (size_t)(k - k0) * 3 * hs;
                    h[0] = p0x;
                    h[hs] = p0y;
                    h[2 * hs] = p0z;
                } else {
                    *h3p = Float3r{p0x, p0y, p0z};
                    h3p += lanes;
                }
            }
            int bvol = -2;
            float3 bb = make_float3(0.f, 0.f, 0.f);
            int acc_m = -1;
            double acc = 0.0;
            // the reverse sweep loads step k-1's kick record and history
            // while it works on step k
            rp -= rs;                    // step k1 - 1
            h3p -= lanes;
            hrp -= 3 * lanes;
            next = make_float3(rp[0], rp[1], rp[2]);
            Float3r nP{0.f, 0.f, 0.f};
            double nx = 0.0, ny = 0.0, nz = 0.0;
            if (!LDSH) nP = *h3p;
            if (MAP) {
                nx = hrp[0];
                ny = hrp[lanes];
                nz = hrp[2 * lanes];
            }
            for (int k = k1 - 1; k >= k0; --k) {
                const float3 cur = next;
                const Float3r P = nP;
                const double rx = nx, ry = ny, rz = nz;
                if (k > k0) {
                    rp -= rs;
                    next = make_float3(rp[0], rp[1], rp[2]);
                    if (!LDSH) {
                        h3p -= lanes;
                        nP = *h3p;
                    }
                    if (MAP) {
                        hrp -= 3 * lanes;
                        nx = hrp[0];
                        ny = hrp[lanes];
                        nz = hrp[2 * lanes];
                    }
                }
                float3 p0;
                if (LDSH) {
                    const float *h = hp + (size_t)(k - k0) * 3 * hs;
                    p0 = make_float3(h[0], h[hs], h[2 * hs]);
                } else {
                    p0 = make_float3(P.x, P.y, P.z);
                }
                const int vol = vh[(k - k0) * bd];
                const float3 a0 = (vol >= 0 && S.mat[vol] >= 0) ? kick_again(p0, cur) : p0;
                if (vol != bvol) {
                    bb = box_field<V>(T, S, R, vol, var);
                    bvol = vol;
                }
                int m;
                double d;
                reverse_step<MAP, V>(T, S, R, sc, kq, p0, a0, rx, ry, rz, vol,
                                  make_float3(cur.x, cur.y, cur.z), bb, lr, lp, m, d);
                // scale gradient: accumulate in a register while the magnet is unchanged
                if (m != acc_m) {
                    if (acc_m >= 0) sgs[acc_m * bd] += acc;
                    acc_m = m;
                    acc = 0.0;
                }
                acc += d;
            }
            if (acc_m >= 0) sgs[acc_m * bd] += acc;
        }
    }
    if (!live) return;
    for (int a = 0; a < 3; ++a) {
        g_in[a * lanes + g] = lr[a];
        g_in[(3 + a) * lanes + g] = lp[a];
    }
    for (int m = 0; m < n_mag; ++m) gs_lane[(size_t)m * lanes + g] = sgs[m * bd];
}

// ---------------------------------------------------------------------------
// Field map tables from the node values b [nz][ny][nx][3].
// ---------------------------------------------------------------------------
__global__ void k_map_nodes(const float *b, int64_t n, float4 *nodes, float *nodesv) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    nodes[i] = make_float4(b[3 * i], b[3 * i + 1], b[3 * i + 2], 0.f);
    if (nodesv) nodesv[i] = b[3 * i + 1];
}

// One thread per cell: the coefficients of its trilinear interpolant (see
// CellPoly), formed in FP64 from the 8 corner values and rounded.
__global__ void k_map_cells(const float4 *nodes, int nx, int ny, int nz, float4 *map,
                            float4 *mapv) {
    const int64_t cell = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t cx = nx - 1, cy = ny - 1;
    if (cell >= cx * cy * (nz - 1)) return;
    const int64_t i = cell % cx, j = cell / cx % cy, k = cell / (cx * cy);
    float kc[3][8];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double C[8];                             // corner c = dx + 2 dy + 4 dz
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const float4 v = nodes[((k + (c >> 2)) * ny + (j + ((c >> 1) & 1))) * nx + (i + (c & 1))];
            C[c] = (double)(a == 0 ? v.x : a == 1 ? v.y : v.z);
        }
        const double q[8] = {C[0],
                             C[1] - C[0],
                             C[2] - C[0],
                             C[4] - C[0],
                             C[3] - C[1] - C[2] + C[0],
                             C[5] - C[1] - C[4] + C[0],
                             C[6] - C[2] - C[4] + C[0],
                             C[7] - C[3] - C[5] - C[6] + C[1] + C[2] + C[4] - C[0]};
#pragma unroll
        for (int c = 0; c < 8; ++c) kc[a][c] = (float)q[c];
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) map[cell * 8 + c] = make_float4(kc[0][c], kc[1][c], kc[2][c], 0.f);
    if (mapv) {
        mapv[cell * 2] = make_float4(kc[1][0], kc[1][1], kc[1][2], kc[1][3]);
        mapv[cell * 2 + 1] = make_float4(kc[1][4], kc[1][5], kc[1][6], kc[1][7]);
    }
}

// ---------------------------------------------------------------------------
// Deterministic per-variant sums (fixed chunking and fixed tree order).
// ---------------------------------------------------------------------------
constexpr int kRedBlock = 256;

template <int NC, typename F>
__device__ __forceinline__ void block_partial(F &&term, int64_t begin, int64_t end,
                                              double *partial_out) {
    __shared__ double red[NC][kRedBlock];
    double acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = 0.0;
    // eight elements per thread in flight; each accumulator still adds its
    // elements in index order
    int64_t i = begin + threadIdx.x;
    for (; i + 7 * kRedBlock < end; i += 8 * kRedBlock) {
#pragma unroll
        for (int u = 0; u < 8; ++u) term(i + u * kRedBlock, acc);
    }
    for (; i < end; i += kRedBlock) term(i, acc);
#pragma unroll
    for (int c = 0; c < NC; ++c) red[c][threadIdx.x] = acc[c];
    __syncthreads();
    for (int w = kRedBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
#pragma unroll
            for (int c = 0; c < NC; ++c) red[c][threadIdx.x] += red[c][threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
#pragma unroll
        for (int c = 0; c < NC; ++c) partial_out[c] = red[c][0];
    }
}

__global__ void __launch_bounds__(kRedBlock) k_tally_pass1(DevIO io, int64_t n, double z_det,
                                                           double r_ap, double r_scale,
                                                           double *partial) {
    const int v = blockIdx.y, b = blockIdx.x, nb = gridDim.x;
    const int64_t chunk = (n + nb - 1) / nb;
    const int64_t base = (int64_t)v * n;
    const int64_t begin = base + min((int64_t)b * chunk, n);
    const int64_t end = base + min((int64_t)(b + 1) * chunk, n);
    auto term = [&](int64_t i, double *acc) {
        if (io.status[i] == MT_ST_ZMAX) {
            const double dz = z_det - io.oz[i];
            const double xd = io.ox[i] + dz * io.opx[i] / io.opz[i];
            const double yd = io.oy[i] + dz * io.opy[i] / io.opz[i];
            const double r = sqrt(xd * xd + yd * yd);
            acc[0] += 1.0;
            acc[1] += (r < r_ap) ? 1.0 : 0.0;
            acc[2] += 1.0 / (1.0 + exp(-(r_ap - r) / r_scale));
        }
    };
    block_partial<3>(term, begin, end, partial + ((size_t)v * nb + b) * 3);
}

// One block per (chunk b, variant v, column c): each column is summed on
// its own, in the same order and tree as every other column.
__global__ void __launch_bounds__(kRedBlock) k_colsum_pass1(const double *vals, int n_cols,
                                                            int64_t n, int64_t lanes,
                                                            double *partial) {
    const int v = blockIdx.y, b = blockIdx.x, nb = gridDim.x, c = blockIdx.z;
    const int64_t chunk = (n + nb - 1) / nb;
    const int64_t base = (int64_t)v * n;
    const int64_t begin = base + min((int64_t)b * chunk, n);
    const int64_t end = base + min((int64_t)(b + 1) * chunk, n);
    const double *col = vals + (size_t)c * lanes;
    auto term = [&](int64_t i, double *acc) { acc[0] += col[i]; };
    block_partial<1>(term, begin, end, partial + ((size_t)v * nb + b) * n_cols + c);
}

// out[v][c] = sum over b of partial[v][b][c], in order of b.
__global__ void k_pass2(const double *partial, int nb, int n_cols, int n_variants, double *out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_variants * n_cols) return;
    const int v = i / n_cols, c = i - v * n_cols;
    const double *p = partial + (size_t)v * nb * n_cols + c;
    double s = 0.0;
    int b = 0;
    for (; b + 8 <= nb; b += 8) {        // loads of eight partials in flight, sums in order of b
        double t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) t[u] = p[(size_t)(b + u) * n_cols];
#pragma unroll
        for (int u = 0; u < 8; ++u) s += t[u];
    }
    for (; b < nb; ++b) s += p[(size_t)b * n_cols];
    out[i] = s;
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------
template <unsigned F, unsigned ROOM>
static const void *plain_kernel() {
    constexpr bool own = !(F & (kStages | kTape | kWide)) &&
                         (blocks_alone(F) || ((F & kMap) && !(F & kVert)));
    if constexpr (!valid_mask(F)) return nullptr;
    else return reinterpret_cast<const void *>(&k_plain<own ? F | ROOM : F>);
}

template <unsigned F, unsigned ROOM>
static const void *persistent_kernel() {
    constexpr bool own = blocks_alone(F) && !(F & kWide);
    if constexpr (valid_mask(F) && !(F & kTape))
        return reinterpret_cast<const void *>(&k_pass<own ? F | ROOM : F>);
    else return nullptr;
}

// Lone muons (the only use with a tape) are always few: their kernel forms
// draws ahead where it can.  The kernels for large tables do not, and have no tape.
template <unsigned F, bool AHEAD>
static const void *variant_waves_kernel() {
    if constexpr (!valid_mask(F) || ((F & kWide) && (AHEAD || (F & kTape)))) return nullptr;
    else if constexpr (!AHEAD && kAhead<F> && (F & kTape)) return nullptr;
    else return reinterpret_cast<const void *>(&k_variant_waves<F, AHEAD && kAhead<F>>);
}

template <bool AHEAD, size_t... I>
static std::array<const void *, sizeof...(I)> variant_waves_kernels(std::index_sequence<I...>) {
    return {variant_waves_kernel<(unsigned)I, AHEAD>()...};
}

template <unsigned ROOM, size_t... I>
static std::array<const void *, sizeof...(I)> plain_kernels(std::index_sequence<I...>) {
    return {plain_kernel<(unsigned)I, ROOM>()...};
}

template <unsigned ROOM, size_t... I>
static std::array<const void *, sizeof...(I)> persistent_kernels(std::index_sequence<I...>) {
    return {persistent_kernel<(unsigned)I, ROOM>()...};
}

// The tables in the layout of the kernel.
static Tables tables_for(const AllTables &T, bool wide) {
    Tables t = T;
    if (wide) {
        t.lds = T.wide_lds;
        t.image = T.wide_image;
    }
    return t;
}

static uint32_t pbin_magic(const Tables &T) { return 0xFFFFFFFFu / (uint32_t)T.hist.n_pbin; }

static unsigned feature_mask(const AllTables &T, const DevRun &R) {
    const bool map = T.field.map != nullptr, wide = R.wide != 0;
    return (map ? kMap : 0u) | (R.ckpt != nullptr ? kTape : 0u) |
           (wide ? kWide : 0u) | (R.sampler == MT_SAMPLER_ALIAS ? kAlias : 0u) |
           (map && R.interp == MT_INTERP_NEAREST ? kNearest : 0u) |
           (R.stage_field ? kStages : 0u) | (T.geom.n_poly > 0 ? kPoly : 0u) |
           (T.hist.log_loss || T.hist.log_scat ? kLog : 0u) |
           (T.geom.vertical && (!map || T.field.vertical) && !wide ? kVert : 0u);
}

hipError_t launch_plain(const AllTables &T, const DevRun &R, const DevIO &io, int block,
                        hipStream_t s) {
    static const auto many = plain_kernels<0u>(std::make_index_sequence<kFeatures>());
    static const auto few = plain_kernels<kRoom>(std::make_index_sequence<kFeatures>());
    const auto &fns = R.room ? few : many;
    if (R.lanes == 0) return hipSuccess;
    const unsigned grid = (unsigned)((R.lanes + block - 1) / block);
    KArgs a{tables_for(T, R.wide != 0), R, io, PassArgs{}, pbin_magic(T)};
    void *args[] = {&a};
    const void *fn = fns[feature_mask(T, R)];
    if (fn == nullptr) return hipErrorInvalidValue;     // excluded by argument validation
    return hipLaunchKernel(fn, dim3(grid), dim3(block), args, (size_t)a.T.lds.bytes, s);
}

hipError_t launch_pass(const AllTables &T, const DevRun &R, const DevIO &io, int block,
                       const PassArgs &P, hipStream_t s) {
    static const auto many = persistent_kernels<0u>(std::make_index_sequence<kFeatures>());
    static const auto few = persistent_kernels<kRoom>(std::make_index_sequence<kFeatures>());
    const auto &fns = R.room ? few : many;
    if (R.lanes == 0) return hipSuccess;
    // sized for every lane (the survivors of a pass are at most that many);
    // blocks past the pass's items exit before staging their tables
    const unsigned grid = (unsigned)((R.lanes + block - 1) / block);
    KArgs a{tables_for(T, R.wide != 0), R, io, P, pbin_magic(T)};
    void *args[] = {&a};
    const void *fn = fns[feature_mask(T, R) & ~kTape];
    if (fn == nullptr) return hipErrorInvalidValue;     // excluded by argument validation
    return hipLaunchKernel(fn, dim3(grid), dim3(block), args, (size_t)a.T.lds.bytes, s);
}

hipError_t launch_variant_waves(const AllTables &T, const DevRun &R, const DevIO &io, int block,
                               hipStream_t s) {
    static const auto now = variant_waves_kernels<false>(std::make_index_sequence<kFeatures>());
    static const auto ahead = variant_waves_kernels<true>(std::make_index_sequence<kFeatures>());
    const bool draw_ahead = (R.solo || R.ahead) && !R.wide;
    const auto &fns = draw_ahead ? ahead : now;
    if (R.lanes == 0) return hipSuccess;
    // (muon, group of G variants) units, 64 / G per wavefront
    const int64_t units = R.solo ? R.lanes : R.lanes >> R.share_shift;
    const int64_t per_wave = kWave >> R.share_shift;
    const int64_t waves = (units + per_wave - 1) / per_wave;
    const int64_t per_block = block / kWave;
    const unsigned grid = (unsigned)((waves + per_block - 1) / per_block);
    KArgs a{tables_for(T, R.wide != 0), R, io, PassArgs{}, pbin_magic(T)};
    void *args[] = {&a};
    const void *fn = fns[feature_mask(T, R)];
    if (fn == nullptr) return hipErrorInvalidValue;     // excluded by argument validation
    const size_t lds = (size_t)a.T.lds.bytes + (draw_ahead ? 2 : 1) * (size_t)block * sizeof(uint4);
    return hipLaunchKernel(fn, dim3(grid), dim3(block), args, lds, s);
}

hipError_t launch_map_nodes(const float *b, int64_t n, float4 *nodes, float *nodesv,
                            hipStream_t s) {
    hipLaunchKernelGGL(k_map_nodes, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, b, n, nodes,
                       nodesv);
    return hipGetLastError();
}

hipError_t launch_map_cells(const float4 *nodes, int nx, int ny, int nz, float4 *map, float4 *mapv,
                            hipStream_t s) {
    const int64_t cells = (int64_t)(nx - 1) * (ny - 1) * (nz - 1);
    hipLaunchKernelGGL(k_map_cells, dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, s, nodes,
                       nx, ny, nz, map, mapv);
    return hipGetLastError();
}

hipError_t launch_queue_reset(unsigned long long *queue, double *zero, int64_t n_zero,
                              hipStream_t s) {
    const int64_t n = n_zero > 1 ? n_zero : 1;
    hipLaunchKernelGGL(k_queue_reset, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, queue,
                       zero, n_zero);
    return hipGetLastError();
}

int64_t adjoint_scratch_bytes(const Tables &T, int64_t lanes) {
    return (int64_t)kCkptEvery * (sizeof(Float3r) + 3 * sizeof(double)) * lanes;
}

// Where the adjoint keeps a segment's start states: device memory (default;
// at 16 steps x 12 B per lane it stays L2/Infinity-Cache resident and leaves
// LDS free for occupancy) or, on request and without a field map, LDS.
hipError_t launch_adjoint(const AllTables &T, const DevRun &R, const DevIO &io,
                          const double *g_out, double *g_in, double *gs_lane, void *scratch,
                          int block, bool lds_history, hipStream_t s) {
    if (R.lanes == 0) return hipSuccess;
    const int64_t grid = (R.lanes + block - 1) / block;
    const bool map = T.field.map != nullptr;
    const bool ldsh = lds_history && !map;
    const Tables t = tables_for(T, true);      // (it looks no momentum bin up: the smaller image)
    size_t shm = (size_t)((t.lds.bytes + 15) & ~15) + (size_t)T.geom.n_mag * block * sizeof(double);
    if (ldsh) shm += (size_t)kCkptEvery * 3 * block * sizeof(float);   // p0 per step
    shm += (size_t)kCkptEvery * block;                                   // volume per step
    char *sc = reinterpret_cast<char *>(scratch);
    const bool vert = T.geom.vertical && (!map || T.field.vertical);
    auto fn = map    ? (vert ? &k_adjoint<true, false, true> : &k_adjoint<true, false, false>)
              : ldsh ? (vert ? &k_adjoint<false, true, true> : &k_adjoint<false, true, false>)
                     : (vert ? &k_adjoint<false, false, true> : &k_adjoint<false, false, false>);
    hipLaunchKernelGGL(fn, dim3((unsigned)grid), dim3(block), shm, s, t, R, io, g_out, g_in, gs_lane,
                       sc);
    return hipGetLastError();
}

hipError_t launch_tally(const DevIO &io, int64_t n, int32_t n_variants, double z_det,
                        double r_ap, double r_scale, double *partial, int32_t n_part_blocks,
                        double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_tally_pass1, dim3(n_part_blocks, n_variants), dim3(kRedBlock), 0, s, io,
                       n, z_det, r_ap, r_scale, partial);
    const int nout = n_variants * 3;
    hipLaunchKernelGGL(k_pass2, dim3((nout + 127) / 128), dim3(128), 0, s, partial, n_part_blocks,
                       3, n_variants, out);
    return hipGetLastError();
}

hipError_t launch_column_sums(const double *vals, int32_t n_cols, int64_t n, int32_t n_variants,
                              double *partial, int32_t n_part_blocks, double *out, hipStream_t s) {
    if (n_cols <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_colsum_pass1, dim3(n_part_blocks, n_variants, n_cols), dim3(kRedBlock),
                       0, s, vals, n_cols, n, n * n_variants, partial);
    const int nout = n_variants * n_cols;
    hipLaunchKernelGGL(k_pass2, dim3((nout + 127) / 128), dim3(128), 0, s, partial, n_part_blocks,
                       n_cols, n_variants, out);
    return hipGetLastError();
}

}  // namespace mt
