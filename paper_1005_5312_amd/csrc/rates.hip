// Photoionization rates of START (Hasegawa & Umemura 2010) on gfx950.
//
// For every target particle i:
//   Gamma_i = sigma / (4 pi) * sum_alpha L_alpha exp(-tau_alpha) / d_alpha^2,
// the monochromatic form of Appendix A eq. (A2) with on-the-spot attenuation
// (eq. 7), summed over the virtual sources the tree walk hands out
// (section 2.2.2, eqs. 12-15) and excluding the target's own emission
// (k_other, eqs. 25-26).  tau_alpha is the optical depth along the straight
// ray between source and target through the gridded n_HI field.
//
// One wavefront owns up to 64 targets that are adjacent in Morton order and
// walks the tree once for all of them: a cell's children are visited when any
// target opens it, and each target has the FP64 opening test of eq. (12) of its
// own.  The rays of the entries are marched 64 at a time, one per lane; those
// of one source sit side by side, so they are nearly parallel and read the same
// grid lines.
//
// Precision: START_FP64 marches and accumulates in FP64.  START_FP32C keeps
// the FP64 opening test (exact lists) and the FP64 ray geometry, reads the
// FP32 copy of the grid (half the bytes), accumulates each column in FP64
// (one FMA per cell, no dearer than a compensated FP32 sum) and sums the
// terms of Gamma with Kahan compensation in FP32.
#include "internal.h"

#include <algorithm>
#include <cstring>
#include <type_traits>

namespace start {

namespace {

constexpr int kWave = 64;
constexpr int kThreads = 256;
constexpr int kWavesPerBlock = kThreads / kWave;

enum Mode { kRates = 0, kCount = 1, kList = 2, kStats = 3, kKeys = 4 };

// One rate problem: a tree, a grid and a run of targets (the item's segment
// of the batch's sorted target arrays).  Read by the kernels from a device
// table, one entry per item of a batch.
struct Item {
    // tree
    int64_t n_nodes;
    int64_t n_src;
    const int4 *geo;
    const int *skip;
    const int *first;
    const int *count;
    const int *ref;
    const double4 *mom;
    const uint4 *momq;
    const double *lscale;   // luminosity unit of the FP32 copies (one value)
    const double4 *src;
    const uint4 *srcq;
    const unsigned *perm;
    const Sibling *sib;     // the same nodes, siblings side by side
    // grid
    const double *grid;
    const float *gridf;
    int G;
    int grid_log2;
    int sx, sy;         // element strides of the grid copies (padded rows and planes)
    int64_t guard;      // zeroed elements before cell 0 (and after the last cell)
    double frac_scale;  // 2^-(32 - grid_log2)
    double gs;          // G / size
    double lo[3];
    double size;
    double inv_size;
    double unit_cm;
    double cell_cm;     // size / G * unit_cm
    double theta2;
    double sigma;
    // channel 0: photoionisation, term L exp(-sigma N) / d^2 (eq. A2);
    // channel 1: H2 photodissociation, term L f_sh(N / 1e14) / d^2 (eq. B1)
    int channel;
    double col_scale;   // column in cells x density -> sigma N (0) or N / 1e14 (1)
    double rate_scale;  // sigma / (4 pi) (0) or 1.13e8 / (4 pi) (1)
    // targets: caller's positions, and this item's run of the sorted arrays
    int64_t n_t;
    const double *tgt_xyz;   // [3][n_t], caller order
    const double4 *tgt;      // sorted target positions
    const unsigned *tgt_orig;// caller index of each sorted target
    const int64_t *self_src; // caller order, may be null
    // outputs (caller order)
    void *gamma;
    int64_t *counts;         // list count mode: entries per target
    const int64_t *offsets;  // list mode
    int64_t *entries;        // list mode
    int64_t *stats;          // counter mode: [n_t][4]
};

// A launch covers the tiles (runs of <= 64 targets of one item) of a batch,
// one wave per tile; the item table and the tiles are kernel arguments of
// their own (const, restrict) so their fields are read with scalar loads.

// Eq. (12): l^2 <= theta^2 d^2 in normalised units, d the distance to the
// closest point of the cube [c 2^-n, (c+1) 2^-n].  Written as the same FP64
// operations as the oracle (explicit fma, no contraction) so that the lists
// agree bit for bit.  b = (lo x, lo y, lo z, side): the cube's corner c 2^-n
// and side 2^-n (exact, c < 2^21), and lo + side = (c + 1) 2^-n is exact too.
__device__ inline bool accept_box(const double4 b, const double u[3], double theta2)
{
    const double lo[3] = {b.x, b.y, b.z};
    double d[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double a = lo[k] - u[k];
        const double c = u[k] - (lo[k] + b.w);
        // max(0, a, c) as two v_max_f64 (the operands are finite, so the
        // value is the same as with compares and selects)
        d[k] = fmax(fmax(a, c), 0.0);
    }
    const double d2 = fma(d[2], d[2], fma(d[1], d[1], d[0] * d[0]));
    return b.w * b.w <= theta2 * d2;
}

__device__ inline int clampi(int v, int G) { return v < 0 ? 0 : (v >= G ? G - 1 : v); }

// Tree records at a wave-uniform index, read through the scalar cache (the
// walk's node pointer is the same in every lane, and the tree is read-only
// while a kernel runs): a generic load would take a vector load per lane
// and wait on the LDS counter as well.
using CI = const __attribute__((address_space(4))) int;
using CU = const __attribute__((address_space(4))) unsigned;
using CD = const __attribute__((address_space(4))) double;
__device__ inline int4 uni_int4(const int4 *a, int i)
{
    CI *p = (CI *)a + 4 * (int64_t)i;
    return make_int4(p[0], p[1], p[2], p[3]);
}
__device__ inline int uni_int(const int *a, int64_t i) { return ((CI *)a)[i]; }
__device__ inline unsigned uni_u32(const unsigned *a, int64_t i) { return ((CU *)a)[i]; }
__device__ inline void uni_sibling(const Sibling *a, int i, double4 &cube, int4 &meta)
{
    CD *p = (CD *)a + 6 * (int64_t)i;
    CI *q = (CI *)(p + 4);
    cube = make_double4(p[0], p[1], p[2], p[3]);
    meta = make_int4(q[0], q[1], q[2], q[3]);
}
// The same at an index that four neighbouring lanes share: lane `part` of the
// four (all of them active) reads its three words, and the words go round by DPP.
__device__ inline void quad_sibling(const Sibling *a, int i, int part, double4 &cube, int4 &meta)
{
    struct Words {
        int w[3];
    };
    const Words r = reinterpret_cast<const Words *>(a)[4 * (int64_t)i + part];
#define FROM(d) __builtin_amdgcn_update_dpp(0, r.w[(d) % 3], (d) / 3 * 0x55, 0xF, 0xF, true)
    cube = make_double4(__hiloint2double(FROM(1), FROM(0)), __hiloint2double(FROM(3), FROM(2)),
                        __hiloint2double(FROM(5), FROM(4)), __hiloint2double(FROM(7), FROM(6)));
    meta = make_int4(FROM(8), FROM(9), FROM(10), FROM(11));
#undef FROM
}
// the luminosity (.w) of a double4 record
__device__ inline double uni_w(const double4 *a, int64_t i) { return ((CD *)a)[4 * i + 3]; }

// Orders LDS traffic between the lanes of one wavefront (no block barrier:
// the waves of a block are independent).
__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline int lanes_below(uint64_t m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// Inclusive sum over the lanes of the first N (the others hold 0), by DPP.
template <int N>
__device__ inline int scan_lanes(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
    if (N > 8) v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
    if (N > 16) v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // row_bcast:15 into rows 1 and 3
    if (N > 32) v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // row_bcast:31 into rows 2 and 3
    return v;
}

// ---------------------------------------------------------------------------
// Ray march through the piecewise-constant grid from its start (t = 0) to
// its end (t = 1); the start is given as its cell (linear index) and its
// fraction fb inside the cell.  The rate kernels start every ray at its
// (virtual) source: the items of one node then leave from one point and fan
// out towards their targets, so the lanes of a gather stay in the same or
// neighbouring cache lines for longer than when each ray starts at its own
// target (~20% fewer L1 accesses per gather on the diffuse benchmark's
// batches).  The geometry (direction D, plane parameters)
// is FP64 in both precisions: an FP32 ray parameter resolves a crossing only
// to ~6e-8 of the ray length (1e-5 cell over 128 cells), which times the
// optical depth of a dense cell (~200 per cell for the 200x clumps) is above
// the 2e-4 target.  TV is the type of the grid values (FP32 or
// FP64); the sum is FP64 in both cases.  Returns sum n_c dt.
//
// The step has no branch: the next crossing is the minimum m of the three
// plane parameters, the first axis whose parameter equals m moves to its next
// plane, and the cell offset moves by that axis's stride (where the ray
// passes exactly through an edge or a corner, the other axes at m follow in
// the next steps with chords of length 0, which add exactly nothing).  The
// cell sequence depends on the geometry only, so the loads run ahead of the
// sum: three cells ahead in the rate kernels, four for FP64 cells (gathers
// in flight per lane hide most of the L1 / L2 latency: three are 7% faster
// in FP32 and 16% in FP64 than one), one ahead in the counter pass, which
// has no registers to spare.
// Cells are addressed by a 32-bit byte offset from the grid base, which the
// hardware adds to the base in the load itself (below 2^32 for FP32 cells at
// G <= 1024 and for FP64 cells at G <= 512, the grids with guard bands;
// FP64 cells of the largest grid take an element index).  The hot loop is
// L1- and VALU-bound: one gather and 14 VALU instructions per step and lane
// in FP32C, 13 in FP64.
//
// The loop ends: each step moves an axis whose parameter equals m, by a_k >=
// 1 / (2 G) (|D| is below 2G for points in the box; the step is exact since
// a_k is far above the spacing of doubles below 1), so after at most
// 3 (2G + 2) steps every parameter is >= 1.  Positions reaching the kernel
// are finite and inside the box (checked on entry), so the parameters are
// finite.  Were m NaN, it would not equal any parameter and z would step
// while t = min(m, 1) is 1 (v_min_f64 returns the non-NaN operand): the
// rate march ends with its turn (three or four steps on) and the counter
// pass at once.  No extra step counter is kept: one costs 4-8% here, as it changes
// how the loop is scheduled.
// ---------------------------------------------------------------------------
// 1 / d for d > 0 to full FP64 precision: hardware reciprocal and two Newton
// steps (the inputs are finite, normal magnitudes: ray components in cells).
__device__ inline double recip(double d)
{
    double r = __builtin_amdgcn_rcp(d);
    double e = fma(-d, r, 1.0);
    r = fma(r, e, r);
    e = fma(-d, r, 1.0);
    return fma(r, e, r);
}

// min of two FP64 values in one instruction (fmin() would first quiet
// signalling NaNs of both operands; the plane parameters are never NaN
// signalling, and a quiet NaN loses the comparison either way)
__device__ inline double vmin(double x, double y)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}

__device__ inline double min3(double x, double y, double z) { return vmin(vmin(x, y), z); }

// H2 self-shielding function of Appendix B: 1 up to x = 1, x^(-3/4) above,
// as (1 / x^(1/4))^3 with two square roots (a few ulp; far lighter than pow)
__device__ inline float fsh(float x)
{
    const float r = 1.0f / sqrtf(sqrtf(x));
    return x <= 1.0f ? 1.0f : r * r * r;
}
__device__ inline double fsh(double x)
{
    const double r = 1.0 / sqrt(sqrt(x));
    return x <= 1.0 ? 1.0 : r * r * r;
}

typedef const __attribute__((address_space(1))) char gchar_t;

// cell value at an offset from the grid base: in bytes (S = 1 byte per unit),
// which the hardware adds to the SGPR base in the load itself, or as an
// element index (S = the cell size, one address computation per load)
template <unsigned S, typename TV>
__device__ inline TV load_cell(const TV *grid, unsigned off)
{
    if constexpr (S == 1)
        return *(const __attribute__((address_space(1))) TV *)((gchar_t *)grid + off);
    else
        return *((const __attribute__((address_space(1))) TV *)grid + off);
}

// One step of the march: the first axis (x, then y, then z) whose plane
// parameter equals the minimum m moves to its next plane, and the cell offset
// by that axis's stride.  Where the ray passes exactly through an edge or a
// corner the other axes at m follow in the next steps, each with a chord of
// length 0 (which adds exactly nothing).  The three moves run under lane
// masks (exec set from the two comparisons), so each is one add per axis
// instead of a select and an add for every axis: 8 vector instructions per
// step for the comparisons and moves against 14.  The masks come from the
// active lanes only and exec is restored at the end of the block.
__device__ inline void step_axis(double tn[3], const double a[3], const int ds[3], double m, unsigned &off)
{
    const uint64_t m0 = __builtin_amdgcn_ballot_w64(tn[0] == m);
    const uint64_t m1 = __builtin_amdgcn_ballot_w64(tn[1] == m);
    uint64_t sv, tmp;
    asm volatile(
        "s_and_saveexec_b64 %[sv], %[m0]\n\t"
        "v_add_f64 %[t0], %[t0], %[a0]\n\t"
        "v_add_u32 %[off], %[off], %[d0]\n\t"
        "s_andn2_b64 exec, %[m1], %[m0]\n\t"
        "v_add_f64 %[t1], %[t1], %[a1]\n\t"
        "v_add_u32 %[off], %[off], %[d1]\n\t"
        "s_or_b64 %[tmp], %[m0], %[m1]\n\t"
        "s_andn2_b64 exec, %[sv], %[tmp]\n\t"
        "v_add_f64 %[t2], %[t2], %[a2]\n\t"
        "v_add_u32 %[off], %[off], %[d2]\n\t"
        "s_mov_b64 exec, %[sv]"
        : [t0] "+v"(tn[0]), [t1] "+v"(tn[1]), [t2] "+v"(tn[2]), [off] "+v"(off), [sv] "=&s"(sv), [tmp] "=&s"(tmp)
        : [m0] "s"(m0), [m1] "s"(m1), [a0] "v"(a[0]), [a1] "v"(a[1]), [a2] "v"(a[2]), [d0] "v"(ds[0]),
          [d1] "v"(ds[1]), [d2] "v"(ds[2]));
}

template <typename TV, bool STATS, bool CLAMP>
__device__ inline TV march(const TV *__restrict__ grid, int sx, int sy, unsigned last, unsigned idx0,
                           const double fb[3], const double D[3], int &ncell)
{
    // Axis k crosses its next plane at tn_k and every 1/|D_k| after it.  In
    // FP64 stepping tn_k by a_k drifts by ~1 ulp per step: over the <= 3G
    // steps of a ray that is ~1e-11 cell, far inside every tolerance.
    // offset units per cell: bytes, except for FP64 cells on a grid without
    // guard bands (G = 1024), whose bytes can pass 2^32
    constexpr unsigned kScale = sizeof(TV) == 8 && CLAMP ? 1u : (unsigned)sizeof(TV);
    constexpr unsigned kUnit = kScale == 1 ? (unsigned)sizeof(TV) : 1u;   // bytes per offset unit
    const int stride[3] = {sx, sy, 1};
    double a[3], tn[3];
    int ds[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (D[k] > 0.0) {
            a[k] = recip(D[k]);
            tn[k] = (1.0 - fb[k]) * a[k];
            ds[k] = stride[k];
        } else if (D[k] < 0.0) {
            a[k] = recip(-D[k]);
            tn[k] = fb[k] * a[k];
            ds[k] = -stride[k];
        } else {
            a[k] = 0.0;
            tn[k] = 2.0;   // never crossed
            ds[k] = 0;
        }
        // a step of 2 carries a parameter past the end (t = 1) whatever it
        // was, so longer steps are cut to 2: every step is then finite
        a[k] = a[k] < 2.0 ? a[k] : 2.0;
        ds[k] *= (int)kScale;
    }
    unsigned off = idx0 * kScale;
    const unsigned off_max = last * kScale;
    double t = 0.0, sum = 0.0;
    auto add = [&](TV v, double len) {
        sum = fma((double)v, len, sum);
        if (STATS) ncell += len > 0.0 ? 1 : 0;
    };
    double m = min3(tn[0], tn[1], tn[2]);
    // leave the current cell (t = m) for the next one and load its value
    auto advance = [&](TV &vnext) {
        t = m;
        step_axis(tn, a, ds, m, off);
        if (CLAMP) off = off > off_max ? off_max : off;   // also catches a step below 0
        vnext = load_cell<kUnit>(grid, off);
        m = min3(tn[0], tn[1], tn[2]);
    };
    if constexpr (!STATS) {
        // Registers take the cells in turn (three for FP32 cells, four for
        // FP64, whose longer gathers gain 2% from the fourth; a fourth for
        // FP32 gains nothing and costs the eighth wave per SIMD); a cell's
        // value is added when the march leaves the cell two (three) places
        // after it, so three (four) loads are in flight.  The march runs in
        // whole turns of three (four) steps with the crossing parameter
        // clamped to 1: once a lane has reached its end its further steps
        // have length 0 and add nothing, so a turn has no exits inside it,
        // and every turn (the first too: the pending registers start as
        // loads of the first cell, added with length 0) enters with the same
        // loads in flight, so no wait for all of them.  Each step is kept in
        // place by a scheduling barrier so that its load is issued within it.
        constexpr bool kFour = sizeof(TV) == 8;
        TV vB = load_cell<kUnit>(grid, off);
        TV vC = load_cell<kUnit>(grid, off);
        TV vD = kFour ? load_cell<kUnit>(grid, off) : TV(0);
        TV vA = load_cell<kUnit>(grid, off);
        double lA = 0.0, lB = 0.0, lC = 0.0, lD = 0.0;
        auto leave = [&](double &len, TV &vnext) {
            const double mc = vmin(m, 1.0);   // a NaN m gives 1: the lane ends
            len = mc - t;
            t = mc;
            step_axis(tn, a, ds, m, off);
            if (CLAMP) off = off > off_max ? off_max : off;   // also catches a step below 0
            vnext = load_cell<kUnit>(grid, off);
            m = min3(tn[0], tn[1], tn[2]);
        };
        for (;;) {
            add(vB, lB);
            leave(lA, vB);
            __builtin_amdgcn_sched_barrier(0);
            add(vC, lC);
            leave(lB, vC);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (kFour) {
                add(vD, lD);
                leave(lC, vD);
                __builtin_amdgcn_sched_barrier(0);
                add(vA, lA);
                leave(lD, vA);
            } else {
                add(vA, lA);
                leave(lC, vA);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (!(t < 1.0)) break;
        }
        add(vB, lB);
        add(vC, lC);
        if constexpr (kFour) add(vD, lD);
        return (TV)sum;
    } else {
        // the counter pass: one load ahead
        TV v = load_cell<kUnit>(grid, off);
        // two steps per turn (no register copies between them)
        for (;;) {
            if (!(m < 1.0)) break;
            add(v, m - t);
            advance(v);
            if (!(m < 1.0)) break;
            add(v, m - t);
            advance(v);
        }
        add(v, 1.0 - t);
        return sum;
    }
}

// ---------------------------------------------------------------------------
// Walk used by the list export (entries only, no march).
// ---------------------------------------------------------------------------
template <int MODE>
__global__ void __launch_bounds__(kThreads) list_kernel(const Item *__restrict__ items, const int4 *__restrict__ tiles,
                                                        int n_tiles)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int ti = __builtin_amdgcn_readfirstlane((int)blockIdx.x * kWavesPerBlock + (int)(threadIdx.x >> 6));
    if (ti >= n_tiles) return;
    const int4 tile = tiles[ti];
    const Item &P = items[__builtin_amdgcn_readfirstlane(tile.x)];
    const int64_t it = (int64_t)tile.y + lane;
    const bool valid = lane < tile.z;
    double u[3] = {0.0, 0.0, 0.0};
    unsigned orig = 0;
    int64_t self = -1;
    if (valid) {
        const double4 p = P.tgt[it];
        const double x[3] = {p.x, p.y, p.z};
        orig = P.tgt_orig[it];
        if (P.self_src) self = P.self_src[orig];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double v = (x[k] - P.lo[k]) * P.inv_size;
            u[k] = v > 1.0 ? 1.0 : (v < 0.0 ? 0.0 : v);
        }
    }
    int64_t n_entries = 0;
    const int64_t out_base = ((MODE == kList || MODE == kKeys) && valid) ? P.offsets[orig] : 0;
    // kList writes the export code (node index, or -(source index)-1);
    // kKeys writes node << 32 | (bucket member + 1, or 0), which increases
    // along the walk, so each target's keys come out sorted
    auto emit = [&](int64_t code, uint64_t key, double L) {
        if (!(L > 0.0)) return;
        if (MODE == kList) P.entries[out_base + n_entries] = code;
        if (MODE == kKeys) P.entries[out_base + n_entries] = (int64_t)key;
        ++n_entries;
    };
    const int4 *const t_geo = P.geo;
    const int *const t_skip = P.skip;
    const int *const t_ref = P.ref;
    const int *const t_first = P.first;
    const int *const t_count = P.count;
    const unsigned *const t_perm = P.perm;
    const double4 *const t_mom = P.mom;
    const double4 *const t_src = P.src;
    const double theta2 = P.theta2;
    int resume = 0, node = 0;
    const int n_nodes = (int)P.n_nodes;
    while (node < n_nodes) {
        node = __builtin_amdgcn_readfirstlane(node);
        const int4 g = uni_int4(t_geo, node);
        const int sk = uni_int(t_skip, node);
        const double lw = uni_w(t_mom, node);
        const int ref = uni_int(t_ref, node);
        const int kind = g.w >> 8;
        const bool active = valid && node >= resume;
        if (kind == kKindLeaf) {
            if (active && (int64_t)ref != self) emit(-(int64_t)ref - 1, (uint64_t)node << 32, lw);
            node += 1;
            continue;
        }
        const bool acc = active && accept_box(cube_of(g), u, theta2);
        if (acc) {
            emit(node, (uint64_t)node << 32, lw);
            resume = sk;
        }
        const bool open = active && !acc;
        if (kind == kKindBucket) {
            if (__any(open)) {
                const int f = uni_int(t_first, node), cnt = uni_int(t_count, node);
                for (int q = f; q < f + cnt; ++q) {
                    const unsigned pq = uni_u32(t_perm, q);
                    const double lq = uni_w(t_src, q);
                    if (open && (int64_t)pq != self)
                        emit(-(int64_t)pq - 1, (uint64_t)node << 32 | (uint64_t)(q - f + 1), lq);
                }
            }
            node += 1;
            continue;
        }
        node = __any(open) ? node + 1 : sk;
    }
    if (valid) {
        if (MODE == kCount) P.counts[orig] = n_entries;
    }
}

// ---------------------------------------------------------------------------
// Rate kernel.  A wave owns NT targets (8, 16, 32 or 64) that are adjacent in
// Morton order.  It walks the tree frame by frame: a frame is the children of
// one opened cell (side by side in Tree::sib) and the targets that opened it.
// Its siblings are tested 64 / NT at a time for all targets, lane = sibling *
// NT + target: what a target uses whole (or a single source) goes to the ring,
// and what some target opens goes to a stack in LDS, from whose top the walk
// goes on.  So each target's terms come in one order whatever the tile: a
// frame's own entries in the siblings' order, then the opened siblings' in
// theirs (from the last to the first it marched 3-6% slower on 128^3 cells).
//
// DF: strictly depth first, for the FP32C rates of the equilibrium loops.
// Their fractions are double precision, and the other order moves one FP32C
// rate in about twenty by its last bit: the fractions would be 1e-8 off what
// the loops have always given.  It cuts a step at every opened sibling, and
// takes 272 us where the other takes 243 (16457 targets that all emit).
//
// An entry is not marched at once: (entry, target) items go to a per-wave ring
// in LDS, and as soon as 64 are pending every lane marches one of them --
// whichever target it belongs to.  Items of one node share the source and sit
// side by side, so a batch is bundles of nearly parallel rays that read the
// same grid lines (sorting a window by ray length instead balanced the lanes
// better but lost this locality and ran 40% slower).  After a batch the terms
// are handed out target by target, in order, and lane t adds target t's to its
// Kahan (FP32) or plain (FP64) sum: results are deterministic and do not depend
// on the tile.
//
// What bounds it: the marches' gathers keep the vector memory path ~83% busy
// (~21 cycles each) and the vector units ~89% (2^20 targets that all emit, in
// tiles of 32).  So the walk stays off that
// path: with 64 or 32 targets the one or two siblings' records come through the
// scalar cache, with fewer each lane loads a quarter of one and has the rest
// from its neighbours by DPP (whole records by vector loads cost 3-4%: 2^17
// targets that all emit 1653 us, now 1589; for tiles of 32 the quarters take
// 18.91 ms and the scalar cache 18.64, 2^20 targets).
//
// Against a walk that visited every node of the tile's union one after the
// other (tiles of 16 and more) or eight siblings in depth-first order (tiles of
// at most 8), us before -> now: 1024 targets that all emit 56 -> 49, 16457 272
// -> 243, 2^17 1740 -> 1610, 300007 7000 -> 6600 (FP64, 128^3 shadow 7790 ->
// 7500), 2^20 18940 -> 18560; 2^17 targets of 1024 sources 970 -> 913.
constexpr int kRing = 128;   // items; a node adds <= 64 and a batch drains 64

// 32-bit fixed point of the box: floor(u 2^32) of the normalised coordinate
// u in [0, 1] (1 itself to 2^32 - 1).  The FP32 path encodes the virtual
// sources and the targets alike, so a target at a source's position is at
// distance 0 exactly (both skipped as in the FP64 path); positions closer
// than 2^-32 of the box count as the same.  The top g bits of a coordinate
// are its cell on a 2^g grid, the rest the fraction inside it (exact in FP64).
__device__ inline unsigned fixed32(double x, double lo, double inv)
{
    double u = (x - lo) * inv;
    u = u < 0.0 ? 0.0 : (u > 1.0 ? 1.0 : u);
    const double q = floor(u * 4294967296.0);
    return q >= 4294967295.0 ? 0xFFFFFFFFu : (unsigned)q;
}

// Frames of siblings that wait on a wave's walk: at most 7 more per level of
// the path than it has taken up, 8 of the last.
constexpr int kStack = 7 * kMaxLevel + 8;

// TF: the target's position in cells (FP64) for the FP64 path; for the FP32
// path its 32-bit box fixed-point coordinates (fixed32), kept in the items.
template <typename T, typename TF, int NT, bool DF>
struct WaveLds {
    static constexpr bool kFp64 = sizeof(TF) == 8;
    // FP32 path: the item whole (code, then the target's fixed32
    // coordinates), so that a march reads it in one access
    uint4 qitem[kFp64 ? 1 : kRing];
    // FP64 path: the item as code
    int code[kFp64 ? kRing : 1];  // node index, or -(sorted source index)-1
    T term[kWave + 8];            // a batch's terms by target, each target's in order
    TF tpos[kFp64 ? NT : 1][3];   // FP64 path: target position in cells
    unsigned char lane[kRing];    // target of the item
    // depth first: the siblings that wait at each level of the path
    int4 rest[DF && NT < kWave ? kMaxLevel + 1 : 1][DF ? kWave / NT : 1];
    // otherwise: (targets that opened the cell (two words), first child's place,
    // children; a bucket: first sorted source, minus its sources)
    int4 stack[DF ? 1 : kStack];
};


template <int PREC, bool STATS, bool CLAMP, int NT, bool DF, typename T, typename TF>
__device__ __forceinline__ void rates_tile(const Item &P, const int4 tile, WaveLds<T, TF, NT, DF> &L, int *lds_ncell);

template <int PREC, bool STATS, bool CLAMP, int NT, bool DF>
__global__ void __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(NT < 64 || PREC == START_FP64 ? 5 : 7))) rates_kernel(const Item *__restrict__ items,
                                                         const int4 *__restrict__ tiles, int n_tiles)
{
    using T = typename std::conditional<PREC == START_FP64, double, float>::type;
    using TF = typename std::conditional<PREC == START_FP64, double, unsigned>::type;
    __shared__ WaveLds<T, TF, NT, DF> lds_all[kWavesPerBlock];
    __shared__ int ncell_all[STATS ? kWavesPerBlock : 1][STATS ? kWave + 8 : 1];   // counter mode only
    const int wv = threadIdx.x >> 6;
    // blocks are dealt round-robin to the 8 XCDs: give each XCD a contiguous
    // run of tiles (Morton-adjacent targets share nodes and grid lines in its L2)
    const int nb = (int)gridDim.x;
    const int per_xcd = nb / 8;
    int blk = (int)blockIdx.x;
    if (per_xcd > 0 && blk < per_xcd * 8) blk = (blk & 7) * per_xcd + (blk >> 3);
    // wave-uniform: tile record and item table are read with scalar loads
    const int ti = __builtin_amdgcn_readfirstlane(blk * kWavesPerBlock + wv);
    if (ti >= n_tiles) return;
    const int4 tile = tiles[ti];
    const int item = __builtin_amdgcn_readfirstlane(tile.x);
    rates_tile<PREC, STATS, CLAMP, NT, DF, T, TF>(items[item], tile, lds_all[wv], ncell_all[STATS ? wv : 0]);
}

template <int PREC, bool STATS, bool CLAMP, int NT, bool DF, typename T, typename TF>
__device__ __forceinline__ void rates_tile(const Item &P, const int4 tile, WaveLds<T, TF, NT, DF> &L, int *lds_ncell)
{
    const int lane = threadIdx.x & (kWave - 1);
    constexpr int kLog = NT == 8 ? 3 : NT == 16 ? 4 : NT == 32 ? 5 : 6;
    constexpr int kSib = kWave / NT;
    const int tgt = lane & (NT - 1), sib = lane >> kLog;   // this lane's target of the tile, and its sibling
    const int64_t it = (int64_t)tile.y + tgt;
    const bool valid = tgt < tile.z;
    wave_sync();   // the previous tile's LDS reads are done

    const int G = P.G;
    const int gl = P.grid_log2;
    // the march addresses the grid from the start of its guard band, which
    // takes the steps past a ray's end (CLAMP: G = 1024, no band, offsets
    // clamped to the last cell's element)
    const int64_t guard = P.guard;
    const int last = (G - 1) * (P.sx + P.sy + 1);
    double u[3] = {0.0, 0.0, 0.0};
    unsigned orig = 0;
    int self = -1;   // source indices fit in 31 bits (n_s <= 2^30)
    unsigned tq[3] = {0u, 0u, 0u};   // FP32 path: this lane's target as fixed32 box coordinates
    {
        double B[3] = {0.0, 0.0, 0.0};
        if (valid) {
            const double4 p = P.tgt[it];
            const double x[3] = {p.x, p.y, p.z};
            orig = P.tgt_orig[it];
            if (P.self_src) self = (int)P.self_src[orig];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const double v = (x[k] - P.lo[k]) * P.inv_size;
                u[k] = v > 1.0 ? 1.0 : (v < 0.0 ? 0.0 : v);
                // the position in cells: its floor (the last cell for a target
                // on the top face) plus the fraction, both exact, sum to it
                B[k] = (x[k] - P.lo[k]) * P.gs;
            }
        }
        if constexpr (PREC == START_FP64) {
            if (lane < NT) {
                L.tpos[lane][0] = B[0];
                L.tpos[lane][1] = B[1];
                L.tpos[lane][2] = B[2];
            }
        } else {
            const double4 p = valid ? P.tgt[it] : make_double4(P.lo[0], P.lo[1], P.lo[2], 0.0);
            tq[0] = fixed32(p.x, P.lo[0], P.inv_size);
            tq[1] = fixed32(p.y, P.lo[1], P.inv_size);
            tq[2] = fixed32(p.z, P.lo[2], P.inv_size);
        }
    }

    T acc = T(0), accc = T(0);
    int64_t st_test = 0, st_entries = 0, st_cells = 0, st_zero = 0;
    int head = 0, tail = 0;   // wave-uniform ring counters
    const T col_scale = (T)P.col_scale;
    const int sh = 32 - gl;

    // the node and source arrays of the item, read once per tile (the item
    // is the same for the whole wave): each march then selects its record's
    // address between two registers instead of loading the array pointer,
    // and reads it as global memory (a generic load would also wait on LDS)
    using GD = const __attribute__((address_space(1))) double;
    using GU = const __attribute__((address_space(1))) unsigned;
    GD *const mom = (GD *)P.mom;
    GD *const src = (GD *)P.src;
    GU *const momq = (GU *)P.momq;
    GU *const srcq = (GU *)P.srcq;
    // the item's scalars, also read once per tile
    const double frac_scale = P.frac_scale, gs = P.gs;
    const double lo[3] = {P.lo[0], P.lo[1], P.lo[2]};
    const int sx = P.sx, sy = P.sy, channel = P.channel;
    const T *const grid_base = (PREC == START_FP64 ? (const T *)P.grid : (const T *)P.gridf) - guard;

    // March one item: the term L e^-tau / d^2 (d in cells) of ring slot `slot`.
    auto march_item = [&](int slot, T &term, int &nc) {
        int code, tl = 0;
        unsigned qt[3] = {0u, 0u, 0u};
        if constexpr (PREC == START_FP64) {
            code = L.code[slot];
            tl = L.lane[slot];
        } else {
            const uint4 q = L.qitem[slot];
            code = (int)q.x;
            qt[0] = q.y;
            qt[1] = q.z;
            qt[2] = q.w;
        }
        double tp[3] = {0.0, 0.0, 0.0};
        if constexpr (PREC == START_FP64) {
#pragma unroll
            for (int k = 0; k < 3; ++k) tp[k] = L.tpos[tl][k];
        }
        // the ray runs from the (virtual) source (t = 0) to the target (t = 1):
        // D = target - source, the march starts in the source's cell
        double D[3], fa[3];
        int ab[3];
        T w;
        if (PREC == START_FP64) {
            GD *const r = code >= 0 ? mom + 4 * (int64_t)code : src + 4 * (int64_t)(-code - 1);
            const double4 m = make_double4(r[0], r[1], r[2], r[3]);
            const double A[3] = {(m.x - lo[0]) * gs, (m.y - lo[1]) * gs, (m.z - lo[2]) * gs};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                // a source on the top face sits in the last cell at fraction 1
                ab[k] = clampi((int)floor(A[k]), G);
                fa[k] = A[k] - (double)ab[k];
                D[k] = tp[k] - A[k];
            }
            w = (T)m.w;
        } else {
            // centre as 32-bit fixed point of the box: the top g bits are the
            // cell, the rest the fraction inside it (exact in FP64); D is the
            // difference of the two fixed-point coordinates in cells, exact
            // (both below 2^32, scaled by a power of two)
            GU *const r = code >= 0 ? momq + 4 * (int64_t)code : srcq + 4 * (int64_t)(-code - 1);
            const uint4 m = make_uint4(r[0], r[1], r[2], r[3]);
            const unsigned q[3] = {m.x, m.y, m.z};
            const unsigned fmask = (1u << sh) - 1u;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                ab[k] = (int)(q[k] >> sh);
                fa[k] = (double)(q[k] & fmask) * frac_scale;
                D[k] = ((double)qt[k] - (double)q[k]) * frac_scale;
            }
            w = (T)__uint_as_float(m.w);
        }
        const double d2 = D[0] * D[0] + D[1] * D[1] + D[2] * D[2];
        if (d2 > 0.0) {
            const unsigned e0 = (unsigned)(ab[0] * sx + ab[1] * sy + ab[2] + guard);
            const T col = march<T, STATS, CLAMP>(grid_base, sx, sy, (unsigned)(last + guard), e0, fa, D, nc);
            // FP32C: the term from the hardware square root, exp2 and
            // reciprocal (each ~1 ulp; the argument of exp2 is rounded to
            // ~6e-8 relative, i.e. 6e-8 tau of the term), FP64 as written
            const T dist = PREC == START_FP64 ? (T)sqrt(d2) : (T)__builtin_amdgcn_sqrtf((float)d2);   // grid units
            const T c = col_scale * (col * dist);
            if (channel == 0)                                  // c = tau
                term = PREC == START_FP64 ? w * exp(-c) / (T)d2
                                          : (T)(w * __builtin_amdgcn_exp2f((float)c * -1.44269504f) *
                                                __builtin_amdgcn_rcpf((float)d2));
            else
                term = w * fsh(c) / (T)d2;                     // c = N_H2 / 1e14
        } else {
            term = T(0);
            nc = -1;                                           // zero distance: skipped
        }
    };

    // March the next (up to) 64 pending items and hand the terms back.
    auto drain = [&]() {
        const int nb_items = (tail - head) < kWave ? (tail - head) : kWave;
        const int slot = (head + lane) & (kRing - 1);
        T term = T(0);
        int nc = 0;
        wave_sync();   // the queue's LDS writes
        if (lane < nb_items) march_item(slot, term, nc);
        // the items are in each target's order of terms: the terms go to LDS
        // target by target.  The ballots of the items' target numbers give the
        // items of target t; their counts, scanned over the lanes t, the place
        // of each target's first term.
        const unsigned tl = L.lane[slot];
        const uint64_t here = __ballot(lane < nb_items);
        uint64_t bits[kLog];
#pragma unroll
        for (int k = 0; k < kLog; ++k) bits[k] = __ballot((tl >> k) & 1u);
        auto of_target = [&](unsigned t) {
            unsigned lo = (unsigned)here, hi = (unsigned)(here >> 32);
#pragma unroll
            for (int k = 0; k < kLog; ++k) {
                const unsigned off = ((t >> k) & 1u) - 1u;   // all ones where the bit is 0
                lo &= (unsigned)bits[k] ^ off;
                hi &= (unsigned)(bits[k] >> 32) ^ off;
            }
            return (uint64_t)lo | (uint64_t)hi << 32;
        };
        const int k = lane < NT ? __popcll(of_target((unsigned)lane)) : 0;   // terms of target `lane`
        const int f = scan_lanes<NT>(k) - k;                                 // and its first place
        const int first_of = __builtin_amdgcn_ds_bpermute((int)(tl << 2), f);
        if (lane < nb_items) {
            const int at = first_of + __popcll(of_target(tl) & ((1ull << lane) - 1ull));
            L.term[at] = term;
            if (STATS) lds_ncell[at] = nc;
        }
        wave_sync();
        if (lane < NT) {
            // lane t adds the terms of target t, the next four read ahead
            const T *const tt = &L.term[f];
            T v[4] = {tt[0], tt[1], tt[2], tt[3]};
            for (int j = 0; j < k; j += 4) {
                T x[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) x[q] = v[q];
                const int nx = j + 4 < k ? j + 4 : 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = tt[nx + q];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (j + q < k) {
                        const T y = x[q] - accc;
                        const T t2 = acc + y;
                        if (sizeof(T) == 4) accc = (t2 - acc) - y;
                        acc = t2;
                        if (STATS) {
                            const int c = lds_ncell[f + j + q];
                            if (c < 0) st_zero++;
                            else st_cells += c;
                        }
                    }
            }
        }
        head += nb_items;
        wave_sync();
    };

    // Queue the entry `code` for the lanes of the mask m (wave-uniform).
    auto queue = [&](uint64_t m, int code) {
        if (__builtin_amdgcn_inverse_ballot_w64(m)) {
            const int s = (tail + lanes_below(m)) & (kRing - 1);
            L.lane[s] = (unsigned char)tgt;
            if constexpr (PREC == START_FP64) {
                L.code[s] = code;
            } else {
                L.qitem[s] = make_uint4((unsigned)code, tq[0], tq[1], tq[2]);
            }
            if (STATS) st_entries++;
        }
        tail += __popcll(m);
    };

    // The walk (see above the kernel).  A frame: `left` siblings from place
    // `first`, for the targets of the lanes `act`; the root is the one sibling
    // of the first.
    constexpr int kLit = PREC == START_FP32C ? 2 : 1;
    const double theta2 = P.theta2;
    const Sibling *const w_sib = P.sib;
    const unsigned *const t_perm = P.perm;
    const double4 *const t_src = P.src;
    const uint4 *const t_srcq = P.srcq;
    bool done = P.n_nodes == 0, bucket = false, fresh = true;
    int first = 0, left = 1, depth = 0;
    uint64_t act = __ballot(valid), held_take = 0, held_open = 0;
    int4 held = make_int4(0, 0, 0, 0);
    auto enter = [&](uint64_t by, int f, int n) {   // n < 0: the members of a bucket
        act = by;
#pragma unroll
        for (int b = NT; b < kWave; b *= 2) act |= act << b;
        first = f;
        bucket = n < 0;
        left = bucket ? -n : n;
        fresh = true;
    };
    // Depth first: the frames that wait, one level per lane: the masks of what
    // is left of the siblings in hand (their records are in L.rest), the place
    // and number of the siblings from those on, the lanes of the targets.
    // Otherwise: the frame's opened siblings, one per lane, until the frame is
    // through (targets that opened it, first child's place, children or minus
    // a bucket's sources).
    unsigned w_take[2] = {0u, 0u}, w_open[2] = {0u, 0u}, w_act[2] = {0u, 0u};
    int w_first = 0, w_left = 0;
    auto put = [&](unsigned *r, uint64_t v) {
        const bool here = lane == depth;
        r[0] = here ? (unsigned)v : r[0];
        r[1] = here ? (unsigned)(v >> 32) : r[1];
    };
    auto get = [&](const unsigned *r, int l) {
        return (uint64_t)(unsigned)__builtin_amdgcn_readlane((int)r[0], l) |
               (uint64_t)(unsigned)__builtin_amdgcn_readlane((int)r[1], l) << 32;
    };
    auto wait = [&](uint64_t lanes, int f, int n) {
        put(w_act, lanes);
        const bool here = lane == depth;
        w_first = here ? f : w_first;
        w_left = here ? n : w_left;
        ++depth;
    };
    int sp = 0;
    while (!done) {
        // (depth first, not fresh: what is left of a frame that waited)
        uint64_t take = held_take, opened = held_open;
        int4 me = held;
        if (!DF || fresh) {
            // kSib siblings for all targets
            const uint64_t lanes = left < kSib ? act & ((1ull << (left * NT & 63)) - 1ull) : act;
            bool tk = false, op = false;
            if (bucket) {
                // members of a level-21 cell
                if (__builtin_amdgcn_inverse_ballot_w64(lanes)) {
                    const int q = first + sib;
                    const bool lit = PREC == START_FP32C ? __uint_as_float(t_srcq[q].w) > 0.f : t_src[q].w > 0.0;
                    tk = (int)t_perm[q] != self && lit;
                    me.x = -q - 1;
                }
            } else {
                double4 cube;
                if constexpr (kSib > 2) {
                    // each lane reads a quarter of its sibling's record (a lane
                    // past the last sibling that one's) and has the rest from
                    // its neighbours
                    quad_sibling(w_sib, first + (sib < left ? sib : left - 1), lane & 3, cube, me);
                } else {
                    // the same records in every lane: through the scalar cache
                    uni_sibling(w_sib, first, cube, me);
                    if constexpr (kSib == 2) {
                        double4 c1;
                        int4 m1;
                        uni_sibling(w_sib, first + (left > 1), c1, m1);
                        me = make_int4(sib ? m1.x : me.x, sib ? m1.y : me.y, sib ? m1.z : me.z, sib ? m1.w : me.w);
                        cube = make_double4(sib ? c1.x : cube.x, sib ? c1.y : cube.y, sib ? c1.z : cube.z,
                                            sib ? c1.w : cube.w);
                    }
                }
                const bool leaf = ((me.z >> 2) & 3) == kKindLeaf;
                // (64 targets: every lane has the same sibling, and a leaf's cube
                // is not tested; else it is along with the others, to no effect)
                if (NT == kWave && leaf) {
                    tk = __builtin_amdgcn_inverse_ballot_w64(lanes) && (me.z & kLit) != 0 && me.w != self;
                } else if (__builtin_amdgcn_inverse_ballot_w64(lanes)) {
                    const bool far = accept_box(cube, u, theta2);
                    const bool lit = (me.z & kLit) != 0;
                    tk = lit && (leaf ? me.w != self : far);
                    op = !leaf && !far;
                    if (STATS) st_test++;
                }
            }
            take = __ballot(tk);
            opened = __ballot(op);
        }
        if constexpr (DF) {
            // the siblings up to the first one that some target opens
            const int so = kSib == 1 ? 0 : opened ? __builtin_ctzll(opened) >> kLog : kSib - 1;
            const uint64_t low = ~0ull >> (kWave - NT - (so << kLog));
            if (take & low) queue(take & low, me.x);
            if (opened) {
                const uint64_t by = kSib == 1 ? opened : opened >> (so << kLog) & ((1ull << (NT & 63)) - 1ull);
                // a lane that opened it holds its record
                const int l = (so << kLog) + __builtin_ctzll(by);
                int4 cell = me;
                if constexpr (kSib > 1) {
                    cell.y = __builtin_amdgcn_readlane(me.y, l);
                    cell.z = __builtin_amdgcn_readlane(me.z, l);
                    cell.w = __builtin_amdgcn_readlane(me.w, l);
                    take &= ~low;
                    opened &= ~low;
                }
                if (kSib == 1 ? left > 1 : (take | opened) != 0 || left > kSib) {
                    // what follows it waits at this level
                    if constexpr (kSib > 1) {
                        if (__builtin_amdgcn_inverse_ballot_w64(take | opened)) L.rest[depth][sib] = me;
                        put(w_take, take);
                        put(w_open, opened);
                    }
                    if constexpr (kSib < 8) wait(act, first, left);
                    else ++depth;
                }
                enter(by, cell.y, ((cell.z >> 2) & 3) == kKindBucket ? -cell.w : cell.z >> 4);
            } else if (left > kSib) {
                first += kSib;
                left -= kSib;
                fresh = true;
            } else if (depth > 0) {
                --depth;
                bucket = false;
                if constexpr (kSib > 1) {
                    wave_sync();
                    held = L.rest[depth][sib];
                    held_take = get(w_take, depth);
                    held_open = get(w_open, depth);
                    left = 0;
                    fresh = false;
                }
                if constexpr (kSib < 8) {
                    act = get(w_act, depth);
                    first = __builtin_amdgcn_readlane(w_first, depth);
                    left = __builtin_amdgcn_readlane(w_left, depth);
                    if (kSib == 1 || (held_take | held_open) == 0) {
                        first += kSib;
                        left -= kSib;
                        fresh = true;
                    }
                }
            } else {
                done = true;
            }
        } else {
            if (take) queue(take, me.x);
            first += kSib;
            left -= kSib;
            if (opened) {
                const int num = ((me.z >> 2) & 3) == kKindBucket ? -me.w : me.z >> 4;
                if constexpr (kSib == 1) {
                    wait(opened, me.y, num);
                } else {
                    const unsigned by = (unsigned)(opened >> (sib << kLog)) & (unsigned)((1ull << (NT & 63)) - 1ull);
                    // one lane for each opened sibling: its first target's
                    uint64_t one = __ballot(__builtin_amdgcn_inverse_ballot_w64(opened) && (by & ((1u << tgt) - 1u)) == 0u);
                    while (one) {
                        const int l = __builtin_ctzll(one);
                        one &= one - 1ull;
                        wait((uint64_t)(unsigned)__builtin_amdgcn_readlane((int)by, l),
                             __builtin_amdgcn_readlane(me.y, l), __builtin_amdgcn_readlane(num, l));
                    }
                }
            }
            if (left > 0) {
                // the frame's next siblings
            } else if (depth > 0) {
                // the opened ones go to the stack, the first of them on top and
                // taken up at once
                if (lane > 0 && lane < depth)
                    L.stack[sp + depth - 1 - lane] = make_int4((int)w_act[0], (int)w_act[1], w_first, w_left);
                sp += depth - 1;
                depth = 0;
                enter(get(w_act, 0), __builtin_amdgcn_readlane(w_first, 0), __builtin_amdgcn_readlane(w_left, 0));
            } else if (sp > 0) {
                wave_sync();
                const int4 e = L.stack[--sp];
                enter((uint64_t)(unsigned)__builtin_amdgcn_readfirstlane(e.x) |
                          (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane(e.y) << 32,
                      __builtin_amdgcn_readfirstlane(e.z), __builtin_amdgcn_readfirstlane(e.w));
            } else {
                done = true;
            }
        }
        while (tail - head >= (done ? 1 : kWave)) drain();
    }

    if (!valid || lane >= NT) return;
    if (STATS) {
        int64_t *o = P.stats + (int64_t)orig * 4;
        o[0] = st_test;
        o[1] = st_entries;
        o[2] = st_cells;
        o[3] = st_zero;
        return;
    }
    if (PREC == START_FP64) {
        // terms are L / d^2 with d in cells: restore cm
        static_cast<double *>(P.gamma)[orig] = P.rate_scale * (double)acc / (P.cell_cm * P.cell_cm);
    } else {
        // L' = L / *lscale and lengths in cells: restore units in FP64
        const double Lref = P.n_nodes > 0 ? *P.lscale : 1.0;   // empty tree: no arrays
        const double sum = (double)acc - (double)accc;
        static_cast<float *>(P.gamma)[orig] = (float)(P.rate_scale * sum * Lref / (P.cell_cm * P.cell_cm));
    }
}

// Batched target preparation: every target of every item gets the key
// (item << mbits | Morton key of its cell, the top mbits of 30), so one radix
// sort groups the targets by item and orders each item's targets along the
// Morton curve (the order only affects speed: no target's result depends on
// its neighbours).  Positions and self indices are validated on the way.
__device__ inline unsigned spread10(unsigned v)
{
    v &= 0x3FFu;
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

__device__ inline int item_of(int64_t g, int n_items, const int64_t *offsets)
{
    int lo = 0, hi = n_items - 1;   // last item with offsets[item] <= g
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (offsets[mid] <= g) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

__global__ void __launch_bounds__(kThreads) batch_keys(int64_t n, int n_items, const int64_t *offsets,
                                                       const Item *__restrict__ items, int mbits, uint64_t *keys,
                                                       unsigned *vals, unsigned *flags)
{
    const int64_t g = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (g >= n) return;
    const int item = item_of(g, n_items, offsets);
    const Item &I = items[item];
    const int64_t j = g - offsets[item];
    unsigned bad = 0, code = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double x = I.tgt_xyz[(int64_t)k * I.n_t + j];
        double u = 0.0;
        if (!isfinite(x)) {
            bad |= kFlagNonFinite;
        } else if (x < I.lo[k] || x > I.lo[k] + I.size) {
            bad |= kFlagOutOfBox;
        } else {
            u = (x - I.lo[k]) * I.inv_size;
            u = u > 1.0 ? 1.0 : u;
        }
        unsigned q = (unsigned)(u * 1024.0);
        q = q > 1023u ? 1023u : q;
        code |= spread10(q) << (2 - k);
    }
    if (I.self_src) {
        const int64_t sv = I.self_src[j];
        if (sv < -1 || sv >= I.n_src) bad |= kFlagBadSelf;
    }
    if (bad) atomicOr(flags, bad);
    keys[g] = ((uint64_t)item << mbits) | (code >> (30 - mbits));
    vals[g] = (unsigned)g;
}

__global__ void __launch_bounds__(kThreads) batch_gather(int64_t n, const int64_t *offsets,
                                                         const Item *__restrict__ items, int mbits,
                                                         const uint64_t *keys, const unsigned *vals, double4 *tgt,
                                                         unsigned *tgt_orig)
{
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (k >= n) return;
    const int item = (int)(keys[k] >> mbits);
    const Item &I = items[item];
    const int64_t j = (int64_t)vals[k] - offsets[item];
    tgt[k] = make_double4(I.tgt_xyz[j], I.tgt_xyz[I.n_t + j], I.tgt_xyz[2 * I.n_t + j], 0.0);
    tgt_orig[k] = (unsigned)j;
}


// FP32-path copies of the virtual sources (fixed32 above, with the targets'
// encoding): the centre as 32-bit fixed-point coordinates of the box and the
// luminosity relative to the root's (every L' <= 1); and whether the node
// shines in each precision, in its sibling record.  BUILD: the whole record.
template <bool BUILD>
__global__ void __launch_bounds__(kThreads) make_fp32(const unsigned *n_nodes, int64_t n, const double4 *mom,
                                                      const double4 *src, const double *lscale, start_box box,
                                                      double inv, uint4 *momq, Sibling *sib, uint4 *srcq,
                                                      const int *order, const int2 *kids, const int4 *geo,
                                                      const int *first, const int *count, const int *ref)
{
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const double Lref = *lscale;
    auto encode = [&](const double4 v) {
        return make_uint4(fixed32(v.x, box.lo[0], inv), fixed32(v.y, box.lo[1], inv), fixed32(v.z, box.lo[2], inv),
                          __float_as_uint((float)(v.w / Lref)));
    };
    if (k < (int64_t)*n_nodes) {
        const int p = BUILD ? order[k] : sib[k].node;
        const double4 v = mom[p];
        const uint4 q = encode(v);
        momq[p] = q;
        const int lit = (v.w > 0.0 ? 1 : 0) | (__uint_as_float(q.w) > 0.f ? 2 : 0);
        if (BUILD) {
            const int4 g = geo[p];
            const int kind = g.w >> 8;
            const int2 kd = kids[p];
            const double4 b = cube_of(g);
            sib[k] = Sibling{{b.x, b.y, b.z, b.w},
                             p,
                             kind == kKindBucket ? first[p] : kd.x,
                             lit | (kind << 2) | (kd.y << 4),
                             kind == kKindLeaf ? ref[p] : (kind == kKindBucket ? count[p] : 0)};
        } else {
            sib[k].bits = (sib[k].bits & ~3) | lit;
        }
    }
    if (k < n) srcq[k] = encode(src[k]);
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

}  // namespace

void make_fp32_tree(Tree *t, hipStream_t s)
{
    if (t->n_nodes == 0) return;
    const int64_t k = std::max(t->n_nodes, t->n_src);
    make_fp32<false><<<blocks_for(k), kThreads, 0, s>>>(t->d_nodes, t->n_src, t->mom, t->src, t->lscale, t->box,
                                                        1.0 / t->box.size, t->momq, t->sib, t->srcq, nullptr, nullptr,
                                                        nullptr, nullptr, nullptr, nullptr);
}

void make_siblings(Tree *t, int64_t max_nodes, const int *order, const int2 *kids, hipStream_t s)
{
    make_fp32<true><<<blocks_for(max_nodes), kThreads, 0, s>>>(t->d_nodes, t->n_src, t->mom, t->src, t->lscale, t->box,
                                                               1.0 / t->box.size, t->momq, t->sib, t->srcq, order, kids,
                                                               t->geo, t->first, t->count, t->ref);
}

// ------------------------------------------------------------------------
// Batch launcher.  All items of a call share one sort of their targets and
// one persistent launch per precision; a single start_compute_rates is a
// batch of one item.
// ------------------------------------------------------------------------
namespace {

struct BatchScratch {
    uint64_t *keys;
    unsigned *vals;
    double4 *tgt;
    unsigned *tgt_orig;
    Item *items;
    int64_t *offsets;
    int4 *tiles;
    void *radix_tmp;
};

size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

size_t stage_bytes(int n_items, int64_t n_tiles)
{
    return al256((size_t)n_items * sizeof(Item)) + al256((size_t)(n_items + 1) * sizeof(int64_t)) +
           al256((size_t)n_tiles * sizeof(int4));
}

BatchScratch carve_batch(void *base, int64_t n, int n_items, int64_t n_tiles)
{
    const int64_t nk = n > 1 ? n : 1;
    char *q = (char *)base;
    BatchScratch b;
    b.items = (Item *)q;   // the staged block first: items, offsets, tiles
    q += al256((size_t)n_items * sizeof(Item));
    b.offsets = (int64_t *)q;
    q += al256((size_t)(n_items + 1) * sizeof(int64_t));
    b.tiles = (int4 *)q;
    q += al256((size_t)n_tiles * sizeof(int4));
    b.keys = (uint64_t *)q;
    q += al256((size_t)nk * sizeof(uint64_t));
    b.vals = (unsigned *)q;
    q += al256((size_t)nk * sizeof(unsigned));
    b.tgt = (double4 *)q;
    q += al256((size_t)nk * sizeof(double4));
    b.tgt_orig = (unsigned *)q;
    q += al256((size_t)nk * sizeof(unsigned));
    b.radix_tmp = q;
    return b;
}

template <int PREC, bool STATS>
void launch_tiles(const Item *items, const int4 *tiles, int64_t n_tiles, const BatchLaunch &b, hipStream_t s)
{
    int64_t blocks = (n_tiles + kWavesPerBlock - 1) / kWavesPerBlock;
    if (blocks >= 64) blocks = (blocks + 7) / 8 * 8;   // whole rounds over the 8 XCDs
    auto go = [&](auto kernel) { kernel<<<(unsigned)blocks, kThreads, 0, s>>>(items, tiles, (int)n_tiles); };
    auto pick = [&](auto nt) {   // targets per wave
        constexpr int NT = decltype(nt)::value;
        constexpr bool kOrdered = PREC == START_FP32C && !STATS;   // (counters have no order)
        if (kOrdered && b.depth_first) {
            if (b.clamp) go(rates_kernel<PREC, STATS, true, NT, kOrdered>);
            else go(rates_kernel<PREC, STATS, false, NT, kOrdered>);
        } else {
            if (b.clamp) go(rates_kernel<PREC, STATS, true, NT, false>);
            else go(rates_kernel<PREC, STATS, false, NT, false>);
        }
    };
    if constexpr (!STATS) {
        if (b.tile <= 8) return pick(std::integral_constant<int, 8>{});
        if (b.tile <= 16) return pick(std::integral_constant<int, 16>{});
        if (b.tile <= 32) return pick(std::integral_constant<int, 32>{});
    }
    pick(std::integral_constant<int, 64>{});
}

// Whether any item's grid has no guard band (G = 1024): the launch then
// clamps every march step.
bool needs_clamp(const RateSpec *specs, int n)
{
    for (int i = 0; i < n; ++i)
        if (specs[i].grid && specs[i].grid->guard == 0) return true;
    return false;
}

}  // namespace

size_t batch_stage_bytes(int n_items, int64_t n_tiles) { return stage_bytes(n_items, n_tiles); }

size_t batch_scratch_bytes(int64_t n, int n_items, int64_t n_tiles)
{
    const int64_t nk = n > 1 ? n : 1;
    return stage_bytes(n_items, n_tiles) + al256((size_t)nk * sizeof(uint64_t)) +
           al256((size_t)nk * sizeof(unsigned)) + al256((size_t)nk * sizeof(double4)) +
           al256((size_t)nk * sizeof(unsigned)) + al256(radix_temp_bytes(nk)) + 256;
}

int64_t batch_tiles(const RateSpec *specs, int n, int tile)
{
    int64_t t = 0;
    for (int i = 0; i < n; ++i) t += (specs[i].n_t + tile - 1) / tile;
    return t;
}

namespace {

// The table entry of one rate problem; its targets are the run [off, off +
// n_t) of the batch's sorted target arrays in bs.
Item make_item(const RateSpec &r, const BatchScratch &bs, int64_t off)
{
    const Tree *t = r.tree;
    const Grid *g = r.grid;
    Item I;
    memset(&I, 0, sizeof(I));
    I.n_nodes = t->n_nodes;
    I.n_src = t->n_src;
    I.geo = t->geo;
    I.skip = t->skip;
    I.first = t->first;
    I.count = t->count;
    I.ref = t->ref;
    I.mom = t->mom;
    I.momq = t->momq;
    I.lscale = t->lscale;
    I.src = t->src;
    I.srcq = t->srcq;
    I.perm = t->perm;
    I.sib = t->sib;
    if (g) {
        I.grid = g->val;
        I.gridf = g->valf;
        I.G = g->G;
        I.grid_log2 = g->grid_log2;
        I.sx = g->sx;
        I.sy = g->sy;
        I.guard = g->guard;
    } else {
        I.G = 1;
        I.grid_log2 = 0;
        I.sx = I.sy = 1;
    }
    I.frac_scale = ldexp(1.0, -(32 - I.grid_log2));
    I.gs = (double)I.G / t->box.size;
    for (int k = 0; k < 3; ++k) I.lo[k] = t->box.lo[k];
    I.size = t->box.size;
    I.inv_size = 1.0 / t->box.size;
    I.unit_cm = t->box.length_unit_cm;
    I.cell_cm = t->box.size / I.G * t->box.length_unit_cm;
    I.theta2 = r.theta * r.theta;
    I.sigma = r.sigma;
    I.channel = r.channel;
    I.col_scale = r.channel == 0 ? r.sigma * I.cell_cm : I.cell_cm * 1e-14;
    I.rate_scale = (r.channel == 0 ? r.sigma : 1.13e8) / (4.0 * M_PI);
    I.n_t = r.n_t;
    I.tgt_xyz = r.tgt_xyz;
    I.tgt = bs.tgt + off;
    I.tgt_orig = bs.tgt_orig + off;
    I.self_src = r.self_src;
    I.gamma = r.gamma;
    I.counts = r.counts;
    I.offsets = r.offsets;
    I.entries = r.entries;
    I.stats = r.stats;
    return I;
}

// Bits of an item's number in the sort keys of a batch.
int item_key_bits(int n_items)
{
    int bits = 0;
    while (((int64_t)1 << bits) < n_items) ++bits;
    return bits;
}

// Morton bits of the targets' order, so that the whole key is a few digits of 8
// bits: a pass of the sort takes 12-14 us (two launches), or ~4 of the one launch
// up to 8192 targets, and the order only has to bring together what a tile
// marches.
// Two digits up to 2^16 targets of at most 1024 sources, whose rays and walks
// are few: a call on 16457 uniform targets of 64 sources takes 137 us with three
// and 126 with two (65536 of 1024 sources: 22 us less with two, in clusters 3
// more).  Where all particles emit, clusters need the third digit (65536 of
// them: 1440 us, 1541 with two).  Three up to
// 2^18 targets (64 cells a target there).  Four beyond, the item's number among
// them as long as no item is larger than that.
int morton_bits(const RateSpec *specs, int n, int64_t n_targets)
{
    const int item_bits = item_key_bits(n);
    int64_t max_src = 0, max_t = 0;
    for (int i = 0; i < n; ++i) {
        max_src = std::max(max_src, specs[i].tree->n_src);
        max_t = std::max(max_t, specs[i].n_t);
    }
    if (item_bits > 9 || max_t > ((int64_t)1 << 18)) return 30;
    if (n_targets > ((int64_t)1 << 18)) return (32 - item_bits) / 3 * 3;
    if (n_targets <= 65536 && max_src <= 1024 && item_bits == 0) return 16;
    return (24 - item_bits) / 3 * 3;
}

// Device part of a batch whose tables are in place: target keys, sort and
// gather, then the kernels of the mode.
void launch_staged(const BatchScratch &bs, int64_t N, int n, int64_t n_tiles, int64_t n64, int mode, bool clamp,
                   int tile, bool depth_first, int mbits, unsigned *flags, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1,
                   BatchLaunch *launch)
{
    if (N == 0) return;
    const unsigned nb = (unsigned)((N + kThreads - 1) / kThreads);
    const int item_bits = item_key_bits(n);
    batch_keys<<<nb, kThreads, 0, s>>>(N, n, bs.offsets, bs.items, mbits, bs.keys, bs.vals, flags);
    const SortedPairs sp = radix_sort_pairs(bs.keys, bs.vals, N, mbits + item_bits, bs.radix_tmp, s);
    batch_gather<<<nb, kThreads, 0, s>>>(N, bs.offsets, bs.items, mbits, sp.keys, sp.vals, bs.tgt, bs.tgt_orig);

    if (mode == 2 || mode == 3 || mode == 4) {
        const unsigned lb = (unsigned)((n_tiles + kWavesPerBlock - 1) / kWavesPerBlock);
        if (mode == 2) list_kernel<kCount><<<lb, kThreads, 0, s>>>(bs.items, bs.tiles, (int)n_tiles);
        else if (mode == 3) list_kernel<kList><<<lb, kThreads, 0, s>>>(bs.items, bs.tiles, (int)n_tiles);
        else list_kernel<kKeys><<<lb, kThreads, 0, s>>>(bs.items, bs.tiles, (int)n_tiles);
        return;
    }
    BatchLaunch bl{bs.items, bs.tiles, n_tiles, n64, mode, clamp, tile, depth_first};
    if (launch) *launch = bl;
    if (ev0) hipEventRecord(ev0, s);
    relaunch_batch(bl, s);
    if (ev1) hipEventRecord(ev1, s);
}

static_assert(sizeof(Item) <= 1024, "the item table entry is passed as a kernel argument");

// The tables of a one-item batch written on the device from the kernel
// argument (no host staging): the item, its offsets (0, n_t) and its tiles.
__global__ void __launch_bounds__(kThreads) single_tables(Item I, int tile, int64_t n_tiles, Item *items,
                                                          int64_t *offsets, int4 *tiles)
{
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (k == 0) {
        *items = I;
        offsets[0] = 0;
        offsets[1] = I.n_t;
    }
    if (k < n_tiles) {
        const int64_t f = k * tile;
        tiles[k] = make_int4(0, (int)f, (int)(I.n_t - f < tile ? I.n_t - f : tile), 0);
    }
}

}  // namespace

// Enqueues a batch (the scratch and the pinned staging area must be large
// enough: batch_scratch_bytes / stage_bytes).  mode: 0 rates, 1 counters,
// 2 list counts, 3 lists.  ev0/ev1 (may be null) bracket the rate kernels.
void run_batch(Ctx *c, const RateSpec *specs, int n, int mode, int tile, void *scratch, hipEvent_t ev0,
               hipEvent_t ev1, BatchLaunch *launch)
{
    hipStream_t s = c->stream;
    int64_t N = 0;
    for (int i = 0; i < n; ++i) N += specs[i].n_t;
    const int64_t n_tiles = batch_tiles(specs, n, tile);
    BatchScratch bs = carve_batch(scratch, N, n, n_tiles);

    // host side: item table, offsets, tiles (FP64 items' tiles first)
    hipEventSynchronize(c->stage_ev);   // the previous upload has been read
    char *h = (char *)c->host_stage;
    Item *hi = (Item *)h;
    int64_t *ho = (int64_t *)(h + al256((size_t)n * sizeof(Item)));
    int4 *ht = (int4 *)(h + al256((size_t)n * sizeof(Item)) + al256((size_t)(n + 1) * sizeof(int64_t)));
    int64_t off = 0;
    for (int i = 0; i < n; ++i) {
        hi[i] = make_item(specs[i], bs, off);
        ho[i] = off;
        off += specs[i].n_t;
    }
    ho[n] = off;
    int64_t t64 = 0;
    for (int pass = 0; pass < 2; ++pass)   // FP64 items, then FP32C items
        for (int i = 0; i < n; ++i) {
            if ((specs[i].prec == START_FP64) != (pass == 0)) continue;
            for (int64_t f = 0; f < specs[i].n_t; f += tile)
                ht[t64++] = make_int4(i, (int)f, (int)(specs[i].n_t - f < tile ? specs[i].n_t - f : tile), 0);
        }
    int64_t n64 = 0;
    for (int i = 0; i < n; ++i)
        if (specs[i].prec == START_FP64) n64 += (specs[i].n_t + tile - 1) / tile;
    hipMemcpyAsync(bs.items, h, stage_bytes(n, n_tiles), hipMemcpyHostToDevice, s);
    hipEventRecord(c->stage_ev, s);
    launch_staged(bs, N, n, n_tiles, n64, mode, needs_clamp(specs, n), tile, specs[0].depth_first,
                  morton_bits(specs, n, N), c->d_flags, s, ev0, ev1, launch);
}

void run_single_fixed(Ctx *c, const RateSpec &r, int tile, void *scratch)
{
    hipStream_t s = c->stream;
    const int64_t n_tiles = batch_tiles(&r, 1, tile);
    BatchScratch bs = carve_batch(scratch, r.n_t, 1, n_tiles);
    const Item I = make_item(r, bs, 0);
    const int64_t nb = (n_tiles + kThreads - 1) / kThreads;
    single_tables<<<(unsigned)(nb > 0 ? nb : 1), kThreads, 0, s>>>(I, tile, n_tiles, bs.items, bs.offsets, bs.tiles);
    launch_staged(bs, r.n_t, 1, n_tiles, r.prec == START_FP64 ? n_tiles : 0, 0, needs_clamp(&r, 1), tile, r.depth_first,
                  morton_bits(&r, 1, r.n_t), c->d_flags, s, nullptr, nullptr, nullptr);
}

void relaunch_batch(const BatchLaunch &b, hipStream_t s)
{
    const Item *items = static_cast<const Item *>(b.items);
    if (b.n64 > 0) {
        if (b.mode == 1) launch_tiles<START_FP64, true>(items, b.tiles, b.n64, b, s);
        else launch_tiles<START_FP64, false>(items, b.tiles, b.n64, b, s);
    }
    if (b.n_tiles - b.n64 > 0) {
        if (b.mode == 1)
            launch_tiles<START_FP32C, true>(items, b.tiles + b.n64, b.n_tiles - b.n64, b, s);
        else
            launch_tiles<START_FP32C, false>(items, b.tiles + b.n64, b.n_tiles - b.n64, b, s);
    }
}

// ---------------------------------------------------------------------------
// Upstream-particle chain: optical depth of the pairs (particle, source) that
// have no upstream particle, integrated along the ray as in the rate kernel
// (FP64).  key: node << 32 | (bucket member + 1, or 0).
// ---------------------------------------------------------------------------
namespace {

template <bool CLAMP>
__global__ void __launch_bounds__(256) upstream_roots(int64_t n_roots, const unsigned *__restrict__ roots,
                                                      const uint64_t *__restrict__ keys,
                                                      const unsigned *__restrict__ owner, const double *__restrict__ xyz,
                                                      int64_t n, const double4 *__restrict__ mom,
                                                      const double4 *__restrict__ src, const int *__restrict__ first,
                                                      const double *__restrict__ grid, int64_t guard, int G, int sx,
                                                      int sy, double lo0,
                                                      double lo1, double lo2, double gs, double tau_scale,
                                                      unsigned *__restrict__ links, int link_words)
{
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r >= n_roots) return;
    const unsigned p = roots[r];
    const unsigned i = owner[p];
    const double4 a = source_of_key(mom, src, first, keys[p]);
    const double lo[3] = {lo0, lo1, lo2};
    const double x[3] = {xyz[i], xyz[n + i], xyz[2 * n + i]};
    const double A[3] = {(a.x - lo[0]) * gs, (a.y - lo[1]) * gs, (a.z - lo[2]) * gs};
    int tb[3];
    double fb[3], D[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double B = (x[k] - lo[k]) * gs;
        int b = (int)floor(B);
        b = b < 0 ? 0 : (b > G - 1 ? G - 1 : b);
        tb[k] = b;
        fb[k] = B - (double)b;
        D[k] = A[k] - ((double)tb[k] + fb[k]);
    }
    const double d2 = D[0] * D[0] + D[1] * D[1] + D[2] * D[2];
    unsigned *const out = links + (int64_t)p * link_words;
    auto put = [&](double tau) {
        out[0] = (unsigned)__double2loint(tau);
        out[1] = (unsigned)__double2hiint(tau);
    };
    if (!(d2 > 0.0)) {
        put(0.0);
        return;
    }
    int nc = 0;
    const unsigned e0 = (unsigned)(tb[0] * sx + tb[1] * sy + tb[2] + guard);
    const double col = march<double, false, CLAMP>(grid - guard, sx, sy, (unsigned)((G - 1) * (sx + sy + 1) + guard),
                                                   e0, fb, D, nc);
    put(tau_scale * (col * sqrt(d2)));
}

}  // namespace

void launch_upstream_roots(Ctx *c, const Tree *t, const Grid *g, int64_t n_roots, const unsigned *roots,
                           const uint64_t *keys, const unsigned *owner, const double *xyz, int64_t n, double sigma,
                           void *links)
{
    if (n_roots <= 0) return;
    const double gs = (double)g->G / t->box.size;
    const double tau_scale = sigma * (t->box.size / g->G * t->box.length_unit_cm);
    const unsigned nb = (unsigned)((n_roots + 255) / 256);
    const int link_words = (int)(upstream_link_bytes() / sizeof(unsigned));
    if (g->guard == 0)
        upstream_roots<true><<<nb, 256, 0, c->stream>>>(n_roots, roots, keys, owner, xyz, n, t->mom, t->src, t->first,
                                                        g->val, g->guard, g->G, g->sx, g->sy, t->box.lo[0],
                                                        t->box.lo[1], t->box.lo[2], gs, tau_scale, (unsigned *)links,
                                                        link_words);
    else
        upstream_roots<false><<<nb, 256, 0, c->stream>>>(n_roots, roots, keys, owner, xyz, n, t->mom, t->src,
                                                         t->first, g->val, g->guard, g->G, g->sx, g->sy, t->box.lo[0],
                                                         t->box.lo[1], t->box.lo[2], gs, tau_scale, (unsigned *)links,
                                                        link_words);
}

}  // namespace start
