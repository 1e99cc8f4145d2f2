// Neutral-hydrogen field for the ray integrals, on a G^3 grid over the box.
//
// The paper integrates the optical depth along each light ray through the SPH
// particles (sections 2.2.1-2.2.2).  Here the field is first interpolated to
// the grid cell centres with the SPH kernel of section 2.1 (cubic spline,
// support 2h) in Shepard-normalised form,
//     n_c = sum_k n_k W(|x_c - r_k|, h_k) / sum_k W(|x_c - r_k|, h_k),
// 0 where no kernel reaches, and every ray then integrates the piecewise-
// constant field exactly.  Particles are split into a few classes by their
// support 2h (chosen from a histogram of 2h to minimise the scan work) and
// counting-sorted by (class, cell), stable, so sums run in a fixed order;
// each cell centre gathers, class by class, from the cells within that
// class's largest support.
#include "internal.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace start {

namespace {

constexpr int kThreads = 256;

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

constexpr int kBins = 256;   // reach bins of a quarter cell; the last also holds every larger reach

// Quarter-cell bin of a particle's kernel support 2h: ceil(4 * 2h / delta).
__device__ inline int reach_bin(double h, double gs)
{
    const double u = ceil(8.0 * h * gs);
    return u < (double)(kBins - 1) ? (int)u : kBins - 1;
}

__global__ void __launch_bounds__(kThreads) grid_keys(start_box box, double gs, int G, int64_t n,
                                                      const double *xyz, const double *h, const double *nhi,
                                                      uint64_t *keys, unsigned *idx, unsigned *flags,
                                                      unsigned *hist, unsigned long long *hmax_bits)
{
    __shared__ unsigned lh[kBins];
    __shared__ double wmax[kThreads / 64];
    for (int t = threadIdx.x; t < kBins; t += kThreads) lh[t] = 0;
    __syncthreads();
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    double reach = 0.0;
    int bin = -1;   // reach bin of a valid particle
    if (k < n) {
        unsigned bad = 0;
        int c[3];
        for (int a = 0; a < 3; ++a) {
            const double x = xyz[(int64_t)a * n + k];
            if (!isfinite(x)) bad |= kFlagNonFinite;
            else if (x < box.lo[a] || x > box.lo[a] + box.size) bad |= kFlagOutOfBox;
            double g = isfinite(x) ? (x - box.lo[a]) * gs : 0.0;
            int v = (int)floor(g);
            c[a] = v < 0 ? 0 : (v >= G ? G - 1 : v);
        }
        const double hk = h[k], nk = nhi[k];
        if (!isfinite(hk) || !isfinite(nk)) bad |= kFlagNonFinite;
        else if (!(hk > 0.0) || nk < 0.0) bad |= kFlagNegative;
        if (bad) {
            atomicOr(flags, bad);
        } else {
            reach = 2.0 * hk;
            bin = reach_bin(hk, gs);
        }
        keys[k] = ((uint64_t)c[0] * G + c[1]) * G + c[2];
        idx[k] = (unsigned)k;
    }
    // histogram: one LDS atomic per distinct bin of the wave (most particles
    // share one or two bins, and same-address atomics serialise)
    for (;;) {
        const uint64_t left = __ballot(bin >= 0);
        if (!left) break;
        const int b = __shfl(bin, __ffsll((unsigned long long)left) - 1, 64);
        const uint64_t same = __ballot(bin == b);
        if (bin == b) {
            if ((__lane_id() == __ffsll((unsigned long long)same) - 1)) atomicAdd(&lh[b], (unsigned)__popcll(same));
            bin = -1;
        }
    }
    // largest reach of the block, one atomic per block (positive doubles
    // order like their bit patterns)
    for (int o = 32; o > 0; o >>= 1) reach = fmax(reach, __shfl_xor(reach, o, 64));
    if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = reach;
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = wmax[0];
        for (int w = 1; w < kThreads / 64; ++w) m = fmax(m, wmax[w]);
        if (m > 0.0) atomicMax(hmax_bits, (unsigned long long)__double_as_longlong(m));
    }
    for (int t = threadIdx.x; t < kBins; t += kThreads)
        if (lh[t]) atomicAdd(&hist[t], lh[t]);
}

// The validation word, the reach histogram and the largest reach bits,
// copied by one block into the context's pinned readback words (one host
// wait for all three).
__global__ void grid_readback(const unsigned *bflags, const unsigned *hist, const unsigned long long *hmax,
                              unsigned *rb)
{
    for (int k = threadIdx.x; k < kBins; k += blockDim.x) rb[1 + k] = hist[k];
    if (threadIdx.x == 0) {
        rb[0] = *bflags;
        const unsigned long long v = *hmax;
        rb[1 + kBins] = (unsigned)v;
        rb[2 + kBins] = (unsigned)(v >> 32);
    }
}

// Class-major keys: class * G^3 + cell; top.{x,y,z} are the last bins of
// classes 0..2 (kBins where the class is unused).
__global__ void __launch_bounds__(kThreads) class_keys(int64_t n, const double *h, double gs, int64_t ncell,
                                                       int4 top, uint64_t *keys)
{
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (k >= n) return;
    const int bin = reach_bin(h[k], gs);
    const int cls = (bin > top.x) + (bin > top.y) + (bin > top.z);
    keys[k] += (uint64_t)cls * (uint64_t)ncell;
}

__global__ void __launch_bounds__(kThreads) cell_counts(const uint64_t *keys, int64_t n, unsigned *start)
{
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (k >= n) return;
    atomicAdd(&start[keys[k]], 1u);
}

__global__ void __launch_bounds__(kThreads) invert_perm(int64_t n, const unsigned *perm, unsigned *inv)
{
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (k >= n) return;
    inv[perm[k]] = (unsigned)k;
}

// The binned particle arrays, written from the particles in input order
// (reads in order, each particle's three records written to its binned
// place; gathering through the permutation instead reads five scattered
// doubles per particle).
__global__ void __launch_bounds__(kThreads) scatter_particles(int64_t n, const unsigned *inv, const double *xyz,
                                                              const double *h, const double *nhi, double4 *pos_h,
                                                              double2 *kern, double *ns)
{
    const int64_t o = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (o >= n) return;
    const unsigned k = inv[o];
    const double hk = h[o];
    pos_h[k] = make_double4(xyz[o], xyz[n + o], xyz[2 * n + o], hk);
    // 1/h and the 3-D normalisation 1/(pi h^3) of the kernel, once per particle
    kern[k] = make_double2(1.0 / hk, 1.0 / (M_PI * hk * hk * hk));
    ns[k] = nhi[o];
}

__global__ void __launch_bounds__(kThreads) gather_values(int64_t n, const unsigned *perm, const double *nhi,
                                                          double *ns)
{
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (k >= n) return;
    ns[k] = nhi[perm[k]];
}

// M4 cubic spline of section 2.1 with 3-D normalisation 1/(pi h^3), from
// q = r / h and the normalisation, without branches: 0.25 (2 - q)^3 less
// (1 - q)^3 below q = 1 is the inner polynomial 1 - 1.5 q^2 + 0.75 q^3, and
// both cubes vanish from q = 2 on.
__device__ inline double kernel_w(double q, double norm)
{
    const double t2 = fmax(2.0 - q, 0.0), t1 = fmax(1.0 - q, 0.0);
    return (0.25 * (t2 * t2 * t2) - t1 * t1 * t1) * norm;
}

// sqrt(x) for 0 <= x (finite): the hardware reciprocal square root and one
// Newton step on the root, ~1e-15 relative (the library sqrt rounds
// correctly but takes ~4x the instructions).  Below 1e-200 the result is
// ~1e-100 instead of x^(1/2): kernel weights are then W(0) either way.
__device__ inline double sqrt_nr(double x)
{
    const double xm = fmax(x, 1e-200);
    const double y = __builtin_amdgcn_rsq(xm);
    const double r = xm * y;
    return fma(0.5 * y, fma(-r, r, xm), r);
}

constexpr int kCellsZ = 4;    // cell centres per group, consecutive along z
constexpr int kSlices = 8;    // lanes of a group
constexpr int kGroups = 64 / kSlices;                 // groups of a wave
constexpr int kRows = 1024;   // stencil rows listed at a time
constexpr int kList = 192;    // particles listed per group: emptied above kList - 64
constexpr int kTake = kSlices;                        // particles a lane lists per round
constexpr int kAhead = 4;                             // rows a lane looks up at once

enum ShepardMode { kGather = 0, kGatherCount = 1, kFillPairs = 2 };
constexpr unsigned long long kMaxPairs = 1ull << 29;   // recorded pairs: at most 6 GiB

// Number of pairs of slices 0..s-1 in a cell's eight one-byte counts.
__device__ inline unsigned pairs_before(uint2 c, int s)
{
    unsigned n = 0;
#pragma unroll
    for (int i = 0; i < kSlices; ++i) n += i < s ? ((i < 4 ? c.x : c.y) >> (8 * (i & 3))) & 0xFFu : 0u;
    return n;
}

// The Shepard sums.  Eight lanes (slices) share a group of kCellsZ consecutive
// cell centres of one z row, which share x and y, so every particle is read
// once for all of them.  Per reach class, the rows of cells within the class
// reach are scanned: a particle in cell (a, b, c) is at least (|a - ia| -
// 1/2)_+ cells from a centre in cell ia along x (likewise y, z), so the
// stencil is the set of cells whose nearest point lies within the reach; the
// row geometry runs in float on a widened reach, so the stencil can only grow.
// The support test itself is exact (FP64).
//
// The block lists the stencil's rows once (offset, half-length, class) in
// LDS, those that lie outside the grid for all its centres left out.  A class
// of fewer particles than its stencil has rows (a few wide kernels, or fewer
// particles than cells) is taken whole instead, in one part per lane: looking
// up its rows would cost more than testing its particles (one kernel of
// 2h = 1.2 boxes among 2^20 particles on 128^3 cells: 62 ms by rows, 0.8 whole;
// the line was measured at 1000 kernels of 2h = 0.2 boxes, 2000 rows: 2.2 ms
// whole, 2.9 by rows).
// Then a group's lanes look up kAhead rows each, their loads under way
// together, and append the rows' particles (at most kTake each per round, in
// lane order) to the group's list in LDS; from there they go to the lanes in
// turn, entry j to lane j mod 8, so the lanes are busy alike whatever the rows
// hold.  (16384 particles on 128^3 cells, whose rows are nearly all empty: the
// build takes 1166 us with one row at a time, 961 with four, 934 with six; one
// particle per cell on 64^3 cells: 290 to 300 with any.)  Each lane sums its
// entries in order and the eight sums are added by a butterfly, a fixed order.
//
// What bounds it: FP64 ALU on large grids (~27 instructions per centre and
// listed particle, of which ~60% lie in the support), latency on small ones.
// A thread per group looping over its rows by itself had 8 times fewer waves
// (128 on a 32^3 grid, on 1024 SIMDs) and waited in each row for the lane with
// the longest run: 195 us on 32^3, 239 on 64^3, 771 on 128^3; now 26, 87 and
// 600 (alone).
//
// kGatherCount also counts the (centre, particle) pairs inside the support of
// each centre and slice; kFillPairs records them with their weights, slice by
// slice in summation order, and the weight sums (for refills with new n_HI at
// the same positions, refill_pairs).  The pairs of 64 consecutive cells are
// stored interleaved (pair q of the group's cell l at q * 64 + l, the group
// padded to its longest list), so that a wave refilling those cells reads
// consecutive addresses at every step.
template <int MODE>
__global__ void __launch_bounds__(kThreads)
__attribute__((amdgpu_waves_per_eu(MODE == kFillPairs ? 3 : 4)))
shepard_gather(start_box box, double delta, int G, ReachClasses cls, const unsigned *__restrict__ start,
               const double4 *__restrict__ pos_h, const double2 *__restrict__ kern, const double *__restrict__ ns,
               double *val, float *valf, int sx, int sy, uint2 *__restrict__ pslice, unsigned *__restrict__ pcount,
               const unsigned *__restrict__ pstart, unsigned *__restrict__ pidx, double *__restrict__ pw,
               double *__restrict__ pden, unsigned *__restrict__ many)
{
    __shared__ int2 row_all[kRows];             // (da << 16 | db & 0xffff, half-length << 2 | class),
                                                // or (part of a class, -1 - class)
    __shared__ unsigned list_all[kThreads / 64][kGroups][kList];
    __shared__ int wrows[kThreads / 64];
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    const int g = lane / kSlices, sl = lane % kSlices;
    unsigned *const list = list_all[w][g];
    const int GZ = (G + kCellsZ - 1) / kCellsZ;   // groups per z row
    const int64_t n_groups = (int64_t)G * G * GZ;
    // blocks are dealt round-robin to the 8 XCDs: each gets a contiguous part
    // of the grid, whose particles stay in its L2
    const int log2g = __builtin_ctz((unsigned)G);
    const int nb = (int)gridDim.x, per_xcd = nb / 8;
    int blk = (int)blockIdx.x;
    if (per_xcd > 0 && blk < per_xcd * 8) blk = (blk & 7) * per_xcd + (blk >> 3);
    const int64_t lin = ((int64_t)blk * (kThreads / 64) + w) * kGroups + g;
    const bool live = lin < n_groups;
    const int64_t ncell = (int64_t)G * G * G;
    const int ia = live ? (int)(lin / ((int64_t)G * GZ)) : 0, ib = live ? (int)((lin / GZ) % G) : 0;
    const int ic0 = live ? (int)(lin % GZ) * kCellsZ : 0;
    const int nz = G - ic0 < kCellsZ ? G - ic0 : kCellsZ;
    const int64_t cell0 = ((int64_t)ia * G + ib) * G + ic0;   // unpadded index of the first centre
    const double xc = box.lo[0] + ((double)ia + 0.5) * delta;
    const double yc = box.lo[1] + ((double)ib + 0.5) * delta;
    double zc[kCellsZ], num[kCellsZ], den[kCellsZ];
    unsigned cnt[kCellsZ];        // this slice's pairs; kFillPairs: the next one's place in the cell's list
#pragma unroll
    for (int j = 0; j < kCellsZ; ++j) {
        zc[j] = box.lo[2] + ((double)(ic0 + j) + 0.5) * delta;
        num[j] = 0.0;
        den[j] = 0.0;
        cnt[j] = MODE == kFillPairs && live && j < nz ? pairs_before(pslice[cell0 + j], sl) : 0u;
    }
    int listed = 0;               // entries of the group's list

    // The listed particles, entry j by lane j mod 8; the next one's record is
    // loaded while this one's weights are computed.
    auto empty_list = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        unsigned at = sl < listed ? list[sl] : 0u;
        double4 pn = make_double4(0.0, 0.0, 0.0, 0.0);
        double2 kn = make_double2(0.0, 0.0);
        double nn = 0.0;
        if (sl < listed) {
            pn = pos_h[at];
            kn = kern[at];
            nn = ns[at];
        }
        for (int j = sl; j < listed; j += kSlices) {
            const unsigned s = at;
            const double4 p = pn;
            const double2 kk = kn;
            const double nk = nn;
            if (j + kSlices < listed) {
                at = list[j + kSlices];
                pn = pos_h[at];
                kn = kern[at];
                nn = ns[at];
            }
            const double dx = xc - p.x, dy = yc - p.y;
            const double dxy2 = dx * dx + dy * dy, h2 = 4.0 * p.w * p.w;
            if (!(dxy2 < h2)) continue;
            // the four centres without branches: a centre outside the support
            // 2h (or past the row's end) adds 0
#pragma unroll
            for (int c = 0; c < kCellsZ; ++c) {
                const double dz = zc[c] - p.z;
                const double r2 = dxy2 + dz * dz;
                const bool in = c < nz && r2 < h2;
                if (MODE == kGatherCount) cnt[c] += in ? 1u : 0u;
                const double wt = in ? kernel_w(sqrt_nr(r2) * kk.x, kk.y) : 0.0;
                num[c] = fma(nk, wt, num[c]);
                den[c] += wt;
                if (MODE == kFillPairs && in) {
                    // pair q of cell c: group c / 64, place q * 64 + c % 64
                    const int64_t cell = cell0 + c;
                    const int64_t to = (int64_t)pstart[cell >> 6] + (int64_t)cnt[c] * 64 + (cell & 63);
                    pidx[to] = s;
                    pw[to] = wt;
                    ++cnt[c];
                }
            }
        }
        listed = 0;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    // the cells of the block's centres: x from A0 to A1, y from B0 to B1
    const int64_t lin0 = (int64_t)blk * (kThreads / kSlices);
    const int64_t lin1 = min(lin0 + kThreads / kSlices, n_groups) - 1;
    const int A0 = (int)(lin0 / ((int64_t)G * GZ)), A1 = (int)(lin1 / ((int64_t)G * GZ));
    const int B0 = A0 == A1 ? (int)((lin0 / GZ) % G) : 0, B1 = A0 == A1 ? (int)((lin1 / GZ) % G) : G - 1;
    // all rows of the classes' squares that meet the grid, kRows at a time
    int first_row[kMaxReachClasses + 1], a_lo[kMaxReachClasses], b_lo[kMaxReachClasses], n_b[kMaxReachClasses];
    first_row[0] = 0;
#pragma unroll
    for (int k = 0; k < kMaxReachClasses; ++k) {
        const int R = cls.R[k];
        a_lo[k] = max(-R, -A1);
        b_lo[k] = max(-R, -B1);
        n_b[k] = min(R, G - 1 - B0) - b_lo[k] + 1;
        const int n_a = min(R, G - 1 - A0) - a_lo[k] + 1;
        first_row[k + 1] = first_row[k] + (k < cls.K ? (cls.whole[k] ? kSlices : n_a * n_b[k]) : 0);
    }
    for (int base = 0; base < first_row[kMaxReachClasses]; base += kRows) {
        // 1. the rows that reach the centres, in order
        int rows = 0;
        __syncthreads();
        for (int q = 0; q < kRows; q += kThreads) {
            const int r = base + q + (int)threadIdx.x;
            bool in = false;
            int2 e = make_int2(0, 0);
            if (r < first_row[kMaxReachClasses]) {
                int k = 0, i = r, al = a_lo[0], bl = b_lo[0], nb = n_b[0], whole = cls.whole[0];
                float q2 = cls.q2[0];
#pragma unroll
                for (int c = 1; c < kMaxReachClasses; ++c)
                    if (c < cls.K && r >= first_row[c]) {
                        k = c, i = r - first_row[c], al = a_lo[c], bl = b_lo[c], nb = n_b[c], whole = cls.whole[c];
                        q2 = cls.q2[c];
                    }
                if (whole) {
                    in = true;
                    e = make_int2(i, -1 - k);
                } else {
                    const int da = i / nb + al, db = i % nb + bl;
                    const float fa = da == 0 ? 0.0f : (float)abs(da) - 0.5f;
                    const float fb = db == 0 ? 0.0f : (float)abs(db) - 0.5f;
                    const float rem = q2 - fa * fa - fb * fb;
                    in = rem >= 0.0f;
                    const float rz = fminf(sqrtf(in ? rem : 0.0f) + 0.5f, (float)G);
                    e = make_int2((int)((unsigned)da << 16 | ((unsigned)db & 0xFFFFu)), ((int)rz << 2) | k);
                }
            }
            const uint64_t m = __ballot(in);
            if (lane == 0) wrows[w] = __popcll(m);
            __syncthreads();
            int at = rows + __popcll(m & ((1ull << lane) - 1ull));
            for (int v = 0; v < kThreads / 64; ++v) {
                if (v < w) at += wrows[v];
                rows += wrows[v];
            }
            if (in) row_all[at] = e;
            __syncthreads();
        }
        // 2. their particles
        // a row's first particle and number of particles (32-bit places: at
        // most 2 classes of 1024^3 cells)
        auto look_up = [&](const int2 e, unsigned &at, unsigned &num) {
            at = num = 0;
            if (e.y < 0) {
                const unsigned *const st = start + (int64_t)(-1 - e.y) * ncell;
                const unsigned s0 = st[0], n = st[ncell] - s0;   // (n < 2^20: a stencil's rows at most)
                at = s0 + n * (unsigned)e.x / kSlices;
                num = live ? s0 + n * (unsigned)(e.x + 1) / kSlices - at : 0u;
                return;
            }
            const unsigned a = (unsigned)(ia + (e.x >> 16)), b = (unsigned)(ib + (int)(short)(e.x & 0xFFFF));
            if (live && a < (unsigned)G && b < (unsigned)G) {
                const int rz = e.y >> 2;
                const unsigned row = ((unsigned)(e.y & 3) * (unsigned)G + a) * (unsigned)G + b;
                const unsigned *const st = start + (row << log2g);
                at = st[max(ic0 - rz, 0)];
                num = st[min(ic0 + nz - 1 + rz, G - 1) + 1] - at;
            }
        };
        for (int r = sl; __any(r < rows); r += kAhead * kSlices) {
            unsigned cur[kAhead], left[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                cur[u] = left[u] = 0;
                if (r + u * kSlices < rows) look_up(row_all[r + u * kSlices], cur[u], left[u]);
            }
            for (;;) {
                unsigned more = 0;
#pragma unroll
                for (int u = 0; u < kAhead; ++u) more |= left[u];
                if (!__any(more != 0)) break;
                unsigned take[kAhead], sum = 0;
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    take[u] = min(left[u], (unsigned)kTake - sum);
                    sum += take[u];
                }
                int incl = (int)sum;
#pragma unroll
                for (int o = 1; o < kSlices; o <<= 1) {
                    const int v = __shfl_up(incl, o, kSlices);
                    if (sl >= o) incl += v;
                }
                unsigned *to = list + listed + incl - sum;
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    for (unsigned i = 0; i < take[u]; ++i) to[i] = cur[u] + i;
                    to += take[u];
                    cur[u] += take[u];
                    left[u] -= take[u];
                }
                listed += __shfl(incl, kSlices - 1, kSlices);
                if (__any(listed > kList - kSlices * kTake)) empty_list();
            }
        }
    }
    empty_list();
    if (MODE == kGatherCount) {
#pragma unroll
        for (int j = 0; j < kCellsZ; ++j) {
            unsigned lo = sl < 4 ? (cnt[j] & 0xFFu) << (8 * sl) : 0u, hi = sl >= 4 ? (cnt[j] & 0xFFu) << (8 * (sl - 4)) : 0u;
            unsigned total = cnt[j];
            if (cnt[j] > 255u) atomicOr(many, 1u);   // no room in a byte: nothing is recorded
#pragma unroll
            for (int o = 1; o < kSlices; o <<= 1) {
                lo |= (unsigned)__shfl_xor((int)lo, o, 64);
                hi |= (unsigned)__shfl_xor((int)hi, o, 64);
                total += (unsigned)__shfl_xor((int)total, o, 64);
            }
            if (live && sl == 0 && j < nz) {
                pslice[cell0 + j] = make_uint2(lo, hi);
                pcount[cell0 + j] = total;
            }
        }
    }
#pragma unroll
    for (int j = 0; j < kCellsZ; ++j) {
#pragma unroll
        for (int o = 1; o < kSlices; o <<= 1) {
            num[j] += __shfl_xor(num[j], o, 64);
            den[j] += __shfl_xor(den[j], o, 64);
        }
        // lane j of the group writes centre j
        if (live && sl == j && j < nz) {
            if (MODE == kFillPairs) pden[cell0 + j] = den[j];
            const double v = den[j] > 0.0 ? num[j] / den[j] : 0.0;
            const int64_t e = (int64_t)ia * sx + (int64_t)ib * sy + ic0 + j;
            val[e] = v;
            valf[e] = (float)v;
        }
    }
}

// Sum of n counts into a 64-bit total (the count scan is 32-bit).
__global__ void __launch_bounds__(kThreads) sum_counts(int64_t n, const unsigned *cnt, unsigned long long *total)
{
    __shared__ unsigned long long part[kThreads / 64];
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    unsigned long long v = i < n ? cnt[i] : 0ull;
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int w = 0; w < kThreads / 64; ++w) t += part[w];
        if (t) atomicAdd(total, t);
    }
}

// The grid from the recorded pairs: the same sums in the same order as
// shepard_gather (each slice's pairs in turn, then the slices' sums two by
// two), so the same values bit for bit, reading each cell's pairs instead of
// searching the stencil.
__global__ void __launch_bounds__(kThreads) refill_pairs(int G, const uint2 *__restrict__ pslice,
                                                         const unsigned *__restrict__ gstart,
                                                         const unsigned *__restrict__ pidx,
                                                         const double *__restrict__ pw,
                                                         const double *__restrict__ pden,
                                                         const double *__restrict__ ns, double *val, float *valf,
                                                         int sx, int sy)
{
    const int64_t lin = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (lin >= (int64_t)G * G * G) return;
    const int ia = (int)(lin / ((int64_t)G * G)), ib = (int)((lin / G) % G), ic = (int)(lin % G);
    const int64_t base = (int64_t)gstart[lin >> 6] + (lin & 63);
    const uint2 c = pslice[lin];
    const unsigned nq = pairs_before(c, kSlices);
    // one loop over all pairs; a slice that ends hands its sum to the pair, the
    // four, the eight that it belongs to
    double sum = 0.0, s1 = 0.0, s2 = 0.0, s4 = 0.0;
    int slice = 0;
    unsigned next = pairs_before(c, 1);
    auto end_slice = [&]() {
        if (slice & 1) {
            sum = s1 + sum;
            if (slice & 2) {
                sum = s2 + sum;
                if (slice & 4) sum = s4 + sum;
                else s4 = sum;
            } else {
                s2 = sum;
            }
        } else {
            s1 = sum;
        }
        ++slice;
        if (slice < kSlices) {
            sum = 0.0;
            next += ((slice < 4 ? c.x : c.y) >> (8 * (slice & 3))) & 0xFFu;
        }
    };
    // eight pairs' loads in flight (one at a time, two dependent loads a pair,
    // took 47 us per refill of 64^3 cells with ~32 pairs each; this 29)
    for (unsigned q0 = 0; q0 < nq; q0 += 8) {
        unsigned i[8];
        double wt[8], v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t at = base + (int64_t)(q0 + u < nq ? q0 + u : q0) * 64;
            i[u] = pidx[at];
            wt[u] = pw[at];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = ns[i[u]];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const unsigned q = q0 + (unsigned)u;
            if (q >= nq) break;
            while (q == next) end_slice();
            sum = fma(v[u], wt[u], sum);
        }
    }
    while (slice < kSlices) end_slice();
    const double den = pden[lin];
    const double v = den > 0.0 ? sum / den : 0.0;
    const int64_t e = (int64_t)ia * sx + (int64_t)ib * sy + ic;
    val[e] = v;
    valf[e] = (float)v;
}

// Size of each group of 64 cells in the interleaved pair arrays: 64 times
// its longest list.
__global__ void __launch_bounds__(kThreads) group_sizes(int64_t ncell, int64_t ngroups, const unsigned *pcount,
                                                        unsigned *gsize)
{
    const int64_t g = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (g >= ngroups) return;
    unsigned m = 0;
    for (int64_t c = g * 64; c < g * 64 + 64 && c < ncell; ++c) m = pcount[c] > m ? pcount[c] : m;
    gsize[g] = 64u * m;
}

__global__ void __launch_bounds__(kThreads) unpad(int G, int sx, int sy, const double *val, double *out)
{
    const int64_t lin = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (lin >= (int64_t)G * G * G) return;
    const int ia = (int)(lin / ((int64_t)G * G)), ib = (int)((lin / G) % G), ic = (int)(lin % G);
    out[lin] = val[(int64_t)ia * sx + (int64_t)ib * sy + ic];
}

}  // namespace

// Splits the non-empty reach bins into at most kmax classes of neighbouring
// bins, minimising an estimate of the gather work per cell centre: for each
// class, the particles it holds per cell times the cells its stencil scans
// (a ball of radius reach + half a cell), plus a fixed cost per row of cells.
// reach_cells is the largest reach in cells; it bounds the last class.
static ReachClasses choose_classes(const unsigned *hist, int G, int64_t ncell, double reach_cells, int kmax,
                                   int4 *top)
{
    constexpr double kRowCost = 3.0;   // one row's look-up, in particle tests
    std::vector<int> bin;
    std::vector<double> pre(1, 0.0);
    for (int u = 0; u < kBins; ++u)
        if (hist[u]) {
            bin.push_back(u);
            pre.push_back(pre.back() + hist[u]);
        }
    const int m = (int)bin.size();
    ReachClasses c;
    *top = make_int4(kBins, kBins, kBins, 0);
    if (m == 0) return c;   // no particle: one empty class
    auto radius = [&](int j) {   // reach in cells of a class ending at bin j
        return bin[j] == kBins - 1 ? reach_cells : std::min(0.25 * bin[j], reach_cells);
    };
    auto cost = [&](int i, int j) {
        const double r = radius(j) + 0.5, rows = M_PI * r * r;
        return (pre[j + 1] - pre[i]) / (double)ncell * (4.0 / 3.0 * M_PI * r * r * r + rows) + kRowCost * rows;
    };
    const double inf = 1e300;
    // best[k][j]: k classes over the first j bins; from[k][j]: first bin of the last class
    std::vector<std::vector<double>> best(kmax + 1, std::vector<double>(m + 1, inf));
    std::vector<std::vector<int>> from(kmax + 1, std::vector<int>(m + 1, 0));
    best[0][0] = 0.0;
    for (int k = 1; k <= kmax; ++k)
        for (int j = 1; j <= m; ++j)
            for (int i = k - 1; i < j; ++i)
                if (best[k - 1][i] < inf) {
                    const double v = best[k - 1][i] + cost(i, j - 1);
                    if (v < best[k][j]) {
                        best[k][j] = v;
                        from[k][j] = i;
                    }
                }
    int K = 1;
    for (int k = 2; k <= kmax && k <= m; ++k)
        if (best[k][m] < best[K][m]) K = k;
    int last[kMaxReachClasses];
    for (int k = K, j = m; k > 0; --k) {
        last[k - 1] = j - 1;
        j = from[k][j];
    }
    c.K = K;
    int t[3] = {kBins, kBins, kBins};
    for (int k = 0; k < K; ++k) {
        const double r = radius(last[k]);
        // a margin far above the rounding of the binning and of the float
        // stencil arithmetic; it only ever adds cells to the scan
        c.q2[k] = (float)(r * r * (1.0 + 1e-4) + 1e-4);
        c.R[k] = (int)std::min(floor(0.5 + sqrt((double)c.q2[k])), (double)(G - 1));   // no row is further
        // fewer particles than the stencil has rows inside the grid
        const double rows = std::min(M_PI * (r + 0.5) * (r + 0.5), (double)G * G);
        c.whole[k] = pre[last[k] + 1] - pre[k > 0 ? last[k - 1] + 1 : 0] <= rows;
        if (k < 3 && k < K - 1) t[k] = bin[last[k]];
    }
    *top = make_int4(t[0], t[1], t[2], 0);
    return c;
}

start_status bin_gas(Ctx *c, const start_box &box, int64_t n, const double *xyz, const double *h,
                     const double *nhi, int grid_log2, GasBins *b)
{
    hipStream_t s = c->stream;
    auto al = [](size_t v) { return (v + 255) & ~(size_t)255; };
    const int G = 1 << grid_log2;
    const int64_t ncell = (int64_t)G * G * G;
    *b = GasBins();
    b->box = box;
    b->n = n;
    b->G = G;
    b->delta = box.size / G;
    if (n == 0) return START_OK;
    const int64_t nk = n;
    b->bytes = al(radix_temp_bytes(nk)) + al(nk * sizeof(uint64_t)) + al(nk * sizeof(unsigned)) +
               al(nk * sizeof(double4)) + al(nk * sizeof(double2)) + al(nk * sizeof(double)) +
               al(kBins * sizeof(unsigned)) + 256;
    if (dmalloc(c, (void **)&b->mem, b->bytes) != hipSuccess) {
        b->mem = nullptr;
        return START_ENOMEM;
    }
    char *q = b->mem;
    auto take = [&](size_t v) { char *r = q; q += al(v); return r; };
    void *radix_tmp = take(radix_temp_bytes(nk));
    uint64_t *keys = (uint64_t *)take(nk * sizeof(uint64_t));
    b->idx = (unsigned *)take(nk * sizeof(unsigned));
    b->pos_h = (double4 *)take(nk * sizeof(double4));
    b->kern = (double2 *)take(nk * sizeof(double2));
    b->ns = (double *)take(nk * sizeof(double));
    unsigned *hist = (unsigned *)take(kBins * sizeof(unsigned));
    unsigned long long *hmax = (unsigned long long *)take(256);

    const double gs = (double)G / box.size;
    unsigned *bflags = c->d_flags + 1;   // build validation word (not the rate calls' one)
    hipMemsetAsync(bflags, 0, sizeof(unsigned), s);
    hipMemsetAsync(hist, 0, kBins * sizeof(unsigned), s);
    hipMemsetAsync(hmax, 0, sizeof(unsigned long long), s);
    grid_keys<<<blocks_for(n), kThreads, 0, s>>>(box, gs, G, n, xyz, h, nhi, keys, b->idx, bflags, hist, hmax);
    unsigned flags = 0;
    unsigned long long hbits = 0;
    unsigned hh[kBins];
    static_assert(kBins + 3 <= kReadbackWords, "readback words");
    if (c->rb) {
        grid_readback<<<1, kBins, 0, s>>>(bflags, hist, hmax, c->rb_dev);
    } else {
        hipMemcpyAsync(&flags, bflags, sizeof(unsigned), hipMemcpyDeviceToHost, s);
        hipMemcpyAsync(hh, hist, sizeof(hh), hipMemcpyDeviceToHost, s);
        hipMemcpyAsync(&hbits, hmax, sizeof(hbits), hipMemcpyDeviceToHost, s);
    }
    hipError_t e = hipStreamSynchronize(s);
    if (e == hipSuccess && c->rb) {
        const volatile unsigned *rb = c->rb;
        flags = rb[0];
        for (int k = 0; k < kBins; ++k) hh[k] = rb[1 + k];
        hbits = (unsigned long long)rb[1 + kBins] | ((unsigned long long)rb[2 + kBins] << 32);
    }
    if (e != hipSuccess || flags) {
        free_bins(c, b);
        if (e != hipSuccess) { c->err = hipGetErrorString(e); return START_EHIP; }
        if (flags & kFlagNonFinite) { c->err = "non-finite gas position, h or n_HI"; return START_ENONFINITE; }
        if (flags & kFlagOutOfBox) { c->err = "gas particle outside the box"; return START_EOUTOFBOX; }
        c->err = "gas h <= 0 or n_HI < 0";
        return START_EINVAL;
    }
    std::memcpy(&b->reach, &hbits, sizeof(double));
    int4 top;
    b->cls = choose_classes(hh, G, ncell, b->reach / b->delta, grid_log2 >= 10 ? 2 : kMaxReachClasses, &top);
    const int K = b->cls.K;
    // per (class, cell) starts, allocated once the number of classes is known
    const int64_t nstart = K * ncell + 1;
    b->bytes2 = al(nstart * sizeof(unsigned)) + al(scan_temp_bytes(nstart));
    if (dmalloc(c, (void **)&b->mem2, b->bytes2) != hipSuccess) {
        b->mem2 = nullptr;
        free_bins(c, b);
        c->err = "allocation failed";
        return START_ENOMEM;
    }
    b->start = (unsigned *)b->mem2;
    void *scan_tmp = b->mem2 + al(nstart * sizeof(unsigned));
    if (K > 1) class_keys<<<blocks_for(n), kThreads, 0, s>>>(n, h, gs, ncell, top, keys);
    const SortedPairs sp = radix_sort_pairs(keys, b->idx, n, 3 * grid_log2 + (K > 2 ? 2 : K - 1), radix_tmp, s);
    keys = sp.keys;   // (both pairs of arrays live as long as the bins)
    b->idx = sp.vals;
    hipMemsetAsync(b->start, 0, nstart * sizeof(unsigned), s);
    cell_counts<<<blocks_for(n), kThreads, 0, s>>>(keys, n, b->start);
    exclusive_scan_u32(b->start, nstart, scan_tmp, s);
    unsigned *inv = (unsigned *)keys;   // the keys are no longer needed
    invert_perm<<<blocks_for(n), kThreads, 0, s>>>(n, b->idx, inv);
    scatter_particles<<<blocks_for(n), kThreads, 0, s>>>(n, inv, xyz, h, nhi, b->pos_h, b->kern, b->ns);
    return START_OK;
}

void free_bins(Ctx *c, GasBins *b)
{
    dfree(c, b->mem, b->bytes);
    dfree(c, b->mem2, b->bytes2);
    dfree(c, b->mem3, b->bytes3);
    dfree(c, b->mem4, b->bytes4);
    b->mem = b->mem2 = b->mem3 = b->mem4 = nullptr;
    b->bytes = b->bytes2 = b->bytes3 = b->bytes4 = 0;
    b->pcount = b->pstart = b->pidx = nullptr;
    b->pslice = nullptr;
    b->counted = nullptr;
    b->pw = b->pden = nullptr;
}

namespace {

// Both copies of an empty grid set to 0 by a kernel (fill_grid may be
// captured into a HIP graph, where memset nodes are avoided).
__global__ void __launch_bounds__(256) zero_grid(int64_t span, double *val, float *valf)
{
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= span) return;
    val[k] = 0.0;
    valf[k] = 0.0f;
}

}  // namespace

// Blocks of a Shepard pass: eight lanes per group of kCellsZ centres.
static unsigned gather_blocks(int G)
{
    return blocks_for((int64_t)G * G * ((G + kCellsZ - 1) / kCellsZ) * kSlices);
}

void fill_grid(Ctx *c, const GasBins &b, const double *nhi, Grid *g)
{
    hipStream_t s = c->stream;
    if (b.n == 0) {
        zero_grid<<<(unsigned)((g->span + 255) / 256), 256, 0, s>>>(g->span, g->val, g->valf);
        return;
    }
    if (nhi) gather_values<<<blocks_for(b.n), kThreads, 0, s>>>(b.n, b.idx, nhi, b.ns);
    if (b.pidx) {
        const int64_t ncell = (int64_t)g->G * g->G * g->G;
        refill_pairs<<<blocks_for(ncell), kThreads, 0, s>>>(g->G, b.pslice, b.pstart, b.pidx, b.pw, b.pden, b.ns,
                                                            g->val, g->valf, g->sx, g->sy);
        return;
    }
    shepard_gather<kGather><<<gather_blocks(g->G), kThreads, 0, s>>>(
        b.box, b.delta, b.G, b.cls, b.start, b.pos_h, b.kern, b.ns, g->val, g->valf, g->sx, g->sy, nullptr, nullptr,
        nullptr, nullptr, nullptr, nullptr, nullptr);
}

// 20 bytes a cell for the counts and what the recorded pairs need per cell.
start_status count_pairs(Ctx *c, GasBins *b, Grid *g)
{
    hipStream_t s = c->stream;
    auto al = [](size_t v) { return (v + 255) & ~(size_t)255; };
    const int64_t ncell = (int64_t)b->G * b->G * b->G, ngroups = (ncell + 63) / 64;
    b->bytes3 = al(ncell * sizeof(uint2)) + al(ncell * sizeof(unsigned)) + al((ngroups + 1) * sizeof(unsigned)) +
                al(scan_temp_bytes(ngroups + 1)) + al(ncell * sizeof(double)) + 256;
    if (dmalloc(c, (void **)&b->mem3, b->bytes3) != hipSuccess) {
        b->mem3 = nullptr;
        b->bytes3 = 0;
        return START_ENOMEM;
    }
    char *q = b->mem3;
    auto take = [&](size_t v) { char *r = q; q += al(v); return r; };
    b->pslice = (uint2 *)take(ncell * sizeof(uint2));
    b->pcount = (unsigned *)take(ncell * sizeof(unsigned));
    b->pstart = (unsigned *)take((ngroups + 1) * sizeof(unsigned));
    b->pscan = take(scan_temp_bytes(ngroups + 1));
    b->pden = (double *)take(ncell * sizeof(double));
    b->counted = (unsigned long long *)take(256);   // [0] pairs with padding, [1] a slice has more than 255
    hipMemsetAsync(b->counted, 0, 2 * sizeof(unsigned long long), s);
    shepard_gather<kGatherCount><<<gather_blocks(b->G), kThreads, 0, s>>>(
        b->box, b->delta, b->G, b->cls, b->start, b->pos_h, b->kern, b->ns, g->val, g->valf, g->sx, g->sy, b->pslice,
        b->pcount, nullptr, nullptr, nullptr, nullptr, (unsigned *)(b->counted + 1));
    return START_OK;
}

start_status record_pairs(Ctx *c, GasBins *b, const double *nhi, Grid *g)
{
    hipStream_t s = c->stream;
    auto al = [](size_t v) { return (v + 255) & ~(size_t)255; };
    const int64_t ncell = (int64_t)b->G * b->G * b->G, ngroups = (ncell + 63) / 64;
    auto drop = [&]() {
        dfree(c, b->mem3, b->bytes3);
        b->mem3 = nullptr;
        b->bytes3 = 0;
        b->pcount = b->pstart = nullptr;
        b->pslice = nullptr;
        b->counted = nullptr;
        b->pden = nullptr;
    };
    // 1. the padded group sizes, their sum and their starts
    hipMemsetAsync(b->pstart + ngroups, 0, sizeof(unsigned), s);
    group_sizes<<<blocks_for(ngroups), kThreads, 0, s>>>(ncell, ngroups, b->pcount, b->pstart);
    sum_counts<<<blocks_for(ngroups), kThreads, 0, s>>>(ngroups, b->pstart, b->counted);
    unsigned long long words[2] = {0, 0};
    hipMemcpyAsync(words, b->counted, sizeof(words), hipMemcpyDeviceToHost, s);
    if (hipStreamSynchronize(s) != hipSuccess) {
        drop();
        return START_EHIP;
    }
    // the starts are 32-bit, the pairs (12 B each) must stay modest, and a
    // cell's slices count theirs in bytes.  (Wider counts gain nothing: a refill
    // waits for its longest cell, where the search has eight lanes for it.  20
    // iterations on 2^20 particles, 3000 of them in one cell: 21.1 ms with
    // recorded pairs, 17.9 without.)
    if (words[0] > kMaxPairs || words[1]) {
        drop();
        return START_ENOMEM;
    }
    exclusive_scan_u32(b->pstart, ngroups + 1, b->pscan, s);
    // 2. the pairs themselves (particle, weight), with the weight sums
    const size_t np = words[0] > 0 ? (size_t)words[0] : 1;
    b->bytes4 = al(np * sizeof(unsigned)) + al(np * sizeof(double));
    if (dmalloc(c, (void **)&b->mem4, b->bytes4) != hipSuccess) {
        b->mem4 = nullptr;
        b->bytes4 = 0;
        hipStreamSynchronize(s);   // the scan may still run
        drop();
        return START_ENOMEM;
    }
    b->pidx = (unsigned *)b->mem4;
    b->pw = (double *)(b->mem4 + al(np * sizeof(unsigned)));
    b->n_pairs = (int64_t)words[0];
    gather_values<<<blocks_for(b->n), kThreads, 0, s>>>(b->n, b->idx, nhi, b->ns);
    shepard_gather<kFillPairs><<<gather_blocks(b->G), kThreads, 0, s>>>(
        b->box, b->delta, b->G, b->cls, b->start, b->pos_h, b->kern, b->ns, g->val, g->valf, g->sx, g->sy, b->pslice,
        nullptr, b->pstart, b->pidx, b->pw, b->pden, nullptr);
    return START_OK;
}

start_status alloc_grid(Ctx *c, const start_box &box, int grid_log2, Grid *g)
{
    auto al = [](size_t v) { return (v + 255) & ~(size_t)255; };
    g->box = box;
    g->grid_log2 = grid_log2;
    const int G = 1 << grid_log2;
    g->G = G;
    const int pad = (G >= 64 && G <= 512) ? 16 : 0;
    g->sy = G + pad;
    g->sx = G * g->sy + pad;
    g->span = (int64_t)(G - 1) * g->sx + (int64_t)(G - 1) * g->sy + G;
    g->guard = G <= 512 ? 6 * ((int64_t)g->sx + g->sy + 1) : 0;
    const int64_t held = g->span + 2 * g->guard;
    size_t persist = al(held * sizeof(double)) + al(held * sizeof(float));
    char *pm = nullptr;
    if (dmalloc(c, (void **)&pm, persist) != hipSuccess) return START_ENOMEM;
    g->bytes = persist;
    g->mem = pm;
    g->val = (double *)pm + g->guard;
    g->valf = (float *)(pm + al(held * sizeof(double))) + g->guard;
    // guards and padding are never written again
    if (pad || g->guard) hipMemsetAsync(pm, 0, persist, c->stream);
    return START_OK;
}

start_status build_grid(Ctx *c, const start_box &box, int64_t n, const double *xyz, const double *h,
                        const double *nhi, int grid_log2, Grid *g)
{
    start_status st = alloc_grid(c, box, grid_log2, g);
    if (st) return st;
    GasBins b;
    st = bin_gas(c, box, n, xyz, h, nhi, grid_log2, &b);
    if (st) {
        hipStreamSynchronize(c->stream);   // the padding clear may still run
        dfree(c, g->mem, g->bytes);
        return st;
    }
    fill_grid(c, b, nullptr, g);   // the binning already gathered n_HI
    hipError_t e = hipStreamSynchronize(c->stream);
    free_bins(c, &b);
    if (e != hipSuccess) {
        c->err = hipGetErrorString(e);
        dfree(c, g->mem, g->bytes);
        return START_EHIP;
    }
    return START_OK;
}

void launch_grid_unpad(Ctx *c, const Grid &g, double *out)
{
    const int64_t n = (int64_t)g.G * g.G * g.G;
    unpad<<<blocks_for(n), kThreads, 0, c->stream>>>(g.G, g.sx, g.sy, g.val, out);
}

}  // namespace start
