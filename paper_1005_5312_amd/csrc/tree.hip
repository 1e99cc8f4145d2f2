// Source octree of START (Hasegawa & Umemura 2010, section 2.2.2) for gfx950.
//
// The paper splits cubic cells into 8 until every cell holds one source.  On
// the GPU the same cells come out of sorted Morton keys:
//   1. keys: each position is normalised to the box, quantised to 21 bits per
//      axis and bit-interleaved (x most significant), so a key's top 3n bits
//      name its level-n cell;
//   2. a stable radix sort orders the sources by (key, original index);
//   3. a binary radix tree over the sorted keys (one internal node per pair of
//      neighbours, built in parallel); a binary node whose common prefix
//      ends in a deeper octal digit than its parent's is a cell of the
//      octree that splits, and a run of identical keys is a level-21 bucket;
//   4. depth-first order is (first source, level): the cells that start at one
//      source have different levels, so one mask of levels per source counts
//      them, a scan of the counts gives every node its place without a sort,
//      and the index of the first node after its subtree (stackless walk);
//   5. the virtual source of each cell, eqs. (14)-(15), is summed bottom-up in
//      FP64, children in depth-first order: subtrees of at most 128 sources by
//      one wave each in LDS, the cells above them level by level.
// Below ~2^18 sources launches are what a build costs (~5 us each), so it has
// as few as it can and waits for the device once, at its end: the node count
// stays on the device until then and the kernels are launched for its bound 2n.
// A cell whose sources all sit in one sub-cube is represented by the deepest
// cube with the same sources: the opening test is monotone from parent to
// child, so testing that cube decides the whole chain.
#include <algorithm>

#include "internal.h"

namespace start {

namespace {

constexpr int kThreads = 256;

// Orders LDS traffic between the lanes of one wavefront.
__device__ inline void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline uint64_t spread3(uint64_t v)
{
    // 21 bits -> every third bit of 63
    v &= 0x1FFFFFull;
    v = (v | (v << 32)) & 0x1F00000000FFFFull;
    v = (v | (v << 16)) & 0x1F0000FF0000FFull;
    v = (v | (v << 8)) & 0x100F00F00F00F00Full;
    v = (v | (v << 4)) & 0x10C30C30C30C30C3ull;
    v = (v | (v << 2)) & 0x1249249249249249ull;
    return v;
}

__device__ inline unsigned compact3(uint64_t v)
{
    v &= 0x1249249249249249ull;
    v = (v ^ (v >> 2)) & 0x10C30C30C30C30C3ull;
    v = (v ^ (v >> 4)) & 0x100F00F00F00F00Full;
    v = (v ^ (v >> 8)) & 0x1F0000FF0000FFull;
    v = (v ^ (v >> 16)) & 0x1F00000000FFFFull;
    v = (v ^ (v >> 32)) & 0x1FFFFFull;
    return (unsigned)v;
}

__global__ void __launch_bounds__(kThreads) keys_kernel(start_box box, double inv, int64_t n, const double *xyz,
                                                        const double *lum, uint64_t *keys, unsigned *idx,
                                                        unsigned *flags)
{
    const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (j >= n) return;
    unsigned bad = 0;
    uint64_t key = 0;
    for (int k = 0; k < 3; ++k) {
        const double x = xyz[(int64_t)k * n + j];
        double u;
        if (!isfinite(x)) {
            bad |= kFlagNonFinite;
            u = 0.0;
        } else if (x < box.lo[k] || x > box.lo[k] + box.size) {
            bad |= kFlagOutOfBox;
            u = x < box.lo[k] ? 0.0 : 1.0;
        } else {
            u = (x - box.lo[k]) * inv;
            u = u > 1.0 ? 1.0 : u;
        }
        unsigned q = (unsigned)(u * 2097152.0);   // exact scaling by 2^21, truncation = floor
        q = q > 2097151u ? 2097151u : q;
        key |= spread3(q) << (2 - k);
    }
    if (lum) {
        const double L = lum[j];
        if (!isfinite(L)) bad |= kFlagNonFinite;
        else if (L < 0.0) bad |= kFlagNegative;
    }
    if (bad) atomicOr(flags, bad);
    keys[j] = key;
    idx[j] = (unsigned)j;
}

// Common prefix length of keys a and b as 63-bit strings followed by the
// 32-bit index (so identical keys still order); -1 outside [0, n).
__device__ inline int prefix_len(const uint64_t *k, int n, int a, int b)
{
    if (b < 0 || b >= n) return -1;
    const uint64_t x = k[a] ^ k[b];
    if (x) return __clzll((long long)x) - 1;
    return 63 + __clz((int)((unsigned)a ^ (unsigned)b));
}

__device__ inline int oct_level(int delta) { return (delta >= 63 ? 63 : delta) / 3; }

// Binary radix tree over n sorted keys (internal nodes 0..n-2, node 0 the
// root), and the items of the octree: canonical cells (internal binary nodes
// whose octal level is deeper than their parent's) and single-source leaves.
// The parent's common prefix is the longer of the two that the node's range
// shares with its neighbours.  levels[f] collects, one bit each, the levels of
// the cells whose first source is f, and bit 22 if f is a single source.
constexpr unsigned kLeafBit = 1u << 22;

__global__ void __launch_bounds__(kThreads) radix_tree_kernel(const uint64_t *k, int n, int2 *range, int *delta_out,
                                                              unsigned *levels)
{
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i < n) {
        const bool single = (i == 0 || k[i - 1] != k[i]) && (i == n - 1 || k[i + 1] != k[i]);
        if (single) atomicOr(&levels[i], kLeafBit);
    }
    if (i >= n - 1) return;
    const int d = (prefix_len(k, n, i, i + 1) - prefix_len(k, n, i, i - 1)) >= 0 ? 1 : -1;
    const int dmin = prefix_len(k, n, i, i - d);
    int lmax = 2;
    while (prefix_len(k, n, i, i + lmax * d) > dmin) lmax <<= 1;
    int l = 0;
    for (int t = lmax >> 1; t >= 1; t >>= 1)
        if (prefix_len(k, n, i, i + (l + t) * d) > dmin) l += t;
    const int j = i + l * d;
    const int dnode = prefix_len(k, n, i, j);
    const int lo = i < j ? i : j;
    const int hi = i < j ? j : i;
    const int dl = prefix_len(k, n, lo, lo - 1), dr = prefix_len(k, n, hi, hi + 1);
    const bool canon = i == 0 || oct_level(dnode) > oct_level(dl > dr ? dl : dr);
    range[i] = make_int2(lo, hi);
    delta_out[i] = canon ? dnode : -1;
    if (canon) atomicOr(&levels[lo], 1u << oct_level(dnode));
}

// The node count (also kept on the device, count) and the validation word,
// written by one lane into the context's pinned readback words.
__global__ void tree_readback(const unsigned *count, const unsigned *bflags, unsigned *rb)
{
    if (threadIdx.x != 0) return;
    rb[0] = *count;
    rb[1] = *bflags;
}

// Every node, by the binary node or single source it stands for, at its
// depth-first place: start[f] nodes have a first source before f, and the
// cells starting at f are in the order of their levels, a leaf last.
__global__ void __launch_bounds__(kThreads) fill_nodes(int n, const uint64_t *k, const unsigned *perm,
                                                       const int2 *range, const int *delta, const unsigned *levels,
                                                       const unsigned *start, const double4 *src, int4 *geo, int *skip,
                                                       int *first, int *count, int *ref, double4 *mom, double *lscale,
                                                       unsigned *n_nodes)
{
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i >= n) return;
    if (i == 0) {
        *n_nodes = start[n];
        if (n == 1) lscale[0] = src[0].w > 0.0 ? src[0].w : 1.0;
    }
    auto put = [&](unsigned p, int f, int c, int level, int kind, int r) {
        const uint64_t prefix = level > 0 ? (k[f] >> (3 * (kMaxLevel - level))) : 0ull;
        const int cx = (int)compact3(prefix >> 2), cy = (int)compact3(prefix >> 1), cz = (int)compact3(prefix);
        geo[p] = make_int4(cx, cy, cz, level | (kind << 8));
        skip[p] = (int)start[f + c];
        first[p] = f;
        count[p] = c;
        ref[p] = r;
    };
    if (i < n - 1 && delta[i] >= 0) {
        const int2 r = range[i];
        const int level = oct_level(delta[i]);
        const unsigned p = start[r.x] + __popc(levels[r.x] & ((1u << level) - 1u));
        put(p, r.x, r.y - r.x + 1, level, delta[i] >= 63 ? kKindBucket : kKindInternal, -1);
    }
    if (levels[i] & kLeafBit) {
        // a leaf's own cube is one level below the deepest cube it shares
        const int dl = i > 0 ? prefix_len(k, n, i, i - 1) : -1;
        const int dr = i < n - 1 ? prefix_len(k, n, i, i + 1) : -1;
        const int dm = dl > dr ? dl : dr;
        int level = dm < 0 ? 0 : oct_level(dm) + 1;
        level = level > kMaxLevel ? kMaxLevel : level;
        const unsigned p = start[i + 1] - 1u;
        put(p, i, 1, level, kKindLeaf, (int)perm[i]);
        mom[p] = src[i];
    }
}

// The sorted sources, and no cells yet at any of them (levels has n + 1 words).
__global__ void __launch_bounds__(kThreads) sorted_sources(int64_t n, const unsigned *perm, const double *xyz,
                                                           const double *lum, double4 *src, unsigned *levels)
{
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (k <= n) levels[k] = 0u;
    if (k >= n) return;
    const unsigned o = perm[k];
    src[k] = make_double4(xyz[o], xyz[n + o], xyz[2 * n + o], lum[o]);
}

// Bottom-up sums S = sum L_j r_j and L = sum L_j (eqs. 14-15), a cell's
// children in depth-first order, a bucket's members in sorted order, and the
// centre of luminosity S / L.
constexpr int kSmallTree = 128;              // sources of a subtree that one wave sums
constexpr int kSmallNodes = 2 * kSmallTree;  // its nodes at most (2 n - 1)

// Lengths of the lists that place_children makes, in words of one block of 256
// bytes: children (word 0), subtrees for moments_small, and the cells above them
// by level, on lines of their own.
constexpr int kRootWord = 16, kLevelWord = 32, kListWords = kLevelWord + kMaxLevel + 1;

__device__ inline double4 weighted(const double4 s) { return make_double4(s.w * s.x, s.w * s.y, s.w * s.z, s.w); }

__device__ inline double4 plus(const double4 a, const double4 b)
{
    return make_double4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

__device__ inline double4 centre_of(const double4 s)
{
    return s.w > 0.0 ? make_double4(s.x / s.w, s.y / s.w, s.z / s.w, s.w) : make_double4(0.0, 0.0, 0.0, 0.0);
}

__device__ inline double4 bucket_sum(const double4 *src, int f, int c)
{
    double4 s = make_double4(0.0, 0.0, 0.0, 0.0);
    for (int q = f; q < f + c; ++q) s = plus(s, weighted(src[q]));
    return s;
}

// The luminosity unit of the FP32 copies for a tree of eq. (14): the root's
// luminosity, which no node or source exceeds (1 for a dark tree).
__device__ inline double unit_of(double root) { return root > 0.0 ? root : 1.0; }

// One wave per subtree of at most kSmallTree sources (the largest ones): a
// lane holds up to four of its nodes, sums and links are in LDS, level by level
// from the deepest.  msum[root] is left for the cells above.
__global__ void __launch_bounds__(kThreads) moments_small(const int *lists, const int2 *roots, const int4 *geo,
                                                          const int *skip, const int *first, const int *count,
                                                          const double4 *src, double4 *msum, double4 *mom,
                                                          double *lscale)
{
    __shared__ double4 sum_all[kThreads / 64][kSmallNodes];
    __shared__ int end_all[kThreads / 64][kSmallNodes];
    const int w = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
    double4 *const sum = sum_all[w];
    int *const end = end_all[w];
    const int n_roots = lists[kRootWord];
    constexpr int kPer = kSmallNodes / 64;
    for (int64_t t = (int64_t)blockIdx.x * (kThreads / 64) + w; t < n_roots; t += (int64_t)gridDim.x * (kThreads / 64)) {
        const int2 r = roots[t];   // (node, first node after the subtree)
        const int m = r.y - r.x;
        int level[kPer];           // of a cell, -1 otherwise
        int top = -1;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int q = j * 64 + lane;
            level[j] = -1;
            if (q < m) {
                const int p = r.x + q;
                const int gw = geo[p].w, kind = gw >> 8, f = first[p];
                end[q] = skip[p] - r.x;
                if (kind == kKindLeaf) {
                    sum[q] = weighted(src[f]);
                } else if (kind == kKindBucket) {
                    sum[q] = bucket_sum(src, f, count[p]);
                    mom[p] = centre_of(sum[q]);
                } else {
                    level[j] = gw & 0xFF;
                    top = level[j] > top ? level[j] : top;
                }
            }
        }
        for (int o = 32; o > 0; o >>= 1) top = max(top, __shfl_xor(top, o, 64));
        const int root_level = geo[r.x].w & 0xFF;
        wave_fence();
        for (int lv = top; lv >= root_level; --lv) {
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                if (level[j] == lv) {
                    const int q = j * 64 + lane;
                    double4 s = make_double4(0.0, 0.0, 0.0, 0.0);
                    for (int c = q + 1; c < end[q]; c = end[c]) s = plus(s, sum[c]);
                    sum[q] = s;
                    mom[r.x + q] = centre_of(s);
                }
            wave_fence();
        }
        if (lane == 0) {
            msum[r.x] = sum[0];
            if (r.x == 0) lscale[0] = unit_of(sum[0].w);
        }
        wave_fence();
    }
}

// The cells of more than kSmallTree sources, level by level from the deepest
// (their children are among them, single sources, or subtrees that
// moments_small has summed).  The children are read through their places
// (place_children), all at once: the chain of links between them would be
// eight dependent loads.
struct TopCells {
    const int *lists, *cells;   // cap places a level
    int cap;
    const int2 *kids;
    const int *order;
    const int4 *geo;
    const int *first, *count;
    const double4 *src;
    double4 *msum, *mom;
    double *lscale;
};

__device__ inline void sum_cell(const TopCells &c, int p)
{
    double4 s = make_double4(0.0, 0.0, 0.0, 0.0);
    if ((c.geo[p].w >> 8) == kKindBucket) {
        s = bucket_sum(c.src, c.first[p], c.count[p]);
    } else {
        const int2 kd = c.kids[p];
        int kid[8];
        bool leaf[8];
        double4 v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) kid[j] = c.order[kd.x + (j < kd.y ? j : 0)];
#pragma unroll
        for (int j = 0; j < 8; ++j) leaf[j] = (c.geo[kid[j]].w >> 8) == kKindLeaf;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = leaf[j] ? c.src[c.first[kid[j]]] : c.msum[kid[j]];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (j < kd.y) s = plus(s, leaf[j] ? weighted(v[j]) : v[j]);
    }
    c.msum[p] = s;
    c.mom[p] = centre_of(s);
    if (p == 0) c.lscale[0] = unit_of(s.w);
}

// All levels by one block up to kOneBlock sources, where a launch per level
// would take longer (a build of 2^18 sources 320 us, 351 by levels); by levels
// beyond, where one CU is too few (2^19 sources 483 us by one block and 451 by
// levels, 2^20 741 and 603, 2^22 2949 and 1946).
constexpr int kTopThreads = 1024;
constexpr int64_t kOneBlock = (int64_t)3 << 17;
__global__ void __launch_bounds__(kTopThreads) moments_top(TopCells c)
{
    for (int lv = kMaxLevel; lv >= 0; --lv) {
        const int n = c.lists[kLevelWord + lv];
        if (n == 0) continue;
        for (int t = (int)threadIdx.x; t < n; t += kTopThreads) sum_cell(c, c.cells[(int64_t)lv * c.cap + t]);
        __threadfence_block();
        __syncthreads();
    }
}

__global__ void __launch_bounds__(kThreads) moments_level(TopCells c, int lv)
{
    const int n = c.lists[kLevelWord + lv];
    for (int t = (int)(blockIdx.x * kThreads + threadIdx.x); t < n; t += (int)gridDim.x * kThreads)
        sum_cell(c, c.cells[(int64_t)lv * c.cap + t]);
}

// ---- siblings side by side ----------------------------------------------
// Places of every cell's children (at most eight, in depth-first order), and
// the lists of the moment sums: the largest subtrees of at most kSmallTree
// sources (node, end) and the cells above them (cells: cap places a level).  A
// block takes one run of each for its nodes, so which run a cell gets depends
// on the schedule, its contents do not.  Blocks of 1024: every block adds to
// the same few words (2^22 sources, blocks of 256: 289 us, now 125).
constexpr int kPlaceThreads = 1024;
__global__ void __launch_bounds__(kPlaceThreads) place_children(const unsigned *n_nodes, const int4 *geo,
                                                                const int *skip, const int *count, int *lists,
                                                                int2 *kids, int *order, int2 *roots, int *cells,
                                                                int cap)
{
    constexpr int kWaves = kPlaceThreads / 64;
    __shared__ unsigned wtot[kWaves];
    __shared__ int run[2], level_n[kMaxLevel + 1], level_run[kMaxLevel + 1];
    const int64_t m = *n_nodes;
    const int64_t p = (int64_t)blockIdx.x * kPlaceThreads + threadIdx.x;
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    if (threadIdx.x <= kMaxLevel) level_n[threadIdx.x] = 0;
    int kid[8], kend[8];
    int k = 0;
    unsigned small = 0;                 // children that root a small subtree
    const int gw = p < m ? geo[p].w : kKindLeaf << 8;
    const int kind = gw >> 8, level = gw & 0xFF;
    const bool big = kind != kKindLeaf && count[p] > kSmallTree;
    if (kind == kKindInternal) {
        const int end = skip[p];
        int c = (int)p + 1;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            kid[j] = kend[j] = 0;
            if (c < end) {
                kid[j] = c;
                kend[j] = skip[c];
                if (big && count[c] > 1 && count[c] <= kSmallTree) small |= 1u << j;
                c = kend[j];
                ++k;
            }
        }
    }
    const bool small_root = p == 0 && kind != kKindLeaf && !big;
    // one scan of the two numbers, 16 bits each (at most 8 * 1024)
    const unsigned mine = (unsigned)k | (unsigned)(__popc(small) + (small_root ? 1 : 0)) << 16;
    unsigned incl = mine;
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    if (lane == 63) wtot[w] = incl;
    __syncthreads();
    int at_level = 0;
    if (big) at_level = atomicAdd(&level_n[level], 1);
    if (threadIdx.x < 2) {
        unsigned total = 0;
        for (int v = 0; v < kWaves; ++v) total += wtot[v];
        const int mine_total = (int)((total >> (16 * threadIdx.x)) & 0xFFFFu);
        run[threadIdx.x] = mine_total ? atomicAdd(&lists[threadIdx.x ? kRootWord : 0], mine_total) : 0;
    }
    __syncthreads();
    if (threadIdx.x <= kMaxLevel) {
        const int n = level_n[threadIdx.x];
        level_run[threadIdx.x] = n ? atomicAdd(&lists[kLevelWord + threadIdx.x], n) : 0;
    }
    __syncthreads();
    unsigned before = incl - mine;
    for (int v = 0; v < w; ++v) before += wtot[v];
    const int at = 1 + run[0] + (int)(before & 0xFFFFu);   // place 0 is the root's
    int rt = run[1] + (int)(before >> 16);
    if (p < m) kids[p] = make_int2(at, k);
    if (p == 0) order[0] = 0;
    if (big) cells[(int64_t)level * cap + level_run[level] + at_level] = (int)p;
    if (small_root) roots[rt++] = make_int2(0, skip[0]);
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (j < k) {
            order[at + j] = kid[j];
            if ((small >> j) & 1u) roots[rt++] = make_int2(kid[j], kend[j]);
        }
}

// ---- kernel-weighted node luminosities (section 2.2.2) -----------------
// Each node of >= 2 sources gets, at its centre of luminosity r (eq. 15),
//   form 1: L = sum_j L_j W_j / sum_j W_j (0 when every W_j = 0),
//   form 2: L = sum_j V_j L_j W_j,
// W_j = W(|r - r_j|, h_j), the cubic spline of section 2.1.  The members of
// a node are a contiguous run of the sorted sources, so a node is split
// into chunks of kLumChunk members, one wave per chunk (the root alone would
// otherwise hold one wave for the whole source list); the chunks' partial
// sums are added per node in chunk order, so the result does not depend on
// the schedule.
constexpr int kLumChunk = 1024;

__device__ inline double spline_w(double d, double h)
{
    const double q = d / h;
    const double a = fmax(2.0 - q, 0.0), b = fmax(1.0 - q, 0.0);
    return (0.25 * a * a * a - b * b * b) / (M_PI * h * h * h);
}

// (h, V) of every source in sorted order, with the arguments' validation.
__global__ void __launch_bounds__(kThreads) lum_gather(int64_t n, const unsigned *perm, const double *h,
                                                       const double *vol, int form, double2 *hv, unsigned *flags)
{
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (k >= n) return;
    const unsigned j = perm[k];
    const double hj = h[j];
    const double vj = form == 2 ? vol[j] : 0.0;
    unsigned bad = 0;
    if (!isfinite(hj) || !isfinite(vj))
        bad = kFlagNonFinite;
    else if (!(hj > 0.0) || vj < 0.0)
        bad = kFlagNegative;
    if (bad) atomicOr(flags, bad);
    hv[k] = make_double2(hj, vj);
}

// Chunks of every node (0 for single sources); element m is 0 so that the
// exclusive scan ends with the total.
__global__ void __launch_bounds__(kThreads) lum_chunks(int64_t m, const int4 *geo, const int *count,
                                                       unsigned *nchunk)
{
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p > m) return;
    unsigned c = 0;
    if (p < m && (geo[p].w >> 8) != kKindLeaf) c = (unsigned)((count[p] + kLumChunk - 1) / kLumChunk);
    nchunk[p] = c;
}

// (The largest nodes' chunks bound these two: 256 of the root of 2^18 sources.
// Their bounds are read once, and lum_finish has eight partial sums under way,
// added in the chunks' order: 34 -> 9 and 26 -> 11 us.)
__global__ void __launch_bounds__(kThreads) lum_owner(int64_t m, const unsigned *__restrict__ off,
                                                      unsigned *__restrict__ owner)
{
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p >= m) return;
    const unsigned a = off[p], b = off[p + 1];
    for (unsigned i = a; i < b; ++i) owner[i] = (unsigned)p;
}

__global__ void __launch_bounds__(kThreads) lum_partial(int64_t n_chunks, const unsigned *owner,
                                                        const unsigned *off, const int *first, const int *count,
                                                        const double4 *mom, const double4 *src, const double2 *hv,
                                                        int form, double2 *part)
{
    const int64_t t = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    const int lane = (int)(threadIdx.x & 63);
    if (t >= n_chunks) return;   // the whole wave
    const unsigned p = owner[t];
    const int64_t beg = (int64_t)first[p] + (t - (int64_t)off[p]) * kLumChunk;
    const int64_t end = min((int64_t)first[p] + count[p], beg + kLumChunk);
    const double4 r = mom[p];
    double num = 0.0, den = 0.0;
    for (int64_t k = beg + lane; k < end; k += 64) {
        const double4 s = src[k];
        const double2 q = hv[k];
        const double dx = r.x - s.x, dy = r.y - s.y, dz = r.z - s.z;
        const double w = spline_w(sqrt(dx * dx + dy * dy + dz * dz), q.x);
        num += (form == 2 ? q.y * s.w : s.w) * w;
        den += w;
    }
    for (int o = 32; o > 0; o >>= 1) {
        num += __shfl_xor(num, o, 64);
        den += __shfl_xor(den, o, 64);
    }
    if (lane == 0) part[t] = make_double2(num, den);
}

__global__ void __launch_bounds__(kThreads) lum_finish(int64_t m, const unsigned *__restrict__ off,
                                                       const double2 *__restrict__ part, int form,
                                                       double4 *__restrict__ mom)
{
    const int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (p >= m) return;
    const unsigned a = off[p], b = off[p + 1];
    if (a == b) return;   // a single source keeps its own luminosity
    double num = 0.0, den = 0.0;
    unsigned i = a;
    for (; i + 8 <= b; i += 8) {
        double2 v[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = part[i + q];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            num += v[q].x;
            den += v[q].y;
        }
    }
    for (; i < b; ++i) {
        num += part[i].x;
        den += part[i].y;
    }
    mom[p].w = form == 1 ? (den > 0.0 ? num / den : 0.0) : num;
}

// Largest luminosity of any node or source (as the bits of a non-negative
// double, which order like the values), one atomic per block.
__global__ void __launch_bounds__(kThreads) lum_max(int64_t m, const double4 *mom, int64_t n, const double4 *src,
                                                    unsigned long long *best)
{
    __shared__ unsigned long long red[kThreads / 64];
    unsigned long long v = 0;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < m + n; i += (int64_t)gridDim.x * kThreads) {
        const double L = i < m ? mom[i].w : src[i - m].w;
        const unsigned long long b = (unsigned long long)__double_as_longlong(L);
        v = b > v ? b : v;
    }
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long u = __shfl_xor(v, o, 64);
        v = u > v ? u : v;
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kThreads / 64; ++w) v = red[w] > v ? red[w] : v;
        if (v) atomicMax(best, v);
    }
}

__global__ void lum_scale(const unsigned long long *best, double *lscale)
{
    if (threadIdx.x == 0) lscale[0] = *best ? __longlong_as_double((long long)*best) : 1.0;
}

// New luminosities of the same sources, in sorted order (for a refit inside
// the equilibrium loop, whose emission they are), also in their leaves; a
// negative or non-finite value raises the equilibrium-input flag of the sticky
// word.
__global__ void __launch_bounds__(kThreads) set_lum(int64_t n, int64_t m, const unsigned *perm, const double *lum,
                                                    const int *ref, double4 *src, double4 *mom, double *lscale,
                                                    unsigned *flags)
{
    const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (k < n) {
        const double L = lum[perm[k]];
        if (!(L >= 0.0) || !isfinite(L)) atomicOr(flags, kFlagEqInput);
        src[k].w = L;
    }
    if (k < m && ref[k] >= 0) {
        const double L = lum[ref[k]];
        mom[k].w = L;
        if (n == 1) lscale[0] = unit_of(L);
    }
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kThreads - 1) / kThreads); }

}  // namespace

// ---- moment sums of a built tree ------------------------------------------
namespace {

// Work arrays of the moment sums of a tree of n sources (at most m nodes):
// sums, the lists' lengths, and the lists (a small subtree has 2 sources or
// more; at each of at most 22 levels there are at most n / kSmallTree cells
// above them).
struct Moments {
    double4 *msum;
    int *lists;
    int2 *roots;
    int *cells;
    int2 *kids;      // places of each node's children, and the nodes at them
    int *order;
};

int64_t top_cells_bound(int64_t n) { return n / kSmallTree + 1; }   // of one level

size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

size_t list_bytes(int64_t n, int64_t m)
{
    return 256 + al256((size_t)(n / 2 + 1) * sizeof(int2)) + al256((size_t)(kMaxLevel + 1) * top_cells_bound(n) * sizeof(int)) +
           al256((size_t)m * sizeof(int2)) + al256((size_t)m * sizeof(int));
}

// Temporaries of a build beside the tree's own arrays.
size_t build_bytes(int64_t n)
{
    return al256(radix_temp_bytes(n)) + al256(n * sizeof(int2)) + al256(n * sizeof(int)) +
           2 * al256((n + 1) * sizeof(unsigned)) + al256(scan_temp_bytes(n + 1)) +
           al256(list_bytes(n, 2 * n));
}

Moments carve_moments(void *lists, double4 *msum, int64_t n, int64_t m)
{
    char *q = (char *)lists;
    auto take = [&](size_t b) { char *r = q; q += al256(b); return r; };
    Moments w;
    w.msum = msum;
    w.lists = (int *)take(256);
    w.roots = (int2 *)take((size_t)(n / 2 + 1) * sizeof(int2));
    w.cells = (int *)take((size_t)(kMaxLevel + 1) * top_cells_bound(n) * sizeof(int));
    w.kids = (int2 *)take((size_t)m * sizeof(int2));
    w.order = (int *)take((size_t)m * sizeof(int));
    return w;
}

void sum_moments(Tree *t, const Moments &w, hipStream_t s)
{
    const int64_t n = t->n_src;
    if (n < 2) return;   // a single source is its own moment
    // one wave per subtree: ~n / 60 of them on random positions; more waves
    // than that walk the list in strides
    const int64_t waves = n / 32 + 1;
    const unsigned nb = (unsigned)std::min<int64_t>((waves + kThreads / 64 - 1) / (kThreads / 64), 65536);
    moments_small<<<nb, kThreads, 0, s>>>(w.lists, w.roots, t->geo, t->skip, t->first, t->count, t->src, w.msum,
                                          t->mom, t->lscale);
    if (n <= kSmallTree) return;
    const TopCells c{w.lists, w.cells, (int)top_cells_bound(n), w.kids, w.order, t->geo,
                     t->first, t->count, t->src, w.msum, t->mom, t->lscale};
    if (n <= kOneBlock) {
        moments_top<<<1, kTopThreads, 0, s>>>(c);
        return;
    }
    const unsigned lb = std::min(blocks_for(c.cap), 1024u);
    for (int lv = kMaxLevel; lv >= 0; --lv) moments_level<<<lb, kThreads, 0, s>>>(c, lv);
}

// m: the number of nodes, or a bound
void list_children(const Tree *t, const Moments &w, int64_t m, hipStream_t s)
{
    hipMemsetAsync(w.lists, 0, kListWords * sizeof(int), s);
    place_children<<<(unsigned)((m + kPlaceThreads - 1) / kPlaceThreads), kPlaceThreads, 0, s>>>(
        t->d_nodes, t->geo, t->skip, t->count, w.lists, w.kids, w.order, w.roots, w.cells,
        (int)top_cells_bound(t->n_src));
}

}  // namespace

// Work arrays of a refit: the moment sums and their lists (made once).
size_t refit_bytes(const Tree *t)
{
    return al256((size_t)t->n_nodes * sizeof(double4)) + list_bytes(t->n_src, t->n_nodes);
}

void refit_prepare(Ctx *c, const Tree *t, void *work)
{
    const int64_t m = t->n_nodes;
    if (m == 0) return;
    const Moments w = carve_moments((char *)work + al256((size_t)m * sizeof(double4)), (double4 *)work, t->n_src, m);
    list_children(t, w, m, c->stream);
}

// The same tree for new luminosities of the same sources: keys, order and
// nodes depend on the positions only, so only the sorted luminosities, the
// moments of eqs. (14)-(15) (with the build's own kernels, so the result is
// the rebuilt tree bit for bit) and the FP32 unit are redone.  Asynchronous;
// bad luminosities are reported by the next start_synchronize (as an
// equilibrium input).  `work` holds refit_bytes(t) after refit_prepare.
void refit_tree(Ctx *c, Tree *t, const double *lum, void *work)
{
    const int64_t m = t->n_nodes, n = t->n_src;
    if (n == 0) return;
    hipStream_t s = c->stream;
    const Moments w = carve_moments((char *)work + al256((size_t)m * sizeof(double4)), (double4 *)work, n, m);
    set_lum<<<blocks_for(std::max(m, n)), kThreads, 0, s>>>(n, m, t->perm, lum, t->ref, t->src, t->mom, t->lscale,
                                                            c->d_flags);
    sum_moments(t, w, s);
}

start_status tree_kernel_luminosity(Ctx *c, Tree *t, const double *h, const double *vol, int form)
{
    const int64_t m = t->n_nodes, n = t->n_src;
    if (n == 0) return START_OK;
    hipStream_t s = c->stream;
    auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t b_hv = al(n * sizeof(double2)), b_off = al((m + 1) * sizeof(unsigned));
    const size_t bytes1 = b_hv + b_off + al(scan_temp_bytes(m + 1)) + 256;
    char *t1 = nullptr;
    if (dmalloc(c, (void **)&t1, bytes1) != hipSuccess) return START_ENOMEM;
    double2 *hv = (double2 *)t1;
    unsigned *off = (unsigned *)(t1 + b_hv);
    void *scan_tmp = t1 + b_hv + b_off;
    unsigned long long *best = (unsigned long long *)(t1 + bytes1 - 256);
    unsigned *bflags = c->d_flags + 1;   // build validation word
    hipMemsetAsync(bflags, 0, sizeof(unsigned), s);
    hipMemsetAsync(best, 0, sizeof(*best), s);
    lum_gather<<<blocks_for(n), kThreads, 0, s>>>(n, t->perm, h, vol, form, hv, bflags);
    lum_chunks<<<blocks_for(m + 1), kThreads, 0, s>>>(m, t->geo, t->count, off);
    exclusive_scan_u32(off, m + 1, scan_tmp, s);
    unsigned flags = 0, n_chunks = 0;
    hipMemcpyAsync(&flags, bflags, sizeof(unsigned), hipMemcpyDeviceToHost, s);
    hipMemcpyAsync(&n_chunks, off + m, sizeof(unsigned), hipMemcpyDeviceToHost, s);
    hipError_t e = hipStreamSynchronize(s);
    if (e != hipSuccess || flags) {
        dfree(c, t1, bytes1);
        if (e != hipSuccess) {
            c->err = hipGetErrorString(e);
            return START_EHIP;
        }
        if (flags & kFlagNonFinite) {
            c->err = "non-finite smoothing length or volume";
            return START_ENONFINITE;
        }
        c->err = "smoothing length <= 0 or negative volume";
        return START_EINVAL;
    }
    char *t2 = nullptr;
    const size_t b_part = al((size_t)n_chunks * sizeof(double2));
    const size_t bytes2 = b_part + al((size_t)n_chunks * sizeof(unsigned));
    if (n_chunks > 0 && dmalloc(c, (void **)&t2, bytes2) != hipSuccess) {
        dfree(c, t1, bytes1);
        return START_ENOMEM;
    }
    if (n_chunks > 0) {
        double2 *part = (double2 *)t2;
        unsigned *owner = (unsigned *)(t2 + b_part);
        lum_owner<<<blocks_for(m), kThreads, 0, s>>>(m, off, owner);
        const unsigned waves_per_block = kThreads / 64;
        lum_partial<<<(unsigned)((n_chunks + waves_per_block - 1) / waves_per_block), kThreads, 0, s>>>(
            n_chunks, owner, off, t->first, t->count, t->mom, t->src, hv, form, part);
        lum_finish<<<blocks_for(m), kThreads, 0, s>>>(m, off, part, form, t->mom);
    }
    const int64_t items = m + n;
    const unsigned mb = (unsigned)std::min<int64_t>((items + kThreads - 1) / kThreads, 1024);
    lum_max<<<mb, kThreads, 0, s>>>(m, t->mom, n, t->src, best);
    lum_scale<<<1, 64, 0, s>>>(best, t->lscale);
    e = hipStreamSynchronize(s);
    if (t2) dfree(c, t2, bytes2);
    dfree(c, t1, bytes1);
    if (e != hipSuccess) {
        c->err = hipGetErrorString(e);
        return START_EHIP;
    }
    return START_OK;
}

void launch_keys(const start_box &box, int64_t n, const double *xyz, const double *lum, uint64_t *keys,
                 unsigned *idx, unsigned *flags, hipStream_t s)
{
    if (n <= 0) return;
    const double inv = 1.0 / box.size;
    keys_kernel<<<blocks_for(n), kThreads, 0, s>>>(box, inv, n, xyz, lum, keys, idx, flags);
}

// Builds the octree with its FP32 copies; all allocations are owned by the
// tree.  Synchronises once, at the end (to learn the node count and the
// validation flags).
start_status build_tree(Ctx *c, const start_box &box, int64_t n, const double *xyz, const double *lum,
                        Tree *t)
{
    hipStream_t s = c->stream;
    t->box = box;
    t->n_src = n;
    t->ctx = c;
    if (n == 0) return START_OK;
    const int ni = (int)n;
    const int64_t max_items = 2 * n;
    // persistent arrays
    const size_t persist = al256(n * sizeof(uint64_t)) + al256(n * sizeof(unsigned)) + al256(n * sizeof(double4)) +
                           al256(n * sizeof(uint4)) + al256(max_items * sizeof(int4)) +
                           4 * al256(max_items * sizeof(int)) + al256(max_items * sizeof(double4)) +
                           al256(max_items * sizeof(uint4)) + 2 * al256(sizeof(double)) +
                           al256(max_items * sizeof(Sibling));
    char *pm = nullptr;
    if (dmalloc(c, (void **)&pm, persist) != hipSuccess) return START_ENOMEM;
    t->bytes = persist;
    char *q = pm;
    auto take = [&](size_t b) { char *r = q; q += al256(b); return r; };
    t->keys = (uint64_t *)take(n * sizeof(uint64_t));
    t->perm = (unsigned *)take(n * sizeof(unsigned));
    t->src = (double4 *)take(n * sizeof(double4));
    t->srcq = (uint4 *)take(n * sizeof(uint4));
    t->geo = (int4 *)take(max_items * sizeof(int4));
    t->skip = (int *)take(max_items * sizeof(int));
    t->first = (int *)take(max_items * sizeof(int));
    t->count = (int *)take(max_items * sizeof(int));
    t->ref = (int *)take(max_items * sizeof(int));
    t->mom = (double4 *)take(max_items * sizeof(double4));
    t->momq = (uint4 *)take(max_items * sizeof(uint4));
    t->lscale = (double *)take(sizeof(double));
    t->d_nodes = (unsigned *)take(sizeof(double));
    t->sib = (Sibling *)take(max_items * sizeof(Sibling));

    // temporaries
    const size_t tmp_bytes = build_bytes(n);
    char *tm = nullptr;
    if (dmalloc(c, (void **)&tm, tmp_bytes) != hipSuccess) {
        dfree(c, pm, persist);
        return START_ENOMEM;
    }
    q = tm;
    void *radix_tmp = take(radix_temp_bytes(n));
    int2 *range = (int2 *)take(n * sizeof(int2));
    int *delta = (int *)take(n * sizeof(int));
    unsigned *levels = (unsigned *)take((n + 1) * sizeof(unsigned));
    unsigned *start = (unsigned *)take((n + 1) * sizeof(unsigned));
    void *scan_tmp = take(scan_temp_bytes(n + 1));
    // the sums use the siblings' records, which are written after them
    const Moments w = carve_moments(take(list_bytes(n, max_items)), (double4 *)t->sib, n, max_items);

    unsigned *bflags = c->d_flags + 1;   // build validation word (not the rate calls' one)
    hipMemsetAsync(bflags, 0, sizeof(unsigned), s);
    launch_keys(box, n, xyz, lum, t->keys, t->perm, bflags, s);
    radix_sort_pairs(t->keys, t->perm, n, 63, radix_tmp, s);   // eight passes: the result ends in place
    sorted_sources<<<blocks_for(n + 1), kThreads, 0, s>>>(n, t->perm, xyz, lum, t->src, levels);
    radix_tree_kernel<<<blocks_for(n), kThreads, 0, s>>>(t->keys, ni, range, delta, levels);
    exclusive_scan_bits(levels, start, n + 1, scan_tmp, s);   // start[i] = nodes with first < i
    fill_nodes<<<blocks_for(n), kThreads, 0, s>>>(ni, t->keys, t->perm, range, delta, levels, start, t->src, t->geo,
                                                  t->skip, t->first, t->count, t->ref, t->mom, t->lscale, t->d_nodes);
    list_children(t, w, max_items, s);
    sum_moments(t, w, s);
    make_siblings(t, max_items, w.order, w.kids, s);
    unsigned h[2] = {0, 0};
    if (c->rb) {
        tree_readback<<<1, 64, 0, s>>>(t->d_nodes, bflags, c->rb_dev);
    } else {
        hipMemcpyAsync(&h[0], t->d_nodes, sizeof(unsigned), hipMemcpyDeviceToHost, s);
        hipMemcpyAsync(&h[1], bflags, sizeof(unsigned), hipMemcpyDeviceToHost, s);
    }
    hipError_t e = hipStreamSynchronize(s);
    if (e == hipSuccess && c->rb) {
        const volatile unsigned *rb = c->rb;
        h[0] = rb[0];
        h[1] = rb[1];
    }
    dfree(c, tm, tmp_bytes);
    if (e != hipSuccess) {
        c->err = hipGetErrorString(e);
        dfree(c, pm, persist);
        return START_EHIP;
    }
    const unsigned flags = h[1];
    if (flags) {
        dfree(c, pm, persist);
        if (flags & kFlagNonFinite) { c->err = "non-finite source position or luminosity"; return START_ENONFINITE; }
        if (flags & kFlagOutOfBox) { c->err = "source outside the box"; return START_EOUTOFBOX; }
        c->err = "negative source luminosity";
        return START_EINVAL;
    }
    t->n_nodes = h[0];
    return START_OK;
}

}  // namespace start
