// Device-wide exclusive scan and stable LSD radix sort for gfx950 (wave64).
//
// The radix sort orders the Morton keys of sources and targets and the
// particles of the gas grid.  Each pass sorts on one 8-bit digit of tiles of
// 4096 items (one block of 16 waves):
//   1. per-tile digit histogram (LDS atomics), one row of 256 counts a tile;
//   2. stable scatter: each block sums the rows itself (its own start of
//      every digit), ranks its items (ranks inside a wave come from one ballot
//      per digit bit, waves are ordered through LDS counters), stages the tile
//      in LDS in digit order and writes it out run by run.
// So a pass is two launches; beyond kFusedTiles tiles the rows are scanned in
// between (two more).  Up to 8192 items one block sorts all digits in LDS, in
// one launch.
//
// What bounds it: launches and latency below ~2^18 items (a pass of two
// launches takes 12 us at 16 thousand items and 14 at 2^18), memory above.  The tile of 4096
// with 4 items a thread keeps a block's serial part short (4 rounds of
// ranking, no block barrier between them; 2048 items in 8 rounds with three
// barriers each took 10.7 us at 4096 items) and makes 256 tiles of 2^20 items,
// one for each CU.
#include "internal.h"

namespace start {

namespace {

constexpr int kScanThreads = 1024;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

constexpr int kSortThreads = 1024;
constexpr int kSortWaves = kSortThreads / 64;
constexpr int kSortItems = 4;
constexpr int kSortTile = kSortThreads * kSortItems;
constexpr int kSmallItems = 8;                               // one-block sorts
constexpr int64_t kSmallSort = (int64_t)kSortThreads * kSmallItems;
// Rows a scatter block sums by itself: 512 rows of 1 KiB take it ~4 us, as
// much as the two launches of a scan; more are scanned.
constexpr int64_t kFusedTiles = 512;
constexpr int kChunk = 64;                                   // rows per block of the scan

// Exclusive scan of v over the block's 1024 threads; wsum: 16 words of LDS.
__device__ inline unsigned block_exclusive_scan(unsigned v, unsigned *wsum, unsigned *total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    unsigned incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned u = __shfl_up(incl, o, 64);
        if (lane >= o) incl += u;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    unsigned add = 0, all = 0;
    for (int k = 0; k < kScanThreads / 64; ++k) {
        add += k < w ? wsum[k] : 0u;
        all += wsum[k];
    }
    *total = all;
    return incl - v + add;
}

// Tiles of 8192 words (one launch scans a whole array of that size); BITS:
// the numbers of bits set in `in`.  The arrays are 16-byte aligned.
template <bool BITS>
__global__ void __launch_bounds__(kScanThreads) scan_tiles(const unsigned *in, unsigned *out, int64_t n,
                                                           unsigned *sums)
{
    __shared__ unsigned wsum[kScanThreads / 64];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    unsigned v[kScanItems];
    unsigned s = 0;
    const bool whole = base + kScanItems <= n;   // two 16-byte accesses each way
    if (whole) {
        const uint4 a = *(const uint4 *)(in + base), b = *(const uint4 *)(in + base + 4);
        v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
    } else {
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) v[k] = base + k < n ? in[base + k] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        if (BITS) v[k] = __popc(v[k]);
        s += v[k];
    }
    unsigned total;
    unsigned run = block_exclusive_scan(s, wsum, &total);
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const unsigned c = v[k];
        v[k] = run;
        run += c;
    }
    if (whole) {
        *(uint4 *)(out + base) = make_uint4(v[0], v[1], v[2], v[3]);
        *(uint4 *)(out + base + 4) = make_uint4(v[4], v[5], v[6], v[7]);
    } else {
#pragma unroll
        for (int k = 0; k < kScanItems; ++k)
            if (base + k < n) out[base + k] = v[k];
    }
    if (threadIdx.x == 0 && sums) sums[blockIdx.x] = total;
}

__global__ void __launch_bounds__(kScanThreads) scan_add(unsigned *data, int64_t n, const unsigned *sums)
{
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    const unsigned add = sums[blockIdx.x];
    if (base + kScanItems <= n) {
        uint4 *const p = (uint4 *)(data + base);
        const uint4 a = p[0], b = p[1];
        p[0] = make_uint4(a.x + add, a.y + add, a.z + add, a.w + add);
        p[1] = make_uint4(b.x + add, b.y + add, b.z + add, b.w + add);
        return;
    }
    for (int k = 0; k < kScanItems; ++k)
        if (base + k < n) data[base + k] += add;
}

// LDS writes of a wave's lanes made visible to the wave's other lanes
__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Exclusive scan of v over threads 0..255 (the other threads pass along);
// wsum: 4 words of LDS.
__device__ inline unsigned scan256(unsigned v, unsigned *wsum)
{
    const int t = threadIdx.x, lane = t & 63;
    unsigned incl = v;
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned u = __shfl_up(incl, o, 64);
        if (lane >= o) incl += u;
    }
    if (t < 256 && lane == 63) wsum[t >> 6] = incl;
    __syncthreads();
    unsigned add = 0;
    for (int w = 0; w < 4; ++w)
        if (w < (t >> 6)) add += wsum[w];
    __syncthreads();
    return incl - v + add;
}

// Places of a block's items in the order of one digit, stable: item r of a
// thread is item (wave * ITEMS + r) * 64 + lane of the tile, items from `n`
// on do not count.  On return cnt[w][d] holds the first place of wave w's
// items of digit d, loc[d] the first place of digit d.
template <int ITEMS>
__device__ inline void rank_tile(const uint64_t (&key)[ITEMS], int n, int shift, int nbits,
                                 unsigned (*cnt)[256], unsigned *loc, unsigned *wsum, unsigned (&at)[ITEMS])
{
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    for (int k = t; k < kSortWaves * 256; k += kSortThreads) (&cnt[0][0])[k] = 0;
    __syncthreads();
    const unsigned dmask = (1u << nbits) - 1u;
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const bool valid = (w * ITEMS + r) * 64 + lane < n;
        const unsigned d = (unsigned)(key[r] >> shift) & dmask;
        uint64_t match = __ballot(valid);
        for (int b = 0; b < nbits; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            match &= bit ? bb : ~bb;
        }
        const unsigned rank = (unsigned)__popcll(match & below);
        const unsigned first = cnt[w][d];   // of this wave's earlier rounds
        wave_sync();
        if (valid && rank == 0) cnt[w][d] = first + (unsigned)__popcll(match);
        wave_sync();
        at[r] = first + rank;
    }
    __syncthreads();
    unsigned total = 0;
    if (t < 256)
        for (int k = 0; k < kSortWaves; ++k) {
            const unsigned c = cnt[k][t];
            cnt[k][t] = total;
            total += c;
        }
    const unsigned start = scan256(total, wsum);
    if (t < 256) {
        loc[t] = start;
        for (int k = 0; k < kSortWaves; ++k) cnt[k][t] += start;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) at[r] += cnt[w][(unsigned)(key[r] >> shift) & dmask];
}

__global__ void __launch_bounds__(kSortThreads) radix_hist(const uint64_t *__restrict__ keys, int64_t n, int shift,
                                                           unsigned dmask, unsigned *__restrict__ counts)
{
    __shared__ unsigned hist[256];
    const int t = threadIdx.x;
    if (t < 256) hist[t] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kSortTile;
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int64_t i = base + r * kSortThreads + t;
        if (i < n) atomicAdd(&hist[(unsigned)(keys[i] >> shift) & dmask], 1u);
    }
    __syncthreads();
    if (t < 256) counts[(int64_t)blockIdx.x * 256 + t] = hist[t];
}

// Many tiles: the rows of each chunk of kChunk tiles become exclusive sums
// within the chunk, tot[chunk] its totals ...
__global__ void __launch_bounds__(256) radix_chunks(int64_t ntiles, unsigned *__restrict__ counts,
                                                    unsigned *__restrict__ tot)
{
    const int t = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * kChunk;
    unsigned run = 0;
#pragma unroll 8
    for (int r = 0; r < kChunk; ++r) {
        const int64_t row = r0 + r;
        if (row >= ntiles) break;
        const unsigned c = counts[row * 256 + t];
        counts[row * 256 + t] = run;
        run += c;
    }
    tot[(int64_t)blockIdx.x * 256 + t] = run;
}

// ... and the chunks' totals the global starts of their digits (one block;
// thread group g of 256 sums a contiguous part of the chunks).
__global__ void __launch_bounds__(kSortThreads) radix_chunk_starts(int64_t nchunks, unsigned *__restrict__ tot)
{
    __shared__ unsigned part[kSortThreads / 256][256];
    __shared__ unsigned wsum[4];
    const int t = threadIdx.x, d = t & 255, g = t >> 8;
    constexpr int kGroups = kSortThreads / 256;
    const int64_t per = (nchunks + kGroups - 1) / kGroups;
    const int64_t c0 = g * per < nchunks ? g * per : nchunks;
    const int64_t c1 = c0 + per < nchunks ? c0 + per : nchunks;
    unsigned s = 0;
    for (int64_t c = c0; c < c1; ++c) s += tot[c * 256 + d];
    part[g][d] = s;
    __syncthreads();
    unsigned total = 0;
    for (int k = 0; k < kGroups; ++k) total += part[k][d];
    const unsigned start = scan256(total, wsum);
    __shared__ unsigned first[256];
    if (t < 256) first[t] = start;
    __syncthreads();
    unsigned run = first[d];
    for (int k = 0; k < g; ++k) run += part[k][d];
    for (int64_t c = c0; c < c1; ++c) {
        const unsigned v = tot[c * 256 + d];
        tot[c * 256 + d] = run;
        run += v;
    }
}

// tot null: `counts` holds the tiles' counts and the block sums them;
// otherwise the exclusive sums within the chunk, with the chunks' starts in tot.
__global__ void __launch_bounds__(kSortThreads) radix_scatter(const uint64_t *__restrict__ keys_in,
                                                              const unsigned *__restrict__ vals_in,
                                                              uint64_t *__restrict__ keys_out,
                                                              unsigned *__restrict__ vals_out, int64_t n, int shift,
                                                              int nbits, const unsigned *__restrict__ counts,
                                                              const unsigned *__restrict__ tot, int ntiles)
{
    __shared__ unsigned base[256];      // global start of each digit's run of this tile
    __shared__ unsigned loc[256];       // start of each digit inside the tile
    __shared__ unsigned cnt[kSortWaves][256];
    __shared__ unsigned wsum[4];
    __shared__ uint64_t skey[kSortTile];
    __shared__ unsigned sval[kSortTile];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t tile = blockIdx.x;
    const int64_t tile0 = tile * kSortTile;
    const int here = n - tile0 < kSortTile ? (int)(n - tile0) : kSortTile;
    uint64_t key[kSortItems];
    unsigned val[kSortItems], at[kSortItems];
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int i = (w * kSortItems + r) * 64 + lane;
        key[r] = i < here ? keys_in[tile0 + i] : 0ull;
        val[r] = i < here ? vals_in[tile0 + i] : 0u;
    }
    if (tot) {
        if (t < 256) base[t] = tot[(tile / kChunk) * 256 + t] + counts[tile * 256 + t];
    } else {
        // four groups of 256 threads sum every fourth row; cnt is free here
        unsigned before = 0, all = 0;
        const int d = t & 255, g = t >> 8;
#pragma unroll 8
        for (int r = g; r < ntiles; r += kSortThreads / 256) {
            const unsigned c = counts[(int64_t)r * 256 + d];
            all += c;
            before += r < tile ? c : 0u;
        }
        cnt[g][d] = before;
        cnt[4 + g][d] = all;
        __syncthreads();
        unsigned mine = 0, total = 0;
        if (t < 256)
            for (int k = 0; k < 4; ++k) {
                mine += cnt[k][t];
                total += cnt[4 + k][t];
            }
        const unsigned start = scan256(total, wsum);
        if (t < 256) base[t] = start + mine;
    }
    __syncthreads();
    rank_tile<kSortItems>(key, here, shift, nbits, cnt, loc, wsum, at);
#pragma unroll
    for (int r = 0; r < kSortItems; ++r)
        if ((w * kSortItems + r) * 64 + lane < here) {
            skey[at[r]] = key[r];
            sval[at[r]] = val[r];
        }
    __syncthreads();
    // out in tile order: neighbouring threads write neighbouring places of
    // one digit's run (coalesced)
    const unsigned dmask = (1u << nbits) - 1u;
#pragma unroll
    for (int r = 0; r < kSortItems; ++r) {
        const int i = r * kSortThreads + t;
        if (i < here) {
            const uint64_t k = skey[i];
            const unsigned d = (unsigned)(k >> shift) & dmask;
            const unsigned dst = base[d] + ((unsigned)i - loc[d]);
            keys_out[dst] = k;
            vals_out[dst] = sval[i];
        }
    }
}

// All digits of up to kSortThreads * ITEMS items in one block, in place: a
// pass ranks the items, stages them in LDS and reads them back in order.
template <int ITEMS>
__global__ void __launch_bounds__(kSortThreads) radix_small(uint64_t *__restrict__ keys, unsigned *__restrict__ vals,
                                                            int n, int bits)
{
    __shared__ unsigned loc[256];
    __shared__ unsigned cnt[kSortWaves][256];
    __shared__ unsigned wsum[4];
    __shared__ uint64_t skey[kSortThreads * ITEMS];
    __shared__ unsigned sval[kSortThreads * ITEMS];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    uint64_t key[ITEMS];
    unsigned val[ITEMS], at[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int i = (w * ITEMS + r) * 64 + lane;
        key[r] = i < n ? keys[i] : 0ull;
        val[r] = i < n ? vals[i] : 0u;
    }
    for (int shift = 0; shift < bits; shift += 8) {
        rank_tile<ITEMS>(key, n, shift, bits - shift < 8 ? bits - shift : 8, cnt, loc, wsum, at);
#pragma unroll
        for (int r = 0; r < ITEMS; ++r)
            if ((w * ITEMS + r) * 64 + lane < n) {
                skey[at[r]] = key[r];
                sval[at[r]] = val[r];
            }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const int i = (w * ITEMS + r) * 64 + lane;
            if (i < n) {
                key[r] = skey[i];
                val[r] = sval[i];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int i = (w * ITEMS + r) * 64 + lane;
        if (i < n) {
            keys[i] = key[r];
            vals[i] = val[r];
        }
    }
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

}  // namespace

size_t scan_temp_bytes(int64_t n)
{
    size_t total = 0;
    int64_t m = ceil_div(n, kScanTile);
    while (m > 1) {
        total += (size_t)m * sizeof(unsigned) + 256;
        m = ceil_div(m, kScanTile);
    }
    return total + 256;
}

namespace {

template <bool BITS>
void exclusive_scan(const unsigned *in, unsigned *out, int64_t n, void *temp, hipStream_t s)
{
    if (n <= 0) return;
    const int64_t blocks = ceil_div(n, kScanTile);
    if (blocks == 1) {
        scan_tiles<BITS><<<1, kScanThreads, 0, s>>>(in, out, n, nullptr);
        return;
    }
    unsigned *sums = reinterpret_cast<unsigned *>(temp);
    char *rest = reinterpret_cast<char *>(temp) + (((size_t)blocks * sizeof(unsigned) + 255) & ~(size_t)255);
    scan_tiles<BITS><<<(unsigned)blocks, kScanThreads, 0, s>>>(in, out, n, sums);
    exclusive_scan<false>(sums, sums, blocks, rest, s);
    scan_add<<<(unsigned)blocks, kScanThreads, 0, s>>>(out, n, sums);
}

}  // namespace

void exclusive_scan_u32(unsigned *d_data, int64_t n, void *temp, hipStream_t s)
{
    exclusive_scan<false>(d_data, d_data, n, temp, s);
}

void exclusive_scan_bits(const unsigned *words, unsigned *out, int64_t n, void *temp, hipStream_t s)
{
    exclusive_scan<true>(words, out, n, temp, s);
}

size_t radix_temp_bytes(int64_t n)
{
    const int64_t ntiles = ceil_div(n > 0 ? n : 1, kSortTile);
    auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    return al((size_t)n * sizeof(uint64_t)) + al((size_t)n * sizeof(unsigned)) +
           al((size_t)ntiles * 256 * sizeof(unsigned)) +
           al((size_t)ceil_div(ntiles, kChunk) * 256 * sizeof(unsigned));
}

SortedPairs radix_sort_pairs(uint64_t *keys, unsigned *vals, int64_t n, int bits, void *temp, hipStream_t s)
{
    if (n <= 1 || bits <= 0) return {keys, vals};
    if (n <= kSortTile) {
        radix_small<kSortItems><<<1, kSortThreads, 0, s>>>(keys, vals, (int)n, bits);
        return {keys, vals};
    }
    if (n <= kSmallSort) {
        radix_small<kSmallItems><<<1, kSortThreads, 0, s>>>(keys, vals, (int)n, bits);
        return {keys, vals};
    }
    auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const int64_t ntiles = ceil_div(n, kSortTile);
    const int64_t nchunks = ceil_div(ntiles, kChunk);
    char *p = reinterpret_cast<char *>(temp);
    uint64_t *k_alt = reinterpret_cast<uint64_t *>(p);
    p += al((size_t)n * sizeof(uint64_t));
    unsigned *v_alt = reinterpret_cast<unsigned *>(p);
    p += al((size_t)n * sizeof(unsigned));
    unsigned *counts = reinterpret_cast<unsigned *>(p);
    p += al((size_t)ntiles * 256 * sizeof(unsigned));
    unsigned *tot = ntiles > kFusedTiles ? reinterpret_cast<unsigned *>(p) : nullptr;

    uint64_t *k_in = keys, *k_out = k_alt;
    unsigned *v_in = vals, *v_out = v_alt;
    for (int shift = 0; shift < bits; shift += 8) {
        const int nb = bits - shift < 8 ? bits - shift : 8;
        radix_hist<<<(unsigned)ntiles, kSortThreads, 0, s>>>(k_in, n, shift, (1u << nb) - 1u, counts);
        if (tot) {
            radix_chunks<<<(unsigned)nchunks, 256, 0, s>>>(ntiles, counts, tot);
            radix_chunk_starts<<<1, kSortThreads, 0, s>>>(nchunks, tot);
        }
        radix_scatter<<<(unsigned)ntiles, kSortThreads, 0, s>>>(k_in, v_in, k_out, v_out, n, shift, nb, counts, tot,
                                                                (int)ntiles);
        uint64_t *tk = k_in;
        k_in = k_out;
        k_out = tk;
        unsigned *tv = v_in;
        v_in = v_out;
        v_out = tv;
    }
    return {k_in, v_in};
}

}  // namespace start
