// Targets per wave of the rate kernels, as plain host arithmetic (no HIP types),
// so that it can be compiled and checked on its own.
#pragma once

#include <stdint.h>

#include <array>

namespace start {

// What the choice is made from: a batch's targets, its largest item's targets,
// sources and grid side, its largest opening angle, and whether any item is FP64.
struct BatchSize {
    int64_t total = 0, max_src = 0, max_t = 0;
    int grid = 0;
    double theta = 0.0;
    bool fp64 = false;
};

// Hundreds of sources and a small opening angle: most are taken one by one.
inline bool long_lists(const BatchSize &b) { return b.theta < 0.4 && b.max_src >= 256 && b.max_src < 4096; }

// Targets per wave by size.  Small calls take about total / 4096 (a power of
// two, at most 8), which keeps ~4096 waves in flight.  Beyond, a larger tile
// marches more rays of each source side by side, and a smaller one balances the
// chip's 8192 waves better, the more so the longer its walk is.  Measured (us,
// tiles of 8 / 16 / 32 / 64, theta = 1, FP32C): every particle a source, 2^17
// targets 1606 / 1685 / 1892 / 2402, 2^18 2972 / 2955 / 3364 / 3554, 370000
// 8550 / 7846 / 8099 / 8785, 2^19 11240 / 10580 / 10370 / 10970, 2^20 21580 /
// 19620 / 18520 / 18870; 1024 sources, 2^16 527 / 537 / 631 / 912, 2^17 954 /
// 930 / 945 / 1109, 2^18 1713 / 1579 / 1642 / 1700; 64 sources, 2^15 70 / 74 /
// 106 / 178, 2^16 221 / 192 / 196 / 272, 2^17 376 / 336 / 335 / 346, 2^18 666 /
// 582 / 574 / 575.  The limits are on the largest item, since a batch's scenes
// are walked apart, and on the total, which fills the chip: scenes of 16384
// targets with 1, 64 or 16384 sources take 1087 / 1124 / 1428 / 1570 us at 2^18
// targets in all, 2987 / 2848 / 3121 / 3423 at 2^20, 10640 / 9760 / 9869 / 9440
// at 2^22 (scenes of 4096: 805 / 863 / 918 / 1196, 2509 / 2419 / 2603 / 2773,
// 9387 / 8700 / 8593 / 8309).  The same lines hold in FP64, but for 64: 2^20 targets of
// 1024 sources take 11150 / 10650 with 32 / 64 (FP32C 10600 / 10680), and
// FP32C gains from it only beyond 1.5 million (2^21: 34720 / 33410).  With few
// sources a tile has enough targets to fill a batch of 64 rays (one source,
// 2^16 targets: 15 us with 64, 33 with 8).
//
// Where the lines depend on more than sizes (us, tiles of 16 / 32 / 64):
// - FP32C, particles that all emit, 128^3 cells: 330001 targets 7558 / 8070 /
//   9422, 420001 9205 / 9360 / 10328, 470001 10058 / 9821 / 11381, so 16 up to
//   7 * 2^16; FP64 9062 / 8912 / 9949 at 330001 and 7998 / 7614 / 8630 at 270001.
// - Few sources (below 4096) in FP64, beyond 2^18 targets: 64 (1024 sources,
//   330001 targets 15286 / 14380 / 13989 at theta = 0.5 and 5740 / 5630 / 5641 at
//   1; 2^19 21164 / 18134 / 16872 and 7834 / 7056 / 6794).
// - Long lists (256 sources or more, theta below 0.4) in FP32C: 64 from 3 * 2^17
//   targets (1024 sources at 0.3: 330001 27144 / 23934 / 24612, 420001 33498 /
//   28629 / 27819, 2^20 - / 57570 / 53620; 64 sources, 2^19: 3650 / 3840 with 32 /
//   64; 256 at 0.2: 420001 14673 / 13172 / 14017, 2^19 17771 / 16051 / 15698, so
//   up to 512 sources from 2^19), and 32 from the targets on whose waves fill the
//   chip (2^18 7288 / 6870 / 7049, FP64 6512 / 6393 / 6713; 200001 6036 / 6223 / -,
//   FP64 5520 / 5812 / -), but 16 there at theta = 0 (1024 sources 13529 / 14156 /
//   15624, FP64 13058 / 13870 / 14775) and beyond 2048 sources (3000 at 0.35: 9226 /
//   9379 / 9978, FP64 8388 / 8769 / 9756).
// - Short lists and short rays (scenes of at most 32^3 cells, us with 8 / 16 / 32 /
//   64): the march of a tile is then short beside its walk, so larger tiles, and
//   the total decides, not the largest scene.  64 sources on 16^3 cells, 64 scenes
//   of 4096 targets 300 / 267 / 265 / 264, 64 of 16384 952 / 812 / 768 / 705; on
//   32^3 1439 / 1283 / 1230 / 1266, FP64 1470 / 1288 / 1203 / 1171; 256 sources
//   2576 / 2324 / 2266 / 2360, FP64 2610 / 2349 / 2270 / 2222; 64 scenes of 4096
//   targets of 256 sources 756 / 724 / 731 / 732.
inline int tile_from_size(const BatchSize &b)
{
    const int64_t k16 = (int64_t)1 << 16;
    const bool few = b.max_src < 4096, lists = long_lists(b);
    const int64_t small_t = b.max_src < 1024 ? k16 / 2 : few ? k16 : 2 * k16;
    const int64_t mid_t = few || b.fp64 ? 4 * k16 : 7 * k16;
    const bool short_rays = b.grid <= 32;
    int h = 1;
    if (short_rays && b.max_src < 256 && b.total >= k16)
        h = b.total < 4 * k16 ? 16 : b.grid <= 16 || b.fp64 ? 64 : 32;
    else if (short_rays && b.max_src < 1024 && b.total >= 8 * k16)
        h = b.fp64 || b.total >= 64 * k16 ? 64 : 32;
    else if (b.max_t <= small_t && b.total <= 8 * k16)
        while (h < 8 && (int64_t)h * 2 * 4096 <= b.total) h *= 2;
    else if (b.max_t <= mid_t && b.total < 64 * k16)
        h = b.total < 32 * k16 ? 16 : 32;
    else if (few && b.fp64)
        h = 64;
    else
        h = b.total < (lists ? (b.max_src > 512 ? 6 : 8) * k16 : b.fp64 ? 16 * k16 : 24 * k16) ? 32 : 64;
    if (lists && b.theta > 0.0 && b.max_src <= 2048 && h == 16 && b.total >= 7 * k16 / 2) h = 32;
    while (h < 64 && h * b.max_src < 64) h *= 2;
    return h;
}

// ceil(log2(v)), at least 0
inline int size_class(int64_t v)
{
    int k = 0;
    while (k < 62 && ((int64_t)1 << k) < v) ++k;
    return k;
}

// The autotuner's size class of a batch: all that the choice above is made from.
using TileClass = std::array<int, 6>;
inline TileClass tile_class(const BatchSize &b)
{
    const int grid = size_class(b.grid);
    return {size_class(b.total), size_class(b.max_src), size_class(b.max_t), grid < 4 ? 4 : grid > 6 ? 6 : grid,
            b.fp64 ? 1 : 0, long_lists(b) ? (b.theta > 0.0 ? 1 : 2) : 0};
}

}  // namespace start
