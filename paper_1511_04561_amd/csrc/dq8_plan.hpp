// Host-side launch planning of the dq8 library: how an array with its scale blocks is cut into units and how
// many wavefronts, teams and workgroups walk them.  Plain C++ (no HIP), so that it can be compiled and checked
// on its own; dq8.hip includes it.
#pragma once
#include <cstddef>
#include <cstdint>

#include "dq8.h"
#include "dq8_units.hpp"

namespace {

// Elements per scale block: `block` as the caller passed it, the whole array for 0 or a longer block.
inline size_t block_length(size_t n, size_t block) { return (block == 0 || block > n) ? n : block; }

// Unit for the kernels in which units are pieces of a block: starting from *quads per lane, the largest
// power of two of them whose unit (quads * 256 elements) is no longer than a block, at least one; every
// halving doubles *waves_per_cu (up to 32) so that the bytes in flight per compute unit stay the same.
inline void fit_unit_to_block(size_t block_len, int *quads, int *waves_per_cu)
{
    while (*quads > 1 && (size_t)*quads * 4 * kWave > block_len) {
        *quads >>= 1;
        *waves_per_cu = *waves_per_cu * 2 > 32 ? 32 : *waves_per_cu * 2;
    }
}

// Workers per chunk for the decode-and-average kernel that takes any number of workers a chunk at a time: the
// size from 3 to 8 with the fewest empty places in the last chunk (an empty place repeats a load), the largest
// such size; fewer than 3 workers are one chunk; K = 0 (the local term alone) has no chunks at all.
inline int chunk_size(int K)
{
    if (K < 3) return K < 1 ? 1 : K;
    int best = 3;
    for (int c = 3, waste = DQ8_MAX_K; c <= 8; ++c) {
        const int w = (K + c - 1) / c * c - K;
        if (w <= waste) {
            waste = w;
            best = c;
        }
    }
    return best;
}

// Unit for the kernels that hold a whole block in registers: the smallest power of two of elements
// between 256 and 4096 that holds a block (4096 for longer blocks).
inline size_t holding_unit(size_t block_len)
{
    size_t unit = 256;
    while (unit < block_len && unit < (size_t)kUnit) unit <<= 1;
    return unit;
}

// The longest block that dq8_encode holds in a team's registers (maximum and quantisation from one read of x).
constexpr size_t kLongestHeldBlock = 16384;

// Elements per unit for compression: the smallest power of two that holds a block, up to 4096 when the scales
// are given and up to 16384 when the kernel computes them.
inline size_t encode_unit(size_t block_len, bool fused)
{
    if (fused && block_len > (size_t)kUnit && block_len <= kLongestHeldBlock) return block_len <= 8192 ? 8192 : 16384;
    return holding_unit(block_len);
}

struct Plan {
    size_t B, nb, upb, n_units, n_teams;
    unsigned grid;
};

// Units, and a grid in which every team (wpb wavefronts) walks the same number of them.
inline Plan make_plan(size_t n, size_t block, int cus, int waves_per_cu, int wpb, int waves_per_wg = kWavesPerWg,
               size_t unit = kUnit)
{
    Plan p;
    p.B = block_length(n, block);
    p.nb = (n + p.B - 1) / p.B;
    p.upb = (p.B + unit - 1) / unit;
    if (p.nb == 1) {
        p.n_units = (n + unit - 1) / unit;
    } else {
        size_t last = n - (p.nb - 1) * p.B;  // the last block may be short
        p.n_units = (p.nb - 1) * p.upb + (last + unit - 1) / unit;
    }
    size_t max_teams = (size_t)cus * (size_t)waves_per_cu / (size_t)wpb;
    if (max_teams < 1) max_teams = 1;
    size_t per_team = (p.n_units + max_teams - 1) / max_teams;
    size_t teams = (p.n_units + per_team - 1) / per_team;
    size_t teams_per_wg = (size_t)waves_per_wg / wpb;
    size_t grid = (teams + teams_per_wg - 1) / teams_per_wg;
    p.grid = (unsigned)grid;
    p.n_teams = grid * teams_per_wg;
    return p;
}

// Whether every unit of the plan has at least four elements (a quad), the array's last one apart: its length goes to
// *tail when it is shorter, else 0.  False when that one is all there is.
inline bool units_of_quads(const Plan &p, size_t n, size_t unit, uint32_t *tail)
{
    const size_t piece = p.B % unit, last = (n - (p.nb - 1) * p.B) % unit;
    *tail = last < 4 ? (uint32_t)last : 0;
    if (p.nb > 1 && piece != 0 && piece < 4) return false;
    return p.n_units > (*tail != 0 ? 1u : 0u);
}

// ---- blocks of 4 .. 128 elements (powers of two): many blocks per 1024-element unit of a wavefront

constexpr int kSmallQ = 4;                          // quads per lane
constexpr size_t kSmallUnit = kSmallQ * 4 * kWave;  // 1024 elements

// Quads per block for those kernels, 0 when the block length does not qualify.  Blocks of 256 to 1024
// elements (one, two or four whole rows of a unit) qualify in the kernels that have to hold a block, up to
// the length from which the general kernel for that call is at least as fast: `longest`.
inline int small_block_lanes(size_t n, size_t block_len, size_t longest = 128)
{
    if (block_len < 4 || block_len > longest || (block_len & (block_len - 1)) != 0 || block_len >= n) return 0;
    return (int)(block_len / 4);
}

struct SmallPlan {
    size_t n_units = 0, n_waves = 0, done = 0;  // whole units, wavefronts in the grid, elements they cover
    unsigned grid = 0;
};

// Whole leading units of the array on `waves_per_cu` wavefronts per compute unit, `wpw` per workgroup.
inline SmallPlan make_small_plan(size_t n, int cus, int waves_per_cu, int wpw)
{
    SmallPlan p;
    p.n_units = n / kSmallUnit;
    if (p.n_units == 0) return p;
    size_t waves = (size_t)cus * (size_t)waves_per_cu;
    const size_t per = (p.n_units + waves - 1) / waves;
    waves = (p.n_units + per - 1) / per;
    p.grid = (unsigned)((waves + wpw - 1) / wpw);
    p.n_waves = (size_t)p.grid * wpw;
    p.done = p.n_units * kSmallUnit;
    return p;
}

// ---- kernels that walk an array by position

// Units of `unit` elements: a last one of fewer than four elements is none, and there are none at all when floats lie at
// addresses that are no multiple of 4.  The elements in no unit go one by one.
inline size_t whole_units(size_t n, size_t unit, bool aligned) { return aligned ? n / unit + (n % unit >= 4) : 0; }

// Grid for an array that is one block: workgroups of kOneWaves wavefronts, up to per_cu on a compute unit.
inline unsigned one_block_grid(int cus, size_t n, size_t unit, int per_cu)
{
    const size_t all = (n + unit * kOneWaves - 1) / (unit * kOneWaves), most = (size_t)cus * (size_t)per_cu;
    return (unsigned)(all < most ? all : most);
}

// The longest array whose maxima every workgroup forms by itself (k_encode_near, k_seg_near): at this length one workgroup reads
// 384 KiB, and one launch takes 5.3 us (one scale; 20 segments 6.6) where three take 7.0 (11.1).
constexpr size_t kNearLongest = 98304;

// Arrays that are read twice, first for their maxima: up to this many floats the first pass reads with plain loads, so that
// the second finds them in the memory-side cache, which holds kCachedFloats; longer arrays with non-temporal loads.
// What follows decides how far beyond the cache that pays (plain against non-temporal, both passes).  A compression, which
// reads the part that is left at the rate of the cache: 100 M floats 145.8 / 149.2 us, 300 M 440 / 448, 500 M 745 / 755,
// 1000 M 1570 / 1531.  The error statistics, which are bound by arithmetic: 50 M 96.3 / 96.4, 68 M 126 / 122, 1000 M 1590 / 1515.
constexpr size_t kCachedFloats = (size_t)1 << 26;
constexpr size_t kPlainBeforeCompression = (size_t)1 << 29, kPlainBeforeStatistics = kCachedFloats;

// Expansion of at least this many elements reads the codes with plain loads: in a graph 61 M codes from
// memory 50.1 / 49.4 us, from the memory-side cache 50.2 / 45.6; 16 Mi 15.6 / 14.2; 8 Mi 8.16 / 8.26.
constexpr size_t kCodesFromCache = (size_t)1 << 24;

// ---- tensors back to back, one scale each

// Expansion of at least this many elements in fewer than 64 segments takes units of 4096 elements (k_seg_decode_long, figures
// there): below, units of 1024 on sixteen wavefronts per compute unit are no more than two or three each.  Only where every quad that is
// stored is a multiple of 16 bytes: four wavefronts per compute unit have too few stores on their way where each touches one cache line
// more (30 segments, out at an odd float, units of 1024 / 4096: 11 M elements 15.2 / 18.1 us, 14 M 18.1 / 23.5, 20 M 24.4 / 27.6, 61 M 73.4 /
// 74.0, with the codes from memory 73.3 / 76.5; aligned 14 M 11.9 / 14.8 and, from memory, 15.8 / 16.3, 20 M 15.6 / 17.0 and 21.6 / 19.5, 36 M 35.7 / 28.1, 61 M
// 57.2 / 46.9).
constexpr size_t kLongSegments = (size_t)10 << 20;
inline bool long_segment_units(size_t n, size_t n_seg, uintptr_t out) { return n_seg < (size_t)kWave && n >= kLongSegments && (out & 15) == 0; }

// Wavefronts per workgroup of the kernels that keep a value table beside the bounds: kSegWaves, two such workgroups on a
// compute unit, or twice that where only one workgroup's tables fit and there are units for more than one each.
constexpr size_t kLdsPerCu = 160 * 1024, kValueTableBytes = 64 * 1024;
inline int segment_waves(int cus, size_t n, size_t n_seg)
{
    const bool two_fit = 2 * (kValueTableBytes + (n_seg + 1) * sizeof(uint64_t)) <= kLdsPerCu;
    return two_fit || n <= (size_t)cus * kSegWaves * kSegUnit ? kSegWaves : 2 * kSegWaves;
}

// Whether the kernels with a value table copy `count` scales to LDS beside the bounds of at most as many segments: two workgroups
// of kSegWaves still fit a compute unit then.
constexpr size_t kNearScales = 1024;
static_assert(2 * (kValueTableBytes + (kNearScales + 1) * sizeof(uint64_t) + kNearScales * sizeof(float)) <= kLdsPerCu, "two workgroups");
inline bool scales_fit_near(size_t count) { return count <= kNearScales; }

// Segments whose maxima the workgroups of the maximum pass leave in scratch memory (one row of kMostParts numbers each) for the
// compression to combine: a wavefront of that one combines four rows at a time, so with 64 segments two rounds of
// loads in front of the first unit, which is what a zero fill costs; rows of one call take 64 KiB.
constexpr size_t kMostSegmentsInParts = 64;

struct SegPlan {
    size_t n_items, n_waves, lds;
    uint32_t group;
    unsigned grid;
};

// Items of work, units of kSegUnit elements, on up to `waves_per_cu` wavefronts per compute unit, `waves_per_wg` per workgroup.
// grouped (the maxima): an item of work is four units when a workgroup per compute unit still gets two items or more
// per wavefront, else one unit (short arrays: as many wavefronts as there are units).
inline SegPlan make_segment_plan(int cus, size_t n, size_t n_seg, int waves_per_cu, bool grouped = false, int waves_per_wg = kSegWaves)
{
    SegPlan p;
    const size_t n_units = (n + kSegUnit - 1) / kSegUnit;
    size_t waves = (size_t)cus * (size_t)waves_per_cu;
    p.group = grouped && n_units >= (size_t)cus * kSegWaves * 8 ? 4u : 1u;
    if (p.group == 4) waves = (size_t)cus * kSegWaves;
    p.n_items = (n_units + p.group - 1) / p.group;
    if (waves > p.n_items) waves = p.n_items;
    p.grid = (unsigned)((waves + waves_per_wg - 1) / waves_per_wg);
    p.n_waves = (size_t)p.grid * waves_per_wg;
    p.lds = (n_seg + 1) * sizeof(uint64_t);
    return p;
}

// Which form of the averaging kernel a call takes, and its launch: the plan is made for the form's wavefronts per workgroup, which
// the kernel numbers its wavefronts by.  near: the scales are in LDS, only beside bounds of which two workgroups' fit (without a
// worker there are no scales, however many segments).  ahead: workers requested at once, figures at the kernel.
struct SegAverage {
    SegPlan plan;
    int waves, ahead;
    bool near;
};
inline SegAverage make_segment_average(int cus, size_t n, size_t n_seg, int K, size_t units)
{
    SegAverage a;
    a.waves = segment_waves(cus, n, n_seg);
    a.plan = make_segment_plan(cus, n, n_seg, 2 * kSegWaves, false, a.waves);
    a.near = a.waves == kSegWaves && scales_fit_near((size_t)K * n_seg);
    if (a.near) a.plan.lds += (size_t)K * n_seg * sizeof(float);
    const bool one_unit = units <= a.plan.n_waves, one_workgroup = a.plan.grid <= (unsigned)cus;
    a.ahead = a.near && one_unit && one_workgroup && K > 4 && K <= 8 ? 8 : (a.near && one_unit && K > 2 ? 4 : 2);
    return a;
}

}  // namespace
