// dq8 kernels for an array cut into segments of any lengths (tensors laid out back to back), one scale per
// segment: the paper's per-matrix maximum (Sec. 3.1, last paragraph) for a whole set of matrices in one launch
// instead of one call per matrix.
//
// bounds[0 .. n_seg] are element offsets, bounds[i] <= bounds[i + 1], segment i = [bounds[i], bounds[i + 1]).
// A workgroup copies them to LDS, every entry clamped to n, so that nothing the array holds can lead an access
// outside [0, n): the kernels walk the array in units of 1024 elements by position, and the segment of an
// element is looked up, never the elements of a segment.  Entries that do not ascend give meaningless
// results inside the arrays.
// A wavefront takes a unit at a time, its loads (which do not depend on the segments) issued before the stores of the unit
// before it (k_seg_decode: a unit ahead, as in k_encode_full).  The segment of the unit's first element comes from two votes over the bounds (64
// evenly spaced ones, then the 64 of the stretch the first vote names).  A unit inside one segment goes on with that
// segment's scale; in any other unit every lane looks the segments of its elements up between the unit's first and last
// segment and the same registers go on with scales per quad (per element in the rows of quads in which a segment ends).
// What bounds the kernels: HBM on long arrays, latency on short ones.  Mixed units used to walk sixteen consecutive
// elements per lane one after the other: the convnet's ten tensors (1.76 M elements), seven workers and the own
// gradients averaged: 30.7 us, 11.8 us now (8.3 us when no segment ends inside a unit); that set compressed 16.0 -> 9.8 us; the
// AlexNet-shaped bucket's sixteen matrices (61 M elements), maxima 53.8 -> 42.4 and compression 59.4 -> 46.6 us.
// Elements that are in no unit (fewer than four at the end of the array; all of them when floats lie at addresses that
// are no multiple of 4) go one by one.
#pragma once
#include "dq8_device.hpp"
#include "dq8_kernels_codec.hpp"

namespace {

constexpr int kSegMax = DQ8_MAX_SEGMENTS;  // segments per call: the bounds fit 32 KiB of LDS
constexpr int kSegWg = kWave * kSegWaves;

// The bounds as a workgroup holds them: all of them in LDS, and, where a wavefront has a lane for each (fewer than 64
// segments), one per lane in a register, so that the segment of a unit is one vote without a wait for LDS.
struct SegBounds {
    const uint64_t *lds;
    uint32_t n_seg;
    uint64_t own;  // bound number lane, the largest number in lanes past the last bound
};

// Copies bounds[0 .. n_seg] to LDS, clamped to n.  The caller synchronises the workgroup.
__device__ __forceinline__ SegBounds load_bounds(const uint64_t *__restrict__ bounds, uint32_t n_seg, size_t n, uint64_t *lds, uint32_t lane)
{
    SegBounds r = {lds, n_seg, ~(uint64_t)0};
    if (n_seg < (uint32_t)kWave) {
        if (lane <= n_seg) {
            const uint64_t b = bounds[lane];
            r.own = b < (uint64_t)n ? b : (uint64_t)n;
            if (threadIdx.x <= n_seg) lds[lane] = r.own;
        }
    } else {
        for (uint32_t i = threadIdx.x; i <= n_seg; i += blockDim.x) {
            const uint64_t b = bounds[i];
            lds[i] = b < (uint64_t)n ? b : (uint64_t)n;
        }
    }
    return r;
}

// The last segment whose first element is at or before element v (the same v in every lane), at most
// n_seg - 1: one vote of the wavefront, or two over the bounds in LDS.
__device__ __forceinline__ uint32_t segment_of_uniform(const SegBounds &sb, uint64_t v, uint32_t lane)
{
    const uint32_t n_seg = sb.n_seg;
    if (n_seg < (uint32_t)kWave) {
        const uint32_t c = (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(sb.own <= v));
        const uint32_t s = c ? c - 1 : 0;
        return s < n_seg - 1 ? s : n_seg - 1;
    }
    const uint64_t *lds = sb.lds;
    const uint32_t stride = (n_seg + kWave) / kWave;  // ceil((n_seg + 1) / 64), at most 64
    uint32_t i = lane * stride;
    i = i < n_seg ? i : n_seg;
    const uint32_t c1 = (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(lds[i] <= v && lane * stride <= n_seg));
    const uint32_t base = (c1 ? c1 - 1 : 0) * stride;
    uint32_t j = base + lane;
    const bool in = lane < stride && j <= n_seg;
    j = j < n_seg ? j : n_seg;
    const uint32_t c2 = (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(in && lds[j] <= v));
    const uint32_t s = base + (c2 ? c2 - 1 : 0);
    return s < n_seg - 1 ? s : n_seg - 1;
}

// The same for a v of the lane's own: binary search.
__device__ __forceinline__ uint32_t segment_of_lane(const uint64_t *lds, uint32_t n_seg, uint64_t v)
{
    uint32_t lo = 0, hi = n_seg;  // the answer is in [lo, hi)
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (lds[mid] <= v)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// The elements [start, start + len) of a unit or of a stretch of one, and the segments of its first and last element.
// first == last: the stretch lies inside that segment (the last segment takes whatever lies beyond its end).
struct SegSpan {
    size_t start;
    uint32_t len, first, last;
};

__device__ __forceinline__ SegSpan open_span(const SegBounds &sb, size_t start, uint32_t len, uint32_t lane)
{
    SegSpan q;
    q.start = start;
    q.len = len;
    q.first = segment_of_uniform(sb, start, lane);
    q.last = q.first;
    if (sb.n_seg < (uint32_t)kWave || (q.first != sb.n_seg - 1 && sb.lds[q.first + 1] < start + len)) {
        const uint32_t s = segment_of_uniform(sb, start + len - 1, lane);
        q.last = s > q.first ? s : q.first;
    }
    return q;
}

// Elements at .. of a short last unit, up to 1024 of them and at least four: where fewer are left, the unit's last four (some of
// them once more).  A short unit of more than 1024 elements is read again for this: its registers would have to be indexed at
// run time.
__device__ __forceinline__ SegSpan open_part(const SegBounds &sb, const SegSpan &unit, uint32_t at, uint32_t lane)
{
    const uint32_t left = unit.len - at;
    if (left >= 4) return open_span(sb, unit.start + at, left < (uint32_t)kSegUnit ? left : (uint32_t)kSegUnit, lane);
    return open_span(sb, unit.start + unit.len - 4, 4, lane);
}

// Segments of the elements that a lane holds of a stretch of 1024: quads quad_start(j * 64 + lane, len), j = 0 .. 3.
// split[j] (the same in all lanes): a segment ends inside a quad of row j, seg[j][1 .. 3] may differ from seg[j][0].
// ROWS: rows of 64 quads; `row` is the first one's quad (0 but where the wavefronts of a workgroup share the stretch).
template <int ROWS>
struct SegQuads {
    uint32_t seg[ROWS][4];
    bool split[ROWS];
};

// Few segments in the stretch (mostly two): every lane counts, for each of its elements, the segments that have begun at or
// before it, one bound after the other; no wait but for the bound, no branch.  More than kCountedSegments: a search per quad
// and steps from element to element, which wait for LDS three to ten times, whatever the number of bounds.  In a graph, search /
// counting: expansion of 200 000 elements in 20 segments 4.9 / 4.0 us; 200 elements with 10 bounds inside 5.3 / 4.7, with 14 5.15 /
// 5.3, with 16 4.4 / 5.7; their compression with given scales with 9 bounds 4.6 / 4.9, 14 4.5 / 5.6; their maxima with 12 7.0 / 6.7, with
// 14 5.7 / 6.7.  (With 16 counted, given scales and maxima of such short sets took up to 1 us longer than with none.)
constexpr uint32_t kCountedSegments = 12;

template <int ROWS = kSegQ>
__device__ __forceinline__ SegQuads<ROWS> segments_of_quads(const SegBounds &sb, const SegSpan &q, uint32_t lane, uint32_t row = 0)
{
    SegQuads<ROWS> r;
    const uint64_t *lds = sb.lds;
    const uint32_t span = q.last - q.first;
    if (span <= kCountedSegments) {
        // the low half of bound i in a scalar register
        auto bound = [&](uint32_t i) {
            if (sb.n_seg < (uint32_t)kWave) return (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)sb.own, (int)i);
            return (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)lds[i]);
        };
#pragma unroll
        for (int j = 0; j < ROWS; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) r.seg[j][c] = q.first;
#pragma unroll 1
        for (uint32_t i = q.first + 1; i <= q.last; ++i) {
            const int32_t at = (int32_t)(bound(i) - (uint32_t)q.start);  // in the stretch, so below 4096
#pragma unroll
            for (int j = 0; j < ROWS; ++j) {
                const int32_t off = (int32_t)quad_start(row + j * kWave + lane, q.len);
#pragma unroll
                for (int c = 0; c < 4; ++c) r.seg[j][c] += off >= at - c ? 1u : 0u;
            }
        }
#pragma unroll
        for (int j = 0; j < ROWS; ++j) r.split[j] = __builtin_amdgcn_ballot_w64(r.seg[j][3] != r.seg[j][0]) != 0;
        return r;
    }
    // Whether segment i has begun at offset off of the stretch, for i in (first, last]: those begin inside the stretch,
    // so the difference fits 32 bits.
    auto begun = [&](uint32_t i, uint32_t off) { return (uint32_t)lds[i] - (uint32_t)q.start <= off; };
    const uint32_t top = 1u << (31 - __builtin_clz(span));
#pragma unroll
    for (int j = 0; j < ROWS; ++j) r.seg[j][0] = q.first;
    for (uint32_t step = top; step != 0; step >>= 1) {
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
            const uint32_t mid = r.seg[j][0] + step, in = mid < q.last ? mid : q.last;
            if (begun(in, quad_start(row + j * kWave + lane, q.len)) && mid <= q.last) r.seg[j][0] = mid;
        }
    }
#pragma unroll
    for (int j = 0; j < ROWS; ++j) {
        const uint32_t off = quad_start(row + j * kWave + lane, q.len);
        uint32_t s = r.seg[j][0];
        const bool ends = s < q.last && begun(s + 1, off + 3);
        r.split[j] = __builtin_amdgcn_ballot_w64(ends) != 0;
#pragma unroll
        for (uint32_t c = 1; c < 4; ++c) {
            if (ends)
                while (s < q.last && begun(s + 1, off + c)) ++s;  // empty segments are stepped over
            r.seg[j][c] = s;
        }
    }
    return r;
}

// Scales of the four elements of row j.
template <int ROWS>
__device__ __forceinline__ v4f scales_of_quad(const float *scales, const SegQuads<ROWS> &sq, int j)
{
    const float s = scales[sq.seg[j][0]];
    v4f r = {s, s, s, s};
    if (sq.split[j]) {
        r.y = scales[sq.seg[j][1]];
        r.z = scales[sq.seg[j][2]];
        r.w = scales[sq.seg[j][3]];
    }
    return r;
}

// Elements of unit u (units of U elements; the last one may be shorter, at least four).
template <int U>
__device__ __forceinline__ uint32_t seg_unit_len(size_t u, size_t n)
{
    return cap_to_unit<U>(n - u * (size_t)U);
}

// Calls f(element, segment) for the elements from `from` on, one per lane of the grid at a time.
template <typename F>
__device__ __forceinline__ void for_each_element(const uint64_t *lds, uint32_t n_seg, size_t from, size_t n, size_t n_waves, F f)
{
    for (size_t i = from + (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += n_waves * kWave)
        f(i, segment_of_lane(lds, n_seg, i));
}

// Maxima of the segments into zeroed scales (non-negative binary32 numbers order like their bit patterns, so the pieces
// of a segment merge with an integer atomic max).  A workgroup keeps the maxima of all segments in LDS and sends those
// that are not zero at its end, sixty-four of them in an instruction: atomics on one address are served one after the
// other, about 10 ns each, and the walk by position brings every workgroup to every long segment.
// Units of Q * 256 elements: 16 quads per lane on long arrays, 4 where that leaves wavefronts without work (the plan's
// items of four units and of one).
// A unit with several segments goes on with the registers it was loaded into (read again, it kept its wavefront and the kernel
// longer: maxima and compression of 25 M elements in 30 segments 42.1 us, 41.2 so).
// NT = 0, plain loads, where the array or much of it is still in the memory-side cache when k_seg_encode reads it again
// (kPlainBeforeCompression; by itself up to kCachedFloats): with non-temporal loads here k_seg_encode takes 33.4 instead of 26.8 us
// at 37.7 M elements and 53 instead of 43 us at 61 M, this one 1 to 2 us less.  By itself, 1000 M: 643 plain, 574 us.
// PARTS: workgroup w stores its maximum of segment i to scales[i * kMostParts + w] instead, scratch memory of the call, for
// k_seg_encode to combine: no zero fill before this kernel and no atomics.
template <int Q, int NT, bool PARTS>
__global__ __launch_bounds__(kSegWg) void k_seg_absmax(const float *__restrict__ x, size_t n, const uint64_t *__restrict__ bounds,
                                                       uint32_t n_seg, size_t n_units, size_t n_waves, float *__restrict__ scales)
{
    constexpr int U = Q * 4 * kWave;
    extern __shared__ uint64_t seg_lds[];  // the bounds, then the maxima
    uint32_t *best = reinterpret_cast<uint32_t *>(seg_lds + n_seg + 1);
    const uint32_t lane = threadIdx.x & 63;
    v4f v[Q];
    auto fetch = [&](size_t u) {
        const uint32_t len = seg_unit_len<U>(u, n);
#pragma unroll
        for (int j = 0; j < Q; ++j) v[j] = ldg_floats<NT>(x + u * (size_t)U, quad_start(j * kWave + lane, len));
    };
    size_t u = first_unit(kSegWaves);
    if (u < n_units) fetch(u);
    const SegBounds sb = load_bounds(bounds, n_seg, n, seg_lds, lane);
    for (uint32_t i = threadIdx.x; i < n_seg; i += kSegWg) best[i] = 0;
    __syncthreads();
    uint32_t run = 0, run_seg = 0;  // of the whole units of one segment so far
    auto post = [&] {
        const uint32_t m = wave_max_u32(run);
        if (lane == 0 && m != 0) atomicMax(best + run_seg, m);
        run = 0;
    };
    for (; u < n_units; u += n_waves) {
        const SegSpan q = open_span(sb, u * (size_t)U, seg_unit_len<U>(u, n), lane);
        if (q.first == q.last) {
            float fm = 0.0f;
#pragma unroll
            for (int j = 0; j < Q; ++j) fm = max4_abs(v[j], fm);
            if (u + n_waves < n_units) fetch(u + n_waves);
            if (q.first != run_seg) {
                post();
                run_seg = q.first;
            }
            run = run > f2u(fm) ? run : f2u(fm);
        } else {
            auto merge = [&](const SegSpan &part, const v4f (&w)[kSegQ]) {
                const SegQuads<kSegQ> sq = segments_of_quads(sb, part, lane);
#pragma unroll
                for (int j = 0; j < kSegQ; ++j) {
                    const uint32_t a[4] = {abs_bits(w[j].x), abs_bits(w[j].y), abs_bits(w[j].z), abs_bits(w[j].w)};
                    if (sq.split[j]) {
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (a[c] != 0) atomicMax(best + sq.seg[j][c], a[c]);
                    } else {
                        const uint32_t m01 = a[0] > a[1] ? a[0] : a[1], m23 = a[2] > a[3] ? a[2] : a[3];
                        const uint32_t m = m01 > m23 ? m01 : m23;
                        if (m != 0) atomicMax(best + sq.seg[j][0], m);
                    }
                }
            };
            if constexpr (Q == kSegQ) {
                merge(q, v);
            } else if (q.len == (uint32_t)U) {
#pragma unroll
                for (int p = 0; p < Q; p += kSegQ) {
                    const v4f w[kSegQ] = {v[p], v[p + 1], v[p + 2], v[p + 3]};
                    merge(open_span(sb, q.start + p * 4 * kWave, kSegUnit, lane), w);
                }
            } else {  // the short last unit
#pragma unroll 1
                for (uint32_t at = 0; at < q.len; at += kSegUnit) {
                    const SegSpan part = open_part(sb, q, at, lane);
                    v4f w[kSegQ];
#pragma unroll
                    for (int j = 0; j < kSegQ; ++j) w[j] = ldg_floats<NT>(x + part.start, quad_start(j * kWave + lane, part.len));
                    merge(part, w);
                }
            }
            if (u + n_waves < n_units) fetch(u + n_waves);
        }
    }
    post();
    for_each_element(seg_lds, n_seg, n_units * (size_t)U, n, n_waves, [&](size_t i, uint32_t seg) {
        const uint32_t a = abs_bits(x[i]);
        if (a != 0) atomicMax(best + seg, a);
    });
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n_seg; i += kSegWg) {
        if (PARTS)
            scales[i * kMostParts + blockIdx.x] = u2f(best[i]);
        else if (best[i] != 0)
            atomicMax(reinterpret_cast<unsigned int *>(scales) + i, best[i]);
    }
}

// Compression with the segments' scales (computed by k_seg_absmax or handed in).
// One unit's registers, requested again as soon as its codes are formed, and one copy of the code: 65 registers and 13 KB
// of instructions, where two sets of registers in turn had 90 and 47 KB, too many for the wavefronts that short arrays live
// on (16 Mi elements, given scales: 15.3 us so, 14.5 us now; 8 Mi 7.8 and 6.9).  The first loads come after the tables: in
// front of them, the tables wait until those loads have come (4 Mi: 5.0 against 4.7 us).
// WAVES: 8, with 24 wavefronts on a compute unit, or, on arrays of at least four units for each of 32 wavefronts, 16 with
// two workgroups per compute unit one after the other: 61 M elements 54.0 against 52.4 us, 16 Mi 14.5 against 14.8, 4 Mi
// 4.7 against 5.4.  (64 registers, so that both workgroups are resident: 53.9 us.)
// FROM: where a unit finds its scale: in memory; in LDS, copied there with the bounds; or in LDS, formed from the maxima that the
// n_parts workgroups of k_seg_absmax<.., true> left in `parts` (a wavefront takes four segments at a time, the first workgroup
// stores the scales).  In a graph, before (zero fill, maxima with atomics, scales in memory) and now: 200 000
// elements in 20 segments 8.9 / 8.3 us, 1.76 M in 10 10.2 / 7.8, 8 Mi in 40 17.3 / 15.8, 61 M in 16 90.4 / 90.0.
enum SegScales { kScalesInMemory, kScalesCopied, kScalesFromParts };

template <bool REMAP, int WAVES, SegScales FROM>
__device__ __forceinline__ void encode_segments_body(const uint32_t *__restrict__ tab, const float *__restrict__ x, size_t n,
                                                     const uint64_t *__restrict__ bounds, uint32_t n_seg, size_t n_units, size_t n_waves,
                                                     const float *__restrict__ scales, float *__restrict__ scales_out,
                                                     const float *__restrict__ parts, uint32_t n_parts, uint8_t *__restrict__ codes)
{
    extern __shared__ uint64_t seg_lds[];  // the bounds (seg_bounds_words(n_seg) entries), the search table, the scales
    const uint32_t lane = threadIdx.x & 63;
    v4f v[kSegQ];
    auto fetch = [&](size_t u) {
        const uint32_t len = seg_unit_len<kSegUnit>(u, n);
#pragma unroll
        for (int j = 0; j < kSegQ; ++j) v[j] = ldg_floats<1>(x + u * (size_t)kSegUnit, quad_start(j * kWave + lane, len));
    };
    const BucketWords<kWave * WAVES> words = request_bucket_table<kWave * WAVES>(tab);
    const SegBounds sb = load_bounds(bounds, n_seg, n, seg_lds, lane);
    uint32_t *table = reinterpret_cast<uint32_t *>(seg_lds + seg_bounds_words(n_seg));
    float *near = reinterpret_cast<float *>(table + (tab[kNBucketOff] + 3) / 4 * 4);
    if (FROM == kScalesCopied)
        for (uint32_t i = threadIdx.x; i < n_seg; i += kWave * WAVES) near[i] = scales[i];
    if (FROM == kScalesFromParts) {
        constexpr uint32_t AT_ONCE = 4;
        for (uint32_t i = wave_in_wg() * AT_ONCE; i < n_seg; i += WAVES * AT_ONCE) {
            uint32_t m[AT_ONCE];
#pragma unroll
            for (uint32_t j = 0; j < AT_ONCE; ++j) m[j] = max_of_parts(parts + (i + j < n_seg ? i + j : i) * kMostParts, n_parts, lane);
#pragma unroll
            for (uint32_t j = 0; j < AT_ONCE; ++j)
                if (lane == 0 && i + j < n_seg) {
                    near[i + j] = u2f(m[j]);
                    if (blockIdx.x == 0) scales_out[i + j] = u2f(m[j]);
                }
        }
    }
    Search sr = place_bucket_table(tab, words, table);
    sr.marks = REMAP;
    __syncthreads();
    const float *sc = FROM == kScalesInMemory ? scales : near;
    size_t u = first_unit(WAVES);
    if (u < n_units) fetch(u);
    while (u < n_units) {
        const SegSpan q = open_span(sb, u * (size_t)kSegUnit, seg_unit_len<kSegUnit>(u, n), lane);
        u += n_waves;
        uint32_t cw[kSegQ];
        if (q.first == q.last) {
            const float s = sc[q.first];
            const float d = s == 0.0f ? 1.0f : s;
            encode_quads<true, kSegQ>(sr, v, d, 1.0f / d, reciprocal_ok(d), cw);
        } else {
            const SegQuads<kSegQ> sq = segments_of_quads(sb, q, lane);
            v4f d[kSegQ];
#pragma unroll
            for (int j = 0; j < kSegQ; ++j) d[j] = scales_of_quad(sc, sq, j);
#pragma unroll
            for (int j = 0; j < kSegQ; ++j) {
                const v4f t = v[j];
                const uint32_t s0 = search_sum_exact(sr, t.x / (d[j].x == 0.0f ? 1.0f : d[j].x));
                const uint32_t s1 = search_sum_exact(sr, t.y / (d[j].y == 0.0f ? 1.0f : d[j].y));
                const uint32_t s2 = search_sum_exact(sr, t.z / (d[j].z == 0.0f ? 1.0f : d[j].z));
                const uint32_t s3 = search_sum_exact(sr, t.w / (d[j].w == 0.0f ? 1.0f : d[j].w));
                cw[j] = pack_codes(sr, s0, s1, s2, s3, t);
            }
        }
        if (u < n_units) fetch(u);  // the next unit's loads fly while the codes are stored and its segment is looked up
        uint8_t *pc = codes + q.start;
        if (q.len == (uint32_t)kSegUnit) {
#pragma unroll
            for (int j = 0; j < kSegQ; ++j) stg_codes<1>(pc, 4 * (j * kWave + lane), cw[j]);
        } else {
#pragma unroll
            for (int j = 0; j < kSegQ; ++j) {
                const uint32_t k = j * kWave + lane;
                if (k * 4 < q.len) stg_codes<1>(pc, quad_start(k, q.len), cw[j]);
            }
        }
    }
    for_each_element(seg_lds, n_seg, n_units * (size_t)kSegUnit, n, n_waves, [&](size_t i, uint32_t seg) {
        const float s = sc[seg];
        codes[i] = (uint8_t)code_exact(sr, x[i], s == 0.0f ? 1.0f : s);
    });
}

template <bool REMAP, int WAVES>
__global__ __launch_bounds__(kWave *WAVES) void k_seg_encode(const uint32_t *__restrict__ tab, const float *__restrict__ x, size_t n,
                                                             const uint64_t *__restrict__ bounds, uint32_t n_seg, size_t n_units,
                                                             size_t n_waves, const float *__restrict__ scales, uint8_t *__restrict__ codes)
{
    encode_segments_body<REMAP, WAVES, kScalesInMemory>(tab, x, n, bounds, n_seg, n_units, n_waves, scales, nullptr, nullptr, 0, codes);
}

template <bool REMAP, int WAVES>
__global__ __launch_bounds__(kWave *WAVES) void k_seg_encode_copied(const uint32_t *__restrict__ tab, const float *__restrict__ x, size_t n,
                                                                    const uint64_t *__restrict__ bounds, uint32_t n_seg, size_t n_units,
                                                                    size_t n_waves, const float *__restrict__ scales,
                                                                    uint8_t *__restrict__ codes)
{
    encode_segments_body<REMAP, WAVES, kScalesCopied>(tab, x, n, bounds, n_seg, n_units, n_waves, scales, nullptr, nullptr, 0, codes);
}

template <bool REMAP, int WAVES>
__global__ __launch_bounds__(kWave *WAVES) void k_seg_encode_parts(const uint32_t *__restrict__ tab, const float *__restrict__ x, size_t n,
                                                                   const uint64_t *__restrict__ bounds, uint32_t n_seg, size_t n_units,
                                                                   size_t n_waves, const float *__restrict__ parts, uint32_t n_parts,
                                                                   float *__restrict__ scales, uint8_t *__restrict__ codes)
{
    encode_segments_body<REMAP, WAVES, kScalesFromParts>(tab, x, n, bounds, n_seg, n_units, n_waves, nullptr, scales, parts, n_parts, codes);
}

// Maxima and compression of a short array in one launch: k_encode_near for segments.  A workgroup of sixteen wavefronts
// compresses a slice of 4096 elements, a quad per thread.  The segments that lie inside the slice get their maxima from those
// quads; the one that the slice begins in and the one that it ends in are read whole, wherever they reach, four elements at
// a time per thread.  Nothing is passed from one workgroup to another, so there is no zero fill, no second launch and no
// atomic outside LDS.  Bytes are read up to once per workgroup, out of the L2, which up to kNearLongest elements costs less
// than the two launches.  The scale of a segment is written by the workgroup in whose 4096 elements it begins, those of empty
// segments at the end by the last one.  n >= 4.  In a graph, before and now: 3000 elements in 2 segments
// 9.7 / 3.9 us, in 60 segments 15.5 / 5.9, 30 000 in 10 10.8 / 6.2, 65 536 in 3 10.0 / 5.3, 98 304 in 20 11.1 / 6.6.
template <bool REMAP>
__global__ __launch_bounds__(kNearWg) void k_seg_near(const uint32_t *__restrict__ tab, const float *__restrict__ x, uint32_t n,
                                                      const uint64_t *__restrict__ bounds, uint32_t n_seg,
                                                      float *__restrict__ scales, uint8_t *__restrict__ codes)
{
    extern __shared__ uint64_t seg_lds[];  // the bounds (seg_bounds_words(n_seg) entries), the search table, the maxima
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t from = blockIdx.x * (uint32_t)kNearSlice, to = n - from < (uint32_t)kNearSlice ? n : from + (uint32_t)kNearSlice;
    const uint32_t begin = to - from < 4 ? n - 4 : from;  // a last slice under a quad takes the elements before it once more
    v4f own[1];
    own[0] = ldg_floats<0>(x + begin, quad_start(threadIdx.x, to - begin));
    const BucketWords<kNearWg> words = request_bucket_table<kNearWg>(tab);
    const SegBounds sb = load_bounds(bounds, n_seg, n, seg_lds, lane);
    uint32_t *table = reinterpret_cast<uint32_t *>(seg_lds + seg_bounds_words(n_seg));
    Search sr = place_bucket_table(tab, words, table);
    sr.marks = REMAP;
    uint32_t *best = table + (tab[kNBucketOff] + 3) / 4 * 4;
    for (uint32_t i = threadIdx.x; i < n_seg; i += kNearWg) best[i] = 0;
    __syncthreads();
    const SegSpan q = open_span(sb, begin, to - begin, lane);
    // Segment 0 takes what lies before its first element, the last one what lies beyond its end.
    auto start_of = [&](uint32_t i) { return i == 0 ? 0u : (uint32_t)seg_lds[i]; };
    auto end_of = [&](uint32_t i) { return i == n_seg - 1 ? n : (uint32_t)seg_lds[i + 1]; };
    auto whole_segment = [&](uint32_t i) {
        const uint32_t s0 = start_of(i), s1 = end_of(i);
        if (!(s0 < s1)) return;
        const uint32_t len = s1 - s0;
        float fm = 0.0f;
        if (len < 4) {
            if (threadIdx.x < len) fm = __builtin_fabsf(x[s0 + threadIdx.x]);
        } else if (len <= (uint32_t)kNearSlice) {
            fm = max4_abs(ldg_floats<0>(x + s0, quad_start(threadIdx.x, len)), 0.0f);
        } else {
            constexpr uint32_t R = 4;
            for (uint32_t k = 0; k * 4 < len; k += R * kNearWg) {
                v4f v[R];
#pragma unroll
                for (uint32_t j = 0; j < R; ++j) v[j] = ldg_floats<0>(x + s0, quad_start(k + j * kNearWg + threadIdx.x, len));
#pragma unroll
                for (uint32_t j = 0; j < R; ++j) fm = max4_abs(v[j], fm);
            }
        }
        const uint32_t m = wave_max_u32(f2u(fm));
        if (lane == 0 && m != 0) atomicMax(best + i, m);
    };
    whole_segment(q.first);
    SegQuads<1> sq;
    if (q.first != q.last) {
        whole_segment(q.last);
        sq = segments_of_quads<1>(sb, q, lane, wave_in_wg() * kWave);
        const uint32_t a[4] = {abs_bits(own[0].x), abs_bits(own[0].y), abs_bits(own[0].z), abs_bits(own[0].w)};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t seg = sq.seg[0][c];
            if (seg != q.first && seg != q.last && a[c] != 0) atomicMax(best + seg, a[c]);
        }
    }
    __syncthreads();
    uint32_t cw[1];
    if (q.first == q.last) {
        const float s = u2f(best[q.first]);
        const float d = s == 0.0f ? 1.0f : s;
        encode_quads<true, 1>(sr, own, d, 1.0f / d, reciprocal_ok(d), cw);
    } else {
        const v4f d = scales_of_quad(reinterpret_cast<const float *>(best), sq, 0), t = own[0];
        const uint32_t s0 = search_sum_exact(sr, t.x / (d.x == 0.0f ? 1.0f : d.x));
        const uint32_t s1 = search_sum_exact(sr, t.y / (d.y == 0.0f ? 1.0f : d.y));
        const uint32_t s2 = search_sum_exact(sr, t.z / (d.z == 0.0f ? 1.0f : d.z));
        const uint32_t s3 = search_sum_exact(sr, t.w / (d.w == 0.0f ? 1.0f : d.w));
        cw[0] = pack_codes(sr, s0, s1, s2, s3, t);
    }
    if (threadIdx.x * 4 < to - begin) stg_codes<0>(codes + begin, quad_start(threadIdx.x, to - begin), cw[0]);
    for (uint32_t i = threadIdx.x; i < n_seg; i += kNearWg) {
        const uint32_t s0 = start_of(i);
        if (s0 >= from && (s0 < to || to == n)) scales[i] = u2f(best[i]);
    }
}

// Decompression with the segments' scales.  (61 M elements: 64.8 us with conditions around the loads, 58.1 us so, with two
// workgroups per compute unit; 61 to 66 us with 8 or 16 code words per lane or a copy of the words instead of two slots.
// Plain stores: 50.8 us, but the kernel that follows waits for the caches to be written back: compression and expansion
// together 180 instead of 150 us.)  The stores of a whole unit stand without a condition: 4 Mi elements 7.4 -> 7.0 us.
// WAVES: 8, or 16 where segment_waves() says so: with 4095 segments only one workgroup's tables fit, and 16 wavefronts
// instead of 8 take 64.3 us for 61 M elements instead of 85.9, 10.4 instead of 17.4 for 8 Mi.
// NEAR: the segments' scales are copied to LDS with the bounds.  Fetched when a unit's segment is known they are one more
// round trip to memory for the wavefront, and four gathers for a unit with several segments: 8 Mi elements in 40 segments 8.6
// / 7.5 us.
template <int WAVES, bool NEAR>
__global__ __launch_bounds__(kWave *WAVES) void k_seg_decode(const uint32_t *__restrict__ tab, const uint8_t *__restrict__ codes,
                                                       const float *__restrict__ scales, size_t n,
                                                       const uint64_t *__restrict__ bounds, uint32_t n_seg, size_t n_units,
                                                       size_t n_waves, float *__restrict__ out)
{
    __shared__ __align__(256) float lut[256 * kLutCopies];
    extern __shared__ uint64_t seg_lds[];
    const uint32_t lane = threadIdx.x & 63, lane4 = lane * 4;
    struct Slot {
        uint32_t w[kSegQ];
    } a, b;
    auto fetch = [&](size_t u, Slot &sl) {
        const uint32_t len = seg_unit_len<kSegUnit>(u, n);
#pragma unroll
        for (int j = 0; j < kSegQ; ++j) sl.w[j] = ldg_codes<1>(codes + u * (size_t)kSegUnit, quad_start(j * kWave + lane, len));
    };
    const size_t u0 = first_unit(WAVES);
    if (u0 < n_units) fetch(u0, a);  // the first loads are in flight while the tables are built
    const float lut_value = request_lut(tab);
    float *near = reinterpret_cast<float *>(seg_lds + n_seg + 1);
    if (NEAR)
        for (uint32_t i = threadIdx.x; i < n_seg; i += kWave * WAVES) near[i] = scales[i];
    const SegBounds sb = load_bounds(bounds, n_seg, n, seg_lds, lane);
    place_lut<kWave * WAVES>(lut_value, lut);
    __syncthreads();
    const float *sc = NEAR ? near : scales;
    walk_units(u0, n_units, n_waves, a, b, fetch, [&](size_t u, Slot &sl) {
        const SegSpan q = open_span(sb, u * (size_t)kSegUnit, seg_unit_len<kSegUnit>(u, n), lane);
        float *po = out + q.start;
        auto expand = [&](int j, v4f s) {
            const uint32_t k = j * kWave + lane;
            v4f r;
            r.x = lut_at<0>(lut, sl.w[j], lane4) * s.x;
            r.y = lut_at<1>(lut, sl.w[j], lane4) * s.y;
            r.z = lut_at<2>(lut, sl.w[j], lane4) * s.z;
            r.w = lut_at<3>(lut, sl.w[j], lane4) * s.w;
            if (q.len == (uint32_t)kSegUnit)
                stg_floats<2>(po + 4 * k, r);
            else if (k * 4 < q.len)
                stg_floats<2>(po + quad_start(k, q.len), r);
        };
        if (q.first == q.last) {
            const float s = sc[q.first];
#pragma unroll
            for (int j = 0; j < kSegQ; ++j) expand(j, v4f{s, s, s, s});
        } else {
            const SegQuads<kSegQ> sq = segments_of_quads(sb, q, lane);
            v4f s[kSegQ];
#pragma unroll
            for (int j = 0; j < kSegQ; ++j) s[j] = scales_of_quad(sc, sq, j);
#pragma unroll
            for (int j = 0; j < kSegQ; ++j) expand(j, s[j]);
        }
    });
    for_each_element(seg_lds, n_seg, n_units * (size_t)kSegUnit, n, n_waves,
                     [&](size_t i, uint32_t seg) { out[i] = lut_code(lut, codes[i], lane4) * sc[seg]; });
}

// The same for long arrays and fewer than 64 segments, in the shape of k_decode: units of 4096 elements, sixteen code words per lane,
// four wavefronts per compute unit, the words copied before the next unit's are requested.  A unit with several segments goes
// on with the same words: read again it kept its wavefront, and with it the kernel, 4 us longer. In
// a graph, k_seg_decode / this: 12 Mi elements in 12 segments 13.7 / 11.4 us, 25 M in 30 24.8 / 22.0, 61 M in 16 56.4 / 51.6 (k_decode on
// one segment: 49.4); 8 Mi in 40 7.5 / 8.5 with the codes in the cache, 9.5 / 9.3 without.
__global__ __launch_bounds__(kWg) void k_seg_decode_long(const uint32_t *__restrict__ tab, const uint8_t *__restrict__ codes,
                                                         const float *__restrict__ scales, size_t n, const uint64_t *__restrict__ bounds,
                                                         uint32_t n_seg, size_t n_units, size_t n_waves, float *__restrict__ out)
{
    constexpr int Q = kUnitQuads;
    __shared__ __align__(256) float lut[256 * kLutCopies];
    extern __shared__ uint64_t seg_lds[];
    const uint32_t lane = threadIdx.x & 63, lane4 = lane * 4;
    float *near = reinterpret_cast<float *>(seg_lds + n_seg + 1);
    uint32_t w[Q];
    auto fetch = [&](size_t u) {
        const uint32_t len = cap_to_unit<kUnit>(n - u * (size_t)kUnit);
#pragma unroll
        for (int j = 0; j < Q; ++j) w[j] = ldg_codes<0>(codes + u * (size_t)kUnit, quad_start(j * kWave + lane, len));
    };
    size_t u = first_unit();
    if (u < n_units) fetch(u);  // the first loads are in flight while the tables are built
    const float lut_value = request_lut(tab);
    if (threadIdx.x < n_seg) near[threadIdx.x] = scales[threadIdx.x];
    const SegBounds sb = load_bounds(bounds, n_seg, n, seg_lds, lane);
    place_lut<kWg>(lut_value, lut);
    __syncthreads();
    auto expand = [&](uint32_t cw, v4f s) {
        v4f r;
        r.x = lut_at<0>(lut, cw, lane4) * s.x;
        r.y = lut_at<1>(lut, cw, lane4) * s.y;
        r.z = lut_at<2>(lut, cw, lane4) * s.z;
        r.w = lut_at<3>(lut, cw, lane4) * s.w;
        return r;
    };
    while (u < n_units) {
        const SegSpan q = open_span(sb, u * (size_t)kUnit, cap_to_unit<kUnit>(n - u * (size_t)kUnit), lane);
        u += n_waves;
        if (q.len == (uint32_t)kUnit) {
            uint32_t cur[Q];
#pragma unroll
            for (int j = 0; j < Q; ++j) cur[j] = w[j];
            if (u < n_units) fetch(u);
            float *po = out + q.start;
            if (q.first == q.last) {
                const float s = near[q.first];
#pragma unroll
                for (int j = 0; j < Q; ++j) stg_floats<2>(po + 4 * (j * kWave + lane), expand(cur[j], v4f{s, s, s, s}));
            } else {
#pragma unroll
                for (int p = 0; p < Q; p += kSegQ) {
                    const SegQuads<kSegQ> sq = segments_of_quads(sb, open_span(sb, q.start + p * 4 * kWave, kSegUnit, lane), lane);
#pragma unroll
                    for (int j = 0; j < kSegQ; ++j) stg_floats<2>(po + 4 * ((p + j) * kWave + lane), expand(cur[p + j], scales_of_quad(near, sq, j)));
                }
            }
        } else {  // the short last unit
#pragma unroll 1
            for (uint32_t at = 0; at < q.len; at += kSegUnit) {
                const SegSpan part = open_part(sb, q, at, lane);
                const SegQuads<kSegQ> sq = segments_of_quads(sb, part, lane);
                uint32_t cur[kSegQ];
#pragma unroll
                for (int j = 0; j < kSegQ; ++j) cur[j] = ldg_codes<0>(codes + part.start, quad_start(j * kWave + lane, part.len));
#pragma unroll
                for (int j = 0; j < kSegQ; ++j) {
                    const uint32_t k = j * kWave + lane;
                    const v4f r = expand(cur[j], scales_of_quad(near, sq, j));
                    if (k * 4 < part.len) stg_floats<2>(out + part.start + quad_start(k, part.len), r);
                }
            }
            if (u < n_units) fetch(u);
        }
    }
    for_each_element(seg_lds, n_seg, n_units * (size_t)kUnit, n, n_waves,
                     [&](size_t i, uint32_t seg) { out[i] = lut_code(lut, codes[i], lane4) * near[seg]; });
}

// Decompression of K workers' buffers and their average (optionally with a local fp32 array as the first term)
// with the segments' scales: the ordered sum of the other averaging kernels (product and sum rounded separately,
// workers in index order, then the division by the number of terms), any number of workers, two at a time in flight: every
// place past the last worker costs the loads of a worker, and every further pair of places registers of wavefronts (30.6 M
// elements in 16 segments with 1, 2, 4, 8, 9 workers: 27.3, 37.5, 49, 72, 80 us with two at a time; 38, 52, 57, 84, 100 us
// with four, 8 workers with eight 83 us).  WAVES as in k_seg_decode.
// AHEAD = 8: on arrays that are no more than a unit for every wavefront there is no next unit whose loads could cover the wait
// for a pair of workers, so all of them are requested before the tables are built.
// Eight ahead only for up to eight workers: the empty places of a second round of eight cost a worker's loads each, from codes at odd bytes
// more than is gained (one tensor of 60 000 elements, in a graph, two / four / eight ahead: nine workers 6.9 / 7.7 / 9.2 us, sixteen
// 8.4 / 9.1 / 10.3; 2 M, 32 workers 20.6 / 19.1 / 20.9).
// NEAR: all workers' scales in LDS (see k_seg_decode), row k for worker k.
// 1.76 M elements in 10 segments, seven workers and a local term, in a graph: 10.4 us with two ahead and the scales in memory, 8.5
// so; 3 M, three workers 10.5 / 8.1.  Four ahead in 128 registers spill two; in 168, without, one workgroup on a compute unit is
// faster (1.76 M, four workers and a local term 7.1 / 6.7 us, 2 M, three 5.7 / 5.3) and two, which then wait for each other, slower (3 M,
// three and a local term 8.1 / 10.5; 4 Mi, five 10.9 / 13.1).  Eight ahead with two workgroups on a compute unit, 4 Mi, eight workers: 20.3 us, 14.7 with two.
template <int WAVES, int AHEAD, bool NEAR>
__global__ __launch_bounds__(kWave *WAVES, AHEAD == 8 ? 2 : 4) void k_seg_avg(const uint32_t *__restrict__ tab, WorkerPtrs p, int K,
                                                    const float *__restrict__ local, size_t n,
                                                    const uint64_t *__restrict__ bounds, uint32_t n_seg, size_t n_units,
                                                    size_t n_waves, float *__restrict__ out)
{
    __shared__ __align__(256) float lut[256 * kLutCopies];
    extern __shared__ uint64_t seg_lds[];
    const uint32_t lane = threadIdx.x & 63, lane4 = lane * 4;
    const int terms = K + (local ? 1 : 0);
    const float fk = (float)terms;
    const bool pow2 = (terms & (terms - 1)) == 0;  // then acc * (1 / terms) equals acc / terms exactly
    const float rk = 1.0f / fk;
    auto mean_of = [&](float acc) { return pow2 ? acc * rk : acc / fk; };
    uint32_t w[AHEAD][kSegQ];
    v4f acc[kSegQ];
    // The local term's quads of unit u and the first AHEAD workers' codes.
    auto fetch_workers = [&](size_t start, uint32_t len, int k0) {
#pragma unroll
        for (int c = 0; c < AHEAD; ++c) {
            const uint8_t *pc = p.codes[k0 + c < K ? k0 + c : K - 1] + start;  // a place past the last worker repeats it and is not added
#pragma unroll
            for (int j = 0; j < kSegQ; ++j) w[c][j] = ldg_codes<1>(pc, quad_start(j * kWave + lane, len));
        }
    };
    auto fetch = [&](size_t u) {
        const size_t start = u * (size_t)kSegUnit;
        const uint32_t len = seg_unit_len<kSegUnit>(u, n);
        if (local) {
#pragma unroll
            for (int j = 0; j < kSegQ; ++j) acc[j] = ldg_floats<1>(local + start, quad_start(j * kWave + lane, len));
        } else {
#pragma unroll
            for (int j = 0; j < kSegQ; ++j) acc[j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
        }
        if (K > 0) fetch_workers(start, len, 0);
    };
    size_t u = first_unit(WAVES);
    if (u < n_units) fetch(u);  // the first loads are in flight while the tables are built
    const float lut_value = request_lut(tab);
    float *near = reinterpret_cast<float *>(seg_lds + n_seg + 1);
    if (NEAR)
        for (uint32_t k = wave_in_wg(); k < (uint32_t)K; k += WAVES)
            for (uint32_t i = lane; i < n_seg; i += kWave) near[k * n_seg + i] = p.scales[k][i];
    const SegBounds sb = load_bounds(bounds, n_seg, n, seg_lds, lane);
    place_lut<kWave * WAVES>(lut_value, lut);
    __syncthreads();
    auto scales_of = [&](int k) -> const float * { return NEAR ? near + (uint32_t)k * n_seg : p.scales[k]; };
    for (; u < n_units; u += n_waves) {
        const SegSpan q = open_span(sb, u * (size_t)kSegUnit, seg_unit_len<kSegUnit>(u, n), lane);
#pragma unroll
        for (int j = 0; j < kSegQ; ++j)  // the sum starts at +0: a local -0 becomes +0
            acc[j] = v4f{0.0f + acc[j].x, 0.0f + acc[j].y, 0.0f + acc[j].z, 0.0f + acc[j].w};
        auto add = [&](int c, int j, v4f s) {
            acc[j].x = acc[j].x + lut_at<0>(lut, w[c][j], lane4) * s.x;
            acc[j].y = acc[j].y + lut_at<1>(lut, w[c][j], lane4) * s.y;
            acc[j].z = acc[j].z + lut_at<2>(lut, w[c][j], lane4) * s.z;
            acc[j].w = acc[j].w + lut_at<3>(lut, w[c][j], lane4) * s.w;
        };
        if (q.first == q.last) {
            for (int k0 = 0; k0 < K; k0 += AHEAD) {
                if (k0 != 0) fetch_workers(q.start, q.len, k0);
                float s[AHEAD];
#pragma unroll
                for (int c = 0; c < AHEAD; ++c) s[c] = scales_of(k0 + c < K ? k0 + c : K - 1)[q.first];
#pragma unroll
                for (int c = 0; c < AHEAD; ++c) {
                    if (k0 + c < K) {
#pragma unroll
                        for (int j = 0; j < kSegQ; ++j) add(c, j, v4f{s[c], s[c], s[c], s[c]});
                    }
                }
            }
        } else {
            const SegQuads<kSegQ> sq = segments_of_quads(sb, q, lane);
            for (int k0 = 0; k0 < K; k0 += AHEAD) {
                if (k0 != 0) fetch_workers(q.start, q.len, k0);
                if (NEAR) {  // LDS: no need to ask for the scales of several workers at once
#pragma unroll
                    for (int c = 0; c < AHEAD; ++c) {
                        if (k0 + c < K) {
                            // The row is the compiler's only here: it would form the addresses of all rows' scales, 16
                            // registers each, before the loop.
                            uint32_t row = (uint32_t)(k0 + c) * n_seg;
                            asm volatile("" : "+s"(row));
                            const float *sk = near + row;
#pragma unroll
                            for (int j = 0; j < kSegQ; ++j) add(c, j, scales_of_quad(sk, sq, j));
                        }
                    }
                } else {
                    float s[AHEAD][kSegQ];
#pragma unroll
                    for (int c = 0; c < AHEAD; ++c)
#pragma unroll
                        for (int j = 0; j < kSegQ; ++j) s[c][j] = scales_of(k0 + c < K ? k0 + c : K - 1)[sq.seg[j][0]];
#pragma unroll
                    for (int j = 0; j < kSegQ; ++j) {
                        if (!sq.split[j]) {
#pragma unroll
                            for (int c = 0; c < AHEAD; ++c)
                                if (k0 + c < K) add(c, j, v4f{s[c][j], s[c][j], s[c][j], s[c][j]});
                        } else {
                            v4f t[AHEAD];
#pragma unroll
                            for (int c = 0; c < AHEAD; ++c) t[c] = scales_of_quad(scales_of(k0 + c < K ? k0 + c : K - 1), sq, j);
#pragma unroll
                            for (int c = 0; c < AHEAD; ++c)
                                if (k0 + c < K) add(c, j, t[c]);
                        }
                    }
                }
            }
        }
        v4f r[kSegQ];
#pragma unroll
        for (int j = 0; j < kSegQ; ++j) r[j] = v4f{mean_of(acc[j].x), mean_of(acc[j].y), mean_of(acc[j].z), mean_of(acc[j].w)};
        if (u + n_waves < n_units) fetch(u + n_waves);
        float *po = out + q.start;
#pragma unroll
        for (int j = 0; j < kSegQ; ++j) {
            const uint32_t k = j * kWave + lane;
            if (k * 4 < q.len) stg_floats<2>(po + quad_start(k, q.len), r[j]);
        }
    }
    for_each_element(seg_lds, n_seg, n_units * (size_t)kSegUnit, n, n_waves, [&](size_t i, uint32_t seg) {
        float a = 0.0f;
        if (local) a = a + local[i];
        for (int k = 0; k < K; ++k) a = a + lut_code(lut, p.codes[k][i], lane4) * scales_of(k)[seg];
        out[i] = mean_of(a);
    });
}

}  // namespace
