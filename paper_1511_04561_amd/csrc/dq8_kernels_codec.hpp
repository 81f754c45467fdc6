// dq8 kernels for one buffer: block maxima, compression, decompression, and the calibration copy.
#pragma once
#include "dq8_device.hpp"

namespace {

__global__ void k_fill_zero(float *p, size_t n)
{
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

// Three arrays at once (the second and third no longer than the grid): one launch instead of three.
__global__ void k_fill_zero_three(float *a, size_t na, float *b, size_t nb, float *c, size_t nc)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < na) a[i] = 0.0f;
    if (i < nb) b[i] = 0.0f;
    if (i < nc) c[i] = 0.0f;
}

// Plain fp32 copy with the access pattern of the codec kernels (units of Q * 256 elements,
// 128-bit accesses).  Exists to calibrate bandwidth and hardware-counter readings against a
// kernel whose traffic is known exactly: 4 bytes read and 4 bytes written per element.
template <int Q, int NT>
__global__ __launch_bounds__(kWg) void k_copy(const float *__restrict__ src, float *__restrict__ dst, size_t n,
                                             size_t n_units, size_t n_waves)
{
    constexpr int U = Q * 4 * kWave;
    const uint32_t lane = threadIdx.x & 63;
    for (size_t u = first_unit(); u < n_units; u += n_waves) {
        Unit un = unit_of<U>(u, n, n, 1, 0);
        const float *ps = src + un.start;
        float *pd = dst + un.start;
        if (un.len == U && (((uintptr_t)ps | (uintptr_t)pd) & 15) == 0) {
            const v4f *s4 = reinterpret_cast<const v4f *>(ps);
            v4f *d4 = reinterpret_cast<v4f *>(pd);
            v4f v[Q];
#pragma unroll
            for (int j = 0; j < Q; ++j) v[j] = ldg<NT>(s4 + j * kWave + lane);
#pragma unroll
            for (int j = 0; j < Q; ++j) stg<NT>(d4 + j * kWave + lane, v[j]);
        } else {
            for (uint32_t i = lane; i < un.len; i += kWave) pd[i] = ps[i];
        }
    }
}

// Block maxima.  One wavefront per unit of Q * 256 elements.  upb == 1: each unit is a whole
// block and stores its maximum.  upb > 1: scales[] was zeroed and the pieces of a block merge
// with an integer atomic max (non-negative binary32 numbers order like their bit patterns).
// per_wave == 0: wavefront w takes units w, w + n_waves, ...  per_wave > 0 (used when blocks span
// several units): it takes the per_wave consecutive units from w * per_wave on, keeps one
// running maximum per lane while the block stays the same and issues one atomic per block it
// touches -- thousands of atomics on one address cost more than reading the array.
__device__ __forceinline__ void merge_max(float *scales, size_t block, size_t upb, uint32_t m)
{
    if (upb == 1)
        scales[block] = u2f(m);
    else
        atomicMax(reinterpret_cast<unsigned int *>(scales) + block, m);
}

// Blocks that are whole units (B a multiple of Q * 256, x a multiple of 4): the loop takes the array's n_units whole units
// by position and nothing else, a shorter last unit is done after it by the last wavefront.  HBM bounds it, with 16 KiB
// in flight per wavefront and few wavefronts, so those bytes have to stay in flight: four quads are reduced as soon as
// they have arrived and their registers requested again for the next unit (the scheduling barrier keeps the compiler
// from moving these loads to either end).  Loads and reduction of a whole unit in turn, waiting for the last quad before
// the first one is reduced and nothing is requested meanwhile: 39.1 us for 61.1 M elements in blocks of 4096; so
// 34.6 us (7.1 TB/s).
template <int Q, int NT>
__global__ __launch_bounds__(kWg) void k_absmax_whole(const float *__restrict__ x, size_t n, size_t upb, size_t n_units,
                                                     size_t n_waves, size_t per_wave, float *__restrict__ scales)
{
    constexpr int U = Q * 4 * kWave;
    constexpr int G = Q < 4 ? Q : 4;
    const uint32_t lane = threadIdx.x & 63;
    const size_t w = first_unit();
    size_t u = per_wave ? w * per_wave : w;
    const size_t stride = per_wave ? 1 : n_waves;
    const size_t end = per_wave ? (u + per_wave < n_units ? u + per_wave : n_units) : n_units;
    v4f v[Q];
    if (u < end) {
        size_t blk = upb == 1 ? u : u / upb;
        size_t left = upb == 1 ? 1 : (blk + 1) * upb - u;  // units of the block from u on
        uint32_t run = 0;  // this lane's maximum over the units of the current block so far
        auto flush = [&] {
            const uint32_t r = wave_max_u32(run);
            run = 0;
            if (lane == 0) merge_max(scales, blk, upb, r);
        };
#pragma unroll
        for (int j = 0; j < Q; ++j) v[j] = ldg_floats<NT>(x + u * (size_t)U, 4 * (j * kWave + lane));
        for (;;) {
            const size_t nx = u + stride;
            if (!(nx < end)) break;
            const float *px = x + nx * (size_t)U;
            float fm = 0.0f;
#pragma unroll
            for (int g = 0; g < Q; g += G) {
#pragma unroll
                for (int j = g; j < g + G; ++j) fm = max4_abs(v[j], fm);
#pragma unroll
                for (int j = g; j < g + G; ++j) v[j] = ldg_floats<NT>(px, 4 * (j * kWave + lane));
                __builtin_amdgcn_sched_barrier(0);
            }
            run = run > f2u(fm) ? run : f2u(fm);
            u = nx;
            if (--left == 0) {
                flush();
                blk = upb == 1 ? u : blk + 1;
                left = upb;
            }
        }
        float fm = 0.0f;
#pragma unroll
        for (int j = 0; j < Q; ++j) fm = max4_abs(v[j], fm);
        run = run > f2u(fm) ? run : f2u(fm);
        flush();
    }
    const uint32_t rest = (uint32_t)(n - n_units * (size_t)U);
    if (rest != 0 && w == n_waves - 1) {
        const float *px = x + n_units * (size_t)U;
        float fm = 0.0f;
        if (rest >= 4) {
#pragma unroll
            for (int j = 0; j < Q; ++j) v[j] = ldg_floats<NT>(px, quad_start(j * kWave + lane, rest));
#pragma unroll
            for (int j = 0; j < Q; ++j) fm = max4_abs(v[j], fm);
        } else if (lane < rest) {
            fm = __builtin_fabsf(px[lane]);
        }
        const uint32_t r = wave_max_u32(f2u(fm));
        if (lane == 0) merge_max(scales, n_units / upb, upb, r);
    }
}

// Any other blocks.
template <int Q, int NT>
__global__ __launch_bounds__(kWg) void k_absmax(const float *__restrict__ x, size_t n, size_t B, size_t nb, size_t upb,
                                               size_t n_units, size_t n_waves, size_t per_wave, float *__restrict__ scales)
{
    constexpr int U = Q * 4 * kWave;
    const uint32_t lane = threadIdx.x & 63;
    const size_t w = first_unit();
    size_t u = per_wave ? w * per_wave : w;
    const size_t stride = per_wave ? 1 : n_waves;
    const size_t end = per_wave ? (u + per_wave < n_units ? u + per_wave : n_units) : n_units;
    Unit un;
    bool fast = false;
    v4f v[Q];
    auto open_unit = [&](size_t uu, Unit &q, bool &f) {
        q = unit_of<U>(uu, n, B, nb, upb);
        f = q.len >= 4 && ((uintptr_t)x & 3) == 0;
        if (f) {
            const float *px = x + q.start;
#pragma unroll
            for (int j = 0; j < Q; ++j) v[j] = ldg_floats<NT>(px, quad_start(j * kWave + lane, q.len));
        }
    };
    if (u < end) open_unit(u, un, fast);
    uint32_t run = 0;  // this lane's maximum over the units of the current block so far
    while (u < end) {
        uint32_t m;
        if (fast) {
            float fm = 0.0f;
#pragma unroll
            for (int j = 0; j < Q; ++j) fm = max4_abs(v[j], fm);
            m = f2u(fm);
        } else {
            m = slow_absmax(x + un.start, un.len, lane);
        }
        const size_t blk = un.block;
        u += stride;
        const bool more = u < end;
        if (more) open_unit(u, un, fast);  // next unit's loads fly during the reduction
        run = run > m ? run : m;
        if (!more || un.block != blk) {
            const uint32_t r = wave_max_u32(run);
            run = 0;
            if (lane == 0) merge_max(scales, blk, upb, r);
        }
    }
}

// Maximum of an array that is one block, into a zeroed scale.  Units of Q * 256 elements, strided over the grid: at any
// moment the chip reads one narrow window of the array (37.7 M elements: 29.7 us while every wavefront had a stretch of
// its own, 27.0 us now).  A workgroup sends one atomic: atomics on one address are served one after the other, about 10 ns
// each.  NT = 0, plain loads, when the array is read again after this: then it stays in the memory-side cache (256 MB),
// which takes the second pass over 37.7 M elements from 33.4 to 26.8 us and costs this one a microsecond.
// n_units: whole units and a last one of at least four elements (see quad_start); the elements past them (at most three;
// all of them when x is no multiple of 4) go one by one.
// PARTS: workgroup w stores its maximum to scale[w] instead, scratch memory of the call, for k_encode_one<.., true> to read: no
// zero fill before this kernel and no atomics in it (both passes, in a graph: 131 072 elements 6.6 -> 5.5 us, 1 Mi 8.0 -> 5.9, 8 Mi
// 16.1 -> 12.8, 37.7 M 57.5 -> 56.3).
constexpr int kOneWg = kWave * kOneWaves;

template <int Q, int NT, bool PARTS>
__global__ __launch_bounds__(kOneWg) void k_absmax_one(const float *__restrict__ x, size_t n, size_t n_units, size_t n_waves,
                                                       float *__restrict__ scale)
{
    constexpr int U = Q * 4 * kWave;
    __shared__ uint32_t part[kOneWaves];
    const uint32_t lane = threadIdx.x & 63;
    uint32_t m = 0;
    v4f v[Q];
    auto fetch = [&](size_t u) {
        const float *px = x + u * (size_t)U;
        const uint32_t len = cap_to_unit<U>(n - u * (size_t)U);
#pragma unroll
        for (int j = 0; j < Q; ++j) v[j] = ldg_floats<NT>(px, quad_start(j * kWave + lane, len));
    };
    size_t u = first_unit(kOneWaves);
    if (u < n_units) fetch(u);
    while (u < n_units) {
        float fm = 0.0f;
#pragma unroll
        for (int j = 0; j < Q; ++j) fm = max4_abs(v[j], fm);
        u += n_waves;
        if (u < n_units) fetch(u);
        m = m > f2u(fm) ? m : f2u(fm);
    }
    for (size_t i = n_units * (size_t)U + (size_t)blockIdx.x * kOneWg + threadIdx.x; i < n; i += n_waves * kWave) {
        const uint32_t a = abs_bits(x[i]);
        m = m > a ? m : a;
    }
    m = wave_max_u32(m);
    if (lane == 0) part[wave_in_wg()] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < kOneWaves; ++w) m = m > part[w] ? m : part[w];
        if (PARTS)
            scale[blockIdx.x] = u2f(m);
        else if (m != 0)
            atomicMax(reinterpret_cast<unsigned int *>(scale), m);
    }
}

// The largest of n_parts <= kMostParts non-negative numbers (1 <= n_parts), by one wavefront, to all its lanes.
__device__ __forceinline__ uint32_t max_of_parts(const float *__restrict__ parts, uint32_t n_parts, uint32_t lane)
{
    uint32_t m = 0;
#pragma unroll
    for (uint32_t j = 0; j < kMostParts / kWave; ++j) {
        const uint32_t i = j * kWave + lane, p = f2u(parts[i < n_parts ? i : n_parts - 1]);
        m = m > p ? m : p;
    }
    return wave_max_u32(m);
}

// Compression of an array that is one block with its scale in memory: units of 1024 elements, the next unit's loads always
// ahead (37.7 M elements right after k_absmax_one: 30.3 us; 36.6 us in k_encode, which has conditions in its loop).
// n_units as in k_absmax_one.
// PARTS: the scale is the largest of the n_parts maxima that k_absmax_one<.., true> left, formed by every wavefront by itself; the
// first workgroup stores it.
template <bool REMAP, bool PARTS>
__global__ __launch_bounds__(kOneWg) void k_encode_one(const uint32_t *__restrict__ tab, const float *__restrict__ x, size_t n,
                                                       size_t n_units, size_t n_waves, float *__restrict__ scale,
                                                       const float *__restrict__ parts, uint32_t n_parts, uint8_t *__restrict__ codes)
{
    constexpr int Q = 4, U = Q * 4 * kWave;
    extern __shared__ uint32_t lds[];  // the bucket table
    const uint32_t lane = threadIdx.x & 63;
    struct Slot {
        v4f v[Q];
    } a, b;
    auto fetch = [&](size_t u, Slot &sl) {
        const uint32_t len = cap_to_unit<U>(n - u * (size_t)U);
#pragma unroll
        for (int j = 0; j < Q; ++j) sl.v[j] = ldg_floats<1>(x + u * (size_t)U, quad_start(j * kWave + lane, len));
    };
    const size_t u0 = first_unit(kOneWaves);
    if (u0 < n_units) fetch(u0, a);  // the first loads are in flight while the table is copied
    const float s = PARTS ? u2f(max_of_parts(parts, n_parts, lane)) : *scale;
    if (PARTS && blockIdx.x == 0 && threadIdx.x == 0) *scale = s;
    const float d = s == 0.0f ? 1.0f : s;
    const float r = 1.0f / d;
    const bool recip = reciprocal_ok(d);
    Search sr = load_bucket_table<kOneWg>(tab, lds);
    sr.marks = REMAP;
    __syncthreads();
    walk_units(u0, n_units, n_waves, a, b, fetch, [&](size_t u, Slot &sl) {
        const uint32_t len = cap_to_unit<U>(n - u * (size_t)U);
        uint8_t *pc = codes + u * (size_t)U;
        uint32_t cw[Q];
        encode_quads<true, Q>(sr, sl.v, d, r, recip, cw);
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const uint32_t q = j * kWave + lane;
            if (q * 4 < len) stg_codes<1>(pc, quad_start(q, len), cw[j]);
        }
    });
    for (size_t i = n_units * (size_t)U + (size_t)blockIdx.x * kOneWg + threadIdx.x; i < n; i += n_waves * kWave)
        codes[i] = (uint8_t)encode_one<true>(sr, x[i], d, r, recip);
}

// Compression of a short array that is one block, in one launch: a workgroup of sixteen wavefronts compresses 4096 elements
// and every workgroup forms the maximum of the whole array by itself, from R quads per thread that are all in flight at
// once (R a power of two with R * 4096 >= n; quads past the end repeat the last one).  What such a call costs is launches
// and the waits inside one, not bytes: the workgroups read up to kNearLongest elements again and again, out of the L2, in
// less time than one more launch takes.  n >= 4.  In a graph, before (up to 16384 elements one workgroup of four
// wavefronts, beyond that a zero fill, a maximum pass and a compression) and now: 4096 elements
// 2.6 / 2.3 us, 10 240 3.9 / 2.8, 16 384 4.7 / 2.9, 32 768 6.9 / 3.3, 65 536 6.9 / 4.2, 98 304 7.0 / 5.3.
constexpr int kNearWaves = 16, kNearWg = kWave * kNearWaves;
constexpr size_t kNearSlice = 4 * (size_t)kNearWg;

template <int R, bool REMAP>
__global__ __launch_bounds__(kNearWg) void k_encode_near(const uint32_t *__restrict__ tab, const float *__restrict__ x, uint32_t n,
                                                         float *__restrict__ scale, uint8_t *__restrict__ codes)
{
    extern __shared__ uint32_t lds[];  // kNearWaves maxima, then the bucket table
    const uint32_t lane = threadIdx.x & 63, q = blockIdx.x * kNearWg + threadIdx.x;
    const BucketWords<kNearWg> words = request_bucket_table<kNearWg>(tab);
    v4f own[1], v[R];
    own[0] = ldg_floats<0>(x, quad_start(q, n));
    if constexpr (R > 1) {
#pragma unroll
        for (int j = 0; j < R; ++j) v[j] = ldg_floats<0>(x, quad_start(j * kNearWg + threadIdx.x, n));
    }
    Search sr = place_bucket_table(tab, words, lds + kNearWaves);
    sr.marks = REMAP;
    float fm = max4_abs(own[0], 0.0f);
    if constexpr (R > 1) {
#pragma unroll
        for (int j = 0; j < R; ++j) fm = max4_abs(v[j], fm);
    }
    const uint32_t m = wave_max_u32(f2u(fm));
    if (lane == 0) lds[wave_in_wg()] = m;
    __syncthreads();
    const uint32_t all = wave_max_u32(lds[lane & (kNearWaves - 1)]);
    const float s = u2f(all);
    if (q == 0) *scale = s;
    const float d = s == 0.0f ? 1.0f : s;
    uint32_t cw[1];
    encode_quads<true, 1>(sr, own, d, 1.0f / d, reciprocal_ok(d), cw);
    if (q * 4 < n) stg_codes<0>(codes, quad_start(q, n), cw[0]);
}

// Compression.  A team of WPB wavefronts owns a unit of WPB * QL * 256 elements, QL quads per lane:
// WPB == 1, each wavefront of the workgroup walks its own units; WPB == 4, the workgroup's four
// wavefronts share a unit and combine their maxima through LDS.
// FUSED: a unit is a whole block (upb == 1); the team reduces the block's maximum from
// registers, stores it and quantises the same registers.  Otherwise the scale of the unit's
// block is read from scales[].
// The loop is software-pipelined: the loads of a team's next unit are issued before the
// current unit is reduced and quantised, so each wavefront always has loads in flight.
// A unit shorter than that (a block that is not a power of two, the end of a block or of the
// array) takes the same path (see quad_start); only units of fewer than four elements, and floats at addresses that
// are not a multiple of 4, go element by element.
// EVERY: the host has seen that there are no such units, but for one at the end of the array that is not counted among the
// units.  The loads then stand in the loop without a condition.  With one, the compiler has to reckon with registers of
// a unit that was loaded and not used, and waits for every load before it forms the next addresses (given scales,
// 61.1 M elements: blocks of 100 175.3 us, of 200 101.5 us; so 87.4 and 59.9 us).
template <int WPB, int QL, int NT, bool FUSED, bool FASTDIV, bool EVERY>
struct Encoder {
    static constexpr int Q = QL;
    static constexpr uint32_t TEAM = kWave * WPB;
    static constexpr int U = QL * 4 * (int)TEAM;
    // Units of 8192 and 16384 elements serve every block length above 4096: a short block leaves whole rows
    // of a unit empty, which are neither loaded nor quantised.
    static constexpr bool kSkipRows = WPB > 1 && QL > 4;

    const float *x;
    uint8_t *codes;
    float *scales;
    size_t n, B, nb, upb;
    uint32_t *slots;
    Search sr;
    uint32_t lane, wave, tl, phase;

    struct Slot {
        Unit un;
        bool fast;
        v4f v[Q];
    };

    __device__ __forceinline__ void fetch(size_t u, Slot &sl) const
    {
        sl.un = unit_of<U>(u, n, B, nb, upb);
        const float *px = x + sl.un.start;
        sl.fast = EVERY || (sl.un.len >= 4 && ((uintptr_t)x & 3) == 0);
        if (sl.fast) {
#pragma unroll
            for (int it = 0; it < Q; ++it) {
                if (kSkipRows && it * TEAM * 4 >= sl.un.len) {  // the same for the whole team: a row past the end of the unit
                    sl.v[it] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
                    continue;
                }
                sl.v[it] = ldg_floats<NT>(px, quad_start(it * TEAM + tl, sl.un.len));
            }
        }
    }

    __device__ __forceinline__ void process(Slot &sl)
    {
        const Unit &un = sl.un;
        const float *px = x + un.start;
        uint8_t *pc = codes + un.start;
        float s;
        if (FUSED) {
            uint32_t m;
            if (sl.fast) {
                float fm = 0.0f;
#pragma unroll
                for (int it = 0; it < Q; ++it) fm = max4_abs(sl.v[it], fm);
                m = f2u(fm);
            } else {
                m = slow_absmax<TEAM>(px, un.len, tl);
            }
            m = wave_max_u32(m);
            if (WPB > 1) {
                if (lane == 0) slots[phase * kWavesPerWg + wave] = m;
                __syncthreads();  // every wavefront of the workgroup walks the same units
                const uint32_t *sp = slots + phase * kWavesPerWg;
                uint32_t a = sp[0] > sp[1] ? sp[0] : sp[1], b = sp[2] > sp[3] ? sp[2] : sp[3];
                m = (uint32_t)__builtin_amdgcn_readfirstlane((int)(a > b ? a : b));
                phase ^= 1;  // the other half of slots next time: one barrier per unit is enough
            }
            s = u2f(m);
            if (tl == 0) scales[un.block] = s;
        } else {
            s = scales[un.block];
        }
        const float d = s == 0.0f ? 1.0f : s;  // a zero scale leaves the value as it is
        const float r = 1.0f / d;
        const bool recip = reciprocal_ok(d);
        if (sl.fast) {
            // quads whose table lookups are issued together; the team variant runs six teams per compute unit
            // and has no registers to spare for that
            constexpr int G = WPB > 1 ? 1 : (Q < 4 ? Q : 4);
#pragma unroll
            for (int g = 0; g < Q; g += G) {
                if (kSkipRows && g * TEAM * 4 >= un.len) continue;
                v4f vv[G];
                uint32_t cw[G];
#pragma unroll
                for (int it = 0; it < G; ++it) vv[it] = sl.v[g + it];
                encode_quads<FASTDIV, G>(sr, vv, d, r, recip, cw);
#pragma unroll
                for (int it = 0; it < G; ++it) {
                    const uint32_t q = (g + it) * TEAM + tl;
                    if (q * 4 < un.len) stg_codes<NT>(pc, quad_start(q, un.len), cw[it]);
                }
            }
        } else {
            for (uint32_t i = tl; i < un.len; i += TEAM) pc[i] = (uint8_t)encode_one<FASTDIV>(sr, px[i], d, r, recip);
        }
    }
};

// One wavefront compresses a last block of fewer than four elements (pointers to its elements, code bytes and scale).
__device__ __forceinline__ void encode_under_a_quad(const Search &sr, const float *px, uint32_t len, float *scale, uint8_t *pc, uint32_t lane)
{
    const float v = lane < len ? px[lane] : 0.0f;
    const float s = u2f(wave_max_u32(abs_bits(v)));
    const float d = s == 0.0f ? 1.0f : s;
    if (lane == 0) *scale = s;
    if (lane < len) pc[lane] = (uint8_t)code_exact(sr, v, d);
}

// tail: with EVERY, the elements of a last unit of fewer than four (0: none); unused otherwise.
template <int WPB, int QL, int NT, bool FUSED, bool FASTDIV, bool EVERY>
__global__ __launch_bounds__(kWg) void k_encode(const uint32_t *__restrict__ tab, const float *__restrict__ x, size_t n,
                                               size_t B, size_t nb, size_t upb, size_t n_units, size_t n_teams, uint32_t tail,
                                               float *__restrict__ scales, uint8_t *__restrict__ codes)
{
    static_assert(WPB == 1 || WPB == kWavesPerWg, "a team is one wavefront or the whole workgroup");
    using Enc = Encoder<WPB, QL, NT, FUSED, FASTDIV, EVERY>;
    extern __shared__ uint32_t lds[];
    Enc e;
    e.x = x;
    e.codes = codes;
    e.scales = scales;
    e.n = n;
    e.B = B;
    e.nb = nb;
    e.upb = upb;
    e.slots = lds;  // kTeamSlots words, then the bucket table
    e.lane = threadIdx.x & 63;
    e.wave = wave_in_wg();
    e.tl = WPB == 1 ? e.lane : threadIdx.x;
    e.phase = 0;
    size_t u = WPB == 1 ? first_unit() : (size_t)blockIdx.x;
    typename Enc::Slot a, b;
    if constexpr (WPB == 1) {
        if (u < n_units) e.fetch(u, a);  // the first loads are in flight while the table is copied
        e.sr = load_bucket_table<kWg, true>(tab, lds + kTeamSlots);
        __syncthreads();
    } else {
        // Teams: the table first.  Its words return after the unit's in any case, and with both under way the loop is compiled with
        // earlier waits (linear type, blocks of 3500: 61 M elements 58.6 us, 10.6 M 13.6; with the words copied one by one 57.1 and
        // 13.0; so 57.2 and 12.7.  Given scales, blocks of 4000 at an odd float 62.9, 60.7, 61.1; 5000, 10.6 M 16.1, 15.5, 14.9; 3 M
        // 6.8, 6.7, 5.9.  Not better: given scales, blocks of 3000, 61 M 61.7, 63.1, 63.0, and 4000 at even ones 57.0, 55.9, 57.0).
        e.sr = load_bucket_table<kWg, FUSED>(tab, lds + kTeamSlots);
        __syncthreads();
        if (u < n_units) e.fetch(u, a);
    }
    if constexpr (EVERY) {
        walk_units(u, n_units, n_teams, a, b, [&](size_t v, typename Enc::Slot &sl) { e.fetch(v, sl); },
                   [&](size_t, typename Enc::Slot &sl) { e.process(sl); });
        if (tail != 0 && blockIdx.x == gridDim.x - 1 && e.wave == 0) {
            const size_t at = n - tail;
            if (FUSED) {
                encode_under_a_quad(e.sr, x + at, tail, scales + nb - 1, codes + at, e.lane);
            } else if (e.lane < tail) {
                const float s = scales[nb - 1];
                codes[at + e.lane] = (uint8_t)code_exact(e.sr, x[at + e.lane], s == 0.0f ? 1.0f : s);
            }
        }
        return;
    }
    while (u < n_units) {
        size_t nx = u + n_teams;
        if (nx < n_units) e.fetch(nx, b);
        e.process(a);
        u = nx;
        if (!(u < n_units)) break;
        nx = u + n_teams;
        if (nx < n_units) e.fetch(nx, a);
        e.process(b);
        u = nx;
    }
}

// Compression of whole, aligned blocks of 4096 elements: the common case of k_encode<4, 4, NT, true,
// FASTDIV> (a team of four wavefronts per block, maximum and quantisation from registers) with
// nothing else in the loop.  Block b starts at element 4096 b, x is 16-byte and codes 4-byte
// aligned, so unit geometry is a multiplication and there is no slow path to branch around.
// A ragged last block of tail_len elements is done by the last workgroup after its loop.
// REMAP says whether code bytes of the data type can carry marks (see fix_marked_codes): known at compile time,
// so the test for it drops out of the loop.
template <int NT, bool FASTDIV, bool REMAP>
__global__ __launch_bounds__(kWg) void k_encode_full(const uint32_t *__restrict__ tab, const float *__restrict__ x,
                                                    uint32_t n_full, uint32_t n_teams, uint32_t tail_len,
                                                    float *__restrict__ scales, uint8_t *__restrict__ codes)
{
    constexpr int Q = kUnitQuads / kWavesPerWg;
    extern __shared__ uint32_t lds[];
    uint32_t *slots = lds;  // kTeamSlots words, then the bucket table
    const uint32_t lane = threadIdx.x & 63, wave = wave_in_wg(), tl = threadIdx.x;
    uint32_t phase = 0;
    Search sr;
    auto fetch = [&](uint32_t u, v4f(&v)[Q]) {
        const v4f *p4 = reinterpret_cast<const v4f *>(x) + (size_t)u * (kUnit / 4);
#pragma unroll
        for (int it = 0; it < Q; ++it) v[it] = ldg_at<NT>(p4, it * kWg + tl);
    };
    // Maximum over the team of the wave maxima m, through LDS; one barrier per call.
    auto team_max = [&](uint32_t m) {
        if (lane == 0) slots[phase * kWavesPerWg + wave] = m;
        __syncthreads();
        const uint32_t *sp = slots + phase * kWavesPerWg;
        const uint32_t a = sp[0] > sp[1] ? sp[0] : sp[1], b = sp[2] > sp[3] ? sp[2] : sp[3];
        phase ^= 1;  // the other half of slots next time
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)(a > b ? a : b));
    };
    auto process = [&](uint32_t u, v4f(&v)[Q]) {
        float fm = 0.0f;
#pragma unroll
        for (int it = 0; it < Q; ++it) fm = max4_abs(v[it], fm);
        const float s = u2f(team_max(wave_max_u32(f2u(fm))));
        if (tl == 0) scales[u] = s;
        const float d = s == 0.0f ? 1.0f : s;
        const float r = 1.0f / d;
        const bool recip = reciprocal_ok(d);
        uint32_t *c4 = reinterpret_cast<uint32_t *>(codes) + (size_t)u * (kUnit / 4);
        uint32_t cw[Q];
        encode_quads<FASTDIV, Q>(sr, v, d, r, recip, cw);
#pragma unroll
        for (int it = 0; it < Q; ++it) stg_at<NT>(c4, it * kWg + tl, cw[it]);
    };
    uint32_t u = blockIdx.x;
    v4f a[Q], b[Q];
    if (u < n_full) fetch(u, a);  // the first loads are in flight while the table is copied
    sr = load_bucket_table<kWg>(tab, lds + kTeamSlots);
    sr.marks = REMAP;  // known at compile time: no test for marked code bytes in the loop
    __syncthreads();
    // Steady state: the fetch of the next block is unconditional and comes before the work on the
    // current one, so at the point where the current block's registers are first read the compiler
    // knows exactly how many younger loads are outstanding and waits for the older ones only.  (A
    // fetch under "if there is a next block" merges with the path that has none, and the merged
    // state makes it wait for the loads it has just issued.)  The last block of a team is done
    // outside the steady state.
    if (u < n_full) {
        for (;;) {
            uint32_t nx = u + n_teams;
            if (!(nx < n_full)) {
                process(u, a);
                break;
            }
            fetch(nx, b);
            process(u, a);
            u = nx;
            nx = u + n_teams;
            if (!(nx < n_full)) {
                process(u, b);
                break;
            }
            fetch(nx, a);
            process(u, b);
            u = nx;
        }
    }
    if (tail_len != 0 && blockIdx.x == gridDim.x - 1) {
        const float *px = x + (size_t)n_full * kUnit;
        uint8_t *pc = codes + (size_t)n_full * kUnit;
        const bool quads = tail_len >= 4;  // see quad_start
        float fm = 0.0f;
        if (quads) {
#pragma unroll
            for (int it = 0; it < Q; ++it) a[it] = ldg_floats<NT>(px, quad_start(it * kWg + tl, tail_len));
#pragma unroll
            for (int it = 0; it < Q; ++it) fm = max4_abs(a[it], fm);
        } else if (tl < tail_len) {
            fm = __builtin_fabsf(px[tl]);
        }
        const float s = u2f(team_max(wave_max_u32(f2u(fm))));
        if (tl == 0) scales[n_full] = s;
        const float d = s == 0.0f ? 1.0f : s;
        const float r = 1.0f / d;
        const bool recip = reciprocal_ok(d);
        if (quads) {
#pragma unroll
            for (int it = 0; it < Q; ++it) {
                const uint32_t q = it * kWg + tl;
                const uint32_t cw = encode_quad<FASTDIV>(sr, a[it], d, r, recip);
                if (q * 4 < tail_len) stg_codes<NT>(pc, quad_start(q, tail_len), cw);
            }
        } else if (tl < tail_len) {
            pc[tl] = (uint8_t)encode_one<FASTDIV>(sr, px[tl], d, r, recip);
        }
    }
}

// Compression of blocks of up to QL * 256 elements, one wavefront per block: k_encode_long without the exchange
// between wavefronts.  Blocks have B >= 4 elements and start at every alignment of an element (see quad_start); the last
// block may be shorter (tail elements, 0: none; one of fewer than four elements is no unit and done after the loop).
// Wavefront w of the grid takes blocks w, w + n_waves, ...
// Rows of 1001 elements (2048 of them) took 14.0 us while such rows went element by element.
template <int QL, int NT, int WPW, bool REMAP>
__global__ __launch_bounds__(kWave * WPW) void k_encode_wave(const uint32_t *__restrict__ tab, const float *__restrict__ x,
                                                            uint32_t n_units, uint32_t n_waves, uint32_t B, uint32_t tail, float *__restrict__ scales,
                                                            uint8_t *__restrict__ codes)
{
    constexpr int Q = QL;
    constexpr int G = Q < 4 ? Q : 4;  // quads whose table lookups are issued together
    static_assert(Q % G == 0, "whole groups of quads");
    extern __shared__ uint32_t lds[];  // the bucket table
    const uint32_t lane = threadIdx.x & 63;
    Search sr;
    auto length_of = [&](uint32_t u) { return (tail >= 4 && u == n_units - 1) ? tail : B; };
    auto fetch = [&](uint32_t u, v4f(&v)[Q]) {
        const float *px = x + (size_t)u * B;
        const uint32_t len = length_of(u);
#pragma unroll
        for (int it = 0; it < Q; ++it) v[it] = ldg_floats<NT>(px, quad_start(it * kWave + lane, len));
    };
    auto process = [&](uint32_t u, v4f(&v)[Q]) {
        float fm = 0.0f;
#pragma unroll
        for (int it = 0; it < Q; ++it) fm = max4_abs(v[it], fm);
        const float s = u2f(wave_max_u32(f2u(fm)));
        if (lane == 0) scales[u] = s;
        const float d = s == 0.0f ? 1.0f : s;
        const float r = 1.0f / d;
        const bool recip = reciprocal_ok(d);
        uint8_t *pc = codes + (size_t)u * B;
        const uint32_t len = length_of(u);
#pragma unroll
        for (int g = 0; g < Q; g += G) {
            v4f vv[G];
            uint32_t cw[G];
#pragma unroll
            for (int it = 0; it < G; ++it) vv[it] = v[g + it];
            encode_quads<true, G>(sr, vv, d, r, recip, cw);
#pragma unroll
            for (int it = 0; it < G; ++it) {
                const uint32_t q = (g + it) * kWave + lane;
                if (q * 4 < len) stg_codes<NT>(pc, quad_start(q, len), cw[it]);
            }
        }
    };
    uint32_t u = (uint32_t)first_unit(WPW);
    v4f a[Q], b[Q];
    if (u < n_units) fetch(u, a);  // the first loads are in flight while the table is copied
    sr = load_bucket_table<kWave * WPW>(tab, lds);
    sr.marks = REMAP;  // known at compile time: no test for marked code bytes in the loop
    __syncthreads();
    // steady state as in k_encode_full: the next block's loads are issued unconditionally before the work on
    // the current one
    if (u < n_units) {
        for (;;) {
            uint32_t nx = u + n_waves;
            if (!(nx < n_units)) {
                process(u, a);
                break;
            }
            fetch(nx, b);
            process(u, a);
            u = nx;
            nx = u + n_waves;
            if (!(nx < n_units)) {
                process(u, b);
                break;
            }
            fetch(nx, a);
            process(u, b);
            u = nx;
        }
    }
    if (tail != 0 && tail < 4 && blockIdx.x == gridDim.x - 1 && wave_in_wg() == 0)
        encode_under_a_quad(sr, x + (size_t)n_units * B, tail, scales + n_units, codes + (size_t)n_units * B, lane);
}

// Decompression with units that do not follow the blocks: unit u is quads [u Q 64, (u + 1) Q 64) of the array
// (a quad = 4 consecutive elements; blocks are whole quads, bq of them, so a quad never straddles two blocks),
// whatever the block length.  The host picks Q and NS with Q 64 <= (NS - 1) bq: a unit then touches at most NS
// blocks, whose scales are NS scalar loads (indices clamped to the last block), and every quad selects its own
// by comparing its offset from the start of the unit's first block with bq, 2 bq, ...  The block index and
// offset of a wavefront's unit advance by the same step every iteration (step_b blocks and step_r < bq
// quads), so there is one division per wavefront.  Buffers may start at any element; the last unit may be
// short (a lane past the end repeats the last code word's load and stores nothing); `left` elements after the
// last whole quad (they belong to the last block) are done one by one by the wavefront that has the last unit.
template <int Q, int NS, int NT, int WPW>
__global__ __launch_bounds__(kWave * WPW) void k_decode_flat(const uint32_t *__restrict__ tab, const uint8_t *__restrict__ codes,
                                                            const float *__restrict__ scales, uint64_t nq, uint32_t left,
                                                            uint32_t bq, uint64_t nb, uint64_t n_units, uint32_t n_waves,
                                                            uint64_t step_b, uint32_t step_r, float *__restrict__ out)
{
    __shared__ __align__(256) float lut[256 * kLutCopies];
    constexpr uint32_t UQ = Q * kWave;  // quads per unit
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t lane4 = lane * 4;
    uint64_t u = first_unit(WPW);
    uint64_t b0 = (u * UQ) / bq;               // block of the unit's first quad
    uint32_t r0 = (uint32_t)((u * UQ) % bq);   // and that quad's offset in it
    uint32_t w[Q], len = 0;
    float sc[NS];
    auto open_unit = [&](uint64_t uu, uint64_t bb) {
        const uint8_t *pc = codes + uu * UQ * 4;
        const uint64_t rest = nq - uu * UQ;
        len = rest < UQ ? (uint32_t)rest : UQ;
        const uint32_t last = len - 1;
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const uint32_t i = j * kWave + lane;
            w[j] = ldg_codes<NT>(pc, 4 * (i < last ? i : last));
        }
#pragma unroll
        for (int t = 0; t < NS; ++t) sc[t] = scales[bb + t < nb ? bb + t : nb - 1];
    };
    if (u < n_units) open_unit(u, b0);  // the first loads are in flight while the table is built
    load_lut<kWave * WPW>(tab, lut);
    __syncthreads();
    while (u < n_units) {
        uint32_t cur[Q];
#pragma unroll
        for (int j = 0; j < Q; ++j) cur[j] = w[j];
        float cs[NS];
#pragma unroll
        for (int t = 0; t < NS; ++t) cs[t] = sc[t];
        const uint32_t nqu = len, base = r0 + lane;
        // The stores take any multiple of 4 bytes in the form of policy 2.  Indexed in quads: indexed in elements, the compiler
        // keeps sixteen offsets in registers through the loop (86 instead of 73), and blocks of 1000 take 57.6 instead
        // of 56.3 us (61.1 M elements; blocks of 3000 52.8 instead of 51.7).
        static_assert(NT == 2, "other policies need the type of unaligned quads");
        v4f *o4 = reinterpret_cast<v4f *>(out + u * UQ * 4);
        const bool last_unit = u == n_units - 1;
        const uint64_t last_block = nb - 1;
        u += n_waves;
        b0 += step_b;
        r0 += step_r;
        if (r0 >= bq) {
            r0 -= bq;
            b0 += 1;
        }
        if (u < n_units) open_unit(u, b0);
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const uint32_t o = base + j * kWave;
            float s = cs[0];
#pragma unroll
            for (int t = 1; t < NS; ++t) s = o >= (uint32_t)t * bq ? cs[t] : s;
            v4f r;
            r.x = lut_at<0>(lut, cur[j], lane4) * s;
            r.y = lut_at<1>(lut, cur[j], lane4) * s;
            r.z = lut_at<2>(lut, cur[j], lane4) * s;
            r.w = lut_at<3>(lut, cur[j], lane4) * s;
            if (j * kWave + lane < nqu) stg<NT>(o4 + j * kWave + lane, r);
        }
        if (last_unit && lane < left) {
            const uint64_t e = nq * 4 + lane;
            out[e] = lut_code(lut, codes[e], lane4) * scales[last_block];
        }
    }
    // an array shorter than a quad has no unit at all
    if (n_units == 0 && blockIdx.x == 0 && wave_in_wg() == 0 && lane < left) out[lane] = lut_code(lut, codes[lane], lane4) * scales[0];
}

// Compression of blocks of up to 16384 elements from one read of x: the scheme of k_encode_full with QPL
// quads per lane (a team of four wavefronts holds up to QPL * 1024 elements) and a block length given
// at run time.  Blocks have B >= 4 elements and start at every alignment of an element (see quad_start).  The last block
// may be shorter (tail elements, 0: none): it is one more unit, with its own length; one of fewer than four elements is
// no unit and done after the loop.
template <int QPL, int NT, bool REMAP>
__global__ __launch_bounds__(kWg) void k_encode_long(const uint32_t *__restrict__ tab, const float *__restrict__ x,
                                                    uint32_t n_units, uint32_t n_teams, uint32_t B, uint32_t tail,
                                                    float *__restrict__ scales, uint8_t *__restrict__ codes)
{
    constexpr int Q = QPL;
    constexpr int G = Q < 4 ? Q : (Q % 4 == 0 ? 4 : 2);  // quads whose table lookups are issued together
    static_assert(Q % G == 0, "whole groups of quads");
    extern __shared__ uint32_t lds[];
    uint32_t *slots = lds;  // kTeamSlots words, then the bucket table
    const uint32_t lane = threadIdx.x & 63, wave = wave_in_wg(), tl = threadIdx.x;
    uint32_t phase = 0;
    Search sr;
    auto length_of = [&](uint32_t u) { return (tail >= 4 && u == n_units - 1) ? tail : B; };
    auto fetch = [&](uint32_t u, v4f(&v)[Q]) {
        const float *px = x + (size_t)u * B;
        const uint32_t len = length_of(u);
#pragma unroll
        for (int it = 0; it < Q; ++it) v[it] = ldg_floats<NT>(px, quad_start(it * kWg + tl, len));
    };
    auto team_max = [&](uint32_t m) {
        if (lane == 0) slots[phase * kWavesPerWg + wave] = m;
        __syncthreads();
        const uint32_t *sp = slots + phase * kWavesPerWg;
        const uint32_t a = sp[0] > sp[1] ? sp[0] : sp[1], b = sp[2] > sp[3] ? sp[2] : sp[3];
        phase ^= 1;  // the other half of slots next time
        return (uint32_t)__builtin_amdgcn_readfirstlane((int)(a > b ? a : b));
    };
    auto process = [&](uint32_t u, v4f(&v)[Q]) {
        float fm = 0.0f;
#pragma unroll
        for (int it = 0; it < Q; ++it) fm = max4_abs(v[it], fm);
        const float s = u2f(team_max(wave_max_u32(f2u(fm))));
        if (tl == 0) scales[u] = s;
        const float d = s == 0.0f ? 1.0f : s;
        const float r = 1.0f / d;
        const bool recip = reciprocal_ok(d);
        uint8_t *pc = codes + (size_t)u * B;
        const uint32_t len = length_of(u);
#pragma unroll
        for (int g = 0; g < Q; g += G) {
            v4f vv[G];
            uint32_t cw[G];
#pragma unroll
            for (int it = 0; it < G; ++it) vv[it] = v[g + it];
            encode_quads<true, G>(sr, vv, d, r, recip, cw);
#pragma unroll
            for (int it = 0; it < G; ++it) {
                const uint32_t q = (g + it) * kWg + tl;
                if (q * 4 < len) stg_codes<NT>(pc, quad_start(q, len), cw[it]);
            }
        }
    };
    uint32_t u = blockIdx.x;
    v4f a[Q], b[Q];
    if (u < n_units) fetch(u, a);  // the first loads are in flight while the table is copied
    sr = load_bucket_table<kWg>(tab, lds + kTeamSlots);
    sr.marks = REMAP;  // known at compile time: no test for marked code bytes in the loop
    __syncthreads();
    // steady state as in k_encode_full: the next block's loads are issued unconditionally before the work on
    // the current one
    if (u < n_units) {
        for (;;) {
            uint32_t nx = u + n_teams;
            if (!(nx < n_units)) {
                process(u, a);
                break;
            }
            fetch(nx, b);
            process(u, a);
            u = nx;
            nx = u + n_teams;
            if (!(nx < n_units)) {
                process(u, b);
                break;
            }
            fetch(nx, a);
            process(u, b);
            u = nx;
        }
    }
    if (tail != 0 && tail < 4 && blockIdx.x == gridDim.x - 1 && wave_in_wg() == 0)
        encode_under_a_quad(sr, x + (size_t)n_units * B, tail, scales + n_units, codes + (size_t)n_units * B, lane);
}

// Decompression of one buffer: out = table[code] * scale.  One wavefront per unit of Q * 256
// elements: Q code words (4 codes each) per lane; the next unit's words are loaded before the
// current ones are expanded.
// RAGGED = true (chosen by the host when blocks are not whole units): a short unit of four elements or more stays on
// the pipelined path (see quad_start).  Otherwise a short unit is the last of the array: its loads are not ahead, but
// in flight together.
// LD: cache policy of the code loads.  Plain (0) on long arrays: codes that were written or read a short while ago are then taken
// from the memory-side cache and stay there (kCodesFromCache).
template <int Q, int NT, int WPW, bool RAGGED, int LD = NT>
__global__ __launch_bounds__(kWave * WPW) void k_decode(const uint32_t *__restrict__ tab, const uint8_t *__restrict__ codes,
                                                       const float *__restrict__ scales, size_t n, size_t B, size_t nb,
                                                       size_t upb, size_t n_units, size_t n_waves, float *__restrict__ out)
{
    __shared__ __align__(256) float lut[256 * kLutCopies];
    constexpr int U = Q * 4 * kWave;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t lane4 = lane * 4;
    size_t u = first_unit(WPW);
    Unit un;
    bool fast = false;
    uint32_t w[Q];
    auto expand = [&](uint32_t cw, float s) {
        v4f r;
        r.x = lut_at<0>(lut, cw, lane4) * s;
        r.y = lut_at<1>(lut, cw, lane4) * s;
        r.z = lut_at<2>(lut, cw, lane4) * s;
        r.w = lut_at<3>(lut, cw, lane4) * s;
        return r;
    };
    auto open_unit = [&](size_t uu, Unit &q, bool &f) {
        q = unit_of<U>(uu, n, B, nb, upb);
        f = ((uintptr_t)out & 3) == 0 && (RAGGED ? q.len >= 4 : q.len == U);
        if (f) {
            const uint8_t *pc = codes + q.start;
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                const uint32_t i = j * kWave + lane;
                w[j] = ldg_codes<LD>(pc, RAGGED ? quad_start(i, q.len) : 4 * i);
            }
        }
    };
    if (u < n_units) open_unit(u, un, fast);  // the first loads are in flight while the table is built
    load_lut<kWave * WPW>(tab, lut);
    __syncthreads();
    while (u < n_units) {
        const float s = scales[un.block];
        float *po = out + un.start;
        if (fast) {
            uint32_t cur[Q];
#pragma unroll
            for (int j = 0; j < Q; ++j) cur[j] = w[j];
            const uint32_t len = un.len;
            u += n_waves;
            if (u < n_units) open_unit(u, un, fast);
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                const uint32_t q = j * kWave + lane;
                const v4f r = expand(cur[j], s);
                if (!RAGGED)
                    stg_floats<NT>(po + 4 * q, r);
                else if (q * 4 < len)
                    stg_floats<NT>(po + quad_start(q, len), r);
            }
        } else {
            const uint8_t *pc = codes + un.start;
            if (!RAGGED && un.len >= 4 && ((uintptr_t)out & 3) == 0) {  // the short last unit of the array
                uint32_t cur[Q];
#pragma unroll
                for (int j = 0; j < Q; ++j) cur[j] = ldg_codes<LD>(pc, quad_start(j * kWave + lane, un.len));
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    const uint32_t q = j * kWave + lane;
                    if (q * 4 < un.len) stg_floats<NT>(po + quad_start(q, un.len), expand(cur[j], s));
                }
            } else {
                for (uint32_t i = lane; i < un.len; i += kWave) po[i] = lut_code(lut, pc[i], lane4) * s;
            }
            u += n_waves;
            if (u < n_units) open_unit(u, un, fast);
        }
    }
}

}  // namespace
