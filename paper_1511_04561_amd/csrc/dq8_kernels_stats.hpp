// dq8 kernels for the approximation-error statistics.
#pragma once
#include "dq8_device.hpp"
#include "dq8_kernels_codec.hpp"

namespace {

// Approximation-error statistics of compress-then-decompress (Sec. 3.4, Table 2).  Per block b,
// stats[4 b + 0] = sum of e, [1] = sum of e / |x| over x != 0, [2] = number of x != 0,
// [3] = largest e, with q = fl32(cb[code] * s) and e = |(double) q - (double) x| (one binary64
// subtraction; the quotient one correctly rounded binary64 division).
//
// What a lane does per element.  The code's sign is the sign of x (scales are not negative), so q and x have
// the same sign and e = | |q| - |x| |: the kernel works on magnitudes and never forms the code byte.  |q| comes
// from a table in LDS that is indexed by byte 2 of the search sum (the code field, marked or not, see
// fix_marked_codes) and holds one copy per lane, so the lookup address is one byte permute and no two lanes
// meet in a bank.  The number of non-zero inputs is counted on the scalar unit from the lanes' votes.
//
// The quotient e / |x|.  Both operands are binary32 magnitudes widened to binary64 (e is a difference of two of
// them): 0 <= e < 2^129, 2^-149 <= |x| < 2^128.  The quotient and every intermediate of the division are
// therefore normal binary64 numbers far from overflow and underflow, which is the one case in which the
// division's range reduction, its rescaling and its special-case selection do nothing.  What is left is the
// reciprocal estimate (v_rcp_f64, 2^29 units in the last place: a relative error of 2^-23), Newton steps on it, the
// quotient estimate and its correction with the remainder.  One Newton step is enough because |x| has 24 bits: it leaves
// a relative error of 2^-46, so e * r is off by as much, the remainder e - |x| q has at most 31 significant bits and is
// exact, and what is rounded in the last operation is off by 2^-92 of the quotient.  The quotient of a 53-bit and a 24-bit
// number that is not halfway between two binary64 numbers is at least 2^-78 of itself away from there, and it cannot be
// halfway (e would need 54 bits): the result is the correctly rounded quotient.
__device__ __forceinline__ double quotient_of_magnitudes(double e, double ax)
{
    double r = __builtin_amdgcn_rcp(ax);
    r = __builtin_fma(__builtin_fma(-ax, r, 1.0), r, r);
    const double q = e * r;
    return __builtin_fma(__builtin_fma(-ax, q, e), r, q);
}

// Magnitude table for the lookup above: row b (b = 0 .. 255, a possibly marked code byte) holds the table value
// of the code that byte stands for, 64 copies (one per lane); entry (b, lane) at byte address b * 256 + lane * 4.
// (see place_lut).
__device__ __forceinline__ float request_magnitude_lut(const uint32_t *tab)
{
    return u2f(tab[kCbOff + (fix_marked_codes(threadIdx.x & 255) & 0x7Fu)]);
}

// wavefronts per workgroup: two workgroups (two value tables) share a compute unit, six wavefronts per SIMD
// (25 million elements in one block: 41 us; one workgroup of 16 wavefronts, whose atomics at the end are half as many, 57 us)
constexpr int kStatsWaves = 12;
constexpr int kStatsWg = kStatsWaves * kWave;

// Running statistics of one wavefront for the block it is in.
struct ErrorSums {
    double sum_abs = 0.0, sum_rel = 0.0, worst = 0.0;
    uint64_t count = 0;  // wave-uniform: non-zero inputs of all lanes so far
};

// OWN = true: a wavefront owns whole blocks (block b of round i goes to wavefront b - i * n_waves; the blocks of the
// last, partial round are spread evenly over the wavefronts), adds a block's terms in a fixed order and stores the
// four numbers: no atomics, stats[] need not be zeroed, and the sums are the same in every launch.
// OWN = false (blocks too long or too few for that): a wavefront walks a contiguous run of `per_wave` units and
// merges its sums into stats[], which a kernel before this one has zeroed, with atomics when the block changes and at
// the end: the count and the maximum are exact in any order (integers below 2^53, and non-negative binary64 numbers
// order like their bit patterns); the two sums depend on the order only in their last bits.  Atomics on one address
// are served one after the other, about 10 ns each whoever sends them, so what the wavefronts of a workgroup still hold
// at the end is combined in LDS first and lanes 0 .. 3 of a group of four send the four numbers in one instruction.
// (25 million elements as one block: four atomics from each of 6104 wavefronts took 304 us, ten times the arithmetic;
// with 512 workgroups that combine first 43 us, 41 us with one Newton step in the quotient instead of two.)
// means (may be NULL; NULL too where there are many blocks): the workgroup that finishes last forms them from stats[], which saves the launch of
// k_error_means.  means[0], zeroed like stats[], counts the workgroups until then; every workgroup counts itself after
// its atomics have been performed, so the one that counts last sees them all (it reads with atomic loads: plain ones
// could come from its own compute unit's cache).  Nothing but atomics has to be seen, so waiting for them is enough: a
// release fence would also write the XCD's L2 back, for every wavefront (120 us in all).
// Units are Q * 256 elements; the loads of a wavefront's next unit are issued before the current one is worked on.
template <int Q, bool OWN>
__global__ __launch_bounds__(kStatsWg, kStatsWaves / 2) void k_error_stats(const uint32_t *__restrict__ tab, const float *__restrict__ x,
                                                         size_t n, size_t B, size_t nb, size_t upb, size_t n_units,
                                                         size_t per_wave, size_t n_waves,
                                                         const float *__restrict__ scales, double *__restrict__ stats,
                                                         double *__restrict__ means)
{
    constexpr int U = Q * 4 * kWave;
    __shared__ __align__(256) float lut[256 * kLutCopies];
    extern __shared__ uint32_t bucket_lds[];
    const float lut_value = request_magnitude_lut(tab);
    const BucketWords<kStatsWg> words = request_bucket_table<kStatsWg>(tab);
    place_lut<kStatsWg>(lut_value, lut);
    const Search sr = place_bucket_table(tab, words, bucket_lds);
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63, lane4 = lane * 4;
    const size_t wave = first_unit(kStatsWaves);

    ErrorSums acc;
    auto add = [&](float xv, float qmag) {
        const double ax = (double)__builtin_fabsf(xv);
        const double e = __builtin_fabs((double)qmag - ax);
        acc.sum_abs += e;
        acc.worst = __builtin_fmax(acc.worst, e);
        const bool nz = xv != 0.0f;
        acc.count += (uint64_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(nz));
        // no branch around the division: a zero's quotient is computed (it is a NaN) and not added, so that the
        // elements of a unit stay in one stretch of code that the scheduler can interleave
        const double rel = quotient_of_magnitudes(e, ax);
        acc.sum_rel += nz ? rel : 0.0;
    };
    // The wave's sums to every lane: a fixed tree over the lanes.
    auto combine_lanes = [&] {
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            acc.sum_abs += __shfl_xor(acc.sum_abs, m);
            acc.sum_rel += __shfl_xor(acc.sum_rel, m);
            acc.worst = __builtin_fmax(acc.worst, __shfl_xor(acc.worst, m));
        }
    };
    // Adds number c (0 .. 3) of a block's four to stats[].
    auto merge = [&](size_t blk, uint32_t c, double v) {
        double *p = stats + 4 * blk + c;
        if (c == 3)
            atomicMax(reinterpret_cast<unsigned long long *>(p), (unsigned long long)__double_as_longlong(v));
        else
            atomicAdd(p, v);
    };
    // The wave's sums for block blk are complete: stored, or merged by four lanes.
    auto flush = [&](size_t blk) {
        combine_lanes();
        const double cnt = (double)acc.count;
        if (OWN) {
            if (lane == 0) {
                double *p = stats + 4 * blk;
                p[0] = acc.sum_abs;
                p[1] = acc.sum_rel;
                p[2] = cnt;
                p[3] = acc.worst;
            }
        } else if (lane < 4) {
            merge(blk, lane, lane == 0 ? acc.sum_abs : (lane == 1 ? acc.sum_rel : (lane == 2 ? cnt : acc.worst)));
        }
        acc = ErrorSums();
    };
    // One unit whose quads are in v (whole, aligned) or that is read element by element.
    auto work = [&](const Unit &un, bool fast, const v4f (&v)[Q]) {
        const float s = scales[un.block];
        const float sa = __builtin_fabsf(s);
        const float d = s == 0.0f ? 1.0f : s;
        const float r = 1.0f / d;
        const bool recip = reciprocal_ok(d);
        if (fast) {
            uint32_t sum[Q][4];
            if (recip) {
                uint32_t all = 0xFFFFu;
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    sum[j][0] = search_sum(sr, v[j].x * r);
                    sum[j][1] = search_sum(sr, v[j].y * r);
                    sum[j][2] = search_sum(sr, v[j].z * r);
                    sum[j][3] = search_sum(sr, v[j].w * r);
                }
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    const uint32_t k01 = near_key(sum[j][0]) < near_key(sum[j][1]) ? near_key(sum[j][0]) : near_key(sum[j][1]);
                    const uint32_t k23 = near_key(sum[j][2]) < near_key(sum[j][3]) ? near_key(sum[j][2]) : near_key(sum[j][3]);
                    const uint32_t k = k01 < k23 ? k01 : k23;
                    all = all < k ? all : k;
                }
                // some value of some lane lies next to a threshold: the whole unit again with true divisions
                if (__builtin_amdgcn_ballot_w64(all <= 2 * kNearWindow) != 0) {
#pragma unroll
                    for (int j = 0; j < Q; ++j) {
                        sum[j][0] = search_sum_exact(sr, v[j].x / d);
                        sum[j][1] = search_sum_exact(sr, v[j].y / d);
                        sum[j][2] = search_sum_exact(sr, v[j].z / d);
                        sum[j][3] = search_sum_exact(sr, v[j].w / d);
                    }
                }
            } else {
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    sum[j][0] = search_sum_exact(sr, v[j].x / d);
                    sum[j][1] = search_sum_exact(sr, v[j].y / d);
                    sum[j][2] = search_sum_exact(sr, v[j].z / d);
                    sum[j][3] = search_sum_exact(sr, v[j].w / d);
                }
            }
            // byte 1 of the address = byte 2 of the sum (the code field), byte 0 = lane * 4
            auto magnitude = [&](uint32_t sm) {
                const uint32_t addr = __builtin_amdgcn_perm(sm, lane4, 0x0C0C0600u);
                return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(lut) + addr) * sa;
            };
            float qm[Q][4];  // all lookups first, so that their latencies overlap
#pragma unroll
            for (int j = 0; j < Q; ++j)
#pragma unroll
                for (int c = 0; c < 4; ++c) qm[j][c] = magnitude(sum[j][c]);
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                add(v[j].x, qm[j][0]);
                add(v[j].y, qm[j][1]);
                add(v[j].z, qm[j][2]);
                add(v[j].w, qm[j][3]);
            }
        } else {
            const float *px = x + un.start;
            for (uint32_t i0 = 0; i0 < un.len; i0 += kWave) {  // every lane takes part in the votes of add()
                const uint32_t i = i0 + lane;
                const bool in = i < un.len;
                const float xv = in ? px[i] : 0.0f;
                const uint32_t sm = search_sum_exact(sr, xv / d);
                const uint32_t addr = __builtin_amdgcn_perm(sm, lane4, 0x0C0C0600u);
                const float q = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(lut) + addr) * sa;
                add(xv, in ? q : 0.0f);  // a lane past the end adds e = 0 and no count
            }
        }
    };
    auto is_fast = [&](const Unit &un) { return un.len == (uint32_t)U && (((uintptr_t)(x + un.start)) & 15) == 0; };
    auto load = [&](const Unit &un, v4f (&v)[Q]) {
        const v4f *p4 = reinterpret_cast<const v4f *>(x + un.start);
#pragma unroll
        for (int j = 0; j < Q; ++j) v[j] = ldg<1>(p4 + j * kWave + lane);
    };

    if (OWN) {
        // blocks of this wavefront: one per full round, and possibly one of the last round
        const size_t rounds = nb / n_waves, rem = nb - rounds * n_waves;
        const size_t extra_lo = wave * rem / n_waves, extra_hi = (wave + 1) * rem / n_waves;
        const size_t mine = rounds + (extra_hi > extra_lo ? 1 : 0);
        if (mine == 0) return;
        auto block_of = [&](size_t i) { return i < rounds ? i * n_waves + wave : rounds * n_waves + extra_lo; };
        v4f va[Q], vb[Q];
        size_t i = 0, c = 0;  // block number i of this wavefront, unit c of it
        Unit cur = unit_of<U>(block_of(0) * upb, n, B, nb, upb);
        bool cur_fast = is_fast(cur);
        if (cur_fast) load(cur, va);
        for (;;) {
            // the unit after this one: the next of the block, or the first of the wavefront's next block
            size_t ni = i, nc = c + 1;
            if (nc * (size_t)U >= (size_t)(B < n - cur.block * B ? B : n - cur.block * B)) {
                ni = i + 1;
                nc = 0;
            }
            const bool more = ni < mine;
            Unit nxt = cur;
            bool nxt_fast = false;
            if (more) {
                nxt = unit_of<U>(block_of(ni) * upb + nc, n, B, nb, upb);
                nxt_fast = is_fast(nxt);
                if (nxt_fast) load(nxt, vb);
            }
            work(cur, cur_fast, va);
            if (!more || ni != i) flush(cur.block);
            if (!more) break;
            for (int j = 0; j < Q; ++j) va[j] = vb[j];
            cur = nxt;
            cur_fast = nxt_fast;
            i = ni;
            c = nc;
        }
    } else {
        const size_t u0 = wave * per_wave;
        const size_t u1 = u0 + per_wave < n_units ? u0 + per_wave : n_units;
        constexpr size_t kNoBlock = ~(size_t)0;
        size_t held = kNoBlock;  // the block that acc belongs to after the walk
        if (u0 < u1) {
            v4f va[Q], vb[Q];
            Unit cur = unit_of<U>(u0, n, B, nb, upb);
            bool cur_fast = is_fast(cur);
            if (cur_fast) load(cur, va);
            for (size_t u = u0; u < u1; ++u) {
                const bool more = u + 1 < u1;
                Unit nxt = cur;
                bool nxt_fast = false;
                if (more) {
                    nxt = unit_of<U>(u + 1, n, B, nb, upb);
                    nxt_fast = is_fast(nxt);
                    if (nxt_fast) load(nxt, vb);
                }
                work(cur, cur_fast, va);
                if (more && nxt.block != cur.block) flush(cur.block);
                for (int j = 0; j < Q; ++j) va[j] = vb[j];
                if (!more) held = cur.block;
                cur = nxt;
                cur_fast = nxt_fast;
            }
            combine_lanes();
        }
        // The workgroup's wavefronts post what they hold (the value table is not needed any more) and four threads per
        // wavefront speak for all that hold the same block, if theirs is the first of them.
        __syncthreads();
        double *post = reinterpret_cast<double *>(lut);                                // 4 numbers per wavefront
        uint64_t *post_block = reinterpret_cast<uint64_t *>(post + 4 * kStatsWaves);  // and their block
        uint32_t *last_flag = reinterpret_cast<uint32_t *>(post_block + kStatsWaves);
        const uint32_t wv = wave_in_wg();
        if (lane == 0) {
            post[4 * wv + 0] = acc.sum_abs;
            post[4 * wv + 1] = acc.sum_rel;
            post[4 * wv + 2] = (double)acc.count;
            post[4 * wv + 3] = acc.worst;
            post_block[wv] = held;
        }
        __syncthreads();
        if (threadIdx.x < 4 * kStatsWaves) {
            const uint32_t w = threadIdx.x >> 2, c = threadIdx.x & 3;
            const uint64_t b = post_block[w];
            if (b != kNoBlock && (w == 0 || post_block[w - 1] != b)) {  // runs are in ascending order: equal blocks are neighbours
                double v = post[4 * w + c];
                for (uint32_t i = w + 1; i < (uint32_t)kStatsWaves && post_block[i] == b; ++i) {
                    const double o = post[4 * i + c];
                    v = c == 3 ? __builtin_fmax(v, o) : v + o;
                }
                merge(b, c, v);
            }
        }
        if (means == nullptr) return;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's atomics, the ones on the way included, are performed
        __syncthreads();
        if (threadIdx.x == 0)
            *last_flag = __hip_atomic_fetch_add(reinterpret_cast<unsigned int *>(means), 1u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
        __syncthreads();
        if (*last_flag == 0) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        double a = 0.0, r = 0.0, c = 0.0;
        for (size_t b = threadIdx.x; b < nb; b += kStatsWg) {
            a += __hip_atomic_load(stats + 4 * b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            r += __hip_atomic_load(stats + 4 * b + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            c += __hip_atomic_load(stats + 4 * b + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) {
            a += __shfl_xor(a, m);
            r += __shfl_xor(r, m);
            c += __shfl_xor(c, m);
        }
        if (lane == 0) {
            post[3 * wv + 0] = a;
            post[3 * wv + 1] = r;
            post[3 * wv + 2] = c;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            for (uint32_t i = 1; i < (uint32_t)kStatsWaves; ++i) {
                a += post[3 * i + 0];
                r += post[3 * i + 1];
                c += post[3 * i + 2];
            }
            means[0] = a / (double)n;
            means[1] = c > 0.0 ? r / c : 0.0;
        }
    }
}

// The statistics of an array that is one block, with scratch memory: workgroup w stores its four numbers to rows[4 w .. 4 w + 3] and
// k_error_finish adds the rows in a fixed order.  k_error_stats<.., false> on one block ends in four atomics and a count from each
// of 512 workgroups, all on one cache line and at the same time, and needs them zeroed before.  The block's scale and reciprocal
// are the same for all units; only the quads with a value next to a threshold are looked up again with true divisions (here
// all sixteen values of a lane were, in one unit of seven).
// FROM_PARTS: the scale is the largest of the n_parts maxima at `parts` and the first workgroup stores it; otherwise *scale.
// WAVES: 12 with two workgroups per compute unit, or 4 where the array is no more than a unit for four wavefronts of every
// compute unit: then the units spread over more of them.  What bounds it is the vector units, see k_error_stats.
// Device time in a graph, k_error_stats and now (with the passes before and after): 25 M elements 57.2 / 46.0 us, of these
// 39 / 27 the statistics; 1 M 16.5 / 10.2; 100 000 14.3 / 8.9; given scale 25 M 40.8 / 28.9.
// n_units whole units, strided over the grid.
template <int WAVES, bool FROM_PARTS>
__global__ __launch_bounds__(kWave *WAVES, WAVES / 2) void k_error_stats_one(const uint32_t *__restrict__ tab, const float *__restrict__ x,
                                                                             size_t n, size_t n_units, size_t n_waves,
                                                                             float *__restrict__ scale, const float *__restrict__ parts,
                                                                             uint32_t n_parts, double *__restrict__ rows)
{
    constexpr int Q = 4, U = Q * 4 * kWave;
    __shared__ __align__(256) float lut[256 * kLutCopies];
    extern __shared__ uint32_t bucket_lds[];
    const uint32_t lane = threadIdx.x & 63, lane4 = lane * 4;
    const float lut_value = request_magnitude_lut(tab);
    const BucketWords<kWave * WAVES> words = request_bucket_table<kWave * WAVES>(tab);
    constexpr int H = 2;  // quads worked on at a time
    v4f v[Q / H][H];
    auto fetch = [&](size_t u, int h) {
#pragma unroll
        for (int j = 0; j < H; ++j) v[h][j] = ldg_floats<1>(x + u * (size_t)U, 4 * ((h * H + j) * kWave + lane));
    };
    const size_t u0 = first_unit(WAVES);
    if (u0 < n_units) {
#pragma unroll
        for (int h = 0; h < Q / H; ++h) fetch(u0, h);
    }
    const float s = FROM_PARTS ? u2f(max_of_parts(parts, n_parts, lane)) : *scale;
    if (FROM_PARTS && blockIdx.x == 0 && threadIdx.x == 0) *scale = s;
    place_lut<kWave * WAVES>(lut_value * __builtin_fabsf(s), lut);  // one scale: the products are formed once per code
    const Search sr = place_bucket_table(tab, words, bucket_lds);
    __syncthreads();
    const float d = s == 0.0f ? 1.0f : s;
    const float r = 1.0f / d;
    const bool recip = reciprocal_ok(d);

    double sum_abs = 0.0, sum_rel = 0.0, worst = 0.0;
    uint64_t count = 0;  // wave-uniform
    auto add = [&](float xv, float qmag) {  // xv not zero
        const double ax = (double)__builtin_fabsf(xv);
        const double e = __builtin_fabs((double)qmag - ax);
        sum_abs += e;
        worst = __builtin_fmax(worst, e);
        sum_rel += quotient_of_magnitudes(e, ax);
    };
    // A zero has an error (a type need not have the value 0) but no relative one: the error is added here, and the pair becomes
    // one that adds nothing.  Whether it was one.
    auto take_zero = [&](float &xv, float &qmag) {
        const bool z = xv == 0.0f;
        const double e = z ? (double)qmag : 0.0;
        sum_abs += e;
        worst = __builtin_fmax(worst, e);
        xv = z ? 1.0f : xv;
        qmag = z ? 1.0f : qmag;
        return z;
    };
    // byte 1 of the address = byte 2 of the sum (the code field), byte 0 = lane * 4
    auto magnitude = [&](uint32_t sm) {
        const uint32_t addr = __builtin_amdgcn_perm(sm, lane4, 0x0C0C0600u);
        return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(lut) + addr);
    };
    auto work = [&](const v4f (&v)[H]) {
        float xs[H][4], qm[H][4], least = u2f(0x7F800000u);
        uint32_t sum[H][4], key[H], all = 0xFFFFu;
#pragma unroll
        for (int j = 0; j < H; ++j) {
            xs[j][0] = v[j].x;
            xs[j][1] = v[j].y;
            xs[j][2] = v[j].z;
            xs[j][3] = v[j].w;
#pragma unroll
            for (int c = 0; c < 4; ++c) sum[j][c] = search_sum(sr, xs[j][c] * r);
        }
#pragma unroll
        for (int j = 0; j < H; ++j) {
            const uint32_t k01 = near_key(sum[j][0]) < near_key(sum[j][1]) ? near_key(sum[j][0]) : near_key(sum[j][1]);
            const uint32_t k23 = near_key(sum[j][2]) < near_key(sum[j][3]) ? near_key(sum[j][2]) : near_key(sum[j][3]);
            key[j] = recip ? (k01 < k23 ? k01 : k23) : 0;
            all = all < key[j] ? all : key[j];
        }
        if (__builtin_amdgcn_ballot_w64(all <= 2 * kNearWindow) != 0) {
#pragma unroll
            for (int j = 0; j < H; ++j)
                if (__builtin_amdgcn_ballot_w64(key[j] <= 2 * kNearWindow) != 0) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) sum[j][c] = search_sum_exact(sr, xs[j][c] / d);
                }
        }
#pragma unroll
        for (int j = 0; j < H; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) {  // all lookups first, so that their latencies overlap
                qm[j][c] = magnitude(sum[j][c]);
                least = __builtin_fminf(least, __builtin_fabsf(xs[j][c]));
            }
        count += (uint64_t)(H * 4 * kWave);
        if (__builtin_amdgcn_ballot_w64(least == 0.0f) != 0) {
#pragma unroll
            for (int j = 0; j < H; ++j)
#pragma unroll
                for (int c = 0; c < 4; ++c) count -= (uint64_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(take_zero(xs[j][c], qm[j][c])));
        }
#pragma unroll
        for (int j = 0; j < H; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) add(xs[j][c], qm[j][c]);
    };
    // One set of registers, two quads requested again as soon as they are done with (from the last unit a second time, where there
    // is no next one): two sets and four quads at a time need more registers than six wavefronts per SIMD have.
    for (size_t u = u0; u < n_units; u += n_waves) {
        const size_t next = u + n_waves < n_units ? u + n_waves : u;
#pragma unroll
        for (int h = 0; h < Q / H; ++h) {
            work(v[h]);
            fetch(next, h);
        }
    }
    // the elements past the units, 64 per wavefront, from the wavefront after the last unit's on
    for (size_t i0 = n_units * (size_t)U + (u0 + n_waves - n_units % n_waves) % n_waves * kWave; i0 < n; i0 += n_waves * kWave) {
        const bool in = i0 + lane < n;
        float xv = in ? x[i0 + lane] : 0.0f;
        float q = in ? magnitude(search_sum_exact(sr, xv / d)) : 0.0f;  // a lane past the end: a zero without an error
        count += (uint64_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(!take_zero(xv, q)));
        add(xv, q);
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        sum_abs += __shfl_xor(sum_abs, m);
        sum_rel += __shfl_xor(sum_rel, m);
        worst = __builtin_fmax(worst, __shfl_xor(worst, m));
    }
    __syncthreads();  // the value table is not needed any more
    double *post = reinterpret_cast<double *>(lut);
    if (lane == 0) {
        double *p = post + 4 * wave_in_wg();
        p[0] = sum_abs;
        p[1] = sum_rel;
        p[2] = (double)count;
        p[3] = worst;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        double v = post[threadIdx.x];
        for (int w = 1; w < WAVES; ++w) {
            const double o = post[4 * w + threadIdx.x];
            v = threadIdx.x == 3 ? __builtin_fmax(v, o) : v + o;
        }
        rows[4 * (size_t)blockIdx.x + threadIdx.x] = v;
    }
}

// The rows of k_error_stats_one to the statistics of the block and, where means is not NULL, its means.  One workgroup; wavefront c
// takes number c of all rows, lane l rows l, l + 64, ..., and the lanes' results are combined by a fixed tree: the same sums in
// every launch.
constexpr uint32_t kFinishThreads = 4 * kWave;
__global__ __launch_bounds__(kFinishThreads) void k_error_finish(const double *__restrict__ rows, uint32_t n_rows, size_t n,
                                                                double *__restrict__ stats, double *__restrict__ means)
{
    __shared__ double all[4];
    const uint32_t lane = threadIdx.x & 63, c = wave_in_wg();
    double v = 0.0;
#pragma unroll 8
    for (uint32_t i = lane; i < n_rows; i += kWave) {
        const double o = rows[4 * i + c];
        v = c == 3 ? __builtin_fmax(v, o) : v + o;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
        const double o = __shfl_xor(v, m);
        v = c == 3 ? __builtin_fmax(v, o) : v + o;
    }
    if (lane == 0) {
        stats[c] = v;
        all[c] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0 && means) {
        means[0] = all[0] / (double)n;
        means[1] = all[2] > 0.0 ? all[1] / all[2] : 0.0;
    }
}

// Means over all blocks from the per-block statistics: means[0] = (sum of absolute errors) / n,
// means[1] = (sum of relative errors) / (number of non-zero inputs), 0 when there is none.
// After the statistics kernel in which wavefronts own whole blocks (that one needs no zeroed memory, and a count of its
// workgroups would) and after the other one where there are many blocks.  One workgroup of 1024 threads; thread t adds
// blocks t, t + 1024, ... in that order and the threads' sums are combined by a fixed tree, so the result is the same
// in every launch.
constexpr uint32_t kMeansThreads = 1024;
__global__ __launch_bounds__(kMeansThreads) void k_error_means(const double *__restrict__ stats, size_t nb, size_t n,
                                                              double *__restrict__ means)
{
    __shared__ double part[3][kMeansThreads];
    double a = 0.0, r = 0.0, c = 0.0;
#pragma unroll 4
    for (size_t b = threadIdx.x; b < nb; b += kMeansThreads) {
        a += stats[4 * b];
        r += stats[4 * b + 1];
        c += stats[4 * b + 2];
    }
    part[0][threadIdx.x] = a;
    part[1][threadIdx.x] = r;
    part[2][threadIdx.x] = c;
    __syncthreads();
    for (uint32_t w = kMeansThreads / 2; w >= 1; w >>= 1) {
        if (threadIdx.x < w) {
            part[0][threadIdx.x] += part[0][threadIdx.x + w];
            part[1][threadIdx.x] += part[1][threadIdx.x + w];
            part[2][threadIdx.x] += part[2][threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        means[0] = part[0][0] / (double)n;
        means[1] = part[2][0] > 0.0 ? part[1][0] / part[2][0] : 0.0;
    }
}

}  // namespace
