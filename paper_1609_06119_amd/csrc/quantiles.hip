// Equal-frequency bin boundaries on the device (section 2.2): boundary k of
// feature j is the value of rank floor(k m / B) among the feature's m
// non-NaN values (NaN values are missing, section 4.2).
//
// The ranks are found without sorting, by counting digits of the values'
// order-preserving 32-bit images, 16 + 8 + 8 bits from the top.  The first
// count fills one counter per 16-bit prefix; the counters place every rank
// in one prefix, at most 255 "active" ones.  The second count takes the
// values with an active prefix and counts their next 8 bits, 256 counters
// per active prefix; the third does the same one digit further, after which
// every rank's value is known bit for bit.  Each count reads the values
// once (4 bytes a value) and keeps its 65,536 counters of 16 bits in the
// LDS of one 1024-thread workgroup per CU, so the boundaries cost three
// reads of the sample; a radix sort of 64-bit keys reads and writes 8 bytes
// a value in each of its passes.  2M x 40 normal values: 2700 us with a sort
// (17 us of rank picks with it), now 112, 119 and 132 us for the counts (2.4 to
// 2.9 TB/s; 62 MB of counters written among them) and 33 us for the picks.
#include "fbdt_internal.h"

#include <hip/hip_runtime.h>

#include <algorithm>

namespace fbdt {
namespace {

constexpr int kQThreads = 1024;
constexpr int kQWave = 64;
constexpr int kQWaves = kQThreads / kQWave;
constexpr int kQSlots = 65536;                  // counters of a count
constexpr int kQWords = kQSlots / 2;            // two 16-bit counters per LDS word
constexpr int kQTab = kQSlots / 32;             // words of a bitmap over the slots
constexpr int kQActive = 255;                   // active prefixes at most (one per rank)
constexpr int kQGroups = 256;                   // groups of 256 counters
constexpr int kQGroupRow = 260;                 // group sums of a workgroup (padded)
constexpr int kQBatch = 4;                      // 4-value vectors per thread and batch
constexpr int kQCommon = 6;                     // crowded slots counted by comparing
// Values between two sweeps: a counter below 2^15 after a sweep cannot pass
// 2^16 - 1 before the next one.
constexpr int64_t kQSweep = 32768;
// Values a workgroup may count without a sweep (16-bit counters).
constexpr int64_t kQNoSweep = 65280;
// Values up to which one workgroup per feature does everything: above, the
// six launches of the shared counts get closer.  Time in one workgroup per
// feature over the time shared, over 1 to 255 features of normal values and of
// five levels: 0.53 to 0.81 at 20,000 values, 0.56 to 1.00 at 32,000, 0.58 to
// 1.00 at 40,000, 0.61 to 1.10 at 50,000, 0.62 to 1.17 at 60,000 (the larger
// ones for few features of few levels).
constexpr int64_t kQSmall = 40960;
static_assert(kQSmall <= kQNoSweep, "the one-workgroup path does not sweep");
static_assert(kQSweep == (int64_t)2 * kQBatch * 4 * kQThreads, "two batches between sweeps");

// Order-preserving image of a non-NaN float: unsigned order of the image =
// numeric order of the floats (-0 sorts just below +0).
__device__ __forceinline__ uint32_t order_key(uint32_t b) {
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

__device__ __forceinline__ uint32_t order_key_inverse(uint32_t k) {
    return (k & 0x80000000u) ? (k & 0x7fffffffu) : ~k;
}

constexpr uint32_t kInfKey = 0xff800000u;   // the image of +inf
constexpr uint32_t kNanSlot = 0xffffu;      // prefix of the NaN image, above every number's

// The image of a value, all ones for every NaN (of either sign).
__device__ __forceinline__ uint32_t value_key(uint32_t b) {
    return (b & 0x7fffffffu) > 0x7f800000u ? 0xffffffffu : order_key(b);
}

// A bitmap over slots with the number of set bits below each word: the
// rank of an active slot among the active ones is one 8-byte LDS read.
struct SlotSet {
    uint2 *w;   // {bits, set bits below} [kQTab]
    __device__ __forceinline__ bool find(uint32_t slot, uint32_t &rank) const {
        const uint2 e = w[slot >> 5];
        const uint32_t bit = slot & 31u;
        rank = e.y + __popc(e.x & ((1u << bit) - 1u));
        return (e.x >> bit) & 1u;
    }
};

// Builds the set of the slots of the first nb threads (slot < kQSlots);
// returns the number of distinct ones.  Called by the whole workgroup.
__device__ __forceinline__ uint32_t build_set(const SlotSet &s, uint32_t slot, int nb, uint32_t *s_wave) {
    const int t = threadIdx.x, lane = t % kQWave, wave = t / kQWave;
    for (int q = t; q < kQTab; q += kQThreads) s.w[q] = make_uint2(0u, 0u);
    __syncthreads();
    if (t < nb) atomicOr(&s.w[slot >> 5].x, 1u << (slot & 31u));
    __syncthreads();
    const uint32_t p0 = __popc(s.w[2 * t].x), p1 = __popc(s.w[2 * t + 1].x);
    uint32_t x = p0 + p1;
    for (int o = 1; o < kQWave; o <<= 1) {
        const uint32_t y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (lane == kQWave - 1) s_wave[wave] = x;
    __syncthreads();
    uint32_t base = 0u, all = 0u;
    for (int w = 0; w < kQWaves; ++w) {
        if (w < wave) base += s_wave[w];
        all += s_wave[w];
    }
    s.w[2 * t].y = base + x - p0 - p1;
    s.w[2 * t + 1].y = base + x - p1;
    __syncthreads();
    return all;
}

// Four consecutive values, read at the alignment of a float (rows may start
// at any element).
typedef float float4_unaligned __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ void load_batch(uint32_t (&v)[kQBatch][4], const float *row,
                                           int64_t base) {
#pragma unroll
    for (int u = 0; u < kQBatch; ++u) {
        const float4_unaligned f = *reinterpret_cast<const float4_unaligned *>(
            row + base + ((int64_t)u * kQThreads + threadIdx.x) * 4);
        v[u][0] = __float_as_uint(f.x);
        v[u][1] = __float_as_uint(f.y);
        v[u][2] = __float_as_uint(f.z);
        v[u][3] = __float_as_uint(f.w);
    }
}

// Slot of a value at digit LEVEL (1, 2, 3); false: counted nowhere.
template <int LEVEL>
__device__ __forceinline__ bool value_slot(uint32_t bits, const SlotSet &s1, const SlotSet &s2,
                                           uint32_t &slot) {
    const uint32_t key = value_key(bits);
    if (LEVEL == 1) {
        slot = key >> 16;
        return true;
    }
    uint32_t a;
    bool hit = s1.find(key >> 16, a);
    slot = (a << 8 | ((key >> 8) & 0xffu)) & (kQSlots - 1);
    if (LEVEL == 3 && hit) {
        uint32_t a2;
        hit = s2.find(slot, a2);
        slot = (a2 << 8 | (key & 0xffu)) & (kQSlots - 1);
    }
    return hit;
}

// Lane `from`'s value (from uniform over the wavefront).
__device__ __forceinline__ uint32_t lane_value(uint32_t v, int from) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, from);
}

__device__ __forceinline__ void count_slot(uint32_t *cnt, uint32_t slot, uint32_t times) {
    atomicAdd(&cnt[slot >> 1], times << ((slot & 1u) * 16u));
}

// Counts a batch whose values mostly fall in the NQ slots `common` (uniform
// over the wavefront; ~0: none): those are counted by comparing, on the
// scalar unit, and added once, the others as usual.
template <int LEVEL, int NQ>
__device__ __forceinline__ void count_common(const uint32_t (&v)[kQBatch][4], const SlotSet &s1,
                                             const SlotSet &s2, uint32_t *cnt,
                                             const uint32_t (&common)[kQCommon]) {
    const int lane = threadIdx.x % kQWave;
    uint32_t c[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) c[q] = 0u;
#pragma unroll
    for (int u = 0; u < kQBatch; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t slot;
            const bool hit = value_slot<LEVEL>(v[u][e], s1, s2, slot);
            if (!hit) slot = ~1u;
            uint32_t left = (uint32_t)__popcll(__ballot(hit));
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const uint32_t k = (uint32_t)__popcll(__ballot(slot == common[q]));
                c[q] += k;
                left -= k;
            }
            if (left) {   // (uniform) some value in none of them
                bool other = hit;
#pragma unroll
                for (int q = 0; q < NQ; ++q) other &= slot != common[q];
                if (other) count_slot(cnt, slot, 1u);
            }
        }
#pragma unroll
    for (int q = 0; q < NQ; ++q)
        if (lane == q && c[q]) count_slot(cnt, common[q], c[q]);
}

// Counts a batch in registers.  Values of few distinct codes put many lanes
// of a wavefront on one counter, whose LDS atomic then takes about 8 clocks
// per lane: where one of the first slots of the batch's first value holds 11
// lanes or more, those of them with 4 or more go to count_common (comparing
// costs about 6 clocks per slot, whatever its lanes).
template <int LEVEL>
__device__ __forceinline__ void count_batch(const uint32_t (&v)[kQBatch][4], const SlotSet &s1,
                                            const SlotSet &s2, uint32_t *cnt) {
    uint32_t common[kQCommon];
    int nq = 0, most = 0;
    {
        uint32_t slot;
        const bool hit = value_slot<LEVEL>(v[0][0], s1, s2, slot);
        uint64_t left = __ballot(hit);
#pragma unroll
        for (int q = 0; q < kQCommon; ++q) {
            common[q] = ~0u;
            if (left && (q == 0 || most >= 3)) {
                const uint32_t s = lane_value(slot, __ffsll((unsigned long long)left) - 1);
                const uint64_t same = __ballot(hit && slot == s);
                const int many = __popcll(same);
                left &= ~same;
                most = max(most, many);
                if (many >= 4) {
                    common[q] = s;
                    nq = q + 1;
                }
            }
        }
    }
    if (most < 11) {
#pragma unroll
        for (int u = 0; u < kQBatch; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint32_t slot;
                if (value_slot<LEVEL>(v[u][e], s1, s2, slot)) count_slot(cnt, slot, 1u);
            }
    } else if (nq <= 3) {
        count_common<LEVEL, 3>(v, s1, s2, cnt, common);
    } else {
        count_common<LEVEL, kQCommon>(v, s1, s2, cnt, common);
    }
}

// The counters of 2^15 or more move to the workgroup's 32-bit counters
// `wide` (thread and counters as where the workgroup writes them out).
template <int LEVEL>
__device__ __forceinline__ void sweep(uint32_t *cnt, uint32_t *wide) {
    const int lane = threadIdx.x % kQWave, wave = threadIdx.x / kQWave;
    constexpr int kAll = LEVEL == 1 ? kQGroups : kQActive;
    constexpr int kAtOnce = 8;
    for (int g0 = wave; g0 < kAll; g0 += kAtOnce * kQWaves) {
        uint2 v[kAtOnce];
#pragma unroll
        for (int u = 0; u < kAtOnce; ++u) {
            const int g = min(g0 + u * kQWaves, kAll - 1);
            v[u] = *reinterpret_cast<const uint2 *>(cnt + g * 128 + 2 * lane);
        }
#pragma unroll
        for (int u = 0; u < kAtOnce; ++u) {
            const int g = g0 + u * kQWaves;
            if (g < kAll && ((v[u].x | v[u].y) & 0x80008000u)) {
                uint4 *o = reinterpret_cast<uint4 *>(wide + g * 256 + 4 * lane);
                uint4 s = *o;
                s.x += v[u].x & 0xffffu;
                s.y += v[u].x >> 16;
                s.z += v[u].y & 0xffffu;
                s.w += v[u].y >> 16;
                *o = s;
                *reinterpret_cast<uint2 *>(cnt + g * 128 + 2 * lane) = make_uint2(0u, 0u);
            }
        }
    }
}

// Workgroup barrier that orders LDS only: loads in flight stay in flight.
__device__ __forceinline__ void lds_barrier() {
    __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Counts the values [lo, hi) of a row into cnt (16-bit counters, cleared
// by the caller).  Two batches are in flight by turns, also across the
// sweeps: a workgroup that counts more than kQNoSweep values sweeps its
// counters every kQSweep values.  (With one batch loaded while the other is
// counted, and all of it awaited before a sweep, 10M x 40 values ran at 2.9
// TB/s.)
template <int LEVEL>
__device__ __forceinline__ void count_values(const float *row, int64_t lo, int64_t hi,
                                             const SlotSet &s1, const SlotSet &s2, uint32_t *cnt,
                                             uint32_t *wide) {
    constexpr int64_t kStep = (int64_t)kQBatch * 4 * kQThreads;   // values of a batch
    const bool sweeps = hi - lo > kQNoSweep;
    const int64_t whole = lo + (hi - lo) / kStep * kStep;   // end of the whole batches
    if (whole > lo) {
        uint32_t a[kQBatch][4], b[kQBatch][4];
        load_batch(a, row, lo);
        for (int64_t base = lo;;) {
            // (the last loads repeat a batch: the waits for the others stay exact)
            const bool more_b = base + kStep < whole;
            load_batch(b, row, more_b ? base + kStep : base);
            count_batch<LEVEL>(a, s1, s2, cnt);
            if (!more_b) break;
            base += 2 * kStep;
            const bool more_a = base < whole;
            load_batch(a, row, more_a ? base : base - kStep);
            count_batch<LEVEL>(b, s1, s2, cnt);
            if (sweeps) {
                lds_barrier();
                sweep<LEVEL>(cnt, wide);
                lds_barrier();
            }
            if (!more_a) break;
        }
    }
    // the last, partial batch (less than a sweep's values since the last one
    // together with a last whole batch), 4 values' loads at a time
    for (int64_t i0 = whole + threadIdx.x; i0 < hi; i0 += 4 * kQThreads) {
        uint32_t v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            v[e] = __float_as_uint(row[min(i0 + (int64_t)e * kQThreads, hi - 1)]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            uint32_t slot;
            if (i0 + (int64_t)e * kQThreads < hi && value_slot<LEVEL>(v[e], s1, s2, slot))
                count_slot(cnt, slot, 1u);
        }
    }
}

// The wavefront's 256 counters, c[e] = counter 4 lane + e: index of the one
// that holds the value of rank r among them (255 if there is none), r
// reduced to the rank within it.
__device__ __forceinline__ uint32_t wave_find(const uint64_t (&c)[4], uint64_t &r) {
    const uint64_t sum = c[0] + c[1] + c[2] + c[3];
    uint64_t below[4];   // counts below each of the lane's counters
    below[0] = wave_inclusive_scan_u64(sum) - sum;
#pragma unroll
    for (int e = 1; e < 4; ++e) below[e] = below[e - 1] + c[e - 1];
    uint32_t at = 0u;    // counters whose inclusive sum is <= r: they rise with the counter
#pragma unroll
    for (int e = 0; e < 4; ++e) at += (uint32_t)__popcll(__ballot(below[e] + c[e] <= r));
    at = min(at, 255u);
    const uint32_t e = at & 3u;
    const uint64_t b = e == 0u ? below[0] : e == 1u ? below[1] : e == 2u ? below[2] : below[3];
    const int from = (int)(at >> 2);
    r -= (uint64_t)lane_value((uint32_t)b, from) |
         (uint64_t)lane_value((uint32_t)(b >> 32), from) << 32;
    return at;
}

// Inclusive prefix of the 256 group sums, by wavefront 0; s_incl[256].
__device__ __forceinline__ void scan_groups(const uint64_t *s_group, uint64_t *s_incl) {
    if (threadIdx.x < kQWave) {
        uint64_t c[4], run = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            c[e] = s_group[4 * threadIdx.x + e];
            run += c[e];
        }
        uint64_t x = wave_inclusive_scan_u64(run) - run;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x += c[e];
            s_incl[4 * threadIdx.x + e] = x;
        }
    }
}

// Group of 256 prefixes that holds rank r (255 if none), r reduced to the
// rank within it.  Called by a wavefront.
__device__ __forceinline__ uint32_t find_group(const uint64_t *s_incl, uint64_t &r) {
    const int lane = threadIdx.x % kQWave;
    uint32_t g = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) g += (uint32_t)__popcll(__ballot(s_incl[e * kQWave + lane] <= r));
    if (g > 0u) r -= s_incl[min(g, 255u) - 1u];
    return min(g, 255u);
}

// Rank of the k-th boundary (k from 0) among m values.
__device__ __forceinline__ uint64_t boundary_rank(int k, uint64_t m, int n_bins) {
    return (uint64_t)(k + 1) * m / (uint64_t)n_bins;
}

// Number of distinct prefixes (key >> shift) among keys[0, k], less one: the
// keys rise with k.  Every thread of the workgroup calls it; s_act[256].
__device__ __forceinline__ void active_index(const uint32_t *keys, int nb, int shift, uint8_t *s_act,
                             uint32_t *s_wave) {
    const int t = threadIdx.x, lane = t % kQWave, wave = t / kQWave;
    bool first = false;
    if (t > 0 && t < nb) first = (keys[t] >> shift) != (keys[t - 1] >> shift);
    const uint64_t m = __ballot(first);
    if (lane == 0) s_wave[wave] = (uint32_t)__popcll(m);
    __syncthreads();
    if (t < nb) {
        uint32_t a = (uint32_t)__popcll(m & ((2ull << lane) - 1ull));
        for (int w = 0; w < wave; ++w) a += s_wave[w];
        s_act[t] = (uint8_t)a;
    }
    __syncthreads();
}

// LDS of a count: the sets of the levels above, then the counters.
__host__ __device__ constexpr size_t rank_lds(int level) {
    return level == 1 ? (size_t)kQWords * 4
                      : (size_t)(level - 1) * kQTab * 8 + (size_t)kQActive * 256 * 2;
}

// The sets of the active prefixes of the levels above LEVEL, from the keys
// found so far (`key`: thread t's is rank t's), at the start of lds; returns
// the distinct prefixes of the level above (the rows of 256 counters that
// this level fills).
template <int LEVEL>
__device__ __forceinline__ uint32_t build_sets(uint32_t *lds, SlotSet &s1, SlotSet &s2,
                                               uint32_t key, int nb, uint32_t *s_wave) {
    s1.w = reinterpret_cast<uint2 *>(lds);
    s2.w = s1.w + kQTab;
    if (LEVEL == 1) return kQGroups;
    uint32_t rows = build_set(s1, key >> 16, nb, s_wave);
    if (LEVEL == 3) {
        uint32_t a;
        s1.find(key >> 16, a);
        rows = build_set(s2, (a << 8 | ((key >> 8) & 0xffu)) & (kQSlots - 1), nb, s_wave);
    }
    return rows;
}

template <int LEVEL>
__device__ __forceinline__ uint32_t *counters(uint32_t *lds) {
    return lds + (LEVEL - 1) * kQTab * 2;
}

template <int LEVEL>
__device__ __forceinline__ void clear_counters(uint32_t *cnt) {
    uint4 *c4 = reinterpret_cast<uint4 *>(cnt);
    constexpr int kVec = (LEVEL == 1 ? kQWords : kQActive * 128) / 4;
    for (int q = threadIdx.x; q < kVec; q += kQThreads) c4[q] = make_uint4(0u, 0u, 0u, 0u);
}

// What a count leaves per workgroup, for the pick.
struct Counted {
    void *partial;      // [feature][chunk][65536] counters (the rows of 256 that the level
                        // fills): 32 bits each in counts that sweep, else 16
    uint32_t *groups;   // [feature][chunk][kQGroupRow]: level 1's sums of 256 counters, then
                        // the NaN values
};

// One count of digit LEVEL: workgroup (feature, chunk) = (blockIdx.x,
// blockIdx.y; features first, so that slow ones spread over the launch) counts
// the values [chunk per, (chunk + 1) per) of its feature.
template <int LEVEL>
__global__ __launch_bounds__(kQThreads) void rank_count_kernel(
    const float *__restrict__ x, int64_t ldx, int64_t n, int64_t per,
    const uint32_t *__restrict__ keys, int nb, Counted out) {
    extern __shared__ uint32_t lds[];
    __shared__ uint32_t s_wave[kQWaves];
    const int lane = threadIdx.x % kQWave, wave = threadIdx.x / kQWave;
    const int j = blockIdx.x;
    const size_t part = (size_t)j * gridDim.y + blockIdx.y;
    const int64_t lo = (int64_t)blockIdx.y * per, hi = min(n, lo + per);
    SlotSet s1, s2;
    const uint32_t key =
        LEVEL > 1 && (int)threadIdx.x < nb ? keys[(size_t)j * 256 + threadIdx.x] : 0u;
    const uint32_t rows = build_sets<LEVEL>(lds, s1, s2, key, nb, s_wave);
    uint32_t *cnt = counters<LEVEL>(lds);
    clear_counters<LEVEL>(cnt);
    const bool swept = per > kQNoSweep;   // (of every workgroup, also a shorter last one)
    uint32_t *wide = static_cast<uint32_t *>(out.partial) + part * kQSlots;
    uint2 *narrow = reinterpret_cast<uint2 *>(static_cast<uint16_t *>(out.partial) +
                                              part * kQSlots);
    if (swept)   // (the same thread sweeps and writes a counter)
        for (uint32_t g = wave; g < rows; g += kQWaves)
            *reinterpret_cast<uint4 *>(wide + g * 256 + 4 * lane) = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    count_values<LEVEL>(x + (int64_t)j * ldx, lo, hi, s1, s2, cnt, wide);
    __syncthreads();
    for (uint32_t g = wave; g < rows; g += kQWaves) {
        const uint2 v = *reinterpret_cast<const uint2 *>(cnt + g * 128 + 2 * lane);
        uint4 s = make_uint4(v.x & 0xffffu, v.x >> 16, v.y & 0xffffu, v.y >> 16);
        if (swept) {
            uint4 *o = reinterpret_cast<uint4 *>(wide + g * 256 + 4 * lane);
            const uint4 w = *o;
            s.x += w.x;
            s.y += w.y;
            s.z += w.z;
            s.w += w.w;
            *o = s;
        } else {
            narrow[g * 64 + lane] = v;
        }
        if (LEVEL == 1) {
            uint32_t t = s.x + s.y + s.z + s.w;
            for (int q = kQWave / 2; q > 0; q >>= 1) t += __shfl_xor(t, q);
            if (lane == 0) out.groups[part * kQGroupRow + g] = t;
            // the last counter: NaN
            if (g == kQGroups - 1 && lane == kQWave - 1)
                out.groups[part * kQGroupRow + kQGroups] = s.w;
        }
    }
}

constexpr int kPickThreads = 256;
constexpr int kPickBlocks = 32;   // workgroups that share a feature's ranks
static_assert(kPickThreads == kQGroups && kPickThreads > kQActive, "a thread per group and rank");

// The digits of LEVEL of every rank of a feature from the counts' partials
// (blockIdx.y = feature; the ranks are shared over the wavefronts of the
// gridDim.x workgroups): keys gain the digit, resid becomes the rank within
// the counter.  Level 1 starts from the ranks floor(k m / B), records m and
// flags NaN with 256 bins; level 3 writes the boundaries.
template <int LEVEL, bool WIDE>
__global__ __launch_bounds__(kPickThreads) void rank_pick_kernel(
    Counted in, int chunks, int64_t n, int n_bins, uint32_t *__restrict__ keys_out,
    const uint32_t *__restrict__ keys_in, uint64_t *__restrict__ resid,
    uint64_t *__restrict__ count, float *__restrict__ bounds, int *__restrict__ err) {
    __shared__ uint64_t s_group[kQGroups], s_incl[kQGroups];
    __shared__ uint64_t s_nan;
    __shared__ uint8_t s_act[256];
    __shared__ uint32_t s_wave[kPickThreads / kQWave];
    const int t = threadIdx.x, lane = t % kQWave, wave = t / kQWave;
    const int j = blockIdx.y, nb = n_bins - 1;
    const size_t part0 = (size_t)j * chunks;
    keys_out += (size_t)j * 256;
    keys_in += (size_t)j * 256;
    resid += (size_t)j * 256;
    if (LEVEL == 1) {
        uint64_t s = 0;
#pragma unroll 4
        for (int c = 0; c < chunks; ++c) s += in.groups[(part0 + c) * kQGroupRow + t];
        s_group[t] = s;
        if (wave == 0) {
            s = 0;
            for (int c = lane; c < chunks; c += kQWave)
                s += in.groups[(part0 + c) * kQGroupRow + kQGroups];
            for (int q = kQWave / 2; q > 0; q >>= 1) s += __shfl_xor((unsigned long long)s, q);
            if (lane == 0) s_nan = s;
        }
        __syncthreads();
        scan_groups(s_group, s_incl);
        __syncthreads();
    } else {
        active_index(keys_in, nb, LEVEL == 2 ? 16 : 8, s_act, s_wave);
    }
    const uint64_t m = LEVEL == 1 ? (uint64_t)n - s_nan : count[j];
    if (LEVEL == 1 && blockIdx.x == 0 && t == 0) {
        count[j] = m;
        // NaN is an error with 256 bins (no room for the missing code)
        if (s_nan && n_bins > kMissingCode) atomicOr(err, kErrNan);
    }
    for (int k = blockIdx.x * (kPickThreads / kQWave) + wave; k < nb;
         k += gridDim.x * (kPickThreads / kQWave)) {
        uint64_t r = LEVEL == 1 ? boundary_rank(k, m, n_bins) : resid[k];
        const uint32_t g = LEVEL == 1 ? find_group(s_incl, r) : s_act[k];
        uint64_t c[4] = {0, 0, 0, 0};
        if (WIDE) {
            const uint4 *row = reinterpret_cast<const uint4 *>(static_cast<const uint32_t *>(
                                   in.partial) + part0 * kQSlots) + g * 64 + lane;
#pragma unroll 4
            for (int p = 0; p < chunks; ++p) {
                const uint4 v = row[(size_t)p * (kQSlots / 4)];
                c[0] += v.x;
                c[1] += v.y;
                c[2] += v.z;
                c[3] += v.w;
            }
        } else {
            const uint2 *row = reinterpret_cast<const uint2 *>(static_cast<const uint16_t *>(
                                   in.partial) + part0 * kQSlots) + g * 64 + lane;
#pragma unroll 4
            for (int p = 0; p < chunks; ++p) {
                const uint2 v = row[(size_t)p * (kQSlots / 4)];
                c[0] += v.x & 0xffffu;
                c[1] += v.x >> 16;
                c[2] += v.y & 0xffffu;
                c[3] += v.y >> 16;
            }
        }
        const uint32_t digit = wave_find(c, r);
        if (lane == 0) {
            // a feature without a number keeps the image of +inf
            const uint32_t key = LEVEL == 1   ? (m ? (g << 8 | digit) << 16 : kInfKey)
                                 : LEVEL == 2 ? keys_in[k] | digit << 8
                                              : keys_in[k] | digit;
            if (LEVEL < 3) {
                keys_out[k] = key;
                resid[k] = r;
            } else {
                bounds[(size_t)j * nb + k] =
                    __uint_as_float(m ? order_key_inverse(key) : 0x7f800000u);
            }
        }
    }
}

// Samples of at most kQSmall values: one workgroup per feature counts and
// picks all three digits in its LDS.  The counters become prefix sums within
// their groups of 256 (they fit 16 bits), and thread k searches rank k's.
template <int LEVEL>
__device__ __forceinline__ void small_level(const float *row, int n, int n_bins, uint32_t *lds,
                                            uint32_t &key, uint32_t &rank, uint32_t &m,
                                            uint32_t *s_wave) {
    const int lane = threadIdx.x % kQWave, wave = threadIdx.x / kQWave, nb = n_bins - 1;
    SlotSet s1, s2;
    const uint32_t rows = build_sets<LEVEL>(lds, s1, s2, key, nb, s_wave);
    uint32_t *cnt = counters<LEVEL>(lds);
    uint32_t *s_incl = lds + kQWords;   // level 1: group sums, behind its counters
    clear_counters<LEVEL>(cnt);
    __syncthreads();
    count_values<LEVEL>(row, 0, n, s1, s2, cnt, nullptr);
    __syncthreads();
    if (LEVEL == 1) m = (uint32_t)n - (cnt[kNanSlot >> 1] >> 16);
    if (LEVEL == 1) __syncthreads();   // (read before the sums below replace it)
    for (uint32_t g = wave; g < rows; g += kQWaves) {
        uint2 *p = reinterpret_cast<uint2 *>(cnt + g * 128 + 2 * lane);
        const uint2 v = *p;
        const uint32_t c0 = v.x & 0xffffu, c1 = c0 + (v.x >> 16), c2 = c1 + (v.y & 0xffffu),
                       c3 = c2 + (v.y >> 16);
        uint32_t x = c3;
        for (int o = 1; o < kQWave; o <<= 1) {
            const uint32_t y = __shfl_up(x, o);
            if (lane >= o) x += y;
        }
        const uint32_t below = x - c3;
        *p = make_uint2((below + c0) | (below + c1) << 16, (below + c2) | x << 16);
        if (LEVEL == 1 && lane == kQWave - 1) s_incl[g] = x;
    }
    __syncthreads();
    if (LEVEL == 1) {
        if (wave == 0) {
            uint32_t c[4], run = 0u;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                run += s_incl[4 * lane + e];
                c[e] = run;
            }
            uint32_t x = run;
            for (int o = 1; o < kQWave; o <<= 1) {
                const uint32_t y = __shfl_up(x, o);
                if (lane >= o) x += y;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) s_incl[4 * lane + e] = x - run + c[e];
        }
        __syncthreads();
    }
    if ((int)threadIdx.x < nb) {
        uint32_t g = 0u;
        if (LEVEL == 1) {
            rank = (threadIdx.x + 1u) * m / (uint32_t)n_bins;   // < 2^24
            for (uint32_t step = 128; step > 0; step >>= 1)     // group sums <= rank
                if (s_incl[g + step - 1] <= rank) g += step;
            if (g > 0u) rank -= s_incl[g - 1];
        } else {
            s1.find(key >> 16, g);
            if (LEVEL == 3) s2.find((g << 8 | ((key >> 8) & 0xffu)) & (kQSlots - 1), g);
        }
        const uint16_t *pre = reinterpret_cast<const uint16_t *>(cnt) + g * 256;
        uint32_t digit = 0u;
        for (uint32_t step = 128; step > 0; step >>= 1)         // prefix sums <= rank
            if (pre[digit + step - 1] <= rank) digit += step;
        if (digit > 0u) rank -= pre[digit - 1];
        key = LEVEL == 1 ? (m ? (g << 8 | digit) << 16 : kInfKey)
                         : key | digit << (LEVEL == 2 ? 8 : 0);
    }
    __syncthreads();
}

__global__ __launch_bounds__(kQThreads) void rank_small_kernel(const float *__restrict__ x,
                                                               int64_t ldx, int n, int n_bins,
                                                               float *__restrict__ bounds,
                                                               int *__restrict__ err) {
    extern __shared__ uint32_t lds[];
    __shared__ uint32_t s_wave[kQWaves];
    const int j = blockIdx.x, nb = n_bins - 1;
    const float *row = x + (int64_t)j * ldx;
    uint32_t key = 0u, rank = 0u, m = 0u;
    small_level<1>(row, n, n_bins, lds, key, rank, m, s_wave);
    small_level<2>(row, n, n_bins, lds, key, rank, m, s_wave);
    small_level<3>(row, n, n_bins, lds, key, rank, m, s_wave);
    if ((int)threadIdx.x < nb)
        bounds[(size_t)j * nb + threadIdx.x] =
            __uint_as_float(m ? order_key_inverse(key) : 0x7f800000u);
    if (threadIdx.x == 0 && m != (uint32_t)n && n_bins > kMissingCode) atomicOr(err, kErrNan);
}

static_assert(rank_lds(3) >= (size_t)kQWords * 4 + kQGroups * 4, "group sums fit behind level 1");

}  // namespace

// Workgroups per feature, from the measured costs of a count: 0.33 us per
// 1000 values of a workgroup and 3 us of its own, once per round of one
// workgroup per CU; 0.03 us (0.06 us with sweeps) of the device per workgroup
// for the counters that it writes and as much for the pick that reads them; and
// at the end half the time of a workgroup's values again, the wait for the
// slowest (features with few distinct values take longer).
QuantileShape plan_quantiles(int64_t n, int d, int cu_count) {
    QuantileShape qs{};
    qs.small = n <= kQSmall;
    qs.chunks = 1;
    qs.per = n;
    if (!qs.small) {
        const int64_t most = std::min<int64_t>(256, (n + 4095) / 4096);
        double best = 0.0;
        for (int64_t c = 1; c <= most; ++c) {
            const int64_t per = ((n + c - 1) / c + 3) / 4 * 4;
            const double rounds = (double)((c * d + cu_count - 1) / cu_count);
            const double us = 3.3e-4 * (double)per;
            const double row = per > kQNoSweep ? 0.12 : 0.06;
            const double cost = rounds * (us + 3.0) + row * (double)(c * d) + us / 2;
            if (per > ((int64_t)1 << 31) && c < most) continue;   // 32-bit partial counters
            if (best == 0.0 || cost < best) {
                best = cost;
                qs.per = per;
                qs.chunks = (int)((n + per - 1) / per);
            }
        }
    }
    return qs;
}

// Scratch bytes of each part (256-byte multiples).
struct QuantileParts {
    size_t partial, groups, keys, resid, count;
};

static QuantileParts quantile_parts(const QuantileShape &qs, int d) {
    const auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t wgs = (size_t)d * qs.chunks;
    return {up(wgs * kQSlots * (qs.per > kQNoSweep ? 4 : 2)), up(wgs * kQGroupRow * 4),
            up((size_t)d * 256 * 4), up((size_t)d * 256 * 8), up((size_t)d * 8)};
}

size_t quantile_scratch_bytes(const QuantileShape &qs, int d) {
    if (qs.small) return 256;
    const QuantileParts p = quantile_parts(qs, d);
    return p.partial + p.groups + 2 * p.keys + p.resid + p.count;
}

hipError_t prepare_quantiles(size_t max_lds) {
    if (max_lds < rank_lds(3) + sizeof(uint32_t) * kQWaves) return hipErrorInvalidValue;
    const auto allow = [](const void *f, size_t bytes) {
        return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    };
    const hipError_t e[] = {
        allow(reinterpret_cast<const void *>(rank_count_kernel<1>), rank_lds(1)),
        allow(reinterpret_cast<const void *>(rank_count_kernel<2>), rank_lds(2)),
        allow(reinterpret_cast<const void *>(rank_count_kernel<3>), rank_lds(3)),
        allow(reinterpret_cast<const void *>(rank_small_kernel), rank_lds(3))};
    for (hipError_t x : e)
        if (x != hipSuccess) return x;
    return hipSuccess;
}

hipError_t launch_quantile_boundaries(const float *x, int64_t ldx, int64_t n, int d, int n_bins,
                                      const QuantileShape &qs, void *scratch, float *bounds,
                                      int *err, hipStream_t s) {
    const int nb = n_bins - 1;
    if (n < 1 || d < 1 || nb < 1 || nb > kQActive) return hipErrorInvalidValue;
    if (qs.small) {
        if (n > kQSmall) return hipErrorInvalidValue;
        rank_small_kernel<<<d, kQThreads, rank_lds(3), s>>>(x, ldx, (int)n, n_bins, bounds, err);
        return hipGetLastError();
    }
    if ((int64_t)qs.chunks * qs.per < n || (int64_t)(qs.chunks - 1) * qs.per >= n)
        return hipErrorInvalidValue;
    const QuantileParts p = quantile_parts(qs, d);
    char *at = static_cast<char *>(scratch);
    const auto take = [&](size_t bytes) {
        char *r = at;
        at += bytes;
        return r;
    };
    Counted c{};
    c.partial = take(p.partial);
    c.groups = reinterpret_cast<uint32_t *>(take(p.groups));
    uint32_t *k0 = reinterpret_cast<uint32_t *>(take(p.keys));
    uint32_t *k1 = reinterpret_cast<uint32_t *>(take(p.keys));
    uint64_t *resid = reinterpret_cast<uint64_t *>(take(p.resid));
    uint64_t *count = reinterpret_cast<uint64_t *>(take(p.count));
    const dim3 grid((unsigned)d, (unsigned)qs.chunks), pick(kPickBlocks, (unsigned)d);
    const bool wide = qs.per > kQNoSweep;
    // each level reads the keys of the one before it and writes its own
    // (the workgroups of a pick read all of a feature's keys)
#define FBDT_PICK(L, W, IN, OUT)                                                                \
    rank_pick_kernel<L, W><<<pick, kPickThreads, 0, s>>>(c, qs.chunks, n, n_bins, OUT, IN,      \
                                                         resid, count, bounds, err)
#define FBDT_RANK(L, IN, OUT)                                                                   \
    rank_count_kernel<L><<<grid, kQThreads, rank_lds(L), s>>>(x, ldx, n, qs.per, IN, nb, c);    \
    if (wide)                                                                                   \
        FBDT_PICK(L, true, IN, OUT);                                                            \
    else                                                                                        \
        FBDT_PICK(L, false, IN, OUT)
    FBDT_RANK(1, k1, k0);
    FBDT_RANK(2, k0, k1);
    FBDT_RANK(3, k1, k0);
#undef FBDT_RANK
#undef FBDT_PICK
    return hipGetLastError();
}

}  // namespace fbdt
