// Sorts of 64-bit keys (unique keys; the maximum key pads) used by the repair
// of the (tile, bin) segments: wavefront and workgroup bitonic networks, and a
// workgroup bucket sort.
#pragma once

#include "common.hpp"

namespace tgs {

// The value of lane l ^ m (m a power of two below 64, a constant after
// unrolling). Distances 1, 2, 4 and 8 stay inside a row of 16 lanes and use
// DPP moves (ALU, no LDS traffic): quad permutations for 1 and 2, a row
// rotation by 8 for 8, and for 4 a rotation by 4 or 12 chosen by lane bit 2.
// Larger distances use the LDS crossbar (ds_bpermute).
__device__ __forceinline__ uint32_t xor_lane_u32(uint32_t v, int m) {
    const int x = (int)v;
    switch (m) {
        case 1:
            return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true);  // quad_perm [1,0,3,2]
        case 2:
            return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true);  // quad_perm [2,3,0,1]
        case 4: {
            const int r4 = __builtin_amdgcn_mov_dpp(x, 0x124, 0xF, 0xF, true);   // row_ror:4
            const int r12 = __builtin_amdgcn_mov_dpp(x, 0x12C, 0xF, 0xF, true);  // row_ror:12
            return (uint32_t)((lane() & 4) ? r4 : r12);
        }
        case 8:
            return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x128, 0xF, 0xF, true);  // row_ror:8
        default:
            return shfl_xor_u32(v, m);
    }
}

__device__ __forceinline__ uint64_t xor_lane_u64(uint64_t v, int m) {
    const uint32_t lo = xor_lane_u32((uint32_t)v, m), hi = xor_lane_u32((uint32_t)(v >> 32), m);
    return ((uint64_t)hi << 32) | lo;
}

// Bitonic network over groups of G lanes, one key per lane (the partner at
// distance j < G is lane l ^ j, inside the group).
template <int G>
__device__ __forceinline__ uint64_t group_bitonic(uint64_t v, int li) {
#pragma unroll
    for (int k = 2; k <= G; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
            // the lower lane of an ascending pair keeps the smaller key, the
            // upper one the larger (descending: the reverse): keep the own
            // key exactly when (own < other) says the same
            const uint64_t o = xor_lane_u64(v, j);
            const bool keep_min = ((li & k) == 0) == ((li & j) == 0);
            v = ((v < o) == keep_min) ? v : o;
        }
    }
    return v;
}

// Segments of 65..512 keys: one wavefront, E = 2, 4 or 8 consecutive keys
// per lane in registers (key i = lane * E + k in register k, padded with
// the maximum key): bitonic network whose comparators at distance j < E
// stay inside a lane and at j >= E exchange register k with lane l ^ (j / E).
// REC: write the records of the sorted positions (rs.put).
template <int E, bool REC>
__device__ __forceinline__ void sort_wave_reg(uint64_t* __restrict__ seg, uint32_t s, uint32_t begin, uint32_t len,
                                              const RecordSink& rs) {
    const int l = lane();
    uint64_t v[E];
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const uint32_t i = (uint32_t)(l * E + k);
        v[k] = i < len ? seg[i] : ~0ull;
    }
#pragma unroll
    for (int kk = 2; kk <= E * kWave; kk <<= 1) {
#pragma unroll
        for (int j = kk >> 1; j > 0; j >>= 1) {
            if (j < E) {
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    if (k & j) continue;
                    const bool up = ((l * E + k) & kk) == 0;
                    const uint64_t a = v[k], b = v[k | j];
                    const bool sw = (a > b) == up;
                    v[k] = sw ? b : a;
                    v[k | j] = sw ? a : b;
                }
            } else {
                const int m = j / E;
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    const uint64_t o = xor_lane_u64(v[k], m);
                    const bool keep_min = (((l * E + k) & kk) == 0) == ((l & m) == 0);
                    v[k] = ((v[k] < o) == keep_min) ? v[k] : o;
                }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const uint32_t i = (uint32_t)(l * E + k);
        if (i < len) {
            seg[i] = v[k];
            if (REC) rs.put(s, begin + i, v[k]);
        }
    }
}

// LDS slot of key i in the workgroup networks below: one pad slot after
// every E keys, so that the E-key runs of consecutive threads start in
// different banks.
template <int E>
__device__ __forceinline__ uint32_t block_slot(uint32_t i) {
    return i + i / E;
}

// Segments of 513..8192 keys: one workgroup of NT threads, E consecutive
// keys per thread in registers (key i = t E + k in register k of thread t,
// padded with the maximum key; P = NT E keys): the bitonic network with the
// comparators at distance j < E inside a thread, E <= j < 64 E between the
// lanes of a wavefront (lane l ^ j / E), and j >= 64 E between wavefronts
// through LDS (lds: block_slot<E>(P) slots). Only the last log2(NT / 64)
// merge levels cross wavefronts, so the network takes 2 barriers per
// cross-wavefront step instead of one per step.
template <int E, int NT>
__device__ __forceinline__ void sort_block_reg(uint64_t (&v)[E], uint64_t* lds) {
    const int t = (int)threadIdx.x, l = lane();
    constexpr int P = NT * E;
#pragma unroll
    for (int kk = 2; kk <= P; kk <<= 1) {
#pragma unroll
        for (int j = kk >> 1; j > 0; j >>= 1) {
            if (j < E) {
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    if (k & j) continue;
                    const bool up = (((uint32_t)(t * E + k)) & (uint32_t)kk) == 0;
                    const uint64_t a = v[k], b = v[k | j];
                    const bool sw = (a > b) == up;
                    v[k] = sw ? b : a;
                    v[k | j] = sw ? a : b;
                }
            } else if (j < kWave * E) {
                const int m = j / E;
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    const uint64_t o = xor_lane_u64(v[k], m);
                    const bool keep_min = ((((uint32_t)(t * E + k)) & (uint32_t)kk) == 0) == ((l & m) == 0);
                    v[k] = ((v[k] < o) == keep_min) ? v[k] : o;
                }
            } else {
#pragma unroll
                for (int k = 0; k < E; ++k) lds[block_slot<E>((uint32_t)(t * E + k))] = v[k];
                __syncthreads();
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    const uint32_t i = (uint32_t)(t * E + k);
                    const uint64_t o = lds[block_slot<E>(i ^ (uint32_t)j)];
                    const bool keep_min = ((i & (uint32_t)kk) == 0) == ((i & (uint32_t)j) == 0);
                    v[k] = ((v[k] < o) == keep_min) ? v[k] : o;
                }
                __syncthreads();
            }
        }
    }
}

// ---- workgroup bucket sort -----------------------------------------------------
// n <= CAP keys in registers (key j NT + t in register j of thread t) are
// counting-sorted into kBucketSlots buckets in LDS; a key's place inside its
// bucket is its rank there. With the buckets spread over the keys' own range a
// bucket holds one or two keys, so this is one LDS atomic, one LDS write and a
// few LDS reads per key against the O(log^2) exchanges of the networks.
// Where the keys are clustered in their range (the first and the last bin hold
// the depths outside the percentiles) a rank takes as many LDS reads as the
// bucket has keys, and buckets of more than kBucketRank keys can be ordered by a
// wavefront's network each (sort_long_buckets).
constexpr int kBucketSlots = 4096;
constexpr int kBucketRank = 64;  // longest bucket ordered by rank

template <int NT, int CAP>
struct BucketLds {
    uint32_t off[kBucketSlots + 1];  // first slot of each bucket
    uint16_t bucket[CAP];            // bucket of each slot
    uint32_t sum[NT / kWave], lo[NT / kWave], hi[NT / kWave];
    uint64_t stage[CAP + 4];
};

// Buckets of the keys by (tile, upper word): the slots are divided evenly
// among the `tiles` tiles (b[j] holds the key's tile, 0 .. tiles - 1 <
// kBucketSlots, on entry), and within a tile spread by a monotone map over the
// range of all keys' upper words. Every register holds a key (repeated ones
// past the last). False when all upper words are equal.
template <int E, int NT, int CAP>
__device__ __forceinline__ bool range_buckets(const uint64_t (&key)[E], uint32_t (&b)[E], uint32_t tiles,
                                              BucketLds<NT, CAP>& L) {
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
    for (int j = 0; j < E; ++j) {
        lo = min(lo, (uint32_t)(key[j] >> 32));
        hi = max(hi, (uint32_t)(key[j] >> 32));
    }
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        lo = min(lo, xor_lane_u32(lo, m));
        hi = max(hi, xor_lane_u32(hi, m));
    }
    if (lane() == 0) {
        L.lo[threadIdx.x / kWave] = lo;
        L.hi[threadIdx.x / kWave] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NT / kWave; ++i) {
        lo = min(lo, L.lo[i]);
        hi = max(hi, L.hi[i]);
    }
    const uint32_t span = hi - lo, slots = kBucketSlots / tiles;
    // floor(2^32 slots / (span + 1)) without a 64-bit division; any smaller
    // value gives a monotone map too
    const uint32_t mul = span < slots ? 0u : (uint32_t)((float)slots * (4294967296.0f * 0.999999f) / ((float)span + 1.0f));
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const uint32_t d = (uint32_t)(key[j] >> 32) - lo;
        b[j] = b[j] * slots + (mul ? __umulhi(d, mul) : d);
    }
    return span != 0;
}

// Places the keys in L.stage by bucket (L.off, L.bucket follow; ends with a
// barrier) and returns 0, or 1 when some bucket has more than kBucketRank keys.
// With MOST > 0 and a bucket of more than that, nothing is placed and 2 is
// returned. L.off must not be in use by another wavefront when this is called.
template <uint32_t MOST, int E, int NT, int CAP>
__device__ __forceinline__ int place_buckets(const uint64_t (&key)[E], const uint32_t (&b)[E], uint32_t n,
                                             BucketLds<NT, CAP>& L) {
    constexpr int kPer = kBucketSlots / NT;
    for (int k = threadIdx.x; k < kBucketSlots; k += NT) L.off[k] = 0;
    __syncthreads();
    uint32_t rank[E];
#pragma unroll
    for (int j = 0; j < E; ++j)
        rank[j] = (uint32_t)(j * NT) + threadIdx.x < n ? atomicAdd(&L.off[b[j]], 1u) : 0u;
    __syncthreads();
    uint32_t c[kPer], s = 0, longest = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        c[j] = L.off[threadIdx.x * kPer + j];
        s += c[j];
        longest = max(longest, c[j]);
    }
    const uint32_t incl = wave_inclusive_sum(s);
    if (lane() == kWave - 1) L.sum[threadIdx.x / kWave] = incl;
    if (MOST == 0)
        __syncthreads();
    else if (__syncthreads_or(longest > MOST))
        return 2;
    uint32_t run = incl - s;
#pragma unroll
    for (int i = 0; i < NT / kWave; ++i) run += i < (int)(threadIdx.x / kWave) ? L.sum[i] : 0u;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        L.off[threadIdx.x * kPer + j] = run;
        run += c[j];
    }
    if (threadIdx.x == 0) L.off[kBucketSlots] = n;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < E; ++j) {
        if ((uint32_t)(j * NT) + threadIdx.x >= n) continue;
        const uint32_t q = L.off[b[j]] + rank[j];
        L.stage[q] = key[j];
        L.bucket[q] = (uint16_t)b[j];
    }
    return __syncthreads_or(longest > (uint32_t)kBucketRank) ? 1 : 0;
}

// Orders the buckets of more than kBucketRank keys, up to kBucketMost, in the
// stage; neighbouring buckets go to different wavefronts. Ends with a barrier.
template <int NT, int CAP>
__device__ __forceinline__ void sort_long_buckets(BucketLds<NT, CAP>& L) {
    constexpr int NW = NT / kWave;
    static_assert(kBucketMost <= 8 * kWave && kBucketSlots % NT == 0, "keys of a wavefront's network, whole rounds");
    const RecordSink none{};
    for (int k0 = 0; k0 < kBucketSlots; k0 += NT) {
        const int k = k0 + lane() * NW + (int)threadIdx.x / kWave;
        const uint32_t at = L.off[k], len = L.off[k + 1] - at;
        uint64_t todo = ballot(len > (uint32_t)kBucketRank && len <= (uint32_t)kBucketMost);
        while (todo) {
            const int src = __builtin_ctzll(todo);
            todo &= todo - 1;
            const uint32_t b = shfl_u32(at, src), n = shfl_u32(len, src);
            if (n <= 2 * kWave)
                sort_wave_reg<2, false>(L.stage + b, 0u, 0u, n, none);
            else if (n <= 4 * kWave)
                sort_wave_reg<4, false>(L.stage + b, 0u, 0u, n, none);
            else
                sort_wave_reg<8, false>(L.stage + b, 0u, 0u, n, none);
        }
    }
    __syncthreads();
}

// Place of the key v within its bucket [b, b + len) of the stage: its rank
// among the bucket's (unique) keys. Four keys are read at a time, so that
// their LDS latencies overlap (the stage has kRankPad slots past its end).
constexpr int kRankPad = 4;
__device__ __forceinline__ uint32_t rank_slot(const uint64_t* stage, uint64_t v, uint32_t b, uint32_t len) {
    uint32_t rank = 0;
    for (uint32_t k = 0; k < len; k += kRankPad) {
        uint64_t x[kRankPad];
#pragma unroll
        for (uint32_t i = 0; i < kRankPad; ++i) x[i] = stage[b + k + i];
#pragma unroll
        for (uint32_t i = 0; i < kRankPad; ++i) rank += (k + i < len && x[i] < v) ? 1u : 0u;
    }
    return b + rank;
}

}  // namespace tgs
