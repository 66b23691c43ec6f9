// Single-pass exclusive prefix sums with decoupled look-back: each workgroup
// takes a ticket (so every workgroup it waits on is already running),
// publishes its aggregate, adds the aggregates / inclusive prefixes of its
// predecessors (a status word per workgroup: 2 flag bits + 62 value bits,
// exchanged with agent-scope relaxed atomics), publishes its inclusive
// prefix and writes its outputs. Items are read in coalesced rounds of 256.
// Used for the per-Gaussian entry offsets (fused with the visible-Gaussian
// list), the per-tile segment bases, the rule-based repair selection and, on
// the per-entry atomic path, the (tile, bin) counts -> bin offsets (fused
// with the per-XCD bases and the repair-bucket classification). Also here:
// the group scan and the per-group counting sort of grouped binning.
#include <algorithm>

#include "common.hpp"
#include "wave_sort.hpp"

namespace tgs {

namespace {

constexpr int kThreads = 256;
constexpr int kRounds = 8;
constexpr int kPerBlock = kThreads * kRounds;
#ifndef TGS_EMIT_THREADS
#define TGS_EMIT_THREADS 1024
#endif
#ifndef TGS_EMIT_ROUNDS
#define TGS_EMIT_ROUNDS 4
#endif
constexpr int kEmitThreads = TGS_EMIT_THREADS;  // threads of an emit-scan workgroup
constexpr int kEmitRounds = TGS_EMIT_ROUNDS;    // items per thread of the emit scan
constexpr int kEmitPerBlock = kEmitThreads * kEmitRounds;
constexpr uint64_t kFlagAgg = 1ull << 62;
constexpr uint64_t kFlagInc = 2ull << 62;
constexpr uint64_t kValMask = (1ull << 62) - 1;

template <int NT = kThreads>
__device__ __forceinline__ uint32_t block_sum_u32(uint32_t v, uint32_t* lds) {
    constexpr int NW = NT / kWave;
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) v += shfl_xor_u32(v, m);
    if (lane() == 0) lds[threadIdx.x / kWave] = v;
    __syncthreads();
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) s += lds[i];
    __syncthreads();
    return s;
}

__device__ __forceinline__ uint64_t block_sum_u64(uint64_t v, uint64_t* lds) {
    constexpr int NW = kThreads / kWave;
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        const uint32_t lo = shfl_xor_u32((uint32_t)v, m), hi = shfl_xor_u32((uint32_t)(v >> 32), m);
        v += ((uint64_t)hi << 32) | lo;
    }
    if (lane() == 0) lds[threadIdx.x / kWave] = v;
    __syncthreads();
    uint64_t s = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) s += lds[i];
    __syncthreads();
    return s;
}

// Exclusive scan of one uint32 per thread across the workgroup; *total
// receives the sum. Ends with a barrier, so lds is reusable.
template <int NT = kThreads>
__device__ __forceinline__ uint32_t block_excl_u32(uint32_t v, uint32_t* lds, uint32_t* total) {
    constexpr int NW = NT / kWave;
    const int w = threadIdx.x / kWave, l = lane();
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t o = shfl_up_u32(inc, d);
        if (l >= d) inc += o;
    }
    if (l == kWave - 1) lds[w] = inc;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const uint32_t t = lds[i];
        before += i < w ? t : 0u;
        all += t;
    }
    __syncthreads();
    *total = all;
    return before + inc - v;
}

__device__ __forceinline__ uint64_t status_load(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void status_store(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t wave_sum_u64(uint64_t v) {
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
        const uint32_t lo = shfl_xor_u32((uint32_t)v, m), hi = shfl_xor_u32((uint32_t)(v >> 32), m);
        v += ((uint64_t)hi << 32) | lo;
    }
    return v;
}

// Sum of the values of workgroups 0..b-1, by one whole wavefront: each
// lane reads one status word of a window of 64 predecessors (nearest in lane
// 0) and waits until it is published; the window's values up to the nearest
// inclusive prefix are summed, else the whole window is added and the next
// window further back is read. Waits only on workgroups with a smaller
// ticket, which are running or done; workgroup 0 always publishes an
// inclusive prefix, and positions before it count as an inclusive zero.
__device__ uint64_t look_back(const uint64_t* status, int64_t b) {
    uint64_t prefix = 0;
    for (int64_t hi = b - 1;; hi -= kWave) {
        const int64_t p = hi - lane();
        uint64_t s = kFlagInc;
        if (p >= 0) {
            do {
                s = status_load(&status[p]);
            } while ((s >> 62) == 0);
        }
        const uint64_t inc = ballot((s & ~kValMask) == kFlagInc);
        const int stop = inc ? __builtin_ctzll(inc) : kWave - 1;
        prefix += wave_sum_u64(lane() <= stop ? (s & kValMask) : 0ull);
        if (inc) return prefix;
    }
}

// Called by every lane of one wavefront: publishes the aggregate, looks
// back and publishes the inclusive prefix; returns the exclusive prefix of
// workgroup b (in every lane).
__device__ __forceinline__ uint64_t publish_and_look_back(uint64_t* status, int64_t b, uint64_t agg) {
    if (b == 0) {
        if (lane() == 0) status_store(&status[0], kFlagInc | agg);
        return 0;
    }
    if (lane() == 0) status_store(&status[b], kFlagAgg | agg);
    const uint64_t prefix = look_back(status, b);
    if (lane() == 0) status_store(&status[b], kFlagInc | ((prefix + agg) & kValMask));
    return prefix;
}

// Exclusive scan of one uint64 per thread across the workgroup; *total
// receives the sum. Ends with a barrier, so lds is reusable.
template <int NT = kThreads>
__device__ __forceinline__ uint64_t block_excl_u64(uint64_t v, uint64_t* lds, uint64_t* total) {
    constexpr int NW = NT / kWave;
    const int w = threadIdx.x / kWave, l = lane();
    uint64_t inc = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t lo = shfl_up_u32((uint32_t)inc, d), hi = shfl_up_u32((uint32_t)(inc >> 32), d);
        if (l >= d) inc += ((uint64_t)hi << 32) | lo;
    }
    if (l == kWave - 1) lds[w] = inc;
    __syncthreads();
    uint64_t before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const uint64_t t = lds[i];
        before += i < w ? t : 0ull;
        all += t;
    }
    __syncthreads();
    *total = all;
    return before + inc - v;
}

// ---- entry-emission scan ---------------------------------------------------
// Per Gaussian: x = number of tiles (entries), y = 1 if visible. Writes
// emit_off[g] (exclusive prefix of x), vis_ids[rank] = g for visible g, and
// counters[0] = M, counters[1] = V, counters[2] = M > capacity. count_host
// (host memory the device can write, or null) = M.
// Items are loaded and stored in coalesced rounds; in between they pass
// through LDS so that each thread scans kEmitRounds consecutive items and one
// workgroup scan of the packed pair (x << 24 | y; y <= kEmitPerBlock) serves
// both prefixes.

__global__ void __launch_bounds__(kEmitThreads) emit_scan_kernel(const uint4* __restrict__ info, int64_t n, int tiles_x,
                                                             int tiles_y, uint32_t* __restrict__ emit_off,
                                                             uint32_t* __restrict__ vis_ids, uint32_t* ticket,
                                                             uint64_t* status_x, uint64_t* status_y,
                                                             int64_t* __restrict__ counters, int64_t capacity,
                                                             int64_t* count_host) {
    static_assert(kEmitRounds % 4 == 0 && kEmitPerBlock < (1 << 24), "packed pair layout");
    __shared__ uint32_t tk;
    __shared__ __align__(16) uint32_t item_x[kEmitPerBlock];  // tile counts, then exclusive x
    __shared__ __align__(16) uint32_t item_y[kEmitPerBlock];  // exclusive y | visible << 31
    __shared__ uint64_t lds64[kEmitThreads / kWave];
    __shared__ uint64_t pre[2];
    if (threadIdx.x == 0) tk = atomicAdd(ticket, 1u);
    __syncthreads();
    const int64_t b = tk;
    const int64_t nb = gridDim.x;
    const int64_t base = b * kEmitPerBlock;
#pragma unroll
    for (int r = 0; r < kEmitRounds; ++r) {
        const int64_t g = base + r * kEmitThreads + threadIdx.x;
        int x0, y0, x1, y1;
        item_x[r * kEmitThreads + threadIdx.x] = g < n ? (uint32_t)rect_of(info[g], tiles_x, tiles_y, x0, y0, x1, y1) : 0u;
    }
    __syncthreads();
    constexpr int kVec = kEmitRounds / 4;
    const uint4* own = reinterpret_cast<const uint4*>(item_x) + kVec * threadIdx.x;
    uint32_t c[kEmitRounds];
#pragma unroll
    for (int q = 0; q < kVec; ++q) {
        const uint4 cq = own[q];
        c[4 * q] = cq.x;
        c[4 * q + 1] = cq.y;
        c[4 * q + 2] = cq.z;
        c[4 * q + 3] = cq.w;
    }
    uint32_t ex[kEmitRounds], ey[kEmitRounds];
    uint64_t sx = 0;
    uint32_t sy = 0;
#pragma unroll
    for (int i = 0; i < kEmitRounds; ++i) {
        ex[i] = (uint32_t)sx;
        ey[i] = sy;
        sx += c[i];
        sy += c[i] ? 1u : 0u;
    }
    uint64_t tot;
    const uint64_t tex = block_excl_u64<kEmitThreads>((sx << 24) | sy, lds64, &tot);
    const uint64_t ax = tot >> 24;
    const uint32_t ay = (uint32_t)(tot & 0xFFFFFFu);
    const uint32_t tx0 = (uint32_t)(tex >> 24), ty0 = (uint32_t)(tex & 0xFFFFFFu);
    uint4* own_x = reinterpret_cast<uint4*>(item_x) + kVec * threadIdx.x;
    uint4* own_y = reinterpret_cast<uint4*>(item_y) + kVec * threadIdx.x;
    auto vy = [&](int i) { return (ty0 + ey[i]) | (c[i] ? 0x80000000u : 0u); };
#pragma unroll
    for (int q = 0; q < kVec; ++q) {
        own_x[q] = make_uint4(tx0 + ex[4 * q], tx0 + ex[4 * q + 1], tx0 + ex[4 * q + 2], tx0 + ex[4 * q + 3]);
        own_y[q] = make_uint4(vy(4 * q), vy(4 * q + 1), vy(4 * q + 2), vy(4 * q + 3));
    }
    if (threadIdx.x < kWave) {
        const uint64_t px = publish_and_look_back(status_x, b, ax);
        if (threadIdx.x == 0) pre[0] = px;
    } else if (threadIdx.x < 2 * kWave) {
        const uint64_t py = publish_and_look_back(status_y, b, ay);
        if (threadIdx.x == kWave) pre[1] = py;
    }
    __syncthreads();
    const uint64_t cx = pre[0];
    const uint32_t cy = (uint32_t)pre[1];
    if (b == nb - 1 && threadIdx.x == 0) {
        counters[0] = (int64_t)(cx + ax);
        if (count_host) __hip_atomic_store(count_host, (int64_t)(cx + ax), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        counters[1] = (int64_t)(cy + ay);
        counters[2] = (int64_t)(cx + ax) > capacity ? 1 : 0;
        counters[3] = 0;
    }
#pragma unroll
    for (int r = 0; r < kEmitRounds; ++r) {
        const int64_t g = base + r * kEmitThreads + threadIdx.x;
        if (g < n) {
            const int i = r * kEmitThreads + threadIdx.x;
            emit_off[g] = (uint32_t)(cx + item_x[i]);
            const uint32_t y = item_y[i];
            if (y >> 31) vis_ids[cy + (y & 0x7FFFFFFFu)] = (uint32_t)g;
        }
    }
}

// ---- bin offsets from the per-XCD count copies ---------------------------

__host__ __device__ __forceinline__ int64_t blocks_for(int64_t n) {
    const int64_t b = (n + kPerBlock - 1) / kPerBlock;
    return b > 0 ? b : 1;
}

// Appends value(r) of the items with bk[r] >= 0 (one per thread and round)
// to the list of their repair bucket: aggregated per wavefront and per
// workgroup, one global atomic per bucket and workgroup. lcount / lbase: LDS
// [kBuckets], lcount zeroed before the first round.
template <int R, int NT, class E, class V>
__device__ __forceinline__ void queue_values(const int (&bk)[R], V&& value, int64_t list_stride, uint32_t* lcount,
                                             uint32_t* lbase, E* __restrict__ lists,
                                             uint32_t* __restrict__ bucket_count) {
    uint32_t slot[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        slot[r] = 0;
        if (ballot(bk[r] >= 0) == 0) continue;
#pragma unroll
        for (int k = 0; k < kBuckets; ++k) {
            const uint64_t m = ballot(bk[r] == k);
            if (m == 0) continue;
            const int leader = __builtin_ctzll(m);
            uint32_t b0 = 0;
            if (lane() == leader) b0 = atomicAdd(&lcount[k], (uint32_t)__builtin_popcountll(m));
            b0 = shfl_u32(b0, leader);
            if (bk[r] == k) slot[r] = b0 + rank_in(m);
        }
    }
    __syncthreads();
    if (threadIdx.x < kBuckets)
        lbase[threadIdx.x] = lcount[threadIdx.x] ? atomicAdd(&bucket_count[threadIdx.x], lcount[threadIdx.x]) : 0u;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (bk[r] < 0) continue;
        lists[(int64_t)bk[r] * list_stride + lbase[bk[r]] + slot[r]] = value(r);
    }
}

// The same with the segment ids base + r NT + threadIdx.x as the values.
template <int R, int NT = kThreads>
__device__ __forceinline__ void queue_segments(const int (&bk)[R], int64_t base, int64_t list_stride,
                                               uint32_t* lcount, uint32_t* lbase, uint32_t* __restrict__ lists,
                                               uint32_t* __restrict__ bucket_count) {
    queue_values<R, NT>(
        bk, [&](int r) { return (uint32_t)(base + r * NT + threadIdx.x); }, list_stride, lcount, lbase, lists,
        bucket_count);
}

// bin_off[s] = exclusive prefix of the summed copies (bin_off[nseg] = M);
// count[x][s] becomes bin_off[s] + the counts of copies 0..x-1 in segment
// s. With queue_all, every segment with two or more entries is appended to
// the list of its repair bucket and its entries are added to counters[3];
// nothing is queued when the stream overflowed (counters[2]). repaired[s]
// (optional) records whether segment s was queued. With nseg_dev, the
// number of segments (and the stride of the count copies) is *nseg_dev and
// the grid is sized for its upper bound: workgroups past the last needed one
// leave after their ticket.
__global__ void __launch_bounds__(kThreads) bin_offsets_kernel(uint32_t* __restrict__ count, int64_t nseg_max,
                                                               const uint32_t* __restrict__ nseg_dev,
                                                               uint32_t* __restrict__ bin_off, uint32_t* ticket,
                                                               uint64_t* status, uint32_t* __restrict__ lists,
                                                               uint32_t* __restrict__ bucket_count,
                                                               int64_t* __restrict__ counters, bool queue_all,
                                                               uint8_t* __restrict__ repaired,
                                                               const int64_t* __restrict__ stop) {
    if (stopped(stop)) return;  // the segment bases were not written either
    __shared__ uint32_t tk;
    __shared__ uint32_t lds32[kThreads / kWave];
    __shared__ uint64_t pre;
    __shared__ uint32_t lcount[kBuckets], lbase[kBuckets];
    __shared__ __align__(16) uint32_t tots[kPerBlock];  // segment totals, then block-exclusive prefixes
    if (threadIdx.x == 0) tk = atomicAdd(ticket, 1u);
    if (threadIdx.x < kBuckets) lcount[threadIdx.x] = 0;
    __syncthreads();
    const int64_t b = tk;
    const int64_t nseg = nseg_dev ? (int64_t)*nseg_dev : nseg_max;
    const int64_t nb = blocks_for(nseg);
    if (b >= nb) return;
    const int64_t base = b * kPerBlock;
    const bool queue = queue_all && counters[2] == 0;
    // the copies' counts stay in registers for the base pass below
    uint32_t cv[kRounds][kCopies];
    uint32_t v[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int64_t sg = base + r * kThreads + threadIdx.x;
        v[r] = 0;
#pragma unroll
        for (int x = 0; x < kCopies; ++x) {
            cv[r][x] = sg < nseg ? count[(int64_t)x * nseg + sg] : 0u;
            v[r] += cv[r][x];
        }
        tots[r * kThreads + threadIdx.x] = v[r];
    }
    __syncthreads();
    // each thread scans kRounds consecutive segment totals
    uint4* own = reinterpret_cast<uint4*>(tots) + 2 * threadIdx.x;
    const uint4 t0 = own[0], t1 = own[1];
    const uint32_t c[kRounds] = {t0.x, t0.y, t0.z, t0.w, t1.x, t1.y, t1.z, t1.w};
    uint32_t ex[kRounds], s = 0;
#pragma unroll
    for (int i = 0; i < kRounds; ++i) {
        ex[i] = s;
        s += c[i];
    }
    uint32_t agg;
    const uint32_t tex = block_excl_u32(s, lds32, &agg);
    own[0] = make_uint4(tex + ex[0], tex + ex[1], tex + ex[2], tex + ex[3]);
    own[1] = make_uint4(tex + ex[4], tex + ex[5], tex + ex[6], tex + ex[7]);
    if (threadIdx.x < kWave) {
        const uint64_t pv = publish_and_look_back(status, b, agg);
        if (threadIdx.x == 0) pre = pv;
    }
    __syncthreads();
    const uint32_t carry = (uint32_t)pre;
    if (b == nb - 1 && threadIdx.x == 0) bin_off[nseg] = carry + agg;
    int bk[kRounds];
    uint32_t queued = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int64_t sg = base + r * kThreads + threadIdx.x;
        uint32_t run = carry + tots[r * kThreads + threadIdx.x];
        bk[r] = -1;
        if (sg < nseg) {
            bin_off[sg] = run;
#pragma unroll
            for (int x = 0; x < kCopies; ++x) {
                count[(int64_t)x * nseg + sg] = run;
                run += cv[r][x];
            }
            if (queue) bk[r] = bucket_of(v[r]);
            if (repaired) repaired[sg] = bk[r] >= 0 ? 1 : 0;
            if (bk[r] >= 0) queued += v[r];
        }
    }
    if (!queue) return;
    queue_segments(bk, base, nseg_max, lcount, lbase, lists, bucket_count);
    const uint32_t qsum = block_sum_u32(queued, lds32);
    if (threadIdx.x == 0 && qsum)
        atomicAdd(reinterpret_cast<unsigned long long*>(&counters[3]), (unsigned long long)qsum);
}

// ---- rule-based repair selection -------------------------------------------
// Table "Exact-repair selection rules" and the supplement's Algorithm
// "Selective repair selection and local exact sorting": a segment of length
// l >= 2, bin b, in a tile of l_tile entries is kept when l >= 320, l > 512,
// 100 l >= 45 l_tile, 129 <= l <= 256 and 100 l >= 10 l_tile, or b < 2 and
// l >= 16; kept segments are selected in (tile, bin) order while the
// selected entries fit the budget B (first fit). Kept length of segment q
// (0 when not kept or past the end).
__device__ __forceinline__ uint32_t kept_length(const uint32_t* __restrict__ bin_off, int64_t q, int K,
                                                int64_t nseg) {
    if (q >= nseg) return 0u;
    const int64_t t = q / K;
    const int b = (int)(q - t * K);
    const uint32_t len = bin_off[q + 1] - bin_off[q];
    if (len <= 1) return 0u;
    const uint64_t tl = bin_off[t * K + K] - bin_off[t * K];
    const uint64_t l100 = 100ull * len;
    const bool keep = len >= 320u || len > 512u || l100 >= 45ull * tl || (len >= 129u && len <= 256u && l100 >= 10ull * tl) ||
                      (b < 2 && len >= 16u);
    return keep ? len : 0u;
}

__device__ __forceinline__ uint64_t budget_of(float frac, uint32_t M) {
    return (uint64_t)floor((double)frac * (double)M);
}

// Pass 1: prefix of the kept lengths by a single-pass scan. A kept segment
// whose inclusive prefix is within B is selected (all kept segments before
// it were selected and fit). The one kept segment whose prefix first
// exceeds B is rejected; it leaves ctl = {its index + 1, B - the exclusive
// prefix} for the sequential continuation. When everything fits,
// counters[3] = the kept total.
__global__ void __launch_bounds__(kThreads) select_prefix_kernel(const uint32_t* __restrict__ bin_off, int64_t nseg,
                                                                 int K, float budget, uint32_t* ticket,
                                                                 uint64_t* status, uint32_t* __restrict__ ctl,
                                                                 uint32_t* __restrict__ lists,
                                                                 uint32_t* __restrict__ bucket_count,
                                                                 int64_t* __restrict__ counters,
                                                                 uint8_t* __restrict__ repaired,
                                                                 const int64_t* __restrict__ stop) {
    if (stopped(stop)) return;
    __shared__ uint32_t tk;
    __shared__ uint32_t lds32[kThreads / kWave];
    __shared__ uint64_t pre;
    __shared__ uint32_t lcount[kBuckets], lbase[kBuckets];
    if (threadIdx.x == 0) tk = atomicAdd(ticket, 1u);
    if (threadIdx.x < kBuckets) lcount[threadIdx.x] = 0;
    __syncthreads();
    const int64_t b = tk;
    const int64_t nb = blocks_for(nseg);
    if (b >= nb) return;
    const int64_t base = b * kPerBlock;
    const bool queue = counters[2] == 0;
    const uint64_t B = budget_of(budget, bin_off[nseg]);
    uint32_t v[kRounds];
    uint32_t s = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        v[r] = kept_length(bin_off, base + r * kThreads + threadIdx.x, K, nseg);
        s += v[r];
    }
    const uint32_t agg = block_sum_u32(s, lds32);
    if (threadIdx.x < kWave) {
        const uint64_t pv = publish_and_look_back(status, b, agg);
        if (threadIdx.x == 0) pre = pv;
    }
    __syncthreads();
    uint64_t carry = pre;
    if (b == nb - 1 && threadIdx.x == 0 && carry + agg <= B) counters[3] = (int64_t)(carry + agg);
    int bk[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int64_t sg = base + r * kThreads + threadIdx.x;
        uint32_t tot;
        const uint64_t excl = carry + block_excl_u32(v[r], lds32, &tot);
        carry += tot;
        const uint64_t incl = excl + v[r];
        const bool sel = v[r] != 0 && incl <= B;
        if (v[r] != 0 && incl > B && excl <= B) {
            ctl[0] = (uint32_t)(sg + 1);
            ctl[1] = (uint32_t)(B - excl);
        }
        if (repaired && sg < nseg) repaired[sg] = sel ? 1 : 0;
        bk[r] = queue && sel ? bucket_of(v[r]) : -1;
    }
    queue_segments(bk, base, nseg, lcount, lbase, lists, bucket_count);
}

constexpr int kTailThreads = 1024;

// Exclusive scan over a workgroup of kTailThreads; *total gets the sum.
// Ends with a barrier.
__device__ __forceinline__ uint32_t tail_excl_u32(uint32_t v, uint32_t* lds, uint32_t* total) {
    constexpr int NW = kTailThreads / kWave;
    const int w = threadIdx.x / kWave, l = lane();
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const uint32_t o = shfl_up_u32(inc, d);
        if (l >= d) inc += o;
    }
    if (l == kWave - 1) lds[w] = inc;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const uint32_t t = lds[i];
        before += i < w ? t : 0u;
        all += t;
    }
    __syncthreads();
    *total = all;
    return before + inc - v;
}

// Pass 2 (one workgroup): first fit over the segments after the first
// rejected one, with the remaining budget R, 1024 segments at a time. In a
// chunk, candidates are the kept segments with length <= R; the longest run
// of candidates whose running sum fits R is selected, the candidate that
// ends it is rejected, R drops by the run's sum and the candidates after it
// are filtered against the new R, until none is left. Stops once R < 2 (a
// kept segment has two or more entries). counters[3] = B - R at the end.
__global__ void __launch_bounds__(kTailThreads) select_tail_kernel(const uint32_t* __restrict__ bin_off,
                                                                   int64_t nseg, int K, float budget,
                                                                   const uint32_t* __restrict__ ctl,
                                                                   uint32_t* __restrict__ lists,
                                                                   uint32_t* __restrict__ bucket_count,
                                                                   int64_t* __restrict__ counters,
                                                                   uint8_t* __restrict__ repaired) {
    __shared__ uint32_t lds[kTailThreads / kWave];
    __shared__ uint32_t first, rem;
    if (ctl[0] == 0 || counters[2] != 0) return;
    const uint64_t B = budget_of(budget, bin_off[nseg]);
    uint32_t R = ctl[1];
    for (int64_t base = ctl[0]; base < nseg && R >= 2u; base += kTailThreads) {
        const int64_t q = base + threadIdx.x;
        const uint32_t kl = kept_length(bin_off, q, K, nseg);
        bool cand = kl != 0u && kl <= R;
        bool sel = false;
        while (__syncthreads_or(cand)) {
            uint32_t tot;
            const uint32_t excl = tail_excl_u32(cand ? kl : 0u, lds, &tot);
            if (threadIdx.x == 0) first = 0xFFFFFFFFu;
            __syncthreads();
            if (cand && excl + kl > R) atomicMin(&first, (uint32_t)threadIdx.x);
            __syncthreads();
            const uint32_t f = first;
            if (f == 0xFFFFFFFFu) {
                sel = sel || cand;
                cand = false;
                R -= tot;
            } else {
                if (threadIdx.x == f) rem = R - excl;
                __syncthreads();
                if (cand && threadIdx.x < f) sel = true;
                if (threadIdx.x <= f) cand = false;
                R = rem;
                cand = cand && kl <= R;
            }
        }
        if (sel) {
            if (repaired) repaired[q] = 1;
            const int bk = bucket_of(kl);
            const uint32_t at = atomicAdd(&bucket_count[bk], 1u);
            lists[(int64_t)bk * nseg + at] = (uint32_t)q;
        }
    }
    if (threadIdx.x == 0) counters[3] = (int64_t)(B - R);
}

// ---- per-tile segment bases -------------------------------------------------
// seg_base[t] = exclusive prefix of the per-tile bin counts, each clamped to
// 1..kmax and rounded down to a power of two; seg_base[T] = S.

__device__ __forceinline__ uint32_t pow2_bins(int32_t k, int kmax) {
    const uint32_t c = (uint32_t)(k < 1 ? 1 : (k > kmax ? kmax : k));
    return 1u << (31 - __builtin_clz(c));
}

__global__ void __launch_bounds__(kThreads) seg_base_kernel(const int32_t* __restrict__ kt, int64_t T, int kmax,
                                                            uint32_t* __restrict__ seg_base, uint2* __restrict__ tile_seg,
                                                            uint32_t* ticket, uint64_t* status,
                                                            const int64_t* __restrict__ stop) {
    const bool write = !stopped(stop);
    __shared__ uint32_t tk;
    __shared__ uint32_t lds32[kThreads / kWave];
    __shared__ uint64_t pre;
    if (threadIdx.x == 0) tk = atomicAdd(ticket, 1u);
    __syncthreads();
    const int64_t b = tk;
    const int64_t nb = gridDim.x;
    const int64_t base = b * kPerBlock;
    uint32_t v[kRounds];
    uint32_t sum = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int64_t t = base + r * kThreads + threadIdx.x;
        v[r] = t < T ? pow2_bins(kt[t], kmax) : 0u;
        sum += v[r];
    }
    const uint32_t agg = block_sum_u32(sum, lds32);
    if (threadIdx.x < kWave) {
        const uint64_t pv = publish_and_look_back(status, b, agg);
        if (threadIdx.x == 0) pre = pv;
    }
    __syncthreads();
    uint32_t carry = (uint32_t)pre;
    if (write && b == nb - 1 && threadIdx.x == 0) seg_base[T] = carry + agg;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int64_t t = base + r * kThreads + threadIdx.x;
        uint32_t tot;
        const uint32_t ex = block_excl_u32(v[r], lds32, &tot);
        if (t < T) {
            if (write) seg_base[t] = carry + ex;
            tile_seg[t] = make_uint2(carry + ex, 32u - (uint32_t)__builtin_ctz(v[r]));
        }
        carry += tot;
    }
}

// ---- grouped binning: group prefix and per-group counting sort ---------------

// group_off[g] = exclusive prefix of gcount over g < G, group_off[G] = total
// (one workgroup; G <= kMaxGroups = 8 per thread), and order[0 .. G) = the
// groups by decreasing floor(log2(count)) (empty groups last; arbitrary
// inside a class), so that the group sort starts the longest groups first.
// A count of 2^32 entries or more wraps the prefix sums, and a position can then
// belong to two groups: every group is empty instead (the stream is flagged as
// truncated). Where the call is stopped (see stopped()), the later launches learn
// it from the words that they read first anyway: order[] = -1, and the word
// behind the bucket counts is set.
// With sp.list, also the slices of kSlice entries of the groups that are
// split, sp.list[i] = {group, index among the split groups, begin, end}, and
// sp.ctl [0] = split groups, [1] = slices.
__global__ void __launch_bounds__(kTailThreads) group_scan_kernel(const uint32_t* __restrict__ gcount, GroupMap gm,
                                                                  const int64_t* __restrict__ counters,
                                                                  uint32_t* __restrict__ group_off,
                                                                  uint32_t* __restrict__ order, int64_t capacity,
                                                                  GroupSplit sp, const int64_t* stop,
                                                                  uint32_t* __restrict__ bucket_count) {
    const int G = gm.G;
    // per-tile bin counts: each group's first segment, segment count and the
    // most sub-bins (up to SB) whose codes fit the group sort's counters
    if (gm.seg_base) {
        for (int g = threadIdx.x; g < G; g += kTailThreads) {
            const int64_t t0 = (int64_t)g * gm.GT, t1 = min(t0 + gm.GT, gm.T);
            const uint32_t first = gm.seg_base[t0], segs = gm.seg_base[t1] - first;
            uint32_t lg = 0;
            while ((2u << lg) <= (uint32_t)gm.SB && (uint64_t)segs << (lg + 1) <= (uint64_t)kMaxGroupSegs) ++lg;
            gm.ginfo[g] = make_uint4(first, segs, lg, 0u);
        }
    }
    static_assert(kMaxGroups <= 8 * kTailThreads, "eight groups per thread");
    constexpr int kClasses = 33;  // class 31 - floor(log2 count) for count > 0, 32 for empty
    __shared__ uint32_t lds[kTailThreads / kWave];
    __shared__ uint32_t chist[kClasses], cbase[kClasses];
    if (threadIdx.x < kClasses) chist[threadIdx.x] = 0;
    // consecutive groups per thread, as few as cover them
    const int per = (G + kTailThreads - 1) / kTailThreads, i0 = per * threadIdx.x;
    const bool wrapped = (uint64_t)counters[0] >> 32 != 0, off = stop && counters[2] != 0;
    if (off && threadIdx.x == 0) bucket_count[kBuckets] = 1;
    uint32_t v[8], s = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        v[j] = j < per && i0 + j < G ? gcount[i0 + j] : 0u;
        if (wrapped) v[j] = 0;
        s += v[j];
    }
    uint32_t total;
    uint32_t run = tail_excl_u32(s, lds, &total);  // ends with a barrier: chist is cleared
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (j < per && i0 + j < G) {
            group_off[i0 + j] = run;
            atomicAdd(&chist[v[j] ? __builtin_clz(v[j]) : 32], 1u);
        }
        run += v[j];
    }
    if (threadIdx.x == 0) group_off[G] = total;
    if (sp.list) {
        // each split group's first slice, then all threads list the slices
        // (binary search over the groups)
        __shared__ uint32_t first_item[kMaxGroups];
        __shared__ uint16_t group_id[kMaxGroups];
        run -= s;  // the thread's first group again
        uint32_t n[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t lo = (uint32_t)min((int64_t)run, capacity);
            run += v[j];
            n[j] = (uint32_t)min((int64_t)run, capacity) - lo;
        }
        uint32_t ng = 0, ns = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool in = split_group(n[j]);
            ng += in ? 1u : 0u;
            ns += in ? (n[j] + kSlice - 1) / kSlice : 0u;
        }
        uint32_t all_g, all_s;
        uint32_t h = tail_excl_u32(ng, lds, &all_g), at = tail_excl_u32(ns, lds, &all_s);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (!split_group(n[j])) continue;
            first_item[h] = at;
            group_id[h++] = (uint16_t)(i0 + j);
            at += (n[j] + kSlice - 1) / kSlice;
        }
        if (threadIdx.x == 0) {
            sp.ctl[0] = all_g;
            sp.ctl[1] = all_s;
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < all_s; i += kTailThreads) {
            uint32_t a = 0, b = all_g;  // first_item[a] <= i < first_item[b]
            while (b - a > 1) {
                const uint32_t mid = (a + b) / 2;
                if (first_item[mid] <= i)
                    a = mid;
                else
                    b = mid;
            }
            const uint32_t g = group_id[a], k = i - first_item[a];
            const uint32_t lo = (uint32_t)min((int64_t)group_off[g], capacity);
            const uint32_t hi = (uint32_t)min((int64_t)group_off[g + 1], capacity);
            sp.list[i] = make_uint4(g, a, lo + k * kSlice, min(lo + (k + 1) * kSlice, hi));
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t b = 0;
        for (int c = 0; c < kClasses; ++c) {
            cbase[c] = b;
            b += chist[c];
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j)
        if (j < per && i0 + j < G) order[atomicAdd(&cbase[v[j] ? __builtin_clz(v[j]) : 32], 1u)] = off ? 0xFFFFFFFFu : (uint32_t)(i0 + j);
}

#ifndef TGS_SORT_THREADS
#define TGS_SORT_THREADS 512
#endif
#ifndef TGS_SORT_BATCH
#define TGS_SORT_BATCH (8192 / TGS_SORT_THREADS)
#endif
constexpr int kSortThreads = TGS_SORT_THREADS;  // threads of a group-sort workgroup
constexpr int kSortBatch = TGS_SORT_BATCH;      // entries per thread and sweep step, loaded before any is used

// Staging of the group sort's output when the lists hold sub-segment
// descriptors (SB > 1: exact repair, no records) and the group has at most
// kStage entries: they are placed at their code offsets in LDS, each
// sub-segment of 2..kRankMax entries is put in pair order there (an entry's
// rank among its sub-segment's pairs), and the group is
// written out in order: the output is written in runs instead of one
// scattered 8-byte store per entry, and the short sub-segments need no
// repair pass.
#ifndef TGS_STAGE
#define TGS_STAGE 4096
#endif
constexpr int kStage = TGS_STAGE;
constexpr int kRankMax = 128;

// The segments and codes of group g: segments [sbase, sbase + segs), SB
// sub-bins each, entry codes 0 .. segs SB - 1; nseg = all segments.
struct GroupCodes {
    int64_t sbase, segs, nseg;
    int SB, codes;
};
__device__ __forceinline__ GroupCodes codes_of(const GroupMap& gm, int g, int64_t nseg) {
    GroupCodes c;
    if (gm.seg_base) {
        const uint4 gi = gm.ginfo[g];
        c.sbase = gi.x;
        c.segs = gi.y;
        c.SB = 1 << gi.z;
        c.nseg = gm.seg_base[gm.T];
    } else {
        c.sbase = (int64_t)g * gm.GS;
        c.segs = min((int64_t)gm.GS, nseg - c.sbase);
        c.SB = gm.SB;
        c.nseg = nseg;
    }
    c.codes = (int)(c.segs * c.SB);
    return c;
}
// First code of tile t of the group (tiles g GT ..).
__device__ __forceinline__ int64_t first_code(const GroupMap& gm, const GroupCodes& c, int g, int64_t t) {
    return gm.seg_base ? ((int64_t)gm.seg_base[t] - c.sbase) * c.SB : (t - (int64_t)g * gm.GT) * gm.K * c.SB;
}

// The grouped pairs with the tile number above the id (GroupMap::tagged): an
// entry's code and its plain pair.
template <bool TAG>
struct GroupedPairs {
    DepthBins bins;
    uint32_t id_mask;
    int shift;
    __device__ __forceinline__ GroupedPairs(const float* __restrict__ zrange, const GroupMap& gm) {
        if (!TAG) return;
        bins = DepthBins(zrange, gm.K * gm.SB);
        shift = 31 - gm.tag_bits;  // (shifted once more: tag_bits may be 0)
        id_mask = 0xFFFFFFFFu >> gm.tag_bits;
    }
    __device__ __forceinline__ uint32_t code_of(uint64_t p) const {
        return __umul24((uint32_t)p >> shift >> 1, (uint32_t)bins.K) + bins((uint32_t)(p >> 32));
    }
    __device__ __forceinline__ uint64_t plain(uint64_t p) const {
        return TAG ? (p & ((uint64_t)0xFFFFFFFFu << 32 | id_mask)) : p;
    }
};

// Per-group results from pre[] (LDS), the exclusive prefix of the group's n
// entries over its codes: the bin offsets and repair flags of its segments,
// the entries of its repaired segments (queued[g]) and of its tiles
// (tile_count[t], optional). lds32: NT / 64 words. Per-group values go to
// arrays that a later launch sums: a thousand workgroups adding to one word
// would wait for each other (25 to 50 ns each).
template <int NT>
__device__ __forceinline__ void group_results(const GroupMap& gm, const GroupCodes& gc, int g, uint32_t lo, uint32_t n,
                                              const uint32_t* pre, bool queue, uint32_t* __restrict__ bin_off,
                                              uint8_t* __restrict__ repaired, uint32_t* __restrict__ queued_out,
                                              uint32_t* __restrict__ tile_count, uint32_t* lds32) {
    if (tile_count) {
        // entries per tile: difference of the prefixes at the tiles' first
        // codes, as the bin offsets will give them
        const int64_t t0 = (int64_t)g * gm.GT, t1 = min(t0 + gm.GT, (int64_t)gm.T);
        auto before = [&](int64_t t) -> uint32_t {
            if (t >= t1) return n;
            const int64_t c = first_code(gm, gc, g, t);
            return c < gc.codes ? pre[c] : n;
        };
        for (int64_t t = t0 + threadIdx.x; t < t1; t += NT) tile_count[t] = before(t + 1) - before(t);
    }
    uint32_t queued = 0;
    for (int c = threadIdx.x; c < gc.segs; c += NT) {
        const uint32_t b = pre[c * gc.SB], len = (c + 1 < gc.segs ? pre[(c + 1) * gc.SB] : n) - b;
        bin_off[gc.sbase + c] = lo + b;
        const bool rep = queue && len >= 2;
        if (repaired) repaired[gc.sbase + c] = rep ? 1 : 0;
        if (rep) queued += len;
    }
    if (g == gm.G - 1 && threadIdx.x == 0) bin_off[gc.nseg] = lo + n;
    const uint32_t qsum = block_sum_u32<NT>(queued, lds32);
    if (threadIdx.x == 0) queued_out[g] = qsum;
}

// Parts of a long group. Its codes are cut into parts that fit the stage:
// every kPartStep entries (at the next code), and around any code of more than
// kPartCode entries, which is a part by itself; so every other part has less
// than kPartStep + kPartCode = kStage entries.
static_assert(kPartStep + kPartCode == kStage, "parts fit the stage");

// Thread t holds the counts cnt[] of codes t PER .. and run, the entries
// before them; prev is the count of the code before. flag[j] = a part starts
// at the thread's code j; returns the number of starts after code 0.
template <int PER>
__device__ __forceinline__ uint32_t part_starts(const uint32_t (&cnt)[PER], uint32_t run, uint32_t prev, int codes,
                                                uint32_t (&flag)[PER]) {
    uint32_t flags = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int k = (int)threadIdx.x * PER + j;
        const uint32_t len = cnt[j];
        flag[j] = k > 0 && k < codes &&
                          (run / kPartStep != (run - prev) / kPartStep || len > kPartCode || prev > kPartCode)
                      ? 1u
                      : 0u;
        flags += flag[j];
        run += len;
        prev = len;
    }
    return flags;
}

// Tile of group g that code k belongs to, relative to the group's first.
__device__ __forceinline__ uint32_t tile_of_code(const GroupMap& gm, const GroupCodes& gc, int g, uint32_t k) {
    if (!gm.seg_base) return k / (uint32_t)(gm.K * gc.SB);
    uint32_t t = 0, end = (uint32_t)min((int64_t)gm.GT, gm.T - (int64_t)g * gm.GT);
    while (end - t > 1) {
        const uint32_t mid = (t + end) / 2;
        if (first_code(gm, gc, g, (int64_t)g * gm.GT + mid) <= (int64_t)k)
            t = mid;
        else
            end = mid;
    }
    return t;
}

// One workgroup per group: its entries [group_off[g], group_off[g + 1])
// (clipped to the capacity) are counted per code (segment, or sub-segment
// when SB > 1) in LDS, the code offsets follow by a workgroup scan, and a
// second sweep places every entry at its code offset + an LDS rank (staged
// as above when SB > 1). Also writes bin_off for the group's segments,
// queues the repair segments (as bin_offsets_kernel; sub-segments as
// {begin, length} when SB > 1, without those the staging ordered), and
// writes the records of single-entry segments.
// With sp.list, the groups that are split are left out here, and the first
// sp.slice_grid workgroups count their entries per code, slice by slice, into
// sp.hist (see group_split_kernel).
template <bool TAG>
__global__ void __launch_bounds__(kSortThreads, 4) group_sort_kernel(
    const uint64_t* __restrict__ tmp_pair, uint16_t* tmp_code, const uint32_t* __restrict__ group_off,
    const uint32_t* __restrict__ order, const float* __restrict__ zrange, GroupMap gm, int64_t nseg, int64_t capacity, uint64_t* __restrict__ pairs,
    uint32_t* __restrict__ bin_off, uint32_t* __restrict__ lists, int64_t list_stride,
    uint32_t* __restrict__ bucket_count, const int64_t* __restrict__ counters, bool queue_all,
    uint8_t* __restrict__ repaired, RecordSink rs, uint32_t* __restrict__ queued, uint32_t* __restrict__ tile_count,
    GroupSplit sp) {
    constexpr int NT = kSortThreads;
    constexpr int kMaxPer = kMaxGroupSegs / NT;
    constexpr uint32_t kNone = 0xFFFFFFFFu;
    __shared__ uint32_t hist[kMaxGroupSegs];
    __shared__ uint32_t cur[kMaxGroupSegs];
    __shared__ uint64_t stage[kStage + kRankPad];
    __shared__ uint16_t scode[kStage];
    __shared__ uint32_t lds32[NT / kWave];
    __shared__ uint32_t lcount[kBuckets], lbase[kBuckets];
    const GroupedPairs<TAG> in(zrange, gm);
    // adds the codes of entries [lo, hi) to hist, and keeps them (for the same
    // thread) when they had to be worked out and will be needed again
    auto count = [&](uint32_t lo, uint32_t hi, bool keep) {
        for (uint32_t base = lo; base < hi; base += NT * kSortBatch) {
            if (TAG) {
                uint64_t pr[kSortBatch];
#pragma unroll
                for (int j = 0; j < kSortBatch; ++j)
                    pr[j] = tmp_pair[min(base + (uint32_t)(j * NT) + threadIdx.x, hi - 1)];
#pragma unroll
                for (int j = 0; j < kSortBatch; ++j) {
                    const uint32_t e = base + (uint32_t)(j * NT) + threadIdx.x;
                    if (e >= hi) continue;
                    const uint32_t c = in.code_of(pr[j]);
                    atomicAdd(&hist[c], 1u);
                    if (keep) tmp_code[e] = (uint16_t)c;
                }
                continue;
            }
            uint32_t c[kSortBatch];
#pragma unroll
            for (int j = 0; j < kSortBatch; ++j) {
                const uint32_t e = base + (uint32_t)(j * NT) + threadIdx.x;
                c[j] = e < hi ? (uint32_t)tmp_code[e] : kNone;
            }
#pragma unroll
            for (int j = 0; j < kSortBatch; ++j)
                if (c[j] != kNone) atomicAdd(&hist[c[j]], 1u);
        }
    };
    if ((int)blockIdx.x < sp.slice_grid) {
        // a run of consecutive slices; those of one group are contiguous and
        // are added to its hist together
        const uint32_t slices = sp.ctl[1], per = (slices + sp.slice_grid - 1) / sp.slice_grid;
        const uint32_t end = min((blockIdx.x + 1) * per, slices);
        for (uint32_t i = blockIdx.x * per; i < end;) {
            const uint4 first = sp.list[i];
            uint32_t stop = first.w;
            for (++i; i < end; ++i) {
                const uint4 next = sp.list[i];
                if (next.y != first.y) break;
                stop = next.w;
            }
            const int codes = codes_of(gm, (int)first.x, nseg).codes;
            for (int c = threadIdx.x; c < codes; c += NT) hist[c] = 0;
            __syncthreads();
            count(first.z, stop, false);
            __syncthreads();
            uint32_t* gh = sp.hist + (int64_t)first.y * sp.stride;
            for (int c = threadIdx.x; c < codes; c += NT)
                if (hist[c]) atomicAdd(&gh[c], hist[c]);
        }
        return;
    }
    const int g = (int)order[blockIdx.x - sp.slice_grid];
    if (g < 0) return;  // stopped
    const int64_t cap = capacity;
    const uint32_t lo = (uint32_t)min((int64_t)group_off[g], cap);
    const uint32_t hi = (uint32_t)min((int64_t)group_off[g + 1], cap);
    if (sp.list && split_group(hi - lo)) return;
    const GroupCodes gc = codes_of(gm, g, nseg);
    if (lo == hi) {  // an empty group: offsets only
        for (int c = threadIdx.x; c < gc.segs; c += NT) {
            bin_off[gc.sbase + c] = lo;
            if (repaired) repaired[gc.sbase + c] = 0;
        }
        const int64_t t0 = (int64_t)g * gm.GT;
        if (tile_count)
            for (int64_t t = t0 + threadIdx.x; t < min(t0 + gm.GT, (int64_t)gm.T); t += NT) tile_count[t] = 0;
        if (threadIdx.x == 0) {
            queued[g] = 0;
            if (g == gm.G - 1) bin_off[gc.nseg] = lo;
        }
        return;
    }
    const int codes = gc.codes;
    const int per = (codes + NT - 1) / NT;  // codes per thread, <= kMaxPer
    for (int c = threadIdx.x; c < per * NT; c += NT) hist[c] = 0;
    if (threadIdx.x < kBuckets) lcount[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t n = hi - lo;
    const bool staged = gm.SB > 1 && n <= (uint32_t)kStage;
    // a staged group's entries stay in registers from the count to the placement
    constexpr int kHeld = kStage / NT;
    uint32_t held_code[kHeld];
    uint64_t held_pair[kHeld];
    auto held = [&](int j) { return (uint32_t)(j * NT) + threadIdx.x < n; };
    if (staged) {
#pragma unroll
        for (int j = 0; j < kHeld; ++j) {
            const uint32_t e = min(lo + (uint32_t)(j * NT) + threadIdx.x, hi - 1);
            held_pair[j] = tmp_pair[e];
            if (!TAG) held_code[j] = tmp_code[e];
        }
#pragma unroll
        for (int j = 0; j < kHeld; ++j) {
            if (!held(j)) continue;
            if (TAG) held_code[j] = in.code_of(held_pair[j]);
            atomicAdd(&hist[held_code[j]], 1u);
        }
    } else {
        count(lo, hi, true);
    }
    __syncthreads();
    // exclusive prefix of the code counts: thread i owns codes i per ..
    uint32_t ex[kMaxPer], sum = 0;
#pragma unroll
    for (int j = 0; j < kMaxPer; ++j) {
        ex[j] = sum;
        if (j < per) sum += hist[threadIdx.x * per + j];
    }
    uint32_t agg;
    const uint32_t tex = block_excl_u32<NT>(sum, lds32, &agg);
#pragma unroll
    for (int j = 0; j < kMaxPer; ++j)
        if (j < per) cur[threadIdx.x * per + j] = tex + ex[j];
    __syncthreads();
    const bool queue = queue_all && counters[2] == 0;
    // sub-segments the staging puts in order (none with an overflow)
    const uint32_t local_max = staged && queue ? (uint32_t)kRankMax : 1u;
    // repair queues per code (segments when SB == 1, sub-segments otherwise)
    int bk[kMaxPer];
#pragma unroll
    for (int r = 0; r < kMaxPer; ++r) {
        const int c = r * NT + threadIdx.x;
        bk[r] = -1;
        if (r < per && c < codes) {
            if (queue && hist[c] > local_max) bk[r] = bucket_of(hist[c]);
        }
    }
    if (gm.SB > 1)
        // sub-segments are queued as {begin, length}: the repair needs no offset lookup
        queue_values<kMaxPer, NT>(
            bk,
            [&](int r) {
                const int c = r * NT + threadIdx.x;
                return make_uint2(lo + cur[c], hist[c]);
            },
            list_stride, lcount, lbase, reinterpret_cast<uint2*>(lists), bucket_count);
    else
        queue_segments<kMaxPer, NT>(bk, gc.sbase, list_stride, lcount, lbase, lists, bucket_count);
    // ends with a barrier: the offsets are read (here and above) before the placement moves them
    group_results<NT>(gm, gc, g, lo, n, cur, queue, bin_off, repaired, queued, tile_count, lds32);
    if (staged) {
        // place at the code offsets in LDS ...
#pragma unroll
        for (int j = 0; j < kHeld; ++j) {
            if (!held(j)) continue;
            const uint32_t q = atomicAdd(&cur[held_code[j]], 1u);
            stage[q] = in.plain(held_pair[j]);
            scode[q] = (uint16_t)held_code[j];
        }
        __syncthreads();
        // ... and write the group out in order, short sub-segments by rank
        for (uint32_t q = threadIdx.x; q < n; q += NT) {
            const uint32_t c = scode[q];
            const uint64_t v = stage[q];
            uint32_t out = q;
            const uint32_t len = hist[c];
            // the code's slots are [cur - len, cur) once placed
            if (len >= 2 && len <= local_max) out = rank_slot(stage, v, cur[c] - len, len);
            pairs[lo + out] = v;
        }
    } else {
        for (uint32_t base = lo; base < hi; base += NT * kSortBatch) {
            uint32_t c[kSortBatch];
            uint64_t pr[kSortBatch];
#pragma unroll
            for (int j = 0; j < kSortBatch; ++j) {
                const uint32_t e = base + (uint32_t)(j * NT) + threadIdx.x;
                c[j] = kNone;
                pr[j] = 0;
                if (e < hi) {
                    c[j] = tmp_code[e];
                    pr[j] = tmp_pair[e];
                }
            }
#pragma unroll
            for (int j = 0; j < kSortBatch; ++j) {
                if (c[j] == kNone) continue;
                const uint32_t p = lo + atomicAdd(&cur[c[j]], 1u);
                const uint64_t v = in.plain(pr[j]);
                pairs[p] = v;
                // records exist only with SB == 1, where a code is a segment
                if (rs.masks && hist[c[j]] == 1u) rs.put((uint32_t)(gc.sbase + c[j]), p, v);
            }
        }
    }
}

// ---- split groups ------------------------------------------------------------
// A long group is cut into parts in passes over its entries, and the parts are
// sorted one per workgroup:
//   slices (group_sort_kernel)  entries per code of every slice of kSlice
//                               entries, added to the group's hist;
//   group_split_kernel          one workgroup per slice: the parts follow from
//                               the complete hist, the slice's entries are
//                               ordered by part in LDS and written to the
//                               parts' places in runs;
//   sort_small_kernel           one workgroup per part: bucket sort in LDS.
// The numbers of slices and parts are known on the device only, so their
// workgroups stride over the lists; the grids are what the 256 CUs hold (an
// upper bound as the grid would launch thousands of empty workgroups, at over
// a microsecond each and CU).
constexpr int kSplitThreads = 512;
constexpr int kSplitGrid = 512;  // two workgroups per CU (LDS)

struct SplitLds {
    union {
        uint64_t stage[kSlice];
        struct {  // before the staging
            uint32_t pre[kMaxGroupSegs];   // exclusive prefix of the code counts
            uint32_t part[kMaxGroupSegs];  // part | tile of the group << kPartBits of each code
        };
    };
    uint32_t meta[kSlice];      // that of each slot
    uint32_t begin[kMaxParts];  // first entry of the part, relative to the group; then its place for this slice
    union {
        uint16_t count[kMaxParts];       // first code; then the slice's entries per part and their exclusive prefix
        uint32_t count2[kMaxParts / 2];  // (two parts to a word, for the additions)
        uint32_t tail[kSplitThreads];    // each thread's last code count
    };
};
constexpr int kPartBits = 12;
static_assert(1 << kPartBits == kMaxParts, "part numbers");

template <bool TAG>
__global__ void __launch_bounds__(kSplitThreads) group_split_kernel(
    const uint64_t* __restrict__ tmp_pair, const uint16_t* __restrict__ tmp_code, const uint32_t* __restrict__ group_off,
    const float* __restrict__ zrange, GroupMap gm, int64_t nseg, int64_t capacity, uint64_t* __restrict__ pairs, uint16_t* __restrict__ part_tile,
    uint32_t* __restrict__ bin_off, const int64_t* __restrict__ counters, uint8_t* __restrict__ repaired,
    uint32_t* __restrict__ queued, uint32_t* __restrict__ tile_count, GroupSplit sp) {
    constexpr int NT = kSplitThreads;
    constexpr int kPer = kMaxGroupSegs / NT;  // codes per thread
    constexpr int kEnt = kSlice / NT;         // entries per thread
    constexpr int kPpt = kMaxParts / NT;      // parts per thread, at most
    __shared__ SplitLds L;
    __shared__ uint32_t lds32[NT / kWave];
    __shared__ uint32_t unit0;
    const GroupedPairs<TAG> in(zrange, gm);
    uint4 next = sp.list[blockIdx.x];  // (the grid is at most the list's length)
    const uint32_t slices = sp.ctl[1];
    for (uint32_t it = blockIdx.x; it < slices; it += gridDim.x) {
        const uint4 sl = next;
        if (it + gridDim.x < slices) next = sp.list[it + gridDim.x];
        const int g = (int)sl.x;
        uint32_t* gh = sp.hist + (int64_t)sl.y * sp.stride;
        uint32_t* cursor = gh + sp.stride - kMaxParts;
        const uint32_t lo = (uint32_t)min((int64_t)group_off[g], capacity);
        const uint32_t n = (uint32_t)min((int64_t)group_off[g + 1], capacity) - lo;
        const GroupCodes gc = codes_of(gm, g, nseg);
        // the slice's entries, requested before the prefix is worked out
        uint32_t c[kEnt];
        uint64_t pr[kEnt];
#pragma unroll
        for (int j = 0; j < kEnt; ++j) {
            const uint32_t e = min(sl.z + (uint32_t)(j * NT) + threadIdx.x, sl.w - 1);
            pr[j] = tmp_pair[e];
            if (!TAG) c[j] = tmp_code[e];
        }
        uint32_t cnt[kPer], s = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int k = (int)threadIdx.x * kPer + j;
            cnt[j] = k < gc.codes ? gh[k] : 0u;
            s += cnt[j];
        }
        uint32_t total;
        const uint32_t before = block_excl_u32<NT>(s, lds32, &total);
        uint32_t run = before;
        // last count of the thread before, for its last code's length
        L.tail[threadIdx.x] = cnt[kPer - 1];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            L.pre[threadIdx.x * kPer + j] = run;
            run += cnt[j];
        }
        __syncthreads();
        uint32_t flag[kPer];
        const uint32_t flags = part_starts(cnt, before, threadIdx.x ? L.tail[threadIdx.x - 1] : 0u, gc.codes, flag);
        uint32_t nflags;
        uint32_t p = block_excl_u32<NT>(flags, lds32, &nflags);
        const uint32_t parts = nflags + 1;  // at most one per code
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int k = (int)threadIdx.x * kPer + j;
            p += flag[j];
            if (k < gc.codes) {
                L.part[k] = p | tile_of_code(gm, gc, g, (uint32_t)k) << kPartBits;
                if (flag[j] || k == 0) {
                    L.begin[p] = L.pre[k];
                    L.count[p] = (uint16_t)k;  // first code, for the unit list
                }
            }
        }
        __syncthreads();
        if (sl.z == lo) {
            // the group's first slice: its results and its parts
            if (threadIdx.x == 0) unit0 = atomicAdd(&sp.ctl[2], parts);
            group_results<NT>(gm, gc, g, lo, n, L.pre, counters[2] == 0, bin_off, repaired, queued, tile_count, lds32);
            __syncthreads();
            for (uint32_t q = threadIdx.x; q < parts; q += NT) {
                const uint32_t b = L.begin[q], e = q + 1 < parts ? L.begin[q + 1] : n;
                const uint32_t k0 = L.count[q], k1 = q + 1 < parts ? L.count[q + 1] : (uint32_t)gc.codes;
                const uint32_t ta = tile_of_code(gm, gc, g, k0);
                sp.units[unit0 + q] = make_uint4(lo + b, e - b, ta, tile_of_code(gm, gc, g, k1 - 1) - ta + 1);
            }
            __syncthreads();
        }
        for (uint32_t q = threadIdx.x; q < (parts + 1) / 2; q += NT) L.count2[q] = 0;
        __syncthreads();
        uint32_t rank[kEnt], mt[kEnt];
#pragma unroll
        for (int j = 0; j < kEnt; ++j) {
            const bool ok = sl.z + (uint32_t)(j * NT) + threadIdx.x < sl.w;
            if (TAG) c[j] = in.code_of(pr[j]);
            mt[j] = L.part[c[j]];
            const uint32_t q = mt[j] & (kMaxParts - 1), sh = (q & 1u) * 16u;
            rank[j] = ok ? (atomicAdd(&L.count2[q / 2], 1u << sh) >> sh) & 0xFFFFu : 0u;
        }
        __syncthreads();
        // exclusive prefix over the parts, and each part's place in the output
        const uint32_t pp = (parts + NT - 1) / NT;  // consecutive parts per thread
        uint32_t pc[kPpt], ps = 0;
#pragma unroll
        for (uint32_t j = 0; j < (uint32_t)kPpt; ++j) {
            const uint32_t q = threadIdx.x * pp + j;
            pc[j] = j < pp && q < parts ? L.count[q] : 0u;
            ps += pc[j];
        }
        uint32_t base[kPpt];
#pragma unroll
        for (uint32_t j = 0; j < (uint32_t)kPpt; ++j)
            base[j] = pc[j] ? atomicAdd(&cursor[threadIdx.x * pp + j], pc[j]) : 0u;
        uint32_t pex = block_excl_u32<NT>(ps, lds32, &total);
#pragma unroll
        for (uint32_t j = 0; j < (uint32_t)kPpt; ++j) {
            const uint32_t q = threadIdx.x * pp + j;
            if (j < pp && q < parts) {
                L.count[q] = (uint16_t)pex;
                L.begin[q] += base[j] - pex;  // slot i of the slice goes to begin + i
            }
            pex += pc[j];
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kEnt; ++j) {
            if (sl.z + (uint32_t)(j * NT) + threadIdx.x >= sl.w) continue;
            const uint32_t i = L.count[mt[j] & (kMaxParts - 1)] + rank[j];
            L.stage[i] = in.plain(pr[j]);
            L.meta[i] = mt[j];
        }
        __syncthreads();
        const uint32_t m = sl.w - sl.z;
        for (uint32_t i = threadIdx.x; i < m; i += NT) {
            const uint32_t k = L.meta[i];
            const uint32_t to = lo + L.begin[k & (kMaxParts - 1)] + i;
            pairs[to] = L.stage[i];
            part_tile[to] = (uint16_t)(k >> kPartBits);
        }
        __syncthreads();
    }
}

__global__ void fill_u32_dyn_kernel(uint32_t* p, uint32_t v, const uint32_t* n_dev, int mult, const int64_t* stop) {
    if (stopped(stop)) return;  // *n_dev was not written
    const int64_t n = (int64_t)*n_dev * mult;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void fill_u32_kernel(uint32_t* p, uint32_t v, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

}  // namespace

int64_t scan_blocks(int64_t n) { return n > 0 ? (n + kPerBlock - 1) / kPerBlock : 1; }

hipError_t launch_emit_scan(const uint32_t* info, int64_t n, int tiles_x, int tiles_y, uint32_t* emit_off,
                            uint32_t* vis_ids, uint32_t* ticket, uint64_t* status_x, uint64_t* status_y,
                            int64_t* counters, int64_t capacity, int64_t* count_host, hipStream_t s) {
    const int64_t blocks = n > 0 ? (n + kEmitPerBlock - 1) / kEmitPerBlock : 1;
    hipLaunchKernelGGL(emit_scan_kernel, dim3((unsigned)blocks), dim3(kEmitThreads), 0, s,
                       reinterpret_cast<const uint4*>(info), n, tiles_x, tiles_y, emit_off, vis_ids, ticket, status_x,
                       status_y, counters, capacity, count_host);
    return hipGetLastError();
}

hipError_t launch_bin_offsets(uint32_t* count, int64_t nseg, const uint32_t* nseg_dev, uint32_t* bin_off,
                              uint32_t* ticket, uint64_t* status, uint32_t* lists, uint32_t* bucket_count,
                              int64_t* counters, bool queue_all, uint8_t* repaired, const int64_t* stop,
                              hipStream_t s) {
    hipLaunchKernelGGL(bin_offsets_kernel, dim3((unsigned)scan_blocks(nseg)), dim3(kThreads), 0, s, count, nseg,
                       nseg_dev, bin_off, ticket, status, lists, bucket_count, counters, queue_all, repaired, stop);
    return hipGetLastError();
}

hipError_t launch_repair_select(const uint32_t* bin_off, int64_t T, int K, float budget, uint32_t* ticket,
                                uint64_t* status, uint32_t* ctl, uint32_t* lists, uint32_t* bucket_count,
                                int64_t* counters, uint8_t* repaired, const int64_t* stop, hipStream_t s) {
    const int64_t nseg = T * K;
    if (nseg == 0) return hipSuccess;
    hipLaunchKernelGGL(select_prefix_kernel, dim3((unsigned)scan_blocks(nseg)), dim3(kThreads), 0, s, bin_off, nseg,
                       K, budget, ticket, status, ctl, lists, bucket_count, counters, repaired, stop);
    hipLaunchKernelGGL(select_tail_kernel, dim3(1), dim3(kTailThreads), 0, s, bin_off, nseg, K, budget, ctl, lists,
                       bucket_count, counters, repaired);
    return hipGetLastError();
}

hipError_t launch_group_scan(const uint32_t* gcount, GroupMap gm, const int64_t* counters, uint32_t* group_off,
                             uint32_t* order, int64_t capacity, const GroupSplit& sp, const int64_t* stop,
                             uint32_t* bucket_count, hipStream_t s) {
    hipLaunchKernelGGL(group_scan_kernel, dim3(1), dim3(kTailThreads), 0, s, gcount, gm, counters, group_off, order,
                       capacity, sp, stop, bucket_count);
    return hipGetLastError();
}

hipError_t launch_group_sort(const uint64_t* tmp_pair, uint16_t* tmp_code, const uint32_t* group_off,
                             const uint32_t* order, const float* zrange, GroupMap gm, int64_t nseg, int64_t capacity, uint64_t* pairs, uint32_t* bin_off,
                             uint32_t* lists, int64_t list_stride, uint32_t* bucket_count,
                             const int64_t* counters, bool queue_all, uint8_t* repaired, RecordSink rs,
                             uint32_t* queued, uint32_t* tile_count, const GroupSplit& sp, uint16_t* part_tile,
                             hipStream_t s) {
    hipLaunchKernelGGL(gm.tagged ? group_sort_kernel<true> : group_sort_kernel<false>, dim3((unsigned)(sp.slice_grid + gm.G)), dim3(kSortThreads), 0, s, tmp_pair,
                       tmp_code, group_off, order, zrange, gm, nseg, capacity, pairs, bin_off, lists, list_stride, bucket_count,
                       counters, queue_all, repaired, rs, queued, tile_count, sp);
    if (sp.list) {
        hipLaunchKernelGGL(gm.tagged ? group_split_kernel<true> : group_split_kernel<false>, dim3((unsigned)std::min(sp.max_slices, kSplitGrid)),
                           dim3(kSplitThreads), 0, s, tmp_pair, tmp_code, group_off, zrange, gm, nseg, capacity, pairs,
                           part_tile, bin_off, counters, repaired, queued, tile_count, sp);
    }
    return hipGetLastError();
}

hipError_t launch_seg_base(const int32_t* per_tile_bins, int64_t T, int kmax, uint32_t* seg_base, uint2* tile_seg,
                           uint32_t* ticket, uint64_t* status, const int64_t* stop, hipStream_t s) {
    hipLaunchKernelGGL(seg_base_kernel, dim3((unsigned)scan_blocks(T)), dim3(kThreads), 0, s, per_tile_bins, T, kmax,
                       seg_base, tile_seg, ticket, status, stop);
    return hipGetLastError();
}

hipError_t launch_fill_u32_dyn(uint32_t* p, uint32_t v, const uint32_t* n_dev, int mult, int64_t max_n,
                               const int64_t* stop, hipStream_t s) {
    if (max_n <= 0) return hipSuccess;
    int64_t grid = (max_n + 255) / 256;
    if (grid > 4096) grid = 4096;
    hipLaunchKernelGGL(fill_u32_dyn_kernel, dim3((unsigned)grid), dim3(256), 0, s, p, v, n_dev, mult, stop);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t v, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    int64_t grid = (n + 255) / 256;
    if (grid > 4096) grid = 4096;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)grid), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

}  // namespace tgs
