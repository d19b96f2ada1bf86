// Last stage of a prefix sort (Sec. 4, Algorithms 4 and 5 with the lower
// digits' passes replaced): the passes of the upper digits have left the keys
// in order of their upper digits, keys of equal upper digits (a run) beside
// each other in input order; here every run is put in order of the lower
// digits, stably.  The plan takes this route only when a sample says that the
// runs are short (write_plan), but any run length is sorted:
//
//   radix_runs_kernel       a tile of keys with kRunMost keys on either side in
//                           LDS; every key counts the larger keys of its run
//                           before it and the smaller ones after it, which is
//                           how far it moves.  Runs longer than kRunMost keys
//                           are copied as they are and listed, and where one of
//                           them is out of order its tile is marked.
//   radix_long_runs_kernel  one workgroup per listed run with a mark (a key that
//                           fills a long run by itself leaves none): the
//                           one-workgroup LSD sort, and above its capacity
//                           merges of such pieces.
//
// Compiled once per (key bytes, value bytes) pair with -DEVOSORT_KB/-DEVOSORT_VB.
#include "block_lsd.hpp"
#include "radix_finish.hpp"
#include "radix_impl.hpp"

#ifndef EVOSORT_KB
#error "EVOSORT_KB must be defined"
#endif
#ifndef EVOSORT_VB
#error "EVOSORT_VB must be defined"
#endif

#define EVOSORT_CAT4(a, b, c, d) a##b##c##d
#define EVOSORT_XCAT4(a, b, c, d) EVOSORT_CAT4(a, b, c, d)
#define EVOSORT_RUNS_NAME(kb, vb) EVOSORT_XCAT4(radix_runs_k, kb, _v, vb)
#define EVOSORT_LONG_NAME(kb, vb) EVOSORT_XCAT4(radix_long_runs_k, kb, _v, vb)

namespace evosort {

namespace {

constexpr int kRunThreads = 512;
constexpr int kRunItems = kRunTile / kRunThreads;

// The buffers of the plan's last stage.
__device__ __forceinline__ PassIo last_stage_io(const RadixRoute& r, uint32_t stages)
{
    PassIo io{};
    route_pass(r, stages - 1, stages, io);
    return io;
}

// In a bit set of 64-bit words: the highest set bit at or below `at`, and the
// lowest one above it, as far as kRunMost bits away (else one that is further).
__device__ __forceinline__ int bit_at_or_below(const uint64_t* set, int at)
{
    int w = at >> 6;
    const int last = at - kRunMost > 0 ? (at - kRunMost) >> 6 : 0;
    uint64_t x = set[w] & (~0ull >> (63 - (at & 63)));
    while (x == 0 && w > last)
        x = set[--w];
    return x ? w * 64 + 63 - __clzll((long long)x) : at - kRunMost - 1;
}
__device__ __forceinline__ int bit_above(const uint64_t* set, int at, int words)
{
    int w = (at + 1) >> 6;
    const int last = (at + 1 + kRunMost) >> 6 < words ? (at + 1 + kRunMost) >> 6 : words - 1;
    uint64_t x = w <= last ? set[w] & (~0ull << ((at + 1) & 63)) : 0;
    while (x == 0 && w < last)
        x = set[++w];
    return x ? w * 64 + __ffsll((unsigned long long)x) - 1 : at + 1 + kRunMost;
}
// Whether any of the bits lo .. hi is set.
__device__ __forceinline__ bool any_bit(const uint64_t* set, int lo, int hi)
{
    for (int w = lo >> 6; w <= hi >> 6; ++w) {
        uint64_t x = set[w];
        if (w == lo >> 6)
            x &= ~0ull << (lo & 63);
        if (w == hi >> 6)
            x &= ~0ull >> (63 - (hi & 63));
        if (x)
            return true;
    }
    return false;
}

// The keys (and values) are read once, the halo from cache, and written once,
// each within its run of the place it was read from.  Bound by latency: 239 to
// 255 registers leave one workgroup of eight waves per CU, too few to cover its
// loads and LDS steps (1e9 int64 keys 8.0 ms, 2.0 TB/s; 3e7 float64 keys with
// 8-byte values 0.26 ms, 3.7 TB/s; 1e7 int64 argsort with 10 copies of each key,
// which writes no keys, 82 us, 2.9 TB/s; a radix pass 3.7-3.9, the copy 5.1).  Two bit sets in LDS, made from one ballot per 64 keys, hold
// where a run starts and where a key is above the next of its run; a key finds
// its run from the first and leaves its place alone when the second is empty
// there (equal keys, keys in order), so that only runs out of order are
// counted, one key after the other.  Counting is VALU work of about the
// longest run per wave: walking every run in both directions without the bit
// sets took 446 us for 1e7 argsort keys with 10 copies of each.
template <int KB, int VB>
__global__ __launch_bounds__(kRunThreads) void radix_runs_kernel(RadixRunArgs a, OrderMap<typename KeyWord<KB>::U> om)
{
    using U = typename KeyWord<KB>::U;
    using V = typename ValWord<VB>::T;
    constexpr int H = kRunMost;
    constexpr int WORDS = (kRunTile + 2 * H) / 64;
    static_assert(H % 64 == 0 && kRunThreads % 64 == 0, "a wave's keys are one word of a bit set");
    __shared__ U s_key[kRunTile + 2 * H];
    __shared__ uint64_t s_start[WORDS];  // a run starts here
    __shared__ uint64_t s_above[WORDS];  // the next key is of the same run and smaller

    const uint32_t plan = *a.route.plan;
    const uint32_t shift = 8 * plan_prefix_pass(plan);
    if (shift == 0) {
        finish_copies(a.route, plan_stages(plan), a.n, KB, VB, (size_t)blockIdx.x * kRunThreads + threadIdx.x,
                      (size_t)gridDim.x * kRunThreads);
        return;
    }
    const PassIo io = last_stage_io(a.route, plan_stages(plan));
    const U* __restrict__ keys_in = reinterpret_cast<const U*>(io.keys_in);
    U* __restrict__ keys_out = reinterpret_cast<U*>(io.keys_out);
    const V* __restrict__ vals_in = reinterpret_cast<const V*>(io.vals_in);
    V* __restrict__ vals_out = reinterpret_cast<V*>(io.vals_out);
    const bool write_keys = !(io.flags & RADIX_FLAG_SKIP_KEYS);
    const int64_t tiles = (a.n + kRunTile - 1) / kRunTile;

    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        // LDS word i holds key t0 + i, for first <= i < end
        const int64_t t0 = t * kRunTile - H;
        const int cnt = a.n - t * kRunTile < kRunTile ? (int)(a.n - t * kRunTile) : kRunTile;
        const int first = t == 0 ? H : 0;
        const int end = a.n - t0 < kRunTile + 2 * H ? (int)(a.n - t0) : kRunTile + 2 * H;
        U k[kRunItems];
        V v[VB ? kRunItems : 1];
#pragma unroll
        for (int q = 0; q < kRunItems; ++q) {
            const int i0 = q * kRunThreads + (int)threadIdx.x;
            const int64_t at = t * kRunTile + (i0 < cnt ? i0 : cnt - 1);
            k[q] = keys_in[at];
            if constexpr (VB != 0)
                v[q] = vals_in[at];
        }
        // the halo: one thread per key on either side
        static_assert(2 * H == kRunThreads, "one halo key per thread");
        const int hi = (int)threadIdx.x < H ? (int)threadIdx.x : kRunTile + (int)threadIdx.x;
        if (hi >= first && hi < end)
            s_key[hi] = om.to_order(keys_in[t0 + hi]);
#pragma unroll
        for (int q = 0; q < kRunItems; ++q) {
            k[q] = om.to_order(k[q]);
            const int i0 = q * kRunThreads + (int)threadIdx.x;
            if (i0 < cnt)
                s_key[H + i0] = k[q];
        }
        __syncthreads();

        // The bit sets.  Of the first key in sight only the array's own is
        // known to start a run; a run that goes on before the others is
        // longer than H for every key of the tile that is in it.
        auto bits = [&](int at) {
            const bool valid = at >= first && at < end;
            const U x = s_key[valid ? at : first];
            const U before = s_key[valid && at > first ? at - 1 : first];
            const U after = s_key[valid && at + 1 < end ? at + 1 : first];
            // one past the array's last key counts as a start
            const bool start = valid ? (at > first ? ((x ^ before) >> shift) != 0 : t == 0)
                                     : at == end && t0 + end == a.n;
            const bool above = valid && at + 1 < end && ((x ^ after) >> shift) == 0 && after < x;
            const uint64_t ms = ballot(start), ma = ballot(above);
            if ((threadIdx.x & (kWave - 1)) == 0) {
                s_start[at >> 6] = ms;
                s_above[at >> 6] = ma;
            }
        };
#pragma unroll
        for (int q = 0; q < kRunItems; ++q)
            bits(H + q * kRunThreads + (int)threadIdx.x);
        bits(hi);
        __syncthreads();

        const int lane = (int)(threadIdx.x & (kWave - 1));
#pragma unroll
        for (int q = 0; q < kRunItems; ++q) {
            const int i0 = q * kRunThreads + (int)threadIdx.x;
            if (i0 >= cnt)
                continue;
            const int at = H + i0;
            const int c = at >> 6;  // the wave's word
            const uint64_t s0 = uniform(s_start[c - 1]), s1 = uniform(s_start[c]), s2 = uniform(s_start[c + 1]);
            const uint64_t a0 = uniform(s_above[c - 1]), a1 = uniform(s_above[c]), a2 = uniform(s_above[c + 1]);
            int run = at, stop = at;  // the run's keys, if it has to be sorted
            bool sort = false;
            if (s0 != 0 && s2 != 0) {
                // every run of the wave's keys lies in these three words
                if ((a0 | a1 | a2) != 0) {
                    const uint64_t upto = s1 & (~0ull >> (63 - lane)), past = s1 & ((~0ull << lane) << 1);
                    const int b0 = 63 - __clzll((long long)s0), b2 = __ffsll((unsigned long long)s2) - 1;
                    const bool before = (a0 >> b0) != 0, after = (a2 & ((1ull << b2) - 1)) != 0;
                    const int lo = upto ? 63 - __clzll((long long)upto) : 0;
                    const uint64_t below = past ? (past & (0 - past)) - 1 : ~0ull;
                    sort = ((a1 & below) >> lo) != 0 || (!upto && before) || (!past && after);
                    run = upto ? c * 64 + lo : c * 64 - 64 + b0;
                    stop = past ? c * 64 + __ffsll((unsigned long long)past) - 1 : c * 64 + 64 + b2;
                }
            } else {
                run = bit_at_or_below(s_start, at);
                stop = bit_above(s_start, at, WORDS);
                if (stop - run > H) {
                    if (run == at)  // its first key
                        a.long_runs[atomicAdd(a.long_count, 1u)] = t0 + at;
                    if ((a1 >> lane) & 1)
                        a.unsorted[t] = 1;
                } else {
                    sort = any_bit(s_above, run, stop - 1);
                }
            }
            int move = 0;
            if (sort) {
                // its place: the smaller keys of the run, and the equal ones before it
                int rank = 0;
                if (KB == 8 && shift <= 32) {
                    // the lower halves decide
                    const uint32_t* low = reinterpret_cast<const uint32_t*>(s_key);
                    const uint32_t mine = (uint32_t)k[q];
                    for (int j = run; j < stop; j += 2) {
                        const int j1 = j + 1 < stop ? j + 1 : j;
                        const uint32_t x0 = low[(KB / 4) * j], x1 = low[(KB / 4) * j1];
                        rank += (x0 < mine || (x0 == mine && j < at)) ? 1 : 0;
                        rank += (j1 > j && (x1 < mine || (x1 == mine && j1 < at))) ? 1 : 0;
                    }
                } else {
                    for (int j = run; j < stop; ++j) {
                        const U x = s_key[j];
                        rank += (x < k[q] || (x == k[q] && j < at)) ? 1 : 0;
                    }
                }
                move = run + rank - at;
            }
            const int64_t dst = t0 + at + move;
            if (write_keys)
                keys_out[dst] = om.from_order(k[q]);
            if constexpr (VB != 0)
                vals_out[dst] = v[q];
        }
        __syncthreads();  // the next tile overwrites the keys and the bit sets
    }
}

// Workgroup shape of the long runs' sort: the largest the one-workgroup sort
// of the pair has (values through the keys' staging area where both together
// would not fit in LDS).
template <int KB, int VB>
struct LongShape {
    static constexpr int THREADS = KB == 8 && VB != 0 ? 512 : 1024;
    static constexpr int ITEMS = 16;
    static constexpr bool SPLIT = (size_t)THREADS * ITEMS * (KB + VB) > 128 * 1024;
    static constexpr int CAP = THREADS * ITEMS;
};

// One level of merges of a workgroup: src[0, len) holds sorted pieces of
// `width` keys (the last one shorter); every key finds its place among the
// other piece of its pair by binary search, the left piece first on ties.
template <int KB, int VB, int THREADS>
__device__ void merge_pieces(const OrderMap<typename KeyWord<KB>::U>& om, const typename KeyWord<KB>::U* src,
                             typename KeyWord<KB>::U* dst, const typename ValWord<VB>::T* vsrc,
                             typename ValWord<VB>::T* vdst, int64_t len, int64_t width)
{
    using U = typename KeyWord<KB>::U;
    constexpr int F = 4;  // searches in flight per thread: each is a chain of dependent loads
    for (int64_t i0 = threadIdx.x; i0 < len; i0 += F * THREADS) {
        U k[F];
        int64_t lo[F], hi[F], from[F], i[F];
        bool left[F];
#pragma unroll
        for (int f = 0; f < F; ++f) {
            i[f] = i0 + f * THREADS < len ? i0 + f * THREADS : len - 1;
            const int64_t base = i[f] / (2 * width) * (2 * width);
            const int64_t mid = base + width < len ? base + width : len;
            const int64_t end = base + 2 * width < len ? base + 2 * width : len;
            left[f] = i[f] < mid;
            from[f] = lo[f] = left[f] ? mid : base;
            hi[f] = left[f] ? end : mid;
            k[f] = om.to_order(src[i[f]]);
        }
        bool more = true;
        while (more) {
            more = false;
#pragma unroll
            for (int f = 0; f < F; ++f) {
                if (lo[f] < hi[f]) {
                    const int64_t c = (lo[f] + hi[f]) >> 1;
                    const U x = om.to_order(src[c]);
                    const bool right = left[f] ? x < k[f] : x <= k[f];
                    lo[f] = right ? c + 1 : lo[f];
                    hi[f] = right ? hi[f] : c;
                    more = true;
                }
            }
        }
#pragma unroll
        for (int f = 0; f < F; ++f) {
            if (i0 + f * THREADS < len) {
                // its place in its own piece and in the other, from the pair's first key
                const int64_t base = i[f] / (2 * width) * (2 * width);
                const int64_t mine = left[f] ? base : (base + width < len ? base + width : len);
                const int64_t d = base + (i[f] - mine) + (lo[f] - from[f]);
                dst[d] = om.from_order(k[f]);
                if constexpr (VB != 0)
                    vdst[d] = vsrc[i[f]];
            }
        }
    }
}

template <int KB, int VB>
__global__ __launch_bounds__((LongShape<KB, VB>::THREADS)) void radix_long_runs_kernel(
    RadixRunArgs a, OrderMap<typename KeyWord<KB>::U> om)
{
    using U = typename KeyWord<KB>::U;
    using V = typename ValWord<VB>::T;
    using S = LongShape<KB, VB>;
    __shared__ BlockLsdLds<KB, VB, S::THREADS, S::ITEMS, S::SPLIT> L;

    const uint32_t plan = *a.route.plan;
    const uint32_t shift = 8 * plan_prefix_pass(plan);
    if (shift == 0)
        return;
    const PassIo io = last_stage_io(a.route, plan_stages(plan));
    const bool write_keys = !(io.flags & RADIX_FLAG_SKIP_KEYS);
    // the stage's input is a buffer of the scratch (it has a pass before it),
    // free once the runs kernel has ended; so is keys_out in an argsort
    U* kx = reinterpret_cast<U*>(const_cast<void*>(io.keys_in));
    U* ky = reinterpret_cast<U*>(io.keys_out);
    V* vx = reinterpret_cast<V*>(const_cast<void*>(io.vals_in));
    V* vy = reinterpret_cast<V*>(io.vals_out);

    const uint32_t count = *a.long_count;
    for (uint32_t r = blockIdx.x; r < count; r += gridDim.x) {
        const int64_t begin = a.long_runs[r];
        const U head = om.to_order(kx[begin]);
        // The run's end: keys are in order of their prefixes, so each round
        // tests THREADS evenly spaced keys and keeps the step between the last
        // that is in the run and the first that is not.
        int64_t last = begin, past = a.n;  // last: in the run; past: not
        while (past - last > 1) {
            const int64_t step = (past - last + S::THREADS - 1) / S::THREADS;
            const int64_t i = last + step * (int64_t)(threadIdx.x + 1);
            const bool in_run = i < past && ((om.to_order(kx[i < past ? i : last]) ^ head) >> shift) == 0;
            const int same = __syncthreads_count(in_run);  // the threads in the run are a prefix
            const int64_t upto = last + step * (int64_t)(same + 1);
            last += step * (int64_t)same;
            past = upto < past ? upto : past;
        }
        const int64_t len = past - begin;
        int marked = 0;
        for (int64_t t = begin / kRunTile + threadIdx.x; t <= last / kRunTile; t += S::THREADS)
            marked |= (int)a.unsorted[t];
        if (!__syncthreads_or(marked))
            continue;  // in order as the runs kernel copied it
        if (len <= S::CAP) {
            block_lsd_sort<KB, VB, S::THREADS, S::ITEMS, S::SPLIT>(
                BlockLsdIo{kx, ky, vx, vy, false, !write_keys}, om, L, begin, (uint32_t)len);
            continue;
        }
        for (int64_t p = 0; p < len; p += S::CAP)
            block_lsd_sort<KB, VB, S::THREADS, S::ITEMS, S::SPLIT>(
                BlockLsdIo{kx, ky, vx, vy, false, false}, om, L, begin + p,
                (uint32_t)(len - p < S::CAP ? len - p : S::CAP));
        bool in_y = true;
        for (int64_t width = S::CAP; width < len; width *= 2) {
            __threadfence_block();
            __syncthreads();
            merge_pieces<KB, VB, S::THREADS>(om, (in_y ? ky : kx) + begin, (in_y ? kx : ky) + begin,
                                             VB ? (in_y ? vy : vx) + begin : nullptr,
                                             VB ? (in_y ? vx : vy) + begin : nullptr, len, width);
            in_y = !in_y;
        }
        __threadfence_block();
        __syncthreads();
        if (!in_y) {
            for (int64_t i = begin + threadIdx.x; i < begin + len; i += S::THREADS) {
                if (write_keys)
                    ky[i] = kx[i];
                if constexpr (VB != 0)
                    vy[i] = vx[i];
            }
            __syncthreads();
        }
    }
}

}  // namespace

hipError_t EVOSORT_RUNS_NAME(EVOSORT_KB, EVOSORT_VB)(const KeyDesc& kd, const RadixRunArgs& a, hipStream_t s)
{
    using U = typename KeyWord<EVOSORT_KB>::U;
    const OrderMap<U> om{(U)kd.flip, (U)kd.neg, (U)kd.desc};
    // four workgroups per CU at most, each looping over its tiles (one at a time
    // is resident, see above): where there is nothing to do, a launch lasts
    // longer the more workgroups it has
    const int64_t tiles = (a.n + kRunTile - 1) / kRunTile;
    const uint32_t grid = (uint32_t)(tiles < 1024 ? tiles : 1024);
    hipLaunchKernelGGL((radix_runs_kernel<EVOSORT_KB, EVOSORT_VB>), dim3(grid), dim3(kRunThreads), 0, s, a, om);
    return hipGetLastError();
}

hipError_t EVOSORT_LONG_NAME(EVOSORT_KB, EVOSORT_VB)(const KeyDesc& kd, const RadixRunArgs& a, hipStream_t s)
{
    using U = typename KeyWord<EVOSORT_KB>::U;
    using S = LongShape<EVOSORT_KB, EVOSORT_VB>;
    static_assert(sizeof(BlockLsdLds<EVOSORT_KB, EVOSORT_VB, S::THREADS, S::ITEMS, S::SPLIT>) <= 160 * 1024,
                  "one workgroup fits in one CU's LDS");
    const OrderMap<U> om{(U)kd.flip, (U)kd.neg, (U)kd.desc};
    // few: a listed run out of order is rare, and this launch mostly finds none
    const int64_t want = a.n / (8 * kRunMost) + 1;
    const uint32_t grid = (uint32_t)(want < 64 ? want : 64);
    hipLaunchKernelGGL((radix_long_runs_kernel<EVOSORT_KB, EVOSORT_VB>), dim3(grid), dim3(S::THREADS), 0, s, a, om);
    return hipGetLastError();
}

}  // namespace evosort
