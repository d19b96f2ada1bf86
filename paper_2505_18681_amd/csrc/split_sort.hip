// Splitter sort: how the automatic choice sorts arrays of some 1e4 to 4e5 keys
// (Sec. 4.3, Algorithm 6 hands arrays to the routine that is fastest at their
// length).  There the radix passes, the histogram before them and the merge
// rounds are chains of short launches, each of which costs 4 to 10 us whatever
// it sorts; this one has two (parallel sorting by regular sampling, Shi and
// Schaeffer 1992, with one workgroup per bucket):
//
//   split_blocks_kernel   every wave, or two or four of them together, sorts a
//                         block of 512 to 2048 keys in registers
//                         (wave_merge.hpp) and writes it, with the values or
//                         indices, to the scratch, and an index row of every
//                         block; one workgroup meanwhile sorts a sample of the
//                         input and writes the splitters that bound the buckets;
//   split_buckets_kernel  one workgroup per bucket: it finds where its two
//                         splitters fall in every block (one thread per block:
//                         the block's index row, then the keys between two of
//                         its entries), which also tells where the bucket goes
//                         in the output, gathers the blocks' pieces, sorts them
//                         and writes them out.
//
// Keys are ordered by (key, block, position), so equal keys keep their input
// order, and a splitter is a key and a block: any number of copies of a key
// spreads over the buckets.  A bucket of more than kSplitBucketMost keys (the
// sample bounds no bucket tightly) is sorted in several steps, each of which
// takes the smallest keys left.
//
// Bound by latency: the chains of dependent loads and compare steps in the two
// kernels.
//
// Compiled once per (key bytes, value bytes) pair with -DEVOSORT_KB/-DEVOSORT_VB.
#include "common.hpp"
#include "split_sort.hpp"
#include "wave_merge.hpp"

#ifndef EVOSORT_KB
#error "EVOSORT_KB must be defined"
#endif
#ifndef EVOSORT_VB
#error "EVOSORT_VB must be defined"
#endif

#define EVOSORT_CAT4(a, b, c, d) a##b##c##d
#define EVOSORT_XCAT4(a, b, c, d) EVOSORT_CAT4(a, b, c, d)
#define EVOSORT_BLOCKS_NAME(kb, vb) EVOSORT_XCAT4(split_blocks_k, kb, _v, vb)
#define EVOSORT_BUCKETS_NAME(kb, vb) EVOSORT_XCAT4(split_buckets_k, kb, _v, vb)

namespace evosort {

namespace {

constexpr int kSplitThreads = 256;  // of a bucket's workgroup
static_assert(kSplitBlocksMost <= kSplitThreads, "one thread per block");
static_assert(kSplitBucketMost == kSplitThreads * 8 && kSplitGroupKeys == kSplitThreads * 8, "eight records per thread");

// ---------------------------------------------------------------- blocks --
// The splitters: 256 * PER keys of the input, one from each of as many equal
// parts of it, in order of (key, block); bucket j begins at the sample of rank
// j / buckets.
template <int KB, int PER>
__device__ __forceinline__ void write_splitters(const SplitArgs& a, const OrderMap<typename KeyWord<KB>::U>& om,
                                                typename Rec<KB>::W* buf)
{
    using U = typename KeyWord<KB>::U;
    using SR = Rec<KB>;
    using SW = typename SR::W;
    constexpr int S = kSplitThreads * PER;
    const uint32_t n = (uint32_t)a.n;
    SW x[PER];
    U k[PER];
    uint32_t at[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const uint32_t i = (uint32_t)(q * kSplitThreads) + threadIdx.x;
        // part i of S, at a place that differs from part to part (the golden ratio's multiples)
        at[q] = (uint32_t)((((uint64_t)i << 32) + i * 2654435769u) / S * n >> 32);
        k[q] = reinterpret_cast<const U*>(a.keys_in)[at[q] < n ? at[q] : n - 1];
    }
#pragma unroll
    for (int q = 0; q < PER; ++q)
        x[q] = SR::make(om.to_order(k[q]), at[q] / a.plan.block_keys);
    sort_striped<kSplitThreads / kWave, false>(x, buf, 0, [](const SW& p, const SW& q) { return SR::less(p, q); });
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q)
        buf[pad16(striped_rank<kSplitThreads / kWave, PER>(q))] = x[q];
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < a.plan.buckets; j += kSplitThreads)
        reinterpret_cast<SW*>(a.splitters)[j] = buf[pad16((int)(j * (uint32_t)S / a.plan.buckets))];
}

// BW: waves per block of 512 * BW keys.
template <int KB, int VB, int BW>
__global__ __launch_bounds__(kSplitThreads) void split_blocks_kernel(SplitArgs a, OrderMap<typename KeyWord<KB>::U> om)
{
    using U = typename KeyWord<KB>::U;
    using V = typename ValWord<VB>::T;
    using R = BlockRec<KB, VB>;
    using W = typename R::W;
    using SW = typename Rec<KB>::W;
    constexpr int PER = 8;
    constexpr int G = kSplitGroupKeys;
    constexpr int PART = kWave * PER * BW / kSplitRow;  // keys per entry of an index row
    constexpr size_t BYTES = sizeof(SW) * padded16(G);  // a sample's record is as large as a block's, or larger
    static_assert(sizeof(SW) >= sizeof(W), "the buffers hold either");
    __shared__ __attribute__((aligned(16))) unsigned char s_buf[BYTES];

    if (blockIdx.x == 0) {  // the first workgroup: its chain is the longest
        if (threadIdx.x == 0 && a.error_word)
            *a.error_word = 0;
        SW* buf = reinterpret_cast<SW*>(s_buf);
        if (a.plan.samples == 1024)
            write_splitters<KB, 4>(a, om, buf);
        else
            write_splitters<KB, 8>(a, om, buf);
        return;
    }
    const int64_t start = (int64_t)(blockIdx.x - 1) * G;
    const int cnt = a.n - start < G ? (int)(a.n - start) : G;
    const U* keys_in = reinterpret_cast<const U*>(a.keys_in) + start;
    const V* vals_in = reinterpret_cast<const V*>(a.vals_in) + start;
    // A wave loads keys of its own block; what is missing in the last block is
    // filled up with records above all of its own.
    U k[PER];
    W x[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int i = striped_rank<kSplitThreads / kWave, PER>(q);
        k[q] = keys_in[i < cnt ? i : cnt - 1];
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int i = striped_rank<kSplitThreads / kWave, PER>(q);
        x[q] = R::make(i < cnt ? om.to_order(k[q]) : ~(U)0, (uint32_t)i);
    }
    const int first = (int)(threadIdx.x / kWave) / BW * (kWave * PER * BW);  // this wave's block
    sort_striped<BW, false>(x, reinterpret_cast<W*>(s_buf), first, [](const W& p, const W& q) { return R::less(p, q); });
    U* keys = reinterpret_cast<U*>(a.keys_tmp) + start;
    V* vals = reinterpret_cast<V*>(a.vals_tmp) + start;
    U* rows = reinterpret_cast<U*>(a.rows) + start / PART;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int i = striped_rank<kSplitThreads / kWave, PER>(q);
        if (i < cnt) {
            keys[i] = R::ord(x[q]);
            if constexpr (VB != 0)
                vals[i] = a.iota ? (V)(start + R::pos(x[q])) : vals_in[R::pos(x[q])];
            if (i % PART == PART - 1)
                rows[i / PART] = R::ord(x[q]);
        }
    }
}

// --------------------------------------------------------------- buckets --
// A splitter in the order (key, block, position in the block).
template <typename U>
struct Splitter {
    U key;
    int block;
    int pos;
};

// Keys of block c, the sorted words blk[lo, hi) of it that may straddle, that
// come before the splitter: the block's first position that does not.  Eight
// candidates per step, all in flight at once.
template <typename U>
__device__ __forceinline__ int split_position(const U* blk, int lo, int hi, int c, const Splitter<U>& s)
{
    if (c == s.block)
        return s.pos;
    const bool ties = c < s.block;  // this block's equal keys come before the splitter
    while (lo < hi) {
        const int step = (hi - lo + 7) >> 3;
        U x[7];
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            const int at = lo + (j + 1) * step - 1;
            x[j] = blk[at < hi ? at : hi - 1];
        }
        int pass = 0;  // candidates before the splitter: a prefix of them
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            const int at = lo + (j + 1) * step - 1;
            pass += at < hi && (x[j] < s.key || (ties && x[j] == s.key)) ? 1 : 0;
        }
        lo += pass * step;
        if (pass < 7 && lo + step - 1 < hi)  // the first candidate that is not
            hi = lo + step - 1;
    }
    return lo;
}

// COUNT sorted words, 16-byte aligned, of which the first `valid` count: how
// many of them come before (key, block), by block c's place against the block.
template <int COUNT, typename U>
__device__ __forceinline__ int count_before(const U* p, int valid, U key, bool ties)
{
    constexpr int VEC = 16 / (int)sizeof(U);
    uint4 v[COUNT / VEC];
#pragma unroll
    for (int j = 0; j < COUNT / VEC; ++j)
        v[j] = reinterpret_cast<const uint4*>(p)[j];
    int before = 0;
#pragma unroll
    for (int j = 0; j < COUNT / VEC; ++j) {
        U x[VEC];
        __builtin_memcpy(x, &v[j], 16);
#pragma unroll
        for (int i = 0; i < VEC; ++i)
            before += j * VEC + i < valid && (x[i] < key || (ties && x[i] == key)) ? 1 : 0;
    }
    return before;
}

template <int KB, int VB, int BW>
__global__ __launch_bounds__(kSplitThreads) void split_buckets_kernel(SplitArgs a,
                                                                      OrderMap<typename KeyWord<KB>::U> om)
{
    using U = typename KeyWord<KB>::U;
    using V = typename ValWord<VB>::T;
    using R = BlockRec<KB, VB>;
    using W = typename R::W;
    using SR = Rec<KB>;  // a sample: key and sample number
    using SW = typename SR::W;
    constexpr int THREADS = kSplitThreads;
    constexpr int WAVES = THREADS / kWave;
    constexpr int PER = 8;
    constexpr int MOST = kSplitBucketMost;
    constexpr int B = kWave * PER * BW;
    constexpr int PART = B / kSplitRow;  // keys per entry of an index row
    __shared__ W s_buf[padded16(MOST)];
    __shared__ uint32_t s_src[MOST];           // where a gathered key comes from
    __shared__ uint32_t s_off[THREADS];        // first gathered key of every block's piece
    __shared__ uint32_t s_from[THREADS];       // where the piece begins in the scratch
    __shared__ uint32_t s_wtot[WAVES], s_wpos[WAVES];
    __shared__ SW s_next[WAVES];

    const int P = (int)a.plan.blocks, NB = (int)a.plan.buckets, bucket = (int)blockIdx.x;
    const U* words = reinterpret_cast<const U*>(a.keys_tmp);
    const int lane = (int)(threadIdx.x & (kWave - 1)), w = (int)(threadIdx.x / kWave);
    const int n = (int)a.n;
    auto block_len = [&](int c) { return n - c * B < B ? n - c * B : B; };

    // ---- this thread's block: the piece [pos, end) of it is in the bucket ---
    const int c = (int)threadIdx.x;
    const int len = c < P ? block_len(c) : 0;
    const U* blk = words + (size_t)(c < P ? c : 0) * B;
    int pos = 0, end = len;
    {
        const SW* split = reinterpret_cast<const SW*>(a.splitters);
        const SW first = split[bucket], next = split[bucket + 1 < NB ? bucket + 1 : bucket];
        const U key0 = SR::ord(first), key1 = SR::ord(next);
        // an equal key of an earlier block comes before the splitter
        const bool ties0 = (uint32_t)c < SR::pos(first), ties1 = (uint32_t)c < SR::pos(next);
        if (c < P) {
            const U* row = reinterpret_cast<const U*>(a.rows) + (size_t)c * kSplitRow;
            const int whole = len / PART;  // entries that are keys of the block
            const int p0 = count_before<kSplitRow>(row, whole, key0, ties0) * PART;
            const int p1 = count_before<kSplitRow>(row, whole, key1, ties1) * PART;
            pos = p0 + count_before<PART>(blk + (p0 < B ? p0 : 0), len - p0, key0, ties0);
            end = p1 + count_before<PART>(blk + (p1 < B ? p1 : 0), len - p1, key1, ties1);
            if (bucket == 0)
                pos = 0;
            if (bucket + 1 == NB)
                end = len;
        }
    }
    // everything before the bucket in any block is before it in the output
    uint32_t total_pos;
    block_exclusive_scan<THREADS>((uint32_t)pos, s_wpos, &total_pos);
    uint32_t base = total_pos;

    U* keys_out = reinterpret_cast<U*>(a.keys_out);
    V* vals_out = reinterpret_cast<V*>(a.vals_out);
    const V* vals_tmp = reinterpret_cast<const V*>(a.vals_tmp);
    for (;;) {
        // ---- the step's keys: all that are left, or the smallest of them ----
        int stop = end;
        uint32_t total;
        uint32_t off = block_exclusive_scan<THREADS>((uint32_t)(stop - pos), s_wtot, &total);
        if (total == 0)
            break;
        if (total > (uint32_t)MOST) {
            // A splitter that at most MOST / P keys of every piece come
            // before: the smallest of the pieces' keys of that rank.  There
            // is one, since pieces without it would hold MOST keys at most.
            const int rank = MOST / P;
            SW mine = SR::top();
            if (end - pos > rank)
                mine = SR::make(blk[pos + rank], (uint32_t)c);
            auto smaller = [&](const SW& y) { mine = pick(SR::less(y, mine), y, mine); };
            smaller(lane_xor<32>(mine, lane));
            smaller(lane_xor<16>(mine, lane));
            smaller(lane_xor<8>(mine, lane));
            smaller(lane_xor<4>(mine, lane));
            smaller(lane_xor<2>(mine, lane));
            smaller(lane_xor<1>(mine, lane));
            __syncthreads();  // every thread has used the scan's words
            if (lane == 0)
                s_next[w] = mine;
            __syncthreads();
            mine = s_next[0];
#pragma unroll
            for (int i = 1; i < WAVES; ++i)
                mine = pick(SR::less(s_next[i], mine), s_next[i], mine);
            const int owner = (int)SR::pos(mine);
            // only the owner uses the position
            const Splitter<U> s{SR::ord(mine), owner, pos + rank};
            if (c < P)
                stop = split_position(blk, pos, end, c, s);
            off = block_exclusive_scan<THREADS>((uint32_t)(stop - pos), s_wtot, &total);
        }
        const int m = (int)total;
        s_off[threadIdx.x] = off;
        s_from[threadIdx.x] = (uint32_t)(c * B + pos);
        __syncthreads();

        // ---- gather the pieces in block order, sort them, write them out ----
        auto step = [&](auto per) {
            constexpr int N = decltype(per)::value;  // records per thread
            U k[N];
            W x[N];
#pragma unroll
            for (int q = 0; q < N; ++q) {
                const int e = q * THREADS + (int)threadIdx.x;
                const int ee = e < m ? e : m - 1;
                // the last block whose piece begins at or before key ee
                int at = 0;
#pragma unroll
                for (int st = kSplitBlocksMost / 2; st >= 1; st >>= 1)
                    if (st < P)  // uniform
                        at = at + st < P && s_off[at + st] <= (uint32_t)ee ? at + st : at;
                const uint32_t src = s_from[at] + ((uint32_t)ee - s_off[at]);
                k[q] = words[src];
                if constexpr (VB != 0) {
                    if (e < m)
                        s_src[e] = src;
                }
            }
#pragma unroll
            for (int q = 0; q < N; ++q) {
                const int e = q * THREADS + (int)threadIdx.x;
                x[q] = R::make(e < m ? k[q] : ~(U)0, (uint32_t)e);
            }
            sort_striped<WAVES, false>(x, s_buf, 0, [](const W& p, const W& q) { return R::less(p, q); });
#pragma unroll
            for (int q = 0; q < N; ++q) {
                const int i = striped_rank<WAVES, N>(q);
                if (i < m) {
                    if (keys_out)
                        keys_out[base + (uint32_t)i] = om.from_order((U)R::ord(x[q]));
                    if constexpr (VB != 0)
                        vals_out[base + (uint32_t)i] = vals_tmp[s_src[R::pos(x[q])]];
                }
            }
        };
        if (m <= THREADS * 4)
            step(std::integral_constant<int, 4>{});
        else
            step(std::integral_constant<int, PER>{});
        base += total;
        pos = stop;
        __syncthreads();  // the buffers are used again
    }
}

template <int BW>
hipError_t launch_t(bool buckets, const KeyDesc& kd, const SplitArgs& a, hipStream_t s)
{
    using U = typename KeyWord<EVOSORT_KB>::U;
    const OrderMap<U> om{(U)kd.flip, (U)kd.neg, (U)kd.desc};
    if (buckets) {
        hipLaunchKernelGGL((split_buckets_kernel<EVOSORT_KB, EVOSORT_VB, BW>), dim3(a.plan.buckets),
                           dim3(kSplitThreads), 0, s, a, om);
    } else {
        const uint32_t groups = (uint32_t)((a.n + kSplitGroupKeys - 1) / kSplitGroupKeys);
        hipLaunchKernelGGL((split_blocks_kernel<EVOSORT_KB, EVOSORT_VB, BW>), dim3(groups + 1), dim3(kSplitThreads), 0,
                           s, a, om);
    }
    return hipGetLastError();
}

hipError_t launch(bool buckets, const KeyDesc& kd, const SplitArgs& a, hipStream_t s)
{
    const SplitPlan& p = a.plan;
    if (a.n < 1 || a.n > 0x7fffffff || p.blocks < 1 || p.blocks > (uint32_t)kSplitBlocksMost || p.buckets < 1 ||
        (p.samples != 1024 && p.samples != 2048) || p.buckets > p.samples || (int64_t)p.samples > a.n ||
        p.blocks != (a.n + p.block_keys - 1) / p.block_keys)
        return hipErrorInvalidValue;
    switch (p.block_keys) {
    case 512:
        return launch_t<1>(buckets, kd, a, s);
    case 1024:
        return launch_t<2>(buckets, kd, a, s);
    case 2048:
        // 1024 keys a block reach the 2^18 keys that these widths go to
        if constexpr (EVOSORT_KB == 4 && EVOSORT_VB == 0)
            return launch_t<4>(buckets, kd, a, s);
        return hipErrorInvalidValue;
    default:
        return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t EVOSORT_BLOCKS_NAME(EVOSORT_KB, EVOSORT_VB)(const KeyDesc& kd, const SplitArgs& a, hipStream_t s)
{
    return launch(false, kd, a, s);
}

hipError_t EVOSORT_BUCKETS_NAME(EVOSORT_KB, EVOSORT_VB)(const KeyDesc& kd, const SplitArgs& a, hipStream_t s)
{
    return launch(true, kd, a, s);
}

}  // namespace evosort
