// Sorting records in the registers of a wave and merging runs of them in LDS:
// what the mergesort's blocks and the splitter sort's blocks and buckets share.
#pragma once

#include "common.hpp"

namespace evosort {

// LDS index of element p of a padded array: one spare element every 16.
__device__ __forceinline__ int pad16(int p) { return p + (p >> 4); }
constexpr int padded16(int n) { return n + (n >> 4) + 1; }

// ---------------------------------------------------------------- records --
template <int KB>
struct Rec;
template <>
struct Rec<4> {
    using W = uint64_t;  // order word << 32 | position in the block
    static __device__ __forceinline__ W make(uint32_t ord, uint32_t pos) { return ((uint64_t)ord << 32) | pos; }
    static __device__ __forceinline__ uint32_t ord(W r) { return (uint32_t)(r >> 32); }
    static __device__ __forceinline__ uint32_t pos(W r) { return (uint32_t)r; }
    static __device__ __forceinline__ bool less(W a, W b) { return a < b; }
    // above every record (positions are below 2^32 - 1)
    static __device__ __forceinline__ W top() { return ~0ull; }
};
template <>
struct Rec<8> {
    struct W {
        uint64_t ord;
        uint32_t pos;
        uint32_t pad;
    };
    static __device__ __forceinline__ W make(uint64_t ord, uint32_t pos) { return W{ord, pos, 0u}; }
    static __device__ __forceinline__ uint64_t ord(const W& r) { return r.ord; }
    static __device__ __forceinline__ uint32_t pos(const W& r) { return r.pos; }
    static __device__ __forceinline__ bool less(const W& a, const W& b)
    {
        return a.ord < b.ord || (a.ord == b.ord && a.pos < b.pos);
    }
    static __device__ __forceinline__ W top() { return W{~0ull, 0xffffffffu, 0u}; }
};

// Records of the block sort.  Keys-only blocks hold bare order words: a
// chunk ranks a key against its chunk mates by (word, position), positions
// being the records' indices, and the merges take the left run's record on
// equal words, so the block is stable without storing positions.  With values
// (or indices) a record also carries the key's position in the block, which
// tells where its value is parked.
template <int KB, int VB>
struct BlockRec {
    using R = Rec<KB>;
    using W = typename R::W;
    static constexpr bool kBare = false;
    static __device__ __forceinline__ W make(typename KeyWord<KB>::U ord, uint32_t pos) { return R::make(ord, pos); }
    static __device__ __forceinline__ typename KeyWord<KB>::U ord(const W& r) { return (typename KeyWord<KB>::U)R::ord(r); }
    static __device__ __forceinline__ uint32_t pos(const W& r) { return R::pos(r); }
    static __device__ __forceinline__ bool less(const W& a, const W& b) { return R::less(a, b); }
    // x (at index jx) comes before y (at index iy) in the stable order
    static __device__ __forceinline__ bool before(const W& x, int, const W& y, int) { return R::less(x, y); }
    static __device__ __forceinline__ W top() { return R::top(); }
};
template <int KB>
struct BlockRec<KB, 0> {
    using W = typename KeyWord<KB>::U;
    static constexpr bool kBare = true;
    static __device__ __forceinline__ W make(W ord, uint32_t) { return ord; }
    static __device__ __forceinline__ W ord(W r) { return r; }
    static __device__ __forceinline__ bool less(W a, W b) { return a < b; }
    static __device__ __forceinline__ bool before(W x, int jx, W y, int iy) { return x < y || (x == y && jx < iy); }
    static __device__ __forceinline__ W top() { return ~(W)0; }
};

// A key with its index in a round's input slice.
template <typename U>
struct KeyIdx;
template <>
struct KeyIdx<uint32_t> {
    uint64_t w;  // key << 32 | index
    static __device__ __forceinline__ KeyIdx make(uint32_t key, uint32_t idx) { return {((uint64_t)key << 32) | idx}; }
    static __device__ __forceinline__ uint32_t key(const KeyIdx& r) { return (uint32_t)(r.w >> 32); }
    static __device__ __forceinline__ uint32_t idx(const KeyIdx& r) { return (uint32_t)r.w; }
    static __device__ __forceinline__ bool less(const KeyIdx& a, const KeyIdx& b) { return a.w < b.w; }
    static __device__ __forceinline__ KeyIdx top() { return {~0ull}; }
};
template <>
struct KeyIdx<uint64_t> {
    uint64_t k;
    uint32_t i;
    static __device__ __forceinline__ KeyIdx make(uint64_t key, uint32_t idx) { return {key, idx}; }
    static __device__ __forceinline__ uint64_t key(const KeyIdx& r) { return r.k; }
    static __device__ __forceinline__ uint32_t idx(const KeyIdx& r) { return r.i; }
    static __device__ __forceinline__ bool less(const KeyIdx& a, const KeyIdx& b)
    {
        return a.k < b.k || (a.k == b.k && a.i < b.i);
    }
    static __device__ __forceinline__ KeyIdx top() { return {~0ull, 0xffffffffu}; }
};

// c ? a : b, field by field for the 16-byte records: a select of the whole
// aggregate can be lowered through private (scratch) memory.
template <typename T>
__device__ __forceinline__ T pick(bool c, const T& a, const T& b)
{
    return c ? a : b;
}
__device__ __forceinline__ Rec<8>::W pick(bool c, const Rec<8>::W& a, const Rec<8>::W& b)
{
    return Rec<8>::W{c ? a.ord : b.ord, c ? a.pos : b.pos, 0u};
}
__device__ __forceinline__ KeyIdx<uint64_t> pick(bool c, const KeyIdx<uint64_t>& a, const KeyIdx<uint64_t>& b)
{
    return KeyIdx<uint64_t>{c ? a.k : b.k, c ? a.i : b.i};
}

// (a, b) <- (the smaller, the larger) under `less`; records that `less`
// does not order are identical.  Bare 32-bit words take min and max.
template <typename W, typename Less>
__device__ __forceinline__ void order2(W& a, W& b, Less less)
{
    const bool sw = less(b, a);
    const W lo = pick(sw, b, a), hi = pick(sw, a, b);
    a = lo;
    b = hi;
}
template <typename Less>
__device__ __forceinline__ void order2(uint32_t& a, uint32_t& b, Less)
{
    const uint32_t lo = a < b ? a : b, hi = a < b ? b : a;
    a = lo;
    b = hi;
}

// Sorts the PER records of a lane with a bitonic network.
template <int PER, typename W, typename Less>
__device__ __forceinline__ void lane_sort(W (&x)[PER], Less less)
{
#pragma unroll
    for (int size = 2; size <= PER; size *= 2) {
#pragma unroll
        for (int st = size / 2; st >= 1; st /= 2) {
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int pq = q ^ st;
                if (pq > q) {
                    if ((q & size) == 0)
                        order2(x[q], x[pq], less);
                    else
                        order2(x[pq], x[q], less);
                }
            }
        }
    }
}

// --------------------------------------------------------- wave exchanges --
// The 32-bit register v of lane (lane ^ M) of the wave.  Masks inside a row
// of 16 lanes are DPP moves (no LDS pipe); 16 and 31 swizzle inside 32 lanes;
// 32 and 63 go through ds_bpermute.
template <int M>
__device__ __forceinline__ uint32_t lane_xor32(uint32_t v, int lane)
{
    const int s = (int)v;
    if constexpr (M == 1)
        return (uint32_t)__builtin_amdgcn_mov_dpp(s, 0xB1, 0xF, 0xF, true);  // quad_perm [1,0,3,2]
    else if constexpr (M == 2)
        return (uint32_t)__builtin_amdgcn_mov_dpp(s, 0x4E, 0xF, 0xF, true);  // quad_perm [2,3,0,1]
    else if constexpr (M == 3)
        return (uint32_t)__builtin_amdgcn_mov_dpp(s, 0x1B, 0xF, 0xF, true);  // quad_perm [3,2,1,0]
    else if constexpr (M == 7)
        return (uint32_t)__builtin_amdgcn_mov_dpp(s, 0x141, 0xF, 0xF, true);  // row_half_mirror
    else if constexpr (M == 15)
        return (uint32_t)__builtin_amdgcn_mov_dpp(s, 0x140, 0xF, 0xF, true);  // row_mirror
    else if constexpr (M == 8)
        return (uint32_t)__builtin_amdgcn_mov_dpp(s, 0x128, 0xF, 0xF, true);  // row_ror:8
    else if constexpr (M == 4)
        return lane_xor32<3>(lane_xor32<7>(v, lane), lane);  // (l ^ 7) ^ 3
    else if constexpr (M == 16 || M == 31)
        return (uint32_t)__builtin_amdgcn_ds_swizzle(s, (M << 10) | 0x1F);  // bit mode: l ^ M in 32 lanes
    else {
        static_assert(M == 32 || M == 63, "mask not provided");
        return (uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ M) << 2, s);
    }
}

template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v, int lane)
{
    return lane_xor32<M>(v, lane);
}
template <int M>
__device__ __forceinline__ uint64_t lane_xor(uint64_t v, int lane)
{
    const uint32_t lo = lane_xor32<M>((uint32_t)v, lane);
    const uint32_t hi = lane_xor32<M>((uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}
template <int M>
__device__ __forceinline__ Rec<8>::W lane_xor(const Rec<8>::W& v, int lane)
{
    return Rec<8>::W{lane_xor<M>(v.ord, lane), lane_xor32<M>(v.pos, lane), 0u};
}

// One step of a network across lanes: of this lane's record x and its
// partner's y the lower lane keeps the smaller and the upper the larger one.
// Bare 32-bit words: the median of both and 0 (the smaller) or all ones (the
// larger), one instruction where the compare and the select are two.
template <typename W>
struct LaneSide {
    bool high;
    __device__ __forceinline__ explicit LaneSide(bool h) : high(h) {}
    template <typename Less>
    __device__ __forceinline__ W keep(const W& x, const W& y, Less less) const
    {
        return pick(less(y, x) != high, y, x);
    }
};
template <>
struct LaneSide<uint32_t> {
    uint32_t bound;
    __device__ __forceinline__ explicit LaneSide(bool h) : bound(h ? ~0u : 0u) {}
    template <typename Less>
    __device__ __forceinline__ uint32_t keep(uint32_t x, uint32_t y, Less) const
    {
        uint32_t r;
        asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(y), "v"(bound));
        return r;
    }
};

// Half-cleaner steps of a bitonic merge across lanes: every register of lane
// l meets the same register of lane l ^ M, for M = M0, M0 / 2, ..., 1; the
// lower lane keeps the smaller.
template <int M, int N, typename W, typename Less>
__device__ __forceinline__ void half_clean_lanes(W (&x)[N], int lane, Less less)
{
    if constexpr (M >= 1) {
        // the lower lane takes y when it is smaller, the upper when it is not
        const LaneSide<W> side((lane & M) != 0);
#pragma unroll
        for (int q = 0; q < N; ++q)
            x[q] = side.keep(x[q], lane_xor<M>(x[q], lane), less);
        half_clean_lanes<M / 2>(x, lane, less);
    }
}

// Merge levels of run length L = PER, 2 PER, ..., 32 PER inside one wave,
// in registers: lane l holds records [l PER, (l + 1) PER) of the wave's
// 64 PER, each lane's PER in order on entry, all 64 PER in order on exit.  A
// level pairs runs of L records (L / PER lanes) and merges each pair with a
// bitonic merge: every record of the left run meets its mirror image in the
// right run, then half-cleaners at distances L/2 down to 1 sort both halves.
// Records compare by `less`, under which no two distinct records are equal,
// so the result is the one unique order the LDS merges would give.
template <int PER, int L, typename W, typename Less>
__device__ __forceinline__ void wave_merge_levels(W (&x)[PER], int lane, Less less)
{
    if constexpr (L < 64 * PER) {
        constexpr int G = 2 * L / PER;  // lanes holding one pair of runs
        const LaneSide<W> side((lane & (G / 2)) != 0);
        W y[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q)
            y[q] = lane_xor<G - 1>(x[PER - 1 - q], lane);
#pragma unroll
        for (int q = 0; q < PER; ++q)
            x[q] = side.keep(x[q], y[q], less);
        half_clean_lanes<L / 2 / PER>(x, lane, less);  // distances L/2 .. PER: across lanes
#pragma unroll
        for (int st = PER / 2; st >= 1; st >>= 1) {
#pragma unroll
            for (int q = 0; q < PER; ++q)
                if ((q & st) == 0)
                    order2(x[q], x[q + st], less);
        }
        wave_merge_levels<PER, 2 * L>(x, lane, less);
    }
}

// Number of A elements among the first k outputs of the merge of the sorted
// runs A = src[a0, a0 + L) and B = src[b0, b0 + L) (merge path, A first on
// ties), found by the whole wave: each round the 64 lanes test 64 evenly
// spaced candidates at once and a ballot keeps the interval between the last
// that passes and the first that fails, so runs of up to 4096 take two
// rounds.  Wave-uniform arguments; every lane returns the same value.
template <typename W, typename Less>
__device__ __forceinline__ int wave_merge_path(const W* src, int a0, int b0, int L, int k, int lane, Less less)
{
    int lo = k - L > 0 ? k - L : 0;
    int hi = k < L ? k : L;
    while (lo < hi) {
        const int step = (hi - lo + 63) >> 6;
        const int c = lo + (lane + 1) * step;
        // A[c - 1] goes before B[k - c]: at least c outputs come from A
        const bool pass = c <= hi && !less(src[pad16(b0 + k - c)], src[pad16(a0 + c - 1)]);
        const int t = __popcll(__ballot(pass));  // the passing lanes are a prefix
        lo += t * step;
        hi = hi < lo + step - 1 ? hi : lo + step - 1;
    }
    return lo;
}

// One LDS merge level of a full block, one wave per 64 PER consecutive
// outputs [o, o + 64 PER) of the merge of the pair of runs of length L that
// starts at s (L >= 64 PER).  The wave finds where its outputs start and end
// on both runs (wave_merge_path), loads its A slice ascending followed by its
// B slice descending -- a bitonic sequence -- lane-striped (element e in
// register e / 64 of lane e % 64, so consecutive lanes read consecutive LDS
// words), and sorts it with the half-cleaners of a bitonic merge (distances of
// 64 and more inside the lane, below 64 across lanes): output o + 64 q + lane
// is left in x[q].
template <int PER, typename W, typename Less>
__device__ __forceinline__ void wave_lds_merge(const W* src, W (&x)[PER], int s, int L, int o, int lane, Less less)
{
    constexpr int OUT = 64 * PER;
    const int a0 = s, b0 = s + L;
    const int k = o - s;
    const int i0 = wave_merge_path(src, a0, b0, L, k, lane, less);
    const int i1 = wave_merge_path(src, a0, b0, L, k + OUT, lane, less);
    const int na = i1 - i0;
    const int b_last = b0 + (k + OUT - i1) - 1;  // the B slice's last element
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int e = q * 64 + lane;
        x[q] = src[pad16(e < na ? a0 + i0 + e : b_last - (e - na))];
    }
#pragma unroll
    for (int d = PER / 2; d >= 1; d >>= 1) {  // distances 64 d, inside the lane
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if ((q & d) == 0)
                order2(x[q], x[q + d], less);
    }
    half_clean_lanes<32>(x, lane, less);
}

// Orders the LDS accesses of a wave before and after it (a wave's LDS
// instructions run in program order; this keeps the compiler to that order).
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Sorts the 64 * WAVES * PER records of a group of WAVES consecutive waves,
// any record of the group in any register, through buf[pad16(first)] .. of
// padded LDS records: 64 * PER per wave in registers, then merge levels in
// LDS.  The record of rank r of the group is left in x[q] of the lane with
// r = (wave of the group) * 64 * PER + 64 q + lane.  With WAVES > 1 every
// thread of the workgroup has to call it; the buffer may be used again after a
// barrier (WAVES == 1: after wave_lds_order).
// LOOPED: called in a loop of the caller, where unrolled merge levels and LDS
// addresses kept from one round to the next would cost twice the registers.
template <int WAVES, bool LOOPED, int PER, typename W, typename Less>
__device__ __forceinline__ void sort_striped(W (&x)[PER], W* buf, int first, Less less)
{
    const int tid = (int)(LOOPED ? materialize(threadIdx.x) : threadIdx.x);
    const int lane = tid & (kWave - 1);
    const int o = first + (tid / kWave) % WAVES * kWave * PER;  // the wave's first record
    lane_sort(x, less);
    wave_merge_levels<PER, PER>(x, lane, less);
    if constexpr (PER == 1 && WAVES == 1)
        return;
#pragma unroll
    for (int q = 0; q < PER; ++q)
        buf[pad16(o + lane * PER + q)] = x[q];
    if constexpr (WAVES == 1) {
        wave_lds_order();
#pragma unroll
        for (int q = 0; q < PER; ++q)
            x[q] = buf[pad16(o + q * kWave + lane)];
    } else {
        __syncthreads();
        auto level = [&](int L) {
            wave_lds_merge<PER>(buf, x, first + (o - first) / (2 * L) * (2 * L), L, o, lane, less);
            if (2 * L < WAVES * kWave * PER) {
                __syncthreads();  // every wave has read its records
#pragma unroll
                for (int q = 0; q < PER; ++q)
                    buf[pad16(o + q * kWave + lane)] = x[q];
                __syncthreads();
            }
        };
        if constexpr (LOOPED) {
#pragma unroll 1
            for (int L = kWave * PER; L < WAVES * kWave * PER; L *= 2)
                level(L);
        } else {
#pragma unroll
            for (int L = kWave * PER; L < WAVES * kWave * PER; L *= 2)
                level(L);
        }
    }
}

// Rank, in its group, of the record that sort_striped leaves in x[q] of this
// thread.
template <int WAVES, int PER>
__device__ __forceinline__ int striped_rank(int q, int tid)
{
    return (tid / kWave % WAVES * PER + q) * kWave + (tid & (kWave - 1));
}
template <int WAVES, int PER>
__device__ __forceinline__ int striped_rank(int q)
{
    return striped_rank<WAVES, PER>(q, (int)threadIdx.x);
}

// Where one sort reads and writes.  Values are read from vals_in, or are the
// input positions when iota is set (argsort); keys are not written when
// skip_keys is set.
struct NetworkIo {
    const void* keys_in;
    void* keys_out;
    const void* vals_in;
    void* vals_out;
    bool iota;
    bool skip_keys;
};

// Sorts keys [begin, begin + len) (1 <= len <= 64 * WAVES * PER), stably, into
// the same range of the outputs; the outputs may be the inputs.  One group of
// WAVES waves, as sort_striped.
template <int KB, int VB, int WAVES, int PER, bool LOOPED>
__device__ __forceinline__ void network_sort(const NetworkIo& io, const OrderMap<typename KeyWord<KB>::U>& om,
                                             typename BlockRec<KB, VB>::W* buf, int first, int64_t begin, int len)
{
    using U = typename KeyWord<KB>::U;
    using V = typename ValWord<VB>::T;
    using R = BlockRec<KB, VB>;
    using W = typename R::W;
    const int tid = (int)(LOOPED ? materialize(threadIdx.x) : threadIdx.x);
    const U* keys_in = reinterpret_cast<const U*>(io.keys_in) + begin;
    W x[PER];
    {
        U k[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int i = striped_rank<WAVES, PER>(q, tid);
            k[q] = keys_in[i < len ? i : len - 1];
        }
        // filled up with records above all others
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int i = striped_rank<WAVES, PER>(q, tid);
            x[q] = R::make(i < len ? om.to_order(k[q]) : ~(U)0, (uint32_t)i);
        }
    }
    sort_striped<WAVES, LOOPED>(x, buf, first, [](const W& p, const W& q) { return R::less(p, q); });
    if constexpr (VB != 0) {
        const V* vals_in = reinterpret_cast<const V*>(io.vals_in) + begin;
        V* vals_out = reinterpret_cast<V*>(io.vals_out) + begin;
        V v[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int i = striped_rank<WAVES, PER>(q, tid);
            const uint32_t at = i < len ? R::pos(x[q]) : 0;
            v[q] = io.iota ? (V)(begin + at) : vals_in[at];
        }
        // in place: every value is read before one is written
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        if constexpr (WAVES > 1)
            __syncthreads();
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int i = striped_rank<WAVES, PER>(q, tid);
            if (i < len)
                vals_out[i] = v[q];
        }
    }
    if (!io.skip_keys) {
        U* keys_out = reinterpret_cast<U*>(io.keys_out) + begin;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int i = striped_rank<WAVES, PER>(q, tid);
            if (i < len)
                keys_out[i] = om.from_order((U)R::ord(x[q]));
        }
    }
}

}  // namespace evosort
