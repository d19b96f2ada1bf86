// One-workgroup sort for arrays below the fallback threshold (the branch of
// Sec. 4.3, Algorithm 6 that hands small arrays to the platform's own sort).
//
// One launch of one workgroup, with the workgroup shape picked by the array
// length.  Up to 4096 keys, and up to 8192 without values, they are sorted in
// registers with bitonic merges across lanes, and merged in LDS
// (wave_merge.hpp); above, by the one-workgroup LSD radix sort (8-bit digits),
// whose work per key does not grow with the length.  Keys, values or indices
// stay in registers and LDS all the time.  Stable, like every routine here.
// Bound by latency; us per call, LSD sort / networks: int32 1000 keys 8.6 / 4.3
// (kernel alone), 8192 21.3 / 14.6; int64 2000 keys 26.9 / 9.6; int32 pairs
// 4096 17.2 / 15.5, 6000 20.6 / 26.7 (kept on the LSD sort).
#include "block_lsd.hpp"
#include "common.hpp"
#include "small_sort.hpp"
#include "wave_merge.hpp"

namespace evosort {

namespace {

// Workgroup shapes of the networks: waves and records per thread.
struct NetShape {
    int waves;
    int per;
};
constexpr int kNetShapeCount = 5;
constexpr NetShape kNetShapes[kNetShapeCount] = {{4, 1}, {4, 4}, {8, 4}, {16, 4}, {16, 8}};
template <int KB, int VB>
constexpr int net_shapes()
{
    return VB == 0 ? kNetShapeCount : kNetShapeCount - 1;
}

// Workgroup shapes of the LSD sort; the last one holds the capacity.
struct SmallShape {
    int threads;
    int items;
};
constexpr int kSmallShapeCount = 2;
// 4-byte keys, and 8-byte keys without values
constexpr SmallShape kSmallShapes[kSmallShapeCount] = {{1024, 8}, {1024, 16}};
// 8-byte keys with values or indices (registers: 16 keys and 16 values per thread need 512 threads)
constexpr SmallShape kSmallShape8V{512, 16};
static_assert(1024 * 16 == kSmallCapacity && 512 * 16 == kSmallCapacity8V, "the largest shape holds the capacity");

// Keys and values share the staging area unless that would not fit in LDS.
template <int KB, int VB, int THREADS, int ITEMS>
constexpr bool split_staging()
{
    return (size_t)THREADS * ITEMS * (KB + VB) > 128 * 1024;
}

template <int KB, int VB, int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void small_sort_kernel(SmallSortArgs a, OrderMap<typename KeyWord<KB>::U> om)
{
    constexpr bool SPLIT = split_staging<KB, VB, THREADS, ITEMS>();
    __shared__ BlockLsdLds<KB, VB, THREADS, ITEMS, SPLIT> L;
    const bool argsort = a.mode == SMALL_MODE_ARGSORT;
    if (a.error_word && threadIdx.x == 0)
        *a.error_word = 0;
    const BlockLsdIo io{a.keys_in, a.keys_out, a.vals_in, a.vals_out, argsort, argsort};
    block_lsd_sort<KB, VB, THREADS, ITEMS, SPLIT>(io, om, L, 0, (uint32_t)a.n);
}

template <int KB, int VB, int THREADS, int ITEMS>
hipError_t launch_shape(const KeyDesc& kd, const SmallSortArgs& a, hipStream_t s)
{
    using U = typename KeyWord<KB>::U;
    static_assert(sizeof(BlockLsdLds<KB, VB, THREADS, ITEMS, split_staging<KB, VB, THREADS, ITEMS>()>) <=
                      160 * 1024,
                  "one workgroup fits in one CU's LDS");
    OrderMap<U> om{(U)kd.flip, (U)kd.neg, (U)kd.desc};
    hipLaunchKernelGGL((small_sort_kernel<KB, VB, THREADS, ITEMS>), dim3(1), dim3(THREADS), 0, s, a, om);
    return hipGetLastError();
}

template <int KB, int VB, int WAVES, int PER>
__global__ __launch_bounds__(WAVES* kWave) void small_network_kernel(SmallSortArgs a,
                                                                     OrderMap<typename KeyWord<KB>::U> om)
{
    __shared__ typename BlockRec<KB, VB>::W buf[padded16(WAVES * kWave * PER)];
    const bool argsort = a.mode == SMALL_MODE_ARGSORT;
    if (a.error_word && threadIdx.x == 0)
        *a.error_word = 0;
    const NetworkIo io{a.keys_in, a.keys_out, a.vals_in, a.vals_out, argsort, argsort};
    network_sort<KB, VB, WAVES, PER, false>(io, om, buf, 0, 0, (int)a.n);
}

// The first shape, from index I on, that holds n keys: the networks', then the
// LSD sort's.
template <int KB, int VB, int I>
hipError_t launch_t(const KeyDesc& kd, const SmallSortArgs& a, hipStream_t s)
{
    if constexpr (I < net_shapes<KB, VB>()) {
        constexpr NetShape sh = kNetShapes[I];
        if (a.n > (int64_t)sh.waves * kWave * sh.per)
            return launch_t<KB, VB, I + 1>(kd, a, s);
        using U = typename KeyWord<KB>::U;
        OrderMap<U> om{(U)kd.flip, (U)kd.neg, (U)kd.desc};
        hipLaunchKernelGGL((small_network_kernel<KB, VB, sh.waves, sh.per>), dim3(1), dim3(sh.waves * kWave), 0, s, a,
                           om);
        return hipGetLastError();
    } else if constexpr (KB == 8 && VB != 0) {
        return launch_shape<KB, VB, kSmallShape8V.threads, kSmallShape8V.items>(kd, a, s);
    } else {
        constexpr int J = I - net_shapes<KB, VB>();
        constexpr SmallShape sh = kSmallShapes[J];
        if constexpr (VB != 0 && J + 1 < kSmallShapeCount) {
            if (a.n > (int64_t)sh.threads * sh.items)
                return launch_t<KB, VB, I + 1>(kd, a, s);
            return launch_shape<KB, VB, sh.threads, sh.items>(kd, a, s);
        } else {  // without values the networks hold as many keys as the first shape
            constexpr SmallShape last = kSmallShapes[kSmallShapeCount - 1];
            return launch_shape<KB, VB, last.threads, last.items>(kd, a, s);
        }
    }
}

}  // namespace

int64_t small_sort_capacity(int key_bytes, int val_bytes)
{
    return key_bytes == 8 && val_bytes != 0 ? kSmallCapacity8V : kSmallCapacity;
}

hipError_t launch_small_sort(const KeyDesc& kd, int val_bytes, const SmallSortArgs& a, hipStream_t s)
{
    if (a.n < 0 || a.n > small_sort_capacity(kd.bytes, val_bytes))
        return hipErrorInvalidValue;
    if (a.n == 0)
        return hipSuccess;
    if (kd.bytes == 4) {
        if (val_bytes == 0)
            return launch_t<4, 0, 0>(kd, a, s);
        if (val_bytes == 4)
            return launch_t<4, 4, 0>(kd, a, s);
        return launch_t<4, 8, 0>(kd, a, s);
    }
    if (val_bytes == 0)
        return launch_t<8, 0, 0>(kd, a, s);
    if (val_bytes == 4)
        return launch_t<8, 4, 0>(kd, a, s);
    return launch_t<8, 8, 0>(kd, a, s);
}

}  // namespace evosort
