// One-workgroup sort of the small segments of a batched segmented sort.
//
// A segment of a class is sorted by one wave (up to 512 keys), or by one
// workgroup: in registers, with bitonic merges across lanes, and above 512 keys
// with merge levels in LDS (wave_merge.hpp), so HBM sees one read and one write
// per key.  Bound by the VALU work of the networks (1.8e3-key segments, uint32,
// 1e8 keys in all: a one-workgroup LSD sort by 8-bit digits here took 1.09 ms).
// Networks here also with values above 4096 records, where a single array goes
// to the LSD sort (small_sort.hip): many workgroups at once are bound otherwise
// than one alone.  Whole calls, LSD sort / networks, 3e7 int32 keys with 4-byte
// values in segments of 4000 keys 911 / 768 us, 5000 778 / 829, 6000 684 / 709,
// 8000 695 / 592 (8192 records are sorted from 4097 keys on).
// Waves and workgroups take their class's segments at a fixed stride: taking
// them from a ticket counter costs about 12 ns per segment, since atomics on one
// word are performed one after the other (1e6 segments of 100 keys: 11.7 ms).
//
// Compiled once per (key bytes, value bytes) pair with -DEVOSORT_KB/-DEVOSORT_VB.
#include "common.hpp"
#include "segmented.hpp"
#include "wave_merge.hpp"

#ifndef EVOSORT_KB
#error "EVOSORT_KB must be defined"
#endif
#ifndef EVOSORT_VB
#error "EVOSORT_VB must be defined"
#endif

#define EVOSORT_CAT4(a, b, c, d) a##b##c##d
#define EVOSORT_XCAT4(a, b, c, d) EVOSORT_CAT4(a, b, c, d)
#define EVOSORT_NAME(kb, vb) EVOSORT_XCAT4(seg_block_dispatch_k, kb, _v, vb)

namespace evosort {

namespace {

constexpr int kWaveClassKeys = 512;  // class 0: one wave per segment

// Workgroup of a class's kernel: waves, and records per thread of a segment
// that fills the class.
struct SegGroup {
    int waves;
    int per;
};
constexpr SegGroup seg_group(int64_t capacity, size_t record)
{
    return capacity <= kWaveClassKeys ? SegGroup{4, 8}
           : capacity <= 2048         ? SegGroup{4, 8}
           : capacity <= 4096         ? SegGroup{8, 8}
           : capacity <= 8192         ? (record <= 4 ? SegGroup{8, 16} : SegGroup{16, 8})
                                      : SegGroup{16, 16};
}

template <int KB, int VB>
__global__ __launch_bounds__(4 * kWave) void seg_wave_sort_kernel(SegBlockArgs a, OrderMap<typename KeyWord<KB>::U> om)
{
    using W = typename BlockRec<KB, VB>::W;
    __shared__ W buf[4 * padded16(kWaveClassKeys)];
    const NetworkIo io{a.keys_in, a.keys_out, a.vals_in, a.vals_out, false, false};
    const uint32_t count = *a.count;
    const int w = (int)(threadIdx.x / kWave);
    W* mine = buf + w * padded16(kWaveClassKeys);
    const uint32_t step = gridDim.x * 4;
    uint32_t j = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (uint32_t)w));
    if (j >= count)
        return;
    uint32_t seg = a.list[j];
    int64_t begin = a.offsets[seg], end = a.offsets[seg + 1];
    for (;;) {
        // the next segment's bounds are on their way while this one is sorted
        const uint32_t next = step < count - j ? j + step : j;
        const uint32_t nseg = a.list[next];
        const int64_t nbegin = a.offsets[nseg], nend = a.offsets[nseg + 1];
        const int len = __builtin_amdgcn_readfirstlane((int)(end - begin));
        const int64_t b = (int64_t)uniform((uint64_t)begin);
        if (len <= 64)
            network_sort<KB, VB, 1, 1, true>(io, om, mine, 0, b, len);
        else if (len <= 128)
            network_sort<KB, VB, 1, 2, true>(io, om, mine, 0, b, len);
        else if (len <= 256)
            network_sort<KB, VB, 1, 4, true>(io, om, mine, 0, b, len);
        else
            network_sort<KB, VB, 1, 8, true>(io, om, mine, 0, b, len);
        if (next == j)
            return;
        wave_lds_order();  // the buffer is used again
        j = next;
        begin = nbegin;
        end = nend;
    }
}

// (1024 threads: two workgroups per CU need 64 registers)
template <int KB, int VB, int WAVES, int PER>
__global__ __launch_bounds__(WAVES* kWave, WAVES == 16 ? 8 : 1) void seg_block_sort_kernel(
    SegBlockArgs a, OrderMap<typename KeyWord<KB>::U> om)
{
    using W = typename BlockRec<KB, VB>::W;
    __shared__ W buf[padded16(WAVES * kWave * PER)];
    const NetworkIo io{a.keys_in, a.keys_out, a.vals_in, a.vals_out, false, false};
    const uint32_t count = *a.count;
    uint32_t j = blockIdx.x;
    if (j >= count)
        return;
    uint32_t seg = a.list[j];
    int64_t begin = a.offsets[seg], end = a.offsets[seg + 1];
    for (;;) {
        // the next segment's bounds are on their way while this one is sorted
        const uint32_t next = gridDim.x < count - j ? j + gridDim.x : j;
        seg = a.list[next];
        const int64_t nbegin = a.offsets[seg], nend = a.offsets[seg + 1];
        const int64_t b = (int64_t)uniform((uint64_t)begin);
        const int len = __builtin_amdgcn_readfirstlane((int)(end - begin));
        if (len <= WAVES * kWave * PER / 2)
            network_sort<KB, VB, WAVES, PER / 2, true>(io, om, buf, 0, b, len);
        else
            network_sort<KB, VB, WAVES, PER, true>(io, om, buf, 0, b, len);
        if (next == j)
            return;
        __syncthreads();  // the buffer is used again
        j = next;
        begin = nbegin;
        end = nend;
    }
}

template <int CLS>
hipError_t launch_class(const KeyDesc& kd, const SegBlockArgs& a, uint32_t max_segments, hipStream_t s)
{
    constexpr int RB = EVOSORT_KB + EVOSORT_VB;
    constexpr int64_t CAP = seg_class_capacity(RB, CLS);
    using U = typename KeyWord<EVOSORT_KB>::U;
    using W = typename BlockRec<EVOSORT_KB, EVOSORT_VB>::W;
    constexpr SegGroup g = seg_group(CAP, sizeof(W));
    constexpr bool WAVE = CAP <= kWaveClassKeys;
    static_assert(WAVE ? CAP <= kWaveClassKeys : CAP <= (int64_t)g.waves * kWave * g.per, "the class fits the group");
    static_assert(sizeof(W) * padded16(g.waves * kWave * g.per) <= 80 * 1024,
                  "two workgroups of a class fit in one CU's LDS");
    auto kernel = [] {
        if constexpr (WAVE)
            return seg_wave_sort_kernel<EVOSORT_KB, EVOSORT_VB>;
        else
            return seg_block_sort_kernel<EVOSORT_KB, EVOSORT_VB, g.waves, g.per>;
    }();
    static int resident = 0;  // one per instantiation
    if (resident == 0) {
        int dev = 0, cus = 0, per_cu = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, g.waves * kWave, 0) == hipSuccess && cus > 0 &&
            per_cu > 0)
            resident = cus * per_cu;
        else {
            (void)hipGetLastError();
            resident = 1024;  // any grid is correct; this only sizes the persistent launch
        }
    }
    const uint32_t want = WAVE ? seg_wave_groups(max_segments) : max_segments;
    const uint32_t grid = want < (uint32_t)resident ? want : (uint32_t)resident;
    if (grid == 0)
        return hipSuccess;
    OrderMap<U> om{(U)kd.flip, (U)kd.neg, (U)kd.desc};
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(g.waves * kWave), 0, s, a, om);
    return hipGetLastError();
}

}  // namespace

hipError_t EVOSORT_NAME(EVOSORT_KB, EVOSORT_VB)(int cls, const KeyDesc& kd, const SegBlockArgs& a,
                                                 uint32_t max_segments, hipStream_t s)
{
    constexpr int classes = seg_class_count(EVOSORT_KB + EVOSORT_VB);
    switch (cls) {
    case 0:
        return launch_class<0>(kd, a, max_segments, s);
    case 1:
        return launch_class<1>(kd, a, max_segments, s);
    case 2:
        return launch_class<2>(kd, a, max_segments, s);
    case 3:
        if constexpr (classes > 3)
            return launch_class<3>(kd, a, max_segments, s);
        return hipErrorInvalidValue;
    default:
        return hipErrorInvalidValue;
    }
}

}  // namespace evosort
