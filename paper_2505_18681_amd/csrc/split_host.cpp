// Shape and dispatch of the splitter sort.
#include "split_sort.hpp"

namespace evosort {

#define EVOSORT_SPLIT_DECL(KB, VB)                                                        \
    hipError_t split_blocks_k##KB##_v##VB(const KeyDesc&, const SplitArgs&, hipStream_t); \
    hipError_t split_buckets_k##KB##_v##VB(const KeyDesc&, const SplitArgs&, hipStream_t);
EVOSORT_SPLIT_DECL(4, 0)
EVOSORT_SPLIT_DECL(4, 4)
EVOSORT_SPLIT_DECL(4, 8)
EVOSORT_SPLIT_DECL(8, 0)
EVOSORT_SPLIT_DECL(8, 4)
EVOSORT_SPLIT_DECL(8, 8)
#undef EVOSORT_SPLIT_DECL

SplitPlan split_plan(int64_t n)
{
    SplitPlan p{};
    p.block_keys = 512;
    while ((n + p.block_keys - 1) / p.block_keys > kSplitBlocksMost && p.block_keys < 2048)
        p.block_keys *= 2;
    p.blocks = (uint32_t)((n + p.block_keys - 1) / p.block_keys);
    p.samples = n <= 131072 ? 1024 : 2048;
    // Buckets of 384 keys on average, so that few have more than the 1024 that
    // four records per thread hold, and at least three (four) samples each.
    const int64_t want = (n + 383) / 384, most = p.samples == 1024 ? 341 : 512;
    p.buckets = (uint32_t)(want < most ? want : most);
    return p;
}

#define EVOSORT_SPLIT_CALL(what)                             \
    if (kd.bytes == 4)                                       \
        return val_bytes == 0   ? what##_k4_v0(kd, a, s)     \
               : val_bytes == 4 ? what##_k4_v4(kd, a, s)     \
                                : what##_k4_v8(kd, a, s);    \
    return val_bytes == 0   ? what##_k8_v0(kd, a, s)         \
           : val_bytes == 4 ? what##_k8_v4(kd, a, s)         \
                            : what##_k8_v8(kd, a, s);

hipError_t launch_split_blocks(const KeyDesc& kd, int val_bytes, const SplitArgs& a, hipStream_t s)
{
    EVOSORT_SPLIT_CALL(split_blocks)
}

hipError_t launch_split_buckets(const KeyDesc& kd, int val_bytes, const SplitArgs& a, hipStream_t s)
{
    EVOSORT_SPLIT_CALL(split_buckets)
}
#undef EVOSORT_SPLIT_CALL

}  // namespace evosort
