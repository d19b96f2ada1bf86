// Copies on the device, and what the last launch of a routed radix sort does.
#pragma once

#include "common.hpp"
#include "kernels.hpp"

namespace evosort {

// bytes is a multiple of 4 (keys, values and indices are 4 or 8 bytes).
__device__ __forceinline__ void copy_range(unsigned char* __restrict__ dst, const unsigned char* __restrict__ src,
                                           size_t bytes, size_t tid, size_t nthreads)
{
    size_t done = 0;
    if (((reinterpret_cast<uintptr_t>(dst) | reinterpret_cast<uintptr_t>(src)) & 15) == 0) {
        const size_t n16 = bytes / 16;
        uint4* d = reinterpret_cast<uint4*>(dst);
        const uint4* s = reinterpret_cast<const uint4*>(src);
        size_t i = tid;
        // eight 16-byte words in flight per thread
        for (; i + 7 * nthreads < n16; i += 8 * nthreads) {
            const uint4 w0 = s[i], w1 = s[i + nthreads], w2 = s[i + 2 * nthreads], w3 = s[i + 3 * nthreads];
            const uint4 w4 = s[i + 4 * nthreads], w5 = s[i + 5 * nthreads], w6 = s[i + 6 * nthreads],
                        w7 = s[i + 7 * nthreads];
            // every load is issued before the first store: the scheduler
            // would otherwise pair each load with its store and wait on each
            __builtin_amdgcn_sched_barrier(0);
            d[i] = w0;
            d[i + nthreads] = w1;
            d[i + 2 * nthreads] = w2;
            d[i + 3 * nthreads] = w3;
            d[i + 4 * nthreads] = w4;
            d[i + 5 * nthreads] = w5;
            d[i + 6 * nthreads] = w6;
            d[i + 7 * nthreads] = w7;
        }
        for (; i < n16; i += nthreads)
            d[i] = s[i];
        done = n16 * 16;
    }
    uint32_t* d4 = reinterpret_cast<uint32_t*>(dst + done);
    const uint32_t* s4 = reinterpret_cast<const uint32_t*>(src + done);
    for (size_t i = tid; i < (bytes - done) / 4; i += nthreads)
        d4[i] = s4[i];
}

// After the passes of a routed sort (see RadixRoute): with no live pass, the
// input goes to the output unchanged (argsort: the identity permutation);
// with an odd number of live passes sorted in place, the last pass's
// temporary buffer goes to the output; otherwise every workgroup leaves.
// (m: stages of the plan; tid of nth threads in the launch)
__device__ __forceinline__ void finish_copies(const RadixRoute& r, uint32_t m, int64_t n, int kb, int vb, size_t tid,
                                              size_t nth)
{
    const bool argsort = (r.flags & ROUTE_ARGSORT) != 0;
    if (m == 0) {
        if (argsort) {
            if (vb == 4) {
                for (size_t i = tid; i < (size_t)n; i += nth)
                    reinterpret_cast<uint32_t*>(r.vals_out)[i] = (uint32_t)i;
            } else {
                for (size_t i = tid; i < (size_t)n; i += nth)
                    reinterpret_cast<uint64_t*>(r.vals_out)[i] = (uint64_t)i;
            }
            return;
        }
        if (r.keys_out != r.keys_in)
            copy_range(reinterpret_cast<unsigned char*>(r.keys_out), reinterpret_cast<const unsigned char*>(r.keys_in),
                       (size_t)n * kb, tid, nth);
        if (vb && r.vals_out != r.vals_in)
            copy_range(reinterpret_cast<unsigned char*>(r.vals_out), reinterpret_cast<const unsigned char*>(r.vals_in),
                       (size_t)n * vb, tid, nth);
        return;
    }
    if (!argsort && (r.flags & ROUTE_COPY_IF_ODD) && (m & 1)) {
        copy_range(reinterpret_cast<unsigned char*>(r.keys_out), reinterpret_cast<const unsigned char*>(r.keys_tmp),
                   (size_t)n * kb, tid, nth);
        if (vb)
            copy_range(reinterpret_cast<unsigned char*>(r.vals_out), reinterpret_cast<const unsigned char*>(r.vals_tmp),
                       (size_t)n * vb, tid, nth);
    }
}

}  // namespace evosort
