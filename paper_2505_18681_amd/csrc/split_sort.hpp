// Splitter sort of mid-size arrays (host-visible part).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "kernels.hpp"

namespace evosort {

constexpr int kSplitBucketMost = 2048;  // keys one bucket step sorts
constexpr int kSplitBlocksMost = 256;   // blocks: one thread of a bucket's workgroup each
constexpr int kSplitGroupKeys = 2048;   // keys per workgroup of the blocks kernel: one or more blocks
constexpr int kSplitRow = 32;           // entries of a block's index row

// Shape of one splitter sort.
struct SplitPlan {
    uint32_t block_keys;  // 512, 1024 or 2048
    uint32_t blocks;
    uint32_t samples;     // 1024 or 2048, at most n
    uint32_t buckets;
};
SplitPlan split_plan(int64_t n);

struct SplitArgs {
    const void* keys_in;
    void* keys_out;       // null for argsort
    const void* vals_in;  // pairs only; argsort: the values are the input positions
    void* vals_out;       // values or indices
    void* keys_tmp;       // n order words, room for a multiple of kSplitGroupKeys
    void* vals_tmp;       // n values or indices
    void* rows;           // kSplitRow order words per block: the last key of each 1 / kSplitRow of the block
    void* splitters;      // 16 bytes per bucket
    int64_t n;
    SplitPlan plan;
    bool iota;
    uint32_t* error_word;  // cleared (no device-side error can occur here); may be null
};
hipError_t launch_split_blocks(const KeyDesc& kd, int val_bytes, const SplitArgs& a, hipStream_t s);
hipError_t launch_split_buckets(const KeyDesc& kd, int val_bytes, const SplitArgs& a, hipStream_t s);

}  // namespace evosort
