// How many KV heads a workgroup of the compaction takes.  Host arithmetic only, so that it can be checked without a GPU.
#pragma once
#include <cstdint>

namespace specvlm {

constexpr int kCompactThreads = 256;
constexpr int kCompactChunksPerThread = 8;   // 16-byte chunks: 64 rows * 32 chunks / 256 threads

// log2 of the heads per workgroup.  `workgroups`: those of one head each; `head_chunks`: 16-byte chunks of one head's rows, a whole
// path of them.  Fewer workgroups always pay where there are many (8192 and more); with fewer of them, what one workgroup has to move
// is what the call waits for once the paths are long.  us by heads per workgroup (1 | 2 | 4 | 8), every row of the path moved:
//   2048 workgroups, 112 chunks 5.25 | 4.71 | 5.07 | 5.48; 320: 6.48 | 6.45 | 7.09; 512: 7.67 | 7.76 | 9.09; 640: 7.89 | 8.16
//   4096             128        7.36 | 5.85 | 5.93 | 6.47; 320: 9.42 | 8.70 | 8.84; 640: 13.25 | 12.63; 1024, a third of the rows: 10.63 | 9.69
//   1024             320        4.65 | 4.67 | 5.51;        512: 5.69 | 6.11 | 7.81; 640: 5.82 | 6.37
//   8192             128        11.1 | 8.38 | 7.83 | 8.08; 320: 14.6 | 13.97 | 13.38
// (Up to 2048 chunks at any number from 512 workgroups on: 80 layers and tensors x 2 requests x 8 heads of 1024 chunks 10.6 -> 12.7.)
inline int compact_head_bits(int64_t workgroups, int head_chunks) {
    int bits = 0;
    while (bits < 3) {
        const int64_t chunks = static_cast<int64_t>(head_chunks) << (bits + 1);
        if (workgroups >> (bits + 1) < 512 || chunks > kCompactThreads * kCompactChunksPerThread) break;
        if (workgroups < 8192 && chunks > workgroups / (bits ? 8 : 2)) break;
        ++bits;
    }
    return bits;
}

}  // namespace specvlm
