// Whether a draft level with its selection gives every row a second workgroup, for its log-sum-exp.  Host arithmetic only, so that it can
// be checked without a GPU.
#pragma once
#include <cstdint>

#include "specvlm.h"

namespace specvlm {

// As long as all workgroups are resident at once and a request's log-sum-exps fit behind its counter.  Not the root's row of up to 65536
// entries, which needs no meeting otherwise (32000 5.6 us, 6.3 with one; 100001 14.8, 11.9).  The row is then read twice, by two compute units:
// what that costs grows with the rows and their bytes, most where the second reading is fp32 and does not end in registers.  Time of two
// workgroups a row over one, logits in cache (a level in a graph; from HBM the line lies 10 - 30 rows further on):
//   rows            10     40     50     60     80    100    120    128
//   bf16  32000    0.88   0.90   0.89   0.91   0.91   0.92   0.91   0.91
//         65000    0.87   0.88   0.88   0.87   0.88   0.85   0.91   1.05
//        100001    0.83   0.84   0.85   0.85   0.88   0.95   1.01   1.04
//        250000    0.73   0.76   0.77   0.77   0.81   0.92   0.98   1.02
//   fp32  32000    0.88   0.91   0.90   0.91   0.92   0.92   0.98   1.03
//         65000    0.85   0.89   0.99   1.05   1.13   1.32   1.42   1.42
//         65537    0.84   0.85   0.85   0.87   1.09   1.22   1.32   1.31
//        152064    0.86   0.96   0.98   1.01   1.17   1.29   1.41   1.44
//        250000    0.76   0.95   1.01   1.09   1.19   1.29   1.38   1.47
inline bool sums_beside(int32_t dtype, int64_t B, int32_t W, int32_t V, bool root) {
    if (W >= SPECVLM_COUNTER_STRIDE || (root && W == 1 && V <= 65536)) return false;
    const int64_t rows = B * W;
    if (dtype == SPECVLM_BF16) return rows <= (V <= 65536 ? 120 : 110);
    return V <= 65536 ? rows <= 128 && rows * V <= 2200000 : rows <= 50;
}

}  // namespace specvlm
