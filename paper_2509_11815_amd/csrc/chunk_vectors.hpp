// A chunk of a row's entries as 16-byte vectors.  Index arithmetic only, so that it can be checked on the host.
#pragma once
#include <cstdint>

#ifdef __HIP__
#define SPECVLM_HOST_DEVICE __host__ __device__
#else
#define SPECVLM_HOST_DEVICE
#endif

namespace specvlm {

// Entries [v0, v1) of a row of V that starts at address `row` (aligned to an entry), `vec` entries per vector, v0 < v1.
// Vector k starts at entry v0 - lead + k vec, on a 16-byte boundary.  Vectors 0 .. count - 1 hold the chunk; of these
// only lo .. hi lie inside the row as a whole: the first of a row and the last may not, their entries are loaded one
// by one.
struct ChunkVectors {
    int lead, count, lo, hi;
    SPECVLM_HOST_DEVICE ChunkVectors(uintptr_t row, int v0, int v1, int V, int vec) {
        const int entry = 16 / vec;
        lead = static_cast<int>(((row + static_cast<uintptr_t>(v0) * entry) & 15) / entry);
        const int first = v0 - lead;
        count = (lead + v1 - v0 + vec - 1) / vec;
        lo = first < 0 ? 1 : 0;
        const int whole = (V - first) / vec;
        hi = (whole < count ? whole : count) - 1;
    }
};

}  // namespace specvlm
