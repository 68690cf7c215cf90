// What the kernels work out from a request's prefix length and node count, which come from the caller's device memory and may
// hold any 32-bit value.  Usable on the host as well, so that it can be checked without a GPU.
#pragma once

namespace specvlm {

constexpr int kSharesRound = 128;   // keys that the four streams of a workgroup take at once (attn_streams.hip)

// Keys of a request, 1 .. capacity whatever its lengths are (a bad request takes part in the division of a batch until it is reported).
constexpr int keys_of(int prefix, int nodes, int nodes_max, int capacity) {
    const int P = prefix < 0 ? 0 : prefix > capacity ? capacity : prefix;
    const int n = nodes < 1 ? 1 : nodes > nodes_max ? nodes_max : nodes;
    return n < capacity - P ? P + n : capacity;            // (P + n of the caller's values may not fit in 32 bits)
}

// Whether a request's prefix and its `nodes` nodes (1 .. 64) lie inside the cache (their sum may not fit in 32 bits).
constexpr bool length_fits(int prefix, int nodes, int capacity) { return prefix >= 0 && prefix <= capacity - nodes; }

// Whether row `node` behind the prefix is a slot of the cache (prefix + node may not fit in 32 bits).
constexpr bool slot_inside(int prefix, int node, int capacity) { return prefix >= 0 && node >= 0 && prefix < capacity - node; }

// ceil(rounds / len), inverse = 1 / len to a few ulp
constexpr int columns_of(int rounds, float len, float inverse) { return static_cast<int>((static_cast<float>(rounds) - 0.5f + len) * inverse); }

// A column a request (attn_streams.hip): the workgroups of the requests up to the mean read rounds of the longest one ahead, each as many as it
// is shorter than the mean, one at least; nothing where the longest has less than two rounds beyond the mean.  These rounds follow one
// another in the order of the requests from first_read_ahead() on, up to the longest request's end and kMostReadAhead at most.
constexpr int kMostReadAhead = 8;   // 64 KB each, of four or five heads on an XCD
constexpr int rounds_read_ahead(int rounds, int longest, int mean) { return longest - mean < 2 || rounds > mean ? 0 : mean - rounds > 1 ? mean - rounds : 1; }
constexpr int first_read_ahead(int longest, int all) { return longest - all > 2 ? longest - all : 2; }

}  // namespace specvlm
