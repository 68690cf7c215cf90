// How a bf16 verification call is divided among workgroups.  Host arithmetic only, so that it can be checked
// without a GPU.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>

#include "specvlm.h"

namespace specvlm {

constexpr int kTile = 32;           // keys per tile
constexpr int kStreamsPerWg = 2;    // key streams of a workgroup that takes all query rows of a head
constexpr int kMostTwoPerCu = 512;  // work items that the launch shape with two workgroups per compute unit holds at once
constexpr int kMaxSplitHeads = 1024;  // (request, head) pairs a split call can have: one set of ticket counters each

// Key-range splits per (request, head) when the caller leaves the choice to the library: the
// count that minimises a small cost model of the kernel on 256 compute units, one workgroup
// each.  A workgroup costs a fixed prologue + merge time plus one step per 32-key tile of its
// longest stream; a step takes the measured time of the loop body with two tiles in flight
// (the same with 160 or 256 units active), or the workgroup's share of HBM bandwidth if that
// is slower; workgroups beyond 256 run as further rounds.  The cache capacity stands in for
// the request lengths, which the host does not know.
inline int32_t single_round_ranges(const specvlm_attn_desc& d) {
    const int64_t heads = static_cast<int64_t>(d.B) * d.H_q;
    if (heads > kMaxSplitHeads) return 1;      // more (request, head) pairs than ticket counters: that many fill the chip unsplit
    if (d.num_splits > 0) return std::min(d.num_splits, 64);
    const int cus = 256;
    const int bh = d.B * d.H_q;
    const int cap = d.paged ? d.max_blocks_per_req * SPECVLM_PAGE_SIZE : d.kv_capacity;
    const int ntile = (cap + kTile - 1) / kTile;
    const double step_bytes = static_cast<double>(kStreamsPerWg) * kTile * d.D * 2 * 2;   // K and V, bf16
    const double bw = 6.0e6;                                     // bytes per microsecond the loop sustains
    const double step_alone = d.D == 128 ? 1.35 : 0.9;           // microseconds per step of one compute unit by itself
    auto wg_time = [&](int splits, int active) {
        const int steps = (ntile + kStreamsPerWg * splits - 1) / (kStreamsPerWg * splits);
        const double step = std::fmax(step_alone, step_bytes * active / bw);
        return (splits > 1 ? 8.0 : 5.0) + steps * step;
    };
    const int most = std::max(1, std::min(64, ntile / kStreamsPerWg));     // never a stream without a whole tile
    int best = 1;
    double best_t = 1e30;
    for (int s = 1; s <= most; ++s) {
        const long wgs = static_cast<long>(bh) * s;
        const long full = wgs / cus;
        const int rest = static_cast<int>(wgs % cus);
        const double t = full * wg_time(s, cus) + (rest ? wg_time(s, rest) : 0.0);
        if (t < best_t * 0.999) { best_t = t; best = s; }
    }
    return best;
}

// How a call is divided among workgroups: query rows and key ranges, or key ranges only.
//
// With few (request, head) pairs the chip can be filled in two ways.  Key ranges (attn_mfma.hip):
// every workgroup takes all 64 query rows, K and V are fetched once, and the 2 - 64 partial results
// of a head meet at the end.  Query rows as well (attn_wave.hip): workgroups of 16 or 32 rows, whose
// K and V come from L2 for all but the first of a head's row blocks, with a quarter or half of the
// arithmetic each, so that fewer or no partial results have to meet, and those are a quarter or half the size.
// As the kernels are now (us; 1 x 32 heads x 128, 60 nodes, on 256 workgroups; by key ranges 8, 32 rows 4, 16 rows 2 ranges):
//   keys        828   1160   1660   2160   2660   3060   3324   3660   4060   4560
//   key ranges 11.1   12.0   13.0   13.8   14.9   15.2   16.3   17.2   17.6   18.6
//   32 rows     8.9   10.1   10.7   12.2   13.7   14.5   15.5   17.0   17.6   18.9
//   16 rows     9.3          13.0   15.6   17.9   19.9   20.6   22.7   24.7   26.5
// so rows win until the repeated K and V traffic (at most ~14 TB/s from L2) costs more than the merge.  plan_rows() was fitted to earlier forms of
// the kernels (it crosses near 3300 keys, and near 2100, where it counts seven ranges); fit_rows() below puts that right for head size 128 in one
// round of workgroups with up to 16 ranges.  Elsewhere (head size 64, more rounds or ranges) plan_rows() decides alone, and its choice has not been
// measured against the kernels as they are.
struct AttnPlan {
    int32_t ranges;        // key ranges per head that the workspace holds
    int32_t block_rows;    // query rows per workgroup, 0: all (key ranges only)
    int32_t splits;        // key ranges the call takes, <= ranges
    int32_t streams = 0;   // key ranges of a request in the kernel with four streams per workgroup (attn_streams.hip) when it divides evenly, <= ranges; 0: that is another kernel's
    int32_t columns = 0;   // workgroups of the kernel with four streams per row block of a KV head, all requests together: it takes the call; 0: one of the others
    int32_t by_length = 0; // the columns are dealt out to the requests by their lengths, on the device
};

inline AttnPlan plan_rows(const specvlm_attn_desc& d, int32_t nominal) {
    const int cus = 256;
    const int group = d.H_q / d.H_kv, rows = group * d.N_max;
    const int cap = d.paged ? d.max_blocks_per_req * SPECVLM_PAGE_SIZE : d.kv_capacity;
    const int ntile = (cap + kTile - 1) / kTile;
    const double half = d.D == 128 ? 1.0 : 0.5;            // tile size relative to head size 128
    auto rounds_of = [&](double items, auto&& one) {       // us of `items` workgroups, 256 at a time
        const int full = static_cast<int>(items / cus), rest = static_cast<int>(items) - full * cus;
        return full * one(cus) + (rest ? one(rest) : 0.0);
    };
    const double heads = static_cast<double>(d.B) * d.H_q;
    const int steps = (ntile + kStreamsPerWg * nominal - 1) / (kStreamsPerWg * nominal);
    const double step = d.D == 128 ? 0.85 : 0.6;
    const double merge = nominal == 1 ? 0.0 : nominal <= 8 ? 2.8 : 0.8 * nominal;
    const double items = heads * nominal;
    AttnPlan best{nominal, 0, nominal};
    double best_t = items > cus && items <= 2 * cus
        ? 6.5 + merge + steps * std::fmax(2 * step, items * half * 32768 / 6.2e6)
        : rounds_of(items, [&](int active) { return 6.5 + merge + steps * std::fmax(step, active * half * 32768 / 8.0e6); });
    // what the row-dividing kernels assume (32-bit offsets into a request's query rows and a half tile)
    if (d.kv_stride_t >= (1 << 22) || (d.N_max * d.q_stride_n + group * d.q_stride_h) >= (1ll << 30) ||
        heads * 4 * nominal >= (1 << 24))
        return best;
    for (int br = 16; br <= 32; br *= 2) {
        if (br == 32 && rows <= 16) break;
        const int rb = (rows + br - 1) / br;
        const double units = static_cast<double>(d.B) * d.H_kv * rb;
        const double a = br == 16 ? (d.D == 128 ? 4.8 : 4.3) : (d.D == 128 ? 5.2 : 4.6);
        const double c = br == 16 ? 1.9 : 2.5, b = (br == 16 ? 0.9 : 1.05) * (d.D == 128 ? 1.0 : 0.57);
        const int s_lo = d.num_splits > 0 ? nominal : 1;      // a caller's count is taken as given
        for (int s = s_lo; s <= nominal; ++s) {
            if (s > 1 && units > kMaxSplitHeads) break;    // one set of ticket counters per unit
            const int r = (ntile + 4 * s - 1) / (4 * s);
            const double t = rounds_of(units * s, [&](int active) {
                return a + (s > 1 ? c + 0.8 * ((s - 1) / 8) : 0.0) + r * std::fmax(b, active * half * 65536 / 13.5e6);
            });
            if (t < best_t * 0.98) { best_t = t; best = AttnPlan{nominal, br, s}; }
        }
    }
    return best;
}

// A batch in which at least four query heads share a KV head takes four key ranges instead of two, in the launch shape
// with two workgroups per compute unit: most of its tiles come from L2, so that a second workgroup's steps cost
// little, and a short request's workgroups make room next to a long one's.
// us per call (head size 128, 60 nodes), 2 -> 4 ranges | 32-row blocks:
//   query / KV heads x requests     equal lengths                            very different lengths
//   32 / 8 x 4                      3000 keys 30.9 -> 29.8 | 29.5            2500 - 300  27.5 -> 21.7 | 24.5
//                                   4500      41.3 -> 39.5 | 42.4
//   64 / 8 x 2                      4500      41.2 -> 37.8 | 37.0            4500 + 900  41.1 -> 29.2 | 36.1
//   40 / 8 x 3                      3000      30.9 -> 29.9 | 27.7            4500 - 1000 40.9 -> 29.9 | 37.7
//   28 / 4 x 4                      3000      30.8 -> 28.8 | 26.8            3000 - 500  31.0 -> 27.9 | 26.3
//   32 / 8 x 3                      3000      30.7 -> 28.4 | 27.8            3000 - 500  30.7 -> 23.2 | 26.9
//   48 / 8 x 2                      4500      40.9 -> 35.8 | 37.0            4500 + 700  41.1 -> 28.9 | 36.4
// (figures of these kernels before attn_streams.hip, which now takes all of these shapes, by length: plan_columns below.  This rule
// then says how large the workspace is, and still chooses the kernel where that one is not taken: blocks of rows less than 55 % full, fewer
// than 180 workgroups, capacities that are no multiple of 16.)  Four ranges in two workgroups per compute unit | attn_streams.hip:
//   (two ranges each)  32 / 8 x 4, 3000: 28.9 | 24.5; 2500 - 300: 21.8 | 21.6; 64 / 8 x 2, 4500: 36.6 | 29.9; 4500 + 900: 28.9 | 29.7, paged 30.3 | 31.9;
//   40 / 8 x 3, 3000: 28.8 | 23.8; 4500 - 1000: 29.3 | 29.7; 28 / 4 x 4, 3000 - 500: 27.7 | 22.6; 48 / 8 x 2, 4500 + 700: 28.5 | 28.8, paged 30.0 | 31.2
// (one request much longer than the other: two ranges of it are all that 256 workgroups of 64 rows leave; up to 5 % slower, equal
// lengths 15 - 22 % faster, and the host does not know the lengths.)
// Row blocks are chosen first, by their comparison with two ranges: where that favours them they also beat four
// at equal lengths (32 / 8 x 4, 2000 keys 25.1 | 22.9; 64 / 8 x 2, 3000 keys 29.3 | 26.8), and where it does not they lose
// little there and much at different ones.
// Not taken where equal lengths lost: no shared KV heads 31.2 -> 32.6, two query heads per KV head
// 25.2 -> 26.1, more than four ranges 21.6 -> 24.6, head size 64 18.7 -> 19.7; nor for a call without key ranges,
// whose results would gain the rounding of partial results; streams shorter than 12 tiles have nothing to divide.
inline AttnPlan plan_of_heads_and_rows(const specvlm_attn_desc& d) {
    AttnPlan plan = plan_rows(d, single_round_ranges(d));
    if (plan.block_rows || d.num_splits > 0 || plan.ranges != 2) return plan;
    if (d.B < 2 || d.D != 128 || d.H_q / d.H_kv < 4) return plan;
    const int cap = d.paged ? d.max_blocks_per_req * SPECVLM_PAGE_SIZE : d.kv_capacity;
    if (cap >= 12 * kStreamsPerWg * kTile * 2 && 4ll * d.B * d.H_q <= kMostTwoPerCu) plan.ranges = plan.splits = 4;
    return plan;
}

// Row blocks (attn_wave.hip) that run in one round of workgroups are beaten by twice their key ranges (196 random shapes, 0.68 -
// 0.99 of their time), not by the same number or half as many more, as long as the blocks of a head share an XCD, that is where
// their workgroups are a multiple of 8.  us by row blocks | here:
//   8 x 40 query / 10 KV heads, 22 nodes, 503 keys 10.3 | 12.3; 6 x 64 / 8 of 64, 18 nodes, 828: 9.4 | 11.6; 4 x 40 / 20, 46 nodes, 3869:
//   40.7 | 43.5 (42 such shapes, all slower here, 6 - 27 %); two ranges | three: 5 x 28 / 4, 24 nodes, 2900: 21.1 | 23.0; but 8 x 20 / 5,
//   22 nodes, 3390: 24.8 | 22.4 (three ranges on 216 workgroups or more, long streams); three | four: 3 x 16 / 8, 36 nodes, 2750: 16.0 | 16.7
// That condition and the lines for other numbers of workgroups date from when only a multiple of 8 gave an XCD a contiguous range of the row blocks
// (other numbers: every XCD fetched a head's K and V again, 5 x 50 / 10, 30 nodes, 2600 keys 60.0 | 34.6; 9 x 20 / 4, 40 nodes, 472: 13.8 | 13.0).
// attn_wave.hip now does so whatever the number, and it makes no difference any more.  Time of row blocks over that of the even division here, 1926
// random shapes, requests as long as the cache (and at a quarter of it); one range: least - most, else the mean:
//     ranges, tiles          one                        three: 40 - 56  56 - 70      70 - 90      90 - 120     four: 70 - 90  90 - 120
//     128, multiple of 8     0.81 - 0.91 (0.77 - 0.85)  0.96 (0.84)     1.01 (0.87)  1.04 (0.87)  1.08 (0.86)  0.93 (0.82)    0.98 (0.86)
//     128, other numbers     0.82 - 0.94 (0.78 - 0.86)  0.98 (0.85)     1.04 (0.87)  1.07 (0.88)  1.11 (0.87)  0.97 (0.85)    1.02 (0.88)
//     64, multiple of 8      0.85 - 1.03 (0.83 - 1.06)  0.98 (0.89)     1.02 (0.90)  1.03 (0.92)  1.07 (0.92)  0.94 (0.87)    0.97 (0.91)
//     64, other numbers      0.85 - 0.97 (0.82 - 0.91)  0.98 (0.89)     1.01 (0.90)  1.05 (0.93)  1.09 (0.93)  0.96 (0.88)    1.01 (0.92)
// So for other numbers of workgroups the line lies too low: of the calls that it sends here evenly divided, those of one range, and of four up
// to 90 tiles, would be better off with row blocks (9 x 20 / 4, 40 nodes, 472 keys among them); not drawn again yet.
inline bool rows_in_one_round_win(const specvlm_attn_desc& d, const AttnPlan& plan, int64_t units, int s) {
    const int ntile = ((d.paged ? d.max_blocks_per_req * SPECVLM_PAGE_SIZE : d.kv_capacity) + kTile - 1) / kTile;
    if (!plan.block_rows) return false;
    const int row_blocks = (d.H_q / d.H_kv * d.N_max + plan.block_rows - 1) / plan.block_rows;
    const int64_t workgroups = static_cast<int64_t>(d.B) * d.H_kv * row_blocks * plan.splits;
    if (workgroups > 256 || s >= 2 * plan.splits) return false;
    if (workgroups % 8 == 0) return !(s == 3 && units * s >= 216 && ntile >= (d.D == 64 ? 56 : 90));
    if (plan.splits > 1) return ntile < 56;
    return row_blocks < 6 && (ntile < 32 || (d.paged && d.D == 64));
}

// Batches that fill the chip with four streams per workgroup of 64 rows (attn_streams.hip) take as many key ranges as make one
// round of 140 (with ranges 180) - 256 workgroups.  Not fewer workgroups (128 x 19 tiles: 15.1 us, 12.8 by row blocks), streams shorter than 3.5 tiles
// (4 x 16 heads of 31 tiles, two ranges: 15.7 against 14.2; with four ranges, whose meeting costs more, 4.25 tiles), nor blocks
// less than 55 % full (28 of 64 rows: 17.0 against 15.5).  A call whose results were not rounded to partial ones before stays
// without them, and one that took key ranges takes at least two: requests of different lengths need them (5 x 32 heads,
// 3568 - 400 keys, three ranges 38.9, one 43.2; equal lengths of 3100: 49.3 and 46.3).
// Nor short unsplit calls of 224 workgroups or more that share no K and V, whose stream from HBM counts more than a tile's step.
// attn_mfma | here: 7 x 32 heads, 424 keys 14.3 | 15.5; 8 x 32, 560: 17.7 | 18.6; 8 x 28, 670: 18.3 | 18.9 (25 of 30 such calls of equal
// lengths are slower here, up to 10 %; at very different ones 10 x 25, 700 - 90: 17.1 | 16.8, in the mean 3 % faster here).  From 24 tiles on
// (paged 18) equal lengths are even to 3 % slower, different ones 2 - 15 % faster.
// Nor a single request, which mostly loses (1 x 32 / 8, 4000 keys, four ranges 16.2 by key ranges | 18.1; 1 x 40, 2000: 14.6 by row blocks | 15.6;
// 1 x 28 / 4, 5200: 18.3 | 21.8), except with 64 query heads on few KV heads and 2000 keys or more (1 x 64 / 8, 4000: 23.0 | 18.5): not taken yet.
// us per call before -> here (head size 128 unless said):
//   unsplit       8 x 32 query / 16 KV heads, 4788 keys 82.4 -> 65.7; 7 x 32 / 8, 852: 21.1 -> 17.2; 4 x 40, 671: 18.5 -> 16.4;
//                 6 x 32, 2800 - 300: 44.7 -> 35.6; 8 x 32, 900: 25.3 -> 25.4; 5 x 32 of 64, 253: 10.6 -> 8.9
//   two ranges    3 x 32 / 4, 2657: 27.7 -> 22.0; 3 x 32, 3529: 38.8 -> 35.6
//   three, four   5 x 16 of 64, 3027: 18.6 -> 16.3; 2 x 40, 3729: 33.0 -> 30.6; 2 x 32, 4474: 30.9 -> 30.7
inline int32_t stream_ranges(const specvlm_attn_desc& d, const AttnPlan& plan) {
    const int cap = d.paged ? d.max_blocks_per_req * SPECVLM_PAGE_SIZE : d.kv_capacity;
    const int group = d.H_q / d.H_kv, rows = group * d.N_max, blocks = (rows + 63) / 64;
    const int64_t units = static_cast<int64_t>(d.B) * d.H_kv * blocks;
    if (d.B < 2 || d.num_splits > 0 || units > 256 || 100 * rows < 55 * 64 * blocks) return 0;
    // what the kernel assumes: whole halves of a tile inside the cache, 32-bit offsets into a request's query rows and a half tile
    if (cap % 16 || d.kv_stride_t >= (1 << 22) || (d.N_max * d.q_stride_n + group * d.q_stride_h) >= (1ll << 30)) return 0;
    const int s = plan.splits == 1 ? 1 : std::min<int64_t>({256 / units, plan.ranges, 4});
    if (s < (plan.splits == 1 ? 1 : 2) || units * s < (s == 1 ? 140 : 180) || rows_in_one_round_win(d, plan, units, s)) return 0;
    const int ntile = (cap + kTile - 1) / kTile;
    if (s == 1 && group == 1 && !plan.block_rows && d.D == 128 && units >= 224 && ntile < (d.paged ? 18 : 24)) return 0;
    return ntile >= (s == 4 ? 17 : 14) * s ? s : 0;
}

constexpr int kMostRanges = 8;      // key ranges of a request that the kernel with four streams adds up
constexpr int kMostByLength = 16;   // requests that it deals columns out to

// The host does not know the requests' lengths, the device does.  A batch with room for more workgroups than `streams` would take, or
// for more than one per request, gets C = 256 / (row blocks of a request) columns, and every workgroup works out from the lengths which
// request and key range its column is (attn_streams.hip): few for short requests, up to eight for long ones, so that the longest stream
// of the batch is as short as C columns allow.  us per call before -> here (head size 128, 60 - 64 nodes):
//   4 x 32 query / 8 KV heads, 2048, 1311, 3000, 777 keys 24.0 -> 20.1; 3 x 32 / 16, 3664, 1500, 500: 27.9 -> 20.4; 8 x 16 / 4, 4500 - 200:
//   29.8 -> 20.5; 6 x 32, 2800 - 300: 42.0 -> 33.8; 2 x 32, 4474 + 800: 29.5 -> 24.7; 2 x 32, 64 / 8, 4500 + 900 paged: 31.9 -> 25.7;
//   4 x 35 / 5, 48 nodes, 2016, from row blocks: 37.8 -> 20.5
// Equal lengths cost what the plan costs, 0.1 - 0.5 us, as the first tile is requested before it.  So only where streams are long:
// x = tiles per column at equal lengths.  The capacity stands in for them, and requests may be much shorter: the lines lie where the
// geometric mean of the time here over the time there, for a longest request of the whole capacity, a half, a quarter and an eighth, falls
// below 1 (320 shapes at four fillings; requests of a batch equal or up to ten times different):
//   in place of                        x        whole  half  quarter  eighth | mean
//   the streams' kernel, evenly    128 26 - 34  0.94   0.97   1.02     1.02   0.99;   34 - 60: 0.97;   above: 0.94
//                                   64 60 - 80  0.82   0.91   0.97     1.01   0.93;   above: 0.95
//   key ranges                     128 20 - 30  0.98   1.05   1.16     1.18   1.09;   30 - 60: 0.92;   above: 0.82
//                                   64 50 - 80  0.85   0.85   0.84     0.80   0.83;   above: 0.87
//   row blocks, one round of a     128 20 - 38  0.90   1.10   1.33     1.36   1.16;   38 - 44: 1.06;   44 - 60: 0.94;   above: 0.87
//     multiple of 8 workgroups      64 26 - 44  0.85   1.05   1.22     1.28   1.09;   44 - 50: 1.04;   50 - 60: 0.97;   above: 0.91
//   row blocks, one round of       128 20 - 30  0.84  1.06  1.28     1.32   1.11;   30 - 38: 1.04;   38 - 44: 0.96;   44 - 60: 0.90;   above: 0.84
//     another number                64 20 - 30  0.85  1.03  1.18     1.24   1.07;   30 - 38: 1.03;   38 - 50: 0.99;   50 - 60: 0.94;   above: 0.90
// (The last two rows are measured with the kernels as they are, 2587 shapes, the others with earlier ones.  A multiple of 8 made a difference to row
// blocks then: 0.77 from 34 on, 0.83 from 30 on, together with calls of more than one round, which share the line of 20 and 26.  With today's figures
// it would be at 38 for one round.  Not drawn again yet: at 20 - 38 requests that fill the cache would lose 1.2 - 1.3, shorter ones gain as much.)
// (3 x 40, 1744 slots: 1700 keys 23.1 -> 19.6, 376 - 58 keys 10.2 -> 14.4 us; so it keeps its row blocks.)  Not where heads are shared and
// equal lengths would leave more than a fifth of the columns idle (5 x 32 / 16, 4916 keys 53.6 | 63.9), and blocks at least 70 % full.
// Below, short unsplit calls with shared heads gain from a column each (x < 12, at 64 16); at 128 from 7 tiles on (140 shapes, equal lengths of the whole
// capacity | different | half of it: 3 tiles 1.06 | 1.06 | 1.06 of their time; 4 - 6: 0.99 | 0.99 | 1.02; 7 - 10: 0.97 | 0.97 | 1.00; 11 - 13: 0.91 | 0.91 | 0.95; at
// 64 3 - 6: 0.93 | 0.93 | 0.95; 7 - 13: 0.85 | 0.85 | 0.91; without shared heads 0.95 - 1.08).
inline void plan_columns(const specvlm_attn_desc& d, AttnPlan& plan) {
    const int group = d.H_q / d.H_kv, rows = group * d.N_max, blocks = (rows + 63) / 64;
    const int64_t units = static_cast<int64_t>(d.H_kv) * blocks;
    if (plan.streams) plan.columns = d.B * plan.streams;
    const int cap = d.paged ? d.max_blocks_per_req * SPECVLM_PAGE_SIZE : d.kv_capacity;
    if (d.B < 2 || d.B > kMostByLength || d.num_splits > 0 || units * d.B > 256 || 100 * rows < (plan.streams ? 55 : 70) * 64 * blocks) return;
    if (cap % 16 || cap > (1 << 24) || d.kv_stride_t >= (1 << 22) || (d.N_max * d.q_stride_n + group * d.q_stride_h) >= (1ll << 30)) return;
    int columns = static_cast<int>(256 / units);
    // blocks of a head and range on one XCD, where that costs an eighth of the columns at most (4 x 28 / 4, 3000 keys 23.8 -> 22.6)
    if (blocks > 1)
        for (int c = columns; c >= d.B && 8 * c >= 7 * columns; --c)
            if (d.H_kv * c % 8 == 0) { columns = c; break; }
    const int ntile = (cap + kTile - 1) / kTile;
    const double x = static_cast<double>(ntile) * d.B / columns;
    const bool wide = d.D == 128;
    if (plan.streams) {
        if (x < (wide ? 26 : 60)) return;
    } else {
        if (group > 1 && !plan.block_rows && plan.splits == 1 && x < (wide ? 12 : 16)) {
            if (!wide || ntile >= 7) plan.columns = d.B;
            return;
        }
        const int used = std::min(columns / d.B, kMostRanges) * d.B;
        double least = wide ? 30 : 40;
        if (plan.block_rows) {
            const int64_t workgroups = static_cast<int64_t>(d.B) * d.H_kv * ((rows + plan.block_rows - 1) / plan.block_rows) * plan.splits;
            if (workgroups <= 256 && workgroups % 8 == 0) least = wide ? 44 : 50;
            else least = wide && group > 1 ? 20 : 26;
        }
        if (x < least) return;
        if (group > 1 && 5 * used < 4 * columns && (!plan.block_rows || x < 32)) return;
    }
    if (columns > d.B) {
        plan.columns = columns;
        plan.by_length = 1;
    } else {
        plan.columns = d.B;
    }
}

// The division into row blocks once more, for head size 128 and one round of workgroups, with the times of the kernels as they are: a
// workgroup's constant, another where partial results meet, and a step that lasts as long as one compute unit needs for its bytes while
// `active` of them fetch (the row blocks of a head, or the heads of a group, fetch together).  Fitted to 2200 random calls (1 - 8 requests,
// 2 - 64 KV heads shared by 1 - 8, 8 - 64 nodes, 64 - 9000 keys) in all their divisions, and held against 1000 others:
//   key ranges -> row blocks, where these are 3 % faster by the model, take about as many compute units (fewer: up to 1.06) and have at most 7
//     tiles a stream (10 where four or more heads share K and V; beyond, K and V fetched once win again: 8 - 11 tiles up to 1.09 of the time of
//     key ranges): 0.91 of their time in the mean of 282 calls, none above 1.02; requests of a half to an eighth of the capacity 0.80, none above 0.88
//   32 -> 16 rows and back, as many ranges, where 5 % faster: 0.92 of 385, none above 0.99; shorter requests 0.90
// us per call: 1 x 32 heads, 2160 keys 13.7 -> 12.3, 2660: 14.6 -> 13.7, 3324: 16.3 -> 15.5 (as the step was made 16.6 -> 16.1); paged 3324:
// 17.7 -> 16.2; 1060 keys in a cache of 3328: 12.1 -> 9.9; 32 / 8 heads, 2660: 14.2 -> 12.1, 4060: 16.2 -> 14.6.  Not taken: other numbers of ranges of row blocks (more: 0.94, but up to 1.22
// where requests are short; fewer: 0.95, and up to 4 % further from 64 bits; here 0.98 - 1.008 of the error before), row blocks -> key ranges (1.07).
// plan_rows() stays for what was measured against its choice: which batches go to the kernel with four streams, and whether a call has
// partial results at all.  Those are rounded to bf16: a call without them does not gain them here.
inline void fit_rows(const specvlm_attn_desc& d, AttnPlan& plan) {
    const int group = d.H_q / d.H_kv, rows = group * d.N_max;
    const int cap = d.paged ? d.max_blocks_per_req * SPECVLM_PAGE_SIZE : d.kv_capacity;
    const int ntile = (cap + kTile - 1) / kTile;
    const int64_t items = static_cast<int64_t>(d.B) * d.H_q * plan.ranges;
    if (d.D != 128 || d.num_splits > 0 || items > 256 || plan.ranges > 16) return;        // (more ranges: their meeting is priced too high here)
    if (d.kv_stride_t >= (1 << 22) || (d.N_max * d.q_stride_n + group * d.q_stride_h) >= (1ll << 30)) return;      // as in plan_rows()
    auto units_of = [&](int br) { return static_cast<int64_t>(d.B) * d.H_kv * ((rows + br - 1) / br); };
    auto steps_of = [&](int s) { return (ntile + 4 * s - 1) / (4 * s); };
    auto row_time = [&](int br, int s) {
        const double meet = s > 1 ? (br == 16 ? 1.65 : 1.85) + 1.35 * ((s - 1) / 8) : 0.0;
        return (br == 16 ? 3.8 : 4.7) + meet + steps_of(s) * (1.02 + 0.0025 * units_of(br) * s / ((rows + br - 1) / br));
    };
    const bool from_rows = plan.block_rows != 0;
    int least = plan.splits, most = plan.splits;
    double best;
    if (from_rows) {
        best = 0.95 * row_time(plan.block_rows, plan.splits);
    } else {
        // (attn_mfma.hip deals workgroups that are no multiple of 8 out to the XCDs in turn, so that the heads of a group share no L2 and key ranges
        // take longer than the model below says.  Row blocks took 0.55 - 0.93 of their time in 164 such calls; not taken yet)
        if (items % 8 != 0 && group > 1) return;
        const int steps = (ntile + kStreamsPerWg * plan.ranges - 1) / (kStreamsPerWg * plan.ranges);
        best = 0.97 * (7.0 + (plan.ranges > 1 ? 1.86 + 1.55 * std::max(0, plan.ranges - 8) : 0.0) + steps * (0.894 + 0.00115 * items / group));
        least = 1;
    }
    for (int br = 16; br <= 32; br *= 2) {
        if (br == 32 && rows <= 16) break;
        for (int s = least; s <= most && units_of(br) * s <= 256; ++s) {
            if (!from_rows && (steps_of(s) > (group < 4 ? 7 : 10) || 10 * units_of(br) * s < 9 * items)) continue;
            const double t = row_time(br, s);
            if (t < best) { best = t; plan.block_rows = br; plan.splits = s; }
        }
    }
}

inline AttnPlan attn_plan(const specvlm_attn_desc& d) {
    AttnPlan plan = plan_of_heads_and_rows(d);
    plan.streams = stream_ranges(d, plan);
    plan_columns(d, plan);
    if (!plan.columns && plan.ranges == single_round_ranges(d)) fit_rows(d, plan);
    return plan;
}

// The same call without columns that are dealt out by length: for a workspace that does not hold their partial results.
inline AttnPlan evenly(const specvlm_attn_desc& d, AttnPlan plan) {
    if (plan.by_length) plan.columns = d.B * plan.streams;
    plan.by_length = 0;
    return plan;
}

// Workspace: the ticket counters, a region of fixed size at the start whatever the shape (a later call of another shape then finds its
// counters where every earlier call left zeros, never where one stored partial results), and a partial result of 64 rows and their
// (max, sum) pairs per (request, head, key range).  One that divides the columns by length takes one per workgroup, in fp32 where the call's
// results are not rounded to partial ones otherwise.
constexpr size_t kCounterBytes = static_cast<size_t>(kMaxSplitHeads) * 4 * 128;
inline size_t attn_workspace_bytes(const specvlm_attn_desc& d, const AttnPlan& plan) {
    size_t parts = plan.ranges == 1 ? 0 : static_cast<size_t>(d.B) * d.H_q * plan.ranges * (64 * d.D * 2 + 64 * 8);
    if (plan.by_length) {
        const size_t workgroups = static_cast<size_t>(plan.columns) * d.H_kv * ((d.H_q / d.H_kv * d.N_max + 63) / 64);
        parts = std::max(parts, workgroups * (64 * d.D * (plan.splits == 1 ? 4 : 2) + 64 * 8));
    }
    return parts ? kCounterBytes + parts : 0;
}

}  // namespace specvlm
