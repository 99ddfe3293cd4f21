// row_plan.hpp -- which launch form the rows of a verification or an update take: a function of their number, their
// length, K and the type only.  Plain host code.
#pragma once
#include <algorithm>
#include <cstdint>

namespace stand {

// Row pass.  Few rows: every row is split over workgroups that hold their parts in registers (row_parts.hpp), where that pays
// (plan_row_parts) and applies (not at the entry point with fixed scratch).  Else rows that fit a workgroup's registers are
// held whole, however many they are (plan_row_whole).  Others stream through the four waves of a workgroup, or through
// sixteen as long as each compute unit has at most one such workgroup: verifications, sixteen / four waves, us: 256 rows of
// 522 KB (bf16) 49.2 / 54.3, 288 rows 63.7 / 59.6.
#ifndef STAND_ROW_WPR
#define STAND_ROW_WPR 4
#endif
constexpr int kRowWPR = STAND_ROW_WPR, kRowWPRFewRows = 16;
constexpr int kRowsSixteenWaves = 256;
constexpr int unsplit_waves(int64_t rows) { return rows <= kRowsSixteenWaves ? kRowWPRFewRows : kRowWPR; }

constexpr int kPartWaves = 8, kPartThreads = 64 * kPartWaves;
constexpr int kPartVectors = 8;                      // most vectors per lane
constexpr int kPartsMax = 32;                        // most parts of a row
constexpr int kPartsTarget = 256;                    // workgroups that few rows are split into
constexpr int kRowsSplit = 512;                      // more rows are held whole (plan_row_whole), in two parts (plan_row_two_parts), or they stream
constexpr int kCommitSlotsSplit = 4096;              // row slots of an update that may be split (most hold no row)
constexpr int kCommitWorkgroups = 2560;              // workgroups that find a row in a split update of short paths

constexpr int64_t row_vectors(int64_t V, int element_bytes) { return (V * element_bytes + 15) / 16; }

// Parts of a row for row_parts_kernel, or 0 where it does not fit.  A part must fit the registers of a workgroup;
// beyond that, few rows are split further until the launch has kPartsTarget workgroups, but not into parts of
// less than one vector per thread (the maxima of their lane groups would no longer bound the K best well).
inline int choose_parts(int64_t vectors, int64_t rows)
{
    const int64_t least = (vectors + kPartThreads * kPartVectors - 1) / (kPartThreads * kPartVectors);
    const int64_t most = std::max<int64_t>(least, vectors / kPartThreads);
    const int64_t want = (kPartsTarget + rows - 1) / rows;
    const int64_t p = std::min(std::max(want, least), most);
    if (least > kPartsMax) return 0;
    return (int)std::max<int64_t>(1, std::min<int64_t>(p, kPartsMax));
}

// Most workgroups (rows x parts) that a split launch of so many rows should have.  A workgroup holds its part in
// registers from its first load to its last candidate, so beyond a few device-fulls (1024 are resident) the streaming
// kernels, which overlap one row's end with the next one's loads, are faster.  Verifications of rows that start on cache
// lines, split / the other form, us (parts; bf16 unless named):
//   up to 256 rows, the other form has sixteen waves:  128 x 16 52.7 / 58.6, x 25 80.3 / 81.9;  160 x 13 52.2 / 55.6, x 20 75.8 / 71.1;
//     192 x 10 49.1 / 49.3, x 13 57.4 / 55.4;  224 x 8 42.8 / 44.0, x 13 61.9 / 58.2;  256 x 4 30.8 / 33.3, x 6 39.2 / 38.5, x 10 56.3 / 54.6
//   more rows, four waves:  288 x 10 61.6 / 68.5, x 16 89.1 / 91.4, fp32 78.6 / 77.4;  320 x 8 52.6 / 59.1, x 16 96.9 / 92.0;
//     384 x 4 38.0 / 40.0, fp32 x 8 53.6 / 50.0;  448 x 3 35.6 / 35.2;  512 x 2 30.8 / 32.5, x 4 44.3 / 40.6
// (Rows that start anywhere slow the other forms down by up to a tenth and leave the split as it is.)
constexpr int64_t split_limit(int64_t rows)
{
    return rows <= kRowsSixteenWaves ? 420000 / std::max<int64_t>(rows, 1) : (rows <= kRowsSplit ? 300000000 / (rows * rows) : 0);
}

// A part's bound needs at least K of its 64 lane groups (8 vectors each) to hold elements, and some more to be a good one:
// K = 32, 256 rows of 32 / 40 lane groups split 23.3 / 18.2 us, sixteen waves 21.4 / 21.5; of 24 31.3 / 21.1 (no bound
// at all: every element is a candidate).
constexpr bool bound_holds(int64_t vectors, int K) { return vectors >= 10 * (int64_t)K; }

// Parts per row of a verification, 0: not split.
inline int plan_row_parts(int64_t V, int element_bytes, int64_t rows, int K)
{
    const int64_t vectors = row_vectors(V, element_bytes);
    const int p = choose_parts(vectors, rows);
    return bound_holds(vectors, K) && rows * p <= split_limit(rows) ? p : 0;
}

// Whether a row that is not split is held whole in the registers of one workgroup of row_parts_kernel, however many rows
// there are: nothing is read twice, no list is kept while streaming, and a workgroup's end is shorter than the streaming
// pass's.  (Rows of one part use none of the memory in which parts meet.)  Streaming with four waves / whole, us:
//   verify 1036 x 2096 vectors (bf16) 32.2 / 29.9, 1440 x 3804 44.3 / 41.4, 2784 x 3800 55.7 / 54.6, 882 x 2064 (fp32) 28.4 / 25.8,
//   16384 x 4000 193.1 / 192.7, fp32 199.9 / 185.2, 16384 x 500 101.0 / 99.5;  step 540 x 1079 37.3 / 34.6, 720 x 1024 33.3 / 29.2
constexpr bool plan_row_whole(int64_t V, int element_bytes, int K)
{
    return row_vectors(V, element_bytes) <= kPartThreads * kPartVectors && bound_holds(row_vectors(V, element_bytes), K);
}

// More rows than plan_row_parts splits, too long for one workgroup, short enough for two: two parts as long as the launch has
// little more than a device-full of workgroups (1024 are resident), beyond 584 rows only if the parts are nearly full.
// Streaming with four waves / two parts, bf16, K = 10 (rows on cache lines), us; verifications:
//   520 rows x 4104 vectors 27.0 / 26.4, x 5000 29.0 / 26.6, x 8192 33.7 / 29.9;  553 x 4288 29.0 / 28.0, x 6248 31.7 / 30.0;
//   584 x 4104 28.4 / 28.3, x 5000 30.2 / 28.8, x 6248 31.5 / 30.6, x 7936 34.8 / 31.8;  not 600 x 4104 29.7 / 30.2, x 6248 33.4 / 33.3,
//   640 x 4288 27.7 / 28.4, x 6248 30.7 / 30.8;  600 x 7936 36.5 / 34.7, 640 x 7936 33.2 / 32.6, x 8192 35.9 / 33.4;
//   misaligned 576 x 4100 fp32 29.3 / 27.3, 640 x 7696, K = 16 35.2 / 33.4;  not 720 x 8125 34.9 / 35.3, 768 x 6250 31.8 / 34.6
// and steps:  520 x 4104 38.2 / 37.3;  553 x 4288 37.9 / 37.5;  584 x 4104 40.9 / 40.9, x 5000 40.3 / 39.5, x 6248 43.1 / 43.0, x 7936 46.8 / 45.9;
//   not 640 x 4288 39.0 / 40.2, x 6248 42.3 / 43.2, x 7176 42.6 / 43.3;  600 x 7936 46.1 / 45.7, 640 x 7696 44.9 / 45.2, K = 16 45.7 / 45.3,
//   x 8192 45.5 / 44.8, 620 x 7800 fp32 44.8 / 44.1
constexpr int kRowsTwoParts = 584, kRowsTwoFullParts = 640;
constexpr bool plan_row_two_parts(int64_t V, int element_bytes, int64_t rows, int K)
{
    const int64_t vectors = row_vectors(V, element_bytes), full = kPartThreads * kPartVectors;
    return rows > kRowsSplit && rows <= (vectors > 15 * full / 8 ? kRowsTwoFullParts : kRowsTwoParts) &&
           vectors > full && vectors <= 2 * full && bound_holds(vectors, K);
}

// Parts per row of an update with R row slots per trajectory, W = longest path, N = nodes; 0: not split.
// Where all slots can be on one path or are merged anyway (chains, all-nodes updates) every slot counts as a row.  Else
// accepted paths are short: the parts are chosen for up to four rows per trajectory, the limit is on two.  Updates,
// split / unsplit, us: 128 trajectories x 300 KB (5 parts), paths of 1 / 2 / 4 / 8: 52 / 74, 68 / 89, 105 / 118, 172 / 160;
// x 800 KB (fp32, 13 parts: not split): 96 / 141, 139 / 167, 220 / 215, 426 / 291; 64 x 800 KB (split): 69 / 80, 84 / 89, 127 / 116, 216 / 157.
inline int plan_commit_parts(int64_t V, int element_bytes, int64_t B, int W, int N, int R, int K)
{
    const int64_t vectors = row_vectors(V, element_bytes);
    const bool all = W == N || R > W;
    const int64_t expect = B * (all ? R : std::min(W, 4)), usual = B * (all ? R : std::min(W, 2));
    if (expect > kRowsSplit || B * R > kCommitSlotsSplit || !bound_holds(vectors, K)) return 0;
    const int p = choose_parts(vectors, expect);
    return usual * p <= (all ? split_limit(usual) : kCommitWorkgroups) ? p : 0;
}

// 16-byte loads per thread and segment of the exact sums in a launch of their own: one round of four, or of two for the few
// path rows of a small batch (the entry point with fixed scratch; steps of deep trees).  That entry point with 2 / 4, us:
// 1 x 32 rows x 152 064 30.4 / 31.2, 8 x 32 x 128 256 31.1 / 32.2, 16 x 48 x 32 003 fp32 32.7 / 32.9, x 32 000 24.5 / 26.0;
// steps of 32 x 64 158.0 / 156.4.  Not where every drafted row is summed, which fills the vector ALUs at any batch size:
// all-nodes steps of 16 x 64 rows 357 / 331, 4 x 64 98 / 94.
constexpr int exact_loads(bool verify, bool all_nodes, int64_t B) { return verify && !all_nodes && B <= 16 ? 2 : 4; }

// Whether the workgroups of B trajectories may wait in step_tail_kernel, for each other and for workgroups that are started
// behind them, on compute units that hold `places` such workgroups at once: they take at most an eighth of the places, so
// that the others have room with launches of seven more such batches beside them.
constexpr bool plan_tail_places(int64_t B, int64_t places) { return 8 * B <= places; }

// Ranges of vectors of a path row in step_tail_kernel, each summed by one wave; workgroups hold `waves` of them.  Rows are cut
// as finely as one vector per lane for a few trajectories, where the latency of a sum counts, else four: steps with 1 / 2
// vectors per lane, us: 1 x 32 rows x 152 064 25.6 / 27.6, 8 x 32 x 128 256 41.4 / 42.0; with 1 / 2 / 4 / 8: 32 x 64 x 152 064,
// long paths 158.6 / 152.0 / 148.3 / 149.6.  But not into more than 2048 ranges (4096 beyond 16 trajectories) of all
// trajectories' rows together, unless they were longer than eight vectors per lane: more workgroups only wait to be started and
// take the trajectories' waves their turn; and never into more than 8192.  Steps of paths of two / five rows, us:
//   finest / 8192 / 4096 / 2048 ranges in all:  16 x 16 rows x 128 256 46.2, 52.6 / same / 46.1, 52.6 / 44.7, 49.8;
//     16 x 16 x 300 000 69.9, 83.6 / same / 64.9, 74.7 / 62.7, 70.7;  32 x 16 x 300 000 91.2, 105.3 / same / 91.8, 106.7 / 91.5, 103.1;
//     32 x 16 x 1 000 003 227.7, 266.5 / 223.4, 256.1 / 221.7, 253.8 / 238.3, 256.3;
//     64 x 16 x 1 000 003 435.9, 520.9 / 417.1, 479.4 / 421.3, 492.4 / 457.9, 492.4 (separate launches 413.7, 466.9)
inline int plan_tail_ranges(int64_t V, int element_bytes, int64_t B, int waves, int most)
{
    const bool few = B <= 16;
    const int64_t vectors = row_vectors(V, element_bytes), finest = 64 * (few ? 1 : 4);
    const int64_t most_ranges = std::min<int64_t>((vectors + finest - 1) / finest, std::min<int64_t>(8192 / B, most));
    const int64_t n = std::min<int64_t>(std::max<int64_t>(vectors / 512, (few ? 2048 : 4096) / B), most_ranges);
    return (int)std::min<int64_t>((n + waves - 1) / waves * waves, most);
}

// Path rows of a verification that have summing workgroups of their own, `groups` each (the others are taken after them): as
// many as 512 workgroups serve, at least three.  2 / 3 / 4 / all, steps of 32 x 64 rows x 152 064 (5 groups) with long paths
// 151.4 / 147.9 / 148.4 / 149.2 us.  Three / as many as 512 workgroups serve, verifications, us (separate launches): 24 x 64 rows
// x 32 000 (1 group), paths of 2 / 5 / up to 11 rows 36.2 / 36.2 (37.9), 40.0 / 36.3 (38.9), 46.7 / 37.1 (41.3); 32 x 31 x 32 000, up to 16
// rows, 40.6 / 32.9 (35.0); 8 x 64 x 152 064 (16 groups), 5 rows, 48.5 / 45.3 (47.1).
constexpr int plan_tail_slots(int64_t B, int W, int groups)
{
    const int64_t n = 512 / (B * groups);
    return (int)(n < 3 ? (W < 3 ? W : 3) : (n < W ? n : W));
}

// Which calls end in step_tail_kernel, where one workgroup finishes a trajectory's rows and applies its records, one wave claims
// them, and workgroups wait to be started for rows that few paths reach.  W: longest path, NO: orders.  Separate launches / one, us:
// Verifications: all but those of many trajectories with long rows and long paths (`groups` summing workgroups per row).
//   64 x 48 rows x 152 064 (5 groups), W = 8, paths of 2 / up to 8 rows: 171.5 / 173, 183 / 189; W = 16: 124.1 / 128.2, 129.7 / 135.8;
//   W = 32, 5 rows: 127.5 / 139.0;  32 x 31 x 152 064, W = 16: 72.6 / 71.2, 77.2 / 80.9;  64 x 32 x 32 000 (1 group), W = 32: 44.4 / 41.7, 47.7 / 46.3
inline bool plan_tail_verify(int64_t B, int W, int groups) { return B <= 32 || B * W * groups <= 2560; }
// Steps: while there are few record slots in all.  Paths of 2 / 4 / up to W rows, 32 000 tokens:
//   B x W x NO  32 x 8 x 8 = 2048: 58.9 / 57.0, 65.3 / 66.6, 70.5 / 71.6;  48 x 8 x 5 = 1920: 66.5 / 64.2, 73.4 / 72.4, 78.2 / 77.9;
//   16 x 16 x 8 = 2048: 46.6 / 45.8, 60.5 / 62.0, 69.2 / 70.8;  64 x 8 x 3 = 1536: 73.9 / 70.4, 79.8 / 78.8, 84.2 / 85.7;  32 x 16 x 3: 49.7 / 45.8, 64.8 / 62.3, 73.2 / 72.2
//   beyond: 64 x 8 x 5 = 2560: 76.4 / 74.6, 84.0 / 85.0, 88.3 / 91.4;  48 x 11 x 5: 76.3 / 75.1, 85.3 / 86.2, 93.0 / 96.2;  32 x 16 x 8 = 4096: 57.9 / 61.1, 74.0 / 75.3, 83.2 / 86.1;
//   64 x 16 x 5: 72.9 / 71.1, 85.8 / 91.9, 96.1 / 103.1
//   (the longest paths cost up to 5 % below the line too: 1 x 11 x 8, paths of 2 / 5 / 11: 31.5 / 25.6, 41.1 / 41.1, 43.6 / 48.4)
inline bool plan_tail_step(int64_t B, int W, int NO) { return B * W * NO <= 2048; }
// Updates: 50 257 tokens, 2 rows / all W rows: W x NO = 5 x 8 (1 trajectory) 24.2 / 19.1, 23.6 / 22.8; 7 x 4 (6 trajectories) 23.5 / 19.9, 24.4 / 25.4;
//   10 x 4 (6) 23.4 / 20.2, 26.0 / 28.5, (64) 29.5 / 25.2, 57.9 / 60.6;  not 15 x 2: (6) 22.5 / 19.9, 28.5 / 31.5; 20 x 2: (8) 23.3 / 20.8, 29.7 / 36.1, (64) 35.2 / 31.3, 79.7 / 91.8;
//   update and draft of 6 x 14 rows x 4 orders 35.7 / 37.4, of 4 x 32 x 4 50.9 / 66.7 (all slots hold a row)
constexpr bool plan_tail_update(int W, int NO) { return W <= 12 && W * NO <= 40; }

// Whether a step of a small batch (row kernel and step_tail_kernel) keeps these two launches where its rows alone would
// allow the one launch (more than kRowsFew).  One launch / two launches, bf16, us:
//   up to 1024 rows: 8 x 100 x 32 000 45.0 / 38.5, 16 x 64 x 64 000 57.0 / 53.6, x 152 064 87.0 / 84.1, 32 x 32 x 152 064 89.7 / 84.7;
//     not of long rows: 13 x 64 x 128 256 fp32 94.8 / 104.8
//   rows held whole, up to 1600: 16 x 81 x 32 000 48.0 / 45.3, 32 x 50 53.5 / 53.4;  2048: 16 x 128 52.7 / 54.7, 32 x 64 54.9 / 57.5
//     others beyond 1024: 16 x 81 x 64 000 58.5 / 63.3, 32 x 50 x 64 000 68.2 / 71.7
//   more than 32 trajectories (one or two tail workgroups each in the one launch): 64 x 32 x 32 000 68.9 / 62.4,
//     x 64 000 85.9 / 82.4;  x 152 064 124.3 / 142.5, 64 x 48 x 128 256 148.5 / 164.4
inline bool plan_two_launches(int64_t B, int64_t rows, int64_t V, int element_bytes, int K)
{
    // (rows of less than one vector per thread, vocabularies of a few thousand tokens, keep the plain rule on rows)
    if (row_vectors(V, element_bytes) < kPartThreads) return false;
    const int64_t bytes = rows * V * element_bytes;
    return (rows <= 1024 && bytes <= 320000000) || (rows <= 1600 && plan_row_whole(V, element_bytes, K)) ||
           (B > 32 && rows <= 2048 && bytes <= 265000000);
}

}  // namespace stand
