// Host-side launchers of the gfx950 kernels (internal to the library; the public surface is
// include/picospec.h).  Every launcher enqueues on `stream` and returns the launch status.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <cmath>

#include "rowspan.hpp"

namespace picospec {

constexpr int kMaxK = 4096;          // candidate buffer in LDS holds 16384 entries; k beyond this is refused
constexpr int kMaxV = 1 << 20;
// picospec_round: draft + target rows up to which the target rows' statistics take the layout of round_stats_shape, and rounds
// without a table stream both kinds of rows in one launch (the chip holds 512 compress workgroups at a time)
constexpr int kRoundSmallRows = 512;

// The optimistic pass of the compress kernel takes its threshold from a sample of m elements of a row of V: the value
// of rank r in the sample, and every row element at or above it becomes a candidate.  With f = m / V the sample holds
// X ~ Binomial(k, f) of the row's k largest; the pass finds fewer than k candidates iff X >= r, so
//     r = k f + z sqrt(k f (1 - f)) + z^2 / 3      (mean + z standard deviations + the term that covers small means)
// with z = 4.5 (or 4, see below).  It overflows a buffer of `cap` slots iff the sample holds fewer than r of the row's
// `cap` largest, Binomial(cap, f): r must stay z_over standard deviations below cap f.  A pass that fails either way is
// repeated the careful way, so the margins only trade a rare slow row against the candidates every row carries.
// 0: no rank satisfies both (the careful pass takes the row).  The host evaluates the same function, with a slightly
// larger z_over, to choose the kernel variant.
__host__ __device__ inline int optimistic_rank(int k, int V, int m, int cap, float z_over = 4.45f) {
    const float f = (float)m / (float)V;
    const float lam = (float)k * f, lam_cap = (float)cap * f;
    const float sd_cap = sqrtf(lam_cap * (1.f - f));
    const float zs[2] = {4.5f, 4.0f};
    for (int i = 0; i < 2; ++i) {
        const float r = ceilf(lam + zs[i] * sqrtf(lam * (1.f - f)) + zs[i] * zs[i] * (1.f / 3.f));
        if (lam_cap - r >= z_over * sd_cap) return (int)r;           // (r may exceed k: a short record still takes the fast pass)
    }
    return 0;
}

// The compression of few rows over many workgroups (split.hip): how a row is split, how many of its elements a workgroup
// hands on (its `rank` largest and what shares the threshold's bin), and how many slots its list has.
// parts = 0: the call is not split.  Lines of the rule:
//   * rows (split_max_rows): with one workgroup per row a call takes the time of one row as long as every row has a CU of its
//     own; split, the first launch's time grows with the rows from about 40 rows on, and the second one's with k.  Measured,
//     unsplit / split, us, fp32 (bf16): k = 256: 192 rows of 151,936 28.8 / 26.8 (23.6 / 23.7), 100,000 23.5 / 21.7 (19.6 / 19.9),
//     16,384 14.0 / 13.8 (13.5 / 13.4); k = 1024: 128 rows of 151,936 29.4 / 24.4 (25.4 / 22.2), 100,000 24.4 / 21.9 (20.8 / 21.2), 20,000 15.5 / 15.3
//     (15.8 / 15.5), 16,384 15.0 / 15.4 (15.1 / 15.6); k = 4096: 80 rows of 151,936 35.0 / 31.0 (34.6 / 31.4), 50,000 25.9 / 26.2 (27.9 / 26.4): of 574
//     points on this side of the line seven are slower by more than 1 %, at V = 16,384 by 3 %.  More rows would gain on fp32 (320 of 151,936, k = 256: 50.4 /
//     39.8; 160 of 128,256, k = 512: 26.3 / 23.3) and are not taken so far; bf16 rows would not (31.5 / 33.0, 22.4 / 21.6).
//   * V: two workgroups' worth, and eight times k.
//   * the margin of the rank is optimistic_rank's (4.5 standard deviations of the share of the k largest that falls to one
//     workgroup); its lists together must fit the candidate buffer of the finishing kernel with room to spare.
//   * a list holds the rank, a crowded pivot bin and some slack.
//   * lanes: of a workgroup's 256 lanes, 256 (1 - exp(-rank / 256)) hold one of its `rank` largest elements on average, so a threshold with that
//     many lanes' maxima at or above it has about `rank` elements above it, with a standard deviation of 4.3 at rank 93, 4.8 at 104 and
//     5.1 at 110 (simulated orders, 4000 a point).  Together with the share's own that leaves of the 4.5 deviations asked for 4.5 to 4.7 up to rank 104 in rows of three
//     parts and more, 4.46 at 106 (3 and 4 parts) and 4.2 at 125 (4), and 4.3 to 4.4 in rows of two parts from 100 on; of 512 lanes, with which calls in one launch
//     select, 4.9 at 102 to 113, 4.7 at 125.  So ranks beyond kSplitLanesRank (lanes = 0) count the elements, which is slower everywhere: us, elements / lanes, fp32 (bf16):
//     8 rows of 32,000, k = 256 (rank 102) 9.9 / 9.6 (9.7 / 9.4), 290 (113) 9.9 / 9.6 (9.7 / 9.4); 48 of 131,072, k = 975 (102) 15.1 / 14.3 (14.5 / 13.7), 1050 (108)
//     15.6 / 14.9 (15.0 / 14.2).
constexpr int kSplitMaxRows = 192;
inline int split_max_rows(int k) { return k <= 256 ? kSplitMaxRows : k <= 1024 ? 128 : 80; }
constexpr int kSplitMinV = 16384;                // (two workgroups per row)
constexpr int kSplitNarrowRank = 240;            // ranks for which 256 elements above the histogram's lower end suffice
constexpr int kSplitLanesRank = 104;             // ... for which the threshold is looked for among the lanes' largest values first
constexpr int kSplitMaxParts = 64;               // lists per row (one per lane of a finishing wave): rows of up to half a million elements
struct SplitPlan { int parts, rank, cap, lanes; };
inline SplitPlan split_plan(int dtype, int64_t rows, int V, int k) {
    const SplitPlan none{0, 0, 0, 0};
    if (rows < 1 || V < kSplitMinV || k < 1 || k > kMaxK || rows > split_max_rows(k) || V / 8 < k) return none;
    const int parts = split_parts(dtype == 1, row_vecs_max(dtype == 1, V));
    if (parts < 2 || parts > kSplitMaxParts) return none;
    const float f = 1.f / (float)parts, lam = (float)k * f;
    const int rank = (int)ceilf(lam + 4.5f * sqrtf(lam * (1.f - f)) + 6.75f);
    if (rank > V / parts / 2 || (float)parts * (float)rank > 7000.f) return none;
    const float m = (float)(rank + (rank / 8 > 16 ? rank / 8 : 16));         // with a crowded pivot bin
    const int cap = ((int)ceilf(m + 2.f * sqrtf(m)) + 7) / 8 * 8;
    const int lanes = rank <= kSplitLanesRank ? (int)ceilf(256.f * (1.f - expf((float)rank * (-1.f / 256.f)))) : 0;
    return SplitPlan{parts, rank, cap, lanes};
}
inline size_t split_scratch_bytes(int dtype, int64_t rows, int V, int k) {
    const SplitPlan p = split_plan(dtype, rows, V, k);
    return (size_t)rows * (size_t)p.parts * (32 + 8 * (size_t)p.cap);
}

// ... in one launch, whose last workgroup of a row finishes it (split_compress_kernel; behind the lists, on a 16-byte boundary, a word per row).  It
// spares the host a launch, 2.5 to 3 us of the 12.6 in which it issues a row's record and draw.  us a call in a replayed graph and called in a row, two
// launches / one: one row of 32,000 fp32, k = 64: 9.0 / 9.3, 8.9 / 9.0 (record and draw, which the host bounds: 13.9 / 11.2); one of 128,256 bf16, k = 10: 9.0 /
// 9.2, 8.9 / 8.9; 2 of 151,936 fp32, k = 64: 9.7 / 9.9, 9.6 / 9.6; 4 of 128,256 bf16, k = 64: 9.6 / 9.6, 9.5 / 9.3; 8, k = 256: 10.5 / 10.2, 10.9 / 9.9; 24 of
// 33,001 fp32, k = 70: 9.6 / 9.6, 10.2 / 9.2.  So captured calls of fewer than kOneLaunchSplitReplayed rows, whose replays no host bounds, take two; all
// calls beyond 128 workgroups do (bf16, 32 rows of 128,256, k = 256, 512 workgroups: 14.7 against 13.5; 16 of 151,936, k = 1024, 304: 17.7
// against 15.4): those of the one launch have the finish's LDS, two to a CU.
constexpr int kOneLaunchSplit = 128, kOneLaunchSplitReplayed = 4;
inline bool split_one_launch(int dtype, int64_t rows, int V, int k) { return rows * split_plan(dtype, rows, V, k).parts <= kOneLaunchSplit; }
inline size_t split_words_at(int dtype, int64_t rows, int V, int k) { return (split_scratch_bytes(dtype, rows, V, k) + 15) / 16 * 16; }
inline size_t split_one_launch_bytes(int dtype, int64_t rows, int V, int k) { return split_words_at(dtype, rows, V, k) + (size_t)rows * kArrivalStride; }

// Kernels whose dynamic LDS exceeds the 64 KB default need their limit raised once per device and kernel.
// `done` is the caller's per-device record for that kernel; the current device's ordinal comes back in `dev`.
// The record is atomic and the attribute call idempotent: two threads that meet here on a kernel's first use
// both set the same value, and a thread that reads `true` (acquire) finds the attribute set.
constexpr int kMaxDevices = 64;
using DeviceFlags = std::atomic<bool>[kMaxDevices];
inline hipError_t raise_lds_limit_once(const void* kernel, size_t bytes, DeviceFlags& done, int& dev) {
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    if (!done[dev].load(std::memory_order_acquire)) {
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
        done[dev].store(true, std::memory_order_release);
    }
    return hipSuccess;
}

// seq_off / n_accept: both null (record r from row r), or the downlink's row map (record b from target
// row seq_off[b] + b + n_accept[b])
hipError_t launch_compress(const void* logits, int dtype, int64_t ld, int n_rows, int V, float temperature,
                           int k, float top_p, int32_t* idx, float* prob, int32_t* count, float* mass,
                           float* lse, const int32_t* seq_off, const int32_t* n_accept, hipStream_t stream);

// the same with every row spread over several workgroups (split_plan(...).parts > 0), in two launches, or in one (split_one_launch) where the
// scratch, on a 16-byte boundary, holds split_one_launch_bytes(...) and not only split_scratch_bytes(...)
hipError_t launch_split_compress(const void* logits, int dtype, int64_t ld, int n_rows, int V, float temperature,
                                 int k, float top_p, int32_t* idx, float* prob, int32_t* count, float* mass,
                                 float* lse, const int32_t* seq_off, const int32_t* n_accept, void* scratch, size_t scratch_bytes, hipStream_t stream);

// ... and besides it, in the first of the two launches, the target rows' segment table in the split layout
hipError_t launch_split_round(const void* draft_logits, int dtype, int64_t ld_d, int n_draft, int V, float temperature,
                              int k, float top_p, int32_t* idx, float* prob, int32_t* count, float* mass, float* lse,
                              const void* tgt_logits, int64_t ld_t, int n_target, void* seg_table, void* scratch, hipStream_t stream);

// the draft rows' compression and the target rows' statistics in one launch (small rounds)
hipError_t launch_round_stream(const void* draft_logits, int dtype, int64_t ld_d, int n_draft, int V, float temperature,
                               int k, float top_p, int32_t* idx, float* prob, int32_t* count, float* mass, float* lse,
                               const void* tgt_logits, int64_t ld_t, int n_target,
                               float* tgt_max, float* tgt_sum, float* tgt_lse, void* seg_table, hipStream_t stream);

hipError_t launch_sample_draft(const int32_t* idx, const float* prob, const int32_t* count, const float* mass,
                               int k, int n_rows, const float* uniforms, int32_t* tok, float* q_scalar,
                               hipStream_t stream);

// Launch shape of the row statistics (threads per row, 16-byte vectors per thread and trip) for a dtype and a row
// count, and with it the layout of the optional segment table: a segment is what one wave reads per trip, seg_vecs
// consecutive vectors; a row owns `stride` entries (float2: sum, reference exponent).
struct StatsShape { int threads, nv, seg_vecs, stride; };
inline StatsShape stats_shape(int dtype, int64_t n_rows, int V) {
    StatsShape sh;
    if (dtype != 1)            { sh.threads = 1024; sh.nv = 4; }   // fp32 rows are HBM-bound with any shape
    else if (n_rows >= 2048)   { sh.threads = 256;  sh.nv = 4; }   // bf16: twice the arithmetic per byte; small workgroups,
    else if (n_rows >= 1024)   { sh.threads = 512;  sh.nv = 2; }   // many per CU, keep the vector ALUs busier as long as
    else                       { sh.threads = 1024; sh.nv = 2; }   // there are rows enough to fill the chip with them
    const int esz = dtype == 1 ? 2 : 4;
    const int64_t nq_max = ((int64_t)V * esz + 15) / 16 + 1;       // (a row off the 16-byte boundary spans one vector more)
    const int tile_vecs = sh.threads * sh.nv;
    sh.seg_vecs = 64 * sh.nv;
    sh.stride = (int)((nq_max + tile_vecs - 1) / tile_vecs) * (sh.threads / 64);
    return sh;
}
// ... and of the target rows of a small round, whose statistics run in 512-thread workgroups next to the compression
// (launch_round_stream): vectors per lane and trip chosen so that a row of the longest vocabulary has as many
// segments as above
template <bool BF16> constexpr int kRoundStatsNV = BF16 ? 2 : 4;
inline StatsShape round_stats_shape(int dtype, int V) {
    StatsShape sh;
    sh.threads = kCompressThreads;
    sh.nv = dtype == 1 ? kRoundStatsNV<true> : kRoundStatsNV<false>;
    const int esz = dtype == 1 ? 2 : 4;
    const int64_t nq_max = ((int64_t)V * esz + 15) / 16 + 1;
    const int tile_vecs = sh.threads * sh.nv;
    sh.seg_vecs = 64 * sh.nv;
    sh.stride = (int)((nq_max + tile_vecs - 1) / tile_vecs) * (sh.threads / 64);
    return sh;
}
// launch_round_stream's work for rounds with a segment table, in the layout `sh`, where the compression's first pass applies
// (round_wide_serves)
bool round_wide_serves(int dtype, int64_t n_draft, int64_t n_target, int V, int k);
hipError_t launch_round_wide(const void* draft_logits, int dtype, int64_t ld_d, int n_draft, int V, float temperature,
                             int k, float top_p, int32_t* idx, float* prob, int32_t* count, float* mass, float* lse,
                             const void* tgt_logits, int64_t ld_t, int n_target,
                             float* tgt_max, float* tgt_sum, float* tgt_lse, void* seg_table, const StatsShape& sh, hipStream_t stream);
// bytes of the segment table of `rows` rows (16-byte header in front: see SegHeader)
struct SegHeader { int32_t magic, seg_vecs, stride, rows; };
constexpr int32_t kSegMagic = 0x53454731;        // entries (sum of 2^(z c - r), r)
constexpr int32_t kSegMagicSplit = 0x53454732;   // split layout: entries (sum of 2^(z c - r), m), m = the segment's largest logit, r = m c (split_ref)
// Calls whose rows leave CUs idle spread every row's statistics over many workgroups: each wave leaves the entries of two
// segments of 256 vectors, nothing else, and the kernel that needs the statistics forms them from the row's table.  One
// workgroup per row is bound by the vector ALUs of one CU.  The line for calls that keep the table for their draw: a row for nearly
// every CU (verification and draw of 224 rows of 151,936, k = 64, us, one workgroup per row / spread: fp32 38.3 / 34.3, bf16 28.9 / 25.0;
// of 16,384: 20.9 / 17.1, 19.1 / 17.2); nor below kSplitMinV, where a row is a few segments.  (More rows would gain as well, 384: 28.4 / 25.1, a
// round's 576: 31.5 / 24.0.  Not taken: the draws of such a call are many, and one in 400 lies so near a step of the cumulative
// sum that sums in another order name its neighbour; the spread sums are the more exact ones.)
constexpr int kSplitStatsRows = 224;
inline StatsShape split_stats_shape(int dtype, int V) {
    return StatsShape{256, kSplitStatsNV, 64 * kSplitStatsNV, stats_segments(row_vecs_max(dtype == 1, V))};
}
inline bool split_stats_serves(int64_t rows, int V) { return rows >= 1 && rows <= kSplitStatsRows && V >= kSplitMinV; }
// Calls that are given no workspace and would need one for their statistics alone.  A verification without a draw gains less
// (its second launch is there either way; the draw that the table serves is another call's).  us, one
// workgroup per row / spread, device time:
//   * verification, fp32: rows of 16,384: 9.4 / 10.6 (160 rows), 20,000: 10.6 / 9.8 (64), 10.8 / 11.0 (192), 32,000: 10.9 / 10.5 (128),
//     12.0 / 12.3 (224), 64,000: 13.6 / 12.9 (128), 14.5 / 14.8 (192), 151,936: 22.5 / 21.9 (160), 24.4 / 24.7 (192);
//     bf16: 16,384: 9.6 / 10.9 (160), 20,000: 10.2 / 9.8 (128), 10.3 / 10.5 (224), 32,000: 10.3 / 10.7 (160), 64,000: 12.6 / 12.3 (192),
//     151,936: 18.6 / 16.8 (192), 18.7 / 18.3 (224);
//   * row_stats (launch_row_stats_spread), on the device alone and called in a row: fp32: 33,001: 6.4 / 4.5, 6.4 / 7.5 (8 rows), 64,000: 6.9 / 5.8, 9.7 / 7.4 (64),
//     151,936: 14.3 / 14.7, 14.5 / 14.5 (128); bf16: 33,001: 6.5 / 5.3, 6.5 / 7.6 (96), 64,000: 6.9 / 4.4, 6.9 / 7.6 (8), 151,936: 11.4 / 11.1 (160), 14.6 / 14.3 (192).
//     (Where calls in a row are the slower ones it is the host, which allocates the scratch.)
inline bool verify_scratch_serves(int dtype, int64_t rows, int V) {
    if (!split_stats_serves(rows, V) || V < 20000) return false;
    return rows <= (dtype != 1 ? 160 : V >= 64000 ? kSplitStatsRows : 128);
}
inline bool row_stats_split_serves(int dtype, int64_t rows, int V) {
    const int64_t row_bytes = (int64_t)V * (dtype == 1 ? 2 : 4);
    return split_stats_serves(rows, V) && row_bytes >= 250000 && rows <= (dtype == 1 ? 160 : row_bytes >= 500000 ? 128 : 64);
}
// Whether a round spreads its draft rows in scratch behind its table (picospec_round; picospec_scratch_bytes asks for that scratch by the same
// rule, and a round that does not spread them uses the table alone).  us, one launch for both streams (launch_round_wide) / drafts spread, of
// 2380 points (4 to 192 drafts, 1 to 400 sequences, V = 16,384 to 151,936, k = 10 to 4096) one in thirty-six on the wrong side by more than 2 %, none by more
// than 7 %:
//   * rounds whose statistics are not spread with the drafts' rows (more than kSplitStatsRows target rows) take three launches behind each
//     other and never do: 128 drafts and 528 target rows, k = 256, of 64,000: fp32 43.7 / 51.9, bf16 29.9 / 42.0, of 151,936: 75.5 / 91.1, 49.2 /
//     69.2; 96 and 296 of 151,936, k = 1024: 51.1 / 68.8, 35.8 / 52.7; 16 and 416 of 64,000: 33.7 / 39.5, 27.5 / 33.8.  But where the one launch does not
//     serve (bf16, k > 2048 or V < 32,768), rounds beyond kRoundSmallRows have three launches either way: 37.2 / 34.8 (128 and 528 of 32,000 bf16, k = 256);
//   * drafts, fp32: k = 256, of 151,936: 128 and 192: 47.7 / 45.6, 160 and 192: 49.4 / 49.3, 192 and 224: 50.5 / 55.5; k = 1024, of 64,000: 96 and 128: 31.1 /
//     29.1; short rows: 64 and 80 of 16,384: 25.7 / 25.2, 96 and 112: 25.8 / 27.4.  bf16, three workgroups per CU in the one launch: k = 256, of 151,936: 96 and 160:
//     33.1 / 32.3, 128 and 192: 32.8 / 36.1; k = 1024, of 64,000: 64 and 80: 27.9 / 26.3, 96 and 128: 28.2 / 29.1.  k = 4096: 48 and 64 of 151,936: 54.2 /
//     49.4, 54.9 / 49.7;
//   * drafts per sequence: with the statistics spread a sequence's decision forms those of all its rows.  One sequence of 96 drafts of
//     64,000, k = 256: 36.6 / 39.5, 34.5 / 40.7; of 64: 33.0 / 31.8, 31.2 / 33.8; four of 32 of 16,384: 25.7 / 26.1, 25.0 / 27.3.
inline bool round_split_serves(int dtype, int64_t n_draft, int64_t rows, int V, int k) {
    if (split_plan(dtype, n_draft, V, k).parts == 0) return false;
    const bool wide = round_wide_serves(dtype, n_draft, rows, V, k), short_rows = V < 24000;
    if (!wide && n_draft + rows > kRoundSmallRows) return true;
    if (!split_stats_serves(rows, V) || n_draft > (short_rows ? 24 : 48) * (rows - n_draft)) return false;
    if (k > 2048) return n_draft <= 48;
    if (dtype == 1 && wide) return n_draft <= 64 || (n_draft <= (k <= 256 ? 96 : 80) && rows <= 160);
    return n_draft <= (k <= 256 ? (wide ? 160 : 128) : (short_rows ? 64 : 128));
}
// Where a draw that was given no table makes one of the rows it draws from (one workgroup per row passes over its row twice, and
// is bound by the vector ALUs of one CU): 64 sequences x 33 001 fp32, k = 64: 17.2 -> 11.3 us; 64 x 151 936, k = 64: fp32 29.5 ->
// 15.4, bf16 24.7 -> 13.2; 512: 73.4 -> 54.7, 50.4 -> 32.2; 1024: 139 -> 105, 98.7 -> 56.7.  The draw from a table gathers one logit per
// record entry: long records cost more than the second pass (256 x 151 936 bf16, k = 4096: 28.0, 37.8), and so do those of up to
// 1024 entries where the pass has the chip filled once (256 x 64 000 bf16, k = 1024: 17.8, 19.2).  On rows of up to 64 KB the second
// launch does not pay for few sequences (8 to 256 x 16 384 bf16, k = 64: 9.4 to 10.8, 10.5 to 12.3; fp32 14.3, 12.5 at 256); more
// sequences on such rows would gain (512: 19.6, 15.0; fp32 26.2, 15.5) and keep the pass so far.
constexpr int kResidualSplitSeqs = 1024, kResidualSplitK = 1024;
inline bool residual_split_serves(int dtype, int64_t B, int V, int k) {
    if (B < 1 || B > kResidualSplitSeqs || k > kResidualSplitK || (int64_t)V * (dtype == 1 ? 2 : 4) <= 65536) return false;
    return k <= 256 || B <= 128 || B > 256;
}
inline size_t seg_table_bytes(int dtype, int64_t rows, int V) {
    return sizeof(SegHeader) + (size_t)rows * (size_t)stats_shape(dtype, rows, V).stride * 8;
}
// ... of a round's target rows, whichever of the two schedules the round takes
inline size_t round_seg_table_bytes(int dtype, int64_t rows, int V) {
    const size_t small = sizeof(SegHeader) + (size_t)rows * (size_t)round_stats_shape(dtype, V).stride * 8;
    return small > seg_table_bytes(dtype, rows, V) ? small : seg_table_bytes(dtype, rows, V);
}

// Scratch of the calls whose last workgroups go on (arrive_last): a table in the split layout and behind it (split_table_end) the groups' words, kArrivalStride bytes apart, one per row (row_stats), per sequence and one more (verify), per sequence (the draw without a table).
// Workgroups per row, of `waves` waves, of these launches: no more of them in all than are on the chip at once, two of eight waves per CU (a
// workgroup that waits for its arrival, 0.7 us, holds its place: with a workgroup for every eight segments a verification of 144 rows of 151,936
// fp32 took 28.3 us, with these 19.5).
constexpr int kSpreadGroups = 512;
inline int spread_parts(int segments, int waves, int64_t rows) {
    const int64_t most = (segments + waves - 1) / waves, fit = (int64_t)kSpreadGroups * 8 / waves / (rows > 0 ? rows : 1);
    return (int)(fit < 1 ? 1 : fit < most ? fit : most);
}
// Where they serve, by the segments (4 KB) of the rows in all.  With few, two launches are a boundary of 1.5 us on the device and 2.5 to 3.5 us on the
// host; with more, the rows stream faster from many small workgroups that wait for nothing.  us a call, two launches / one, in a replayed graph
// and called in a row:
//   * verification of a range of positions, up to 5500: fp32: 24 rows of 24,576: 8.0 / 7.2, 8.2 / 7.2; 48 of 64,000 (3024): 9.0 / 8.3, 9.3 / 8.1; 76 of 64,000 (4788): 10.2 /
//     10.1, 11.1 / 9.6; 144 of 33,001 (4752): 10.1 / 10.6, 10.3 / 9.8; 32 of 151,936 (4768): 10.2 / 11.8, 11.3 / 11.2; 108 of 50,000 (5292): 10.4 / 11.4, 11.2 / 10.8;
//     bf16: 48 of 128,256 (3024): 9.4 / 8.3, 9.6 / 8.0; 144 of 64,000 (4608): 10.9 / 10.8, 10.9 / 10.1; 64 of 151,936 (4800): 10.1 / 12.7, 11.3 / 11.9.  That is, of 74 points from 2300 to
//     5500 one launch is the faster in 72 called in a row (1 to 29 %), and in a replayed graph, where no host waits, in 25 of 26 up to 3300 and in 16 of 48
//     beyond (9 % faster to 20 % slower): captured calls take two there;
//   * of all positions, whose workgroups look their sequences up and all have rows to sum, up to 2000: fp32: 24 of 64,000 (1512): 7.8 / 7.5, 8.0 / 7.4; 48 of
//     33,001: 8.1 / 7.5, 8.3 / 7.4; bf16: 24 of 128,256: 8.1 / 7.5, 8.3 / 7.5; 96 of 33,001 (1632): 9.1 / 8.2, 9.3 / 8.0;
//   * the draw, up to 2500: fp32: 24 sequences of 33,001, k = 70: 9.0 / 8.0, 9.8 / 7.8; 64, k = 256 (2112): 9.9 / 9.1, 10.6 / 8.9; bf16: 64 of 64,000 (2048): 9.8 / 9.4, 11.0 / 9.0; beyond
//     (on the device alone) fp32 64 of 64,000 (4032): 10.1 / 10.8, bf16 64 of 151,936 (4800): 11.8 / 13.6.  And from 512 sequences on for records of 513 entries or more, whose
//     workgroups sum a row alone: 512 of 33,001, k = 700: 23.6 / 19.9, bf16 18.7 / 16.5, of 151,936 bf16 38.5 / 34.6; shorter records (k = 64: 18.0 / 20.1) do not gain.
constexpr int kOneLaunchRange = 5500, kOneLaunchRangeReplayed = 3300, kOneLaunchVerify = 2000, kOneLaunchDraw = 2500;
inline bool verify_one_launch(bool ranged, int dtype, int64_t rows, int V) { return rows * split_stats_shape(dtype, V).stride <= (ranged ? kOneLaunchRange : kOneLaunchVerify); }
// (asked only where it makes a difference: `stream` is being captured.  A stream that cannot be asked is not.)
inline bool is_captured(hipStream_t stream) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) == hipSuccess) return status == hipStreamCaptureStatusActive;
    (void)hipGetLastError();
    return false;
}
inline bool residual_one_launch(int dtype, int64_t B, int V, int k) {
    return B * split_stats_shape(dtype, V).stride <= kOneLaunchDraw || (k > 512 && B >= 512);
}
// (behind the larger of the two layouts' tables: a buffer of picospec_scratch_bytes or picospec_workspace_bytes, which holds either, never reaches the words,
// so that its owner gets two launches, and one of picospec_one_launch_bytes one)
inline size_t split_table_end(int dtype, int64_t rows, int V) {
    const size_t split = sizeof(SegHeader) + (size_t)rows * (size_t)split_stats_shape(dtype, V).stride * 8, table = seg_table_bytes(dtype, rows, V);
    return ((split > table ? split : table) + 15) / 16 * 16;
}
inline size_t row_stats_words_at(int dtype, int64_t rows, int V) { return split_table_end(dtype, rows, V); }
inline size_t row_stats_scratch_bytes(int dtype, int64_t rows, int V) { return row_stats_words_at(dtype, rows, V) + (size_t)rows * kArrivalStride; }
inline size_t verify_words_at(int dtype, int64_t rows, int V) { return split_table_end(dtype, rows, V); }
constexpr int kFoundWords = 3;                   // 64-bit words per position looked up
inline size_t verify_found_at(int dtype, int64_t rows, int64_t B, int V) { return verify_words_at(dtype, rows, V) + (size_t)(B + 1) * kArrivalStride; }
inline size_t verify_scratch_bytes(int dtype, int64_t rows, int64_t B, int V) { return verify_found_at(dtype, rows, B, V) + (size_t)rows * kFoundWords * 8; }
inline size_t residual_words_at(int dtype, int64_t B, int V) { return split_table_end(dtype, B, V); }
inline size_t residual_scratch_bytes(int dtype, int64_t B, int V) { return residual_words_at(dtype, B, V) + (size_t)B * kArrivalStride; }

// seg (nullable): the segment table, seg_stride entries per row
hipError_t launch_row_stats(const void* logits, int dtype, int64_t ld, int n_rows, int V, float temperature,
                            float* row_max, float* row_sum, float* row_lse, void* seg_table, hipStream_t stream);

// the table of the rows alone, in the split layout (split_stats_serves): seq_off == nullptr: rows 0 .. n_rows - 1; else the
// target rows pos_begin[b]..pos_end[b] of every sequence (nullable: 0 / gamma_b)
hipError_t launch_row_stats_parts(const void* logits, int dtype, int64_t ld, int n_rows, int V, float temperature, int B, int gamma_max, const int32_t* seq_off, const int32_t* pos_begin, const int32_t* pos_end,
                                  void* seg_table, hipStream_t stream, const int32_t* n_accept = nullptr);   // n_accept: every sequence's row at that position only
// ... and the statistics from it
hipError_t launch_row_stats_finish(const void* logits, int dtype, int64_t ld, int n_rows, int V, float temperature,
                                   const void* seg_table, float* row_max, float* row_sum, float* row_lse, hipStream_t stream);

// both in one launch; scratch holds row_stats_scratch_bytes(...)
hipError_t launch_row_stats_spread(const void* logits, int dtype, int64_t ld, int n_rows, int V, float temperature,
                                   void* scratch, float* row_max, float* row_sum, float* row_lse, hipStream_t stream);

// launch_row_stats_parts and launch_accept in one launch; scratch holds verify_scratch_bytes(...)
hipError_t launch_verify_spread(const void* tgt_logits, int dtype, int64_t ld, int V, float temperature,
                                int B, int64_t n_rows, const int32_t* seq_off, const int32_t* draft_tok,
                                const int32_t* q_idx, const float* q_prob, const int32_t* q_count, const float* q_mass,
                                int k, int renorm, const float* q_scalar, const float* uniforms,
                                float* tgt_max, float* tgt_sum, float* tgt_lse,
                                int32_t* n_accept, float* p_tok, float* q_tok, uint32_t* flags,
                                bool ranged, const int32_t* pos_begin, const int32_t* pos_end, int gamma_max,
                                void* scratch, hipStream_t stream);

// the same for the target rows pos_begin[b]..pos_end[b] of every sequence only (nullable: 0 / gamma_b)
hipError_t launch_row_stats_range(const void* logits, int dtype, int64_t ld, int V, float temperature, int B,
                                  int gamma_max, const int32_t* seq_off, const int32_t* pos_begin,
                                  const int32_t* pos_end, float* row_max, float* row_sum, float* row_lse,
                                  hipStream_t stream);

hipError_t launch_accept(const void* tgt_logits, int dtype, int64_t ld, int V, float temperature,
                         int B, const int32_t* seq_off, const int32_t* draft_tok,
                         const int32_t* q_idx, const float* q_prob, const int32_t* q_count, const float* q_mass,
                         int k, int renorm, const float* q_scalar, const float* uniforms,
                         float* tgt_max, float* tgt_sum, float* tgt_lse,
                         int32_t* n_accept, float* p_tok, float* q_tok, uint32_t* flags,
                         const int32_t* pos_begin, const int32_t* pos_end,
                         const void* split_table, int64_t n_rows, bool all_rows, hipStream_t stream);

// threads of the draw from the segment table: a thread holds two record entries of records of up to 512 entries, four of
// longer ones
inline int residual_seg_threads(int k) { return k <= 512 ? 256 : k <= 2048 ? 512 : 1024; }

hipError_t launch_residual(const void* tgt_logits, int dtype, int64_t ld, int V, float temperature,
                           int B, const int32_t* seq_off, const int32_t* n_accept,
                           const float* tgt_max, const float* tgt_sum,
                           const int32_t* q_idx, const float* q_prob, const int32_t* q_count, const float* q_mass,
                           int k, int renorm, const float* uniforms,
                           int32_t* out_tok, float* resid_mass, uint32_t* flags, const void* seg_table, int64_t n_rows, hipStream_t stream);
// the same with a scratch table of its own (residual_split_serves): the sequences' rows at n_accept are spread over many workgroups, and the
// draw reads their segments: in one launch where the scratch holds residual_scratch_bytes(...), in two where it holds the table alone
hipError_t launch_residual_split(const void* tgt_logits, int dtype, int64_t ld, int V, float temperature,
                                 int B, const int32_t* seq_off, const int32_t* n_accept, const float* tgt_max,
                                 const int32_t* q_idx, const float* q_prob, const int32_t* q_count, const float* q_mass,
                                 int k, int renorm, const float* uniforms,
                                 int32_t* out_tok, float* resid_mass, uint32_t* flags, void* scratch, size_t scratch_bytes, int64_t n_rows, hipStream_t stream);

// (launch_accept: split_table non-null: the rows' statistics are formed from that table, tgt_max / tgt_sum / tgt_lse written;
// all_rows: those of all n_rows rows of the call, else of the sequences' positions in the range)
// acceptance and residual draw of every sequence in one launch; split_table: the table holds the split layout, and the rows'
// statistics are formed from it and written; seg_table (nullable, also in launch_residual): the
// table of the n_rows target rows from launch_row_stats (small_round_table: from launch_round_stream, whose layout
// differs), with which the draw does not stream its row again
hipError_t launch_decide(const void* tgt_logits, int dtype, int64_t ld, int V, float temperature,
                         int B, const int32_t* seq_off, const int32_t* draft_tok,
                         const int32_t* q_idx, const float* q_prob, const int32_t* q_count, const float* q_mass,
                         int k, int renorm, const float* uniforms, float* tgt_max, float* tgt_sum, float* tgt_lse,
                         int32_t* n_accept, float* p_tok, float* q_tok, uint32_t* flags,
                         int32_t* out_tok, float* resid_mass, uint32_t* res_flags, const void* seg_table, int64_t n_rows,
                         bool small_round_table, bool split_table, hipStream_t stream);

hipError_t launch_resample_sparse(const void* draft_logits, int dtype, int64_t ld, int V, float temperature,
                                  int B, const int32_t* seq_off, const int32_t* n_accept,
                                  const float* draft_max, const float* draft_sum,
                                  const int32_t* p_idx, const float* p_prob, const int32_t* p_count, const float* p_mass,
                                  int k, int renorm, const float* uniforms,
                                  int32_t* out_tok, float* resid_mass, uint32_t* flags, hipStream_t stream);

// device self-check of the buffer loads' range check (csrc/selfcheck.hip); the workspace holds kCheckBytes
constexpr int kCheckBytes = 64 * 1024;
hipError_t launch_check_device(void* workspace, uint32_t* status, hipStream_t stream);
hipError_t launch_probe_clock(uint64_t* out, hipStream_t stream);

// ---- wire messages (csrc/wire.hip); fmt: 0 fp32, 1 fp16, 2 bf16 probabilities
int64_t downlink_bytes_max(int B, int k, int fmt);
int64_t uplink_bytes(int B, int n_draft, int fmt);

hipError_t launch_pack_downlink(int B, const int32_t* seq_off, const int32_t* n_accept, const int32_t* token,
                                const int32_t* idx, const float* prob, const int32_t* count, int k, int fmt,
                                void* wire, int64_t capacity, int64_t* wire_bytes, uint32_t* status, hipStream_t stream);

hipError_t launch_unpack_downlink(const void* wire, int64_t wire_bytes, int B, int k, int32_t* n_accept,
                                  int32_t* token, int32_t* idx, float* prob, int32_t* count, float* mass,
                                  uint32_t* status, hipStream_t stream);

hipError_t launch_pack_uplink(int B, int n_draft, const int32_t* seq_off, const int32_t* draft_tok,
                              const float* q_scalar, int fmt, void* wire, int64_t* wire_bytes, hipStream_t stream);

hipError_t launch_unpack_uplink(const void* wire, int64_t wire_bytes, int B, int n_max, int32_t* seq_off,
                                int32_t* draft_tok, float* q_scalar, uint32_t* status, hipStream_t stream);

}  // namespace picospec
