// Parallel verification (paper Section 3.3): softmax statistics of every target row in one
// streaming pass, then per sequence the sparse lookup of the drafted token's probability, the
// acceptance test u < min(1, p/qhat) and the first rejected position.
#include <algorithm>

#include "common.hpp"
#include "decide.hpp"
#include "kernels.hpp"

namespace picospec {

namespace {

template <bool BF16, int NV, int THREADS>
__global__ __launch_bounds__(THREADS) void row_stats_kernel(
    const void* __restrict__ logits, int64_t ld, int V, float inv_T,
    float* __restrict__ row_max, float* __restrict__ row_sum, float* __restrict__ row_lse)
{
    row_stats_row<BF16, NV, THREADS>(blockIdx.x, logits, ld, V, inv_T, row_max, row_sum, row_lse);
}

// The statistics together with the row's segment table (row_stats_seg_row); workgroup 0 also writes the table's header.
template <bool BF16, int NV, int THREADS>
__global__ __launch_bounds__(THREADS) void row_stats_seg_kernel(
    const void* __restrict__ logits, int64_t ld, int V, float inv_T,
    float* __restrict__ row_max, float* __restrict__ row_sum, float* __restrict__ row_lse,
    SegHeader* __restrict__ header, int seg_stride)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *header = SegHeader{kSegMagic, NV * kWave, seg_stride, (int32_t)gridDim.x};
    row_stats_seg_row<BF16, NV, THREADS>(blockIdx.x, logits, ld, V, inv_T, row_max, row_sum, row_lse,
                                         reinterpret_cast<float2*>(header + 1), seg_stride);
}

// The same for the target rows begin_b..end_b of every sequence only (verification of a part of the
// draft): workgroup (t, b) of a (gamma_max + 1) x B grid takes position t of sequence b or leaves.
template <bool BF16, int NV, int THREADS>
__global__ __launch_bounds__(THREADS) void row_stats_range_kernel(
    const void* __restrict__ logits, int64_t ld, int V, float inv_T,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ pos_begin, const int32_t* __restrict__ pos_end,
    float* __restrict__ row_max, float* __restrict__ row_sum, float* __restrict__ row_lse)
{
    const int b = blockIdx.y, t = blockIdx.x;
    const int d0 = seq_off[b];
    int g = seq_off[b + 1] - d0;
    if (g < 0) g = 0;
    int begin, end;
    clamp_range(pos_begin, pos_end, b, g, begin, end);
    if (t < begin || t > end) return;
    row_stats_row<BF16, NV, THREADS>((int64_t)d0 + b + t, logits, ld, V, inv_T, row_max, row_sum, row_lse);
}

// Rows that leave the chip partly idle: the segment tables alone (split layout).  Bound by the memory's latency up to some
// 100 rows and by its rate from there (196 bf16 rows of 128,256 in 10.9 us: 4.6 TB/s).  One workgroup per row -> here: 16 sequences of 1 to 8 drafts, fp32 rows of 151,936: 17.8 -> 9.3 us; half of 24 such drafts, rows of 33,001: 8.2 -> 5.0 us.  grid: (workgroups per row, rows), or (.., gamma_max + 1, B) for the
// target rows of a range of positions, or (.., 1, B) for every sequence's row at n_accept (row b of the table).
template <bool BF16>
__global__ __launch_bounds__(256) void row_stats_parts_kernel(
    const void* __restrict__ logits, int64_t ld, int V, float inv_T, int n_rows, int seg_stride,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ pos_begin, const int32_t* __restrict__ pos_end,
    const int32_t* __restrict__ n_accept, SegHeader* __restrict__ header)
{
    if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0)
        *header = SegHeader{kSegMagicSplit, kSplitStatsNV * kWave, seg_stride, n_rows};
    int64_t row = blockIdx.y;
    if (seq_off) {                                    // position t of sequence b, or nothing
        const int b = blockIdx.z, d0 = seq_off[b];
        const int g = max(seq_off[b + 1] - d0, 0);
        int t = blockIdx.y;
        if (n_accept) {
            t = min(max(n_accept[b], 0), g);          // (as the draw takes it)
        } else {
            int begin, end;
            clamp_range(pos_begin, pos_end, b, g, begin, end);
            if (t < begin || t > end) return;
        }
        row = (int64_t)d0 + b + t;
        if (row < 0 || row >= n_rows) return;           // (offsets that leave the call's rows)
    }
    row_stats_parts<BF16>(row, n_accept ? (int64_t)blockIdx.z : row, (int)blockIdx.x, logits, ld, V, inv_T, reinterpret_cast<float2*>(header + 1), seg_stride);
}

// The statistics of rows whose table stands in the split layout: one wave per row.
template <bool BF16>
__global__ __launch_bounds__(256) void row_stats_finish_kernel(
    const void* __restrict__ logits, int64_t ld, int V, float inv_T, int n_rows, const SegHeader* __restrict__ header,
    int seg_vecs, int seg_stride, float* __restrict__ row_max, float* __restrict__ row_sum, float* __restrict__ row_lse)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t row = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (row >= n_rows) return;
    const RowView rv = row_view<BF16>(logits, ld, row, V);
    const int nq = (rv.L + Vec<BF16>::N - 1) / Vec<BF16>::N, n_seg = (nq + seg_vecs - 1) / seg_vecs;
    float M;
    double S;
    const float2* const seg_row = reinterpret_cast<const float2*>(header + 1) + row * (int64_t)seg_stride;
    TableStats stats;
    stats.load(seg_row, n_seg);
    stats.combine(seg_row, n_seg, 1.4426950408889634f * inv_T, M, S);
    if (lane == 0) {
        row_max[row] = M;
        row_sum[row] = (float)S;
        if (row_lse) row_lse[row] = (float)((double)M * (double)inv_T + log(S));
    }
}

// The same in one launch: the last workgroup of a row to arrive (word `row` of `words`) forms its statistics.
template <bool BF16>
__global__ __launch_bounds__(512) void row_stats_spread_kernel(
    const void* __restrict__ logits, int64_t ld, int V, float inv_T, float2* __restrict__ table, int seg_stride, unsigned long long* __restrict__ words,
    float* __restrict__ row_max, float* __restrict__ row_sum, float* __restrict__ row_lse)
{
    const int64_t row = blockIdx.y;
    row_stats_shared<BF16, 8>(row, row, (int)blockIdx.x, (int)gridDim.x, logits, ld, V, inv_T, table, seg_stride,
                              [&] { if (threadIdx.x == 0) open_arrival(arrival_word(words, row)); });
    if (!arrive_last(arrival_word(words, row), gridDim.x, threadIdx.x == 0) || threadIdx.x >= kWave) return;
    const RowView rv = row_view<BF16>(logits, ld, row, V);
    const int n_seg = stats_segments((rv.L + Vec<BF16>::N - 1) / Vec<BF16>::N);
    const float2* const seg_row = table + row * (int64_t)seg_stride;
    float M;
    double S;
    TableStats stats;
    stats.load<true>(seg_row, n_seg);
    stats.combine<true>(seg_row, n_seg, 1.4426950408889634f * inv_T, M, S);
    if (threadIdx.x == 0) {
        row_max[row] = M;
        row_sum[row] = (float)S;
        if (row_lse) row_lse[row] = (float)((double)M * (double)inv_T + log(S));
    }
}

// Verification of few rows in one launch: the workgroups that sum a sequence's target rows, and one that looks its positions up, arrive at its
// word, and the last of them decides (decide_spread).  ranged: pos_begin / pos_end as in row_stats_range_kernel, grid (workgroups per row, 1 + gamma_max + 1,
// B), y = 0 the looking ones; else grid (.., look_rows + rows), the first look_rows * gridDim.x the looking ones: a row belongs to the
// sequence whose offsets hold it, those in front of the first to the first and those behind the last to the last.  Where the offsets do
// not ascend or leave the call's rows all workgroups arrive at one word, and the last of all takes the sequences one by one.  words: B of the
// sequences, one more.
struct VerifySpreadArgs {
    global_ptr<const void> tgt_logits;
    int64_t ld;
    int V;
    float inv_T;
    int B, n_rows, look_rows, stride;
    bool ranged;
    global_ptr<const int32_t> seq_off, pos_begin, pos_end;
    global_ptr<SegHeader> table;
    global_ptr<unsigned long long> words, found;
    global_ptr<const int32_t> draft_tok, q_idx;
    global_ptr<const float> q_prob;
    global_ptr<const int32_t> q_count;
    global_ptr<const float> q_mass;
    int k, renorm;
    global_ptr<const float> q_scalar, uniforms;
    global_ptr<float> tgt_max, tgt_sum, tgt_lse;
    global_ptr<int32_t> n_accept;
    global_ptr<float> p_tok, q_tok;
    global_ptr<uint32_t> flags;
};

template <bool BF16>
__global__ __launch_bounds__(512, 6) void verify_spread_kernel(const VerifySpreadArgs)
{
    constexpr int kWavesHere = 8;
    // the sequence whose word this workgroup arrives at (B: all of them at one), its first draft row, its positions and what was wrong with them
    __shared__ int s_group, s_d0, s_begin, s_end;
    __shared__ unsigned s_wrong;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int parts = (int)gridDim.x;
    // the positions of sequence s, whose offsets are d0 and d1
    auto span_of = [](auto a, int s, int d0, int d1, int& begin, int& end) {
        const int g = max(d1 - d0, 0);
        unsigned fl = d1 < d0 ? 8u : 0u;
        if (clamp_range(plain(a->pos_begin), plain(a->pos_end), s, g, begin, end)) fl |= 8u;
        return fl;
    };
    auto look_up = [](auto a, int s, int d0, int begin, int end) {
        look_up_positions<BF16, kWavesHere>(s, d0, begin, end, plain(a->tgt_logits), a->ld, a->V, a->n_rows, a->n_rows - a->B, plain(a->draft_tok), plain(a->q_idx), plain(a->q_prob),
                                            plain(a->q_count), plain(a->q_mass), a->k, a->renorm, plain(a->q_scalar), plain(a->found));
    };
    int arrivals = 1;
    bool looks;
    {
        const auto a = args_here<VerifySpreadArgs>();
        const int B = a->B, n_rows = a->n_rows;
        const int32_t* const seq_off = plain(a->seq_off);
        const bool ranged = a->ranged;
        looks = (int)blockIdx.y < a->look_rows;
        int b = looks ? (int)blockIdx.y * parts + (int)blockIdx.x : -1, d0 = 0, begin = 0, end = 0;
        unsigned wrong = 0;
        int64_t row = (int64_t)blockIdx.y - a->look_rows;
        if (ranged) {
            if (looks && blockIdx.x > 0) return;
            b = blockIdx.z;
            d0 = seq_off[b];
            wrong = span_of(a, b, d0, seq_off[b + 1], begin, end);
            const int t = (int)row, last = min(end, (int)gridDim.y - 2), first = min(begin, last + 1);     // (positions the grid does not reach arrive nowhere)
            if (!looks && (t < first || t > last)) return;
            arrivals = (last - first + 1) * parts + 1;
            row += (int64_t)d0 + b;
        } else if (looks && b >= B) {
            return;
        }
        const bool streams = !looks && row >= 0 && row < n_rows;
        if (ranged && looks) look_up(a, b, d0, begin, end);
        auto open = [&] {
            if (wave != 0) return;
            int group = b;
            if (!ranged) {
                // the row's sequence, and whether the offsets are sound (split_stats_serves: at most kSplitStatsRows sequences)
                static_assert(kSplitStatsRows < 4 * kWave, "four offsets per lane");
                int off[4], next[4], in_front = 0;
                bool sound = true;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = min(u * kWave + lane, B);
                    off[u] = seq_off[i];
                    next[u] = seq_off[min(i + 1, B)];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = u * kWave + lane;
                    sound = sound && off[u] >= 0 && next[u] >= off[u] && next[u] <= n_rows - B;
                    in_front += __popcll(__ballot(i > 0 && i < B && off[u] + i <= row));          // sequences 1 .. B - 1 that begin at or in front of the row
                }
                if (__ballot(!sound) == 0ull) {
                    if (!looks) group = in_front;
                    const int g0 = __builtin_amdgcn_readfirstlane(group);
                    const int d1 = seq_off[g0 + 1];
                    d0 = seq_off[g0];
                    end = d1 - d0;
                    const int start = g0 > 0 ? d0 + g0 : 0, stop = g0 + 1 < B ? d1 + g0 + 1 : n_rows;
                    arrivals = (stop - start) * parts + 1;
                } else {
                    group = B;
                    arrivals = n_rows * parts + B;
                }
            }
            if (threadIdx.x == 0) {
                s_group = group; s_d0 = d0; s_begin = begin; s_end = end; s_wrong = wrong;
                open_arrival(arrival_word(plain(a->words), group));
            }
        };
        if (blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0 && threadIdx.x == 0) *plain(a->table) = SegHeader{kSegMagicSplit, kSplitStatsNV * kWave, a->stride, n_rows};
        if (streams) row_stats_shared<BF16, kWavesHere>(row, row, (int)blockIdx.x, parts, plain(a->tgt_logits), a->ld, a->V, a->inv_T, reinterpret_cast<float2*>(plain(a->table) + 1), a->stride, open);
        else open();
    }
    auto here = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    if (looks) {
        const auto a = args_here<VerifySpreadArgs>();
        __syncthreads();
        if (!a->ranged && here(s_group) < a->B) look_up(a, here(s_group), here(s_d0), here(s_begin), here(s_end));
    }
    {
        const auto a = args_here<VerifySpreadArgs>();
        // (the word's place is formed by the thread that uses it: s_group is its own)
        if (!arrive_last(arrival_word(plain(a->words), threadIdx.x == 0 ? s_group : 0), (unsigned)arrivals, threadIdx.x == 0)) return;
    }
    const auto a = args_here<VerifySpreadArgs>();
    const int B = a->B, group = here(s_group);
    const bool ranged = a->ranged;
    int d0 = here(s_d0), begin = here(s_begin), end = here(s_end);
    unsigned wrong = (unsigned)here((int)s_wrong);
    auto look_again = [](int64_t rd, int64_t rt) {
        const auto a = args_here<VerifySpreadArgs>();
        return look_up_position<BF16>(rd, rt, plain(a->tgt_logits), a->ld, a->V, plain(a->draft_tok), plain(a->q_idx), plain(a->q_prob), plain(a->q_count),
                                      plain(a->q_mass), a->k, a->renorm, plain(a->q_scalar));
    };
    for (int s = group < B ? group : 0, n = group < B ? 1 : B; n > 0; --n, ++s) {
        if (group == B) {
            d0 = plain(a->seq_off)[s];
            wrong = span_of(a, s, d0, plain(a->seq_off)[s + 1], begin, end);
            look_up(a, s, d0, begin, end);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
        }
        const int t0 = d0 + s;
        decide_spread<BF16, kWavesHere>(s, d0, wrong, begin, end, !ranged && s == 0 ? min(begin, -t0) : begin,
                                        !ranged && s + 1 == B ? max(end + 1, a->n_rows - t0) : end + 1, plain(a->tgt_logits), a->ld, a->V, a->inv_T, a->n_rows, a->n_rows - B,
                                        plain(a->uniforms), plain(a->tgt_max), plain(a->tgt_sum), plain(a->tgt_lse), plain(a->n_accept), plain(a->p_tok), plain(a->q_tok), plain(a->flags),
                                        plain(a->table), a->stride, plain(a->found), look_again);
        __syncthreads();
    }
}

// picospec_verify's second kernel: one workgroup per sequence (accept_sequence, decide.hpp).
// Up to 64 registers without a table: two workgroups share a CU (512 sequences, k = 2048: 14.3 -> 10.4 us); calls with one have a CU for each.
template <bool BF16, bool TABLE>
__global__ __launch_bounds__(kThreads, TABLE ? 4 : 8) void accept_kernel(
    const void* __restrict__ tgt_logits, int64_t ld, int V, float inv_T, int B,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ draft_tok,
    const int32_t* __restrict__ q_idx, const float* __restrict__ q_prob,
    const int32_t* __restrict__ q_count, const float* __restrict__ q_mass, int k, int renorm,
    const float* __restrict__ q_scalar, const float* __restrict__ uniforms,
    float* __restrict__ tgt_max, float* __restrict__ tgt_sum, float* __restrict__ tgt_lse,
    int32_t* __restrict__ n_accept, float* __restrict__ p_tok, float* __restrict__ q_tok,
    uint32_t* __restrict__ flags, const int32_t* __restrict__ pos_begin, const int32_t* __restrict__ pos_end,
    const SegHeader* __restrict__ table, int seg_vecs, int stride, int n_rows, bool all_rows)
{
    accept_sequence<BF16, TABLE>(blockIdx.x, (int)gridDim.x, n_rows, tgt_logits, ld, V, inv_T, seq_off, draft_tok, q_idx, q_prob, q_count, q_mass, k,
                                 renorm, q_scalar, uniforms, tgt_max, tgt_sum, n_accept, p_tok, q_tok, flags, pos_begin, pos_end,
                                 tgt_lse, table, seg_vecs, stride, all_rows);
}

}  // namespace

hipError_t launch_row_stats_range(const void* logits, int dtype, int64_t ld, int V, float temperature, int B,
                                  int gamma_max, const int32_t* seq_off, const int32_t* pos_begin,
                                  const int32_t* pos_end, float* row_max, float* row_sum, float* row_lse,
                                  hipStream_t stream)
{
    if (B == 0) return hipSuccess;
    const float inv_T = 1.0f / temperature;
    const int64_t n_rows = (int64_t)B * (gamma_max + 1);          // (an upper bound: workgroups outside the ranges leave at once)
    const dim3 grid(gamma_max + 1, B);
#define PICOSPEC_ROW_STATS_RANGE(BF, NVV, TH) \
    hipLaunchKernelGGL((row_stats_range_kernel<BF, NVV, TH>), grid, dim3(TH), 0, stream, logits, ld, V, inv_T, seq_off, pos_begin, pos_end, row_max, row_sum, row_lse)
    if (dtype != 1)           PICOSPEC_ROW_STATS_RANGE(false, 4, kThreads);
    else if (n_rows >= 2048)  PICOSPEC_ROW_STATS_RANGE(true, 4, 256);
    else if (n_rows >= 1024)  PICOSPEC_ROW_STATS_RANGE(true, 2, 512);
    else                      PICOSPEC_ROW_STATS_RANGE(true, 2, kThreads);
#undef PICOSPEC_ROW_STATS_RANGE
    return hipGetLastError();
}

hipError_t launch_row_stats(const void* logits, int dtype, int64_t ld, int n_rows, int V, float temperature,
                            float* row_max, float* row_sum, float* row_lse, void* seg_table, hipStream_t stream)
{
    if (n_rows == 0) return hipSuccess;
    const float inv_T = 1.0f / temperature;
    const StatsShape sh = stats_shape(dtype, n_rows, V);
#define PICOSPEC_ROW_STATS(BF, NVV, TH) \
    do { if (seg_table) hipLaunchKernelGGL((row_stats_seg_kernel<BF, NVV, TH>), dim3(n_rows), dim3(TH), 0, stream, logits, ld, V, inv_T, row_max, row_sum, row_lse, (SegHeader*)seg_table, sh.stride); \
         else hipLaunchKernelGGL((row_stats_kernel<BF, NVV, TH>), dim3(n_rows), dim3(TH), 0, stream, logits, ld, V, inv_T, row_max, row_sum, row_lse); } while (0)
    if (dtype != 1)              PICOSPEC_ROW_STATS(false, 4, kThreads);
    else if (sh.threads == 256)  PICOSPEC_ROW_STATS(true, 4, 256);
    else if (sh.threads == 512)  PICOSPEC_ROW_STATS(true, 2, 512);
    else                         PICOSPEC_ROW_STATS(true, 2, kThreads);
#undef PICOSPEC_ROW_STATS
    return hipGetLastError();
}

hipError_t launch_row_stats_parts(const void* logits, int dtype, int64_t ld, int n_rows, int V, float temperature, int B, int gamma_max, const int32_t* seq_off, const int32_t* pos_begin, const int32_t* pos_end,
                                  void* seg_table, hipStream_t stream, const int32_t* n_accept)
{
    if (n_rows == 0 || (seq_off && B == 0)) return hipSuccess;
    const float inv_T = 1.0f / temperature;
    const StatsShape sh = split_stats_shape(dtype, V);
    const dim3 grid(stats_parts(sh.stride), n_accept ? 1 : seq_off ? gamma_max + 1 : n_rows, seq_off ? B : 1);
    if (dtype == 1) hipLaunchKernelGGL(row_stats_parts_kernel<true>, grid, dim3(256), 0, stream, logits, ld, V, inv_T, n_rows, sh.stride, seq_off, pos_begin, pos_end, n_accept, (SegHeader*)seg_table);
    else            hipLaunchKernelGGL(row_stats_parts_kernel<false>, grid, dim3(256), 0, stream, logits, ld, V, inv_T, n_rows, sh.stride, seq_off, pos_begin, pos_end, n_accept, (SegHeader*)seg_table);
    return hipGetLastError();
}

hipError_t launch_row_stats_finish(const void* logits, int dtype, int64_t ld, int n_rows, int V, float temperature,
                                   const void* seg_table, float* row_max, float* row_sum, float* row_lse, hipStream_t stream)
{
    if (n_rows == 0) return hipSuccess;
    const float inv_T = 1.0f / temperature;
    const StatsShape sh = split_stats_shape(dtype, V);
    const dim3 grid((n_rows + 3) / 4);
    if (dtype == 1) hipLaunchKernelGGL(row_stats_finish_kernel<true>, grid, dim3(256), 0, stream, logits, ld, V, inv_T, n_rows, (const SegHeader*)seg_table, sh.seg_vecs, sh.stride, row_max, row_sum, row_lse);
    else            hipLaunchKernelGGL(row_stats_finish_kernel<false>, grid, dim3(256), 0, stream, logits, ld, V, inv_T, n_rows, (const SegHeader*)seg_table, sh.seg_vecs, sh.stride, row_max, row_sum, row_lse);
    return hipGetLastError();
}

hipError_t launch_row_stats_spread(const void* logits, int dtype, int64_t ld, int n_rows, int V, float temperature,
                                   void* scratch, float* row_max, float* row_sum, float* row_lse, hipStream_t stream)
{
    if (n_rows == 0) return hipSuccess;
    const float inv_T = 1.0f / temperature;
    const StatsShape sh = split_stats_shape(dtype, V);
    const dim3 grid(spread_parts(sh.stride, 8, n_rows), n_rows);
    unsigned long long* const words = (unsigned long long*)((char*)scratch + row_stats_words_at(dtype, n_rows, V));
    float2* const table = (float2*)scratch;
    if (dtype == 1) hipLaunchKernelGGL(row_stats_spread_kernel<true>, grid, dim3(512), 0, stream, logits, ld, V, inv_T, table, sh.stride, words, row_max, row_sum, row_lse);
    else            hipLaunchKernelGGL(row_stats_spread_kernel<false>, grid, dim3(512), 0, stream, logits, ld, V, inv_T, table, sh.stride, words, row_max, row_sum, row_lse);
    return hipGetLastError();
}

hipError_t launch_verify_spread(const void* tgt_logits, int dtype, int64_t ld, int V, float temperature,
                                int B, int64_t n_rows, const int32_t* seq_off, const int32_t* draft_tok,
                                const int32_t* q_idx, const float* q_prob, const int32_t* q_count, const float* q_mass,
                                int k, int renorm, const float* q_scalar, const float* uniforms,
                                float* tgt_max, float* tgt_sum, float* tgt_lse,
                                int32_t* n_accept, float* p_tok, float* q_tok, uint32_t* flags,
                                bool ranged, const int32_t* pos_begin, const int32_t* pos_end, int gamma_max,
                                void* scratch, hipStream_t stream)
{
    const float inv_T = 1.0f / temperature;
    const StatsShape sh = split_stats_shape(dtype, V);
    const int parts = spread_parts(sh.stride, 8, ranged ? std::min<int64_t>(n_rows, (int64_t)B * (gamma_max + 1)) : n_rows), look_rows = ranged ? 1 : (B + parts - 1) / parts;
    const dim3 grid = ranged ? dim3(parts, look_rows + gamma_max + 1, B) : dim3(parts, (unsigned)(look_rows + n_rows));
    unsigned long long* const words = (unsigned long long*)((char*)scratch + verify_words_at(dtype, n_rows, V));
    unsigned long long* const found = (unsigned long long*)((char*)scratch + verify_found_at(dtype, n_rows, B, V));
#define PICOSPEC_GLOBAL(T, p) (global_ptr<T>)(p)
    const VerifySpreadArgs args{PICOSPEC_GLOBAL(const void, tgt_logits), ld, V, inv_T, B, (int)n_rows, look_rows, sh.stride, ranged,
                                PICOSPEC_GLOBAL(const int32_t, seq_off), PICOSPEC_GLOBAL(const int32_t, pos_begin), PICOSPEC_GLOBAL(const int32_t, pos_end),
                                PICOSPEC_GLOBAL(SegHeader, scratch), PICOSPEC_GLOBAL(unsigned long long, words), PICOSPEC_GLOBAL(unsigned long long, found),
                                PICOSPEC_GLOBAL(const int32_t, draft_tok), PICOSPEC_GLOBAL(const int32_t, q_idx), PICOSPEC_GLOBAL(const float, q_prob),
                                PICOSPEC_GLOBAL(const int32_t, q_count), PICOSPEC_GLOBAL(const float, q_mass), k, renorm,
                                PICOSPEC_GLOBAL(const float, q_scalar), PICOSPEC_GLOBAL(const float, uniforms),
                                PICOSPEC_GLOBAL(float, tgt_max), PICOSPEC_GLOBAL(float, tgt_sum), PICOSPEC_GLOBAL(float, tgt_lse),
                                PICOSPEC_GLOBAL(int32_t, n_accept), PICOSPEC_GLOBAL(float, p_tok), PICOSPEC_GLOBAL(float, q_tok), PICOSPEC_GLOBAL(uint32_t, flags)};
#undef PICOSPEC_GLOBAL
    if (dtype == 1) hipLaunchKernelGGL(verify_spread_kernel<true>, grid, dim3(512), 0, stream, args);
    else            hipLaunchKernelGGL(verify_spread_kernel<false>, grid, dim3(512), 0, stream, args);
    return hipGetLastError();
}

hipError_t launch_accept(const void* tgt_logits, int dtype, int64_t ld, int V, float temperature,
                         int B, const int32_t* seq_off, const int32_t* draft_tok,
                         const int32_t* q_idx, const float* q_prob, const int32_t* q_count, const float* q_mass,
                         int k, int renorm, const float* q_scalar, const float* uniforms,
                         float* tgt_max, float* tgt_sum, float* tgt_lse,
                         int32_t* n_accept, float* p_tok, float* q_tok, uint32_t* flags,
                         const int32_t* pos_begin, const int32_t* pos_end,
                         const void* split_table, int64_t n_rows, bool all_rows, hipStream_t stream)
{
    if (B == 0) return hipSuccess;
    const float inv_T = 1.0f / temperature;
    const StatsShape sh = split_stats_shape(dtype, V);
#define PICOSPEC_ACCEPT(BF, TA) \
    hipLaunchKernelGGL((accept_kernel<BF, TA>), dim3(B), dim3(kThreads), 0, stream, tgt_logits, ld, V, inv_T, B, seq_off, draft_tok, q_idx, q_prob, q_count, q_mass, k, renorm, q_scalar, uniforms, tgt_max, tgt_sum, tgt_lse, n_accept, p_tok, q_tok, flags, pos_begin, pos_end, (const SegHeader*)split_table, sh.seg_vecs, sh.stride, (int)n_rows, all_rows)
    if (split_table) { if (dtype == 1) PICOSPEC_ACCEPT(true, true); else PICOSPEC_ACCEPT(false, true); }
    else             { if (dtype == 1) PICOSPEC_ACCEPT(true, false); else PICOSPEC_ACCEPT(false, false); }
#undef PICOSPEC_ACCEPT
    return hipGetLastError();
}

}  // namespace picospec
