// Correction / bonus token (paper Section 3.3): one draw per sequence from
// norm(max(0, P_j - qhat_j)) by inverse CDF in ascending vocabulary id.
//
// One workgroup per sequence streams target row j once, in tiles of 16384 elements.  The sparse qhat
// of the matching draft row is scattered into an LDS image of the tile, so the dense pass sees
// qhat(x) at LDS speed; two images alternate, and instead of clearing an image the entries written
// for a tile are taken back after it, so that an image costs k writes per row, not V.  Within a tile
// each wave owns 1024 consecutive ids (a "segment") and leaves one partial sum per segment; the
// segment sums are kept in LDS in id order.  The crossing of u*R is then located among the segments
// and only that one segment (4 KB at most) is read again to name the token.
#include "common.hpp"
#include "decide.hpp"
#include "kernels.hpp"

namespace picospec {

namespace {

template <bool BF16>
__global__ __launch_bounds__(kThreads) void residual_kernel(
    const void* __restrict__ tgt_logits, int64_t ld, int V, float inv_T,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ n_accept,
    const float* __restrict__ tgt_max, const float* __restrict__ tgt_sum,
    const int32_t* __restrict__ q_idx, const float* __restrict__ q_prob,
    const int32_t* __restrict__ q_count, const float* __restrict__ q_mass, int k, int renorm,
    const float* __restrict__ uniforms,
    int32_t* __restrict__ out_tok, float* __restrict__ resid_mass, uint32_t* __restrict__ flags)
{
    residual_sequence<BF16>(blockIdx.x, n_accept[blockIdx.x], tgt_logits, ld, V, inv_T, seq_off, tgt_max, tgt_sum,
                            q_idx, q_prob, q_count, q_mass, k, renorm, uniforms, out_tok, resid_mass, flags);
}

// The two decisions of a sequence in one workgroup (small rounds): acceptance of its draft positions, then the
// draw at the first rejected position, without the trip of that position through device memory.
template <bool BF16>
__global__ __launch_bounds__(kThreads) void decide_kernel(
    const void* __restrict__ tgt_logits, int64_t ld, int V, float inv_T,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ draft_tok,
    const int32_t* __restrict__ q_idx, const float* __restrict__ q_prob,
    const int32_t* __restrict__ q_count, const float* __restrict__ q_mass, int k, int renorm,
    const float* __restrict__ uniforms, float* __restrict__ tgt_max, float* __restrict__ tgt_sum,
    int32_t* __restrict__ n_accept, float* __restrict__ p_tok, float* __restrict__ q_tok, uint32_t* __restrict__ flags,
    int32_t* __restrict__ out_tok, float* __restrict__ resid_mass, uint32_t* __restrict__ res_flags, int n_rows)
{
    const int first = accept_sequence<BF16>(blockIdx.x, (int)gridDim.x, n_rows, tgt_logits, ld, V, inv_T, seq_off, draft_tok, q_idx, q_prob,
                                            q_count, q_mass, k, renorm, nullptr, uniforms, tgt_max, tgt_sum,
                                            n_accept, p_tok, q_tok, flags, nullptr, nullptr);
    residual_sequence<BF16>(blockIdx.x, first, tgt_logits, ld, V, inv_T, seq_off, tgt_max, tgt_sum,
                            q_idx, q_prob, q_count, q_mass, k, renorm, uniforms, out_tok, resid_mass, res_flags);
}

// The same two kernels with the target rows' segment table at hand (no second pass over a row).
template <bool BF16, int RT>
__global__ __launch_bounds__(RT) void residual_seg_kernel(
    const void* __restrict__ tgt_logits, int64_t ld, int V, float inv_T,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ n_accept,
    const float* __restrict__ tgt_max, const SegHeader* __restrict__ table, int seg_vecs, int stride,
    const int32_t* __restrict__ q_idx, const float* __restrict__ q_prob,
    const int32_t* __restrict__ q_count, const float* __restrict__ q_mass, int k, int renorm,
    const float* __restrict__ uniforms,
    int32_t* __restrict__ out_tok, float* __restrict__ resid_mass, uint32_t* __restrict__ flags, bool by_sequence, int n_rows)
{
    residual_seg_sequence<BF16, RT>(blockIdx.x, n_accept[blockIdx.x], n_rows, n_rows - (int)gridDim.x, tgt_logits, ld, V, inv_T, seq_off, tgt_max, table, seg_vecs, stride,
                                q_idx, q_prob, q_count, q_mass, k, renorm, uniforms, out_tok, resid_mass, flags, nullptr, by_sequence);
}

// The draw that is given no table in one launch: the workgroups that sum a sequence's row (row b of the table) arrive at its word, and the last
// of them draws.
template <bool BF16, int RT>
__global__ __launch_bounds__(RT) void residual_spread_kernel(
    const void* __restrict__ tgt_logits, int64_t ld, int V, float inv_T, int n_rows,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ n_accept,
    const float* __restrict__ tgt_max, SegHeader* __restrict__ table, int seg_vecs, int stride, unsigned long long* __restrict__ words,
    const int32_t* __restrict__ q_idx, const float* __restrict__ q_prob,
    const int32_t* __restrict__ q_count, const float* __restrict__ q_mass, int k, int renorm,
    const float* __restrict__ uniforms,
    int32_t* __restrict__ out_tok, float* __restrict__ resid_mass, uint32_t* __restrict__ flags)
{
    const int b = blockIdx.y, d0 = seq_off[b], g = max(seq_off[b + 1] - d0, 0), j = n_accept[b];
    const int64_t row = (int64_t)d0 + b + min(max(j, 0), g);          // (as the draw takes it)
    const bool streams = row >= 0 && row < n_rows;                    // (offsets that leave the call's rows)
    auto open = [&] { if (threadIdx.x == 0) open_arrival(arrival_word(words, b)); };
    if (streams) row_stats_shared<BF16, RT / kWave>(row, b, (int)blockIdx.x, (int)gridDim.x, tgt_logits, ld, V, inv_T, reinterpret_cast<float2*>(table + 1), stride, open);
    else open();
    if (!arrive_last(arrival_word(words, b), gridDim.x, threadIdx.x == 0)) return;
    residual_seg_sequence<BF16, RT, true>(b, j, n_rows, n_rows - (int)gridDim.y, tgt_logits, ld, V, inv_T, seq_off, tgt_max, table, seg_vecs, stride,
                                          q_idx, q_prob, q_count, q_mass, k, renorm, uniforms, out_tok, resid_mass, flags, nullptr, true);
}

// SPLIT: the table stands in the split layout, and the rows' statistics are formed here.  PIN: RecordScan::find's, and no GUARD in the draw: 0.2 us faster in
// decide_rows_kernel, whose registers this code sets (a round of one sequence 15.7 us, 16.0 without), 0.4 slower in kernels of its own (64 sequences of 8 drafts of 128,256
// bf16 67.0, 67.5 with).
template <bool BF16, bool SPLIT, int RT, bool PIN>
__device__ __forceinline__ void decide_seg(
    const void* __restrict__ tgt_logits, int64_t ld, int V, float inv_T,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ draft_tok,
    const int32_t* __restrict__ q_idx, const float* __restrict__ q_prob,
    const int32_t* __restrict__ q_count, const float* __restrict__ q_mass, int k, int renorm,
    const float* __restrict__ uniforms, float* __restrict__ tgt_max, float* __restrict__ tgt_sum, float* __restrict__ tgt_lse,
    const SegHeader* __restrict__ table, int seg_vecs, int stride,
    int32_t* __restrict__ n_accept, float* __restrict__ p_tok, float* __restrict__ q_tok, uint32_t* __restrict__ flags,
    int32_t* __restrict__ out_tok, float* __restrict__ resid_mass, uint32_t* __restrict__ res_flags, int n_rows)
{
    __shared__ SplitStats s_stats[SPLIT ? kSplitStatsRows : 1];
    int2 rows = make_int2(0, 0);
    const int first = accept_sequence<BF16, SPLIT, PIN>(blockIdx.x, (int)gridDim.x, n_rows, tgt_logits, ld, V, inv_T, seq_off, draft_tok, q_idx, q_prob,
                                                   q_count, q_mass, k, renorm, nullptr, uniforms, tgt_max, tgt_sum,
                                                   n_accept, p_tok, q_tok, flags, nullptr, nullptr,
                                                   tgt_lse, table, seg_vecs, stride, true, SPLIT ? s_stats : nullptr, &rows);
    const int64_t t0 = (int64_t)seq_off[blockIdx.x] + blockIdx.x;
    // the waves that the draw has no use for write the log-sum-exps and end here (a barrier waits for those that are left)
    if (RT < kThreads) {
        if (__builtin_amdgcn_readfirstlane(threadIdx.x / kWave) >= RT / kWave) {
            if (SPLIT) write_split_lse(s_stats, rows, t0, inv_T, tgt_lse, RT, kThreads - RT);
            return;
        }
    } else if (SPLIT) {
        write_split_lse(s_stats, rows, t0, inv_T, tgt_lse, 0, kThreads);
    }
    residual_seg_sequence<BF16, RT, false, !PIN>(blockIdx.x, first, n_rows, n_rows - (int)gridDim.x, tgt_logits, ld, V, inv_T, seq_off, tgt_max, table, seg_vecs, stride,
                                    q_idx, q_prob, q_count, q_mass, k, renorm, uniforms, out_tok, resid_mass, res_flags,
                                    SPLIT ? s_stats : nullptr);
}

template <bool BF16, bool SPLIT, int RT>
__global__ __launch_bounds__(kThreads) void decide_seg_kernel(
    const void* __restrict__ tgt_logits, int64_t ld, int V, float inv_T,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ draft_tok,
    const int32_t* __restrict__ q_idx, const float* __restrict__ q_prob,
    const int32_t* __restrict__ q_count, const float* __restrict__ q_mass, int k, int renorm,
    const float* __restrict__ uniforms, float* __restrict__ tgt_max, float* __restrict__ tgt_sum, float* __restrict__ tgt_lse,
    const SegHeader* __restrict__ table, int seg_vecs, int stride,
    int32_t* __restrict__ n_accept, float* __restrict__ p_tok, float* __restrict__ q_tok, uint32_t* __restrict__ flags,
    int32_t* __restrict__ out_tok, float* __restrict__ resid_mass, uint32_t* __restrict__ res_flags, int n_rows)
{
    decide_seg<BF16, SPLIT, RT, false>(tgt_logits, ld, V, inv_T, seq_off, draft_tok, q_idx, q_prob, q_count, q_mass, k, renorm, uniforms, tgt_max, tgt_sum, tgt_lse,
                                table, seg_vecs, stride, n_accept, p_tok, q_tok, flags, out_tok, resid_mass, res_flags, n_rows);
}

// Short records on a table in the split layout: decide_rows, and the kernel above's code for the sequences that it leaves.
template <bool BF16>
__global__ __launch_bounds__(kThreads) void decide_rows_kernel(
    const void* __restrict__ tgt_logits, int64_t ld, int V, float inv_T,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ draft_tok,
    const int32_t* __restrict__ q_idx, const float* __restrict__ q_prob,
    const int32_t* __restrict__ q_count, const float* __restrict__ q_mass, int k, int renorm,
    const float* __restrict__ uniforms, float* __restrict__ tgt_max, float* __restrict__ tgt_sum, float* __restrict__ tgt_lse,
    const SegHeader* __restrict__ table, int seg_vecs, int stride,
    int32_t* __restrict__ n_accept, float* __restrict__ p_tok, float* __restrict__ q_tok, uint32_t* __restrict__ flags,
    int32_t* __restrict__ out_tok, float* __restrict__ resid_mass, uint32_t* __restrict__ res_flags, int n_rows)
{
    const int b = blockIdx.x, d0 = seq_off[b], d1 = seq_off[b + 1];
    if (decide_rows_serves(b, (int)gridDim.x, d0, d1, n_rows))
        decide_rows<BF16>(b, d0, d1, tgt_logits, ld, V, inv_T, draft_tok, q_idx, q_prob, q_count, q_mass, k, renorm, uniforms, tgt_max, tgt_sum,
                          tgt_lse, table, stride, n_accept, p_tok, q_tok, flags, out_tok, resid_mass, res_flags);
    else
        decide_seg<BF16, true, 256, true>(tgt_logits, ld, V, inv_T, seq_off, draft_tok, q_idx, q_prob, q_count, q_mass, k, renorm, uniforms, tgt_max, tgt_sum,
                                    tgt_lse, table, seg_vecs, stride, n_accept, p_tok, q_tok, flags, out_tok, resid_mass, res_flags, n_rows);
}

}  // namespace

static hipError_t launch_residual_seg(const void* tgt_logits, int dtype, int64_t ld, int V, float it, int B, const int32_t* seq_off,
                                      const int32_t* n_accept, const float* tgt_max, const int32_t* q_idx, const float* q_prob,
                                      const int32_t* q_count, const float* q_mass, int k, int renorm, const float* uniforms,
                                      int32_t* out_tok, float* resid_mass, uint32_t* flags, const void* seg_table, const StatsShape& sh, bool by_sequence, int64_t n_rows, hipStream_t stream)
{
#define PICOSPEC_RESIDUAL(BF, RT) \
    hipLaunchKernelGGL((residual_seg_kernel<BF, RT>), dim3(B), dim3(RT), 0, stream, tgt_logits, ld, V, it, seq_off, n_accept, tgt_max, (const SegHeader*)seg_table, sh.seg_vecs, sh.stride, q_idx, q_prob, q_count, q_mass, k, renorm, uniforms, out_tok, resid_mass, flags, by_sequence, (int)n_rows)
#define PICOSPEC_RESIDUAL_RT(BF) \
    switch (residual_seg_threads(k)) { case 256: PICOSPEC_RESIDUAL(BF, 256); break; case 512: PICOSPEC_RESIDUAL(BF, 512); break; default: PICOSPEC_RESIDUAL(BF, 1024); }
    if (dtype == 1) { PICOSPEC_RESIDUAL_RT(true) } else { PICOSPEC_RESIDUAL_RT(false) }
#undef PICOSPEC_RESIDUAL_RT
#undef PICOSPEC_RESIDUAL
    return hipGetLastError();
}

hipError_t launch_residual_split(const void* tgt_logits, int dtype, int64_t ld, int V, float temperature,
                                 int B, const int32_t* seq_off, const int32_t* n_accept, const float* tgt_max,
                                 const int32_t* q_idx, const float* q_prob, const int32_t* q_count, const float* q_mass,
                                 int k, int renorm, const float* uniforms,
                                 int32_t* out_tok, float* resid_mass, uint32_t* flags, void* scratch, size_t scratch_bytes, int64_t n_rows, hipStream_t stream)
{
    const StatsShape sh = split_stats_shape(dtype, V);
    const float inv_T = 1.0f / temperature;
    if (residual_one_launch(dtype, B, V, k) && scratch_bytes >= residual_scratch_bytes(dtype, B, V)) {
        const dim3 grid(spread_parts(sh.stride, residual_seg_threads(k) / 64, B), B);
        unsigned long long* const words = (unsigned long long*)((char*)scratch + residual_words_at(dtype, B, V));
#define PICOSPEC_RESIDUAL_SPREAD(BF, RT) \
        hipLaunchKernelGGL((residual_spread_kernel<BF, RT>), grid, dim3(RT), 0, stream, tgt_logits, ld, V, inv_T, (int)n_rows, seq_off, n_accept, tgt_max, (SegHeader*)scratch, sh.seg_vecs, sh.stride, words, q_idx, q_prob, q_count, q_mass, k, renorm, uniforms, out_tok, resid_mass, flags)
        static_assert(kResidualSplitK <= 2048, "records for 512 threads");
        if (residual_seg_threads(k) == 256) { if (dtype == 1) PICOSPEC_RESIDUAL_SPREAD(true, 256); else PICOSPEC_RESIDUAL_SPREAD(false, 256); }
        else                                { if (dtype == 1) PICOSPEC_RESIDUAL_SPREAD(true, 512); else PICOSPEC_RESIDUAL_SPREAD(false, 512); }
#undef PICOSPEC_RESIDUAL_SPREAD
        return hipGetLastError();
    }
    if (hipError_t e = launch_row_stats_parts(tgt_logits, dtype, ld, (int)n_rows, V, temperature, B, 0, seq_off, nullptr, nullptr, scratch, stream, n_accept))
        return e;
    return launch_residual_seg(tgt_logits, dtype, ld, V, inv_T, B, seq_off, n_accept, tgt_max, q_idx, q_prob, q_count, q_mass,
                               k, renorm, uniforms, out_tok, resid_mass, flags, scratch, sh, true, n_rows, stream);
}

hipError_t launch_residual(const void* tgt_logits, int dtype, int64_t ld, int V, float temperature,
                           int B, const int32_t* seq_off, const int32_t* n_accept,
                           const float* tgt_max, const float* tgt_sum,
                           const int32_t* q_idx, const float* q_prob, const int32_t* q_count, const float* q_mass,
                           int k, int renorm, const float* uniforms,
                           int32_t* out_tok, float* resid_mass, uint32_t* flags, const void* seg_table, int64_t n_rows, hipStream_t stream)
{
    if (seg_table) {
        if (B == 0) return hipSuccess;
        const StatsShape sh = split_stats_serves(n_rows, V) ? split_stats_shape(dtype, V) : stats_shape(dtype, n_rows, V);   // (as the verification laid it out)
        return launch_residual_seg(tgt_logits, dtype, ld, V, 1.0f / temperature, B, seq_off, n_accept, tgt_max, q_idx, q_prob, q_count, q_mass,
                                   k, renorm, uniforms, out_tok, resid_mass, flags, seg_table, sh, false, n_rows, stream);
    }
    static DeviceFlags limit_raised[2] = {};
    const size_t smem = sizeof(ResidualShared);
    auto f32 = residual_kernel<false>;
    auto b16 = residual_kernel<true>;
    const int which = dtype == 1;
    {
        int dev = 0;
        hipError_t e = raise_lds_limit_once(which ? (const void*)b16 : (const void*)f32, smem, limit_raised[which], dev);
        if (e != hipSuccess) return e;
    }
    if (B == 0) return hipSuccess;
    const float inv_T = 1.0f / temperature;
    if (which) hipLaunchKernelGGL(b16, dim3(B), dim3(kThreads), smem, stream, tgt_logits, ld, V, inv_T, seq_off, n_accept, tgt_max, tgt_sum, q_idx, q_prob, q_count, q_mass, k, renorm, uniforms, out_tok, resid_mass, flags);
    else       hipLaunchKernelGGL(f32, dim3(B), dim3(kThreads), smem, stream, tgt_logits, ld, V, inv_T, seq_off, n_accept, tgt_max, tgt_sum, q_idx, q_prob, q_count, q_mass, k, renorm, uniforms, out_tok, resid_mass, flags);
    return hipGetLastError();
}

hipError_t launch_decide(const void* tgt_logits, int dtype, int64_t ld, int V, float temperature,
                         int B, const int32_t* seq_off, const int32_t* draft_tok,
                         const int32_t* q_idx, const float* q_prob, const int32_t* q_count, const float* q_mass,
                         int k, int renorm, const float* uniforms, float* tgt_max, float* tgt_sum, float* tgt_lse,
                         int32_t* n_accept, float* p_tok, float* q_tok, uint32_t* flags,
                         int32_t* out_tok, float* resid_mass, uint32_t* res_flags, const void* seg_table, int64_t n_rows,
                         bool small_round_table, bool split_table, hipStream_t stream)
{
    if (seg_table) {
        if (B == 0) return hipSuccess;
        const float it = 1.0f / temperature;
        const StatsShape sh = split_table ? split_stats_shape(dtype, V) : small_round_table ? round_stats_shape(dtype, V) : stats_shape(dtype, n_rows, V);
#define PICOSPEC_DECIDE_ARGS dim3(B), dim3(kThreads), 0, stream, tgt_logits, ld, V, it, seq_off, draft_tok, q_idx, q_prob, q_count, q_mass, k, renorm, uniforms, tgt_max, tgt_sum, tgt_lse, (const SegHeader*)seg_table, sh.seg_vecs, sh.stride, n_accept, p_tok, q_tok, flags, out_tok, resid_mass, res_flags, (int)n_rows
#define PICOSPEC_DECIDE(BF, SP, RT) hipLaunchKernelGGL((decide_seg_kernel<BF, SP, RT>), PICOSPEC_DECIDE_ARGS)
#define PICOSPEC_DECIDE_RT(BF, SP) \
        switch (residual_seg_threads(k)) { case 256: PICOSPEC_DECIDE(BF, SP, 256); break; case 512: PICOSPEC_DECIDE(BF, SP, 512); break; default: PICOSPEC_DECIDE(BF, SP, 1024); }
        // (the table of a row has to fit the registers of one wave: fp32 rows of up to 327,680, bf16 of up to 655,360)
        if (split_table && k <= kDecideRowsK && sh.stride <= kDecideRowsSegs) {
            if (dtype == 1) hipLaunchKernelGGL(decide_rows_kernel<true>, PICOSPEC_DECIDE_ARGS);
            else            hipLaunchKernelGGL(decide_rows_kernel<false>, PICOSPEC_DECIDE_ARGS);
        }
        else if (split_table) { if (dtype == 1) { PICOSPEC_DECIDE_RT(true, true) } else { PICOSPEC_DECIDE_RT(false, true) } }
        else             { if (dtype == 1) { PICOSPEC_DECIDE_RT(true, false) } else { PICOSPEC_DECIDE_RT(false, false) } }
#undef PICOSPEC_DECIDE_RT
#undef PICOSPEC_DECIDE
#undef PICOSPEC_DECIDE_ARGS
        return hipGetLastError();
    }
    static DeviceFlags limit_raised[2] = {};
    const size_t smem = sizeof(ResidualShared);
    auto f32 = decide_kernel<false>;
    auto b16 = decide_kernel<true>;
    const int which = dtype == 1;
    {
        int dev = 0;
        hipError_t e = raise_lds_limit_once(which ? (const void*)b16 : (const void*)f32, smem, limit_raised[which], dev);
        if (e != hipSuccess) return e;
    }
    if (B == 0) return hipSuccess;
    const float inv_T = 1.0f / temperature;
    if (which) hipLaunchKernelGGL(b16, dim3(B), dim3(kThreads), smem, stream, tgt_logits, ld, V, inv_T, seq_off, draft_tok, q_idx, q_prob, q_count, q_mass, k, renorm, uniforms, tgt_max, tgt_sum, n_accept, p_tok, q_tok, flags, out_tok, resid_mass, res_flags, (int)n_rows);
    else       hipLaunchKernelGGL(f32, dim3(B), dim3(kThreads), smem, stream, tgt_logits, ld, V, inv_T, seq_off, draft_tok, q_idx, q_prob, q_count, q_mass, k, renorm, uniforms, tgt_max, tgt_sum, n_accept, p_tok, q_tok, flags, out_tok, resid_mass, res_flags, (int)n_rows);
    return hipGetLastError();
}

}  // namespace picospec
