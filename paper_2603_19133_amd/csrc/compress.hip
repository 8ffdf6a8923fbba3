// The kernels of the sparse Top-K compression (compress_row.hpp holds what a workgroup does with a row): the fast
// variants and the careful one, the kernels that stream a round's draft and target rows at once, and the drafter's
// draw from a record.
#include "compress_row.hpp"

namespace picospec {

namespace {

template <bool BF16, bool SMALL>
__global__ __launch_bounds__(kT, SMALL ? 6 : 4) void compress_kernel(
    const void* __restrict__ logits, int64_t ld, int V, float inv_T, int k, float top_p,
    int32_t* __restrict__ idx, float* __restrict__ prob, int32_t* __restrict__ count,
    float* __restrict__ mass, float* __restrict__ lse,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ n_accept, int rank_opt)
{
    compress_row<BF16, SMALL>(blockIdx.x, record_source<BF16>(blockIdx.x, logits, ld, V, seq_off, n_accept), V, inv_T, k, top_p, idx, prob, count, mass, lse, rank_opt);
}

// What the optimistic pass does not serve: rows of up to its sample's length, records it has no rank for.  (3000 fp32 rows of 8000, us: k = 10
// 104.8, k = 4096 159.0 when one kernel held both passes, at 128 registers and some 150 scalar spills; 89.8 and 145.2 so.)
template <bool BF16>
__global__ __launch_bounds__(kT, 4) void compress_careful_kernel(
    const void* __restrict__ logits, int64_t ld, int V, float inv_T, int k, float top_p,
    int32_t* __restrict__ idx, float* __restrict__ prob, int32_t* __restrict__ count,
    float* __restrict__ mass, float* __restrict__ lse,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ n_accept)
{
    compress_row_careful<BF16, false>(blockIdx.x, record_source<BF16>(blockIdx.x, logits, ld, V, seq_off, n_accept), V, inv_T, k, top_p, idx, prob, count, mass, lse);
}

// Both streams of a small round in one launch (the draft rows' compression and the target rows' statistics do
// not depend on each other): workgroups 0..n_draft-1 compress, the others take one target row each.
// (For what round_wide_kernel does not serve: rounds without a table, and rows and records that the optimistic pass does not serve:
// CAREFUL.  With the rows' function of the fast kernels, us of a round without a workspace: 200 drafts and 240 target rows of 151,936, k = 256: fp32 88.9 -> 75.4,
// bf16 64.2 -> 49.9; of 6000, CAREFUL: 32.4 -> 30.4, 30.8 -> 29.1.)
template <bool BF16, bool CAREFUL>
__global__ __launch_bounds__(kT, 4) void round_stream_kernel(
    const void* __restrict__ draft_logits, int64_t ld_d, int n_draft, int V, float inv_T, int k, float top_p,
    int32_t* __restrict__ idx, float* __restrict__ prob, int32_t* __restrict__ count,
    float* __restrict__ mass, float* __restrict__ lse,
    const void* __restrict__ tgt_logits, int64_t ld_t,
    float* __restrict__ tgt_max, float* __restrict__ tgt_sum, float* __restrict__ tgt_lse,
    SegHeader* __restrict__ seg_header, int seg_stride, int rank_opt)
{
    if ((int)blockIdx.x < n_draft) {
        const RowView rv = row_view<BF16>(draft_logits, ld_d, blockIdx.x, V);
        if constexpr (CAREFUL) compress_row_careful<BF16, false>(blockIdx.x, rv, V, inv_T, k, top_p, idx, prob, count, mass, lse);
        else                   compress_row<BF16, false>(blockIdx.x, rv, V, inv_T, k, top_p, idx, prob, count, mass, lse, rank_opt);
    } else if (seg_header) {
        // with the target rows' segment table (the draw then needs no second pass over its row); the row's table is
        // staged in the LDS that a compressing workgroup uses for its candidates
        extern __shared__ __align__(16) unsigned char smem_raw[];
        static_assert(sizeof(CompressShared<kCapBig>) >= kSegStage * sizeof(float2), "the staged table fits the candidate buffer");
        if ((int)blockIdx.x == n_draft && threadIdx.x == 0)
            *seg_header = SegHeader{kSegMagic, kRoundStatsNV<BF16> * kWave, seg_stride, (int32_t)(gridDim.x - n_draft)};
        row_stats_seg_row<BF16, kRoundStatsNV<BF16>, kT, true>((int64_t)blockIdx.x - n_draft, tgt_logits, ld_t, V, inv_T, tgt_max, tgt_sum,
                                                                tgt_lse, reinterpret_cast<float2*>(seg_header + 1), seg_stride,
                                                                reinterpret_cast<float2*>(smem_raw));
    } else {
        row_stats_row<BF16, 2, kT>((int64_t)blockIdx.x - n_draft, tgt_logits, ld_t, V, inv_T, tgt_max, tgt_sum, tgt_lse);
    }
}

// The same with the fast kernels' rows, for rounds of any size whose target rows get a segment table: statistics in the layout
// and in the order of summation of whichever launch the draw expects (stats_threads: stats_shape, round_stats_shape).  `turns` times two drafts
// and a target row, then the drafts that are left, then the target rows that are left.  The compression of a row is bound by the vector ALUs and by its serial phases,
// the statistics by memory: 512 bf16 drafts of 128,256 (k = 1024) and 576 target rows take 55 us here, 36.5 + 31.4 in launches of their
// own; rounds of 40 to 128 sequences, 33,000 to 152,064, k = 64 to 2048, us, two launches / here: bf16 76.5 / 55.2 (40 of 8 drafts), 134.6 /
// 117.7 (64 of 16), 185 / 161 (100 of 14), fp32 107.7 / 82.7, 207.5 / 192.8, 299.5 / 282.7.  (More than 1000 drafts before the first target
// row: up to 3 % slower; four segments in flight per wave of a target row: bf16 2 % faster, fp32 7 % slower.)
template <bool BF16>
__global__ __launch_bounds__(kT, BF16 ? 6 : 4) void round_wide_kernel(
    const void* __restrict__ draft_logits, int64_t ld_d, int n_draft, int V, float inv_T, int k, float top_p,
    int32_t* __restrict__ idx, float* __restrict__ prob, int32_t* __restrict__ count,
    float* __restrict__ mass, float* __restrict__ lse,
    const void* __restrict__ tgt_logits, int64_t ld_t,
    float* __restrict__ tgt_max, float* __restrict__ tgt_sum, float* __restrict__ tgt_lse,
    SegHeader* __restrict__ seg_header, int seg_vecs, int seg_stride, int stats_threads, int rank_opt, int turns)
{
    const int n_target = (int)gridDim.x - n_draft, x = (int)blockIdx.x, turn = x / 3;
    int draft, target;                           // (n_draft or more: none)
    if (turn < turns) {
        draft = x - 3 * turn < 2 ? x - turn : n_draft;
        target = turn;
    } else {                                     // the drafts that are left, then the target rows that are left
        draft = x - turns;
        target = x - n_draft;
    }
    if (__builtin_expect(draft < n_draft, 1)) {   // (the longer code first)
        compress_row<BF16, BF16>(draft, row_view<BF16>(draft_logits, ld_d, draft, V), V, inv_T, k, top_p, idx, prob, count, mass, lse, rank_opt);
    } else {
        extern __shared__ __align__(16) unsigned char smem_raw[];
        if (target == 0 && threadIdx.x == 0) *seg_header = SegHeader{kSegMagic, seg_vecs, seg_stride, n_target};
        float2* const seg = reinterpret_cast<float2*>(seg_header + 1);
        float2* const stage = reinterpret_cast<float2*>(smem_raw);
        static_assert(sizeof(CompressShared<kCapSmall>) >= kSegStage * sizeof(float2), "the staged table fits the candidate buffer");
        constexpr int NV = kRoundStatsNV<BF16>;
        if (stats_threads == kT) row_stats_seg_row<BF16, NV, kT, true>(target, tgt_logits, ld_t, V, inv_T, tgt_max, tgt_sum, tgt_lse, seg, seg_stride, stage);
        else                     row_stats_seg_row<BF16, NV, 2 * kT, true, 2>(target, tgt_logits, ld_t, V, inv_T, tgt_max, tgt_sum, tgt_lse, seg, seg_stride, stage);
    }
}

// The drafter's draw from a record of any length: inverse CDF over the used slots, one wave per row.  (Records beyond kMaxK:
// they do not come from this library's compression.)
__global__ __launch_bounds__(256) void sample_draft_kernel(
    const int32_t* __restrict__ idx, const float* __restrict__ prob, const int32_t* __restrict__ count,
    const float* __restrict__ mass, int k, int n_rows, const float* __restrict__ uniforms,
    int32_t* __restrict__ tok, float* __restrict__ q_scalar)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t row = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (row >= n_rows) return;
    const float* p = prob + row * k;
    int cnt = count[row];
    cnt = cnt < 0 ? 0 : (cnt > k ? k : cnt);
    if (cnt == 0) { if (lane == 0) { tok[row] = -1; if (q_scalar) q_scalar[row] = 0.f; } return; }
    // lane l owns the contiguous slots [l*per, (l+1)*per)
    const int per = (cnt + kWave - 1) / kWave;
    const int s0 = min(cnt, lane * per), s1 = min(cnt, s0 + per);
    double mine = 0.0;
    for (int s = s0; s < s1; ++s) mine += (double)p[s];
    const double incl = wave_scan_incl(mine);
    const double total = __shfl(incl, kWave - 1, kWave);
    const double target = (double)uniforms[row] * total;
    // first lane whose inclusive sum exceeds the target holds the slot
    const unsigned long long ball = __ballot(incl > target);
    int pick = -1;
    if (ball) {
        const int owner = __ffsll((long long)ball) - 1;
        if (lane == owner) {
            double cum = incl - mine;
            for (int s = s0; s < s1; ++s) { cum += (double)p[s]; if (cum > target) { pick = s; break; } }
            if (pick < 0) pick = s1 - 1;
        }
        pick = __shfl(pick, owner, kWave);
    } else {   // rounding: last slot with weight
        if (lane == 0) { pick = cnt - 1; while (pick > 0 && !(p[pick] > 0.f)) --pick; }
        pick = __shfl(pick, 0, kWave);
    }
    if (lane == 0) {
        tok[row] = idx[row * k + pick];
        if (q_scalar) q_scalar[row] = p[pick] / mass[row];
    }
}

// The same draw for records of up to CHUNKS * 256 slots: the wave reads the row in 16-byte pieces, 1 KB per instruction
// (global loads need four-byte alignment only; the last piece of a row whose length is no multiple of four goes slot by
// slot), and keeps it in registers; lane l of piece i owns the four slots 4 * (64 i + l) ..., so a chunk of 256 slots is summed
// by a wave scan and the chunks by a running carry.  What depends on the row alone - count, mass, uniform, probabilities, and
// with IDS the ids - is asked for in one trip to memory; IDS spares the trip for the drawn id, at the price of reading as many
// bytes again: for calls that are bound by their trips.
template <int CHUNKS, bool IDS>
__global__ __launch_bounds__(256) void sample_draft_vec_kernel(
    const int32_t* __restrict__ idx, const float* __restrict__ prob, const int32_t* __restrict__ count,
    const float* __restrict__ mass, int k, int n_rows, const float* __restrict__ uniforms,
    int32_t* __restrict__ tok, float* __restrict__ q_scalar)
{
    struct __attribute__((packed, aligned(4))) Four { uint32_t w[4]; };
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t row = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (row >= n_rows) return;
    const float* p = prob + row * k;
    const int32_t* ids = idx + row * k;
    int cnt = count[row];
    const float mass_row = mass[row], u = uniforms[row];
    Four v[CHUNKS], t[IDS ? CHUNKS : 1] = {};
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
        const int s0 = 4 * (i * kWave + lane);
        v[i] = Four{{0u, 0u, 0u, 0u}};
        if constexpr (IDS) t[i] = v[i];
        if (s0 + 4 <= k) {
            v[i] = *reinterpret_cast<const Four*>(p + s0);
            if constexpr (IDS) t[i] = *reinterpret_cast<const Four*>(ids + s0);
        } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (s0 + e < k) {
                    v[i].w[e] = __float_as_uint(p[s0 + e]);
                    if constexpr (IDS) t[i].w[e] = (uint32_t)ids[s0 + e];
                }
        }
    }
    cnt = cnt < 0 ? 0 : (cnt > k ? k : cnt);
    if (cnt == 0) { if (lane == 0) { tok[row] = -1; if (q_scalar) q_scalar[row] = 0.f; } return; }
    double incl[CHUNKS];                      // inclusive sum over the chunk up to and including this lane's four
    double carry[CHUNKS + 1];                 // sum of the chunks in front
    carry[0] = 0.0;
    auto weight = [&](int i, int e) { return (double)__uint_as_float(v[i].w[e]); };
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[i].w[e] = 4 * (i * kWave + lane) + e < cnt ? v[i].w[e] : 0u;   // slots behind the count carry no weight
        const double mine = ((weight(i, 0) + weight(i, 1)) + weight(i, 2)) + weight(i, 3);
        incl[i] = wave_scan_incl(mine);
        carry[i + 1] = carry[i] + read_lane(incl[i], kWave - 1);
    }
    const double target = (double)u * carry[CHUNKS];
    // the chunk and the lane in which the cumulative weight crosses the target (uniform across the wave), then the lane's slot
    int chunk = -1, owner = 0;
    Four w = v[0], id = t[0];
    double upto = 0.0;
#pragma unroll
    for (int i = 0; i < CHUNKS; ++i) {
        const unsigned long long ball = chunk < 0 ? __ballot(carry[i] + incl[i] > target) : 0ull;
        if (ball) {
            chunk = i;
            owner = __ffsll((long long)ball) - 1;
            w = v[i];
            if constexpr (IDS) id = t[i];
            upto = carry[i] + incl[i] - (((weight(i, 0) + weight(i, 1)) + weight(i, 2)) + weight(i, 3));
        }
    }
    int pick = -1;
    uint32_t pick_w = 0u, pick_id = 0u;
    if (chunk >= 0) {
        int at = 3;                           // first slot of the lane's four whose cumulative weight exceeds the target
        bool found = false;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            upto += (double)__uint_as_float(w.w[e]);
            if (!found && upto > target) { at = e; found = true; }
        }
        uint32_t x = w.w[0], y = id.w[0];
#pragma unroll
        for (int e = 1; e < 4; ++e) { x = at == e ? w.w[e] : x; y = at == e ? id.w[e] : y; }
        pick = 4 * (chunk * kWave + owner) + __builtin_amdgcn_readlane(at, owner);
        pick_w = (uint32_t)__builtin_amdgcn_readlane((int)x, owner);
        pick_id = (uint32_t)__builtin_amdgcn_readlane((int)y, owner);
    }
    if (lane == 0) {
        bool known = true;
        if (pick < 0 || pick >= cnt) {        // rounding: the last slot with weight
            pick = cnt - 1;
            while (pick > 0 && !(p[pick] > 0.f)) --pick;
            pick_w = __float_as_uint(p[pick]);
            known = false;
        }
        tok[row] = IDS && known ? (int32_t)pick_id : ids[pick];
        if (q_scalar) q_scalar[row] = __uint_as_float(pick_w) / mass_row;
    }
}

}  // namespace

// The small variant (three workgroups per CU) serves records of up to kMaxK / 2 entries on rows long enough that the
// optimistic pass applies and its expected candidates fit the smaller buffer with room to spare (the kernel evaluates
// the same function with a slightly smaller allowance, so it agrees).
static bool small_variant_serves(int k, int V)
{
    return k <= CompressShared<kCapSmall>::kRecMax && V >= 4 * kCompressSample &&
           optimistic_rank(k, V, kCompressSample, kCapSmall, 4.5f) > 0;
}

// CUs of device `dev` (-1: not known)
static int cus_of(int dev)
{
    static std::atomic<int> count[kMaxDevices] = {};
    int cus = count[dev].load(std::memory_order_relaxed);
    if (cus == 0) {                              // (first use on this device; a second thread here computes the same value)
        cus = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0 ? cus : -1;
        count[dev].store(cus, std::memory_order_relaxed);
    }
    return cus;
}

// bf16: statistics of 2048 rows and more run in workgroups of 256 threads, which the launch for both streams has no form of.  fp32: the more of the time
// both streams are bound by memory, the less one hides in the other, and each then has its better launch shape alone.  us, a round in three
// launches / two, drafts of 151,936: 1000 257 / 252, 1400 348 / 338, 1600 385 / 382 and 376 / 377, 1760 (k = 4096) 405 / 413, (k = 64) 360 / 349, 2048 462 / 474,
// 4096 876 / 940; of 100,000: 1900 296 / 289, 2048 298 / 296; of 64,000: 2048 258 / 245; of 33,000: 1350 111 / 104, 4000 245 / 246.
constexpr int64_t kWideRowsF32 = 4608, kWideBytesF32 = 1800000000;
bool round_wide_serves(int dtype, int64_t n_draft, int64_t n_target, int V, int k)
{
    if (n_draft < 1 || n_draft + n_target > INT32_MAX) return false;
    if (dtype == 1) return n_target < 2048 && small_variant_serves(k, V);
    const int64_t rows = n_draft + n_target;
    return rows <= kWideRowsF32 && rows * V * 4 <= kWideBytesF32 && compress_rank(k, V, false) > 0;
}

hipError_t launch_compress(const void* logits, int dtype, int64_t ld, int n_rows, int V, float temperature,
                           int k, float top_p, int32_t* idx, float* prob, int32_t* count, float* mass,
                           float* lse, const int32_t* seq_off, const int32_t* n_accept, hipStream_t stream)
{
    static DeviceFlags limit_raised[6] = {};
    const int bf = dtype == 1 ? 1 : 0;
    // the optimistic pass with the large or the small candidate buffer, and the careful pass
    const void* const kernels[6] = {(const void*)compress_kernel<false, false>, (const void*)compress_kernel<true, false>,
                                    nullptr /* (the small buffer serves bf16 rows only) */, (const void*)compress_kernel<true, true>,
                                    (const void*)compress_careful_kernel<false>, (const void*)compress_careful_kernel<true>};
    const size_t smem_big = sizeof(CompressShared<kCapBig>), smem_small = sizeof(CompressShared<kCapSmall>);
    {   // (every variant of the dtype: which of them a call takes depends on its sizes)
        hipError_t e = hipSuccess;
        int dev = 0;
        for (int v = 0; v < 3 && e == hipSuccess; ++v)
            if (kernels[2 * v + bf]) e = raise_lds_limit_once(kernels[2 * v + bf], v == 1 ? smem_small : smem_big, limit_raised[2 * v + bf], dev);
        if (e != hipSuccess) return e;
    }
    if (n_rows == 0) return hipSuccess;
    // (fp32 rows stream faster from two workgroups per CU with the large buffer than from three with the small one,
    //  measured at every record length; bf16 rows, which cost twice the arithmetic per byte, gain from the third)
    const bool small = bf && small_variant_serves(k, V);
    const int rank_opt = compress_rank(k, V, small);
    const float inv_T = 1.0f / temperature;
#define PICOSPEC_COMPRESS(KERNEL, SMEM, ...) \
    hipLaunchKernelGGL(KERNEL, dim3(n_rows), dim3(kT), SMEM, stream, logits, ld, V, inv_T, k, top_p, idx, prob, count, mass, lse, seq_off, n_accept, ##__VA_ARGS__)
    if (small) PICOSPEC_COMPRESS((compress_kernel<true, true>), smem_small, rank_opt);
    else if (rank_opt > 0) { if (bf) PICOSPEC_COMPRESS((compress_kernel<true, false>), smem_big, rank_opt); else PICOSPEC_COMPRESS((compress_kernel<false, false>), smem_big, rank_opt); }
    else                   { if (bf) PICOSPEC_COMPRESS((compress_careful_kernel<true>), smem_big); else PICOSPEC_COMPRESS((compress_careful_kernel<false>), smem_big); }
#undef PICOSPEC_COMPRESS
    return hipGetLastError();
}

hipError_t launch_round_wide(const void* draft_logits, int dtype, int64_t ld_d, int n_draft, int V, float temperature,
                             int k, float top_p, int32_t* idx, float* prob, int32_t* count, float* mass, float* lse,
                             const void* tgt_logits, int64_t ld_t, int n_target,
                             float* tgt_max, float* tgt_sum, float* tgt_lse, void* seg_table, const StatsShape& sh, hipStream_t stream)
{
    static DeviceFlags limit_raised[2] = {};
    const int bf = dtype == 1;
    const size_t smem = bf ? sizeof(CompressShared<kCapSmall>) : sizeof(CompressShared<kCapBig>);
    const void* const kernel = bf ? (const void*)round_wide_kernel<true> : (const void*)round_wide_kernel<false>;
    int dev = 0;
    if (hipError_t e = raise_lds_limit_once(kernel, smem, limit_raised[bf], dev)) return e;
    const float inv_T = 1.0f / temperature;
    const int rank_opt = compress_rank(k, V, bf);
    const int cus = cus_of(dev);
    // (a draft's row is the longer job: up to one per CU start at once, each on a CU of its own - 182 fp32 drafts of 33,000, k = 2048, with 196
    //  target rows: 42.4 us in turns, 36.5 drafts first; 200 bf16 of 100,000: 38.1 / 32.8; 288 of 152,064 64.0 / 64.6, 512 of 128,256 69.7 / 73.7)
    const int turns = n_draft > cus ? min(n_draft / 2, n_target) : 0;
#define PICOSPEC_WIDE(BF) \
    hipLaunchKernelGGL(round_wide_kernel<BF>, dim3(n_draft + n_target), dim3(kT), smem, stream, draft_logits, ld_d, n_draft, V, inv_T, k, top_p, idx, prob, count, mass, lse, tgt_logits, ld_t, tgt_max, tgt_sum, tgt_lse, (SegHeader*)seg_table, sh.seg_vecs, sh.stride, sh.threads, rank_opt, turns)
    if (bf) PICOSPEC_WIDE(true); else PICOSPEC_WIDE(false);
#undef PICOSPEC_WIDE
    return hipGetLastError();
}

hipError_t launch_round_stream(const void* draft_logits, int dtype, int64_t ld_d, int n_draft, int V, float temperature,
                               int k, float top_p, int32_t* idx, float* prob, int32_t* count, float* mass, float* lse,
                               const void* tgt_logits, int64_t ld_t, int n_target,
                               float* tgt_max, float* tgt_sum, float* tgt_lse, void* seg_table, hipStream_t stream)
{
    static DeviceFlags limit_raised[4] = {};
    const size_t smem = sizeof(CompressShared<kCapBig>);
    const void* const kernels[4] = {(const void*)round_stream_kernel<false, false>, (const void*)round_stream_kernel<true, false>,
                                    (const void*)round_stream_kernel<false, true>, (const void*)round_stream_kernel<true, true>};
    const int bf = dtype == 1, rank_opt = compress_rank(k, V, false);
    for (int v = 0; v < 2; ++v) {                // (both variants of the dtype: which of them a call takes depends on its sizes)
        int dev = 0;
        if (hipError_t e = raise_lds_limit_once(kernels[2 * v + bf], smem, limit_raised[2 * v + bf], dev)) return e;
    }
    if (n_draft + n_target == 0) return hipSuccess;
    const float inv_T = 1.0f / temperature;
    if (n_target == 0) seg_table = nullptr;
    SegHeader* const header = (SegHeader*)seg_table;
    const int stride = round_stats_shape(dtype, V).stride;
#define PICOSPEC_STREAM(BF, CA) \
    hipLaunchKernelGGL((round_stream_kernel<BF, CA>), dim3(n_draft + n_target), dim3(kT), smem, stream, draft_logits, ld_d, n_draft, V, inv_T, k, top_p, idx, prob, count, mass, lse, tgt_logits, ld_t, tgt_max, tgt_sum, tgt_lse, header, stride, rank_opt)
    if (rank_opt > 0) { if (bf) PICOSPEC_STREAM(true, false); else PICOSPEC_STREAM(false, false); }
    else              { if (bf) PICOSPEC_STREAM(true, true); else PICOSPEC_STREAM(false, true); }
#undef PICOSPEC_STREAM
    return hipGetLastError();
}

hipError_t launch_sample_draft(const int32_t* idx, const float* prob, const int32_t* count, const float* mass,
                               int k, int n_rows, const float* uniforms, int32_t* tok, float* q_scalar,
                               hipStream_t stream)
{
    if (n_rows == 0) return hipSuccess;
    const int rows_per_block = 256 / kWave;
    const dim3 grid((n_rows + rows_per_block - 1) / rows_per_block);
    if (k <= kMaxK) {
        // the row in registers, as many 256-slot chunks as k needs; up to 512 rows (two waves per CU) the ids as well: such calls
        // wait for their trips to memory (64 rows of 1024: 5.2 us with a trip of its own for the drawn id)
        const bool few = n_rows <= 512;
#define PICOSPEC_SAMPLE_DRAFT(C, I) \
        hipLaunchKernelGGL((sample_draft_vec_kernel<C, I>), grid, dim3(256), 0, stream, idx, prob, count, mass, k, n_rows, uniforms, tok, q_scalar)
        if (k <= 256)       { if (few) PICOSPEC_SAMPLE_DRAFT(1, true); else PICOSPEC_SAMPLE_DRAFT(1, false); }
        else if (k <= 1024) { if (few) PICOSPEC_SAMPLE_DRAFT(4, true); else PICOSPEC_SAMPLE_DRAFT(4, false); }
        else if (k <= 2048) PICOSPEC_SAMPLE_DRAFT(8, false);
        else                PICOSPEC_SAMPLE_DRAFT(16, false);
#undef PICOSPEC_SAMPLE_DRAFT
        static_assert(kMaxK <= 16 * 256, "sixteen chunks hold the longest record");
        return hipGetLastError();
    }
    hipLaunchKernelGGL(sample_draft_kernel, grid, dim3(256), 0, stream,
                       idx, prob, count, mass, k, n_rows, uniforms, tok, q_scalar);
    return hipGetLastError();
}

}  // namespace picospec
