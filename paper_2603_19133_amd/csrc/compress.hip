// The kernels of the sparse Top-K compression (compress_row.hpp holds what a workgroup does with a row): the general
// and the fast variants, the retry launch behind the fast ones, the small rounds' streaming kernel, and the drafter's
// draw from a record.
#include "compress_row.hpp"

namespace picospec {

namespace {

template <bool BF16, bool SMALL, bool FAST>
__global__ __launch_bounds__(kT, SMALL ? 6 : 4) void compress_kernel(
    const void* __restrict__ logits, int64_t ld, int V, float inv_T, int k, float top_p,
    int32_t* __restrict__ idx, float* __restrict__ prob, int32_t* __restrict__ count,
    float* __restrict__ mass, float* __restrict__ lse,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ n_accept, int ahead, int rank_opt)
{
    compress_row<BF16, SMALL, FAST>(blockIdx.x, (int)gridDim.x, logits, ld, V, inv_T, k, top_p, idx, prob, count, mass, lse,
                                    seq_off, n_accept, ahead, rank_opt);
}

// The rows that the fast kernel with the large buffer marked with count = kRetryRow, through the general code: a few workgroups, each
// looking through its share of the counts (one row per thread and step) and compressing the rows it finds marked.
// (Launching one general workgroup per row just to look would cost tens of microseconds: its LDS makes the launch slow.)
template <bool BF16>
__global__ __launch_bounds__(kT, 4) void compress_retry_kernel(
    const void* __restrict__ logits, int64_t ld, int n_rows, int V, float inv_T, int k, float top_p,
    int32_t* __restrict__ idx, float* __restrict__ prob, int32_t* __restrict__ count,
    float* __restrict__ mass, float* __restrict__ lse,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ n_accept, int rank_opt)
{
    __shared__ int marked[kT];
    __shared__ int n_marked;
    const int per = (n_rows + (int)gridDim.x - 1) / (int)gridDim.x;
    const int first = (int)blockIdx.x * per, last = min(first + per, n_rows);
    for (int r0 = first; r0 < last; r0 += kT) {
        if (threadIdx.x == 0) n_marked = 0;
        __syncthreads();
        const int r = r0 + (int)threadIdx.x;
        if (r < last && count[r] == kRetryRow) marked[atomicAdd(&n_marked, 1)] = r;
        __syncthreads();
        const int n = n_marked;
        for (int i = 0; i < n; ++i) {
            const int row = marked[i];
            compress_row<BF16, false, false>(row, n_rows, logits, ld, V, inv_T, k, top_p, idx, prob, count, mass, lse,
                                      seq_off, n_accept, 0, rank_opt);
            __syncthreads();                     // (the row's last reads of LDS are done before the next one resets it)
        }
        __syncthreads();
    }
}

// Both streams of a small round in one launch (the draft rows' compression and the target rows' statistics do
// not depend on each other): workgroups 0..n_draft-1 compress, the others take one target row each.
// (For rounds of a few rows: registers are not held down to four waves per SIMD here.)
template <bool BF16>
__global__ __launch_bounds__(kT, 2) void round_stream_kernel(
    const void* __restrict__ draft_logits, int64_t ld_d, int n_draft, int V, float inv_T, int k, float top_p,
    int32_t* __restrict__ idx, float* __restrict__ prob, int32_t* __restrict__ count,
    float* __restrict__ mass, float* __restrict__ lse,
    const void* __restrict__ tgt_logits, int64_t ld_t,
    float* __restrict__ tgt_max, float* __restrict__ tgt_sum, float* __restrict__ tgt_lse,
    SegHeader* __restrict__ seg_header, int seg_stride, int rank_opt)
{
    if ((int)blockIdx.x < n_draft) {
        compress_row<BF16, false, false>(blockIdx.x, n_draft, draft_logits, ld_d, V, inv_T, k, top_p, idx, prob, count, mass, lse,
                                  nullptr, nullptr, 0, rank_opt);
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

hipError_t launch_compress(const void* logits, int dtype, int64_t ld, int n_rows, int V, float temperature,
                           int k, float top_p, int32_t* idx, float* prob, int32_t* count, float* mass,
                           float* lse, const int32_t* seq_off, const int32_t* n_accept, hipStream_t stream)
{
    static DeviceFlags limit_raised[8] = {};
    static std::atomic<int> cu_count[kMaxDevices] = {};
    const int bf = dtype == 1 ? 1 : 0;
    // general (both passes in one kernel) / fast (optimistic pass only, rows it gives up marked for the retry kernel),
    // the latter with the large or the small candidate buffer
    const void* const kernels[8] = {(const void*)compress_kernel<false, false, false>, (const void*)compress_kernel<true, false, false>,
                                    (const void*)compress_kernel<false, false, true>, (const void*)compress_kernel<true, false, true>,
                                    nullptr /* (the small buffer serves bf16 rows only) */, (const void*)compress_kernel<true, true, true>,
                                    (const void*)compress_retry_kernel<false>, (const void*)compress_retry_kernel<true>};
    const size_t smem_big = sizeof(CompressShared<kCapBig>), smem_small = sizeof(CompressShared<kCapSmall>);
    int dev = 0;
    {   // (every variant of the dtype: which of them a call takes depends on its sizes)
        hipError_t e = hipSuccess;
        for (int v = 0; v < 4 && e == hipSuccess; ++v)
            if (kernels[2 * v + bf]) e = raise_lds_limit_once(kernels[2 * v + bf], v == 2 ? smem_small : smem_big, limit_raised[2 * v + bf], dev);
        if (e != hipSuccess) return e;
    }
    if (n_rows == 0) return hipSuccess;
    int cus = cu_count[dev].load(std::memory_order_relaxed);
    if (cus == 0) {                              // (first use on this device; a second thread here computes the same value)
        cus = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0 ? cus : -1;
        cu_count[dev].store(cus, std::memory_order_relaxed);
    }
    // (fp32 rows stream faster from two workgroups per CU with the large buffer than from three with the small one,
    //  measured at every record length; bf16 rows, which cost twice the arithmetic per byte, gain from the third, and calls
    //  of any number of rows from the kernel without the careful pass: 1 to 512 rows of 33,000, 64,000 and 152,064, k = 10 to
    //  2048, are 15 to 22, 11 to 14 and 7 to 10 % faster than from the general kernel)
    const bool small = bf && small_variant_serves(k, V);
    // With the large buffer, calls of more rows than the chip holds at a time take the fast kernel (fewer registers: the careful
    // pass is not in it) and pay one small launch more; smaller calls are bound by that launch and take the general kernel.
    const bool fast = small || (cus > 0 && n_rows > 2 * cus && V > kCompressSample);
    // rows resident at a time (2 workgroups per CU, 3 of the small variant): the distance of the look-ahead loads
    // (no look-ahead with a row map: the next row is not known from the row number)
    const int ahead = (!seq_off && cus > 0) ? (small ? 3 : 2) * cus : 0;
    const float inv_T = 1.0f / temperature;
    const int rank_opt = compress_rank(k, V, small);
#define PICOSPEC_COMPRESS(BF, SM, FA, SMEM) \
    hipLaunchKernelGGL((compress_kernel<BF, SM, FA>), dim3(n_rows), dim3(kT), SMEM, stream, logits, ld, V, inv_T, k, top_p, idx, prob, count, mass, lse, seq_off, n_accept, ahead, rank_opt)
#define PICOSPEC_RETRY(BF) \
    hipLaunchKernelGGL((compress_retry_kernel<BF>), dim3(min(64, (n_rows + kT - 1) / kT)), dim3(kT), smem_big, stream, logits, ld, n_rows, V, inv_T, k, top_p, idx, prob, count, mass, lse, seq_off, n_accept, compress_rank(k, V, false))
    if (small) {
        PICOSPEC_COMPRESS(true, true, true, smem_small);
    } else if (fast) {
        if (bf) PICOSPEC_COMPRESS(true, false, true, smem_big); else PICOSPEC_COMPRESS(false, false, true, smem_big);
    } else {
        if (bf) PICOSPEC_COMPRESS(true, false, false, smem_big); else PICOSPEC_COMPRESS(false, false, false, smem_big);
    }
    if (fast && !small) {
        if (hipError_t e = hipGetLastError()) return e;
        if (bf) PICOSPEC_RETRY(true); else PICOSPEC_RETRY(false);
    }
#undef PICOSPEC_RETRY
#undef PICOSPEC_COMPRESS
    return hipGetLastError();
}

hipError_t launch_round_stream(const void* draft_logits, int dtype, int64_t ld_d, int n_draft, int V, float temperature,
                               int k, float top_p, int32_t* idx, float* prob, int32_t* count, float* mass, float* lse,
                               const void* tgt_logits, int64_t ld_t, int n_target,
                               float* tgt_max, float* tgt_sum, float* tgt_lse, void* seg_table, hipStream_t stream)
{
    static DeviceFlags limit_raised[2] = {};
    const size_t smem = sizeof(CompressShared<kCapBig>);
    auto f32 = round_stream_kernel<false>;
    auto b16 = round_stream_kernel<true>;
    const int which = dtype == 1;
    {
        int dev = 0;
        hipError_t e = raise_lds_limit_once(which ? (const void*)b16 : (const void*)f32, smem, limit_raised[which], dev);
        if (e != hipSuccess) return e;
    }
    if (n_draft + n_target == 0) return hipSuccess;
    const float inv_T = 1.0f / temperature;
    if (n_target == 0) seg_table = nullptr;
    SegHeader* const header = (SegHeader*)seg_table;
    const int stride = round_stats_shape(dtype, V).stride;
    if (which) hipLaunchKernelGGL(b16, dim3(n_draft + n_target), dim3(kT), smem, stream, draft_logits, ld_d, n_draft, V, inv_T, k, top_p, idx, prob, count, mass, lse, tgt_logits, ld_t, tgt_max, tgt_sum, tgt_lse, header, stride, compress_rank(k, V, false));
    else       hipLaunchKernelGGL(f32, dim3(n_draft + n_target), dim3(kT), smem, stream, draft_logits, ld_d, n_draft, V, inv_T, k, top_p, idx, prob, count, mass, lse, tgt_logits, ld_t, tgt_max, tgt_sum, tgt_lse, header, stride, compress_rank(k, V, false));
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
