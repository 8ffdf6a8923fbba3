// Sparse Top-K compression of few rows (paper Section 3.3, Eq. 4): a call that leaves most of the chip idle spreads every
// row over many small workgroups and finishes it in a second launch, or in the same one by the last of the row's workgroups.
//
// One workgroup per row (compress_row.hpp) is a chain of phases on one CU: 25 us for a bf16 row of 128,256 whatever k is, of
// which 13 us are the streaming of the row by eight waves and the rest serial phases that issue one instruction per wave
// every eight to ten cycles with two waves on a SIMD.  Here
//   * split_select_kernel: P = V / 8192 workgroups of four waves per row.  A workgroup takes every P-th block of 1 KB of the
//     row (so that each sees the whole row evenly: logits trend with the vocabulary id) and holds its 8192 elements in
//     registers: one trip to memory, nothing read twice, no sample.  A histogram over the upper part of its values finds a
//     threshold with at least `rank` of its elements above it; rank is optimistic_rank's bound for a share of 1 / P of the
//     row's k largest, so the elements above it hold the row's top k but for a chance of some 1e-6.  The workgroup writes
//     them to a list of its own in the scratch, and its share of the statistics in front of it.
//   * split_finish_kernel: one workgroup per row gathers the lists (about k plus the ranks' margins), orders them and writes
//     the record: from registers (finish_few), or with the code of the unsplit kernels.  The answer is exact iff the k-th value lies above every workgroup's
//     threshold, which is tested; a row that fails it (or whose lists overflow) is compressed from the start by the
//     unsplit kernels' code in the same workgroup.
//   * split_compress_kernel: both, for calls of up to 128 workgroups whose scratch has room for the rows' words (split_one_launch).
// Device time of a call, one workgroup per row -> split: one bf16 row of 128,256, k = 10: 25.5 -> 4.8 + 4.3 us; 64 fp32 rows of
// 151,936, k = 1024: 31.0 -> 10.5 + 6.6 us, of which the first launch reads 39 MB (5.8 us at 6.8 TB/s).  The line between the two
// is split_plan's.
#include "compress_row.hpp"

namespace picospec {

namespace {

constexpr int kSplitThreads = 256;
constexpr int kSplitBins = 512;                // histogram of a workgroup's values: eight bins per lane in the pivot scan
constexpr int kImageVecs = 4;                  // vectors per lane that pass through LDS at a time
// THREADS: 256, or 512 of which wave w + 4 holds the second half of what wave w holds otherwise.
template <bool BF16, int THREADS> struct SplitGeom {
    using elem_t = typename std::conditional<BF16, uint16_t, uint32_t>::type;
    static constexpr int N = Vec<BF16>::N;
    static constexpr int NV = kSplitElems / (THREADS * N);                 // vectors per lane
    static constexpr int E = NV * N;                                  // elements per lane
    static constexpr int IV = NV < kImageVecs ? NV : kImageVecs;
    static constexpr int WAVES = THREADS / kWave;
    static constexpr int HIST = kSplitBins + kWave, IMAGE = 4 * IV * THREADS;      // words of LDS; behind the bins: a slot per lane for what lies below them
    static_assert(NV % IV == 0 && E <= 32 && THREADS % 256 == 0 && kSplitBins % THREADS == 0, "one bit of a word per element");
    __device__ static __forceinline__ int nth(int j, int wave) { return (wave >> 2) * NV + j; }       // a wave's block j: split_block(nth(j, wave), wave & 3, ..)
};

// What a workgroup leaves of its share of the row; its list of (value, id) pairs stands in an array of its own.
struct __align__(16) SplitHead {
    float mx, tau, r;                          // largest value; threshold (every element above it is in the list); reference exponent
    int count;                                 // entries of the list (more than the list holds: the row is given up)
    double s;                                  // sum of 2^(z c - r) over the share
};
static_assert(sizeof(SplitHead) == 32, "a 16-byte load and one of eight");

// Workgroup `part` of the P workgroups of row `row` of the call.  hist, image: LDS on 16-byte boundaries.  SHARED: for another workgroup of this
// launch to read.  `meanwhile` is run behind the loads.  The share's sum is formed in the same order by workgroups of either size.
template <bool BF16, int THREADS, bool SHARED, class F>
__device__ __forceinline__ void split_select(
    unsigned* const hist, unsigned* const image,
    const int64_t row, const int part, const int P,
    const void* __restrict__ logits, int64_t ld, int V, float inv_T, int rank, int cap, int narrow, int lanes,
    SplitHead* __restrict__ heads, uint2* __restrict__ lists,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ n_accept, const F& meanwhile)
{
    using G = SplitGeom<BF16, THREADS>;
    constexpr int N = G::N, NV = G::NV, E = G::E, kSplitWaves = G::WAVES;
    __shared__ float red[2 * kSplitWaves];
    __shared__ float lane_s[THREADS > 256 ? THREADS : 1];
    __shared__ double wave_s[kSplitWaves];
    __shared__ int wave_held[kSplitWaves];
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const RowView rv = record_source<BF16>(row, logits, ld, V, seq_off, n_accept);
    const int nq = (rv.L + N - 1) / N;
    const int n_blocks = (nq + kWave - 1) / kWave;
    const float c = 1.4426950408889634f * inv_T;
    // (the same range rule as the other row kernels, rowspan.hpp: vectors behind the row read as zero and touch no memory)
    const __amdgpu_buffer_rsrc_t row_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)rv.base, 0, nq * 16, 0x00020000);
    uint4 raw[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const u32x4_t t = __builtin_amdgcn_raw_buffer_load_b128(row_rsrc, lane * 16, split_block(G::nth(j, wave), wave & 3, part, P) * (kWave * 16), 2 /* non-temporal */);
        raw[j] = make_uint4(t.x, t.y, t.z, t.w);
    }
    auto clear = [&] {
#pragma unroll
        for (int i = 0; i < kSplitBins / THREADS; ++i) hist[i * THREADS + tid] = 0u;
    };
    clear();
    meanwhile();
    float v[E];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        float t[N];
        unpack<BF16>(raw[j], t);
#pragma unroll
        for (int e = 0; e < N; ++e) v[j * N + e] = t[e];
    }
    // elements outside the row (in front of its first, behind its last) count as masked ones: -inf.  Only the row's first and
    // last blocks hold any.
    if ((part == 0 && wave == 0) || split_block(G::nth(NV - 1, wave), wave & 3, part, P) >= n_blocks - 1) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const unsigned vm = vec_valid_mask<BF16>(rv, split_block(G::nth(j, wave), wave & 3, part, P) * kWave + lane);
#pragma unroll
            for (int e = 0; e < N; ++e) v[j * N + e] = (vm >> e) & 1u ? v[j * N + e] : kNegInf;
        }
    }
    float bm = kNegInf;
#pragma unroll
    for (int e = 0; e < E; ++e) bm = fmaxf(bm, v[e]);
    // Lower end of the histogram: at least `rank` elements must lie at or above it.  narrow: the smallest of the lanes' largest
    // values will do (256 elements at or above it); else the smallest value above -inf.
    float bl = bm;
    if (!narrow) {
        bl = __builtin_huge_valf();
#pragma unroll
        for (int e = 0; e < E; ++e) bl = fminf(bl, v[e] > kNegInf ? v[e] : __builtin_huge_valf());
    }
    if (!(bl > kNegInf)) bl = __builtin_huge_valf();
    const float wm = wave_max(bm), wl = -wave_max(-bl);
    if (lane == 0) { red[wave] = wm; red[kSplitWaves + wave] = wl; }
    __syncthreads();
    float hi = red[0], lo = red[kSplitWaves];
#pragma unroll
    for (int w = 1; w < kSplitWaves; ++w) { hi = fmaxf(hi, red[w]); lo = fminf(lo, red[kSplitWaves + w]); }
    const float mx = hi;
    // the share's softmax sum, against an integer reference exponent
    const float ref = hi > kNegInf ? ceilf(hi * c) : 0.f;
    const float acc = tree_sum<0, E>([&](int e) { return __builtin_amdgcn_exp2f(fmaf(v[e], c, -ref)); });   // (masked: 2^-inf = 0)

    // ---- threshold: a linear histogram of [lo, hi]; a pivot bin that is crowded is refined over the keys (the order-preserving
    //      integers) of its values.  A linear scale that outliers or masked entries of a finite value stretch (the type's
    //      lowest, -1e9) holds all that matters in one bin however often it is cut; the keys of two values of one binade lie
    //      2^23 apart at most, so three passes of nine bits resolve any bin.
    float tau = kNegInf;
    const bool finite = hi > kNegInf && hi < __builtin_huge_valf();
    int bin, before, cnt;                        // the pivot bin of a pass, elements in the bins in front of it and in it
    const int crowd = max(16, rank >> 3);
    // every wave scans the bins for itself, eight consecutive ones per lane; false: fewer than `need` elements in all of them
    auto find_pivot = [&](int need) {
        const uint4 h0 = *reinterpret_cast<const uint4*>(&hist[8 * lane]), h1 = *reinterpret_cast<const uint4*>(&hist[8 * lane + 4]);
        const int h[8] = {(int)h0.x, (int)h0.y, (int)h0.z, (int)h0.w, (int)h1.x, (int)h1.y, (int)h1.z, (int)h1.w};
        const int loc = ((h[0] + h[1]) + (h[2] + h[3])) + ((h[4] + h[5]) + (h[6] + h[7]));
        const int incl = wave_scan_incl(loc);
        const unsigned long long reach = __ballot(incl >= need);
        if (!reach) return false;
        const int owner = __ffsll((long long)reach) - 1;
        // (the walk through the owner's eight bins in scalar registers)
        before = read_lane(incl - loc, owner); bin = 8 * owner; cnt = read_lane(h[0], owner);
#pragma unroll
        for (int u = 1; u < 8; ++u) {
            const int next = read_lane(h[u], owner);
            if (before + cnt < need && bin == 8 * owner + u - 1) { before += cnt; ++bin; cnt = next; }
        }
        return true;
    };
    const double ws = THREADS > 256 ? 0.0 : wave_sum((double)acc);
    unsigned marks = 0;
    int at = 0, held = 0;
    // First (lanes > 0) by the lanes' largest values alone, one bin and atomic per lane instead of 32: with n of 256 lanes at or above it, a
    // threshold has some -256 ln(1 - n / 256) elements above it, as the host chose n (split_plan); a list that comes out too long for
    // its slots or too few lanes with a value (masks, values that trend within a lane) fall to the elements.  (A crowded pivot bin alone does not: where
    // values tie its elements are one value, which no finer bins divide.  24 fp32 rows of 33,001 on quarters, k = 70, 11.0 -> 9.9 us in two
    // launches, in one, whose 512 lanes meet more ties, 14.4 -> 9.9; 8 bf16 of 128,256, k = 256: 16.2 -> 10.3.)
    // 64 fp32 rows of 151,936, k = 1024: 12.2 -> 10.5 us, 32 bf16 of 128,256, k = 256: 7.5 -> 6.7, one, k = 10: 5.1 -> 4.8.
    // A share with no two values to tell apart (narrow: whose lanes have none) lists everything above -inf, as a share with fewer entries
    // than the rank does: a vocabulary mask may leave it one.  If that is too much, what lies below the one value goes.  (40 rows of 128,256
    // with 13 entries above -inf, k = 512, us: cut at their one value, which sends the row to split_row_again, fp32 39.6, bf16 34.2; so 15.3 and 14.8.)
    const bool one = finite && !(hi > lo);
    bool whole = one;
    for (int by_lanes = lanes;; by_lanes = 0, whole = false) {
    bool again = false;
    if (one) {
        if (!whole && hi == lo) tau = float_below(lo);
    } else if (finite) {
        int need = by_lanes ? by_lanes : rank;
        bool open = true;                        // the threshold is not fine enough yet
        bool counted = false;                    // the histogram holds a pass
        uint32_t top = key_of_bits(__float_as_uint(hi)), bottom = key_of_bits(__float_as_uint(lo));
        const float width = (hi - lo) * (1.0f / (float)kSplitBins);
        float scale = __builtin_amdgcn_rcpf(width);
        asm volatile("" : "+v"(scale));          // (the elements' bins are formed in each round, not held from in front of it)
        if (scale < __builtin_huge_valf() && width < __builtin_huge_valf()) {
            const float at0 = hi * scale;
            // bin 0 holds the largest values; what lies below lo goes to the lane's own slot behind the bins
            auto bin_of = [&](float x) {
                unsigned b;
                asm("v_cvt_u32_f32 %0, %1" : "=v"(b) : "v"(fmaf(x, -scale, at0)));     // (saturates: below 0 and NaN 0, large 2^32 - 1)
                return b;
            };
            if (by_lanes) {
                atomicAdd(&hist[min(bin_of(bm), (unsigned)(kSplitBins + lane))], 1u);
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) atomicAdd(&hist[min(bin_of(v[e]), (unsigned)(kSplitBins + lane))], 1u);
            }
            __syncthreads();
            counted = true;
            if (!find_pivot(need)) {
                if (by_lanes) again = true;      // (too few lanes with an element above -inf)
                open = false;                    // fewer than `need` elements above -inf (a masked row): tau stays -inf, all of them are listed
            } else if (by_lanes) {
                tau = float_below(hi - ((float)(bin + 1) + 0.02f) * width);
                open = false;
                again = before + cnt > cap;      // (a lane's largest is an element: more than the list has slots for)
            } else {
                const float edge = hi - ((float)(bin + 1) + 0.02f) * width;    // below every element of the bins up to the pivot
                tau = float_below(edge);
                open = cnt > crowd;
                need -= before;
                top = min(top, key_of_bits(__float_as_uint(hi - ((float)bin - 0.02f) * width)));
                bottom = max(bottom, key_of_bits(__float_as_uint(edge)));
            }
        }
        if (by_lanes && !counted) again = true;
        for (int pass = 0; open && !by_lanes && pass < 4; ++pass) {       // (a pass too many for the widest bin: one bin is one value by then)
            if (counted) {
                __syncthreads();
                clear();
                __syncthreads();
            }
            const uint32_t span = top - bottom;
            const int shift = max(0, 23 - (int)__clz((int)span));              // span >> shift < 2^9 = kSplitBins
            static_assert(kSplitBins == 1 << 9, "a bin for every value of nine bits");
#pragma unroll
            for (int e = 0; e < E; ++e) {
                uint32_t bits = __float_as_uint(v[e]);
                asm volatile("" : "+v"(bits));                       // (the keys are formed in each pass, not held from in front of the loop)
                const uint32_t d = top - key_of_bits(bits);          // (keys above top wrap far above span)
                if (d <= span) atomicAdd(&hist[d >> shift], 1u);
            }
            __syncthreads();
            counted = true;
            if (!find_pivot(need)) break;        // (the linear bins' margins: tau as it stands has them)
            const uint32_t last = min(span, ((uint32_t)(bin + 1) << shift) - 1u);
            tau = float_below(__uint_as_float(bits_of_key(top - last)));
            open = cnt > crowd && shift > 0;
            need -= before;
            bottom = top - last;
            top -= (uint32_t)bin << shift;
        }
    }

    // ---- the list: the elements above the threshold, in any order.  A lane marks its elements in a word, a scan over the
    //      counts gives it its slots, and it takes the few it marked from the image.
    marks = 0;                                   // bit 31 - e: element e
    // (v > tau is v >= the next larger float: the sign of v - that, shifted in and turned over.  It is finite also for a tau of -inf, whose own
    //  difference to a masked entry is a NaN)
    const float least = __uint_as_float(__float_as_uint(tau) + (tau < 0.f ? -1u : 1u));
#pragma unroll
    for (int e = 0; e < E; ++e) marks = __builtin_amdgcn_alignbit(marks, __float_as_uint(v[e] - least), 31);
    marks = ~marks << (32 - E);
    const int mine = __popc(marks);
    const int incl = wave_scan_incl(mine);
    if (lane == kWave - 1) wave_held[wave] = incl;
    if (THREADS > 256) lane_s[tid] = acc;
    else if (lane == 0) wave_s[wave] = ws;
    __syncthreads();
    at = incl - mine;
    held = 0;
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) { at += w < wave ? wave_held[w] : 0; held += wave_held[w]; }
    if (!(by_lanes || whole) || (!again && held <= cap)) break;
    // the elements themselves, then (the histogram is cleared; every wave has read the counts)
    tau = kNegInf;
    clear();
    __syncthreads();
    }
    const int64_t list = row * P + part;
    uint2* const out = lists + list * cap;
    const typename G::elem_t* const my_image = reinterpret_cast<const typename G::elem_t*>(image) + tid * N;
    if (held <= cap) {
        // (a lane's vectors go through LDS four at a time, so that it picks its marked elements by a computed address)
#pragma unroll
        for (int j0 = 0; j0 < NV; j0 += G::IV) {
#pragma unroll
            for (int j = 0; j < G::IV; ++j) {
                unsigned* const dst = &image[(j * THREADS + tid) * 4];
                if constexpr (BF16) {                // (packed again: the vectors as they were read would hold registers throughout)
                    unsigned p[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        p[q] = __builtin_amdgcn_perm(__float_as_uint(v[(j0 + j) * N + 2 * q + 1]), __float_as_uint(v[(j0 + j) * N + 2 * q]), 0x07060302u);
                    *reinterpret_cast<uint4*>(dst) = make_uint4(p[0], p[1], p[2], p[3]);
                } else *reinterpret_cast<float4*>(dst) = make_float4(v[(j0 + j) * N], v[(j0 + j) * N + 1], v[(j0 + j) * N + 2], v[(j0 + j) * N + 3]);
            }
            constexpr int kPer = G::IV * N;          // elements per batch
            unsigned m = (marks << (j0 * N)) & (0xFFFFFFFFu << (32 - kPer));
            while (m) {
                const int e = __clz((int)m);
                m &= ~(0x80000000u >> e);
                const int j = e / N, el = e % N;
                const unsigned bits = (unsigned)my_image[j * (THREADS * N) + el] << (BF16 ? 16 : 0);
                const int x = (split_block(G::nth(j0 + j, wave), wave & 3, part, P) * kWave + lane) * N - rv.o + el;
                if (SHARED) put_shared(reinterpret_cast<unsigned long long*>(&out[at++]), (unsigned long long)bits | (unsigned long long)(unsigned)x << 32);
                else out[at++] = make_uint2(bits, (unsigned)x);
            }
        }
    }
    if (THREADS > 256 && wave == 0) {                // (the two halves of what a lane of four waves holds, then its wave's lanes)
#pragma unroll
        for (int w = 0; w < 4; ++w) wave_s[w] = wave_sum((double)(lane_s[w * kWave + lane] + lane_s[(THREADS > 256 ? 256 : 0) + w * kWave + lane]));
    }
    if (tid == 0) {
        // (+inf in the row: given up, as by the other kernels' first pass; so is a share of NaN and nothing above -inf, whose sum the
        //  finishing kernel leaves out with its reference: any other NaN it finds in the row's sum)
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < 4; ++w) s += wave_s[w];
        SplitHead h{mx, tau, ref, finite || (!(mx > kNegInf) && s == s) ? held : cap + 1, s};
        if (SHARED) {
            const unsigned long long* src = reinterpret_cast<const unsigned long long*>(&h);
            unsigned long long* dst = reinterpret_cast<unsigned long long*>(heads + list);
#pragma unroll
            for (int i = 0; i < 3; ++i) put_shared(dst + i, src[i]);
        } else {
            heads[list] = h;
        }
    }
}

template <bool BF16> using SplitGeom256 = SplitGeom<BF16, kSplitThreads>;

template <bool BF16>
__global__ __launch_bounds__(kSplitThreads) void split_select_kernel(
    const void* __restrict__ logits, int64_t ld, int V, float inv_T, int rank, int cap, int narrow, int lanes,
    SplitHead* __restrict__ heads, uint2* __restrict__ lists,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ n_accept)
{
    __shared__ __align__(16) unsigned hist[SplitGeom256<BF16>::HIST], image[SplitGeom256<BF16>::IMAGE];
    split_select<BF16, kSplitThreads, false>(hist, image, blockIdx.y, (int)blockIdx.x, (int)gridDim.x, logits, ld, V, inv_T, rank, cap, narrow, lanes, heads, lists, seq_off, n_accept, [] {});
}

// A small round's draft rows and, in the same launch, the segment tables of its target rows: workgroups (x, y) with
// y < n_draft and x < parts select, those with y >= n_draft and x < stats_per_row sum.
template <bool BF16>
__global__ __launch_bounds__(kSplitThreads) void split_round_kernel(
    const void* __restrict__ draft_logits, int64_t ld_d, int n_draft, int V, float inv_T, int rank, int cap, int narrow, int lanes,
    SplitHead* __restrict__ heads, uint2* __restrict__ lists, int parts,
    const void* __restrict__ tgt_logits, int64_t ld_t, int stats_per_row, SegHeader* __restrict__ header, int seg_stride)
{
    __shared__ __align__(16) unsigned hist[SplitGeom256<BF16>::HIST], image[SplitGeom256<BF16>::IMAGE];
    const int x = blockIdx.x, y = blockIdx.y;
    if (y < n_draft) {
        if (x < parts) split_select<BF16, kSplitThreads, false>(hist, image, y, x, parts, draft_logits, ld_d, V, inv_T, rank, cap, narrow, lanes, heads, lists, nullptr, nullptr, [] {});
        return;
    }
    if (y == n_draft && x == 0 && threadIdx.x == 0)
        *header = SegHeader{kSegMagicSplit, kSplitStatsNV * kWave, seg_stride, (int32_t)gridDim.y - n_draft};
    if (x < stats_per_row)
        row_stats_parts<BF16>(y - n_draft, y - n_draft, x, tgt_logits, ld_t, V, inv_T, reinterpret_cast<float2*>(header + 1), seg_stride);
}

// A row whose lists do not hold its answer, from the start.  A function that is called: inlined, what that code keeps alive
// costs every row 0.8 to 1.1 us (one row of 128,256 bf16, k = 10: 6.0 -> 5.1; 64 of 151,936 fp32, k = 1024: 9.5 -> 8.4).
// (It is the fast kernels' code, which calls the careful pass in turn: a call, us, of 40 rows of 128,256, k = 512, that all came here, 13 entries above -inf in
// each: fp32 49.2 with both passes in the one function, 42.6 so, bf16 40.2 and 37.5; inlined, at every other row's cost, 37 and 36 to 38.)
template <bool BF16>
__device__ __attribute__((noinline)) void split_row_again(
    int64_t row, const void* logits, int64_t ld, int V, float inv_T, int k, float top_p,
    int32_t* idx, float* prob, int32_t* count, float* mass, float* lse, const int32_t* seq_off, const int32_t* n_accept, int rank_opt)
{
    row = uniform(row); V = uniform(V);
    compress_row<BF16, false>(row, record_source<BF16>(row, uniform(logits), uniform(ld), V, uniform(seq_off), uniform(n_accept)), V, uniform(inv_T),
                              uniform(k), uniform(top_p), uniform(idx), uniform(prob), uniform(count), uniform(mass), uniform(lse), uniform(rank_opt));
}

// The record of a row whose candidates are few enough to stay in the registers they were loaded into: SLOTS per thread, those of them valid
// of which `valid` has the bit.  As order_top_k and emit_row, with less between: one histogram, on a linear scale of the values (bf16: with
// the id, as its LINEAR places), whose bins hold one or two candidates of the upper end of any smooth distribution; the candidates of the
// bins up to the one that holds the n-th are laid out bin by bin, and whoever reads position i of that ranks it in its bin and writes it:
// positions i and their ranks are a bin apart, so the stores are as good as in order.  The scale goes from `low` to `high`; what lies above shares bin 0.
// Few::crowded, with nothing written: a bin is too crowded (values on a coarse grid); missing: the n-th does not lie above `above`, below which candidates are missing.
// `meanwhile` forms the row's sum of exponentials while the histogram's atomics are on their way.
// Bound by the chain of barriers, six of them (ten before): the finish of one row of 32,000 fp32, k = 64: 4.5 -> 3.6 us from its first instruction, of 64 of
// 151,936, k = 1024: 7.4 -> 5.6; a round of that row 16.4 -> 15.6, the draft of those 22.0 -> 20.0.
constexpr int kFewBins = kBins;                         // (a bin per word of the histogram)
// Entries of a bin that are ranked by comparing all: as many as values on a grid put there, which order_top_k, where fp32 values tie, would sort by a network.
// (64 rows of 151,936, k = 1024, us, in front of finish_few / up to 64 / so, with the selection as it is: fp32 on eighths 40.0 / 42.0 / 22.2, sixths 41.2 / 43.2 / 24.8,
// quarters 46.6 / 48.8 / 39.0; bf16 on sixths 22.0 / 23.4 / 16.7, whose places the ids spread: with up to 512, and the selection as it was, 24.6 for 21.8.)
template <bool BF16> constexpr int kFewMost = BF16 ? 256 : 512;
enum class Few { crowded, missing, done };
template <bool BF16, int SLOTS, class SH, class F>
__device__ __forceinline__ Few finish_few(
    SH& sh, const uint2 (&e)[SLOTS], const unsigned valid, const int n, const int V, const float low, const float high, const float M, const uint32_t above,
    const int64_t row, const int k, const bool direct, const float inv_T, int32_t* __restrict__ idx, float* __restrict__ prob,
    int32_t* __restrict__ count, float* __restrict__ mass, const F& meanwhile)
{
    static_assert(kFewBins == 4 * kT, "four bins per thread");
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    uint64_t* const buf = reinterpret_cast<uint64_t*>(sh.cand_val);
    const float id_step = __uint_as_float((unsigned)(127 - 8 - (32 - __clz(V - 1))) << 23);
    const float scale = (float)(kFewBins - 1) * __builtin_amdgcn_rcpf((high - low) + (BF16 ? fabsf(low) * 0.0078125f : 0.f));
    const float top = high * scale;
    auto bin_of = [&](float v, unsigned id) {
        const float w = BF16 ? fmaf(-(float)id, fabsf(v) * id_step, v) : v;
        unsigned b;
        asm("v_cvt_u32_f32 %0, %1" : "=v"(b) : "v"(fmaf(w, -scale, top)));       // (saturates)
        return min(b, (unsigned)(kFewBins - 1));
    };
    unsigned meta[SLOTS];                              // (bin << 16) | arrival order within the bin
    unsigned seen = 0;                                 // (an arrival of kFewMost or later leaves a bit)
    static_assert((kFewMost<BF16> & (kFewMost<BF16> - 1)) == 0, "one bit and those above it");
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        meta[u] = 0;
        if (valid >> u & 1u) {
            const unsigned b = bin_of(__uint_as_float(e[u].x), e[u].y);
            meta[u] = b << 16 | atomicAdd(&sh.hist[b], 1u);
            seen |= meta[u];
        }
    }
    const double S = meanwhile();
    if (seen & (0xFFFFu & ~(unsigned)(kFewMost<BF16> - 1))) sh.maxbin = 1;
    __syncthreads();
    if (sh.maxbin) return Few::crowded;                // (uniform)
    const uint4 h4 = *reinterpret_cast<const uint4*>(&sh.hist[4 * tid]);
    const int h[4] = {(int)h4.x, (int)h4.y, (int)h4.z, (int)h4.w};
    const int loc = (h[0] + h[1]) + (h[2] + h[3]), incl = wave_scan_incl(loc);
    if (lane == kWave - 1) sh.wtot[wave] = incl;
    __syncthreads();
    int at = incl - loc;
#pragma unroll
    for (int w = 0; w < kW; ++w) at += w < wave ? sh.wtot[w] : 0;
    unsigned first[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        first[j] = (unsigned)at;
        if (at < n && at + h[j] >= n) { sh.piv_bin = 4 * tid + j; sh.piv_before = at + h[j]; }
        at += h[j];
    }
    *reinterpret_cast<uint4*>(&sh.hist[4 * tid]) = make_uint4(first[0], first[1], first[2], first[3]);
    __syncthreads();
    const int piv = sh.piv_bin, n_keep = sh.piv_before;
#pragma unroll
    for (int u = 0; u < SLOTS; ++u)
        if ((valid >> u & 1u) && (int)(meta[u] >> 16) <= piv) buf[sh.hist[meta[u] >> 16] + (meta[u] & 0xFFFFu)] = composite<BF16>(e[u].x, e[u].y);
    __syncthreads();
    uint64_t* const ordered = buf + SH::kCap / 2;
    const double cd = 1.4426950408889634 * (double)inv_T, invS = 1.0 / S;
    int32_t* const idx_row = idx + row * (int64_t)k;
    float* const prob_row = prob + row * (int64_t)k;
    double my_mass = 0.0;
    for (int i = tid; i < n_keep; i += kT) {
        const uint64_t c = buf[i];
        const float v = __uint_as_float(bits_of_short_key<BF16>((uint32_t)(c >> kIdBits)));
        const unsigned id = kIdMask - ((uint32_t)c & kIdMask), b = bin_of(v, id);
        const int s = (int)sh.hist[b], end = (int)b < piv ? (int)sh.hist[b + 1] : n_keep;
        int larger = 0;
        for (int q = s; q < end; q += 4) {             // (four bin-mates per round trip to LDS)
            uint64_t m[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) m[u] = buf[min(q + u, SH::kCap / 2 - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) larger += (q + u < end && m[u] > c) ? 1 : 0;
        }
        const int pos = s + larger;
        if (pos >= n) continue;
        if (pos == n - 1 && (uint32_t)(c >> kIdBits) <= above) sh.overflowed = 1;
        if (direct) {
            const float p = (float)(exp_emit(v, M, cd) * invS);
            idx_row[pos] = (int)id;
            prob_row[pos] = p;
            my_mass += (double)p;
        } else {
            ordered[pos] = c;
        }
    }
    if (direct) {
        const double wm = wave_sum(my_mass);
        if (lane == 0) sh.red[wave] = wm;
    }
    __syncthreads();
    if (direct && tid == 0) {
        double tm = 0.0;
#pragma unroll
        for (int w = 0; w < kW; ++w) tm += sh.red[w];
        mass[row] = (float)tm;
        count[row] = n;
    }
    return sh.overflowed ? Few::missing : Few::done;
}

// SHARED: the lists were written by other workgroups of this launch.
template <bool BF16, bool SHARED>
__device__ __forceinline__ void split_finish(
    CompressShared<kCapBig>& sh, const int64_t row, const void* __restrict__ logits, int64_t ld, int V, float inv_T, int k, float top_p,
    int32_t* __restrict__ idx, float* __restrict__ prob, int32_t* __restrict__ count,
    float* __restrict__ mass, float* __restrict__ lse,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ n_accept,
    const SplitHead* __restrict__ heads, const uint2* __restrict__ lists, int n_lists, int cap, int rank_opt)
{
    using SH = CompressShared<kCapBig>;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const SplitHead* const head = heads + row * n_lists;
    const uint2* const list = lists + row * n_lists * (int64_t)cap;
    const float c = 1.4426950408889634f * inv_T;
    // ---- Everything is asked for at once: the lists' heads (by every wave for itself, one per lane) and the first kAhead * kT
    //      slots of the row's lists, whatever those turn out to hold.  Slot f of the row's lists: position f / n_lists of list f mod n_lists,
    //      so that what the lists do not fill are the last slots.
    constexpr int kAhead = 8;
    const int n_slots = n_lists * cap;
    const float per_round = 1.0f / (float)n_lists;
    auto place_of = [&](int f, int& l, int& q) { q = (int)(((float)f + 0.5f) * per_round); l = f - q * n_lists; };     // (f < 2^15: exact)
    auto entry = [&](int l, int q) {
        const uint2* const at = &list[l * cap + q];
        if (!SHARED) return *at;
        const unsigned long long t = get_shared(reinterpret_cast<const unsigned long long*>(at));
        return make_uint2((unsigned)t, (unsigned)(t >> 32));
    };
    uint4 h;
    double s_head;
    {
        const SplitHead* const my = head + min(lane, n_lists - 1);
        if (SHARED) {
            const unsigned long long* const w = reinterpret_cast<const unsigned long long*>(my);
            const unsigned long long h0 = get_shared(w), h1 = get_shared(w + 1), h2 = get_shared(w + 2);
            h = make_uint4((unsigned)h0, (unsigned)(h0 >> 32), (unsigned)h1, (unsigned)(h1 >> 32));
            s_head = __longlong_as_double((long long)h2);
        } else {
            h = *reinterpret_cast<const uint4*>(my);
            s_head = my->s;
        }
    }
    uint2 e[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
        int l, q;
        place_of(min(u * kT + tid, n_slots - 1), l, q);
        if (u * kT < n_slots) e[u] = entry(l, q);
    }
    zero_hist(sh);
    if (tid == 0) { sh.maxbin = 0; sh.overflowed = 0; }
    const bool mine = lane < n_lists;
    const float mx = mine ? __uint_as_float(h.x) : kNegInf, tau = mine ? __uint_as_float(h.y) : kNegInf;
    const float ref = mx > kNegInf ? __uint_as_float(h.z) : kNegInf;
    const int held = mine ? (int)h.w : 0;
    const float M = wave_max(mx), T = wave_max(tau);
    const float low = -wave_max(mine ? -tau : kNegInf);
    const bool over = __ballot(held > cap) != 0ull;
    const int incl = wave_scan_incl(held), total = read_lane(incl, kWave - 1);
    // (the share's sums meet in fp64; whole exponents: exact)
    auto sum_of_lists = [&] {
        const float R = wave_max(ref);
        const double S = wave_sum(ref > kNegInf ? ldexp(s_head, max((int)(ref - R), -2000)) : 0.0);
        return S * exp2_split((double)R - (double)M * (double)c);
    };
    const int n = min(total, k);
    const bool fill = total < k;
    bool ok = !over && total <= SH::kCap && total >= 1 && M > kNegInf && M < __builtin_huge_valf() &&
              (total >= k || T == kNegInf);      // (a threshold of -inf: every entry above -inf is listed)
    double S = 0.0;
    auto sound = [&] { return S > 0.0 && S < 1e300; };
    // finish_few's scale ends at the row's largest value, unless at least a quarter of the lists have theirs in the lowest eighth below it; then at the
    // largest of those: a few values far above the others would leave the others a few bins.  (us, in front of finish_few / with it, its scale up to M / so:
    // 64 rows of 151,936 fp32, k = 1024, one value of 200 in each 20.8 / 22.6 / 15.7; 8 of 128,256 bf16, k = 256: 14.4 / 15.8 / 10.1.)
    float high = M;
    const float near = fmaf(0.125f, M - low, low);
    if (4 * __popcll(__ballot(mx > near)) <= 3 * n_lists) high = wave_max(mx > near ? kNegInf : mx);
    const float spread = (float)(kFewBins - 1) / (high - low);
    if (ok && n_slots <= kAhead * kT && low > kNegInf && high > low && spread < __builtin_huge_valf() && fabsf(high) * spread < 1e9f) {
        const bool use_top_p = top_p > 0.f && top_p < 1.f;
        unsigned valid = 0;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            int l, q;
            const int f = u * kT + tid;
            place_of(f, l, q);
            if (u * kT < n_slots) valid |= f < n_slots && q < __shfl(held, l, kWave) ? 1u << u : 0u;
        }
        __syncthreads();
        const Few did = finish_few<BF16>(sh, e, valid, n, V, low, high, M, T == kNegInf ? 0u : short_key<BF16>(__float_as_uint(T)), row, k,
                                         !use_top_p && !fill, inv_T, idx, prob, count, mass, [&] { S = sum_of_lists(); return S; });
        if (did == Few::done && sound()) {
            if (tid == kT - 1) lse[row] = (float)((double)M * (double)inv_T + log(S));
            if (use_top_p || fill) emit_row<BF16>(sh, reinterpret_cast<uint64_t*>(sh.cand_val) + SH::kCap / 2, row, n, fill, M, S, inv_T, k, top_p, idx, prob, count, mass);
            return;
        }
        ok = did == Few::crowded;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");               // (what was written is written again)
        __syncthreads();
    }
    if (ok) {
        S = sum_of_lists();
        ok = sound();
    }
    if (ok) {
        const int first = incl - held;           // first slot, in the ordering's buffer, of list `lane`
        auto take = [&](int f, uint2 t) {
            int l, q;
            place_of(f, l, q);
            const int m = __shfl(held, l, kWave), s0 = __shfl(first, l, kWave);
            if (f < n_slots && q < m) { sh.cand_val[s0 + q] = t.x; sh.cand_id[s0 + q] = t.y; }
        };
#pragma unroll
        for (int u = 0; u < kAhead; ++u) if (u * kT < n_slots) take(u * kT + tid, e[u]);
        for (int f0 = kAhead * kT; f0 < n_slots; f0 += kT) {
            int l, q;
            place_of(min(f0 + tid, n_slots - 1), l, q);
            take(f0 + tid, entry(l, q));
        }
        order_prepare(sh, total);
        if (tid == kT - 1) lse[row] = (float)((double)M * (double)inv_T + log(S));
        __syncthreads();
        const uint32_t key_lo = short_key<BF16>(__float_as_uint(low)), key_hi = short_key<BF16>(__float_as_uint(M));
        const uint64_t* sorted;
        if (total <= 4 * kT)      sorted = order_top_k<BF16, 4>(sh, total, n, V, key_lo, key_hi);
        else if (total <= 8 * kT) sorted = order_top_k<BF16, 8>(sh, total, n, V, key_lo, key_hi);
        else                      sorted = order_top_k<BF16>(sh, total, n, V, key_lo, key_hi);
        // the lists hold every element above T: they hold the top k iff the k-th lies above it
        // (bf16: the short key of a T between two values is that of the lower one)
        if (T == kNegInf || (uint32_t)(sorted[n - 1] >> kIdBits) > short_key<BF16>(__float_as_uint(T))) {
            emit_row<BF16>(sh, sorted, row, n, fill, M, S, inv_T, k, top_p, idx, prob, count, mass);
            return;
        }
    }
    __syncthreads();
    split_row_again<BF16>(row, logits, ld, V, inv_T, k, top_p, idx, prob, count, mass, lse, seq_off, n_accept, rank_opt);
}

template <bool BF16>
__global__ __launch_bounds__(kT, 4) void split_finish_kernel(
    const void* __restrict__ logits, int64_t ld, int V, float inv_T, int k, float top_p,
    int32_t* __restrict__ idx, float* __restrict__ prob, int32_t* __restrict__ count,
    float* __restrict__ mass, float* __restrict__ lse,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ n_accept,
    const SplitHead* __restrict__ heads, const uint2* __restrict__ lists, int n_lists, int cap, int rank_opt)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    split_finish<BF16, false>(*reinterpret_cast<CompressShared<kCapBig>*>(smem_raw), blockIdx.x, logits, ld, V, inv_T, k, top_p, idx, prob, count, mass, lse,
                              seq_off, n_accept, heads, lists, n_lists, cap, rank_opt);
}

// Both in one launch: the last workgroup of a row to arrive (arrive_last) finishes it.  512 threads do the selection as well, half of a lane's
// elements each, and form the share's sum in the order of 256 (the same bits).  What it gives and the calls it serves: split_one_launch.
template <bool BF16>
__global__ __launch_bounds__(kT, 4) void split_compress_kernel(
    const void* __restrict__ logits, int64_t ld, int V, float inv_T, int rank, int cap, int narrow, int lanes, int k, float top_p,
    int32_t* __restrict__ idx, float* __restrict__ prob, int32_t* __restrict__ count,
    float* __restrict__ mass, float* __restrict__ lse,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ n_accept,
    SplitHead* __restrict__ heads, uint2* __restrict__ lists, unsigned long long* __restrict__ words, int rank_opt)
{
    using G = SplitGeom<BF16, kT>;
    using SH = CompressShared<kCapBig>;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    SH& sh = *reinterpret_cast<SH*>(smem_raw);
    static_assert(G::IMAGE <= SH::kCap && G::HIST <= SH::kCap, "the selection's arrays lie where the candidates will");
    const int64_t row = blockIdx.y;
    unsigned long long* const word = arrival_word(words, row);
    split_select<BF16, kT, true>(sh.cand_id, sh.cand_val, row, (int)blockIdx.x, (int)gridDim.x, logits, ld, V, inv_T, rank, cap, narrow, lanes, heads, lists,
                                 seq_off, n_accept, [&] { if (threadIdx.x == 0) open_arrival(word); });
    if (!arrive_last(word, gridDim.x, threadIdx.x == 0)) return;
    split_finish<BF16, true>(sh, row, logits, ld, V, inv_T, k, top_p, idx, prob, count, mass, lse, seq_off, n_accept, heads, lists, (int)gridDim.x, cap, rank_opt);
}

}  // namespace

namespace {

hipError_t launch_split_finish(const void* logits, int dtype, int64_t ld, int n_rows, int V, float temperature,
                               int k, float top_p, int32_t* idx, float* prob, int32_t* count, float* mass, float* lse,
                               const int32_t* seq_off, const int32_t* n_accept, const SplitPlan& p, const SplitHead* heads,
                               const uint2* lists, hipStream_t stream)
{
    static DeviceFlags limit_raised[2] = {};
    const int bf = dtype == 1;
    const size_t smem = sizeof(CompressShared<kCapBig>);
    int dev = 0;
    const void* const finish = bf ? (const void*)split_finish_kernel<true> : (const void*)split_finish_kernel<false>;
    if (hipError_t e = raise_lds_limit_once(finish, smem, limit_raised[bf], dev)) return e;
    const float inv_T = 1.0f / temperature;
    if (bf) hipLaunchKernelGGL(split_finish_kernel<true>, dim3(n_rows), dim3(kT), smem, stream, logits, ld, V, inv_T, k, top_p, idx, prob, count, mass, lse, seq_off, n_accept, heads, lists, p.parts, p.cap, compress_rank(k, V, false));
    else    hipLaunchKernelGGL(split_finish_kernel<false>, dim3(n_rows), dim3(kT), smem, stream, logits, ld, V, inv_T, k, top_p, idx, prob, count, mass, lse, seq_off, n_accept, heads, lists, p.parts, p.cap, compress_rank(k, V, false));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_split_compress(const void* logits, int dtype, int64_t ld, int n_rows, int V, float temperature,
                                 int k, float top_p, int32_t* idx, float* prob, int32_t* count, float* mass,
                                 float* lse, const int32_t* seq_off, const int32_t* n_accept, void* scratch, size_t scratch_bytes, hipStream_t stream)
{
    const SplitPlan p = split_plan(dtype, n_rows, V, k);
    const float inv_T = 1.0f / temperature;
    SplitHead* const heads = (SplitHead*)scratch;
    uint2* const lists = (uint2*)(heads + (size_t)n_rows * p.parts);
    const int narrow = p.rank <= kSplitNarrowRank;
    const dim3 grid(p.parts, n_rows);
    if (split_one_launch(dtype, n_rows, V, k) && scratch_bytes >= split_one_launch_bytes(dtype, n_rows, V, k) && !(n_rows < kOneLaunchSplitReplayed && is_captured(stream))) {
        static DeviceFlags limit_raised[2] = {};
        const int bf = dtype == 1;
        const size_t smem = sizeof(CompressShared<kCapBig>);
        int dev = 0;
        if (hipError_t e = raise_lds_limit_once(bf ? (const void*)split_compress_kernel<true> : (const void*)split_compress_kernel<false>, smem, limit_raised[bf], dev)) return e;
        unsigned long long* const words = (unsigned long long*)((char*)scratch + split_words_at(dtype, n_rows, V, k));
        // (twice the lanes, each with half as many elements)
        const int lanes = p.lanes ? (int)ceilf(512.f * (1.f - expf((float)p.rank * (-1.f / 512.f)))) : 0;
#define PICOSPEC_SPLIT(BF) \
        hipLaunchKernelGGL(split_compress_kernel<BF>, grid, dim3(kT), smem, stream, logits, ld, V, inv_T, p.rank, p.cap, narrow, lanes, k, top_p, idx, prob, count, mass, lse, seq_off, n_accept, heads, lists, words, compress_rank(k, V, false))
        if (bf) PICOSPEC_SPLIT(true); else PICOSPEC_SPLIT(false);
#undef PICOSPEC_SPLIT
        return hipGetLastError();
    }
    if (dtype == 1) hipLaunchKernelGGL(split_select_kernel<true>, grid, dim3(kSplitThreads), 0, stream, logits, ld, V, inv_T, p.rank, p.cap, narrow, p.lanes, heads, lists, seq_off, n_accept);
    else            hipLaunchKernelGGL(split_select_kernel<false>, grid, dim3(kSplitThreads), 0, stream, logits, ld, V, inv_T, p.rank, p.cap, narrow, p.lanes, heads, lists, seq_off, n_accept);
    if (hipError_t e = hipGetLastError()) return e;
    return launch_split_finish(logits, dtype, ld, n_rows, V, temperature, k, top_p, idx, prob, count, mass, lse, seq_off, n_accept, p, heads, lists, stream);
}

hipError_t launch_split_round(const void* draft_logits, int dtype, int64_t ld_d, int n_draft, int V, float temperature,
                              int k, float top_p, int32_t* idx, float* prob, int32_t* count, float* mass, float* lse,
                              const void* tgt_logits, int64_t ld_t, int n_target, void* seg_table, void* scratch, hipStream_t stream)
{
    const SplitPlan p = split_plan(dtype, n_draft, V, k);
    const StatsShape sh = split_stats_shape(dtype, V);
    const int per_row = stats_parts(sh.stride);
    const float inv_T = 1.0f / temperature;
    SplitHead* const heads = (SplitHead*)scratch;
    uint2* const lists = (uint2*)(heads + (size_t)n_draft * p.parts);
    const int narrow = p.rank <= kSplitNarrowRank;
    const dim3 grid(p.parts > per_row ? p.parts : per_row, n_draft + n_target);
    if (dtype == 1) hipLaunchKernelGGL(split_round_kernel<true>, grid, dim3(kSplitThreads), 0, stream, draft_logits, ld_d, n_draft, V, inv_T, p.rank, p.cap, narrow, p.lanes, heads, lists, p.parts, tgt_logits, ld_t, per_row, (SegHeader*)seg_table, sh.stride);
    else            hipLaunchKernelGGL(split_round_kernel<false>, grid, dim3(kSplitThreads), 0, stream, draft_logits, ld_d, n_draft, V, inv_T, p.rank, p.cap, narrow, p.lanes, heads, lists, p.parts, tgt_logits, ld_t, per_row, (SegHeader*)seg_table, sh.stride);
    if (hipError_t e = hipGetLastError()) return e;
    return launch_split_finish(draft_logits, dtype, ld_d, n_draft, V, temperature, k, top_p, idx, prob, count, mass, lse, nullptr, nullptr, p, heads, lists, stream);
}

}  // namespace picospec
