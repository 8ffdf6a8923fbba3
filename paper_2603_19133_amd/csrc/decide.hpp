// The per-sequence decisions of a round (paper Section 3.3), as device functions that a workgroup of kThreads
// threads runs for one sequence: accept_sequence (the acceptance test of every draft position and the first
// rejection) and residual_sequence (the correction or bonus token from norm(max(0, P_j - qhat_j))).  The
// library's kernels call them one per launch, or both from one workgroup.
#pragma once

#include "common.hpp"
#include "kernels.hpp"
#include "rowspan.hpp"

namespace picospec {

namespace {

// Clamp a range of draft positions to 0 <= begin <= end <= g; reports whether it had to.
__device__ __forceinline__ bool clamp_range(const int32_t* pos_begin, const int32_t* pos_end, int b, int g, int& begin, int& end) {
    const int rb = pos_begin ? pos_begin[b] : 0, re = pos_end ? pos_end[b] : g;
    end = re < 0 ? 0 : (re > g ? g : re);
    begin = rb < 0 ? 0 : (rb > end ? end : rb);
    return rb != begin || re != end;
}

// The statistics of one target row from its segment table in the split layout (row_stats_parts_kernel): M = the largest of
// the segments' maxima, S = their sums brought to M in fp64.  One wave, the result in every lane; the entries are asked for (load)
// apart from what is made of them.
struct TableStats {
    static constexpr int kAhead = 5;                 // entries per lane in flight (rows of up to 320 segments: one trip)
    float2 e[kAhead];
    // (lanes behind the last segment read that one again and are masked in combine: a load under a condition is waited for where the
    //  branch ends, and the next one is asked for behind it)
    template <bool SHARED = false>
    __device__ __forceinline__ void load(const float2* __restrict__ seg_row, int n_seg) {
        const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const float2* const p = &seg_row[min(u * kWave + lane, n_seg - 1)];
            e[u] = SHARED ? get_shared(p) : *p;
        }
    }
    template <bool SHARED = false>
    __device__ __forceinline__ void combine(const float2* __restrict__ seg_row, int n_seg, float c, float& M, double& S) {
        const int lane = threadIdx.x & (kWave - 1);
        float m = kNegInf;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) if (u * kWave + lane >= n_seg) e[u] = make_float2(0.f, kNegInf);
#pragma unroll
        for (int u = 0; u < kAhead; ++u) m = fmaxf(m, e[u].y);
        for (int s = kAhead * kWave + lane; s < n_seg; s += kWave) m = fmaxf(m, (SHARED ? get_shared(&seg_row[s]) : seg_row[s]).y);
        M = wave_max(m);
        const double top = (double)M * (double)c;
        auto term = [&](float2 t) { return t.x > 0.f || t.x != t.x ? (double)t.x * exp2_split(split_ref(t.y, c) - top) : 0.0; };
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) if (u * kWave < n_seg) s += term(e[u]);
        for (int q = kAhead * kWave + lane; q < n_seg; q += kWave) s += term(SHARED ? get_shared(&seg_row[q]) : seg_row[q]);
        S = wave_sum(s);
    }
};

// Where one wave finds a token in a position's record: the first 1024 ids (512 where the record is off the 16-byte boundary) are asked for apart
// from the search.
struct RecordScan {
    int4 front[4];
    bool aligned;
    __device__ __forceinline__ void load(const int32_t* __restrict__ ids, int k) {
        const int lane = threadIdx.x & (kWave - 1);
        aligned = ((uintptr_t)ids & 15u) == 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int s = u * kWave + lane;
            if (aligned) { if (s < (k >> 2)) front[u] = reinterpret_cast<const int4*>(ids)[s]; }
            else { if (s < k) front[u].x = ids[s]; if (s + 4 * kWave < k) front[u].y = ids[s + 4 * kWave]; }
        }
    }
    // the slot among the record's first cnt that holds x, or -1; in every lane.  PIN: fewer registers, some instructions more
    template <bool PIN = true>
    __device__ __forceinline__ int find(const int32_t* __restrict__ ids, int cnt, int x) const {
        int lane = threadIdx.x & (kWave - 1);
        if (PIN) asm volatile("" : "+v"(lane));           // (the slots are formed here, not held from in front of a caller's loop)
        int slot = -1;
        // The record is ordered by probability and the token was drawn from it, so it sits near the
        // front more often than not: the scan goes in rounds of 1024 ids and stops at the round
        // that holds it.
        if (aligned) {
            const int4* ids4 = reinterpret_cast<const int4*>(ids);
            const int n4 = cnt >> 2;
            auto look = [&](int s, const int4& q) {
                if (s < n4) {
                    if (q.x == x) slot = 4 * s;
                    if (q.y == x) slot = 4 * s + 1;
                    if (q.z == x) slot = 4 * s + 2;
                    if (q.w == x) slot = 4 * s + 3;
                }
            };
#pragma unroll
            for (int u = 0; u < 4; ++u) look(u * kWave + lane, front[u]);
            if (!__ballot(slot >= 0))
                for (int s0 = 4 * kWave; s0 < n4; s0 += 4 * kWave) {
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int s = s0 + u * kWave + lane;
                        if (s < n4) look(s, ids4[s]);
                    }
                    if (__ballot(slot >= 0)) break;
                }
            if (!__ballot(slot >= 0))
                for (int s = 4 * n4 + lane; s < cnt; s += kWave)
                    if (ids[s] == x) slot = s;
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int s = u * kWave + lane;
                if (s < cnt && front[u].x == x) slot = s;
                if (s + 4 * kWave < cnt && front[u].y == x) slot = s + 4 * kWave;
            }
            if (!__ballot(slot >= 0))
                for (int s0 = 8 * kWave; s0 < cnt; s0 += 8 * kWave) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int s = s0 + u * kWave + lane;
                        if (s < cnt && ids[s] == x) slot = s;
                    }
                    if (__ballot(slot >= 0)) break;
                }
        }
        const unsigned long long found = __ballot(slot >= 0);    // (one lane: the ids of a record are distinct)
        return found ? __builtin_amdgcn_readlane(slot, 63 - __clzll((long long)found)) : -1;
    }
};

struct SplitStats { double S; float M; };
// tgt_lse of the positions rows.x .. rows.y - 1 from what accept_sequence<.., TABLE> left in LDS, by `n` threads from thread
// `first` on (a logarithm in fp64: some hundred instructions that the deciding waves need not wait for).
__device__ __forceinline__ void write_split_lse(const SplitStats* s_stats, int2 rows, int64_t t0, float inv_T, float* tgt_lse, int first, int n) {
    for (int i = rows.x + (int)threadIdx.x - first; tgt_lse && i < min(rows.y, kSplitStatsRows); i += n)
        tgt_lse[t0 + i] = (float)((double)s_stats[i].M * (double)inv_T + log(s_stats[i].S));
}

// One workgroup (16 waves) per sequence, one wave per draft position.  The wave looks the drafted
// token up in the position's sparse record with 16-byte loads (four in flight per lane), front
// first, and stops once it is found.  What a position needs is asked for in two trips to memory: everything that depends
// only on the position (token, uniform, statistics, the record's first 1024 ids), then the target's logit and the
// record's probability of the token.  (Twelve loads in flight for a token behind the first 1024 ids: 10.4 -> 18 us at 512 sequences, k = 2048.)
// Returns the sequence's first rejected position (in every thread; a barrier stands behind the decision).
// TABLE: the rows' statistics are not known yet; their sums stand in the segment table (split layout,
// split_stats_serves): they are formed here and written to tgt_max / tgt_sum / tgt_lse.  s_stats (nullable, LDS): they
// are left there by position as well, and tgt_lse is not written: the caller does that off the critical path
// (write_split_lse), for the positions that come back in `rows`.
// Positions whose row lies outside the call's n_rows, or whose draft outside its n_rows - B drafts (offsets that leave them), are flagged and
// rejected; nothing is read or written for them.
// PIN: RecordScan::find's.
template <bool BF16, bool TABLE = false, bool PIN = true>
__device__ __forceinline__ int accept_sequence(
    const int b, const int B, const int n_rows, const void* __restrict__ tgt_logits, int64_t ld, int V, float inv_T,
    const int32_t* __restrict__ seq_off, const int32_t* __restrict__ draft_tok,
    const int32_t* __restrict__ q_idx, const float* __restrict__ q_prob,
    const int32_t* __restrict__ q_count, const float* __restrict__ q_mass, int k, int renorm,
    const float* __restrict__ q_scalar, const float* __restrict__ uniforms,
    float* __restrict__ tgt_max, float* __restrict__ tgt_sum,
    int32_t* __restrict__ n_accept, float* __restrict__ p_tok, float* __restrict__ q_tok,
    uint32_t* __restrict__ flags, const int32_t* __restrict__ pos_begin, const int32_t* __restrict__ pos_end,
    float* __restrict__ tgt_lse = nullptr, const SegHeader* __restrict__ table = nullptr, int seg_vecs = 0, int stride = 0,
    bool all_rows = false, SplitStats* s_stats = nullptr, int2* rows = nullptr)
{
    __shared__ int s_first;
    __shared__ unsigned s_flags;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);   // uniform: so are a position's addresses
    const int d0 = seq_off[b];
    int g = seq_off[b + 1] - d0;
    unsigned fl = 0;
    if (g < 0) { fl |= 8u; g = 0; }
    int begin, end;                                   // the draft positions this call verifies (all of them by default)
    if (clamp_range(pos_begin, pos_end, b, g, begin, end)) fl |= 8u;
    if (tid == 0) { s_first = end; s_flags = 0; }
    __syncthreads();
    const int64_t t0 = (int64_t)d0 + b;
    const float c = 1.4426950408889634f * inv_T;
    const double cd = 1.4426950408889634 * (double)inv_T;
    auto nonfinite = [](float M, float S) { return !(fabsf(M) < __builtin_huge_valf()) || !(S > 0.f) || !(S < __builtin_huge_valf()); };

    // every target row of the range must have finite statistics
    if constexpr (!TABLE) {
        if (t0 + begin < 0 || t0 + end >= n_rows) fl |= 8u;
        const int64_t row_end = min(t0 + end + 1, (int64_t)n_rows);
        for (int64_t r = max(t0 + begin, (int64_t)0) + tid; r < row_end; r += kThreads)
            if (nonfinite(tgt_max[r], tgt_sum[r])) fl |= 2u;
    }

    // (TABLE: the row behind the last position as well, and, where all of the call's rows get statistics, by the first and the last
    //  sequence's workgroup those in front of the first and behind the last sequence: seq_off may start above 0, and n_draft may be
    //  larger than seq_off[B], as for a batch that an uplink message clamped)
    int rows_begin = begin, rows_end = end;           // positions rows_begin .. rows_end - 1
    if constexpr (TABLE) {
        rows_begin = all_rows && b == 0 ? min(begin, -(int)t0) : begin;
        rows_end = all_rows && b + 1 == B ? max(end + 1, (int)(n_rows - t0)) : end + 1;
    }
    for (int i = rows_begin + wave; i < rows_end; i += kWaves) {
        const int64_t rt = t0 + i;
        bool decides = !TABLE || (i >= begin && i < end);             // (the other rows have statistics only)
        const int64_t rd = (int64_t)d0 + (decides ? i : 0);
        const bool outside = (PIN || !decides) && (rt < 0 || rt >= n_rows);           // (a draft of the call's has its row there)
        if (outside || (decides && (rd < 0 || rd >= n_rows - B))) {
            fl |= 8u;
            if (decides && lane == 0) atomicMin(&s_first, i);
            decides = false;
            if (outside || !TABLE || rt < 0 || rt >= n_rows) continue;
        }
        int x = -1, cnt = 0;
        float u_t = 0.f, mass_d = 1.f, M_t = 0.f, S_t = 1.f;
        double qh = 0.0;
        const int32_t* ids = q_idx;
        RecordScan scan;
        if (decides) {
            x = draft_tok[rd];
            u_t = uniforms[rt];
            if (!TABLE) { M_t = tgt_max[rt]; S_t = tgt_sum[rt]; }
            if (q_scalar) {
                qh = (double)q_scalar[rd];
            } else {
                cnt = q_count[rd];
                if (renorm) mass_d = q_mass[rd];
                ids = q_idx + rd * k;
                scan.load(ids, k);
            }
        }
        const float2* table_row = nullptr;
        int n_seg = 0;
        TableStats stats;
        if constexpr (TABLE) {
            const RowView rv = row_view<BF16>(tgt_logits, ld, rt, V);
            const int nq = (rv.L + Vec<BF16>::N - 1) / Vec<BF16>::N;
            n_seg = (nq + seg_vecs - 1) / seg_vecs;
            table_row = reinterpret_cast<const float2*>(table + 1) + rt * (int64_t)stride;
            stats.load(table_row, n_seg);
        }
        const bool bad = x < 0 || x >= V;
        const float z_t = bad || !decides ? 0.f : logit_at<BF16>(tgt_logits, ld, rt, x);
        float q_at = 0.f;                             // the record's probability of the token
        bool in_record = false;
        if (decides && !q_scalar) {
            cnt = cnt < 0 ? 0 : (cnt > k ? k : cnt);
            const int slot = scan.template find<PIN>(ids, cnt, x);
            in_record = slot >= 0 && !bad;
            if (in_record) q_at = q_prob[rd * k + slot];
        }
        // (the row's statistics are formed while the last two loads are on their way)
        if constexpr (TABLE) {
            double S;
            stats.combine(table_row, n_seg, c, M_t, S);
            S_t = (float)S;
            if (lane == 0) {
                tgt_max[rt] = M_t;
                tgt_sum[rt] = S_t;
                if (s_stats && i >= begin && i < kSplitStatsRows) s_stats[i] = SplitStats{S, M_t};
                else if (tgt_lse) tgt_lse[rt] = (float)((double)M_t * (double)inv_T + log(S));
                if (i >= begin && i <= end && nonfinite(M_t, S_t)) fl |= 2u;
            }
            if (!decides) continue;
        }
        if (!q_scalar) {
            if (in_record) {
                qh = (double)q_at;
                if (renorm) qh /= (double)mass_d;
            } else if (lane == 0) {
                fl |= 1u;
            }
        }
        if (lane == 0) {
            if (bad) fl |= 8u;
            double p = 0.0;
            if (!bad) p = exp_emit(z_t, M_t, cd) / (double)S_t;
            const double u = (double)u_t;
            // u < min(1, p/qhat), without forming the quotient; qhat = 0 counts as ratio = +inf.  An id outside the
            // vocabulary has p = 0 whatever qhat is said to be: it is rejected, so the accepted prefix ends in front of it
            const bool accept = !bad && (u < 1.0) && (qh > 0.0 ? (u * qh < p) : true);
            if (!accept) atomicMin(&s_first, i);
            if (p_tok) p_tok[rd] = (float)p;
            if (q_tok) q_tok[rd] = (float)qh;
        }
    }
    if (fl) atomicOr(&s_flags, fl);
    if (rows) *rows = make_int2(begin, rows_end);
    __syncthreads();
    const int first = s_first;
    if (tid == 0) {
        n_accept[b] = first;
        flags[b] = s_flags;
    }
    return first;
}

// What the acceptance of a position needs besides its row's statistics: qhat, the target's logit at the token, and flags (1: not in the record,
// 8: no id).  One wave, in every lane.
struct Looked { double qh; float z; unsigned fl; };
template <bool BF16>
__device__ __forceinline__ Looked look_up_position(
    const int64_t rd, const int64_t rt, const void* __restrict__ tgt_logits, int64_t ld, int V, const int32_t* __restrict__ draft_tok,
    const int32_t* __restrict__ q_idx, const float* __restrict__ q_prob, const int32_t* __restrict__ q_count, const float* __restrict__ q_mass,
    int k, int renorm, const float* __restrict__ q_scalar)
{
    const int x = draft_tok[rd];
    const bool bad = x < 0 || x >= V;
    Looked at{0.0, 0.f, bad ? 8u : 0u};
    float mass_d = 1.f;
    int cnt = 0;
    const int32_t* ids = q_idx;
    RecordScan scan;
    if (q_scalar) {
        at.qh = (double)q_scalar[rd];
    } else {
        cnt = q_count[rd];
        if (renorm) mass_d = q_mass[rd];
        ids = q_idx + rd * k;
        scan.load(ids, k);
    }
    at.z = bad ? 0.f : logit_at<BF16>(tgt_logits, ld, rt, x);
    if (!q_scalar) {
        const int slot = scan.find(ids, cnt < 0 ? 0 : (cnt > k ? k : cnt), x);
        if (slot >= 0 && !bad) {
            at.qh = (double)q_prob[rd * k + slot];
            if (renorm) at.qh /= (double)mass_d;
        } else {
            at.fl |= 1u;
        }
    }
    return at;
}

// The lookups of a sequence's positions by a workgroup of its own while others stream the rows, one wave per position: entry rt of `found` is kFoundWords
// words for the workgroup that decides to read (get_shared), the logit and the halves of qhat, each with the sequence it was looked up for and the first
// with the flags.  (Where offsets descend, positions of two sequences share a target row and its entry, which then holds words of
// either: the sequence that does not find its own looks up again.)
__device__ __forceinline__ void put_found(unsigned long long* entry, int b, const Looked& at) {
    const unsigned long long tag = (unsigned long long)(b + 1) << 40, qh = (unsigned long long)__double_as_longlong(at.qh);
    put_shared(entry, tag | (unsigned long long)at.fl << 32 | __float_as_uint(at.z));
    put_shared(entry + 1, tag | (qh & 0xFFFFFFFFull));
    put_shared(entry + 2, tag | qh >> 32);
}
struct Found {
    unsigned long long w[kFoundWords];
    __device__ __forceinline__ explicit Found(const unsigned long long* entry) {
#pragma unroll
        for (int i = 0; i < kFoundWords; ++i) w[i] = get_shared(entry + i);
    }
    // (uniform: every lane reads the same entry)
    __device__ __forceinline__ bool of(int b) const {
        const auto tag = [](unsigned long long v) { return (int)(v >> 40) - 1; };
        return __builtin_amdgcn_readfirstlane(tag(w[0]) == b && tag(w[1]) == b && tag(w[2]) == b);
    }
    __device__ __forceinline__ Looked looked() const {
        return Looked{__longlong_as_double((long long)(w[2] << 32 | (w[1] & 0xFFFFFFFFull))), __uint_as_float((unsigned)w[0]), (unsigned)(w[0] >> 32) & 0xFFu};
    }
};

template <bool BF16, int WAVES>
__device__ __forceinline__ void look_up_positions(
    const int b, const int d0, const int begin, const int end, const void* __restrict__ tgt_logits, int64_t ld, int V, int n_rows, int n_draft,
    const int32_t* __restrict__ draft_tok, const int32_t* __restrict__ q_idx, const float* __restrict__ q_prob,
    const int32_t* __restrict__ q_count, const float* __restrict__ q_mass, int k, int renorm, const float* __restrict__ q_scalar,
    unsigned long long* __restrict__ found)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    for (int i = begin + wave; i < end; i += WAVES) {
        const int64_t rd = (int64_t)d0 + i, rt = rd + b;
        if (rt < 0 || rt >= n_rows || rd < 0 || rd >= n_draft) continue;      // (offsets that leave the call's rows or drafts)
        const Looked at = look_up_position<BF16>(rd, rt, tgt_logits, ld, V, draft_tok, q_idx, q_prob, q_count, q_mass, k, renorm, q_scalar);
        if (lane == 0) put_found(found + kFoundWords * rt, b, at);
    }
}

// accept_sequence<.., TABLE> of a sequence whose table rows and lookups other workgroups of this launch have left: one wave per row, one trip
// to memory.  rows_begin .. rows_end - 1: the positions whose rows get statistics.  look_again(rd, rt) is look_up_position.
template <bool BF16, int WAVES, class F>
__device__ __forceinline__ void decide_spread(
    const int b, const int d0, unsigned fl, const int begin, const int end, const int rows_begin, const int rows_end,
    const void* __restrict__ tgt_logits, int64_t ld, int V, float inv_T, int n_rows, int n_draft, const float* __restrict__ uniforms,
    float* __restrict__ tgt_max, float* __restrict__ tgt_sum, float* __restrict__ tgt_lse,
    int32_t* __restrict__ n_accept, float* __restrict__ p_tok, float* __restrict__ q_tok, uint32_t* __restrict__ flags,
    const SegHeader* __restrict__ table, int stride, const unsigned long long* __restrict__ found, const F& look_again)
{
    __shared__ int s_first;
    __shared__ unsigned s_flags;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int64_t t0 = (int64_t)d0 + b;
    const float c = 1.4426950408889634f * inv_T;
    const double cd = 1.4426950408889634 * (double)inv_T;
    if (tid == 0) { s_first = end; s_flags = 0; }
    __syncthreads();
    float M = 0.f;
    double S = 1.0;
    int64_t wait_lse = -1;                            // the row whose log-sum-exp is still to be written
    auto write_lse = [&] { if (wait_lse >= 0 && tgt_lse && lane == 0) tgt_lse[wait_lse] = (float)((double)M * (double)inv_T + log(S)); };
    auto is_draft = [&](int i, int64_t rd) { return i >= begin && i < end && rd >= 0 && rd < n_draft; };
    // (one lane: the acceptance test of accept_sequence)
    auto decide = [&](int i, int64_t rd, const Looked& at, float M_t, float S_t, float u_t) {
        const bool bad = at.fl & 8u;
        const double u = (double)u_t, qh = at.qh;
        const double p = bad ? 0.0 : exp_emit(at.z, M_t, cd) / (double)S_t;
        fl |= at.fl;
        if (bad || !(u < 1.0) || !(qh > 0.0 ? (u * qh < p) : true)) atomicMin(&s_first, i);
        if (p_tok) p_tok[rd] = (float)p;
        if (q_tok) q_tok[rd] = (float)qh;
    };
    bool again = false;                               // some position's entry is another sequence's
    for (int i = rows_begin + wave; i < rows_end; i += WAVES) {
        const int64_t rt = t0 + i, rd = (int64_t)d0 + i;
        const bool outside = rt < 0 || rt >= n_rows, decides = is_draft(i, rd);
        if (outside || (i >= begin && i < end && !decides)) {        // (offsets that leave the call's rows, or its drafts: nothing is read or written there)
            fl |= 8u;
            if (i >= begin && i < end && lane == 0) atomicMin(&s_first, i);
            if (outside) continue;
        }
        const RowView rv = row_view<BF16>(tgt_logits, ld, rt, V);
        const int n_seg = stats_segments((rv.L + Vec<BF16>::N - 1) / Vec<BF16>::N);
        const float2* const table_row = reinterpret_cast<const float2*>(table + 1) + rt * (int64_t)stride;
        const Found entry(found + kFoundWords * rt);                 // (used where the row decides)
        const float u_t = uniforms[rt];
        TableStats stats;
        stats.load<true>(table_row, n_seg);
        write_lse();
        stats.combine<true>(table_row, n_seg, c, M, S);
        wait_lse = rt;
        const float S_t = (float)S;
        const bool mine = entry.of(b);
        again = again || (decides && !mine);
        if (lane == 0) {
            tgt_max[rt] = M;
            tgt_sum[rt] = S_t;
            if (i >= begin && i <= end && (!(fabsf(M) < __builtin_huge_valf()) || !(S_t > 0.f) || !(S_t < __builtin_huge_valf()))) fl |= 2u;
            if (decides && mine) decide(i, rd, entry.looked(), M, S_t, u_t);
        }
    }
    if (again) {                                      // (uniform; a pass of its own, which holds no row's statistics in registers: each wave reads those it wrote)
        write_lse();
        wait_lse = -1;
        for (int i = rows_begin + wave; i < rows_end; i += WAVES) {
            const int64_t rt = t0 + i, rd = (int64_t)d0 + i;
            if (rt < 0 || rt >= n_rows || !is_draft(i, rd) || Found(found + kFoundWords * rt).of(b)) continue;
            const Looked at = look_again(rd, rt);
            if (lane == 0) decide(i, rd, at, tgt_max[rt], tgt_sum[rt], uniforms[rt]);
        }
    }
    if (fl) atomicOr(&s_flags, fl);
    __syncthreads();
    if (tid == 0) {
        n_accept[b] = s_first;
        flags[b] = s_flags;
    }
    write_lse();
}


constexpr int kTile = kResidualTile;                          // elements per tile (both dtypes)
static_assert(kResidualThreads == kThreads, "one workgroup of kThreads threads per sequence");
constexpr int kSegLen = kTile / kWaves;                       // 1024 consecutive ids per wave and tile
constexpr int kMaxTiles = (kMaxV + 16) / kTile + 1;
constexpr int kMaxSeg = kMaxTiles * kWaves;

struct __align__(16) ResidualShared {
    float qimg[2][kTile];       // qhat images of two consecutive tiles (0 off-support)
    double seg[kMaxSeg];        // residual mass of each segment, id order
    double red[2 * kWaves];
    double before;              // cumulative residual in front of the chosen segment
    int seg_pick, seg_last;
};

static_assert(sizeof(ResidualShared) <= 160 * 1024, "LDS budget of one gfx950 CU");

// The draw of sequence b at its target row j_in (the first rejected position, or gamma_b for the bonus token).
template <bool BF16>
__device__ __forceinline__ void residual_sequence(
    const int b, const int j_in, const void* __restrict__ tgt_logits, int64_t ld, int V, float inv_T,
    const int32_t* __restrict__ seq_off,
    const float* __restrict__ tgt_max, const float* __restrict__ tgt_sum,
    const int32_t* __restrict__ q_idx, const float* __restrict__ q_prob,
    const int32_t* __restrict__ q_count, const float* __restrict__ q_mass, int k, int renorm,
    const float* __restrict__ uniforms,
    int32_t* __restrict__ out_tok, float* __restrict__ resid_mass, uint32_t* __restrict__ flags)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    ResidualShared& sh = *reinterpret_cast<ResidualShared*>(smem_raw);
    using Geom = ResidualGeom<BF16>;
    constexpr int N = Vec<BF16>::N, NV = Geom::NV;                     // vectors per thread and tile
    constexpr int kSegVec = Geom::SEG_VECS;                            // vectors per segment
    static_assert(Geom::TILE_VECS == kThreads * NV && kSegVec == NV * kWave, "tile geometry");
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);   // uniform: it forms scalar load offsets
    const int d0 = seq_off[b];
    int g = seq_off[b + 1] - d0;
    unsigned fl = 0;
    if (g < 0) { fl |= 8u; g = 0; }
    int j = j_in;
    if (j < 0 || j > g) { fl |= 8u; j = j < 0 ? 0 : g; }
    const int64_t rt = (int64_t)d0 + b + j;
    const int64_t rd = (int64_t)d0 + j;
    bool has_q = j < g;
    int cnt = 0;
    float q_scale = 1.f;
    if (has_q) {
        cnt = q_count[rd];
        cnt = cnt < 0 ? 0 : (cnt > k ? k : cnt);
        if (renorm) q_scale = 1.f / q_mass[rd];
    }
    const float M = tgt_max[rt];
    const float c = 1.4426950408889634f * inv_T;
    const RowView rv = row_view<BF16>(tgt_logits, ld, rt, V);
    const int n_tiles = (rv.L + kTile - 1) / kTile;
    const int n_seg = n_tiles * kWaves;
    const int32_t* ids = q_idx + rd * k;
    const float* qp = q_prob + rd * k;
    const int nq = (rv.L + N - 1) / N;
    // row loads: descriptor base + scalar offset of the vector group + this lane's offset.  On gfx950 a raw
    // buffer load compares scalar offset + lane offset + 16 with the descriptor's size (measured;
    // picospec_check_device() tests it), so vectors behind the row read as zero without touching memory
    const __amdgpu_buffer_rsrc_t row_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)rv.base, 0, nq * 16, 0x00020000);
    // vector `first + lane` of the row (first is uniform across the wave)
    auto load_vec = [&](int first) {
        const u32x4_t t = __builtin_amdgcn_raw_buffer_load_b128(row_rsrc, lane * 16, first * 16, 2 /* non-temporal */);
        return make_uint4(t.x, t.y, t.z, t.w);
    };

    // P(x) = 2^(z*c + kappa), kappa = -M*c - log2 S, so that one fused multiply-add and one exponential
    // form each probability.  kappa is rounded to fp32 once; that would scale every P by the same
    // factor 1 + eps, so qhat is scaled by it as well (the residuals then all carry it) and the sums
    // are divided by it at the end: the arithmetic stays that of P - qhat.
    const double kappa_d = -(double)M * (double)c - log2((double)tgt_sum[rt]);
    const float kappa = (float)kappa_d;
    const double common = exp2((double)kappa - kappa_d);       // 1 + eps
    // residual of the N elements of the 16-byte vector `raw` = vector q of the row, given the qhat image
    auto residual_of = [&](const uint4& raw, int q, const float* qimg, bool edge, float (&r)[N]) {
        float v[N];
        unpack<BF16>(raw, v);
        if (edge) {
            const unsigned vm = vec_valid_mask<BF16>(rv, q);
#pragma unroll
            for (int e = 0; e < N; ++e) {
                const float d = __builtin_amdgcn_exp2f(fmaf(v[e], c, kappa)) - qimg[e];
                r[e] = ((vm >> e) & 1u) && d > 0.f ? d : 0.f;
            }
        } else {
#pragma unroll
            for (int e = 0; e < N; ++e) r[e] = fmaxf(__builtin_amdgcn_exp2f(fmaf(v[e], c, kappa)) - qimg[e], 0.f);
        }
    };

    // this thread's share of the sparse record (k <= kMaxK), kept in registers across tiles
    constexpr int SP = kMaxK / kThreads;
    int my_id[SP];
    float my_q[SP];
#pragma unroll
    for (int z = 0; z < SP; ++z) {
        const int s = z * kThreads + tid;
        my_id[z] = -1;
        my_q[z] = 0.f;
        if (s < cnt) { my_id[z] = ids[s]; my_q[z] = (float)((double)qp[s] * (double)q_scale * common); }
    }
    // write (or take back) this thread's record entries that fall into ids [lo, lo + len)
    auto scatter = [&](float* img, int lo, int len, bool take_back) {
#pragma unroll
        for (int z = 0; z < SP; ++z) {
            const int off = my_id[z] - lo;
            if (my_id[z] >= 0 && off >= 0 && off < len) img[off] = take_back ? 0.f : my_q[z];
        }
    };

    {   // both images start empty
        float4* z4 = reinterpret_cast<float4*>(&sh.qimg[0][0]);
#pragma unroll
        for (int z = 0; z < 2 * kTile / 4 / kThreads; ++z) z4[z * kThreads + tid] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();

    // vector of (tile it, wave, jv, lane): it * (kThreads * NV) + wave * kSegVec + jv * kWave + lane
    const int wave_vec = wave * kSegVec;
    double R = 0.0;
    for (int attempt = 0; attempt < 2; ++attempt) {
        // three tiles in registers: one in use, two in flight (loads behind the row read zeros)
        uint4 tb[3][NV];
        auto load_tile = [&](int it, uint4 (&dst)[NV]) {
#pragma unroll
            for (int jv = 0; jv < NV; ++jv) dst[jv] = load_vec(Geom::group_first(it, wave, jv));
        };
        load_tile(0, tb[0]);
        load_tile(1, tb[1]);
        load_tile(2, tb[2]);
        if (has_q) scatter(sh.qimg[0], -rv.o, kTile, false);
        __syncthreads();
        auto step = [&](int it, uint4 (&buf)[NV]) {
            const float* img = sh.qimg[it & 1];
            const bool edge = it == 0 || it + 1 == n_tiles;
            double sum = 0.0;
#pragma unroll
            for (int jv = 0; jv < NV; ++jv) {
                float r[N];
                const int ql = wave_vec + jv * kWave + lane;             // vector within the tile
                residual_of(buf[jv], it * (kThreads * NV) + ql, img + ql * N, edge, r);
                float part = 0.f;
#pragma unroll
                for (int e = 0; e < N; ++e) part += r[e];
                sum += (double)part;
            }
            load_tile(it + 3, buf);
            sum = wave_sum(sum);
            if (lane == 0) sh.seg[it * kWaves + wave] = sum;
            __syncthreads();                                             // the image of this tile has been read
            if (has_q) {
                scatter(sh.qimg[it & 1], it * kTile - rv.o, kTile, true);
                if (it + 1 < n_tiles) scatter(sh.qimg[(it + 1) & 1], (it + 1) * kTile - rv.o, kTile, false);
            }
            __syncthreads();
        };
        // (whole groups of three in the loop, so that its body has one path and the waits for the loads
        // in flight stay exact; the last one or two tiles follow it)
        int it = 0;
        for (; it + 3 <= n_tiles; it += 3) {
            step(it, tb[0]);
            step(it + 1, tb[1]);
            step(it + 2, tb[2]);
        }
        if (it < n_tiles) step(it, tb[0]);
        if (it + 1 < n_tiles) step(it + 1, tb[1]);
        // total residual mass
        double part = 0.0;
        for (int s = tid; s < n_seg; s += kThreads) part += sh.seg[s];
        part = wave_sum(part);
        if (lane == 0) sh.red[wave] = part;
        __syncthreads();
        R = 0.0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) R += sh.red[w];
        __syncthreads();
        if (R > 0.0 || !has_q) break;   // (R still carries the common factor)
        // P == qhat numerically: draw from P itself
        fl |= 4u;
        has_q = false;
    }

    // locate the segment in which the cumulative residual first exceeds u*R
    const double target = (double)uniforms[(int64_t)d0 + b + g] * R;
    const int per = (n_seg + kThreads - 1) / kThreads;       // contiguous segments per thread
    const int s0 = min(n_seg, tid * per), s1 = min(n_seg, s0 + per);
    double mine = 0.0;
    for (int s = s0; s < s1; ++s) mine += sh.seg[s];
    double incl = wave_scan_incl(mine);
    if (lane == kWave - 1) sh.red[wave] = incl;
    if (tid == 0) { sh.seg_pick = 0x7FFFFFFF; sh.seg_last = -1; sh.before = 0.0; }
    __syncthreads();
    double before = 0.0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) if (w < wave) before += sh.red[w];
    double cum = before + incl - mine;
    int my_pick = 0x7FFFFFFF, my_last = -1;
    for (int s = s0; s < s1; ++s) {
        const double v = sh.seg[s];
        if (v > 0.0) my_last = s;
        if (my_pick == 0x7FFFFFFF && cum + v > target) my_pick = s;
        if (my_pick == 0x7FFFFFFF) cum += v;
    }
    if (my_pick != 0x7FFFFFFF) atomicMin(&sh.seg_pick, my_pick);
    if (my_last >= 0) atomicMax(&sh.seg_last, my_last);
    __syncthreads();
    int pick = __builtin_amdgcn_readfirstlane(sh.seg_pick);   // (uniform: it forms scalar load offsets below)
    const bool crossed = pick != 0x7FFFFFFF;
    if (!crossed) pick = max(__builtin_amdgcn_readfirstlane(sh.seg_last), 0);   // rounding: last segment with mass
    if (crossed && my_pick == pick) sh.before = cum;          // exactly one thread owns the chosen segment
    // (both images are empty again: every entry was taken back after its tile)
    const int pt = pick / kWaves, pw = pick % kWaves;
    const int seg_vec = pt * (kThreads * NV) + pw * kSegVec;  // first vector of the segment
    const int seg_lo = seg_vec * N - rv.o;                    // id of its first element
    if (has_q) scatter(sh.qimg[0], seg_lo, kSegLen, false);
    __syncthreads();

    // re-read that one segment and name the token (wave 0): ids ascend with (jv, lane, element)
    if (wave == 0) {
        const double base0 = sh.before;
        double base = base0;
        int tok = -1, last_tok = -1;
#pragma unroll
        for (int jv = 0; jv < NV; ++jv) {
            float r[N];
            const int ql = jv * kWave + lane;
            residual_of(load_vec(Geom::group_first(pt, pw, jv)), seg_vec + ql, sh.qimg[0] + ql * N, true, r);
            double sum = 0.0;
#pragma unroll
            for (int e = 0; e < N; ++e) sum += (double)r[e];
            const double inc = wave_scan_incl(sum);
            const unsigned long long hit = (crossed && tok < 0) ? __ballot(base + inc > target) : 0ull;
            if (hit) {
                const int owner = __ffsll((long long)hit) - 1;
                int t = -1;
                if (lane == owner) {
                    double cu = base + inc - sum;
#pragma unroll
                    for (int e = 0; e < N; ++e) {
                        cu += (double)r[e];
                        if (t < 0 && cu > target) t = seg_lo + ql * N + e;
                    }
                    if (t < 0) t = seg_lo + ql * N + N - 1;
                }
                tok = __shfl(t, owner, kWave);
            }
            // rounding fallback: the last id of the segment with residual mass
            const unsigned long long any = __ballot(sum > 0.0);
            if (any) {
                const int owner = 63 - __clzll((long long)any);
                int t = -1;
                if (lane == owner) {
#pragma unroll
                    for (int e = 0; e < N; ++e) if (r[e] > 0.f) t = seg_lo + ql * N + e;
                }
                last_tok = __shfl(t, owner, kWave);
            }
            base += __shfl(inc, kWave - 1, kWave);
        }
        if (tok < 0) tok = last_tok >= 0 ? last_tok : min(max(seg_lo, 0), V - 1);
        if (lane == 0) {
            out_tok[b] = tok;
            resid_mass[b] = (fl & 4u) ? 0.f : (float)(R / common);
            flags[b] = fl;
        }
    }
}

// ---------------------------------------------------------------- the same draw from the row's segment table
//
// With the exponential sums of the target row's segments at hand (written by the statistics pass: row_stats_seg_row)
// the row is not streamed again.  R = sum_x max(0, P(x) - qhat(x)) = sum over segments of (P(segment) - T(segment)),
// T = sum over the record's entries in the segment of min(P(x), qhat(x)): one gathered logit per record entry.  The
// segment in which the cumulative residual crosses u R is then read (one to four KB) and the token named as before.
// T is summed in 2^-62 fixed point (integer LDS atomics: the order of the additions does not change the result).
// Bound by latency: three dependent trips to memory and a chain of scans and barriers of 0.3 to 0.6 us each - one scan for the total and
// the place, the sum taken from the acceptance where that has it, no logarithm: 9.0 -> 8.3 us with the acceptance for one sequence of 32,000,
// 6.7 -> 6.25 alone for 24 of 33,001 - and for many sequences by the gathered logits (256 of 4096 entries: 13.7 of 24.5 us at 8 TB/s of lines).

constexpr int kMaxSegTable = 1040;                               // segments of the longest row (2^20 elements: 1025 of 4 KB or of 2 KB)
constexpr int kMaxSegElems = 256 * 8;                            // elements of the largest segment (256 vectors of bf16)

struct __align__(16) SegResidualShared {
    double pseg[kMaxSegTable];                 // P of each segment, then its residual mass
    unsigned long long tfix[kMaxSegTable];     // T of each segment, 2^-62 fixed point
    float qimg[kMaxSegElems];                  // qhat image of the chosen segment
    double red[2 * kWaves];
    double before;
    int seg_pick, seg_last;
    int tok, last_tok;                         // first id behind the crossing, last id with mass
};

// s_stats (nullable): the target rows' statistics by position, left in LDS by accept_sequence<.., TABLE>.
// by_sequence: the table holds one row per sequence, the one it draws from (launch_residual_split).
// RT: threads (whole waves from thread 0 on) that run this, at least k / 4: every wave more is one more that goes through the
// chain of scans and barriers, four instructions' time each once a SIMD holds several (residual_seg_threads).
// SHARED: the table was written by other workgroups of this launch (and has no header).
// A row outside the call's n_rows, or a record outside its n_draft (offsets that leave them), is flagged and gives token 0; nothing of it is read.
// GUARD: the place is looked at behind a branch.
template <bool BF16, int RT, bool SHARED = false, bool GUARD = false>
__device__ __forceinline__ void residual_seg_sequence(
    const int b, const int j_in, const int n_rows, const int n_draft, const void* __restrict__ tgt_logits, int64_t ld, int V, float inv_T,
    const int32_t* __restrict__ seq_off, const float* __restrict__ tgt_max, const SegHeader* __restrict__ table,
    const int seg_vecs, const int stride,
    const int32_t* __restrict__ q_idx, const float* __restrict__ q_prob,
    const int32_t* __restrict__ q_count, const float* __restrict__ q_mass, int k, int renorm,
    const float* __restrict__ uniforms,
    int32_t* __restrict__ out_tok, float* __restrict__ resid_mass, uint32_t* __restrict__ flags, const SplitStats* s_stats = nullptr,
    const bool by_sequence = false)
{
    __shared__ SegResidualShared sh;
    constexpr int N = Vec<BF16>::N;
    constexpr int SP = RT == kThreads ? kMaxK / kThreads : (RT == 512 ? 4 : 2);
    constexpr int RW = RT / kWave;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int d0 = seq_off[b];
    int g = seq_off[b + 1] - d0;
    unsigned fl = 0;
    if (g < 0) { fl |= 8u; g = 0; }
    int j = j_in;
    if (j < 0 || j > g) { fl |= 8u; j = j < 0 ? 0 : g; }
    int64_t rt = (int64_t)d0 + b + j;
    const int64_t rd = (int64_t)d0 + j;
    bool has_q = j < g;
    // (the answer is given where the table's header is looked at: a branch in front of the loads below costs 0.3 us.  The call's first row is read instead)
    bool outside = false;
    if (!GUARD || __builtin_expect(d0 < 0 || (int64_t)d0 + g > n_draft, 0)) {       // (uniform: whether some position of the sequence may be)
        outside = rt < 0 || rt >= n_rows || (has_q && (rd < 0 || rd >= n_draft));
        if (outside) { rt = 0; has_q = false; }
    }
    const RowView rv = row_view<BF16>(tgt_logits, ld, rt, V);
    const int nq = (rv.L + N - 1) / N;
    const int seg_elems = seg_vecs * N;
    const int n_seg = (nq + seg_vecs - 1) / seg_vecs;
    const float2* seg_row = reinterpret_cast<const float2*>(table + 1) + (by_sequence ? (int64_t)b : rt) * (int64_t)stride;
    // Everything that depends only on the two rows is asked for at once (one trip to memory): the table's header
    // (checked below), the target row's maximum, the record's count and mass, this thread's entries of the record and
    // its entries of the segment table.
    SegHeader hd{kSegMagicSplit, seg_vecs, stride, 0x7FFFFFFF};
    if (!SHARED) hd = *table;
    const float M = s_stats ? s_stats[min(j, kSplitStatsRows - 1)].M : tgt_max[rt];
    double S = s_stats ? s_stats[min(j, kSplitStatsRows - 1)].S : 0.0;
    const bool known = S > 0.0 && S < (double)__builtin_huge_valf();       // (else: the sum over the table's rows below)
    int cnt = 0;
    float mass_d = 1.f;
    int my_id[SP];
    float my_p[SP];
    if (has_q) {
        cnt = q_count[rd];
        if (renorm) mass_d = q_mass[rd];
#pragma unroll
        for (int z = 0; z < SP; ++z) {
            const int sl = z * RT + tid;
            my_id[z] = -1;
            my_p[z] = 0.f;
            if (sl < k) { my_id[z] = q_idx[rd * k + sl]; my_p[z] = q_prob[rd * k + sl]; }
        }
        cnt = cnt < 0 ? 0 : (cnt > k ? k : cnt);
    } else {
#pragma unroll
        for (int z = 0; z < SP; ++z) { my_id[z] = -1; my_p[z] = 0.f; }
    }
    const bool table_ok = n_seg <= stride && n_seg <= kMaxSegTable && seg_elems <= kMaxSegElems;
    float2 my_seg[(kMaxSegTable + RT - 1) / RT];
#pragma unroll
    for (int u = 0; u < (kMaxSegTable + RT - 1) / RT; ++u) {
        const int sg = u * RT + tid;
        my_seg[u] = make_float2(0.f, 0.f);
        if (table_ok && sg < n_seg) my_seg[u] = SHARED ? get_shared(&seg_row[sg]) : seg_row[sg];
    }
    // ... and, one trip later, the target's logit at each of this thread's record entries
    float my_z[SP];
#pragma unroll
    for (int z = 0; z < SP; ++z) {
        const int sl = z * RT + tid;
        if (!(sl < cnt && my_id[z] >= 0 && my_id[z] < V)) my_id[z] = -1;
        my_z[z] = my_id[z] >= 0 ? logit_at<BF16>(tgt_logits, ld, rt, my_id[z]) : 0.f;
    }
    const float c = 1.4426950408889634f * inv_T;
    const double cd = 1.4426950408889634 * (double)inv_T;
    const double q_scale = 1.0 / (double)mass_d;
    if (outside || !table_ok || (hd.magic != kSegMagic && hd.magic != kSegMagicSplit) || rt >= hd.rows || hd.stride != stride || hd.seg_vecs != seg_vecs) {
        if (tid == 0) { out_tok[b] = 0; resid_mass[b] = 0.f; flags[b] = fl | 8u; }     // (not the table of these rows)
        return;
    }

    // P of every segment, up to the common factor 1 / S
    double part = 0.0;
#pragma unroll
    for (int u = 0; u < (kMaxSegTable + RT - 1) / RT; ++u) {
        const int sg = u * RT + tid;
        if (sg < n_seg) {
            const float2 e = my_seg[u];
            // (the split layout keeps the segment's maximum, the other one its reference exponent)
            const double up = (hd.magic == kSegMagicSplit ? split_ref(e.y, c) : (double)e.y) - (double)M * (double)c;
            const double p = e.x > 0.f ? (double)e.x * exp2_split(up) : 0.0;
            sh.pseg[sg] = p;
            sh.tfix[sg] = 0ull;
            part += p;
        }
    }
    for (int i = tid; i < seg_elems; i += RT) sh.qimg[i] = 0.f;
    if (tid == 0) { sh.seg_pick = 0x7FFFFFFF; sh.seg_last = -1; sh.before = 0.0; sh.tok = 0x7FFFFFFF; sh.last_tok = -1; }
    if (!known) {                                 // (uniform)
        part = wave_sum(part);
        if (lane == 0) sh.red[wave] = part;
    }
    __syncthreads();
    if (!known) {
        S = 0.0;
#pragma unroll
        for (int w = 0; w < RW; ++w) S += sh.red[w];
    }
    const double invS = 1.0 / S;

    // this thread's share of the record: qhat and min(P, qhat) into the segment's T
    float my_q[SP];
#pragma unroll
    for (int z = 0; z < SP; ++z) {
        my_q[z] = 0.f;
        if (my_id[z] >= 0) {
            const double qh = (double)my_p[z] * q_scale;
            const double p = exp_emit(my_z[z], M, cd) * invS;
            const double m = p < qh ? p : qh;
            my_q[z] = (float)qh;
            atomicAdd(&sh.tfix[(my_id[z] + rv.o) / seg_elems], (unsigned long long)llrint(m * 4611686018427387904.0));
        }
    }
    __syncthreads();

    // residual mass of every segment, the total, and the segment in which the cumulative residual crosses u R
    const int per = (n_seg + RT - 1) / RT;        // contiguous segments per thread
    const int s0 = min(n_seg, tid * per), s1 = min(n_seg, s0 + per);
    auto seg_mass = [&](int s) {
        double r = sh.pseg[s] * invS;
        if (has_q) { r -= (double)sh.tfix[s] * (1.0 / 4611686018427387904.0); r = r > 0.0 ? r : 0.0; }
        return r;
    };
    // (one scan serves the total and the place: a wave's last lane holds its sum, and each attempt has words of its own for them)
    double R = 0.0, mine = 0.0, incl = 0.0, cum = 0.0;
    for (int attempt = 0; attempt < 2; ++attempt) {
        mine = 0.0;
        for (int s = s0; s < s1; ++s) mine += seg_mass(s);
        incl = wave_scan_incl(mine);
        double* const sums = sh.red + attempt * RW;
        if (lane == kWave - 1) sums[wave] = incl;
        __syncthreads();
        R = 0.0;
        double before = 0.0;
#pragma unroll
        for (int w = 0; w < RW; ++w) { const double t = sums[w]; if (w < wave) before += t; R += t; }
        cum = before + incl - mine;
        if (R > 0.0 || !has_q) break;
        fl |= 4u;                                              // P == qhat numerically: draw from P itself
        has_q = false;
    }
    const double target = (double)uniforms[(int64_t)d0 + b + g] * R;
    int my_pick = 0x7FFFFFFF, my_last = -1;
    for (int s = s0; s < s1; ++s) {
        const double v = seg_mass(s);
        if (v > 0.0) my_last = s;
        if (my_pick == 0x7FFFFFFF && cum + v > target) my_pick = s;
        if (my_pick == 0x7FFFFFFF) cum += v;
    }
    if (my_pick != 0x7FFFFFFF) atomicMin(&sh.seg_pick, my_pick);
    if (my_last >= 0) atomicMax(&sh.seg_last, my_last);
    __syncthreads();
    int pick = __builtin_amdgcn_readfirstlane(sh.seg_pick);
    const bool crossed = pick != 0x7FFFFFFF;
    if (!crossed) pick = max(__builtin_amdgcn_readfirstlane(sh.seg_last), 0);     // rounding: last segment with mass
    if (crossed && my_pick == pick) sh.before = cum;          // exactly one thread owns the chosen segment
    const int seg_vec = pick * seg_vecs;                      // first vector of the segment
    const int seg_lo = seg_vec * N - rv.o;                    // id of its first element
    // Wave w reads the segment's vectors w * 64 + lane (a segment has at most four times 64 of them); the loads are on their
    // way while the record's entries are laid out.
    static_assert(RW >= 4 && kMaxSegElems <= 4 * kWave * 8, "one wave per 64 vectors of the segment");
    const bool reads = wave * kWave < seg_vecs;               // (uniform)
    const int ql = wave * kWave + lane, q = seg_vec + ql;
    uint4 raw = make_uint4(0, 0, 0, 0);
    if (reads && vec_in_row<BF16>(rv, q)) raw = load16_stream(rv.base + q);
    if (has_q) {
#pragma unroll
        for (int z = 0; z < SP; ++z) {
            const int off = my_id[z] - seg_lo;
            if (my_id[z] >= 0 && off >= 0 && off < seg_elems) sh.qimg[off] = my_q[z];
        }
    }
    __syncthreads();

    // the token: ids ascend with (wave, lane, element)
    double r[N], sum = 0.0, inc = 0.0;
    if (reads) {
        float v[N];
        unpack<BF16>(raw, v);
        const unsigned vm = vec_valid_mask<BF16>(rv, q);
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const double d = exp_emit(v[e], M, cd) * invS - (double)sh.qimg[ql * N + e];
            r[e] = ((vm >> e) & 1u) && d > 0.0 ? d : 0.0;
            sum += r[e];
        }
        inc = wave_scan_incl(sum);
        if (lane == kWave - 1) sh.red[wave] = inc;
    }
    __syncthreads();
    if (reads) {
        double base = sh.before;
        for (int w = 0; w < wave; ++w) base += sh.red[w];
        const unsigned long long hit = crossed ? __ballot(base + inc > target) : 0ull;
        if (hit && lane == __ffsll((long long)hit) - 1) {
            double cu = base + inc - sum;
            int t = -1;
#pragma unroll
            for (int e = 0; e < N; ++e) {
                cu += r[e];
                if (t < 0 && cu > target) t = seg_lo + ql * N + e;
            }
            if (t < 0) t = seg_lo + ql * N + N - 1;
            atomicMin(&sh.tok, t);
        }
        const unsigned long long any = __ballot(sum > 0.0);   // rounding fallback: the last id of the segment with mass
        if (any && lane == 63 - __clzll((long long)any)) {
            int t = -1;
#pragma unroll
            for (int e = 0; e < N; ++e) if (r[e] > 0.0) t = seg_lo + ql * N + e;
            atomicMax(&sh.last_tok, t);
        }
    }
    __syncthreads();
    if (tid == 0) {
        int tok = sh.tok;
        if (tok == 0x7FFFFFFF) tok = sh.last_tok >= 0 ? sh.last_tok : min(max(seg_lo, 0), V - 1);
        out_tok[b] = tok;
        resid_mass[b] = (fl & 4u) ? 0.f : (float)R;
        flags[b] = fl;
    }
}

// ---------------------------------------------------------------- both decisions of a short draft, one wave per position
//
// The two functions above behind each other make five dependent trips to memory: offsets; the positions' tokens, ids and table rows; their
// logits; then the chosen row's record and table again; its gathered logits; the segment.  Here the wave of a position asks for its
// record's probabilities with the ids, and for the target's logits at all of them together with the token's, so that when the first
// rejection is known its wave holds all the draw needs in registers, its entries with their logits and its row's segments.  It
// sums, scans and picks the segment alone, without a barrier, and the whole workgroup names the token, one dword of the segment per thread.
// For records of up to 256 entries (kDecideRowsK) and drafts of up to 15 positions in a call whose table stands in the split layout: longer records
// pay for the gathers of the positions that are not drawn from, and with registers for 512 entries all calls take 0.9 us more.  Verification and draw in a replayed graph, us,
// general code / 256 entries / 512: 8 sequences of 8 drafts of 32,000 fp32, k = 64 12.5 / 10.8 / 11.9, 256 12.4 / 11.2 / 12.3, 320 13.0 / - / 12.4, 512 13.0 / - / 13.0; 16 of 8 of
// 151,936, k = 256 22.2 / 21.6 / 22.7, 320 22.5 / - / 23.0, 512 22.6 / - / 25.1; 12 of 14 of 128,256, k = 256 23.7 / 23.9 / 25.1, 320 24.5 / - / 26.9; bf16 17.9 / 17.4 / 18.4, 18.4 / - / 19.5.
// Bound by the chain of latencies: of 5.8 us
// for one sequence of 32,000 fp32, k = 64, the three trips are 0.7, 0.7 and 0.5, the scan of the segments and the token 1.0 each.
// General code / here, us a call: that round 18.7 / 16.4, 8 sequences of 8 drafts of 32,000 bf16, k = 256: 21.8 / 19.7, verification and draw of 16 of
// 151,936 fp32, k = 64: 18.9 / 17.1.
constexpr int kDecideRowsK = 256, kDecideRowsSegs = TableStats::kAhead * kWave;

// Whether sequence b can be decided so (uniform in the workgroup); rows of the call in front of the first and behind the last sequence,
// whose statistics accept_sequence writes, and offsets that leave the call's rows stay with the general code.
__device__ __forceinline__ bool decide_rows_serves(int b, int B, int d0, int d1, int n_rows) {
    const int g = d1 - d0, t0 = d0 + b;
    return g >= 0 && g < kWaves && d0 >= 0 && d1 <= n_rows - B && (b > 0 || t0 == 0) && (b + 1 < B || d1 + b + 1 == n_rows);
}

template <bool BF16>
__device__ __forceinline__ void decide_rows(
    const int b, const int d0, const int d1, const void* __restrict__ tgt_logits, int64_t ld, int V, float inv_T,
    const int32_t* __restrict__ draft_tok, const int32_t* __restrict__ q_idx, const float* __restrict__ q_prob,
    const int32_t* __restrict__ q_count, const float* __restrict__ q_mass, int k, int renorm,
    const float* __restrict__ uniforms, float* __restrict__ tgt_max, float* __restrict__ tgt_sum, float* __restrict__ tgt_lse,
    const SegHeader* __restrict__ table, int stride,
    int32_t* __restrict__ n_accept, float* __restrict__ p_tok, float* __restrict__ q_tok, uint32_t* __restrict__ flags,
    int32_t* __restrict__ out_tok, float* __restrict__ resid_mass, uint32_t* __restrict__ res_flags)
{
    constexpr int N = Vec<BF16>::N, SP = kDecideRowsK / kWave, U = TableStats::kAhead;
    constexpr int kSegVecs = kSplitStatsNV * kWave, kSegElems = kSegVecs * N;
    constexpr double kFix = 4611686018427387904.0;                 // 2^62
    static_assert(kSegVecs * 4 == kThreads, "one dword of the segment per thread");
    __shared__ unsigned long long tfix[kDecideRowsSegs];           // T of each segment of the chosen row, 2^-62 fixed point
    __shared__ float qimg[kSegElems];                              // qhat image of the chosen segment
    __shared__ double wave_mass[kWaves];
    __shared__ double s_before, s_target, s_R, s_invS;
    __shared__ float s_M;
    __shared__ int s_first, s_pick;                                // (s_pick: -1 - segment where the sum is not crossed)
    __shared__ unsigned s_flags, s_res_flags;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int g = d1 - d0;
    const int64_t t0 = (int64_t)d0 + b;
    const int i = min(wave, g);                                    // this wave's position; the last one is the bonus row's
    const bool mine = wave <= g, drafted = wave < g;
    const int64_t rt = t0 + i, rd = (int64_t)d0 + (drafted ? i : 0);
    const RowView rv = row_view<BF16>(tgt_logits, ld, rt, V);
    const int nq = (rv.L + N - 1) / N, n_seg = stats_segments(nq);
    const float2* const table_row = reinterpret_cast<const float2*>(table + 1) + rt * (int64_t)stride;
    const float c = 1.4426950408889634f * inv_T;
    const double cd = 1.4426950408889634 * (double)inv_T;
    // ---- one trip: what depends on the position alone.  Without a condition anywhere, since a load under one is waited for where its
    //      branch ends: the bonus row's wave asks for the first position's values and uses none, a sequence without drafts reads some float.
    TableStats stats;
    int my_id[SP];
    float my_p[SP];
    const float u_draw = uniforms[t0 + g];
    const bool any_q = g > 0;
    const int32_t* const ids = any_q ? q_idx + rd * k : (const int32_t*)uniforms;
    const float* const qp = any_q ? q_prob + rd * k : uniforms;
    const int last = any_q ? k - 1 : 0;
    const int tok_x = *(any_q ? draft_tok + rd : (const int32_t*)uniforms), count_d = *(any_q ? q_count + rd : (const int32_t*)uniforms);
    const float u_t = uniforms[rt], q_mass_d = *(any_q ? q_mass + rd : uniforms);
    stats.load(table_row, n_seg);
#pragma unroll
    for (int z = 0; z < SP; ++z) {
        const int sl = min(z * kWave + lane, last);
        my_id[z] = ids[sl];
        my_p[z] = qp[sl];
    }
    // (all of it: which row is drawn from is not known yet, and rows at other offsets of a 16-byte block differ by a segment)
    static_assert(kDecideRowsSegs <= kThreads, "one word per thread");
    if (tid < kDecideRowsSegs) tfix[tid] = 0ull;
    for (int s = tid; s < kSegElems; s += kThreads) qimg[s] = 0.f;
    if (tid == 0) { s_first = g; s_flags = 0; }
    __syncthreads();
    const int x = drafted ? tok_x : -1, cnt = !drafted || count_d < 0 ? 0 : (count_d > k ? k : count_d);
    const float mass_d = renorm ? q_mass_d : 1.f;
    float M = 0.f;
    double S = 0.0;
    float my_z[SP];
    if (mine) {
        // ---- one more: the target's logits at the record's ids and at the token
        unsigned fl = 0;
        bool found = false;
        float q_at = 0.f;
#pragma unroll
        for (int z = 0; z < SP; ++z) {
            const bool held = z * kWave + lane < cnt;
            if (held && my_id[z] == x) { found = true; q_at = my_p[z]; }
            if (!(held && my_id[z] >= 0 && my_id[z] < V)) my_id[z] = -1;
            my_z[z] = logit_at<BF16>(tgt_logits, ld, rt, max(my_id[z], 0));
        }
        const bool bad = x < 0 || x >= V;
        int x_at = bad ? 0 : x;
        asm("" : "+v"(x_at));                                      // (a vector load: a scalar one would be waited for here)
        const float z_t = logit_at<BF16>(tgt_logits, ld, rt, x_at);
        const unsigned long long at = __ballot(found);             // (one lane: the ids of a record are distinct)
        const bool in_record = at != 0ull && !bad;
        stats.combine(table_row, n_seg, c, M, S);
        const float S_t = (float)S;
        if (!(fabsf(M) < __builtin_huge_valf()) || !(S_t > 0.f) || !(S_t < __builtin_huge_valf())) fl |= 2u;
        if (drafted) {
            double qh = 0.0;
            if (in_record) {
                qh = (double)read_lane(q_at, 63 - __clzll((long long)at));
                if (renorm) qh /= (double)mass_d;
            } else {
                fl |= 1u;
            }
            if (bad) fl |= 8u;
            const double p = bad ? 0.0 : exp_emit(z_t, M, cd) / (double)S_t;
            const double u = (double)u_t;
            const bool accept = !bad && (u < 1.0) && (qh > 0.0 ? (u * qh < p) : true);   // (accept_sequence's test)
            if (lane == 0) {
                if (!accept) atomicMin(&s_first, i);
                if (p_tok) p_tok[rd] = (float)p;
                if (q_tok) q_tok[rd] = (float)qh;
            }
        }
        if (lane == 0) {
            tgt_max[rt] = M;
            tgt_sum[rt] = S_t;
            if (fl) atomicOr(&s_flags, fl);
        }
    }
    __syncthreads();
    const int j = s_first;
    if (tid == kThreads - 1) { n_accept[b] = j; flags[b] = s_flags; }
    if (wave == j) {                                               // (j <= g: this wave holds row j)
        // ---- the chosen row: residual mass of its segments, the total, and the segment in which the cumulative residual crosses u R
        // (as the draw from a table takes it: a sum that is no number is formed again from the segments that have one)
        double Sd = S;
        if (!(S > 0.0 && S < (double)__builtin_huge_valf())) {
            double s = 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) s += stats.e[u].x > 0.f ? (double)stats.e[u].x * exp2_split(split_ref(stats.e[u].y, c) - (double)M * (double)c) : 0.0;
            Sd = wave_sum(s);
        }
        const double invS = 1.0 / Sd, q_scale = 1.0 / (double)mass_d;
        float my_q[SP];
#pragma unroll
        for (int z = 0; z < SP; ++z) {
            my_q[z] = 0.f;
            if (z * kWave < k && my_id[z] >= 0) {
                const double qh = (double)my_p[z] * q_scale, p = exp_emit(my_z[z], M, cd) * invS;
                my_q[z] = (float)qh;
                atomicAdd(&tfix[(my_id[z] + rv.o) / kSegElems], (unsigned long long)llrint((p < qh ? p : qh) * kFix));
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // (LDS serves a wave in order)
        double p[U], r[U], incl[U], R = 0.0;
        const double top = (double)M * (double)c;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float2 e = stats.e[u];
            p[u] = u * kWave < n_seg && e.x > 0.f ? (double)e.x * exp2_split(split_ref(e.y, c) - top) * invS : 0.0;
        }
        bool has_q = drafted;
        unsigned fl = 0;
        for (int attempt = 0; attempt < 2; ++attempt) {
            R = 0.0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                r[u] = p[u];
                if (has_q && u * kWave < n_seg && u * kWave + lane < n_seg) {
                    r[u] -= (double)tfix[u * kWave + lane] * (1.0 / kFix);
                    r[u] = r[u] > 0.0 ? r[u] : 0.0;
                }
                incl[u] = 0.0;
                if (u * kWave < n_seg) incl[u] = R + wave_scan_incl(r[u]);
                if (u * kWave < n_seg) R = read_lane(incl[u], kWave - 1);
            }
            if (R > 0.0 || !has_q) break;
            fl |= 4u;                                              // P == qhat numerically: draw from P itself
            has_q = false;
        }
        const double target = (double)u_draw * R;
        int pick = -1, last = 0;
        double before = 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (u * kWave >= n_seg) break;
            const unsigned long long over = __ballot(incl[u] > target), any = __ballot(r[u] > 0.0);
            if (any) last = u * kWave + 63 - __clzll((long long)any);
            if (pick < 0 && over) {
                const int owner = __ffsll((long long)over) - 1;
                pick = u * kWave + owner;
                before = read_lane(incl[u] - r[u], owner);
            }
        }
        const int seg = pick >= 0 ? pick : last;                   // rounding: the last segment with mass
        const int seg_lo = seg * kSegElems - rv.o;
        if (has_q)
#pragma unroll
            for (int z = 0; z < SP; ++z) {
                const int off = my_id[z] - seg_lo;
                if (my_id[z] >= 0 && off >= 0 && off < kSegElems) qimg[off] = my_q[z];
            }
        if (lane == 0) {
            s_pick = pick >= 0 ? seg : -1 - seg;
            s_before = before;
            s_target = target;
            s_R = R;
            s_invS = invS;
            s_M = M;
            s_res_flags = fl;
        }
    }
    __syncthreads();
    // ---- the token: one dword of the segment per thread, ids ascend with (wave, lane, element)
    const bool crossed = s_pick >= 0;
    const int seg = __builtin_amdgcn_readfirstlane(crossed ? s_pick : -1 - s_pick);
    const RowView rj = row_view<BF16>(tgt_logits, ld, t0 + j, V);
    const int q = seg * kSegVecs + tid / 4, seg_lo = seg * kSegElems - rj.o;
    uint32_t raw = 0;
    if (vec_in_row<BF16>(rj, q)) raw = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(rj.base) + (int64_t)seg * kThreads + tid);
    if (mine && lane == 0 && tgt_lse) tgt_lse[rt] = (float)((double)M * (double)inv_T + log(S));     // (while that load is on its way)
    constexpr int E = BF16 ? 2 : 1;
    const double target = s_target, inv = s_invS;
    const float Mj = s_M;
    double r[E], sum = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int id = seg_lo + tid * E + e;
        const float v = BF16 ? __uint_as_float(e ? raw & 0xFFFF0000u : raw << 16) : __uint_as_float(raw);
        const double d = exp_emit(v, Mj, cd) * inv - (double)qimg[tid * E + e];
        r[e] = id >= 0 && id < V && d > 0.0 ? d : 0.0;
        sum += r[e];
    }
    const double inc = wave_scan_incl(sum);
    if (lane == kWave - 1) wave_mass[wave] = inc;
    __syncthreads();
    // every wave places the crossing for itself, by the waves' sums; the one it falls to names the token
    const double w_sum = lane < kWaves ? wave_mass[lane] : 0.0, w_incl = s_before + wave_scan_incl(w_sum);
    const unsigned long long over = crossed ? __ballot(lane < kWaves && w_incl > target) : 0ull, any = __ballot(w_sum > 0.0);
    const int owner = over ? __ffsll((long long)over) - 1 : any ? 63 - __clzll((long long)any) : 0;
    if (wave != owner) return;
    const double base = owner ? read_lane(w_incl, owner - 1) : s_before;
    const unsigned long long hit = over ? __ballot(base + inc > target) : 0ull, some = __ballot(sum > 0.0);
    const int who = hit ? __ffsll((long long)hit) - 1 : some ? 63 - __clzll((long long)some) : 0;
    if (lane != who) return;
    int tok = -1;
    if (hit) {
        double cu = base + inc - sum;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            cu += r[e];
            if (tok < 0 && cu > target) tok = seg_lo + tid * E + e;
        }
        if (tok < 0) tok = seg_lo + tid * E + E - 1;
    } else {                                                       // rounding fallback: the last id of the segment with mass
#pragma unroll
        for (int e = 0; e < E; ++e) if (r[e] > 0.0) tok = seg_lo + tid * E + e;
        if (tok < 0) tok = min(max(seg_lo, 0), V - 1);
    }
    out_tok[b] = tok;
    resid_mass[b] = s_res_flags & 4u ? 0.f : (float)s_R;
    res_flags[b] = s_res_flags;
}

}  // namespace

}  // namespace picospec
