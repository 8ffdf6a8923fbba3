"""Calls of few rows, whose rows are spread over many workgroups: the compression and the target rows' statistics against the
oracle at the edges of the rule and of its parts (two parts, a part with one block, the longest rows, the most rows), and
against the same calls with one workgroup per row."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_19133_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ps():
    from paper_2603_19133_amd import binding
    return binding


@pytest.fixture(scope="module")
def pu():
    import parity_util
    return parity_util


def _announce(*a):
    print("[case]", *a, flush=True)


def _unsplit(ps, z, V, T, k, top_p=0.0):
    """picospec_compress without a workspace: one workgroup per row."""
    out = ps.alloc_compressed(z.shape[0], k, z.device)
    p = lambda t: t.data_ptr()
    ps._check(ps.lib.picospec_compress(p(z), ps._dtype_code(z), z.stride(0), z.shape[0], V, T, k, top_p, p(out.idx), p(out.prob),
                                       p(out.count), p(out.mass), p(out.lse), None, 0, torch.cuda.current_stream().cuda_stream))
    return out


def _rows(rng, pattern, R, V):
    z = rng.standard_normal((R, V)) * 3
    if pattern == "trend":
        z = z + np.linspace(6, -6, V)
    elif pattern == "few_values":
        z = np.round(z)
    elif pattern == "one_value":
        z = np.full((R, V), -0.5)
    elif pattern == "outlier":
        z[:, V // 3] = 1e4
    elif pattern == "masked":
        z = np.where(rng.random((R, V)) < 0.97, -np.inf, z)
    elif pattern == "masked_lowest":
        z = np.where(rng.random((R, V)) < 0.9, np.finfo(np.float32).min, z)
    elif pattern == "masked_to_a_few":
        z = np.where(rng.random((R, V)) < 0.9999, -np.inf, z)
    elif pattern == "periodic":                  # one workgroup's blocks hold all of the large values
        z = z + 8.0 * ((np.arange(V) // 256) % 64 == 5)
    elif pattern == "plus_inf":
        z[:, 7] = np.inf
    return z.astype(np.float32)


# 8192 elements per workgroup: two parts, a block more, the longest row of 64 parts and the first that is not split
@pytest.mark.parametrize("V,R,k", [(16383, 2, 64), (16384, 2, 64), (16385, 3, 1), (16640, 2, 500), (24576, 192, 32), (24577, 193, 32),
                                   (50001, 4, 4096), (40000, 128, 1024), (40000, 80, 4096), (40000, 81, 4096), (32767, 2, 4096), (128256, 2, 10), (151936, 3, 1024), (152064, 1, 4096), (524288 - 64, 1, 4000),
                                   (524289, 1, 100)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_sizes_match_the_oracle_and_one_workgroup_per_row(gpu, pu, ps, V, R, k, dtype):
    _announce("split sizes", V, R, k, dtype)
    z = _rows(np.random.default_rng(V + k), "normal", R, V)
    stored = z if dtype == "f32" else W.to_bf16_bits(z)
    dev = pu.to_device(stored, gpu)
    g, u = ps.compress(dev, V, 0.9, k), _unsplit(ps, dev, V, 0.9, k)
    torch.cuda.synchronize()
    n = min(R, 4)
    pu.compare_compress(ps.Compressed(g.idx[:n], g.prob[:n], g.count[:n], g.mass[:n], g.lse[:n], k), oracle.compress(stored[:n], V, 0.9, k), 0.0)
    assert torch.equal(g.idx, u.idx) and torch.equal(g.count, u.count)
    pu.assert_close(pu.n(g.prob), pu.n(u.prob).astype(np.float64), 1e-6, "prob", atol=1e-38)


@pytest.mark.parametrize("pattern", ["trend", "few_values", "one_value", "outlier", "masked", "masked_lowest", "masked_to_a_few", "periodic"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("k,top_p", [(40, 0.0), (2000, 0.9)])
def test_patterns_match_the_oracle(gpu, pu, ps, pattern, dtype, k, top_p):
    _announce("split patterns", pattern, dtype, k, top_p)
    V, R, shift = 40003, 3, 1                    # rows off the 16-byte boundary
    z = _rows(np.random.default_rng(k), pattern, R, V + shift)
    stored = z if dtype == "f32" else W.to_bf16_bits(z)
    g = ps.compress(pu.to_device(stored, gpu)[:, shift:], V, 1.1, k, top_p)
    torch.cuda.synchronize()
    pu.compare_compress(g, oracle.compress(np.ascontiguousarray(stored[:, shift:]), V, 1.1, k, top_p), top_p)


def _share_heads(ps, z, V, k):
    """A compression in scratch of its own: the record, and per row and workgroup its threshold, the length of its list (what the
    selecting workgroups leave first in the scratch: 32 bytes each, third to last words unread here) and how many entries above -inf its
    share has (every P-th kilobyte of the row)."""
    dt, R = ps._dtype_code(z), z.shape[0]
    out = ps.alloc_compressed(R, k, z.device)
    ws = torch.zeros(ps.workspace_bytes(ps.CALL_COMPRESS, dt, R, V, k), dtype=torch.uint8, device=z.device)
    p = lambda t: t.data_ptr()
    ps._check(ps.lib.picospec_compress(p(z), dt, z.stride(0), R, V, 1.0, k, 0.0, p(out.idx), p(out.prob), p(out.count), p(out.mass), p(out.lse),
                                       p(ws), ws.numel(), torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    esz = z.element_size()
    per_block, blocks = 1024 // esz, ((V * esz + 15) // 16 + 1 + 63) // 64
    P = -(-blocks // (8192 // per_block))
    head = ws[:R * P * 32].view(R, P, 32)
    share = torch.zeros((R, blocks * per_block), dtype=torch.bool, device=z.device)
    share[:, :V] = z[:, :V] > float("-inf")
    share = share.view(R, blocks, per_block).sum(2)
    held = torch.stack([share[:, q::P].sum(1) for q in range(P)], 1)
    return out, head[:, :, 4:8].contiguous().view(torch.float32)[:, :, 0], head[:, :, 12:16].contiguous().view(torch.int32)[:, :, 0], held


@pytest.mark.parametrize("k", [10, 512, 1100])           # (ranks that are looked for among the lanes' largest values, and one that is not)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_a_share_with_fewer_entries_than_its_rank_lists_those_alone(gpu, pu, ps, dtype, k):
    """Vocabulary masks: a list of a share's entries above -inf holds none of the masked ones, and the row keeps its lists."""
    _announce("few entries in a share", dtype, k)
    V, rng = 128256, np.random.default_rng(k)
    z = np.full((4, V), -np.inf, np.float32)
    for r, n in enumerate((200, 60, 3000, 2)):
        at = rng.permutation(V)[:n]
        z[r, at] = rng.standard_normal(n)
    z[3, 100:103] = (1.0, 2.0, 3.0)              # (all in one share: the others have nothing)
    stored = z if dtype == torch.float32 else W.to_bf16_bits(z)
    out, tau, count, held = _share_heads(ps, pu.to_device(stored, gpu), V, k)
    pu.compare_compress(out, oracle.compress(stored, V, 1.0, k), 0.0)
    open_ = tau == float("-inf")
    assert open_[[0, 1, 3]].any(1).all() and torch.equal(count[open_].long(), held[open_].long())
    assert bool((count <= held).all())


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("k", [10, 40, 1100])
def test_a_share_of_one_value_lists_what_it_has(gpu, pu, ps, dtype, k):
    """One entry above -inf in every share, equal ones, and one value in all lanes but for smaller ones beside it: the lists hold the
    whole answer and say so; a share of nothing but one value is cut there."""
    _announce("one value in a share", dtype, k)
    V, rng = 128256, np.random.default_rng(k)
    block = 256 if dtype == torch.float32 else 512
    z = np.full((4, V), -np.inf, np.float32)
    z[0, np.arange(7, 16 * block, block)] = rng.standard_normal(16)               # (16 workgroups: the first block of each)
    z[1, np.arange(3, V - 1, 997)] = 0.5
    z[2, np.arange(8, 16 * block, block)] = 2.0
    z[2, np.arange(9, 16 * block, block)] = 1.0  # (the same lane's second entry)
    z[3] = -1.5
    stored = z if dtype == torch.float32 else W.to_bf16_bits(z)
    out, tau, count, held = _share_heads(ps, pu.to_device(stored, gpu), V, k)
    pu.compare_compress(out, oracle.compress(stored, V, 1.0, k), 0.0)
    assert bool((tau[:3] == float("-inf")).all()) and torch.equal(count[:3].long(), held[:3].long())
    assert bool((tau[3] > -2.0).all()) and bool((tau[3] < -1.5).all())


def _grid_rows(rng, pattern, R, V):
    """Rows whose k-th value is shared by more entries than there are candidate slots."""
    z = rng.standard_normal((R, V)) * 3
    if pattern == "steps":
        z = np.round(z / 2) * 2
    elif pattern == "early":                     # the ties that count stand at low ids, more densely than further on
        z = np.round((z + np.linspace(5, -5, V)) / 2) * 2
    elif pattern == "late":
        z = np.round((z + np.linspace(-5, 5, V)) / 2) * 2
    elif pattern == "zeros":                     # the threshold is zero, of either sign
        z = np.where(z > 7.5, z, np.where(rng.random((R, V)) < 0.5, 0.0, -0.0) * (z > -1) + np.where(z > -1, 0, -4))
    elif pattern == "negative":
        z = np.where(z > 8, 1.0, np.where(z > -2, -2.0, -6.0))
    elif pattern == "lowest":                    # a mask of the type's lowest value reaches into the record
        z = np.where(z > 7, z, -3.3895e38)
    return z.astype(np.float32)


@pytest.mark.parametrize("pattern", ["steps", "early", "late", "zeros", "negative", "lowest"])
@pytest.mark.parametrize("V,shift,k,top_p", [(32768, 0, 700, 0.0), (33001, 3, 2048, 0.0), (100003, 1, 777, 0.9), (152064, 0, 2048, 0.0), (152064, 0, 3000, 0.0)])
def test_rows_that_tie_at_the_threshold(gpu, pu, ps, pattern, V, shift, k, top_p):
    """Lower ids first among equal logits, also where only the ties of the lowest ids are looked at."""
    _announce("ties at the threshold", pattern, V, k, top_p)
    stored = W.to_bf16_bits(_grid_rows(np.random.default_rng(V + k), pattern, 3, V + shift))
    g = _unsplit(ps, pu.to_device(stored, gpu)[:, shift:], V, 0.9, k, top_p)
    torch.cuda.synchronize()
    pu.compare_compress(g, oracle.compress(np.ascontiguousarray(stored[:, shift:]), V, 0.9, k, top_p), top_p)


def test_rows_that_tie_at_the_threshold_keep_the_first_pass(gpu, ps):
    """A row streamed a second time, the careful way, takes four to five times a row that is not.  (Measured: 1.3 times.)"""
    _announce("time of ties at the threshold")
    B, V, k = 400, 128256, 1024
    g = torch.Generator(device=gpu)
    g.manual_seed(1)
    z = torch.randn((B, V), device=gpu, generator=g) * 3
    us = []
    for rows in (z.to(torch.bfloat16), ((z / 2).round() * 2).to(torch.bfloat16)):
        runs = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(10):
                ps.compress(rows, V, 1.0, k)
            b.record()
            torch.cuda.synchronize()
            runs.append(a.elapsed_time(b))
        us.append(sorted(runs[2:])[0])
    assert us[1] < 2.5 * us[0], us


# (the kernel of the small candidate buffer: the shortest rows it serves, its longest record; the safe pass keeps one sub-tile of
# 4096 elements as its first candidates there and fills the 5120 slots at once)
@pytest.mark.parametrize("pattern", ["one_value", "few_values", "ascending", "spike", "none"])
@pytest.mark.parametrize("V,ld,k,top_p", [(32768, 32768, 1, 0.0), (33001, 33004, 2048, 0.0), (33001, 33004, 777, 0.9)])
def test_rows_that_lose_the_first_pass_with_one_workgroup_per_row(gpu, pu, ps, pattern, V, ld, k, top_p):
    _announce("lost rows", pattern, V, k, top_p)
    rng = np.random.default_rng(V + k)
    z = _rows(rng, pattern, 5, ld)
    if pattern == "ascending":
        z = np.tile(np.linspace(-8, 8, ld, dtype=np.float32), (5, 1))
    elif pattern == "spike":                     # beside the sample's runs in most rows
        z[np.arange(5), (np.arange(5) * 6151 + 1234) % V] = 160.0
    elif pattern == "none":
        z[:] = -np.inf
        z[1:, 3] = 1.0
    stored = W.to_bf16_bits(z)
    g = _unsplit(ps, pu.to_device(stored, gpu)[:, :V], V, 0.9, k, top_p)
    torch.cuda.synchronize()
    if pattern == "none":                        # (a row without a finite value has ids in ascending order and no distribution)
        assert torch.equal(g.idx[0].cpu(), torch.arange(k, dtype=torch.int32)) or top_p
        g = ps.Compressed(g.idx[1:], g.prob[1:], g.count[1:], g.mass[1:], g.lse[1:], k)
        stored = stored[1:]
    pu.compare_compress(g, oracle.compress(np.ascontiguousarray(stored[:, :V]), V, 0.9, k, top_p), top_p)


# (candidates are claimed by 32-bit words, two elements of a bf16 row: words that begin in front of a row or end behind it, with values there that
# would head the record, and rows whose candidates come in pairs)
@pytest.mark.parametrize("V,ld,k", [(33001, 33003, 300), (33000, 33001, 2048), (33001, 33002, 3000), (12001, 12001, 64)])
def test_words_on_the_rows_edges_and_pairs_with_one_workgroup_per_row(gpu, pu, ps, V, ld, k):
    _announce("words on the edges", V, ld, k)
    rng = np.random.default_rng(V + ld)
    R = 6
    flat = np.full(R * ld + 8, 50.0, np.float32)                 # (what lies between the rows)
    rows = _rows(rng, "normal", R, V)
    rows[1::2, 1:] = np.maximum(rows[1::2, 1:], rows[1::2, :-1])   # neighbours share their larger value: ties in pairs
    for r in range(R):
        flat[1 + r * ld:1 + r * ld + V] = rows[r]
    bits = W.to_bf16_bits(flat)
    dev = pu.to_device(bits, gpu)
    z = torch.as_strided(dev, (R, V), (ld, 1), 1)
    g = _unsplit(ps, z, V, 0.9, k)
    torch.cuda.synchronize()
    stored = np.stack([bits[1 + r * ld:1 + r * ld + V] for r in range(R)])
    pu.compare_compress(g, oracle.compress(np.ascontiguousarray(stored), V, 0.9, k), 0.0)


# (bf16 candidates are ordered by places on a linear scale: equal values spread by id between two neighbours of the type, also where the
# neighbours' distance changes - powers of two, next to zero - and where the scale ends; hundreds of zeros at the cut share one place)
@pytest.mark.parametrize("pattern", ["across_zero", "zeros_at_the_cut", "powers_of_two", "tiny", "subnormal", "huge", "few_across_zero", "zipf"])
@pytest.mark.parametrize("V,k", [(32768, 2048), (131072, 2048), (40001, 3000), (33001, 10)])
def test_orders_of_bf16_values_with_one_workgroup_per_row(gpu, pu, ps, pattern, V, k):
    _announce("bf16 orders", pattern, V, k)
    rng = np.random.default_rng(V + k)
    R = 4
    z = rng.standard_normal((R, V))
    share = 1.1 * k / V                                          # of the values above the middle of the pattern
    if pattern == "across_zero":
        z = z - np.quantile(z, 1 - share / 2)
    elif pattern == "zeros_at_the_cut":
        z = np.where(rng.random((R, V)) < share / 2, np.abs(z), np.where(rng.random((R, V)) < share, 0.0, -1.0 - np.abs(z)))
    elif pattern == "powers_of_two":
        z = np.sign(z) * np.exp2(np.round(np.abs(z) * 4) - 4)
    elif pattern == "tiny":
        z = (z - np.quantile(z, 1 - share)) * 1e-20
    elif pattern == "subnormal":
        z = z * 2e-39
    elif pattern == "huge":
        z = z * 3e37
    elif pattern == "few_across_zero":
        z = np.round((z - np.quantile(z, 1 - share / 2)) * 4) / 4
    else:
        z = 0.5 * z - 1.2 * np.log(np.floor(rng.random((R, V)) * V) + 1) + rng.standard_normal((R, V))
    stored = W.to_bf16_bits(z.astype(np.float32))
    T = 1e-20 if pattern == "tiny" else 1e37 if pattern == "huge" else 0.9
    g = _unsplit(ps, pu.to_device(stored, gpu), V, T, k)
    torch.cuda.synchronize()
    pu.compare_compress(g, oracle.compress(stored, V, T, k), 0.0)


@pytest.mark.parametrize("V,k,top_p", [(33001, 1, 0.0), (33001, 777, 0.9), (152064, 2048, 0.0)])
@pytest.mark.parametrize("zeros,masked", [(129, False), (900, False), (900, True), (1, True)])
def test_equal_values_next_to_zero_with_one_workgroup_per_row(gpu, pu, ps, V, k, top_p, zeros, masked):
    """Zeros (of either sign) among the candidates of bf16 rows, which a linear scale of the values cannot tell apart; also in rows that
    hold fewer entries above -inf than the record is long."""
    _announce("equal values next to zero", V, k, top_p, zeros, masked)
    rng = np.random.default_rng(zeros)
    z = (rng.standard_normal((5, V)) - 6).astype(np.float32)
    if masked:
        z[:, rng.random(V) < 0.995] = -np.inf
    for r in range(5):
        at = rng.permutation(V)[:zeros]
        z[r, at] = np.where(rng.random(zeros) < 0.5 * (r % 3), np.float32(-0.0), np.float32(0.0))
        z[r, rng.permutation(V)[:20]] = 3.0
    stored = W.to_bf16_bits(z)
    u = _unsplit(ps, pu.to_device(stored, gpu), V, 1.0, k, top_p)
    torch.cuda.synchronize()
    pu.compare_compress(u, oracle.compress(stored, V, 1.0, k, top_p), top_p)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_infinities_and_nan_as_with_one_workgroup_per_row(gpu, ps, dtype):
    _announce("split infinities", dtype)
    V, k = 30000, 20
    z = torch.from_numpy(_rows(np.random.default_rng(3), "plus_inf", 4, V)).to(gpu).to(dtype)
    z[1] = float("-inf")
    z[2, 5] = float("nan")
    z[2, 7] = 0.0
    z[3] = torch.finfo(dtype).min
    g, u = ps.compress(z, V, 1.0, k), _unsplit(ps, z, V, 1.0, k)
    torch.cuda.synchronize()
    for r in (0, 1, 3):                          # (the entries of a row with a NaN are whatever they are; the statistics are NaN)
        assert torch.equal(g.idx[r], u.idx[r]) and torch.equal(g.count[r], u.count[r])
        assert torch.allclose(g.prob[r], u.prob[r], rtol=1e-6, atol=0, equal_nan=True)
    assert torch.allclose(g.lse, u.lse, rtol=1e-6, atol=0, equal_nan=True)


# (ranks up to 100 find their threshold by the lanes' largest values first: k = 308 and 1129 are the last that do in 5 and 19 parts)
@pytest.mark.parametrize("pattern", ["normal", "one_lane", "few_lanes", "masked_but_a_lane", "masked_but_many", "crowded"])
@pytest.mark.parametrize("V,k", [(16384, 1), (33001, 308), (33001, 309), (151936, 1129), (151936, 1130)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_thresholds_by_lanes_match_the_oracle_and_one_workgroup_per_row(gpu, pu, ps, pattern, V, k, dtype):
    """Large values in one lane or few of every wave (lists too long for the lanes' threshold), masks that leave too few lanes, equal values."""
    _announce("thresholds by lanes", pattern, V, k, dtype)
    z = np.random.default_rng(k).standard_normal((3, V)).astype(np.float32) * 3
    lane = np.arange(V) // (4 if dtype == "f32" else 8) % 64
    if pattern == "one_lane":
        z += np.float32(20) * (lane == 17)
    elif pattern == "few_lanes":
        z += np.float32(20) * (lane % 16 == 5)
    elif pattern == "masked_but_a_lane":
        z[:, lane != 63] = -np.inf
    elif pattern == "masked_but_many":
        z[:, lane % 3 > 0] = -np.inf
    elif pattern == "crowded":
        z = np.minimum(z, np.float32(2))
    stored = z if dtype == "f32" else W.to_bf16_bits(z)
    dev = pu.to_device(stored, gpu)
    g, u = ps.compress(dev, V, 0.9, k), _unsplit(ps, dev, V, 0.9, k)
    torch.cuda.synchronize()
    pu.compare_compress(g, oracle.compress(stored, V, 0.9, k), 0.0)
    assert torch.equal(g.idx, u.idx) and torch.equal(g.count, u.count)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V,R,T", [(16384, 3, 1.0), (33001, 224, 0.7), (128256, 5, 0.05), ((1 << 20) - 5, 2, 1.0)])
def test_row_statistics(gpu, pu, ps, dtype, V, R, T):
    _announce("split statistics", dtype, V, R, T)
    g = torch.Generator(device=gpu)
    g.manual_seed(V)
    z = (torch.randn((R, V + 3), device=gpu, generator=g) * 4).to(dtype)[:, 1:V + 1]
    z[0, : V // 2] = torch.finfo(dtype).min     # whole segments of masked entries, by the type's lowest value and by -inf
    z[1, V // 2:] = float("-inf")
    mx, sm, lse = ps.row_stats(z, V, T)
    x = z.double().cpu()
    m = x.max(1).values
    s = torch.exp((x - m[:, None]) / T).sum(1)
    assert torch.equal(mx.double().cpu(), m)
    pu.assert_close(pu.n(sm), s.numpy(), pu.RTOL, "sum")
    pu.assert_close(pu.n(lse), (m / T + torch.log(s)).numpy(), pu.RTOL_LSE, "lse", atol=2e-6)


@pytest.mark.parametrize("rows", ["all_lowest", "all_neg_inf", "nan", "plus_inf"])
def test_statistics_of_degenerate_rows(gpu, ps, rows):
    """What a row of nothing but masked entries, or with a NaN or an infinity in it, gave before it gives with its statistics
    spread over many workgroups."""
    _announce("split degenerate statistics", rows)
    V = 20000
    z = torch.randn((2, V), device=gpu)
    z[1] = {"all_lowest": torch.finfo(torch.float32).min, "all_neg_inf": float("-inf")}.get(rows, 0.0)
    if rows == "nan":
        z[1, 9] = float("nan")
    if rows == "plus_inf":
        z[1, 9] = float("inf")
    got = ps.row_stats(z, V, 1.0)
    want = [torch.empty(2, device=gpu) for _ in range(3)]
    ps._check(ps.lib.picospec_row_stats(z.data_ptr(), ps.F32, V, 2, V, 1.0, *[t.data_ptr() for t in want],
                                        torch.cuda.current_stream().cuda_stream))
    # (row_stats takes one workgroup per row at this size; a verification that is given a workspace spreads them)
    off, tok = torch.tensor([0, 1], dtype=torch.int32, device=gpu), torch.zeros(1, dtype=torch.int32, device=gpu)
    v = ps.verify(z, V, 1.0, off, 1, tok, None, torch.rand(2, device=gpu), q_scalar=torch.rand(1, device=gpu),
                  workspace=ps.alloc_workspace(torch.float32, 2, V, gpu))
    torch.cuda.synchronize()
    for got in (got, (v.tgt_max, v.tgt_sum, v.tgt_lse)):
        for a, b in zip(got, want):
            assert torch.allclose(a, b, rtol=1e-6, atol=0, equal_nan=True), (a, b)


def test_rows_behind_the_last_sequence_keep_their_statistics(gpu, ps):
    """n_draft may be larger than seq_off[B] (a batch that an uplink message clamped): all n_draft + B rows get statistics."""
    _announce("split statistics behind the last sequence")
    V, B, N = 20000, 2, 7
    tgt = torch.randn((N + B, V), device=gpu)
    off = torch.tensor([0, 2, 4], dtype=torch.int32, device=gpu)
    tok = torch.zeros(N, dtype=torch.int32, device=gpu)
    v = ps.verify(tgt, V, 1.0, off, N, tok, None, torch.rand(N + B, device=gpu), q_scalar=torch.rand(N, device=gpu))
    assert torch.equal(v.tgt_max, tgt.max(1).values)
    assert torch.allclose(v.tgt_lse, torch.logsumexp(tgt, 1), rtol=1e-5)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("R", [223, 224, 225])
def test_long_sequences_on_either_side_of_the_rule(gpu, ps, monkeypatch, R, dtype):
    """One sequence of R - 1 drafts, rejected at its last or its first but two: the edge of the rule by rows, and the most
    positions whose statistics the deciding workgroup keeps in LDS."""
    _announce("split statistics of long sequences", R, dtype)
    V, k, T, N = 16384, 64, 0.9, R - 1
    g = torch.Generator(device=gpu)
    g.manual_seed(R)
    tgt = (torch.randn((R, V), device=gpu, generator=g) * 2).to(dtype)
    q = ps.compress(tgt[:N].contiguous(), V, T, k)               # (mass < 1: q > p on every entry of the record)
    off = torch.tensor([0, N], dtype=torch.int32, device=gpu)
    tok = q.idx[:, 0].contiguous()
    for reject in (N - 1, 2):
        u = torch.zeros(R, device=gpu)
        u[reject], u[-1] = 0.9999999, 0.37
        res = []
        for split in (True, False):
            if not split:
                monkeypatch.setattr(ps, "_split_stats", lambda *a: False)
            res.append(ps.verify_sample(tgt, V, T, off, N, tok, q, u))
            monkeypatch.undo()
        (v, r), (v0, r0) = res
        assert int(v.n_accept[0]) == reject and int(v0.n_accept[0]) == reject and not v.flags.any() and not r.flags.any()
        assert torch.equal(v.tgt_max, tgt.float().max(1).values)
        assert torch.allclose(v.tgt_lse.double(), torch.logsumexp(tgt.double() / T, 1), rtol=1e-6, atol=2e-6)
        assert torch.allclose(v.p_tok, v0.p_tok, rtol=2e-6, atol=0)
        assert torch.equal(r.out_tok, r0.out_tok) and torch.allclose(r.resid_mass, r0.resid_mass, rtol=1e-5, atol=1e-7)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V,B,k", [(16385, 1, 1), (33001, 24, 70), (128256, 3, 1024), (40000, 2, 1025), (32768, 2, 5), (33000, 129, 257), (33000, 257, 257), (33000, 1024, 10), (33000, 1025, 10)])
def test_draw_without_a_table_makes_one(gpu, pu, ps, V, B, k, dtype):
    """The correction draw of few sequences from a table that it forms itself: against the oracle, at first rejections from
    the first position to the bonus row, with one out of range (clamped and flagged, as without the table)."""
    _announce("draw with a table of its own", V, B, k, dtype)
    T, g = 0.9, torch.Generator(device=gpu)
    g.manual_seed(V + B)
    gam = torch.tensor([b % 3 for b in range(B)], dtype=torch.int32)
    gam[0] = 2
    off = torch.zeros(B + 1, dtype=torch.int32)
    off[1:] = gam.cumsum(0)
    N = int(off[-1])
    tgt = (torch.randn((N + B, V + 1), device=gpu, generator=g) * 2).to(dtype)[:, 1:]     # (rows off the 16-byte boundary)
    rows = [int(off[b]) + b + i for b in range(B) for i in range(int(gam[b]))]
    draft = (tgt[rows].float() + torch.randn((N, V), device=gpu, generator=g)).to(dtype)
    q = ps.compress(draft, V, T, k)
    u = torch.rand(N + B, device=gpu, generator=g)
    tok = q.idx[:, 0].contiguous()
    ver = ps.verify(tgt, V, T, off.to(gpu), N, tok, q, u)
    na = torch.tensor([b % (int(gam[b]) + 1) for b in range(B)], dtype=torch.int32)
    if B > 1:
        na[1] = 9
    d = lambda t: t.to(gpu)
    got = ps.sample_residual(tgt, V, T, d(off), N, ver, q, u, n_accept=d(na))
    plain = ps.alloc_residual(B, tgt.device)
    p = lambda t: t.data_ptr()
    o_d, na_d = d(off), d(na)
    ps._check(ps.lib.picospec_sample_residual(p(tgt), ps._dtype_code(tgt), tgt.stride(0), V, T, B, N, p(o_d), p(na_d), p(ver.tgt_max), p(ver.tgt_sum),
                                              p(q.idx), p(q.prob), p(q.count), p(q.mass), k, 1, p(u), p(plain.out_tok), p(plain.resid_mass), p(plain.flags),
                                              None, 0, torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert torch.equal(got.flags, plain.flags) and int(got.flags.sum()) == (8 if B > 1 else 0)
    # two fp32 sums of the row: the mass agrees to their rounding, and the token unless the uniform falls within it of a step
    assert torch.allclose(got.resid_mass, plain.resid_mass, rtol=1e-5, atol=1e-6)
    assert (got.out_tok != plain.out_tok).sum().item() <= B // 200
    for b in range(min(B, 4)):
        j = min(int(na[b]), int(gam[b]))
        r = int(off[b]) + b + j
        pr = torch.softmax(tgt[r].double() / T, 0)
        if j < int(gam[b]):
            i, n = int(off[b]) + j, int(q.count[int(off[b]) + j])
            pr[q.idx[i, :n].long()] -= q.prob[i, :n].double() / q.mass[i].double()
        res = pr.clamp_min(0).cpu()
        cum = res.cumsum(0) / res.sum()
        x, uu = int(got.out_tok[b]), float(u[int(off[b]) + b + int(gam[b])])
        assert abs(float(got.resid_mass[b]) - float(res.sum())) < 2e-6 * max(1.0, float(res.sum()))
        assert float(cum[x]) > uu - 1e-5 and (x == 0 or float(cum[x - 1]) < uu + 1e-5)


@pytest.mark.parametrize("k", [1, 3, 10, 255, 256, 257, 777, 1021, 1024, 1025, 2047, 2049, 4093, 4096])
@pytest.mark.parametrize("R", [1, 5, 513])
def test_draw_from_records_of_every_length(gpu, pu, ps, k, R):
    """The drafter's draw against the oracle: pieces of four slots, the last one cut, counts of 1 to k, up to 512 rows and more."""
    _announce("draw", k, R)
    rng = np.random.default_rng(k * 1000 + R)
    p = np.sort(rng.random((R, k)).astype(np.float32) ** 4, axis=1)[:, ::-1].copy()
    cnt = rng.integers(1, k + 1, R).astype(np.int32)
    cnt[0] = k
    p[np.arange(k)[None, :] >= cnt[:, None]] = 0
    ids = rng.integers(0, 1 << 20, (R, k)).astype(np.int32)
    mass = p.astype(np.float64).sum(1).astype(np.float32)
    u = rng.random(R, dtype=np.float32)
    q = oracle.Compressed(ids, p.astype(np.float64), cnt, mass.astype(np.float64), mass.astype(np.float64), np.ones(R), k)
    tok, slot, margin = oracle.sample_draft(q, u)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(gpu)
    g_tok, g_q = ps.sample_draft(ps.Compressed(d(ids), d(p), d(cnt), d(mass), d(mass), k), d(u))
    torch.cuda.synchronize()
    # (fp64 sums in another order: a uniform within 1e-12 of a step is the only way to differ)
    sure = margin > 1e-12
    assert sure.mean() > 0.99 and np.array_equal(pu.n(g_tok)[sure], tok[sure])
    want = p[np.arange(R), slot].astype(np.float64) / mass
    pu.assert_close(pu.n(g_q)[sure], want[sure], pu.RTOL, "q_scalar", atol=1e-37)


def test_a_workspace_that_is_refused_stays_refused(gpu, ps):
    """Calls that bring a buffer of their own still look at the one they are given."""
    _announce("refused workspace")
    V, k = 20000, 8
    d, t = torch.randn((2, V), device=gpu), torch.randn((3, V), device=gpu)
    off = torch.tensor([0, 2], dtype=torch.int32, device=gpu)
    tok, u = torch.zeros(2, dtype=torch.int32, device=gpu), torch.rand(3, device=gpu)
    good = torch.empty(ps.workspace_bytes(ps.CALL_ROUND, ps.F32, 3, V, 0) + 16, dtype=torch.uint8, device=gpu)
    q, v, _ = ps.round(d, t, V, 1.0, off, 2, tok, k, u, workspace=good)
    for bad in (good[:64], good[8:]):
        for call in (lambda: ps.round(d, t, V, 1.0, off, 2, tok, k, u, workspace=bad), lambda: ps.verify(t, V, 1.0, off, 2, tok, q, u, workspace=bad),
                     lambda: ps.verify_sample(t, V, 1.0, off, 2, tok, q, u, workspace=bad),
                     lambda: ps.sample_residual(t, V, 1.0, off, 2, v, q, u, workspace=bad)):
            with pytest.raises(ps.PicoSpecError) as e:
                call()
            assert e.value.code == ps.EWORKSPACE


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("where", ["whole_segment", "among_masked", "last_segment", "masked_row"])
def test_nan_in_a_segment_without_a_finite_value_is_flagged(gpu, ps, dtype, where):
    """A segment (256 vectors of 16 bytes) that holds NaN and nothing above -inf: the row's log-sum-exp is not finite, with its
    statistics spread over many workgroups as with one workgroup per row."""
    _announce("NaN in a segment without a finite value", dtype, where)
    seg = 1024 if dtype == torch.float32 else 2048
    V, B = 20 * seg + 3, 3
    tgt = torch.randn((2 * B, V), device=gpu).to(dtype)          # one draft per sequence: rows 2 b and 2 b + 1
    bad = 3                                      # (the second row of sequence 1)
    if where == "whole_segment":
        tgt[bad, 4 * seg:5 * seg] = float("nan")
    elif where == "among_masked":
        tgt[bad, 4 * seg:5 * seg] = float("-inf")
        tgt[bad, 4 * seg + 777] = float("nan")
    elif where == "last_segment":
        tgt[bad, 20 * seg:] = float("nan")
    else:
        tgt[bad] = float("-inf")
        tgt[bad, 12] = 1.0
        tgt[bad, 7 * seg + 5] = float("nan")
    base = torch.zeros((2 * B, (V + 7) // 8 * 8), dtype=dtype, device=gpu)   # (rows on the 16-byte boundary: a segment is whole ids)
    base[:, :V] = tgt
    z = base[:, :V]
    off = torch.arange(B + 1, dtype=torch.int32, device=gpu)
    tok, u = torch.zeros(B, dtype=torch.int32, device=gpu), torch.rand(2 * B, device=gpu)
    q = ps.compress(torch.randn((B, V), device=gpu).to(dtype), V, 1.0, 8)
    ws = ps.alloc_workspace(dtype, 2 * B, V, gpu)
    for ver in (ps.verify(z, V, 1.0, off, B, tok, q, u, workspace=ws), ps.verify_sample(z, V, 1.0, off, B, tok, q, u, workspace=ws)[0],
                ps.verify_range(z, V, 1.0, off, B, tok, q, u, None, None, 1)):
        torch.cuda.synchronize()
        assert [bool(f & ps.FLAG_NONFINITE) for f in ver.flags.tolist()] == [False, True, False], (ver.flags, ver.tgt_sum)
        assert ver.tgt_sum.isnan().tolist() == [r == bad for r in range(2 * B)] and ver.tgt_lse.isnan().tolist() == ver.tgt_sum.isnan().tolist()
    assert ps.row_stats(z, V, 1.0)[1].isnan().tolist() == [r == bad for r in range(2 * B)]
    # one workgroup per row, without and with the table of its own layout
    out, p = ps.alloc_verified(B, B, gpu), lambda t: t.data_ptr()
    ps._check(ps.lib.picospec_verify(p(z), ps._dtype_code(z), z.stride(0), V, 1.0, B, B, p(off), p(tok), p(q.idx), p(q.prob), p(q.count), p(q.mass), 8, 1,
                                     None, p(u), p(out.n_accept), p(out.p_tok), p(out.q_tok), p(out.tgt_max), p(out.tgt_sum), p(out.tgt_lse),
                                     p(out.flags), None, 0, torch.cuda.current_stream().cuda_stream))
    many = z.repeat(40, 1) if z.stride(0) == V else torch.cat([base] * 40)[:, :V]       # (240 rows: more than are spread)
    off40 = torch.arange(40 * B + 1, dtype=torch.int32, device=gpu)
    tab = ps.verify(many, V, 1.0, off40, 40 * B, tok.repeat(40), None, u.repeat(40), q_scalar=u.repeat(40)[:40 * B].contiguous(),
                    workspace=ps.alloc_workspace(dtype, 80 * B, V, gpu))
    torch.cuda.synchronize()
    assert [bool(f & ps.FLAG_NONFINITE) for f in out.flags.tolist()] == [False, True, False], out.flags
    assert [bool(f & ps.FLAG_NONFINITE) for f in tab.flags.tolist()] == [False, True, False] * 40, tab.flags


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("others", ["masked", "nan"])
def test_nan_in_a_share_without_a_finite_value_reaches_the_record(gpu, ps, dtype, others):
    """The blocks of one workgroup's share of a row (every P-th kilobyte) hold a NaN and nothing above -inf: the row's sum is NaN as
    with one workgroup per row."""
    _announce("NaN in a share without a finite value", dtype, others)
    P, blk, k = 5, 256 if dtype == torch.float32 else 512, 24
    V = 8192 * P - 8                             # (a row is split as if it spanned a vector more)
    z = torch.randn((3, V), device=gpu)
    share = (torch.arange(V, device=gpu) // blk) % P == 3
    z[1, share] = float("-inf") if others == "masked" else float("nan")
    z[1, 3 * blk + 100] = float("nan")
    z = z.to(dtype)
    g, u = ps.compress(z, V, 1.0, k), _unsplit(ps, z, V, 1.0, k)
    torch.cuda.synchronize()
    assert g.lse.isnan().tolist() == u.lse.isnan().tolist() == [False, True, False]
    assert g.mass.isnan().tolist() == u.mass.isnan().tolist()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("k,share", [(10, 0.9), (1024, 0.5), (1024, 0.9)])
@pytest.mark.parametrize("mask", ["lowest", "-1e9"])
def test_masks_of_a_finite_value_are_compressed_once(gpu, ps, dtype, mask, k, share):
    """Rows masked by the type's lowest value or by -1e9: every workgroup's list holds what it found, so no row is compressed a
    second time from the start (which costs more than one workgroup per row)."""
    _announce("split finite masks", dtype, mask, k, share)
    V, R = 32000, 3
    g = torch.Generator(device=gpu)
    g.manual_seed(k)
    z = torch.randn((R, V), device=gpu, generator=g) * 3
    hidden = torch.rand((R, V), device=gpu, generator=g) < share
    z[hidden] = {"lowest": torch.finfo(dtype).min, "-1e9": -1e9}[mask]
    z = z.to(dtype)
    n = ps.workspace_bytes(ps.CALL_COMPRESS, ps._dtype_code(z), R, V, k)
    ws = torch.zeros(n, dtype=torch.uint8, device=gpu)
    out = ps.alloc_compressed(R, k, gpu)
    p = lambda t: t.data_ptr()
    ps._check(ps.lib.picospec_compress(p(z), ps._dtype_code(z), V, R, V, 1.0, k, 0.0, p(out.idx), p(out.prob), p(out.count), p(out.mass),
                                       p(out.lse), p(ws), n, torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    u = _unsplit(ps, z, V, 1.0, k)
    assert torch.equal(out.idx, u.idx) and torch.allclose(out.prob, u.prob, rtol=1e-6, atol=1e-38)
    # the scratch begins with a 32-byte head per share (its fourth word the entries found), lists of `cap` pairs follow
    vecs = (V * z.element_size() + 15) // 16 + 1
    parts = -(-(-(-vecs // 64)) // (8192 * z.element_size() // 1024))
    cap = (n // (R * parts) - 32) // 8
    found = ws.view(torch.int32)[:R * parts * 8].view(R * parts, 8)[:, 3]
    assert cap > 8 and int(found.max()) <= cap and int(found.view(R, parts).sum(1).min()) >= k, (cap, found)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V,R,T", [(16384, 4, 1.0), (33001, 224, 0.7), (64000, 64, 1.0), (128256, 128, 0.05), ((1 << 20) - 5, 2, 1.0)])
def test_target_statistics_in_a_given_workspace(gpu, pu, ps, dtype, V, R, T):
    """The statistics from the split table wherever a verification is given one, whole segments masked among them, against 64 bits;
    and row_stats of the same rows, which takes the table or one workgroup per row by its own rule."""
    _announce("split statistics in a given workspace", dtype, V, R, T)
    g = torch.Generator(device=gpu)
    g.manual_seed(V)
    z = (torch.randn((R, V + 3), device=gpu, generator=g) * 4).to(dtype)[:, 1:V + 1]
    z[0, : V // 2] = torch.finfo(dtype).min
    z[1, V // 2:] = float("-inf")
    off = torch.tensor([0, R - 1], dtype=torch.int32, device=gpu)
    tok, u = torch.zeros(R - 1, dtype=torch.int32, device=gpu), torch.rand(R, device=gpu, generator=g)
    ver = ps.verify(z, V, T, off, R - 1, tok, None, u, q_scalar=torch.rand(R - 1, device=gpu, generator=g), workspace=ps.alloc_workspace(dtype, R, V, gpu))
    x = z.double().cpu()
    m = x.max(1).values
    s = torch.exp((x - m[:, None]) / T).sum(1)
    for mx, sm, lse in ((ver.tgt_max, ver.tgt_sum, ver.tgt_lse), ps.row_stats(z, V, T)):
        assert torch.equal(mx.double().cpu(), m)
        pu.assert_close(pu.n(sm), s.numpy(), pu.RTOL, "sum")
        pu.assert_close(pu.n(lse), (m / T + torch.log(s)).numpy(), pu.RTOL_LSE, "lse", atol=2e-6)


def test_rows_in_front_of_the_first_sequence_keep_their_statistics(gpu, ps):
    """seq_off may start above 0: all n_draft + B rows get statistics, as with one workgroup per row."""
    _announce("split statistics in front of the first sequence")
    V, B, N = 20000, 2, 7
    tgt = torch.randn((N + B, V), device=gpu)
    off = torch.tensor([3, 4, 6], dtype=torch.int32, device=gpu)
    tok, u = torch.zeros(N, dtype=torch.int32, device=gpu), torch.rand(N + B, device=gpu)
    q = ps.compress(torch.randn((N, V), device=gpu), V, 1.0, 8)
    for v in (ps.verify(tgt, V, 1.0, off, N, tok, None, u, q_scalar=torch.rand(N, device=gpu)), ps.verify_sample(tgt, V, 1.0, off, N, tok, q, u)[0]):
        assert torch.equal(v.tgt_max, tgt.max(1).values)
        assert torch.allclose(v.tgt_lse, torch.logsumexp(tgt, 1), rtol=1e-5)
        assert not (v.flags & (ps.FLAG_BAD_INPUT | ps.FLAG_NONFINITE)).any()


def test_offsets_beyond_the_rows_write_nothing_behind_them(gpu, ps):
    """A negative gamma_b is flagged; the sequence it belongs to may start behind the call's rows, and what is behind those rows'
    entries of the outputs stays as it was."""
    _announce("split statistics, offsets beyond the rows")
    V, B, N, room = 20000, 3, 3, 12
    tgt = torch.randn((room, V), device=gpu)                      # (rows behind the call's six exist: nothing is read out of range)
    off = torch.tensor([0, 5, 2, 3], dtype=torch.int32, device=gpu)
    tok, u, qs = torch.zeros(room, dtype=torch.int32, device=gpu), torch.rand(room, device=gpu), torch.rand(room, device=gpu)
    out = ps.alloc_verified(B, room, gpu)
    for t in (out.tgt_max, out.tgt_sum, out.tgt_lse):
        t.fill_(-7.0)
    ps.verify(tgt, V, 1.0, off, N, tok, None, u, q_scalar=qs, out=out)
    torch.cuda.synchronize()
    for t in (out.tgt_max, out.tgt_sum, out.tgt_lse):
        assert (t[:N + B] != -7.0).all() and (t[N + B:] == -7.0).all()
    assert int(out.flags[1]) & ps.FLAG_BAD_INPUT


def test_a_round_takes_its_scratch_from_a_workspace_that_holds_it(gpu, ps):
    """A caller that sizes the workspace for the round allocates once: the round spreads its rows in it and allocates nothing; what it
    gives is what it gives without one."""
    _announce("round in the caller's workspace")
    V, k, B, N, T = 32000, 64, 2, 8, 0.8
    g = torch.Generator(device=gpu)
    g.manual_seed(5)
    tgt = torch.randn((N + B, V), device=gpu, generator=g) * 2
    draft = torch.randn((N, V), device=gpu, generator=g) * 2
    off = torch.tensor([0, 4, 8], dtype=torch.int32, device=gpu)
    u = torch.rand(N + B, device=gpu, generator=g)
    tok = ps.compress(draft, V, T, k).idx[:, 0].contiguous()
    ws = ps.alloc_workspace(torch.float32, N + B, V, gpu, ps.CALL_ROUND, k=k, n_draft=N)
    assert ws.numel() > ps.alloc_workspace(torch.float32, N + B, V, gpu, ps.CALL_ROUND).numel()
    want = ps.round(draft, tgt, V, T, off, N, tok, k, u)
    out = dict(q=ps.alloc_compressed(N, k, gpu), ver=ps.alloc_verified(B, N, gpu), res=ps.alloc_residual(B, gpu))
    torch.cuda.synchronize()
    made = lambda: torch.cuda.memory_stats()["allocation.all.allocated"]
    before = made()
    ps.round(draft, tgt, V, T, off, N, tok, k, u, workspace=ws, **out)
    assert made() == before
    for a, b in zip(want, (out["q"], out["ver"], out["res"])):
        for name, x in vars(a).items():
            assert not torch.is_tensor(x) or torch.equal(x, getattr(b, name)), name


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_a_round_that_spreads_nothing_takes_its_table_from_a_workspace_that_holds_it(gpu, ps, dtype):
    """What the call asks for is what it uses: a workspace that holds the table will do, and nothing is allocated beside it."""
    _announce("round in the table alone", dtype)
    V, k, B, N, T = 40000, 64, 4, 192, 0.8
    assert ps.scratch_bytes(ps.CALL_ROUND, ps.F32 if dtype == torch.float32 else ps.BF16, N, B, V, k) == 0
    g = torch.Generator(device=gpu)
    g.manual_seed(5)
    tgt = (torch.randn((N + B, V), device=gpu, generator=g) * 2).to(dtype)
    draft = (torch.randn((N, V), device=gpu, generator=g) * 2).to(dtype)
    off = torch.tensor([0, 48, 96, 144, 192], dtype=torch.int32, device=gpu)
    u = torch.rand(N + B, device=gpu, generator=g)
    ws = ps.alloc_workspace(dtype, N + B, V, gpu, ps.CALL_ROUND, k=k, n_draft=N)
    assert ws.numel() == ps.alloc_workspace(dtype, N + B, V, gpu, ps.CALL_ROUND).numel()
    with_scratch = torch.empty(ws.numel() + 16 + ps.workspace_bytes(ps.CALL_COMPRESS, ps._dtype_code(tgt), N, V, k), dtype=torch.uint8, device=gpu)
    tok = draft.float().argmax(1).to(torch.int32)
    outs = []
    for w in (ws, with_scratch):
        out = dict(q=ps.alloc_compressed(N, k, gpu), ver=ps.alloc_verified(B, N, gpu), res=ps.alloc_residual(B, gpu))
        torch.cuda.synchronize()
        before = torch.cuda.memory_stats()["allocation.all.allocated"]
        ps.round(draft, tgt, V, T, off, N, tok, k, u, workspace=w, **out)
        assert torch.cuda.memory_stats()["allocation.all.allocated"] == before
        outs.append(out)
    torch.cuda.synchronize()
    for key in outs[0]:
        for name, x in vars(outs[0][key]).items():
            assert not torch.is_tensor(x) or torch.equal(x, getattr(outs[1][key], name)), name


@pytest.mark.parametrize("dtype,N,B,V,k", [(torch.bfloat16, 160, 80, 98304, 40), (torch.bfloat16, 159, 80, 98303, 40),  # one launch for both streams
                                           (torch.bfloat16, 96, 64, 32768, 256), (torch.bfloat16, 97, 63, 32768, 256),  # its line, the rows that it
                                           (torch.bfloat16, 97, 63, 32767, 256),                                       # serves, and one beside them
                                           (torch.bfloat16, 64, 32, 32768, 2048), (torch.bfloat16, 48, 32, 32768, 2049),
                                           (torch.float32, 160, 64, 20000, 256), (torch.float32, 160, 65, 20000, 256),
                                           (torch.float32, 24, 1, 16384, 64), (torch.float32, 25, 1, 16384, 64),         # drafts per sequence
                                           (torch.float32, 64, 450, 16384, 16), (torch.bfloat16, 16, 500, 16400, 300),   # large rounds
                                           (torch.float32, 112, 112, 16384, 700), (torch.float32, 113, 112, 16384, 700),  # 224 rows and more
                                           (torch.float32, 48, 4, 32768, 4096), (torch.float32, 49, 4, 32768, 4096)])
def test_rounds_on_either_side_of_the_rule(gpu, pu, ps, dtype, N, B, V, k):
    """Every schedule that a round's sizes can choose against the one without scratch: the same ids, sums to rounding, and the same
    decisions but where a uniform lies within that of a step."""
    _announce("rounds on either side of the rule", dtype, N, B, V, k)
    T, g = 0.9, torch.Generator(device=gpu)
    g.manual_seed(N + V)
    off_l = [N * b // B for b in range(B + 1)]
    at = torch.tensor([off_l[b] + b + i for b in range(B) for i in range(off_l[b + 1] - off_l[b])], device=gpu)
    tgt = (torch.randn((N + B, V), device=gpu, generator=g) * 2).to(dtype)
    draft = (tgt[at].float() + torch.randn((N, V), device=gpu, generator=g)).to(dtype)
    off = torch.tensor(off_l, dtype=torch.int32, device=gpu)
    u = torch.rand(N + B, device=gpu, generator=g)
    tok = ps.compress(draft, V, T, k).idx[:, 0].contiguous()
    q, v, r = ps.round(draft, tgt, V, T, off, N, tok, k, u)
    with pu.no_scratch():
        q0, v0, r0 = ps.round(draft, tgt, V, T, off, N, tok, k, u)
    torch.cuda.synchronize()
    assert torch.equal(q.idx, q0.idx) and torch.equal(q.count, q0.count) and torch.equal(v.tgt_max, v0.tgt_max)
    for a, b in ((q.prob, q0.prob), (q.mass, q0.mass), (v.p_tok, v0.p_tok), (v.q_tok, v0.q_tok), (v.tgt_sum, v0.tgt_sum), (v.tgt_lse, v0.tgt_lse)):
        assert torch.allclose(a, b, rtol=2e-6, atol=1e-37)
    assert torch.equal(v.flags, v0.flags) and torch.equal(r.flags, r0.flags)
    # (the first positions that differ: a uniform within the acceptance margin of p / q there)
    for b in torch.nonzero(v.n_accept != v0.n_accept)[:, 0].tolist():
        d, t = off_l[b] + int(min(v.n_accept[b], v0.n_accept[b])), off_l[b] + b + int(min(v.n_accept[b], v0.n_accept[b]))
        assert abs(float(u[t]) * float(v.q_tok[d]) / float(v.p_tok[d]) - 1) < pu.ACCEPT_MARGIN
    same = v.n_accept == v0.n_accept
    assert torch.allclose(r.resid_mass[same], r0.resid_mass[same], rtol=1e-5, atol=1e-6)
    # (tokens that differ: the uniform lies within the sums' rounding of both tokens' steps of the residual's cumulative sum)
    for b in torch.nonzero(same & (r.out_tok != r0.out_tok))[:, 0].tolist():
        j, n = int(v.n_accept[b]), off_l[b + 1] - off_l[b]
        res = torch.softmax(tgt[off_l[b] + b + j].double() / T, 0)
        if j < n:
            res[q.idx[off_l[b] + j].long()] -= q.prob[off_l[b] + j].double() / q.mass[off_l[b] + j].double()
        res = res.clamp_min(0)
        cum, at_u = res.cumsum(0), float(u[off_l[b] + b + n]) * float(res.sum())
        for x in (int(r.out_tok[b]), int(r0.out_tok[b])):
            assert float(cum[x]) > at_u - pu.CDF_MARGIN and (x == 0 or float(cum[x - 1]) < at_u + pu.CDF_MARGIN)
