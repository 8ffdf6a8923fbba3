"""Calls whose last workgroup goes on (verification, the draw without a table, row statistics in one launch) against the same calls in two, which
a workspace that holds the table alone takes: the same bits.  Scratch that holds anything, offsets of every kind, repeated use and
captured launches.  (The verification is compared with one workgroup per row as well, the statistics with 64 bits.)"""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ps():
    from paper_2603_19133_amd import binding
    return binding


NV, WORD, FRONT = 4, 256, 4


def _segments(dtype, V):
    n = 8 if dtype == torch.bfloat16 else 4
    return ((V * (16 // n) + 15) // 16 + 1 + 64 * NV - 1) // (64 * NV)


def _table_bytes(ps, dtype, rows, V):
    """What picospec_workspace_bytes asks for: two launches (test_boundary_cpu.py holds that it is less than one launch needs)."""
    return ps.workspace_bytes(ps.CALL_VERIFY, ps.BF16 if dtype == torch.bfloat16 else ps.F32, rows, V, 0)


def _scratch_bytes(ps, dtype, rows, groups, V):
    return (max(16 + rows * 8 * _segments(dtype, V), _table_bytes(ps, dtype, rows, V)) + 15) // 16 * 16 + groups * WORD


class _Case:
    def __init__(self, ps, seed, dtype, V, ld, gammas, k, extra=0, off=None):
        self.ps, self.dtype, self.V, self.k = ps, dtype, V, k
        dev = torch.device("cuda")
        g = torch.Generator(device=dev); g.manual_seed(seed)
        self.B = len(gammas)
        self.off = torch.tensor(np.concatenate([[0], np.cumsum(gammas)]) if off is None else off, dtype=torch.int32, device=dev)
        self.N = int(sum(gammas)) + extra
        self.rows = self.N + self.B
        room = self.rows + 8                          # (offsets that leave the call's rows stay inside the tensors)
        self.z = torch.zeros((room, ld), dtype=dtype, device=dev)[:, :V]
        self.z.copy_(torch.randn((room, V), device=dev, generator=g) * 3)
        self.uni = torch.rand(room, device=dev, generator=g)
        self.q = ps.compress(self.z, V, 1.0, k)
        pick = torch.randint(0, min(3, k), (room,), device=dev, generator=g)
        self.tok = self.q.idx.gather(1, pick.unsqueeze(1).long())[:, 0].contiguous()
        self.scalar = torch.rand(room, device=dev, generator=g)
        behind = lambda t: torch.cat([t[:FRONT], t])[FRONT:]      # (room in front of what is read by draft row)
        self.q = ps.Compressed(*[behind(t) for t in (self.q.idx, self.q.prob, self.q.count, self.q.mass, self.q.lse)], k)
        self.tok, self.scalar = behind(self.tok), behind(self.scalar)
        self.code = ps._dtype_code(self.z)

    def fresh(self):
        ver, res = self.ps.alloc_verified(self.B, self.N + 8, self.z.device), self.ps.alloc_residual(self.B, self.z.device)
        self.fronts = [torch.empty(FRONT + self.N + 8, device=self.z.device) for _ in range(2)]
        ver.p_tok, ver.q_tok = [t[FRONT:] for t in self.fronts]
        for t in list(vars(ver).values()) + list(vars(res).values()) + self.fronts:
            t.fill_(-7)
        return ver, res

    def verify(self, ws, ver, q_scalar, ranged=None):
        q = self.q
        rec = ps_none if q_scalar else (q.idx, q.prob, q.count, q.mass, q.k)
        outs = (ver.n_accept, ver.p_tok, ver.q_tok, ver.tgt_max, ver.tgt_sum, ver.tgt_lse, ver.flags, ws, self.ps._stream())
        head = (self.z, self.code, self.z.stride(0), self.V, 0.9, self.B, self.N, self.off, self.tok, *rec, 1, self.scalar if q_scalar else None, self.uni)
        if ranged is None:
            self.ps._check(self.ps._nat.verify(*head, *outs))
        else:
            self.ps._check(self.ps._nat.verify_range(*head, *ranged, *outs))


ps_none = (None, None, None, None, 0)


def _same(a, b):
    for name, x in vars(a).items():
        np.testing.assert_array_equal(x.cpu().numpy(), vars(b)[name].cpu().numpy(), err_msg=name)


CASES = [(16384, 16384, [1], 64, 0, None), (20000, 20003, [0, 3, 15, 0, 16], 70, 0, None), (33001, 33001, [4] * 9, 257, 3, None),
         (40000, 40001, [2, 2, 2], 10, 2, [2, 4, 6, 8]),          # rows in front of the first sequence
         (33000, 33000, [3, 3, 3], 10, 0, [0, 5, 3, 9]),          # offsets that descend
         (33000, 33000, [3, 3, 3], 10, 0, [0, 6, 2, 9]),          # ... so far that positions of two sequences share a target row
         (16384, 16387, [4] * 8, 64, 0, [0, 9, 1, 10, 2, 11, 3, 12, 32]),
         (33000, 33000, [3, 3, 3], 10, 0, [0, 3, 6, 12]),         # ... that leave the call's rows
         (33000, 33000, [3, 3, 3], 10, 0, [0, -1, 2, 9])]         # ... and whose drafts lie in front of the call's


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V,ld,gammas,k,extra,off", CASES)
@pytest.mark.parametrize("q_scalar", [False, True])
def test_verification(gpu, ps, dtype, V, ld, gammas, k, extra, off, q_scalar):
    print("[case]", V, gammas, k, extra, off, dtype, q_scalar, flush=True)
    c = _Case(ps, V + k, dtype, V, ld, gammas, k, extra, off)
    full = _scratch_bytes(ps, dtype, c.rows, c.B + 1, V) + c.rows * 24
    asked = ps.lib.picospec_one_launch_bytes(ps.CALL_VERIFY, c.code, c.N, c.B, V, 0)
    assert asked in (0, full)
    assert _table_bytes(ps, dtype, c.rows, V) < full
    garbage = torch.randint(0, 256, (full,), dtype=torch.uint8, device=c.z.device)
    table = garbage.clone()[:_table_bytes(ps, dtype, c.rows, V)]
    ranges = [None]
    if off is None or off[-1] <= c.N:
        g = (c.off[1:] - c.off[:-1]).clamp_min(0)
        top = int(g.max())
        ranges += [(None, None, top), ((g + 1) // 2, g, top), (torch.zeros_like(g), (g + 1) // 2, top), (g, g, top), (g + 5, g - 9, top)]
    for r in ranges:
        want, _ = c.fresh()
        c.verify(None, want, q_scalar, r)
        assert all(bool((t[:FRONT] == -7).all()) for t in c.fronts)
        two = None
        for fill in ("two launches", "random", "ones", "again"):
            if fill == "ones":
                garbage.fill_(255)
            got, _ = c.fresh()
            c.verify(table if fill == "two launches" else garbage, got, q_scalar, r)
            torch.cuda.synchronize()
            assert all(bool((t[:FRONT] == -7).all()) for t in c.fronts)
            if off is not None and min(off) < 0 and r is None:
                assert got.n_accept[1] == 0 and got.flags[1] & 8
            a, w = [{n: t.cpu().numpy() for n, t in vars(v).items()} for v in (got, want)]
            if off is not None and off[-1] > c.N:
                # rows behind the call's are neither read nor written here: flagged and rejected
                assert (a["p_tok"][c.N:] == -7).all() and (a["tgt_sum"][c.rows:] == -7).all()
                assert a["flags"][-1] & 8 and a["n_accept"][-1] <= 3
                continue
            two = two or a
            np.testing.assert_array_equal(a["n_accept"], w["n_accept"])
            np.testing.assert_array_equal(a["flags"], w["flags"])
            shared = off is not None and (np.diff(off) < 0).any()     # (positions of two sequences: whose p comes last is anyone's)
            if not shared:
                np.testing.assert_array_equal(a["q_tok"], w["q_tok"])
                np.testing.assert_array_equal(a["p_tok"], two["p_tok"])
            for name in ("tgt_max", "tgt_sum", "tgt_lse"):
                np.testing.assert_array_equal(a[name], two[name], err_msg=name)
            for name in ("tgt_max", "tgt_sum", "tgt_lse") + (() if shared else ("p_tok",)):
                # (two fp32 sums of up to 40,000 terms, by 1024 threads and by segments: a few 2^-24 each)
                np.testing.assert_allclose(a[name], w[name], rtol=2e-6, err_msg=name)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V,B,k", [(33001, 1, 1), (33001, 24, 70), (33003, 37, 600), (40000, 512, 600), (33000, 600, 513)])
def test_draw(gpu, ps, dtype, V, B, k):
    print("[case]", V, B, k, dtype, flush=True)
    c = _Case(ps, B + k, dtype, V, V + 3, [b % 3 for b in range(B)], k)
    ver, _ = c.fresh()
    mx, sm, lse = ps.row_stats(c.z, V, 0.9)
    g = c.off[1:] - c.off[:-1]
    n = torch.minimum(g, torch.arange(B, device=g.device, dtype=torch.int32) % 4 - 1)       # (-1: clamped and flagged)
    def draw(ws):
        _, res = c.fresh()
        ps._check(ps._nat.sample_residual_ws(c.z, c.code, c.z.stride(0), V, 0.9, B, c.N, c.off, n, mx, sm, c.q.idx, c.q.prob, c.q.count, c.q.mass, k, 1, c.uni,
                                             res.out_tok, res.resid_mass, res.flags, ws, ps._stream()))
        return res
    room = torch.randint(0, 256, (_scratch_bytes(ps, dtype, B, B, V),), dtype=torch.uint8, device=c.z.device)
    table = room.clone()[:_table_bytes(ps, dtype, B, V)]
    want = draw(table)
    for _ in range(3):
        _same(draw(room), want)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("off,n,outside", [([0, 3, 6, 12], [1, 3, 5], [2]),          # the drawn row lies behind the call's
                                           ([0, 3, 6, 12], [1, 3, 3], [2]),          # ... its draft's record alone
                                           ([0, 3, 12, 9], [3, 7, 0], [1, 2]),       # offsets that descend
                                           ([0, -1, 2, 9], [0, 0, 2], [1]),          # a record in front of the call's
                                           ([-2, -1, 2, 9], [0, 0, 2], [0, 1])])
def test_a_draw_that_leaves_the_call(gpu, ps, dtype, off, n, outside):
    """The drawn row or the record lies outside the call's (inside the tensors, which are larger): token 0, flagged, in one launch, in two and from a
    verification's table; the other sequences draw as ever."""
    V, k, front = 33001, 64, 8
    print("[case]", off, n, dtype, flush=True)
    c = _Case(ps, 5, dtype, V, V + 1, [3, 3, 3], k)
    mx, sm, _ = ps.row_stats(c.z, V, 0.9)
    # (everything once more with room in front of it)
    z = torch.cat([c.z[:front], c.z])
    pad = lambda t: torch.cat([t[:front], t])[front:]
    z, mx, sm, uni, idx, prob, count, mass = z[front:], *[pad(t) for t in (mx, sm, c.uni, c.q.idx, c.q.prob, c.q.count, c.q.mass)]
    seq, na = torch.tensor(off, dtype=torch.int32, device=z.device), torch.tensor(n, dtype=torch.int32, device=z.device)
    def draw(ws, call, seq=seq, na=na):
        _, res = c.fresh()
        ps._check(call(z, c.code, z.stride(0), V, 0.9, c.B, c.N, seq, na, mx, sm, idx, prob, count, mass, k, 1, uni,
                       res.out_tok, res.resid_mass, res.flags, ws, ps._stream()))
        return [t.cpu().numpy() for t in vars(res).values()]
    room = torch.randint(0, 256, (_scratch_bytes(ps, dtype, c.B, c.B, V),), dtype=torch.uint8, device=z.device)
    one, two = draw(room, ps._nat.sample_residual_ws), draw(room[:_table_bytes(ps, dtype, c.B, V)], ps._nat.sample_residual_ws)
    ws = ps.alloc_workspace(dtype, c.rows, V, z.device)
    ver, _ = c.fresh()
    c.z = z
    c.verify(ws, ver, False)
    table = draw(ws, ps._nat.sample_residual)
    inside = [b for b in range(c.B) if b not in outside]
    for tok, resid, flags in (one, two, table):
        assert all(tok[b] == 0 and resid[b] == 0 and flags[b] & 8 for b in outside), (tok, resid, flags)
        assert all(0 < resid[b] <= 1.0 and 0 <= tok[b] < V and (flags[b] & 8 == 0 or off[b + 1] < off[b]) for b in inside), (tok, resid, flags)
        np.testing.assert_array_equal(tok, one[0])
        np.testing.assert_array_equal(flags, one[2])
        np.testing.assert_allclose(resid, one[1], rtol=1e-6)


@pytest.mark.parametrize("dtype,V,rows", [(torch.float32, 62500, 1), (torch.float32, 125003, 100), (torch.float32, 64000, 64), (torch.float32, 128256, 128),
                                          (torch.float32, 1048576, 2), (torch.bfloat16, 125001, 1), (torch.bfloat16, 128256, 160), (torch.bfloat16, 151937, 37),
                                          (torch.bfloat16, 1048576, 2)])
def test_row_statistics(gpu, ps, dtype, V, rows):
    print("[case]", V, rows, dtype, flush=True)
    z = (torch.randn((rows, V + 1), device="cuda") * 3).to(dtype)[:, :V]
    code, T = ps._dtype_code(z), 0.9
    one, two = ps.lib.picospec_one_launch_bytes(ps.CALL_ROW_STATS, code, rows, 0, V, 0), _table_bytes(ps, dtype, rows, V)
    assert one == _scratch_bytes(ps, dtype, rows, rows, V) > two > 0            # (spread, in one launch and in two)
    z[rows - 1, V // 2:] = float("-inf")
    def stats(ws):
        out = [torch.full((rows,), -7.0, device="cuda") for _ in range(3)]
        ps._check(ps._nat.row_stats(z, code, z.stride(0), rows, V, T, *out, ws, ps._stream()))
        return [o.cpu().numpy() for o in out]
    room = torch.randint(0, 256, (one,), dtype=torch.uint8, device="cuda")
    x = z.double() / T
    top, lse = x.max(1).values, torch.logsumexp(x, 1)
    # each term 2^e, e of up to 2^6 rounded to fp32, so 2^-18 ln 2 at most and 2^-22 for the terms that matter (e > -2^2); the log-sum-exp is rounded once
    exact = [z.float().max(1).values, torch.exp(lse - top), lse]
    for name, got, want, tol in zip("max sum lse".split(), stats(room), exact, (0.0, 2e-6, 3e-7)):
        np.testing.assert_allclose(got, want.double().cpu().numpy(), rtol=tol, err_msg=name)
    z[0, 7] = float("inf")
    want = stats(room.clone()[:two])
    for _ in range(3):
        for got, w in zip(stats(room), want):
            np.testing.assert_array_equal(got, w)


def test_captured_calls_replay(gpu, ps):
    c = _Case(ps, 3, torch.float32, 33001, 33001, [4, 0, 7, 2], 64)
    ver, res = c.fresh()
    ws = torch.empty(_scratch_bytes(ps, torch.float32, c.rows, c.B + 1, 33001) + c.rows * 24 + 65536, dtype=torch.uint8, device="cuda")
    ws2 = torch.empty(_scratch_bytes(ps, torch.float32, c.B, c.B, 33001) + 65536, dtype=torch.uint8, device="cuda")
    def both(v, r):
        c.verify(ws, v, False)
        ps._check(ps._nat.sample_residual_ws(c.z, c.code, c.z.stride(0), c.V, 0.9, c.B, c.N, c.off, v.n_accept, v.tgt_max, v.tgt_sum, c.q.idx, c.q.prob, c.q.count,
                                             c.q.mass, c.k, 1, c.uni, r.out_tok, r.resid_mass, r.flags, ws2, ps._stream()))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        both(ver, res)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        both(ver, res)
    for i in range(4):
        c.z.copy_(torch.randn_like(c.z) * (2 + i))
        want_v, want_r = c.fresh()
        both(want_v, want_r)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        _same(ver, want_v)
        _same(res, want_r)


def _kernels(graph):
    """Kernels of a captured graph (its only nodes)."""
    n = ctypes.c_size_t(0)
    assert ctypes.CDLL("libamdhip64.so").hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,V,launches", [(24, 33001, 1), (112, 64000, 2)])     # (up to 3300 segments of a range's rows, and beyond)
def test_a_captured_range_takes_the_launches_that_replay_faster(gpu, ps, dtype, rows, V, launches):
    V *= 1 if dtype == torch.float32 else 2
    c = _Case(ps, 4, dtype, V, V, [3] * (rows // 8), 64, extra=rows // 2)
    assert ps.lib.picospec_one_launch_bytes(ps.CALL_VERIFY, c.code, c.N, c.B, V, 0) > ps.scratch_bytes(ps.CALL_VERIFY, c.code, c.N, c.B, V, 0) or launches == 2
    ws = torch.empty(_scratch_bytes(ps, dtype, c.rows, c.B + 1, V) + c.rows * 24, dtype=torch.uint8, device="cuda")
    r = (None, None, 3)
    want, _ = c.fresh()
    c.verify(ws, want, False, r)
    ver, _ = c.fresh()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        c.verify(ws, ver, False, r)
    assert _kernels(graph) == launches
    graph.instantiate()
    for _ in range(3):
        ws.random_(0, 256)
        graph.replay()
        torch.cuda.synchronize()
        _same(ver, want)
