"""GPU parity of picospec_round (the three calls of a round as one; two launches for small rounds, Section 3.3)
against the oracle and, bit for bit, against the separate calls."""
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


CASES = [("cfg1", {}, 0), ("cfg2", {}, 0), ("cfg3", {"B": 6}, 0), ("cfg3", {"B": 40}, 0), ("cfg5", {"B": 10}, 0),
         ("cfg5", {"B": 70, "V": 20011, "k": 512}, 1), ("cfg4", {"B": 3}, 0)]


@pytest.mark.parametrize("name,scale,rnd", CASES)
@pytest.mark.parametrize("renorm", [1, 0])
def test_round_call_matches_oracle_and_separate_calls(gpu, pu, ps, name, scale, rnd, renorm):
    _announce("picospec_round", name, scale, rnd, renorm)
    w = W.WORKLOADS[name].scaled(**scale) if scale else W.WORKLOADS[name]
    r = W.build_round(w, rnd)
    o = pu.oracle_round(r, renorm=renorm)
    sep = pu.gpu_round(r, o.tok, gpu, renorm=renorm)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(gpu)
    q, ver, res = ps.round(pu.to_device(r.draft_logits, gpu), pu.to_device(r.tgt_logits, gpu), w.V, w.T, d(r.seq_off),
                           r.N, d(o.tok), w.k, d(r.uniforms), top_p=w.top_p, renorm=renorm)
    torch.cuda.synchronize()
    one = pu.GpuRound(q, ver, res)
    pu.compare_round(one, o, r, max_excluded_frac=0.34)
    # the same call with the workspace (the draw works from the target rows' segment table), and the fused call on
    # the existing records, with and without it
    ws = ps.alloc_workspace(torch.float32 if w.dtype == "f32" else torch.bfloat16, r.N + r.B, w.V, gpu, ps.CALL_ROUND)
    q3, ver3, res3 = ps.round(pu.to_device(r.draft_logits, gpu), pu.to_device(r.tgt_logits, gpu), w.V, w.T, d(r.seq_off),
                              r.N, d(o.tok), w.k, d(r.uniforms), top_p=w.top_p, renorm=renorm, workspace=ws)
    torch.cuda.synchronize()
    pu.compare_round(pu.GpuRound(q3, ver3, res3), o, r, max_excluded_frac=0.34)
    for wsp in (None, ws):
        ver4, res4 = ps.verify_sample(pu.to_device(r.tgt_logits, gpu), w.V, w.T, d(r.seq_off), r.N, d(o.tok), sep.q, d(r.uniforms),
                                      renorm=renorm, workspace=wsp)
        torch.cuda.synchronize()
        pu.compare_round(pu.GpuRound(sep.q, ver4, res4), o, r, max_excluded_frac=0.34)
    # the same calls as a caller makes them that has no scratch: nothing at all, and the table only
    with pu.no_scratch():
        for wsp in (None, ws):
            bare = pu.GpuRound(*ps.round(pu.to_device(r.draft_logits, gpu), pu.to_device(r.tgt_logits, gpu), w.V, w.T, d(r.seq_off), r.N, d(o.tok), w.k,
                                         d(r.uniforms), top_p=w.top_p, renorm=renorm, workspace=wsp))
            ver5, res5 = ps.verify_sample(pu.to_device(r.tgt_logits, gpu), w.V, w.T, d(r.seq_off), r.N, d(o.tok), sep.q, d(r.uniforms),
                                          renorm=renorm, workspace=wsp)
            torch.cuda.synchronize()
            pu.compare_round(bare, o, r, max_excluded_frac=0.34)
            pu.compare_round(pu.GpuRound(sep.q, ver5, res5), o, r, max_excluded_frac=0.34)
    # the records come from the same code: bit for bit; the target statistics of the two-launch schedule are summed by
    # 512 threads instead of 1024, so everything behind them agrees to rounding and the decisions wherever the oracle
    # does not call them knife-edge
    for a, b in ((q.idx, sep.q.idx), (q.prob, sep.q.prob), (q.count, sep.q.count), (q.mass, sep.q.mass), (q.lse, sep.q.lse)):
        assert torch.equal(a, b)
    for a, b, what in ((ver.p_tok, sep.ver.p_tok, "p_tok"), (ver.q_tok, sep.ver.q_tok, "q_tok"), (ver.tgt_sum, sep.ver.tgt_sum, "tgt_sum"),
                       (ver.tgt_lse, sep.ver.tgt_lse, "tgt_lse")):
        pu.assert_close(pu.n(a), pu.n(b).astype(np.float64), 2e-6, what, atol=1e-37)
    assert torch.equal(ver.tgt_max, sep.ver.tgt_max) and torch.equal(ver.flags, sep.ver.flags)
    off = r.seq_off
    clear = np.array([o.ver.margin[off[b]:off[b + 1]].min(initial=np.inf) >= pu.ACCEPT_MARGIN for b in range(r.B)])
    assert np.array_equal(pu.n(ver.n_accept)[clear], pu.n(sep.ver.n_accept)[clear])
    same_row = pu.n(ver.n_accept) == pu.n(sep.ver.n_accept)
    pu.assert_close(pu.n(res.resid_mass)[same_row], pu.n(sep.res.resid_mass)[same_row].astype(np.float64), 1e-5, "resid_mass", atol=1e-30)
    sure = clear & same_row & (o.res.cdf_margin >= pu.CDF_MARGIN)
    assert np.array_equal(pu.n(res.out_tok)[sure], pu.n(sep.res.out_tok)[sure])


# (drafts and target rows take turns, two to one: one draft, an odd number of them, more targets than turns, drafts left over; the layouts
# of the statistics change at 1024 and 2048 target rows, the last of which bf16 rounds take in launches of their own)
@pytest.mark.parametrize("dtype,N,B,V,pad,k", [(torch.bfloat16, 1, 520, 32768, 0, 40), (torch.bfloat16, 301, 222, 33001, 3, 2048),
                                               (torch.bfloat16, 1001, 22, 32768, 0, 64), (torch.bfloat16, 1001, 23, 32768, 0, 64),
                                               (torch.bfloat16, 2000, 47, 32768, 0, 64), (torch.bfloat16, 2000, 48, 32768, 0, 64),
                                               (torch.float32, 1, 520, 16385, 0, 4), (torch.float32, 301, 222, 33001, 3, 4096),
                                               (torch.float32, 700, 2, 20000, 0, 1024),
                                               (torch.float32, 4300, 308, 16385, 0, 64), (torch.float32, 4300, 309, 16385, 0, 64)])     # the most rows, and one more
def test_both_streams_in_one_launch_match_the_separate_calls(gpu, pu, ps, dtype, N, B, V, pad, k):
    """Bit for bit, with rows among them that lose the first pass of the compression."""
    _announce("both streams in one launch", dtype, N, B, V, k)
    T, g = 0.9, torch.Generator(device=gpu)
    g.manual_seed(N + B)
    off_l = [N * b // B for b in range(B + 1)]
    at = torch.tensor([off_l[b] + b + i for b in range(B) for i in range(off_l[b + 1] - off_l[b])], device=gpu)
    tgt = (torch.randn((N + B, V + pad), device=gpu, generator=g) * 2).to(dtype)[:, :V]
    draft = (tgt[at].float() + torch.randn((N, V), device=gpu, generator=g)).to(dtype)
    draft[3::7] = 0.5
    draft[4::7, (V // 3):] = -20.0
    draft[5::7] = torch.linspace(-8, 8, V, device=gpu).to(dtype)
    off = torch.tensor(off_l, dtype=torch.int32, device=gpu)
    u = torch.rand(N + B, device=gpu, generator=g)
    tok = draft.float().argmax(1).to(torch.int32)
    ws = ps.alloc_workspace(dtype, N + B, V, gpu, ps.CALL_ROUND)
    with pu.no_scratch():
        q, v, r = ps.round(draft, tgt, V, T, off, N, tok, k, u, workspace=ws)
        q0 = ps.compress(draft, V, T, k)
        v0 = ps.verify(tgt, V, T, off, N, tok, q0, u, workspace=ws)
        r0 = ps.sample_residual(tgt, V, T, off, N, v0, q0, u, workspace=ws)
    torch.cuda.synchronize()
    for a, b in ((q, q0), (v, v0), (r, r0)):
        for name, x in vars(a).items():
            assert not torch.is_tensor(x) or torch.equal(x, getattr(b, name)), name


# (up to 512 rows in all: statistics in a layout of their own, by workgroups of 512 threads; drafts first up to the number of CUs, in turns beyond)
@pytest.mark.parametrize("dtype,N,B,V,pad,k", [(torch.bfloat16, 1, 1, 32768, 0, 1), (torch.bfloat16, 200, 100, 33001, 3, 2048), (torch.bfloat16, 256, 0, 64000, 0, 777),
                                               (torch.float32, 1, 1, 8185, 0, 4), (torch.float32, 200, 100, 33001, 3, 4096), (torch.float32, 253, 3, 100000, 1, 64)])
def test_both_streams_of_a_small_round_in_one_launch(gpu, pu, ps, dtype, N, B, V, pad, k):
    """Records bit for bit those of the call of its own, statistics to rounding, with rows among them that lose the first pass; the segment sums
    of every target row add up to its sum."""
    B = B or N
    _announce("both streams of a small round", dtype, N, B, V, k)
    T, g = 0.9, torch.Generator(device=gpu)
    g.manual_seed(N + B)
    off_l = [N * b // B for b in range(B + 1)]
    tgt = (torch.randn((N + B, V + pad), device=gpu, generator=g) * 2).to(dtype)[:, :V]
    draft = (torch.randn((N, V + pad), device=gpu, generator=g) * 2).to(dtype)[:, :V]
    draft[3::7] = 0.5
    draft[5::7] = torch.linspace(-8, 8, V, device=gpu).to(dtype)
    off = torch.tensor(off_l, dtype=torch.int32, device=gpu)
    u = torch.rand(N + B, device=gpu, generator=g)
    tok = draft.float().argmax(1).to(torch.int32)
    ws = ps.alloc_workspace(dtype, N + B, V, gpu, ps.CALL_ROUND)
    with pu.no_scratch():
        q, v, r = ps.round(draft, tgt, V, T, off, N, tok, k, u, workspace=ws)
        q0 = ps.compress(draft, V, T, k)
        v0 = ps.verify(tgt, V, T, off, N, tok, q0, u)
    torch.cuda.synchronize()
    for name, x in vars(q).items():
        assert not torch.is_tensor(x) or torch.equal(x, getattr(q0, name)), name
    exact = torch.logsumexp(tgt.double() / T, 1)
    assert torch.equal(v.tgt_max, v0.tgt_max) and torch.allclose(v.tgt_lse.double(), exact, rtol=0, atol=2e-6)
    assert torch.allclose(v.tgt_sum.double(), torch.exp(exact - v.tgt_max.double() / T), rtol=2e-6)
    magic, seg_vecs, stride, rows = ws[:16].view(torch.int32).tolist()
    n_vec = 16 // tgt.element_size()
    assert rows == N + B and stride >= -(-V // (seg_vecs * n_vec))
    table = ws[16:16 + rows * stride * 8].view(torch.float32).view(rows, stride, 2)
    first = (tgt.data_ptr() // tgt.element_size() + torch.arange(rows, device=gpu) * tgt.stride(0)) % n_vec     # elements in front of a row's first vector
    n_seg = (first + V + seg_vecs * n_vec - 1) // (seg_vecs * n_vec)
    used = torch.arange(stride, device=gpu)[None, :] < n_seg[:, None]
    total = torch.where(used & (table[:, :, 0] > 0), table[:, :, 0].double() * torch.exp2(table[:, :, 1].double()), torch.zeros((), dtype=torch.float64, device=gpu)).sum(1)
    assert torch.allclose(torch.log(total), exact, rtol=0, atol=2e-6)
    assert torch.equal(v.flags, v0.flags)


def test_round_call_empty_and_misuse(gpu, ps):
    _announce("picospec_round empty")
    V = 64
    z = torch.zeros((0, V), device=gpu)
    off = torch.zeros(1, dtype=torch.int32, device=gpu)
    q, ver, res = ps.round(z, z, V, 1.0, off, 0, torch.zeros(0, dtype=torch.int32, device=gpu), 8, torch.zeros(0, device=gpu))
    torch.cuda.synchronize()
    assert q.idx.shape == (0, 8) and ver.n_accept.numel() == 0 and res.out_tok.numel() == 0
    # a sequence without draft positions: only its bonus token
    tgt = torch.randn((1, V), device=gpu)
    off = torch.tensor([0, 0], dtype=torch.int32, device=gpu)
    q, ver, res = ps.round(z, tgt, V, 1.0, off, 0, torch.zeros(0, dtype=torch.int32, device=gpu), 8, torch.full((1,), 0.5, device=gpu))
    torch.cuda.synchronize()
    assert int(ver.n_accept.item()) == 0 and 0 <= int(res.out_tok.item()) < V
    with pytest.raises(ps.PicoSpecError):
        ps.round(z, tgt, V, 1.0, off, 0, torch.zeros(0, dtype=torch.int32, device=gpu), 0, torch.full((1,), 0.5, device=gpu))
    with pytest.raises(ps.PicoSpecError):
        ps.round(z, tgt.to(torch.bfloat16), V, 1.0, off, 0, torch.zeros(0, dtype=torch.int32, device=gpu), 8,
                 torch.full((1,), 0.5, device=gpu), renorm=3)
