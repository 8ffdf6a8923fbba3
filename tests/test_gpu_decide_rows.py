"""Acceptance and draw with one wave per position (records of up to 256 entries, drafts of up to 15 positions) against the general
kernel, which the same records with one more unused slot are given to: the same decisions, statistics and tokens."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ps():
    from paper_2603_19133_amd import binding
    return binding


def _case(seed, V, ld, k, gammas, dtype, kind, dev):
    rng = np.random.default_rng(seed)
    off = np.concatenate([[0], np.cumsum(gammas)]).astype(np.int32)
    N, B = int(off[-1]), len(gammas)
    z = (rng.standard_normal((N + B, V)) * 3).astype(np.float32)
    if kind == "masked":
        z = np.where(rng.random(z.shape) < 0.999, -np.inf, z)
        z[:, V // 2] = 1.0
    tgt = torch.zeros((N + B, ld), dtype=dtype, device=dev)[:, :V]
    tgt.copy_(torch.from_numpy(z))
    rows = np.array([off[b] + b + i for b in range(B) for i in range(gammas[b])], dtype=np.int64)
    d = tgt.float().cpu().numpy()[rows].astype(np.float64)
    if kind != "same":
        with np.errstate(invalid="ignore"):
            d = d + rng.standard_normal(d.shape)
    if kind == "nan":
        tgt[1, 5] = float("nan")
        tgt[3, :] = float("-inf")
    idx = np.argsort(-d, axis=1, kind="stable")[:, :k]
    top = np.take_along_axis(d, idx, 1)
    p = np.exp(top - d.max(1, keepdims=True)) / np.exp(d - d.max(1, keepdims=True)).sum(1, keepdims=True) if N else np.zeros((0, k))
    count = rng.integers(max(1, k // 2), k + 1, N).astype(np.int32)
    tok = np.array([idx[i, rng.integers(0, min(3, count[i]))] for i in range(N)], dtype=np.int32)
    if N > 4 and kind == "outside":
        tok[0], tok[1], tok[3] = V, -1, int(np.setdiff1d(np.arange(V), idx[3])[0])
        count[2] = 0
    mass = np.where(np.arange(k)[None] < count[:, None], p, 0).sum(1)
    t = lambda a, dt=np.float32: torch.from_numpy(np.ascontiguousarray(a, dtype=dt)).to(dev)
    return dict(tgt=tgt, off=t(off, np.int32), N=N, B=B, idx=idx, p=p, count=t(count, np.int32), mass=t(mass), tok=t(tok, np.int32), uni=t(rng.random(N + B)))


def _run(ps, c, V, k, width, renorm, n_draft=None):
    dev = c["tgt"].device
    n_draft = c["N"] if n_draft is None else n_draft
    q = ps.alloc_compressed(max(n_draft, 1), width, dev)
    q.idx.fill_(-1); q.prob.zero_(); q.count.zero_(); q.mass.fill_(1.0)
    q.idx[:c["N"], :k] = torch.from_numpy(c["idx"].astype(np.int32)).to(dev)
    q.prob[:c["N"], :k] = torch.from_numpy(c["p"].astype(np.float32)).to(dev)
    q.count[:c["N"]] = c["count"]
    q.mass[:c["N"]] = c["mass"]
    extra = n_draft - c["N"]
    tgt = torch.cat([c["tgt"], c["tgt"][:extra]]) if extra else c["tgt"]
    uni = torch.cat([c["uni"], c["uni"][:extra]]) if extra else c["uni"]
    tok = torch.cat([c["tok"], c["tok"].new_zeros(extra)]) if extra else c["tok"]
    ver, res = ps.alloc_verified(c["B"], n_draft, dev), ps.alloc_residual(c["B"], dev)
    for t in (ver.p_tok, ver.q_tok, ver.tgt_max, ver.tgt_sum, ver.tgt_lse):
        t.fill_(-7.0)
    ws = ps.alloc_workspace(tgt.dtype, n_draft + c["B"], V, dev, ps.CALL_VERIFY_SAMPLE)
    ps.verify_sample(tgt, V, 0.8, c["off"], n_draft, tok, q, uni, renorm=renorm, ver=ver, res=res, workspace=ws)
    torch.cuda.synchronize()
    return {k2: v.cpu().numpy() for o in (ver, res) for k2, v in vars(o).items() if isinstance(v, torch.Tensor)} | {"rflags": res.flags.cpu().numpy(), "vflags": ver.flags.cpu().numpy()}


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V,ld,k,gammas,kind", [
    (16384, 16384, 1, [1, 4], "normal"), (16385, 16387, 63, [0, 15, 16, 3, 1], "normal"), (33001, 33003, 64, [15, 2], "outside"),
    (33001, 33001, 65, [8, 0, 0, 5], "masked"), (40000, 40000, 256, [15, 14, 1], "same"), (33001, 33002, 200, [3, 3, 4], "nan"),
    (327679, 327679, 100, [2, 1], "normal"), (327681, 327681, 100, [2, 1], "normal"), (16384, 16384, 10, [0, 0], "normal")])
@pytest.mark.parametrize("renorm", [0, 1])
def test_one_wave_per_position_matches_the_general_kernel(gpu, ps, V, ld, k, gammas, kind, dtype, renorm):
    print("[case]", V, ld, k, gammas, kind, dtype, renorm, flush=True)
    c = _case(V + k, V, ld, k, gammas, dtype, kind, torch.device("cuda"))
    for n_draft in (c["N"], c["N"] + 2):                   # (rows behind the last sequence: the general code takes its workgroup)
        got, want = _run(ps, c, V, k, k, renorm, n_draft), _run(ps, c, V, k, 257, renorm, n_draft)
        for name, w in want.items():
            # (fp64 sums of up to 320 segments in another order, rounded to fp32 once: one unit in the last place)
            if name == "resid_mass":
                np.testing.assert_allclose(got[name], w, rtol=1.2e-7, err_msg=name)
            else:
                np.testing.assert_array_equal(got[name], w, err_msg=name)


def _uncleared(V, ld, N, gammas):
    """Sequences whose row at position 1 has a segment more than the row of the wave that would clear it by its own row's count."""
    segs = lambda r: -(-(-(-((r * ld) % N + V) // N)) // 256)
    first = np.concatenate([[0], np.cumsum(gammas)])
    return [b for b, g in enumerate(gammas)
            if segs(first[b] + b + 1) > segs(first[b] + b + min((segs(first[b] + b + 1) - 1) // 64, g))]


@pytest.mark.parametrize("dtype,V,ld", [(torch.float32, 32768, 32769), (torch.float32, 32767, 32767), (torch.bfloat16, 65535, 65535)])
def test_the_drawn_row_may_have_a_segment_more(gpu, ps, dtype, V, ld):
    """Rows at other offsets of a 16-byte block can be a segment longer than the sequence's first row: most of the target's mass on the last
    ids, the first position accepted, the second rejected, LDS that holds what another kernel left there."""
    print("[case]", V, ld, dtype, flush=True)
    dev, k, gammas = torch.device("cuda"), 64, [3] * 24
    assert len(_uncleared(V, ld, 4 if dtype == torch.float32 else 8, gammas)) >= 4
    c = _case(V, V, ld, k, gammas, dtype, "normal", dev)
    c["tgt"][:, V - 2:] += 30.0
    c["uni"].fill_(0.5)
    for b in range(len(gammas)):
        c["uni"][4 * b] = 0.0
        c["uni"][4 * b + 1:4 * b + 3] = 0.9999
    dirty = torch.randn((1024, 40000), device=dev)
    ps.compress(dirty, 40000, 1.0, 2048)                   # (every CU, 73 KB of LDS each)
    got = _run(ps, c, V, k, k, 1)
    want = _run(ps, c, V, k, 257, 1)
    assert (want["n_accept"] == 1).mean() > 0.9 and (want["out_tok"] >= V - 2).mean() > 0.9
    for name, w in want.items():
        if name == "resid_mass":
            np.testing.assert_allclose(got[name], w, rtol=1.2e-7, err_msg=name)
        else:
            np.testing.assert_array_equal(got[name], w, err_msg=name)
