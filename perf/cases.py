"""The calls that a program built on this library makes, as cases with a time, a floor and an expected result.

Every case is one pass through the public calls (paper_2603_19133_amd.binding) on inputs that are already on the GPU and
into outputs that the program keeps, as a serving loop does it:

  draft   the drafter's step: compress the logits of one position of B sequences, draw a token from each record
          (gamma of these run one after the other in every round, so their latency counts most of all)
  round   picospec_round: compress, verify and draw in one call
  calls   the same round as three calls (compress, verify, sample_residual): what bench.py times
  verify  picospec_verify_sample: the cloud's part when the records arrive with the tokens
  cloud   the paper's own direction (Section 3.3): uplink message in, verification with the scalar q_i, Top-K record of
          the rejected target rows, downlink message out
  edge    the other end of it: uplink message out, dense draft statistics, downlink message in, local resampling
  pieces  a draft verified in two parts as its positions become known (Section 3.2), then the draw without a workspace

The listed sizes are the five workloads of workloads.py (cfg1 .. cfg5) and generic ones between them: the smallest calls (one
sequence), ordinary batches, calls that fill the chip; fp32 and bf16; plain Top-K and top-p; fixed and ragged draft
lengths; vocabularies and leading dimensions off every power of two and off the 16-byte boundary.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2603_19133_amd import binding as ps

_DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
_CHUNK = 1 << 26          # elements handled at a time by the torch code below


def _case(name, kind, B, gamma, V, dtype, T, k, recipe, top_p=0.0, pad=0, fmt=0):
    c = dict(kind=kind, B=B, gamma_lo=gamma[0], gamma_hi=gamma[1], V=V, dtype=dtype, T=T, k=k, recipe=recipe, top_p=top_p,
             pad=pad, fmt=fmt)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one user, one draft (cfg1): bound by launches and latency
        _case("round_b1", "round", 1, (4, 4), 32000, "f32", 1.0, 64, "normal3"),
        # a small batch (cfg2)
        _case("round_b8", "round", 8, (8, 8), 32000, "bf16", 1.0, 256, "mix4"),
        # an ordinary serving batch (cfg3)
        _case("round_b64", "round", 64, (8, 8), 128256, "bf16", 0.7, 1024, "zipf1.1"),
        # the largest configuration (cfg4): the chip is full many times over
        _case("calls_b256", "calls", 256, (16, 16), 151936, "f32", 1.0, 4096, "resample5"),
        # ragged drafts, nucleus records, bf16 (cfg5)
        _case("calls_b512_topp", "calls", 512, (1, 16), 152064, "bf16", 1.0, 2048, "zipf1.2", top_p=0.95),
        # one user's drafting step with the paper's record length K = 10
        _case("draft_b1", "draft", 1, (1, 1), 128256, "bf16", 0.7, 10, "zipf1.1"),
        # a serving batch's drafting step
        _case("draft_b64", "draft", 64, (1, 1), 151936, "f32", 1.0, 1024, "mix4"),
        # a large batch, odd vocabulary and leading dimension, nucleus records of odd length
        _case("draft_b300_odd", "draft", 300, (1, 1), 50001, "bf16", 0.9, 777, "zipf1.2", top_p=0.9, pad=2),
        # the cloud's part of a ragged batch, records at hand
        _case("verify_b16", "verify", 16, (1, 8), 151936, "f32", 0.8, 64, "normal3"),
        # the paper's direction at a serving batch: both ends of it
        _case("cloud_b32", "cloud", 32, (4, 6), 128256, "bf16", 1.0, 256, "zipf1.1", fmt=1),
        _case("edge_b32", "edge", 32, (4, 6), 128256, "bf16", 1.0, 256, "zipf1.1", fmt=1),
        # a draft verified in two parts, odd rows
        _case("pieces_b24", "pieces", 24, (2, 8), 33001, "f32", 0.8, 70, "normal3", pad=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_MOST = 256 * 33 * 151936 * 4          # row bytes of the largest listed case


def draw(rng: random.Random):
    kind = rng.choice(["draft", "draft", "round", "calls", "verify", "cloud", "edge", "pieces"])
    dtype = rng.choice(["f32", "bf16"])
    V = _log_int(rng, 32000, 152064)
    if rng.random() < 0.5:
        V &= ~7                                             # (most vocabularies are padded to a multiple of 8 or more)
    pad = 0 if rng.random() < 0.7 else rng.randint(1, 8)
    k = _log_int(rng, 10, 4096)
    if rng.random() < 0.5:
        k = max(8, k & ~3)
    top_p = rng.choice([0.0, 0.0, 0.9, 0.95]) if kind in ("draft", "round", "calls") else 0.0
    recipe = rng.choice(["normal3", "mix4", "resample5", "zipf1.1", "zipf1.2"])
    lo = rng.randint(1, 8)
    gamma = (lo, lo) if rng.random() < 0.4 else (lo, rng.randint(lo, 16))
    B = {"draft": lambda: _log_int(rng, 1, 1024), "round": lambda: _log_int(rng, 1, 128),
         "calls": lambda: _log_int(rng, 64, 512)}.get(kind, lambda: _log_int(rng, 1, 128))()
    if kind == "draft":
        gamma = (1, 1)
    esz = 4 if dtype == "f32" else 2
    while B > 1 and B * (2 * gamma[1] + 1) * (V + pad) * esz > _MOST:
        B //= 2
    return _case(None, kind, B, gamma, V, dtype, round(rng.uniform(0.6, 1.2), 2), k, recipe, top_p, pad,
                 rng.choice([0, 1, 2]) if kind in ("cloud", "edge") else 0)


# ---------------------------------------------------------------- inputs

def _gen(seed, what, device):
    g = torch.Generator(device=device)
    g.manual_seed((int(seed) * 16 + what) & 0x7FFFFFFFFFFF)
    return g


def _offsets(c):
    r = random.Random(17)                                   # (draft lengths belong to the case: they are its outputs' shapes)
    off = [0]
    for _ in range(c["B"]):
        off.append(off[-1] + r.randint(c["gamma_lo"], c["gamma_hi"]))
    return off


def _device():
    return torch.device("cuda")


def _logits(c, rows, seed, what, like=None):
    """[rows, V] logits (stride V + pad): like=None the target recipe, else the draft's, row by row from `like`."""
    dev, V, dt = _device(), c["V"], _DTYPES[c["dtype"]]
    g = _gen(seed, what, dev)
    out = torch.zeros((rows, V + c["pad"]), dtype=dt, device=dev)[:, :V]
    step = max(1, _CHUNK // V)
    for r0 in range(0, rows, step):
        n = min(step, rows - r0)
        z = torch.randn((n, V), device=dev, generator=g)
        rec = c["recipe"]
        if like is None:
            if rec.startswith("zipf"):
                s = float(rec[4:])
                rank = torch.floor(torch.rand((n, V), device=dev, generator=g) * V) + 1.0
                z = z * 0.5 - s * torch.log(rank)
            else:
                z = z * {"normal3": 3.0, "mix4": 4.0, "resample5": 5.0}[rec]
        else:
            t = like(r0, n)
            if rec == "mix4":
                z = 0.8 * t + 1.5 * z
            elif rec == "resample5":
                z = torch.where(torch.rand((n, V), device=dev, generator=g) < 0.1, z * 5.0, t)
            else:
                z = t + (1.2 if rec == "zipf1.2" else 1.0) * z
        out[r0:r0 + n] = z.to(dt)
    return out


def _draft_tokens(c, logits, seed):
    """One token per row from the row's record (its Top-K, cut to the top-p prefix), renormalised."""
    dev, rows = logits.device, logits.shape[0]
    g = _gen(seed, 9, dev)
    tok = torch.empty(rows, dtype=torch.int32, device=dev)
    k = min(c["k"], c["V"])
    step = max(1, _CHUNK // c["V"])
    for r0 in range(0, rows, step):
        z = logits[r0:r0 + step].float() / c["T"]
        top = torch.topk(z, k, dim=1, sorted=True).values
        if 0 < c["top_p"] < 1:
            p = torch.exp(top.double() - torch.logsumexp(z.double(), 1, keepdim=True))
            n_keep = ((torch.cumsum(p, 1) - p) < c["top_p"]).sum(1)
            edge = top.gather(1, (n_keep - 1).clamp(min=0).unsqueeze(1))
        else:
            edge = top[:, -1:]
        inside = (z > edge) | (z == top[:, :1])             # (strictly above the last entry: ties at the cut may be outside)
        u = torch.rand(z.shape, device=dev, generator=g).clamp_(1e-20, 1 - 1e-7)
        tok[r0:r0 + step] = torch.where(inside, z - torch.log(-torch.log(u)), -math.inf).argmax(1).to(torch.int32)
    return tok


def _records(c, logits):
    """Records of the rows in the library's layout: larger logit first, lower id first among equal ones."""
    rows, k = logits.shape[0], c["k"]
    q = ps.alloc_compressed(rows, k, logits.device)
    step = max(1, _CHUNK // c["V"])
    for r0 in range(0, rows, step):
        z = logits[r0:r0 + step].float()
        v, i = torch.sort(z, dim=1, descending=True, stable=True)
        zd = z.double() / c["T"]
        lse = torch.logsumexp(zd, 1)
        p = torch.exp(v[:, :k].double() / c["T"] - lse.unsqueeze(1)).float()
        q.idx[r0:r0 + step] = i[:, :k].to(torch.int32)
        q.prob[r0:r0 + step] = p
        q.count[r0:r0 + step] = k
        q.mass[r0:r0 + step] = p.double().sum(1).float()
        q.lse[r0:r0 + step] = lse.float()
    return q


def _take(q, rows):
    return ps.Compressed(q.idx[rows], q.prob[rows], q.count[rows], q.mass[rows], q.lse[rows], q.k)


class _State:
    pass


def _inputs(case, seed):
    """The tensors of the case that are made from the seed alone."""
    c, s, dev = case, _State(), _device()
    s.c, s.B, s.V, s.T, s.k = c, c["B"], c["V"], c["T"], c["k"]
    off = _offsets(c)
    s.off, s.N = off, off[-1]
    if c["kind"] == "draft":
        tgt = _logits(c, s.B, seed, 1)
        s.draft = _logits(c, s.B, seed, 2, like=lambda r0, n: tgt[r0:r0 + n].float())
        s.duni = torch.rand(s.B, device=dev, generator=_gen(seed, 4, dev))
        return s
    s.tgt = _logits(c, s.N + s.B, seed, 1)
    rows = torch.tensor([off[b] + b + i for b in range(s.B) for i in range(off[b + 1] - off[b])], device=dev)
    s.draft = _logits(c, s.N, seed, 2, like=lambda r0, n: s.tgt[rows[r0:r0 + n]].float())
    s.seq_off = torch.tensor(off, dtype=torch.int32, device=dev)
    s.uni = torch.rand(s.N + s.B, device=dev, generator=_gen(seed, 3, dev))
    s.tok = _draft_tokens(c, s.draft, seed)
    return s


def _scalars(s):
    """q_i of the drafted tokens (renormalised on the record), fp32."""
    z = s.draft.float()
    out = torch.empty(s.N, device=z.device)
    step = max(1, _CHUNK // s.V)
    for r0 in range(0, s.N, step):
        zz = z[r0:r0 + step].double() / s.T
        top = torch.topk(zz, min(s.k, s.V), dim=1).values
        x = zz.gather(1, s.tok[r0:r0 + step].long().unsqueeze(1))
        out[r0:r0 + step] = torch.exp(x[:, 0] - torch.logsumexp(top, 1)).float()
    return out


def prepare(case, seed):
    s, c, dev = _inputs(case, seed), case, _device()
    kind = c["kind"]
    if kind == "draft":
        s.q = ps.alloc_compressed(s.B, s.k, dev)
        s.out_tok = torch.empty(s.B, dtype=torch.int32, device=dev)
        s.out_q = torch.empty(s.B, device=dev)
        return s
    if kind in ("round", "calls", "verify", "pieces"):
        s.ver = ps.alloc_verified(s.B, s.N, dev)
        s.res = ps.alloc_residual(s.B, dev)
        if kind in ("round", "calls"):
            s.q = ps.alloc_compressed(s.N, s.k, dev)
        else:
            s.q = _records(c, s.draft)
            del s.draft
        if kind != "pieces":
            which = {"round": ps.CALL_ROUND, "calls": ps.CALL_VERIFY, "verify": ps.CALL_VERIFY_SAMPLE}[kind]
            s.ws = ps.alloc_workspace(s.tgt.dtype, s.N + s.B, s.V, dev, which)
        else:
            s.gamma_max = c["gamma_hi"]
            g = s.seq_off[1:] - s.seq_off[:-1]
            s.gamma_max = min(s.gamma_max, s.N)
            s.mid, s.zero, s.end = (g + 1) // 2, torch.zeros_like(g), g
            s.first = ps.Verified(torch.empty_like(s.ver.n_accept), s.ver.p_tok, s.ver.q_tok, s.ver.tgt_max, s.ver.tgt_sum,
                                  s.ver.tgt_lse, torch.empty_like(s.ver.flags))
        return s
    q = _scalars(s)
    if kind == "cloud":
        del s.draft
        s.up, n = ps.pack_uplink(s.seq_off, s.N, s.tok, q, c["fmt"])
        s.up_bytes = int(n.item())
        s.ver = ps.alloc_verified(s.B, s.N, dev)
        s.rec = ps.alloc_compressed(s.B, s.k, dev)
        s.down = torch.zeros(ps.downlink_bytes_max(s.B, s.k, c["fmt"]), dtype=torch.uint8, device=dev)
    else:
        s.q = q
        # what the cloud answers: the number of accepted tokens and the record of the rejected target row
        r = random.Random(int(seed) * 31 + 5)
        na = [min(s.off[b + 1] - s.off[b], r.randint(0, 6)) for b in range(s.B)]
        rows = torch.tensor([s.off[b] + b + na[b] for b in range(s.B)], device=dev)
        rec = _records(c, s.tgt[rows])
        na = torch.tensor(na, dtype=torch.int32, device=dev)
        bonus = torch.randint(0, s.V, (s.B,), device=dev, generator=_gen(seed, 6, dev)).to(torch.int32)
        s.down, n, _ = ps.pack_downlink(s.seq_off, na, bonus, rec, c["fmt"])
        s.down_bytes = int(n.item())
        s.up = torch.zeros(ps.uplink_bytes(s.B, s.N, c["fmt"]), dtype=torch.uint8, device=dev)
        s.res = ps.alloc_residual(s.B, dev)
        del s.tgt
    return s


# ---------------------------------------------------------------- one pass

def _out_q(q):
    return {"idx": q.idx, "prob": q.prob, "count": q.count, "mass": q.mass, "lse": q.lse}


def _out_v(v):
    return {"n_accept": v.n_accept, "p_tok": v.p_tok, "q_tok": v.q_tok, "max": v.tgt_max, "sum": v.tgt_sum, "lse": v.tgt_lse,
            "flags": v.flags}


def _out_r(r):
    return {"tok": r.out_tok, "mass": r.resid_mass, "flags": r.flags}


def run(s):
    c = s.c
    kind, fmt = c["kind"], c["fmt"]
    if kind == "draft":
        ps.compress(s.draft, s.V, s.T, s.k, c["top_p"], out=s.q)
        ps.sample_draft(s.q, s.duni, s.out_tok, s.out_q)
        return {"q": _out_q(s.q), "tok": s.out_tok, "q_scalar": s.out_q}
    if kind == "round":
        ps.round(s.draft, s.tgt, s.V, s.T, s.seq_off, s.N, s.tok, s.k, s.uni, top_p=c["top_p"], q=s.q, ver=s.ver, res=s.res,
                 workspace=s.ws)
        return {"q": _out_q(s.q), "v": _out_v(s.ver), "r": _out_r(s.res)}
    if kind == "calls":
        ps.compress(s.draft, s.V, s.T, s.k, c["top_p"], out=s.q)
        ps.verify(s.tgt, s.V, s.T, s.seq_off, s.N, s.tok, s.q, s.uni, out=s.ver, workspace=s.ws)
        ps.sample_residual(s.tgt, s.V, s.T, s.seq_off, s.N, s.ver, s.q, s.uni, out=s.res, workspace=s.ws)
        return {"q": _out_q(s.q), "v": _out_v(s.ver), "r": _out_r(s.res)}
    if kind == "verify":
        ps.verify_sample(s.tgt, s.V, s.T, s.seq_off, s.N, s.tok, s.q, s.uni, ver=s.ver, res=s.res, workspace=s.ws)
        return {"v": _out_v(s.ver), "r": _out_r(s.res)}
    if kind == "pieces":
        ps.verify_range(s.tgt, s.V, s.T, s.seq_off, s.N, s.tok, s.q, s.uni, s.zero, s.mid, s.gamma_max, out=s.first)
        ps.verify_range(s.tgt, s.V, s.T, s.seq_off, s.N, s.tok, s.q, s.uni, s.mid, s.end, s.gamma_max, out=s.ver)
        n = torch.where(s.first.n_accept < s.mid, s.first.n_accept, s.ver.n_accept)
        ps.sample_residual(s.tgt, s.V, s.T, s.seq_off, s.N, s.ver, s.q, s.uni, out=s.res, n_accept=n)
        return {"n": n, "v": _out_v(s.ver), "r": _out_r(s.res)}
    if kind == "cloud":
        seq_off, tok, q, up_status = ps.unpack_uplink(s.up, s.up_bytes, s.B, s.N)
        ps.verify(s.tgt, s.V, s.T, seq_off, s.N, tok, None, s.uni, q_scalar=q, out=s.ver)
        ps.compress_rejected(s.tgt, s.V, s.T, seq_off, s.N, s.ver.n_accept, s.k, out=s.rec)
        down, n, status = ps.pack_downlink(seq_off, s.ver.n_accept, None, s.rec, fmt, wire=s.down)
        return {"up": [seq_off, tok, q, up_status], "v": _out_v(s.ver), "rec": _out_q(s.rec), "down": [down, n, status]}
    up, n = ps.pack_uplink(s.seq_off, s.N, s.tok, s.q, fmt, wire=s.up)
    mx, sm, lse = ps.row_stats(s.draft, s.V, s.T)
    d = ps.unpack_downlink(s.down, s.down_bytes, s.B, s.k)
    ps.resample_sparse(s.draft, s.V, s.T, s.seq_off, s.N, d.n_accept, mx, sm, d.rec, s.uni, out=s.res)
    return {"up": [up, n], "stats": [mx, sm, lse], "rec": [d.rec.idx, d.rec.prob, d.rec.count, d.rec.mass, d.n_accept, d.token, d.status],
            "r": _out_r(s.res)}


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    c = case
    esz = 4 if c["dtype"] == "f32" else 2
    B, V, k = c["B"], c["V"], c["k"]
    N = B * (c["gamma_lo"] + c["gamma_hi"]) / 2
    row, rec = V * esz, 8 * k
    kind = c["kind"]
    rows = {"draft": B, "round": 2 * N + B, "calls": 2 * N + B, "verify": N + B, "pieces": N + B, "cloud": N + B, "edge": N}[kind]
    recs = {"draft": B, "round": N, "calls": N, "verify": B, "pieces": B, "cloud": 2 * B, "edge": 2 * B}[kind]
    # (a record entry is read for the draw; the records that the acceptance test only looks one token up in are not counted)
    return {"bytes": float(rows * row + recs * rec), "flops": float(4 * rows * V)}


def tolerance(case):
    # fp32 sums in another order, one v_exp_f32 each: 32-bit results agree to a few 1e-7; a whole value may differ where a
    # uniform falls on a step of the cumulative sum or a ratio (about one draw in a thousand)
    return {"rel": 1e-6, "max": 1e-5, "differ": 0.01}


# ---------------------------------------------------------------- the same in 64 bits

def _stats64(z, T):
    """(max of the raw logits, sum exp((z - max)/T), lse) of fp64 rows."""
    m = z.max(1).values
    s = torch.exp((z - m.unsqueeze(1)) / T).sum(1)
    return m, s, m / T + torch.log(s)


def _rows64(fn, logits, V, *per_row):
    """fn over chunks of rows in fp64, its results concatenated."""
    step, got = max(1, (_CHUNK >> 1) // V), []
    for r0 in range(0, logits.shape[0], step):
        got.append(fn(logits[r0:r0 + step].double(), *[p[r0:r0 + step] for p in per_row]))
    return [torch.cat(x) for x in zip(*got)]


def _record64(c, z):
    """(prob [n, k] with zeros behind the count, count, mass, lse) of fp64 rows."""
    m, s, lse = _stats64(z, c["T"])
    k = c["k"]
    top = torch.topk(z, k, dim=1, sorted=True).values
    p = torch.exp((top - m.unsqueeze(1)) / c["T"]) / s.unsqueeze(1)
    n = torch.full_like(m, k).long()
    if 0 < c["top_p"] < 1:
        pf = p.float().double()
        keep = (torch.cumsum(pf, 1) - pf) < c["top_p"]
        n = keep.sum(1)
        p = torch.where(keep, p, 0.0)
    return p, n, p.sum(1), lse


def exact(case, seed):
    c, s = case, _inputs(case, seed)
    V, T, k, kind = s.V, s.T, s.k, case["kind"]
    none_q = {"idx": None, "count": None}

    def records(z):
        return _rows64(lambda zz: _record64(c, zz), z, V)

    if kind == "draft":
        p, n, mass, lse = records(s.draft)
        return {"q": dict(none_q, prob=p, mass=mass, lse=lse), "tok": None, "q_scalar": None}
    if kind == "edge":
        mx, sm, lse = _rows64(lambda z: _stats64(z, T), s.draft, V)
        return {"up": [None, None], "stats": [mx, sm, lse], "rec": [None] * 7, "r": {"tok": None, "mass": None, "flags": None}}

    mx, sm, lse = _rows64(lambda z: _stats64(z, T), s.tgt, V)
    dev = mx.device
    rows_t = torch.tensor([s.off[b] + b + i for b in range(s.B) for i in range(s.off[b + 1] - s.off[b])], device=dev)
    x = s.tok.long()
    p_tok = torch.exp((s.tgt[rows_t, x].double() - mx[rows_t]) / T) / sm[rows_t]
    v = {"n_accept": None, "p_tok": p_tok, "q_tok": None, "max": mx, "sum": sm, "lse": lse, "flags": None}
    if kind == "cloud":
        return {"up": [None] * 4, "v": v, "rec": dict(none_q, prob=None, mass=None, lse=None), "down": [None] * 3}

    prob, count, mass, dlse = records(s.draft)
    ids = torch.arange(V, device=dev)

    def q_of(z, xx, n, ml):                                 # qhat of the drafted token: 0 outside its record
        zx = z.gather(1, xx.unsqueeze(1))
        rank = ((z > zx) | ((z == zx) & (ids.unsqueeze(0) < xx.unsqueeze(1)))).sum(1)
        return [torch.where(rank < n, torch.exp(zx[:, 0] / T - ml[:, 1]) / ml[:, 0], 0.0)]

    (q_tok,) = _rows64(q_of, s.draft, V, x, count, torch.stack([mass, dlse], 1))
    v["q_tok"] = q_tok
    u = s.uni[rows_t].double()
    ok = ((u < 1) & torch.where(q_tok > 0, u * q_tok < p_tok, True)).tolist()
    resid = []
    for b in range(s.B):
        d0, g = s.off[b], s.off[b + 1] - s.off[b]
        j = next((i for i in range(g) if not ok[d0 + i]), g)
        z = s.tgt[d0 + b + j].double()
        r = torch.exp((z - mx[d0 + b + j]) / T) / sm[d0 + b + j]
        if j < g:
            n = int(count[d0 + j])
            at = torch.sort(s.draft[d0 + j].float(), descending=True, stable=True).indices[:n]
            qd = torch.zeros(V, dtype=torch.float64, device=dev)
            qd[at] = prob[d0 + j, :n] / mass[d0 + j]
            r = (r - qd).clamp(min=0)
        resid.append(r.sum())
    r = {"tok": None, "mass": torch.stack(resid), "flags": None}
    if kind == "verify":
        return {"v": v, "r": r}
    if kind == "pieces":
        return {"n": None, "v": v, "r": r}
    return {"q": dict(none_q, prob=prob, mass=mass, lse=dlse), "v": v, "r": r}
