"""Rules of the gfx950 instruction set that hand-written assembly has to keep by itself, held against the generated code (the
sources are cross-compiled here, no GPU needed)."""
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

SOURCES = ["split.hip", "compress.hip", "verify.hip", "residual.hip"]


@pytest.fixture(scope="module")
def listings(tmp_path_factory):
    """Source name -> its kernels' instructions as (kernel, written by hand, mnemonic, operands)."""
    from paper_2603_19133_amd import build as bld
    if not os.path.exists(bld.HIPCC):
        pytest.skip("hipcc not found")
    tmp = tmp_path_factory.mktemp("isa")
    flags = [f for f in bld.FLAGS if f not in ("-shared", "-fPIC")]

    def listing(src):
        asm = str(tmp / (src + ".s"))
        out = subprocess.run([bld.HIPCC, *flags, "-S", "--cuda-device-only", "-o", asm, os.path.join(bld.CSRC, src)],
                             capture_output=True, text=True)
        assert out.returncode == 0, out.stderr[-2000:]
        code, name, hand = [], None, False
        for line in open(asm):
            m = re.match(r"^(_ZN8picospec\S+):", line)
            if m:
                name = m.group(1)
            t = line.strip()
            if t.startswith(";;#ASMSTART") or t.startswith(";;#ASMEND"):
                hand = t.startswith(";;#ASMSTART")
                continue
            t = t.split(";")[0].strip()
            if name and re.match(r"[a-z]+_", t):
                op, _, args = t.partition(" ")
                code.append((name, hand, op, [a.strip() for a in re.split(r",(?![^\[]*\])", args)]))
        return code

    with ThreadPoolExecutor(len(SOURCES)) as pool:
        return dict(zip(SOURCES, pool.map(listing, SOURCES)))


def _regs(text, kind):
    out = set()
    for m in re.finditer(rf"\b{kind}\[(\d+):(\d+)\]|\b{kind}(\d+)\b", text):
        out.update([int(m.group(3))] if m.group(3) else range(int(m.group(1)), int(m.group(2)) + 1))
    if kind == "s" and re.search(r"\bvcc\b", text):
        out.add("vcc")
    return out


TWO_RESULTS = re.compile(r"v_(add|sub|subrev|addc|subb|subbrev)_co_|v_div_scale|v_mad_[iu]64")


@pytest.mark.parametrize("src", SOURCES)
def test_scalar_results_of_vector_instructions_have_their_wait_states(listings, src):
    """Two wait states between a vector instruction that writes an SGPR or VCC and a vector instruction that reads it.  The compiler
    pads its own code; nobody pads inside an asm statement."""
    broken, seen, kernel, pending = [], 0, None, []
    for name, hand, op, ops in listings[src]:
        if name != kernel:
            kernel, pending = name, []
        written = set()
        if op.startswith("v_"):
            n = 2 if TWO_RESULTS.match(op) else 1
            for i, a in enumerate(ops):
                if i < n:
                    written |= _regs(a, "s")
                elif any(_regs(a, "s") & regs for regs, left in pending):
                    broken.append((name, hand, op, ops))
            seen += bool(written)
        passed = int(ops[0], 0) + 1 if op == "s_nop" else 1
        pending = [(regs, left - passed) for regs, left in pending if left > passed]
        if written:
            pending.append((written, 2))
    assert seen > 100                            # (the listing was understood)
    assert not broken, (len(broken), broken[:3])


@pytest.mark.parametrize("src", SOURCES)
def test_hand_issued_loads_keep_their_registers(listings, src):
    """A load written in an asm statement lands behind the compiler's back: nothing names its registers before the wait for it."""
    broken, kernel, flying = [], None, set()
    for name, hand, op, ops in listings[src]:
        if name != kernel:
            assert not flying, kernel
            kernel = name
        if hand and op.startswith("global_load"):
            flying |= _regs(ops[0], "v")
            if _regs(ops[1], "v") & flying:
                broken.append((name, op, ops))
        elif op == "s_waitcnt" and "vmcnt(0)" in " ".join(ops):
            flying = set()
        elif flying & _regs(" ".join(ops), "v"):
            broken.append((name, op, ops))
    assert not broken, (len(broken), broken[:3])


@pytest.mark.parametrize("src,claiming", [("compress.hip", 7), ("split.hip", 2)])
def test_hand_issued_lds_results_keep_their_registers(listings, src, claiming):
    """The slots that an asm statement claims in LDS, and the counter it reads behind them, land behind the compiler's back as well: between
    the instruction and the wait nothing names their registers, nor moves them to scratch memory or another register."""
    broken, kernel, flying, claims, reads = [], None, set(), {}, {}
    for name, hand, op, ops in listings[src]:
        if name != kernel:
            assert not flying, kernel
            kernel = name
        if hand and (op.startswith("ds_add_rtn") or op.startswith("ds_read")):
            if _regs(" ".join(ops), "v") & flying:
                broken.append((name, op, ops))
            flying |= _regs(ops[0], "v")
            (claims if op.startswith("ds_add") else reads)[name] = (claims if op.startswith("ds_add") else reads).get(name, 0) + 1
        elif op == "s_waitcnt" and "lgkmcnt(0)" in " ".join(ops):
            flying = set()
        elif flying & _regs(" ".join(ops), "v"):
            broken.append((name, op, ops))
    assert len(claims) == claiming and all(n >= 8 for n in claims.values()), claims
    assert reads.keys() == claims.keys() and all(claims[k] in (4 * n, 8 * n) for k, n in reads.items()), (claims, reads)
    assert not broken, (len(broken), broken[:3])


def test_every_range_checked_load_takes_its_place_from_the_shared_rule():
    """What picospec_max_load_byte evaluates on the host is what the kernels address: every raw buffer load of a row names its
    vectors through a function of rowspan.hpp (or the spread sample's, whose vectors lie inside the row)."""
    from paper_2603_19133_amd import build as bld
    shared = ("group_first(", "split_block(", "stats_group_first(", "sample_vec(")
    loads = 0
    for name in sorted(os.listdir(bld.CSRC)):
        if name == "selfcheck.hip":              # (the probes of the range check itself)
            continue
        text = open(os.path.join(bld.CSRC, name)).read()
        for m in re.finditer(r"raw_buffer_load_b128\((\w+), ([^;]*);", text):
            loads += 1
            where = m.group(2)
            if where.startswith("lane * 16, first * 16"):        # (a helper whose callers pass the place)
                assert all(any(f in call for f in shared) for call in re.findall(r"load_vec\((?!int)[^;]*", text)), name
            else:
                assert any(f in where for f in shared), (name, where)
    assert loads >= 5
    # ... and a row's segments are chosen by functions of it as well
    text = open(os.path.join(bld.CSRC, "common.hpp")).read()
    chosen = re.findall(r"segs\.load\(([^;]*);", text)
    assert len(chosen) >= 3 and all("stats_segment(" in c or "shared_segment(" in c for c in chosen), chosen
    assert "shared_segment(" in open(os.path.join(bld.CSRC, "api.hip")).read()
