"""The rule by which a call's rows are split over workgroups, and the split kernels' code, without a GPU."""
import os
import re
import subprocess
import tempfile

import pytest


@pytest.fixture(scope="module")
def B():
    from paper_2603_19133_amd import binding
    return binding


def test_scratch_is_asked_for_where_rows_are_split_only(B):
    f = B.workspace_bytes
    for dt in (B.F32, B.BF16):
        for rows, k in ((192, 256), (128, 1024), (80, 4096)):        # more rows fill the chip by themselves
            assert f(B.CALL_COMPRESS, dt, 1, 151936, k) > 0 and f(B.CALL_COMPRESS, dt, rows, 151936, k) > 0
            assert f(B.CALL_COMPRESS, dt, rows + 1, 151936, k) == 0
        assert f(B.CALL_COMPRESS, dt, 1, 16384, 64) > 0
        assert f(B.CALL_COMPRESS, dt, 2, 32767, 4096) == 0           # a record of more than an eighth of the row
        assert f(B.CALL_COMPRESS, dt, 4, 16383, 64) == 0             # too short to split
        assert f(B.CALL_COMPRESS, dt, 1, 1 << 20, 64) == 0           # more lists than a finishing wave has lanes
        assert f(B.CALL_COMPRESS, dt, 0, 32000, 64) == 0
        sizes = [f(B.CALL_COMPRESS, dt, r, 40000, 100) for r in range(1, 193)]
        assert all(b > a for a, b in zip(sizes, sizes[1:]))
        # a round's workspace without k is its segment table; with k it holds the scratch of up to that many draft rows as well
        table = f(B.CALL_ROUND, dt, 20, 32000, 0)
        assert f(B.CALL_ROUND, dt, 20, 32000, 64) >= table + f(B.CALL_COMPRESS, dt, 20, 32000, 64)


FAKE = 0x1000


def test_a_smaller_workspace_is_accepted_and_a_misaligned_one_is_not(B):
    """Both calls fail later checks of theirs in no case: no rows, nothing is launched (the calls return before that only where the
    workspace is refused)."""
    call = lambda ws, n: B.lib.picospec_compress(None, B.F32, 100, 0, 100, 1.0, 10, 0.0, None, None, None, None, None, ws, n, None)
    assert call(FAKE + 4, 1 << 20) == B.EWORKSPACE
    rs = lambda ws, n, rows=2: B.lib.picospec_row_stats_ws(FAKE, B.F32, 100, rows, 100, 1.0, FAKE, FAKE, None, ws, n, None)
    assert rs(FAKE + 4, 1 << 20) == B.EWORKSPACE and rs(FAKE, 16) == B.EWORKSPACE
    assert B.lib.picospec_row_stats_ws(FAKE, B.F32, 100, 2, 100, 0.0, FAKE, FAKE, None, None, 0, None) == B.EINVAL
    assert B.lib.picospec_row_stats_ws(FAKE, B.F32, 100, 2, 100, 1.0, None, FAKE, None, None, 0, None) == B.EINVAL
    assert B.lib.picospec_row_stats_ws(FAKE, 9, 100, 2, 100, 1.0, FAKE, FAKE, None, None, 0, None) == B.EDTYPE


def test_split_kernels_keep_claimed_slots_in_registers():
    """The finishing kernel holds the general compression for the rows it gives up, with that code's hand-issued LDS atomics: no
    scratch access may stand between one of them and the wait that follows (see the same test of the compress kernels)."""
    from paper_2603_19133_amd import build as bld
    if not os.path.exists(bld.HIPCC):
        pytest.skip("hipcc not found")
    flags = [f for f in bld.FLAGS if f not in ("-shared", "-fPIC")]
    with tempfile.TemporaryDirectory() as tmp:
        asm = os.path.join(tmp, "split.s")
        out = subprocess.run([bld.HIPCC, *flags, "-S", "--cuda-device-only", "-o", asm, os.path.join(bld.CSRC, "split.hip")],
                             capture_output=True, text=True)
        assert out.returncode == 0, out.stderr[-2000:]
        lines = open(asm).read().split("\n")
    seen, name, pending, by_hand = {}, None, False, False
    for line in lines:
        m = re.match(r"^(_ZN8picospec\S+):", line)
        if m:
            name, pending, by_hand = m.group(1), False, False
            seen[name] = dict(atomics=0, scratch=0, in_window=0)
            continue
        if name is None:
            continue
        ins = line.strip()
        if ins.startswith(";;#ASMSTART") or ins.startswith(";;#ASMEND"):
            by_hand = ins.startswith(";;#ASMSTART")
        elif ins.startswith("s_endpgm"):
            name = None
        elif ins.startswith("ds_add_rtn") and by_hand:
            seen[name]["atomics"] += 1
            pending = True
        elif ins.startswith("s_waitcnt") and "lgkmcnt(0)" in ins:
            pending = False
        elif ins.startswith("scratch_"):
            seen[name]["scratch"] += 1
            seen[name]["in_window"] += pending
    claiming = [k for k, v in seen.items() if v["atomics"] >= 8]                # what the finishing kernel calls, both types
    assert len(claiming) == 2 and all("split_row_again" in k for k in claiming), seen
    assert all(v["in_window"] == 0 for v in seen.values()), seen
    assert all(v["scratch"] == 0 for k, v in seen.items() if "select" in k or "split_round" in k), seen


def test_the_binding_asks_the_library_for_its_scratch(B):
    """One copy of the rules: what the binding allocates is what picospec_scratch_bytes says, 0 where a call has no use for it."""
    f, w = B.scratch_bytes, B.workspace_bytes
    for dt in (B.F32, B.BF16):
        for rows in (0, 1, 8, 64, 80, 128, 129, 192, 193, 224, 225, 1000):
            for V in (4096, 16383, 16384, 33001, 151936):
                for k in (10, 1024, 4096):
                    assert f(B.CALL_COMPRESS, dt, rows, 0, V, k) == f(B.CALL_COMPRESS_REJECTED, dt, 7, rows, V, k) == w(B.CALL_COMPRESS, dt, rows, V, k)
                    for which in (B.CALL_VERIFY, B.CALL_VERIFY_SAMPLE, B.CALL_ROW_STATS):
                        n = f(which, dt, rows, 0, V, k)
                        assert n in (0, w(B.CALL_VERIFY, dt, rows, V, 0)) and B._split_stats(which, dt, rows, 0, V) == (n > 0)
                    # a round's is its table and, behind it, the scratch of its draft rows
                    n = f(B.CALL_ROUND, dt, rows, 3, V, k)
                    assert n == 0 or n == -(-w(B.CALL_ROUND, dt, rows + 3, V, 0) // 16) * 16 + w(B.CALL_COMPRESS, dt, rows, V, k)
    assert f(B.CALL_SAMPLE_RESIDUAL, B.F32, 8, 8, 151936, 64) > 0 and f(B.CALL_SAMPLE_RESIDUAL, B.F32, 8, 8, 4096, 64) == 0
    for bad in ((B.CALL_VERIFY, 7, 8, 1, 151936), (B.CALL_VERIFY, B.F32, -1, 1, 151936), (B.CALL_VERIFY, B.F32, 8, 1, 0),
                (B.CALL_VERIFY, B.F32, 8, 1, (1 << 20) + 1), (B.CALL_VERIFY, B.F32, 2 ** 31 - 1, 1, 151936), (B.CALL_SAMPLE_DRAFT, B.F32, 8, 1, 151936)):
        assert f(*bad, 64) == 0


def test_a_round_spreads_its_drafts_only_where_that_was_faster(B):
    """By (drafts, sequences, V, k) as measured against the one launch for both streams: slower ones keep it, whatever the caller's
    buffer."""
    f = lambda dt, n, b, V, k: B.scratch_bytes(B.CALL_ROUND, dt, n, b, V, k) > 0
    for dt in (B.F32, B.BF16):
        for n, b, k in ((20, 300, 64), (20, 300, 4096), (64, 300, 4096), (128, 128, 1024), (128, 128, 64), (80, 80, 4096), (49, 10, 4096),
                        (64, 450, 64), (16, 497, 64), (161, 32, 64)):
            assert not f(dt, n, b, 64000, k), (n, b, k)
        for n, b, k in ((4, 1, 64), (64, 8, 256), (80, 20, 1024), (80, 20, 2048), (48, 3, 4096), (96, 64, 256)):
            assert f(dt, n, b, 151936, k), (n, b, k)
        for n, b, V in ((48, 1, 24000), (24, 1, 23999), (72, 3, 23999)):                 # drafts per sequence
            assert f(dt, n, b, V, 64) and not f(dt, n + 1, b, V, 64), (n, b, V)
    assert f(B.F32, 160, 64, 64000, 256) and not f(B.F32, 160, 65, 64000, 256)
    assert f(B.F32, 128, 64, 24000, 257) and f(B.F32, 64, 64, 23999, 257) and not f(B.F32, 65, 64, 23999, 257)
    # bf16: fewer drafts where one launch for both streams takes three workgroups per CU, up to its longest record and shortest row
    assert f(B.BF16, 96, 64, 32768, 256) and not f(B.BF16, 97, 63, 32768, 256) and not f(B.BF16, 96, 65, 32768, 256)
    assert f(B.BF16, 80, 80, 64000, 257) and not f(B.BF16, 81, 79, 64000, 257) and f(B.BF16, 64, 160, 64000, 257)
    assert not f(B.BF16, 128, 64, 32768, 256) and f(B.BF16, 128, 64, 32767, 256) and not f(B.BF16, 129, 64, 32767, 256)
    assert not f(B.BF16, 20, 480, 32768, 64) and f(B.BF16, 20, 480, 32767, 64)             # (beyond 512 rows in all)
    assert not f(B.BF16, 20, 480, 64000, 2048) and f(B.BF16, 20, 480, 64000, 2049)
    assert not f(B.BF16, 160, 80, 151936, 64) and not f(B.BF16, 0, 4, 151936, 64) and not f(B.BF16, 193, 4, 151936, 64)


def test_statistics_are_spread_without_a_workspace_only_where_that_was_faster(B):
    f = lambda which, dt, rows, V: B.scratch_bytes(which, dt, rows, 0, V, 0) > 0
    for V, f32, bf16 in ((16384, 0, 0), (20000, 160, 128), (32000, 160, 128), (64000, 160, 224), (151936, 160, 224)):
        for dt, most in ((B.F32, f32), (B.BF16, bf16)):
            assert f(B.CALL_VERIFY, dt, most or 1, V) == (most > 0) and not f(B.CALL_VERIFY, dt, most + 1, V)
            assert f(B.CALL_VERIFY_SAMPLE, dt, 224, V) and not f(B.CALL_VERIFY_SAMPLE, dt, 225, V)       # (the draw works from the table)
    for V, f32, bf16 in ((32000, 0, 0), (62500, 64, 0), (64000, 64, 0), (128256, 128, 160), (151936, 128, 160)):
        for dt, most in ((B.F32, f32), (B.BF16, bf16)):
            assert f(B.CALL_ROW_STATS, dt, most or 1, V) == (most > 0) and not f(B.CALL_ROW_STATS, dt, most + 1, V)


def test_a_draw_with_a_table_of_its_own_asks_for_a_row_per_sequence(B):
    for dt in (B.F32, B.BF16):
        for n, b in ((3, 2), (1024 * 16, 1024), (0, 300)):
            got = B.scratch_bytes(B.CALL_SAMPLE_RESIDUAL, dt, n, b, 151936, 64)
            assert got == B.workspace_bytes(B.CALL_SAMPLE_RESIDUAL, dt, b, 151936, 64) and got < 3000 * b + 16
