"""Rows spread over several workgroups of which a row's last goes on (the records of few rows in one launch) against the same call in two launches, which a
workspace without room for the rows' words still takes: the same bits.  Scratch that holds anything, repeated use, captured launches."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# two parts, odd strides and sizes, the rank by lanes and by elements, lists longer than the registers take, one launch's most workgroups, the most parts
CASES = [(16384, 16384, 1, 1), (20001, 20003, 3, 330), (32000, 32000, 8, 256), (33001, 33001, 24, 1000), (128256, 128259, 2, 10), (128256, 128256, 8, 256),
         (151936, 151936, 5, 1024), (500000, 500000, 2, 2048)]


@pytest.fixture(scope="module")
def ps():
    from paper_2603_19133_amd import binding
    return binding


def _rows(g, pattern, rows, ld):
    z = torch.randn((rows, ld), device="cuda", generator=g) * 3
    if pattern == "masked":
        z[torch.rand((rows, ld), device="cuda", generator=g) < 0.999] = float("-inf")
    elif pattern == "grid":                      # values that tie: the two forms' lanes find other thresholds
        z = torch.round(z * 4) / 4
    elif pattern == "far":                       # a few values far above the others
        z[:, 7:ld:ld // 3] = 300.0
    elif pattern == "lost":                      # +-inf, NaN, one value: rows that the lists cannot give
        z[0, 5] = float("inf")
        z[rows - 1] = 0.25
        z[rows // 2, 9] = float("nan") if rows > 2 else 40.0
    return z


def _compress(ps, z, V, k, top_p, ws, out=None):
    out = out or ps.alloc_compressed(z.shape[0], k, z.device)
    for t in (out.idx, out.prob, out.count, out.mass, out.lse):
        t.fill_(-7)
    ps._check(ps._nat.compress(z, ps._dtype_code(z), z.stride(0), z.shape[0], V, 0.9, k, top_p, out.idx, out.prob, out.count, out.mass, out.lse, ws, ps._stream()))
    return out


def _same(a, b):
    for name in ("idx", "prob", "count", "mass", "lse"):
        np.testing.assert_array_equal(getattr(a, name).cpu().numpy(), getattr(b, name).cpu().numpy(), err_msg=name)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V,ld,rows,k", CASES)
@pytest.mark.parametrize("pattern", ["normal", "masked", "grid", "far", "lost"])
def test_one_launch_is_two(gpu, ps, dtype, V, ld, rows, k, pattern):
    print("[case]", V, rows, k, dtype, pattern, flush=True)
    g = torch.Generator(device="cuda"); g.manual_seed(V + k)
    z = _rows(g, pattern, rows, ld).to(dtype)[:, :V]
    code = ps._dtype_code(z)
    two = ps.scratch_bytes(ps.CALL_COMPRESS, code, rows, 0, V, k)
    one = ps.lib.picospec_one_launch_bytes(ps.CALL_COMPRESS, code, rows, 0, V, k)
    assert two > 0 and one == (two + 15) // 16 * 16 + 256 * rows
    room = torch.randint(0, 256, (one,), dtype=torch.uint8, device="cuda", generator=g)
    for top_p in (0.0, 0.9):
        want = _compress(ps, z, V, k, top_p, torch.empty(one - 1, dtype=torch.uint8, device="cuda"))
        for _ in range(3):
            _same(_compress(ps, z, V, k, top_p, room), want)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_rejected_rows(gpu, ps, dtype):
    g = torch.Generator(device="cuda"); g.manual_seed(5)
    V, k, B = 33001, 70, 7
    off = torch.tensor([0, 3, 3, 4, 9, 9, 11, 12], dtype=torch.int32, device="cuda")
    n = torch.tensor([2, 0, 1, 9, -1, 0, 1], dtype=torch.int32, device="cuda")      # (clamped to the draft's length)
    z = (torch.randn((12 + B, V), device="cuda", generator=g) * 3).to(dtype)
    code = ps._dtype_code(z)
    one = ps.lib.picospec_one_launch_bytes(ps.CALL_COMPRESS_REJECTED, code, 12, B, V, k)
    def call(size):
        out = ps.alloc_compressed(B, k, z.device)
        ws = torch.randint(0, 256, (size,), dtype=torch.uint8, device="cuda", generator=g)
        ps._check(ps._nat.compress_rejected(z, code, z.stride(0), V, 0.9, B, 12, off, n, k, 0.0, out.idx, out.prob, out.count, out.mass, out.lse, ws, ps._stream()))
        return out
    _same(call(one), call(one - 1))


def test_captured_calls_replay(gpu, ps):
    V, k, rows = 33001, 64, 6
    z = torch.randn((rows, V), device="cuda")
    out = ps.alloc_compressed(rows, k, z.device)
    ws = torch.empty(ps.lib.picospec_one_launch_bytes(ps.CALL_COMPRESS, ps.F32, rows, 0, V, k), dtype=torch.uint8, device="cuda")
    call = lambda o: ps._check(ps._nat.compress(z, ps.F32, V, rows, V, 0.9, k, 0.0, o.idx, o.prob, o.count, o.mass, o.lse, ws, ps._stream()))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call(out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(out)
    for i in range(4):
        z.copy_(torch.randn_like(z) * (2 + i))
        want = ps.alloc_compressed(rows, k, z.device)
        call(want)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        _same(out, want)


@pytest.mark.parametrize("rows,launches", [(1, 2), (3, 2), (4, 1)])
def test_captured_calls_of_very_few_rows_take_two_launches(gpu, ps, rows, launches):
    import ctypes
    V, k = 33001, 64
    z = torch.randn((rows, V), device="cuda")
    out, want = ps.alloc_compressed(rows, k, z.device), ps.alloc_compressed(rows, k, z.device)
    ws = torch.empty(ps.lib.picospec_one_launch_bytes(ps.CALL_COMPRESS, ps.F32, rows, 0, V, k), dtype=torch.uint8, device="cuda")
    _compress(ps, z, V, k, 0.0, ws, want)
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        ps._check(ps._nat.compress(z, ps.F32, V, rows, V, 0.9, k, 0.0, out.idx, out.prob, out.count, out.mass, out.lse, ws, ps._stream()))
    n = ctypes.c_size_t(0)
    assert ctypes.CDLL("libamdhip64.so").hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0 and n.value == launches
    graph.instantiate()
    for _ in range(3):
        ws.random_(0, 256)
        graph.replay()
        torch.cuda.synchronize()
        _same(out, want)
