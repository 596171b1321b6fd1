"""Workspaces, the caller's and the library's: results against the FP64 oracle
at the tolerances of the forms."""
import ctypes
import threading

import pytest
import torch

import oracle
import paper_2002_03258_amd as tsm
import seeded_inputs as si
from paper_2002_03258_amd import _lib

from helpers import TOL, dev_matrix, err, host_matrix, to_np

pytestmark = pytest.mark.gpu

DT = {torch.float64: tsm.F64, torch.float32: tsm.F32}


def _ws(nbytes, dev):
    """A 256-byte aligned workspace of exactly nbytes, and the bytes behind it."""
    store = torch.full((nbytes + 512,), 0xA5, dtype=torch.uint8, device=dev)
    off = -store.data_ptr() % 256
    return store[off:off + nbytes], store[off + nbytes:]


def _operands(seed, form, m, k, n, rowA, dev):
    """(A for the binding, B, reference, dtype code, tolerance)"""
    dtype = torch.float64 if form == "f64" else torch.float32
    A = dev_matrix(seed, si.STREAM_A, m, k, dtype, dev)
    B = dev_matrix(seed, si.STREAM_B, k, n, dtype, dev)
    if form in ("f64", "f32"):
        ref = oracle.matmul(host_matrix(seed, si.STREAM_A, m, k, dtype),
                            host_matrix(seed, si.STREAM_B, k, n, dtype))
        return (A.contiguous() if rowA else A), B, ref, DT[dtype], TOL[dtype]
    S = tsm.split(A, form, lo=False)
    ref = oracle.matmul(to_np(S.hi), host_matrix(seed, si.STREAM_B, k, n, dtype))
    return S, B, ref, S.dtype_code, 3e-6


@pytest.mark.parametrize("form,m,k,n,rowA", [("bf16", 5120, 400, 33, False),
                                             ("bf16", 775, 8570, 114, False),
                                             ("f64", 5200, 1980, 33, True),
                                             ("f32", 16, 1764, 137, False),
                                             ("f32", 300, 9001, 97, False)])
def test_wide_products_in_the_queried_workspace(dev, form, m, k, n, rowA):
    """The queried bytes serve every panel, B in either order, beta != 0, and
    nothing behind them is written."""
    A, B, ref, code, tol = _operands(4000 + m + k + n, form, m, k, n, rowA, dev)
    op = tsm.OP_TSM2R_ROWMAJOR if rowA else tsm.OP_TSM2R
    need = tsm.workspace_size(op, m, k, n, code)
    ws, behind = _ws(need, dev)
    for b in (B, B.contiguous()):
        C = torch.ones((n, m), dtype=b.dtype, device=dev).t()
        tsm.tsm2r(A, b, out=C, beta=2.0, workspace=ws)
        assert err(to_np(C), ref + 2.0) <= tol
    assert bool((behind == 0xA5).all())


def test_workspace_too_small_for_the_last_panel(dev):
    """Panels of 32 columns need nothing here, the last one of 4 does: refused
    before the first one runs."""
    m, k, n = 139, 2285, 100
    A, B, ref, code, tol = _operands(4050, "f32", m, k, n, False, dev)
    C = torch.full((n, m), 7.0, dtype=torch.float32, device=dev).t()
    ws, _ = _ws(1, dev)
    tsm.tsm2r(A, B[:, :32], workspace=ws)
    with pytest.raises(tsm.TSMError) as e:
        tsm.tsm2r(A, B, out=C, beta=1.0, workspace=ws)
    assert e.value.code == 3
    torch.cuda.synchronize()
    assert bool((C == 7.0).all())


@pytest.mark.parametrize("form,m,k,n,rowA", [("f32", 3001, 3001, 20, False), ("f64", 512, 1000, 32, False),
                                             ("f32", 4096, 700, 16, False), ("f32", 600, 2000, 1, True),
                                             ("f32", 50, 1500, 40, False), ("bf16", 3779, 1024, 11, False)])
def test_small_caller_workspace_runs_the_coarser_split(dev, form, m, k, n, rowA):
    """A workspace that holds the coarser split's bytes (none for the plain
    forms here), but not the finer split's, serves; so does one off the
    256-byte alignment where nothing is put there."""
    A, B, ref, code, tol = _operands(4100 + m + k + n, form, m, k, n, rowA, dev)
    op = tsm.OP_TSM2R_ROWMAJOR if rowA else tsm.OP_TSM2R
    least = k // 32 * 3 * 64 * 16 if form == "bf16" else 0
    assert tsm.workspace_size(op, m, k, n, code) > least
    ws, behind = _ws(max(least, 1), dev)
    for w in (ws, behind[16:32]) if least == 0 else (ws,):
        C = torch.ones((n, m), dtype=B.dtype, device=dev).t()
        tsm.tsm2r(A, B, out=C, beta=-1.0, workspace=w)
        assert err(to_np(C), ref - 1.0) <= tol
    assert bool((behind == 0xA5).all())


@pytest.mark.parametrize("form,m,k,n", [("f64", 1000, 1000, 20), ("f32", 4000, 1500, 5)])
def test_small_caller_workspace_grad_b(dev, form, m, k, n):
    dtype = torch.float64 if form == "f64" else torch.float32
    A = dev_matrix(4200, si.STREAM_A, m, k, dtype, dev)
    dC = dev_matrix(4200, si.STREAM_DC, m, n, dtype, dev)
    ref = oracle.matmul(host_matrix(4200, si.STREAM_A, m, k, dtype).T,
                        host_matrix(4200, si.STREAM_DC, m, n, dtype))
    assert tsm.workspace_size(tsm.OP_GRAD_B, m, k, n, DT[dtype]) > 0
    ws, behind = _ws(1, dev)
    for w in (ws, behind[16:32]):
        assert err(to_np(tsm.grad_b(A, dC, workspace=w)), ref) <= TOL[dtype]
    assert bool((behind == 0xA5).all())


# shapes whose split needs a workspace only to fill the GPU, one per kernel
SPLIT = [(3001, 3001, 20, False), (1500, 1000, 8, True), (16, 5000, 16, False)]


def _many(dtype, dev, count, seed):
    """[(A, B, eager result)] over the shapes of SPLIT"""
    out = []
    for i in range(count):
        m, k, n, row = SPLIT[i % len(SPLIT)]
        A = dev_matrix(seed + i, si.STREAM_A, m, k, dtype, dev)
        A = A.contiguous() if row else A
        B = dev_matrix(seed + i, si.STREAM_B, k, n, dtype, dev)
        out.append((A, B, tsm.tsm2r(A, B)))
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("dtype", list(DT))
def test_streams_are_independent(dev, dtype):
    """Products on several streams at a time, each on its stream's buffer, give
    the bits of the products one after the other."""
    ins = _many(dtype, dev, 6, 4300)
    streams = [torch.cuda.Stream() for _ in range(3)]
    outs = []
    for _ in range(20):
        for i, (A, B, want) in enumerate(ins):
            with torch.cuda.stream(streams[i % 2 if i % 3 else 2]):
                outs.append((tsm.tsm2r(A, B), want))
    torch.cuda.synchronize()
    assert all(torch.equal(got, want) for got, want in outs)


@pytest.mark.parametrize("dtype", list(DT))
def test_threads_on_one_stream(dev, dtype):
    """Threads that share a stream: the launches of one product are enqueued
    together."""
    ins = _many(dtype, dev, 4, 4400)
    outs = [[] for _ in ins]

    def work(i):
        for _ in range(50):
            outs[i].append(tsm.tsm2r(ins[i][0], ins[i][1]))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(ins))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for got, (_, _, want) in zip(outs, ins):
        assert len(got) == 50 and all(torch.equal(g, want) for g in got)


def _direct(A, B, out):
    """The C entry without a workspace, column-major A and B."""
    rc = _lib.lib().tsm2r(A.shape[0], A.shape[1], B.shape[1], A.data_ptr(), A.stride(1),
                          B.data_ptr(), B.stride(1), out.data_ptr(), out.stride(1),
                          DT[A.dtype], torch.cuda.current_stream().cuda_stream)
    assert rc == 0, rc


@pytest.mark.parametrize("dtype", list(DT))
@pytest.mark.parametrize("direct", [False, True])
def test_captured_products_outlive_a_growing_buffer(dev, dtype, direct):
    """Captured before the library owns a buffer, then larger eager products on
    the same stream, whose buffer grows past the captured one: every replay
    gives the eager bits.  Through the binding (the graph owns the workspace)
    and through the C entry (the library keeps it)."""
    m, k, n = 3001, 3001, 20
    A = dev_matrix(4500, si.STREAM_A, m, k, dtype, dev)
    B = dev_matrix(4500, si.STREAM_B, k, n, dtype, dev)
    want = tsm.tsm2r(A, B)
    big = [(dev_matrix(4501 + i, si.STREAM_A, s, s, dtype, dev), dev_matrix(4501 + i, si.STREAM_B, s, w, dtype, dev))
           for i, (s, w) in enumerate([(4099, 64), (6001, 64), (9001, 48)])]
    wants = [tsm.tsm2r(a, b) for a, b in big]
    out = tsm.empty_colmajor(m, n, dtype, dev)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    _lib.lib().tsm2x_finalize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        if direct:
            _direct(A, B, out)
        else:
            tsm.tsm2r(A, B, out=out)
    for (a, b), w in zip(big, wants):
        out.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            got = tsm.tsm2r(a, b)
        torch.cuda.synchronize()
        assert torch.equal(got, w)
        # memory given back in the meantime would be handed out here
        filler = [torch.full((1 << 22,), float("nan"), device=dev) for _ in range(8)]
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        del filler
        torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype", list(DT))
def test_graphs_of_one_stream_replayed_together(dev, dtype):
    ins = _many(dtype, dev, 4, 4600)
    capture = torch.cuda.Stream()
    graphs, outs = [], []
    for A, B, want in ins:
        outs.append(torch.zeros_like(want))
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=capture):
            tsm.tsm2r(A, B, out=outs[-1])
        graphs.append(g)
    streams = [torch.cuda.Stream() for _ in graphs]
    for _ in range(5):
        for o in outs:
            o.zero_()
        torch.cuda.synchronize()
        for _ in range(8):
            for g, s in zip(graphs, streams):
                with torch.cuda.stream(s):
                    g.replay()
        torch.cuda.synchronize()
        for o, (_, _, want) in zip(outs, ins):
            assert torch.equal(o, want)


def test_buffers_of_many_streams_are_bounded(dev):
    """More streams than the library keeps buffers for: the results are right,
    and the buffers of the streams longest unused are given back."""
    dtype = torch.float32
    m, k, n = 3001, 3001, 20
    A = dev_matrix(4700, si.STREAM_A, m, k, dtype, dev)
    B = dev_matrix(4700, si.STREAM_B, k, n, dtype, dev)
    want = tsm.tsm2r(A, B)
    out = torch.zeros_like(want)
    per = tsm.workspace_size(tsm.OP_TSM2R, m, k, n, tsm.F32)
    hip = ctypes.CDLL(_lib.LIB_PATH)          # the runtime the library is linked with
    torch.cuda.synchronize()
    _lib.lib().tsm2x_finalize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    handles = []
    for _ in range(100):
        h = ctypes.c_void_p()
        assert hip.hipStreamCreate(ctypes.byref(h)) == 0
        handles.append(h)
        with torch.cuda.stream(torch.cuda.ExternalStream(h.value)):
            out.zero_()
            _direct(A, B, out)
        torch.cuda.synchronize()
        assert torch.equal(out, want)
    kept = free - torch.cuda.mem_get_info()[0]
    assert kept <= 80 * per, (kept, per)
    _lib.lib().tsm2x_finalize()
    for h in handles:
        assert hip.hipStreamDestroy(h) == 0


def test_ordered_sum_of_more_threads_than_one_launch_has(dev):
    """A pinned split of a very tall product: the ordered sum of its slices
    takes eight threads for each of 2^29 outputs, 2^32 threads in all, more than
    one launch may have.  Small integers, every row exact."""
    m, k, n = (1 << 24) + 256, 288, 32
    col = (torch.arange(m, device=dev) % 7 - 3).to(torch.float32)
    A = col.expand(k, m).contiguous().t()
    B = torch.ones((n, k), dtype=torch.float32, device=dev).t()
    tsm.pin_tsm2r(m, k, n, tsm.F32, 9, 1)
    try:
        assert tsm.tsm2r_plan(m, k, n, tsm.F32)["slices"] == 9
        C = tsm.tsm2r(A, B)
        torch.cuda.synchronize()
    finally:
        tsm.unpin_tsm2r(m, k, n, tsm.F32)
    want = col * k
    assert all(torch.equal(C[:, p], want) for p in range(n))
    del A, B, C
    _lib.lib().tsm2x_finalize()
    torch.cuda.empty_cache()
