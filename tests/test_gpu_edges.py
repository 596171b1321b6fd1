"""Edges of the tiles and steps: matrices of odd sizes and odd leading
dimensions, whose columns start at any element, against the FP64 oracle at
the tolerances of the plain forms."""
import numpy as np
import pytest
import torch

import oracle
import paper_2002_03258_amd as tsm
import seeded_inputs as si
from paper_2002_03258_amd import kmeans

from helpers import TOL, dev_matrix, err, host_matrix, to_np

pytestmark = pytest.mark.gpu

DTYPES = [torch.float64, torch.float32]


def _odd_ld(x, shift=1):
    """x as a column-major view with an odd leading dimension, `shift`
    elements into its storage, NaN around it."""
    rows, cols = x.shape
    store = torch.full((cols, (rows + shift) | 1), float("nan"), dtype=x.dtype, device=x.device)
    v = store[:, shift:shift + rows].t()
    v.copy_(x)
    return v


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("m,k,n", [(127, 2050, 5), (128, 2049, 20), (129, 4099, 4), (511, 8191, 17),
                                   (3001, 3001, 20), (65, 70, 32)])
def test_tsm2r_any_alignment(dev, monkeypatch, dtype, m, k, n):
    """A whole last tile moved up, a clamped last chunk: with the next chunk in
    flight and without, equal bit for bit; beta != 0 added once per row."""
    seed = 3000 + m + k + n
    A = _odd_ld(dev_matrix(seed, si.STREAM_A, m, k, dtype, dev))
    B = _odd_ld(dev_matrix(seed, si.STREAM_B, k, n, dtype, dev))
    ref = oracle.matmul(host_matrix(seed, si.STREAM_A, m, k, dtype),
                        host_matrix(seed, si.STREAM_B, k, n, dtype))
    got = []
    for pf in ("0", "1"):
        monkeypatch.setenv("TSM2X_NN_PF", pf)
        got.append(tsm.tsm2r(A, B))
        C = _odd_ld(torch.ones((n, m), dtype=dtype, device=dev).t())
        tsm.tsm2r(A, B, out=C, beta=2.0)
        assert err(to_np(C), ref + 2.0) <= TOL[dtype]
    assert torch.equal(got[0], got[1])
    assert err(to_np(got[1]), ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", DTYPES)
def test_tsm2r_infinite_last_column(dev, monkeypatch, dtype):
    """The clamped loads of the last chunk leave an infinity in A's last column
    to its own row."""
    m, k, n = 300, 1037, 6
    A = dev_matrix(3, si.STREAM_A, m, k, dtype, dev)
    B = torch.ones((n, k), dtype=dtype, device=dev).t()
    A[7, k - 1] = float("inf")
    for pf in ("0", "1"):
        monkeypatch.setenv("TSM2X_NN_PF", pf)
        C = tsm.tsm2r(A, B)
        assert torch.isinf(C[7]).all()
        assert torch.isfinite(C).sum().item() == (m - 1) * n


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("m,k,n", [(2049, 33, 20), (4097, 95, 5), (8193, 31, 24), (70, 130, 32)])
def test_grad_b_any_alignment(dev, monkeypatch, dtype, m, k, n):
    seed = 3100 + m + k + n
    A = _odd_ld(dev_matrix(seed, si.STREAM_A, m, k, dtype, dev))
    dC = _odd_ld(dev_matrix(seed, si.STREAM_DC, m, n, dtype, dev))
    got = []
    for pf in ("0", "1"):
        monkeypatch.setenv("TSM2X_TN_PF", pf)
        got.append(tsm.grad_b(A, dC))
    ref = oracle.matmul(host_matrix(seed, si.STREAM_A, m, k, dtype).T,
                        host_matrix(seed, si.STREAM_DC, m, n, dtype))
    assert torch.equal(got[0], got[1])
    assert err(to_np(got[1]), ref) <= TOL[dtype]


@pytest.mark.parametrize("lo", [False, True])
@pytest.mark.parametrize("m,k,n", [(1029, 2079, 9), (517, 4127, 32), (4099, 90, 8), (2051, 130, 24)])
def test_planes_with_odd_sizes(dev, lo, m, k, n):
    """The 16-bit forms on odd sizes: forward, dB and the TSM2L forms with
    float operands at any alignment, against the oracle on the stored values."""
    seed = 3200 + m + k + n
    A = _odd_ld(dev_matrix(seed, si.STREAM_A, m, k, torch.float32, dev))
    B = dev_matrix(seed, si.STREAM_B, k, n, torch.float32, dev)
    dC = _odd_ld(dev_matrix(seed, si.STREAM_DC, m, n, torch.float32, dev))
    S = tsm.split(A, "bf16", lo=lo)
    hi, low = oracle.split(np.asfortranarray(host_matrix(seed, si.STREAM_A, m, k, torch.float32)
                                             .astype(np.float32)), oracle.BF16)
    stored = oracle.decode_plane(hi, oracle.BF16)
    if lo:
        stored = stored + oracle.decode_plane(low, oracle.BF16)
    ref = oracle.matmul(stored, host_matrix(seed, si.STREAM_B, k, n, torch.float32))
    assert err(to_np(tsm.tsm2r(S, B)), ref) <= 3e-6
    ref = oracle.matmul(stored.T, host_matrix(seed, si.STREAM_DC, m, n, torch.float32))
    assert err(to_np(tsm.grad_b(S, dC)), ref) <= 3e-6


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("m,k,n", [(1, 1, 1), (63, 2, 3), (64, 3, 16), (65, 4, 17), (129, 5, 32),
                                   (1000, 7, 8), (4097, 8, 31), (127, 9, 5), (333, 15, 16),
                                   (128, 16, 33), (4099, 17, 20), (257, 30, 7), (5000, 31, 32),
                                   (31, 32, 40)])
@pytest.mark.parametrize("pad", [0, 3])
def test_rowmajor_tall_product(dev, dtype, m, k, n, pad):
    """A row-major A with k <= 32 on the TSM2L kernel, rows `pad` elements
    apart (NaN between them, an infinity in one row), through every entry; a
    beta is applied once, in double."""
    seed = 3300 + m + k + n
    src = dev_matrix(seed, si.STREAM_A, m, k, dtype, dev)
    store = torch.full((m, k + pad), float("nan"), dtype=dtype, device=dev)
    A = store[:, pad // 2:pad // 2 + k]
    A.copy_(src)
    B = dev_matrix(seed, si.STREAM_B, k, n, dtype, dev)
    ref = oracle.matmul(host_matrix(seed, si.STREAM_A, m, k, dtype),
                        host_matrix(seed, si.STREAM_B, k, n, dtype))
    for fn in (tsm.tsm2l, tsm.tsm2r, tsm.gemm):
        assert err(to_np(fn(A, B)), ref) <= TOL[dtype]
        assert err(to_np(fn(A, B.contiguous())), ref) <= TOL[dtype]
    C = _odd_ld(torch.ones((n, m), dtype=dtype, device=dev).t())
    tsm.gemm(A, B, out=C, beta=-0.5)
    assert err(to_np(C), ref - 0.5) <= TOL[dtype]
    if m > 2:
        A[m // 2, k - 1] = float("inf")
        C = tsm.tsm2l(A, torch.ones((n, k), dtype=dtype, device=dev).t())
        assert torch.isinf(C[m // 2]).all()
        assert torch.isfinite(C).sum().item() == (m - 1) * n


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("R,ma,n", [(33, 1, 1), (255, 3, 5), (256, 16, 16), (257, 17, 16),
                                    (8191, 16, 33), (8193, 32, 17), (131073, 31, 32),
                                    (1000003, 5, 2)])
def test_short_and_long_product(dev, dtype, R, ma, n):
    """A column-major A of few rows (tt kernel), B by rows and by columns, with
    padded rows; a beta applied once; an infinity in the last row stays in its
    own outputs; a caller's workspace, also one that holds no more than the
    TSM2R plan's partials; the pinned TSM2R kernel gives the same product."""
    seed = 3400 + R + ma + n
    X = dev_matrix(seed, si.STREAM_A, R, ma, dtype, dev).contiguous()
    Y = _odd_ld(dev_matrix(seed, si.STREAM_B, R, n, dtype, dev))
    ref = oracle.matmul(host_matrix(seed, si.STREAM_A, R, ma, dtype).T,
                        host_matrix(seed, si.STREAM_B, R, n, dtype))
    rows = torch.full((R, n + 3), float("nan"), dtype=dtype, device=dev)
    Yr = rows[:, 1:n + 1]
    Yr.copy_(Y)
    code = tsm.F64 if dtype == torch.float64 else tsm.F32
    for y in (Y, Yr):
        got = tsm.tsmttsm(X, y)
        assert err(to_np(got), ref) <= TOL[dtype]
        assert torch.equal(got, tsm.tsmttsm(X, y))
        ws = torch.empty(tsm.workspace_size(tsm.OP_TSM2R, ma, R, n, code) + 256,
                         dtype=torch.uint8, device=dev)
        assert torch.equal(got, tsm.tsmttsm(X, y, workspace=ws))
        C = torch.ones((n, ma), dtype=dtype, device=dev).t()
        tsm.tsmttsm(X, y, out=C, beta=3.0)
        assert err(to_np(C), ref + 3.0) <= TOL[dtype]
    if n <= 32:
        tsm.pin_tsm2r(ma, R, n, code, 1, 0)
        try:
            assert err(to_np(tsm.tsmttsm(X, Yr)), ref) <= TOL[dtype]
        finally:
            tsm.unpin_tsm2r(ma, R, n, code)
    X[R - 1, ma - 1] = float("inf")
    C = tsm.tsmttsm(X, torch.ones((R, n), dtype=dtype, device=dev))
    assert torch.isinf(C[ma - 1]).all()
    assert torch.isfinite(C).sum().item() == (ma - 1) * n


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("k,n", [(1, 3), (2, 40), (3, 5), (4, 5), (5, 40), (7, 3), (13, 16), (23, 23),
                                 (31, 40), (33, 5), (34, 40), (63, 17), (65, 33)])
@pytest.mark.parametrize("shift", [0, 1])
def test_rowmajor_points_ragged_pieces(dev, dtype, k, n, shift):
    """Row-major points whose k values end inside a 16-byte piece, from an
    aligned base and one element past it; integer data, labels and distances
    exact; NaN around every point."""
    m = 1000 + k
    seed = 3500 + k + n
    store = torch.full((m, k + 2 * shift), float("nan"), dtype=dtype, device=dev)
    X = store[:, shift:shift + k]
    X.copy_(dev_matrix(seed, si.STREAM_A, m, k, dtype, dev, dist="int", r=6))
    Mu = dev_matrix(seed, si.STREAM_B, k, n, dtype, dev, dist="int", r=6)
    lab, dist = kmeans.assign(X, Mu.t())
    rlab, rdist = oracle.kmeans_assign(host_matrix(seed, si.STREAM_A, m, k, dtype, dist="int", r=6),
                                       host_matrix(seed, si.STREAM_B, k, n, dtype, dist="int", r=6))
    assert np.array_equal(lab.cpu().numpy(), rlab)
    assert np.array_equal(to_np(dist), rdist)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("m,k,n", [(33, 40, 33), (65, 130, 64), (63, 2049, 48), (1025, 1000, 49),
                                   (4097, 4099, 63), (300, 9001, 65), (2000, 700, 130)])
def test_wide_products(dev, dtype, m, k, n):
    """More than 32 columns: one pass over A up to 64; a beta applied once; a
    caller's workspace, also one that holds the partials of 32 columns only,
    and a pinned 32-column plan, which keeps passes of 32."""
    seed = 3600 + m + k + n
    A = _odd_ld(dev_matrix(seed, si.STREAM_A, m, k, dtype, dev))
    B = dev_matrix(seed, si.STREAM_B, k, n, dtype, dev)
    ref = oracle.matmul(host_matrix(seed, si.STREAM_A, m, k, dtype),
                        host_matrix(seed, si.STREAM_B, k, n, dtype))
    got = tsm.tsm2r(A, B)
    assert err(to_np(got), ref) <= TOL[dtype]
    assert err(to_np(tsm.tsm2r(A, B.contiguous())), ref) <= TOL[dtype]
    C = torch.ones((n, m), dtype=dtype, device=dev).t()
    tsm.gemm(A, B, out=C, beta=-2.0)
    assert err(to_np(C), ref - 2.0) <= TOL[dtype]
    code = tsm.F64 if dtype == torch.float64 else tsm.F32
    ws = torch.empty(tsm.workspace_size(tsm.OP_TSM2R, m, k, n, code) + 256, dtype=torch.uint8,
                     device=dev)
    assert torch.equal(tsm.tsm2r(A, B, workspace=ws), got)
    small = max(tsm.workspace_size(tsm.OP_TSM2R, m, k, w, code) for w in {32, n % 32 or 32})
    if small > 0:
        assert err(to_np(tsm.tsm2r(A, B, workspace=ws[:small])), ref) <= TOL[dtype]
    tsm.pin_tsm2r(m, k, 32, code, 1, 0)
    try:
        assert err(to_np(tsm.tsm2r(A, B)), ref) <= TOL[dtype]
    finally:
        tsm.unpin_tsm2r(m, k, 32, code)


@pytest.mark.parametrize("fmt", ["bf16", "f16"])
@pytest.mark.parametrize("lo", [False, True])
@pytest.mark.parametrize("m,k,n", [(1, 1, 1), (127, 3, 5), (128, 8, 16), (129, 9, 17), (513, 16, 16),
                                   (4097, 17, 32), (100003, 31, 7), (640, 32, 32)])
def test_split_and_product_in_one_pass(dev, fmt, lo, m, k, n):
    """The forward of a float A in a 16-bit mode: planes and product equal
    split() and tsm2l() on them bit for bit, also for values that overflow
    or are not numbers, from any alignment of A and either order of B."""
    seed = 3700 + m + k + n
    A = _odd_ld(dev_matrix(seed, si.STREAM_A, m, k, torch.float32, dev))
    if m > 8:
        A[3, 0], A[4, k - 1], A[5, 0] = float("inf"), float("nan"), 1e30
        A[6, 0], A[7, k - 1] = 1e-41, -0.0
    B = dev_matrix(seed, si.STREAM_B, k, n, torch.float32, dev)
    for a in (A, A.t().contiguous().t(), A.contiguous()):
        for b in (B, B.contiguous()):
            S = tsm.split(a, fmt, lo=lo)
            want = tsm.tsm2l(S, b)
            got_s, got = tsm._split_tsm2l(a, b, fmt, lo)
            assert got_s.planes[:, :, :m].view(torch.int16).equal(S.planes[:, :, :m].view(torch.int16))
            assert got.view(torch.int32).equal(want.view(torch.int32))
            mode = fmt + ("_split" if lo else "")
            C = tsm.matmul(a, b, mode=mode, kind="L")
            assert C.view(torch.int32).equal(want.view(torch.int32))


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("m,k,n", [(1, 1, 1), (130, 7, 3), (4099, 16, 16), (1000, 32, 31),
                                   (513, 1000, 8), (2000, 33, 32)])
def test_gradients_rowmajor_b(dev, dtype, m, k, n):
    """A row-major B (padded rows too) gives the bits of its column-major copy."""
    seed = 3800 + m + k + n
    A = dev_matrix(seed, si.STREAM_A, m, k, dtype, dev)
    B = dev_matrix(seed, si.STREAM_B, k, n, dtype, dev)
    dC = dev_matrix(seed, si.STREAM_DC, m, n, dtype, dev, dist="normal")
    rows = torch.full((k, n + 3), float("nan"), dtype=dtype, device=dev)
    Bp = rows[:, 2:2 + n]
    Bp.copy_(B)
    for b in (B.contiguous(), Bp):
        assert torch.equal(tsm.grad_a(dC, b), tsm.grad_a(dC, B))
        if k <= 32:
            for got, want in zip(tsm.tsm2l_backward(A, b, dC), tsm.tsm2l_backward(A, B, dC)):
                assert torch.equal(got, want)


@pytest.mark.parametrize("dtype", DTYPES)
def test_products_captured_before_any_workspace(dev, dtype):
    """Captured before the library owns a workspace, where none can be
    allocated, the plain products run unsplit; every replay equals the eager
    result within rounding."""
    from paper_2002_03258_amd import _lib
    shapes = [(3001, 3001, 20, False), (1024, 1000, 4, True), (1000, 2000, 50, False),
              (16, 5000, 16, False)]
    ins = []
    for i, (m, k, n, row) in enumerate(shapes):
        A = dev_matrix(3900 + i, si.STREAM_A, m, k, dtype, dev)
        A = A.contiguous() if row else A
        ins.append((A, dev_matrix(3900 + i, si.STREAM_B, k, n, dtype, dev).contiguous()))
    outs = [tsm.empty_colmajor(a.shape[0], b.shape[1], dtype, dev) for a, b in ins]
    torch.cuda.synchronize()
    _lib.lib().tsm2x_finalize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for (a, b), o in zip(ins, outs):
            tsm.tsm2r(a, b, out=o)
    for _ in range(3):
        for o in outs:
            o.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for (a, b), o in zip(ins, outs):
            want = tsm.tsm2r(a, b)
            assert err(to_np(o), to_np(want)) <= TOL[dtype]


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("m,k,n", [(5, 4000, 3), (32, 4000, 32), (64, 4000, 20), (1024, 1024, 8)])
def test_kernel_name_is_the_launched_kernel(dev, dtype, m, k, n):
    A = dev_matrix(4800, si.STREAM_A, m, k, dtype, dev, ld=(m + 31) // 32 * 32)
    B = dev_matrix(4800, si.STREAM_B, k, n, dtype, dev)
    tsm.timing_start()
    tsm.tsm2r(A, B)
    tsm.timing_stop()
    names = [r["kernel"] for r in tsm.timing_collect()]
    assert tsm.kernel_name(tsm.OP_TSM2R, m, k, n, tsm.F64 if dtype == torch.float64 else tsm.F32) in names


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("m,k,n,shift", [(1000, 3, 5, 1), (1027, 40, 16, 2), (2049, 70, 33, 1),
                                         (130, 33, 17, 4), (4000003, 2, 3, 1)])
def test_colmajor_points_off_lines(dev, dtype, m, k, n, shift):
    """Column-major points whose columns start off the 128-byte lines: the
    non-temporal instance, and the cached one on a grid that goes round often
    enough; integer data, labels and distances exact."""
    seed = 4900 + k + n
    X = _odd_ld(dev_matrix(seed, si.STREAM_A, m, k, dtype, dev, dist="int", r=6), shift)
    Mu = dev_matrix(seed, si.STREAM_B, k, n, dtype, dev, dist="int", r=6)
    lab, dist = kmeans.assign(X, Mu.t())
    rlab, rdist = oracle.kmeans_assign(host_matrix(seed, si.STREAM_A, m, k, dtype, dist="int", r=6),
                                       host_matrix(seed, si.STREAM_B, k, n, dtype, dist="int", r=6))
    assert np.array_equal(lab.cpu().numpy(), rlab)
    assert np.array_equal(to_np(dist), rdist)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("m", [136, 144, 257, 300, 1011])
@pytest.mark.parametrize("k,n", [(70, 5), (33, 16), (129, 20), (40, 32)])
def test_wide_output_off_lines(dev, dtype, m, k, n):
    """dA on 64 bytes (136 and 144 rows), and by half-height tiles on any
    alignment: non-temporal stores of whole and of ragged tiles."""
    seed = 5000 + m + k + n
    dC = dev_matrix(seed, si.STREAM_DC, m, n, dtype, dev)
    B = dev_matrix(seed, si.STREAM_B, k, n, dtype, dev)
    ref = oracle.matmul(host_matrix(seed, si.STREAM_DC, m, n, dtype),
                        host_matrix(seed, si.STREAM_B, k, n, dtype).T)
    for d in (dC, _odd_ld(dC)):
        for b in (B, B.contiguous()):
            assert err(to_np(tsm.grad_a(d, b)), ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("m,k,n", [(136, 6, 32), (144, 16, 16), (1008, 30, 8), (5003, 3, 2), (5003, 1, 5),
                                   (1000, 4, 4)])
def test_tall_product_on_64_bytes(dev, dtype, m, k, n):
    """A and C on 64 bytes, or few columns on any alignment: non-temporal."""
    seed = 5100 + m + k + n
    A = dev_matrix(seed, si.STREAM_A, m, k, dtype, dev)
    B = dev_matrix(seed, si.STREAM_B, k, n, dtype, dev)
    ref = oracle.matmul(host_matrix(seed, si.STREAM_A, m, k, dtype),
                        host_matrix(seed, si.STREAM_B, k, n, dtype))
    assert err(to_np(tsm.tsm2l(A, B)), ref) <= TOL[dtype]
    C = torch.ones((n, m), dtype=dtype, device=dev).t()
    tsm.tsm2l(_odd_ld(A), B, out=C, beta=3.0)
    assert err(to_np(C), ref + 3.0) <= TOL[dtype]


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("m,k,n", [(1000, 33, 24), (77, 40, 5), (65, 65, 32), (500, 200, 17), (40, 35, 1),
                                   (31, 130, 16), (33, 67, 20), (17, 4099, 8)])
@pytest.mark.parametrize("pad", [0, 3])
def test_rowmajor_ragged_contraction(dev, dtype, m, k, n, pad):
    """A row-major A whose k is no whole number of the reduction kernel's
    steps, rows `pad` elements apart (NaN between them): the clamped rows of
    the last step, B in either order, an infinity in the last column."""
    seed = 5200 + m + k + n
    store = torch.full((m, k + pad), float("nan"), dtype=dtype, device=dev)
    A = store[:, pad // 2:pad // 2 + k]
    A.copy_(dev_matrix(seed, si.STREAM_A, m, k, dtype, dev))
    B = _odd_ld(dev_matrix(seed, si.STREAM_B, k, n, dtype, dev))
    ref = oracle.matmul(host_matrix(seed, si.STREAM_A, m, k, dtype),
                        host_matrix(seed, si.STREAM_B, k, n, dtype))
    for b in (B, B.contiguous()):
        C = torch.ones((n, m), dtype=dtype, device=dev).t()
        tsm.tsm2r(A, b, out=C, beta=-0.5)
        assert err(to_np(C), ref - 0.5) <= TOL[dtype]
    A[m // 2, k - 1] = float("inf")
    C = tsm.tsm2r(A, torch.ones((n, k), dtype=dtype, device=dev).t())
    assert torch.isinf(C[m // 2]).all()
    assert torch.isfinite(C).sum().item() == (m - 1) * n


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("m,k,n", [(1, 40, 5), (2, 16, 16), (3, 33, 20), (3, 5, 32), (5, 64, 3),
                                   (70001, 6, 24), (40003, 24, 16), (2047, 31, 20), (300, 12, 1)])
def test_grad_b_few_rows_or_columns(dev, dtype, m, k, n):
    """Fewer rows than a 16-byte run, or fewer columns than a workgroup takes."""
    seed = 5300 + m + k + n
    A = _odd_ld(dev_matrix(seed, si.STREAM_A, m, k, dtype, dev))
    dC = _odd_ld(dev_matrix(seed, si.STREAM_DC, m, n, dtype, dev))
    ref = oracle.matmul(host_matrix(seed, si.STREAM_A, m, k, dtype).T,
                        host_matrix(seed, si.STREAM_DC, m, n, dtype))
    assert err(to_np(tsm.grad_b(A, dC)), ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("m,k,n", [(262152, 40, 5), (262160, 33, 16), (262147, 40, 40), (32771, 40, 50),
                                   (40, 3000, 40), (100, 9000, 5)])
def test_tall_products_of_few_columns(dev, dtype, m, k, n):
    """Columns on 64 bytes (262152 and 262160 rows), more than 32 columns in
    two passes, and fewer rows than a tile."""
    seed = 5400 + m + k + n
    A = dev_matrix(seed, si.STREAM_A, m, k, dtype, dev)
    B = dev_matrix(seed, si.STREAM_B, k, n, dtype, dev)
    ref = oracle.matmul(host_matrix(seed, si.STREAM_A, m, k, dtype),
                        host_matrix(seed, si.STREAM_B, k, n, dtype))
    got = tsm.tsm2r(A, B)
    assert err(to_np(got), ref) <= TOL[dtype]
    code = tsm.F64 if dtype == torch.float64 else tsm.F32
    ws = torch.empty(tsm.workspace_size(tsm.OP_TSM2R, m, k, n, code) + 256, dtype=torch.uint8, device=dev)
    assert torch.equal(tsm.tsm2r(A, B.contiguous(), workspace=ws), tsm.tsm2r(A, B.contiguous()))


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("m,k,n", [(1025, 1024, 4), (2048, 2048, 8), (200, 5000, 16), (1448, 1448, 4),
                                   (64, 16384, 3), (20000, 100, 5), (257, 300, 16), (33, 256, 17)])
def test_rowmajor_b_of_the_reduction_kernel(dev, dtype, m, k, n):
    """Read in place or copied first, a row-major B gives the bits of its
    column-major copy, with rows padded too."""
    A = dev_matrix(5500, si.STREAM_A, m, k, dtype, dev).contiguous()
    B = dev_matrix(5500, si.STREAM_B, k, n, dtype, dev)
    rows = torch.full((k, n + 3), float("nan"), dtype=dtype, device=dev)
    Bp = rows[:, 2:2 + n]
    Bp.copy_(B)
    want = tsm.tsm2r(A, B)
    for b in (B.contiguous(), Bp):
        assert torch.equal(tsm.tsm2r(A, b), want)
    ref = oracle.matmul(host_matrix(5500, si.STREAM_A, m, k, dtype),
                        host_matrix(5500, si.STREAM_B, k, n, dtype))
    assert err(to_np(want), ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("m,k,n", [(4096, 4100, 8), (2049, 2048, 9), (2048, 2048, 32)])
def test_large_da_rowmajor_b(dev, dtype, m, k, n):
    dC = dev_matrix(5600, si.STREAM_DC, m, n, dtype, dev)
    B = dev_matrix(5600, si.STREAM_B, k, n, dtype, dev)
    assert torch.equal(tsm.grad_a(dC, B.contiguous()), tsm.grad_a(dC, B))
