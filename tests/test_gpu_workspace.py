"""Workspaces, the caller's and the library's: results against the FP64 oracle
at the tolerances of the forms."""
import pytest
import torch

import oracle
import paper_2002_03258_amd as tsm
import seeded_inputs as si

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
