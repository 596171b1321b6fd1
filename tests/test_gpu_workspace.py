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
    nothing behind them is written; a workspace too small for the last panel
    is refused before the first one runs."""
    A, B, ref, code, tol = _operands(4000 + m + k + n, form, m, k, n, rowA, dev)
    op = tsm.OP_TSM2R_ROWMAJOR if rowA else tsm.OP_TSM2R
    need = tsm.workspace_size(op, m, k, n, code)
    ws, behind = _ws(need, dev)
    for b in (B, B.contiguous()):
        C = torch.ones((n, m), dtype=b.dtype, device=dev).t()
        tsm.tsm2r(A, b, out=C, beta=2.0, workspace=ws)
        assert err(to_np(C), ref + 2.0) <= tol
    assert bool((behind == 0xA5).all())
    if form == "bf16":
        C = torch.full((n, m), 7.0, dtype=torch.float32, device=dev).t()
        # room for a panel of 32 columns, but not for the last one
        small = tsm.workspace_size(op, m, k, 32, code)
        assert small < need
        with pytest.raises(tsm.TSMError) as e:
            tsm.tsm2r(A, B, out=C, beta=1.0, workspace=ws[:small])
        assert e.value.code == 3
        torch.cuda.synchronize()
        assert bool((C == 7.0).all())
