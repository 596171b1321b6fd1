"""The workspace query on the host: no GPU call is made."""
import time

import pytest
import torch

import paper_2002_03258_amd as tsm
from paper_2002_03258_amd import _lib

WIDE = [(tsm.OP_TSM2R, 5120, 400, 33, tsm.BF16), (tsm.OP_TSM2R, 775, 8570, 114, tsm.BF16),
        (tsm.OP_TSM2R_ROWMAJOR, 5200, 1980, 33, tsm.F64),
        (tsm.OP_TSM2R_ROWMAJOR, 13629, 3922, 73, tsm.F64), (tsm.OP_TSM2R, 16, 1764, 137, tsm.F32),
        (tsm.OP_TSM2L, 600, 9001, 70, tsm.F16_SPLIT), (tsm.OP_TSM2R, 300, 9001, 97, tsm.F32)]


@pytest.mark.parametrize("op,m,k,n,dtype", WIDE)
def test_query_covers_every_panel(op, m, k, n, dtype):
    """More than 32 columns run in panels that share the workspace: the query
    gives what the largest needs, which may be a narrower last one."""
    need = tsm.workspace_size(op, m, k, n, dtype)
    for width in (32, n % 32, n % 64):
        if width > 0:
            assert need >= tsm.workspace_size(op, m, k, width, dtype), width


NO_GPU = pytest.mark.skipif(torch.cuda.is_available(), reason="made-up pointers: no launch may succeed")
P = 4096         # a non-null, 256-byte aligned address that nothing reads
UNSPLIT = [(3001, 3001, 20, tsm.F32), (1024, 1024, 8, tsm.F32), (512, 1000, 32, tsm.F64),
           (8192, 1000, 8, tsm.F32), (4096, 700, 16, tsm.F32)]


@NO_GPU
@pytest.mark.parametrize("m,k,n,dtype", UNSPLIT)
def test_caller_workspace_without_room_for_the_finer_split(m, k, n, dtype):
    """Shapes that fill the GPU only by a finer split than their size asks for
    run without it in a workspace that cannot hold its partials (here the call
    then ends at its first launch, for want of a GPU); the coarser split's own
    partials are still demanded."""
    L = _lib.lib()
    for ws, nbytes in ((P, 0), (P + 16, 1 << 30)):
        rc = L.tsm2r_ex(0, 0, m, k, n, P, m, P, k, 0.0, P, m, dtype, ws, nbytes, None)
        assert rc not in (0, 3), rc
    assert L.tsm2r_ex(0, 0, 2000, 8000, 16, P, 2000, P, 8000, 0.0, P, 2000, tsm.F64, P, 256, None) == 3


@NO_GPU
def test_caller_workspace_without_room_for_the_finer_split_grad_b():
    L = _lib.lib()
    assert L.tsm_grad_b(1000, 1000, 20, P, 1000, P, 1000, P, 1000, tsm.F64, P, 0, None) not in (0, 3)
    assert L.tsm_grad_b(100000, 300, 8, P, 100000, P, 100000, P, 300, tsm.F64, P, 256, None) == 3


@NO_GPU
def test_caller_workspace_without_room_for_the_finer_split_planes():
    """16-bit planes, a k too short for the coarser split: B's packed terms (32
    rows to a chunk, three terms of 64 lanes of 16 bytes) are all it demands."""
    m, k, n = 3779, 1024, 11
    terms = k // 32 * 3 * 64 * 16
    call = lambda nbytes: _lib.lib().tsm2r_ex(0, 0, m, k, n, P, 3784, P, k, 0.0, P, m, tsm.BF16, P,
                                              nbytes, None)
    assert tsm.workspace_size(tsm.OP_TSM2R, m, k, n, tsm.BF16) > terms
    assert call(terms) not in (0, 3)
    assert call(terms - 1) == 3


def test_wide_plans_are_cheap_on_the_host():
    """A product of 33 to 64 columns looks at one split per slice length, not
    at every split: at 33 x 1048576 the six plans of a query took 28 times
    those of 32 columns, now 7."""
    def seconds(n):
        best = 1.0
        for _ in range(20):
            t0 = time.perf_counter()
            for _ in range(20):
                tsm.workspace_size(tsm.OP_TSM2R, 33, 1 << 20, n, tsm.F32)
            best = min(best, time.perf_counter() - t0)
        return best
    assert seconds(33) < 15 * seconds(32)
