"""The workspace query on the host: no GPU call is made."""
import pytest

import paper_2002_03258_amd as tsm

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
