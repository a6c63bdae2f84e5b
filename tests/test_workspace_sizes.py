"""The sizes of mgs_workspace_size for the calls that keep partial sums: a
qd sum takes the place of a qd number (64 bytes), so a buffer sized for a
shape stays large enough for it.
"""
import pytest

from paper_1210_0800_amd import _lib


def up(b):
    return (b + 255) // 256 * 256


@pytest.mark.parametrize("m,n", [(1, 1), (65, 64), (320, 256), (1000, 757), (2048, 2048)])
def test_adjoint_and_refinement(m, n):
    for prec, part in ((2, 32), (4, 64)):
        chunks = (n + 7) // 8
        assert _lib.workspace_size(m, n, prec, _lib.MGS_OP_ADJOINT) == \
            2 * up(16 * prec * n) + up(16 * prec * m) + up(part * 2 * chunks * m)
        panels = (n + 63) // 64
        res = 1024 + up(16 * m * min(n, 64))
        assert _lib.workspace_size(m, n, prec, _lib.MGS_OP_REFINE) == \
            up(16 * m * (n + 1)) + up(16 * n * (n + 1)) + 2 * up(16 * n) + up(16 * m) + up(64 * panels * m) + \
            256 + up(res)
