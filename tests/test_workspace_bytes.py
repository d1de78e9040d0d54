"""Workspace sizes that callers may have fixed in their programs: the bytes that
the library asked for when its interface was first laid down (CPU only)."""
import pytest

import paper_2001_07809_amd as sbs


def up256(v):
    return (v + 255) // 256 * 256


@pytest.mark.parametrize("W,H", [(1, 1), (3, 5), (1, 100000), (40, 30), (640, 480), (1390, 1110), (4096, 2304), (9000, 7)])
def test_reconstruct_workspace_bytes(W, H):
    """Eight bytes per pixel in three arrays: slots, rows' and columns' values."""
    assert sbs.lib().sbs_reconstruct_workspace_bytes(W, H) == up256(4 * W * H) + 2 * up256(2 * W * H)
