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


@pytest.mark.parametrize("nframes,W,H,C,block,dmax,nbytes", [
    (1, 384, 288, 1, 15, 15, 2786816), (40, 640, 480, 3, 11, 31, 245424128), (100, 384, 288, 1, 15, 15, 278557184),
    (250, 4096, 2304, 3, 31, 127, 33320135168), (333, 8, 8, 1, 3, 3, 17399808)])
def test_search_workspace_bytes(nframes, W, H, C, block, dmax, nbytes):
    """20% lists; a frame's descriptor takes 280 bytes of a batch's workspace."""
    f = sbs.Frame(1, 1, W, H, C, W * C, 1, W * H // 5, block, dmax, 1, None)
    assert sbs.workspace_bytes([f] * nframes) == nbytes
