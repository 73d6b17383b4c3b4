"""The collapse to 4-wide nodes on both sides of the size from which it is
planned (512 triangles): every triangle in exactly one leaf, inside every box
of its chain of nodes, no node with fewer than two children, for soups,
coinciding triangles (all areas zero or equal) and a huge extent (areas
overflow to infinity)."""
import numpy as np
import pytest

from paper_2605_27323_amd import ptmi, scenes
from test_capi_cpu import _walk


@pytest.mark.parametrize("kind", ["soup", "same", "points", "huge"])
@pytest.mark.parametrize("nt", [511, 512, 513, 3000])
def test_collapse(nt, kind):
    scene = scenes.random_soup(11, nt)
    pos = np.array(scene["positions"], np.float32)
    idx = np.asarray(scene["indices"])
    if kind == "same":
        pos[idx] = pos[idx[0]]
    elif kind == "points":
        pos[:] = pos[0]
    elif kind == "huge":
        pos *= np.float32(1e25)
    ctx = ptmi.Context(dict(scene, positions=pos), device=-1)
    nodes, tris, _ = ctx.host_bvh()
    leaves, depth = _walk(nodes, nt)
    assert depth == ctx.info.depth and ctx.info.stack_entries == 3 * depth + 1
    assert (nodes.view(np.uint32).reshape(-1, 20)[:, 17] != 0xFFFFFFFF).all()
    covered = np.zeros(nt, int)
    ids = tris[:, 3].view(np.uint32)
    for first, cnt, boxes in leaves:
        for j in range(first, first + cnt):
            covered[int(ids[j])] += 1
            v = pos[idx[int(ids[j])]].astype(np.float64)
            for lo, hi in boxes:
                assert (v >= lo).all() and (v <= hi).all()
    assert (covered == 1).all()
