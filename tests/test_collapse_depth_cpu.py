"""Planned 4-wide nodes make no tree deeper than opening by area does: the
levels size every lane's stack, so a deeper tree needs larger workspaces and
may not fit the scratch of pt_render_frame_noalloc any more.  The levels of
the tree opened by area are computed here from the same splits: `LEVELS` holds
those of the builder without the plan, for scenes whose plan alone is one to
four levels deeper."""
import pytest

from paper_2605_27323_amd import ptmi, scenes

LEVELS = [("procedural", 0, 2, 8), ("procedural", 1, 4, 7), ("procedural", 2, 2, 7), ("procedural", 2, 250, 14),
          ("soup", 0, 512, 7), ("soup", 2, 512, 6), ("soup", 0, 10000, 10), ("soup", 3, 50000, 14),
          ("instanced", 0, 40, 10), ("instanced", 1, 1000, 13), ("instanced", 2, 4000, 15)]


@pytest.mark.parametrize("kind,seed,n,levels", LEVELS)
def test_no_deeper_than_opened_by_area(kind, seed, n, levels):
    inst = None
    if kind == "procedural":
        scene, _ = scenes.procedural(seed=seed, n_objects=n)
    elif kind == "soup":
        scene = scenes.random_soup(seed, n)
    else:
        scene, inst, _ = scenes.instanced_procedural(seed=seed, n_instances=n)
    info = ptmi.Context(scene, device=-1, instances=inst).info
    assert info.depth <= levels
    assert info.stack_entries <= 3 * levels + (2 if inst else 1)
