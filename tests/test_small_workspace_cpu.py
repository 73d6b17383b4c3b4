"""Workspaces of small frames: a frame that runs as one launch asks for what
the stages (or the megakernel) ask for with the same arguments, plus at most
one row of ray counts per workgroup, whatever the launch shape; so a workspace
sized for a large frame holds a small one but for those rows.  (Per-stage
timing keeps the stages: PT_FLAG_PROFILE asks for their size.)"""
import ctypes as C

import pytest

from paper_2605_27323_amd import ptmi, scenes

DEPTH = 8
MOST_GROUPS = 8192  # 2^19 paths, 64 to a workgroup


@pytest.fixture(scope="module")
def deep():
    scene, cam = scenes.procedural(seed=2, n_objects=120)  # spills beyond the LDS entries
    ctx = ptmi.Context(scene, device=-1)
    assert ctx.info.stack_entries > 32
    return ctx, cam


def _size(ctx, cam, w, h, fn, spp=1, mode=ptmi.MODE_WAVE, flags=0, block=0, grid_mult=0):
    c = ptmi.Camera((C.c_double * 3)(*cam["eye"]), (C.c_double * 3)(*cam["target"]), (C.c_double * 3)(*cam["up"]),
                    float(cam["vfov_deg"]), w, h)
    ptmi.check(ptmi.lib().pt_set_camera(ctx.h, C.byref(c)))
    a = ptmi.RenderArgs(spp, DEPTH, 0, 0, 0, 1, -1, mode, flags, block, grid_mult)
    n = C.c_uint64()
    ptmi.check(getattr(ptmi.lib(), fn)(ctx.h, C.byref(a), C.byref(n)))
    return n.value


@pytest.mark.parametrize("fn", ["pt_workspace_size", "pt_frames_workspace_size", "pt_backward_workspace_size"])
@pytest.mark.parametrize("mode", [ptmi.MODE_WAVE, ptmi.MODE_MEGA])
@pytest.mark.parametrize("block,grid_mult", [(0, 0), (64, 1), (64, 4), (256, 4)])
def test_no_larger_than_the_stages(deep, fn, mode, block, grid_mult):
    ctx, cam = deep
    slots = 8 if fn == "pt_frames_workspace_size" else 1  # at most eight frames in flight
    for w, h, spp in ((1, 1, 1), (32, 24, 2), (64, 64, 33), (256, 128, 2), (512, 384, 1), (1024, 512, 1)):
        kw = dict(spp=spp, mode=mode, block=block, grid_mult=grid_mult)
        small, stages = (_size(ctx, cam, w, h, fn, flags=f, **kw) for f in (0, ptmi.FLAG_PROFILE))
        rows = 4 * (2 * (DEPTH + 2) + 1) * min(w * h * spp, MOST_GROUPS) + 256
        assert stages <= small <= stages + slots * rows, (w, h, spp)


def test_a_smaller_window_asks_for_no_more(deep):
    ctx, cam = deep
    large = _size(ctx, cam, 1920, 1080, "pt_workspace_size", mode=ptmi.MODE_MEGA)
    small = _size(ctx, cam, 1024, 512, "pt_workspace_size", mode=ptmi.MODE_MEGA)
    assert small <= large + 4 * (2 * (DEPTH + 2) + 1) * MOST_GROUPS + 256
