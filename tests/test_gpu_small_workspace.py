"""Small frames in workspaces that hold just the stages' buffers (a workspace
sized for a larger frame, or for the same frame with per-stage timing): taken
as ever, the same images and gradients as in a workspace of the size asked
for; and small frames with more chunks of paths than workgroups, whose spill
areas bound them: every launch shape gives the stages' image bit for bit.  And
pt_render_frame_noalloc with the default launch shape on scenes whose tree has
just the levels that its scratch holds stacks for."""
import ctypes as C

import numpy as np
import pytest

from paper_2605_27323_amd import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2605_27323_amd import ptmi  # noqa: E402


def _bits(t):
    return t.cpu().numpy().view(np.uint32)


@pytest.fixture(scope="module")
def renderers():
    room, cam = scenes.cornell()  # stacks entirely in LDS
    deep, dcam = scenes.procedural(seed=2, n_objects=120)
    inst_scene, inst, icam = scenes.instanced_procedural(seed=6, n_instances=60)
    return {"room": (ptmi.Renderer(room, cam), cam), "deep": (ptmi.Renderer(deep, dcam), dcam),
            "instanced": (ptmi.Renderer(inst_scene, icam, instances=inst), icam)}


def _size(R, fn, a):
    n = C.c_uint64()
    ptmi.check(getattr(ptmi.lib(), fn)(R.h, C.byref(a), C.byref(n)))
    return n.value


@pytest.mark.parametrize("which", ["room", "deep"])
@pytest.mark.parametrize("mode", ["wave", "mega"])
def test_workspace_of_the_stages_is_enough(renderers, which, mode):
    R, cam = renderers[which]
    w, h = 96, 64
    R.set_camera(dict(cam, width=w, height=h))
    L, kw = ptmi.lib(), dict(spp=2, max_depth=4, seed=3, mode=mode)
    a, pa = R.args(**kw), R.args(flags=ptmi.FLAG_PROFILE, **kw)
    img, ref = torch.empty((h, w, 3), device="cuda"), R.render(**kw)
    for fn in ("pt_workspace_size", "pt_frames_workspace_size", "pt_backward_workspace_size"):
        n = _size(R, fn, pa)
        keep, ptr = ptmi._aligned_empty(n, R.torch_device)
        print("workspace", which, mode, fn, n, flush=True)
        if fn == "pt_workspace_size":
            ptmi.check(L.pt_render_frame(R.h, C.byref(a), img.data_ptr(), None, ptr, n, R._stream()))
            assert np.array_equal(_bits(img), _bits(ref))
            assert L.pt_render_frame(R.h, C.byref(a), img.data_ptr(), None, ptr, n - 256, R._stream()) == ptmi.PT_ENOMEM
        elif fn == "pt_frames_workspace_size":
            acc, racc = torch.empty_like(img), torch.empty_like(img)
            ptmi.check(L.pt_render_frames(R.h, C.byref(a), 11, img.data_ptr(), acc.data_ptr(), ptr, n, R._stream()))
            last = R.render_frames(11, accum=racc, **kw)
            assert np.array_equal(_bits(img), _bits(last)) and np.array_equal(_bits(acc), _bits(racc))
        else:
            d = torch.ones((h, w, 3), device="cuda")
            ga, ge = torch.zeros_like(R.albedo), torch.zeros_like(R.emission)
            ra, re = torch.zeros_like(R.albedo), torch.zeros_like(R.emission)
            ptmi.check(L.pt_render_backward(R.h, C.byref(a), d.data_ptr(), ga.data_ptr(), ge.data_ptr(), ptr, n,
                                            R._stream()))
            R.backward(d, ra, re, **kw)
            # the same terms, their sums in another order: at most one per
            # vertex of every path, each addition rounded by 2^-24
            for g, r in ((ga, ra), (ge, re)):
                bound = 2.0 ** -24 * w * h * 2 * 5 * float(r.abs().max())
                assert float((g.double() - r.double()).abs().max()) <= bound
        torch.cuda.synchronize()
        del keep


@pytest.mark.parametrize("which", ["deep", "instanced"])
@pytest.mark.parametrize("mode", ["wave", "mega"])
@pytest.mark.parametrize("shape", [dict(block=64, grid_mult=1), dict(block=64, grid_mult=4),
                                   dict(block=256, grid_mult=2), dict(block=256, grid_mult=4, stack_lds=32)])
@pytest.mark.parametrize("size", [(30, 30, 33), (211, 151, 2), (479, 409, 1), (719, 727, 1)])
def test_more_chunks_than_workgroups(renderers, which, mode, shape, size):
    R, cam = renderers[which]
    w, h, spp = size
    R.set_camera(dict(cam, width=w, height=h))
    kw = dict(spp=spp, max_depth=3, seed=3, mode=mode, **shape)
    print("chunks", which, mode, shape, size, flush=True)
    img = R.render(**kw).clone()
    rays = R.stats()["extension_rays"], R.stats()["shadow_rays"]
    ref = R.render(flags=ptmi.FLAG_PROFILE, **kw)
    assert np.array_equal(_bits(img), _bits(ref))
    assert rays == (R.stats()["extension_rays"], R.stats()["shadow_rays"])


@pytest.mark.parametrize("seed,n_objects", [(1, 4), (2, 2)])
@pytest.mark.parametrize("size", [(40, 30), (800, 700)])
def test_noalloc_with_default_shape(seed, n_objects, size):
    w, h = size  # a small frame, and one of the megakernel (560000 paths)
    scene, cam = scenes.procedural(seed=seed, n_objects=n_objects, width=w, height=h)
    R = ptmi.Renderer(scene, cam)
    print("noalloc", seed, n_objects, size, R.info.stack_entries, flush=True)
    kw = dict(spp=1, max_depth=4, rr_start=2, seed=6)
    assert np.array_equal(_bits(R.render_noalloc(**kw)), _bits(R.render(mode="mega", **kw)))
