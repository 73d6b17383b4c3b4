"""The traversal kernels' shares of a queue (sections handed to workgroups in
turn, a cursor per workgroup) at the sizes where they can go wrong: queues of
one ray, shorter than a wave per SIMD, at the edges of a section, workgroups
of one, two, three and four waves, grids of one workgroup per compute unit,
the XCD-local split.  Every frame must equal the megakernel's bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def room():
    from paper_2605_27323_amd import ptmi, scenes
    scene, cam = scenes.cornell()
    return ptmi.Renderer(scene, cam), cam


@pytest.mark.parametrize("xcd", [False, True])
@pytest.mark.parametrize("block", [64, 128, 192, 256])
@pytest.mark.parametrize("size", [(1, 1, 1), (5, 3, 1), (32, 32, 1), (33, 31, 1), (255, 257, 1), (181, 181, 2)])
def test_queue_shares_cover_every_ray_once(room, size, block, xcd):
    from paper_2605_27323_amd import ptmi
    R, cam = room
    w, h, spp = size
    R.set_camera(dict(cam, width=w, height=h))
    kw = dict(spp=spp, max_depth=4, seed=3)
    ref = R.render(mode="mega", **kw).cpu().numpy()
    for mult in (1, 8):
        img = R.render(mode="wave", block=block, grid_mult=mult, flags=ptmi.FLAG_XCD_LOCAL if xcd else 0, **kw)
        st = R.stats()
        assert np.array_equal(img.cpu().numpy().view(np.uint32), ref.view(np.uint32))
        assert st["items"]["raygen"] == w * h * spp
