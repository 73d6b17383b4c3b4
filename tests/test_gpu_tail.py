"""The hybrid tail's two mappings of its queue to lanes: spread over the
resident waves up to half of their lanes (131072 paths on 256 compute units),
full waves above, asked to spread or not: the megakernel's image bit for bit."""
import numpy as np
import pytest

from paper_2605_27323_amd import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2605_27323_amd import ptmi  # noqa: E402


@pytest.mark.parametrize("size", [(512, 256), (513, 256), (1, 1), (61, 67), (640, 480)])
@pytest.mark.parametrize("shape", [{}, dict(block=64, grid_mult=1)])
def test_tail_mapping(size, shape):
    scene, cam = scenes.procedural(seed=5, n_objects=12, width=size[0], height=size[1])
    R = ptmi.Renderer(scene, cam)
    kw = dict(spp=1, max_depth=4, seed=3, frame=2)
    ref = R.render(mode="mega", **kw).cpu().numpy().view(np.uint32)
    # FLAG_PROFILE: by the stages, however few paths there are
    for tail in (dict(tail_threshold=1 << 30), dict(tail_bounce=1), dict(tail_threshold=1 << 30, tail_spread=True)):
        print("tail", size, shape, tail, flush=True)
        img = R.render(mode="wave", flags=ptmi.FLAG_PROFILE, **kw, **tail, **shape)
        assert np.array_equal(img.cpu().numpy().view(np.uint32), ref)
        assert R.stats()["items"]["tail"] > 0
