"""Replay B's accumulation and its hand-out of paths where they can go wrong:
one lane with a gradient in a wave, full waves of one triangle (every sample
of one pixel), counts of paths on both sides of a wave, of one wave per SIMD
and of a workgroup's share, emissive triangles outside the largest, and the
three ways its vertices come to it (traced, kept in the records' own memory,
kept in the queues of a small replay A, up to depth 16).

The terms are the same bit for bit in every schedule and only the order of
their additions differs: a sum of n terms in binary32, in any order, is
within n * 2^-24 of the sum of the terms' magnitudes (the oracle's).  Against
the oracle's binary64 gradient, up to depth 4, 1e-4 of that sum more for the
shading and 1e-7 of the largest entry for cancellation within a path."""
import numpy as np
import pytest

import oracle
from paper_2605_27323_amd import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2605_27323_amd import ptmi  # noqa: E402


@pytest.fixture(scope="module")
def setups():
    out = {}
    for which in ("lights", "emissive"):
        scene, cam = scenes.procedural(seed=71, n_objects=30, width=80, height=50)
        if which == "emissive":  # small triangles that emit
            scene = {k: np.array(v) for k, v in scene.items()}
            scene["emission"][::37] = (0.5, 1.0, 2.0)
        out[which] = (cam, ptmi.Renderer(scene, cam), oracle.Scene(scene))
    return out


@pytest.mark.parametrize("which", ["lights", "emissive"])
@pytest.mark.parametrize("size", [(1, 1, 1, 2), (1, 1, 65, 3), (9, 7, 1, 4), (8, 8, 16, 3), (43, 31, 1, 2),
                                  (40, 30, 5, 3), (13, 11, 2, 15), (13, 11, 2, 17),
                                  (80, 60, 5, 1), (100, 70, 5, 1)])
def test_gradients(setups, which, size):
    cam, R, O = setups[which]
    w, h, spp, depth = size
    cam = dict(cam, width=w, height=h)
    R.set_camera(cam)
    d = np.random.default_rng(3).normal(size=(w * h, 3)).astype(np.float32)
    kw = dict(spp=spp, max_depth=depth, seed=5, frame=1)
    oa, oe, aa, ae = O.backward(cam, d, **kw)
    order = w * h * spp * (depth + 1) * 2 * 2.0 ** -24
    # grids of 16384 lanes: paths beyond those dealt, and a cursor for all (from 32768)
    shapes = dict(block=64, grid_mult=1) if h >= 60 else dict(block=64, grid_mult=64) if h == 31 else dict(block=128, grid_mult=1) if h == 30 else {}
    grads, rays = {}, set()
    for mode, flags in (("mega", 0), ("mega", ptmi.FLAG_KEEP_HITS), ("wave", 0), ("wave", ptmi.FLAG_KEEP_HITS),
                        ("wave", ptmi.FLAG_PROFILE)):
        print("gradients", which, size, mode, flags, flush=True)
        ga, ge = torch.zeros_like(R.albedo), torch.zeros_like(R.emission)
        R.backward(torch.from_numpy(d).cuda(), ga, ge, mode=mode, flags=flags, **kw, **shapes)
        st = R.stats()
        rays.add((st["extension_rays"], st["shadow_rays"]))
        grads[mode, flags] = [g.cpu().numpy()[:R.nt].astype(np.float64) for g in (ga, ge)]
    assert len(rays) == 1
    first = grads["mega", 0]
    for key, g in grads.items():
        for k, (o, a) in enumerate(((oa, aa), (oe, ae))):
            assert (np.abs(g[k] - first[k]) <= 2.0 * order * 1.001 * a).all(), key
            if depth <= 4:
                assert (np.abs(g[k] - o) <= (1e-4 + order) * a + 1e-7 * np.abs(o).max()).all(), key
