"""Small frames (whole paths in one launch, pairs of waves) against the stage
kernels and the megakernel, which the same arguments with per-stage timing
take: images, running averages, ray counts and per-stage items bit for bit, at
the sizes where the launch can go wrong (one path, the edges of a wave, the
largest small frame and one more, 64 and 65 samples, the deepest path, more
chunks than workgroups), and the backward's first replay."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _bits(t):
    return t.cpu().numpy().view(np.uint32)


@pytest.fixture(scope="module")
def renderers():
    from paper_2605_27323_amd import ptmi, scenes
    room, cam = scenes.cornell()
    attr, acam = scenes.cornell_attributes()
    inst_scene, inst, icam = scenes.instanced_procedural(seed=6, n_instances=60)
    return {"room": (ptmi.Renderer(room, cam), cam), "attributes": (ptmi.Renderer(attr, acam), acam),
            "instanced": (ptmi.Renderer(inst_scene, icam, instances=inst), icam)}


@pytest.mark.parametrize("which", ["room", "attributes", "instanced"])
@pytest.mark.parametrize("mode", ["wave", "mega"])
@pytest.mark.parametrize("size", [(1, 1, 1, 3), (9, 7, 1, 5), (8, 8, 1, 0), (13, 5, 1, 4), (31, 17, 3, 5),
                                  (5, 3, 64, 2), (5, 3, 65, 2), (40, 30, 2, 62), (40, 30, 2, 63),
                                  (512, 384, 1, 3), (511, 385, 1, 3), (1024, 512, 1, 2), (1023, 513, 1, 2)])
def test_small_frames_equal_the_stages(renderers, which, mode, size):
    import torch
    from paper_2605_27323_amd import ptmi
    R, cam = renderers[which]
    w, h, spp, depth = size
    R.set_camera(dict(cam, width=w, height=h))
    for extra in (dict(), dict(block=64, grid_mult=1, rr_start=2, sampler="halton"), dict(tail_threshold=200), dict(tail_bounce=1)):
        if extra.get("tail_bounce", 0) > depth:
            continue
        kw = dict(spp=spp, max_depth=depth, seed=4, frame=2, mode=mode, **extra)
        accs = [torch.full((h, w, 3), 0.25, device="cuda") for _ in range(2)]
        img = R.render(accum=accs[0], **kw).clone()
        st = R.stats()
        ref = R.render(accum=accs[1], flags=ptmi.FLAG_PROFILE, **kw)
        rst = R.stats()
        assert np.array_equal(_bits(img), _bits(ref)) and np.array_equal(_bits(accs[0]), _bits(accs[1]))
        for key in ("extension_rays", "shadow_rays", "items", "bytes"):
            assert st[key] == rst[key], key


@pytest.mark.parametrize("mode", ["wave", "mega"])
def test_small_frames_in_flight(renderers, mode):
    import torch
    R, cam = renderers["room"]
    kw = dict(spp=2, max_depth=4, seed=9, mode=mode)
    for w, h in ((37, 29), (256, 128), (257, 128)):
        R.set_camera(dict(cam, width=w, height=h))
        acc, ref = torch.empty((h, w, 3), device="cuda"), torch.empty((h, w, 3), device="cuda")
        img = R.render_frames(7, accum=acc, **kw)
        for f in range(7):
            last = R.render(accum=ref, frame=f, **kw)
        assert np.array_equal(_bits(img), _bits(last)) and np.array_equal(_bits(acc), _bits(ref))


@pytest.mark.parametrize("which", ["room", "attributes"])
@pytest.mark.parametrize("size", [(1, 1, 1, 2), (23, 11, 3, 4), (5, 3, 70, 3)])
def test_backward_from_a_small_replay(renderers, which, size):
    # the path radiances (and kept records) of the small replay feed the same
    # gradient kernel: equal up to the order of the atomic additions
    import torch
    from paper_2605_27323_amd import ptmi
    R, cam = renderers[which]
    w, h, spp, depth = size
    R.set_camera(dict(cam, width=w, height=h))
    d = torch.rand((h, w, 3), generator=torch.Generator().manual_seed(1)).cuda()
    kw = dict(spp=spp, max_depth=depth, seed=4, mode="wave")
    grads = []
    for flags in (0, ptmi.FLAG_KEEP_HITS, ptmi.FLAG_PROFILE, ptmi.FLAG_PROFILE | ptmi.FLAG_KEEP_HITS):
        ga, ge = torch.zeros_like(R.albedo), torch.zeros_like(R.emission)
        R.backward(d, ga, ge, flags=flags, **kw)
        grads.append((ga.double().cpu(), ge.double().cpu(), R.stats()["extension_rays"]))
    # at most npaths * (depth + 1) terms a sum, each rounded once: 2^-24 of
    # the sum of magnitudes per addition, bounded by the largest entry times
    # the number of terms
    n = w * h * spp * (depth + 1)
    for ga, ge, rays in grads[:2]:
        assert rays == grads[2][2]
        for a, b in ((ga, grads[2][0]), (ge, grads[2][1])):
            assert (a - b).abs().max() <= 2.0 ** -24 * n * max(float(b.abs().max()), 1e-30)
