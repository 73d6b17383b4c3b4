"""The stage kernels, the megakernel and the two-level stages at small sizes.
Frames of few paths run as one launch whatever their schedule and launch
shape, so these frames ask for per-stage timing (PT_FLAG_PROFILE), which keeps
the kernels that the arguments name, and check from the launch counts that
those ran: the shares of a queue at their edges (one ray, less than a wave per
SIMD, sections of workgroups of one to four waves, the XCD split), leaves of
several triangles, LDS stacks of 8 and 32 entries, launch shapes, both
occupancies, the tail, one stream or two, frames in flight, the batch and the
adjoint.  Every image equals the one-launch frame's bit for bit, and that one
the oracle's within the parity bounds."""
import numpy as np
import pytest

import oracle
from paper_2605_27323_amd import scenes
from tests._parity import assert_parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2605_27323_amd import ptmi  # noqa: E402

P, XCD = ptmi.FLAG_PROFILE, ptmi.FLAG_XCD_LOCAL


def _bits(t):
    return t.cpu().numpy().view(np.uint32)


def _staged(R, mode, flags=0, **kw):
    """The frame by the kernels that its arguments name; its bits."""
    img = _bits(R.render(mode=mode, flags=flags | P, **kw))
    ran = R.stats()["launches"]
    want = {"mega"} if mode == "mega" else {"raygen", "extend", "accumulate"}
    assert want <= set(ran) and ("mega" in ran) == (mode == "mega"), ran
    return img


@pytest.fixture(scope="module")
def room():
    scene, cam = scenes.cornell()
    return ptmi.Renderer(scene, cam), cam


@pytest.mark.parametrize("xcd", [0, XCD])
@pytest.mark.parametrize("block", [64, 128, 192, 256])
@pytest.mark.parametrize("size", [(1, 1, 1), (5, 3, 1), (8, 8, 1), (13, 5, 1), (32, 32, 1), (33, 31, 1), (255, 257, 1),
                                  (181, 181, 2)])
def test_queue_shares(room, size, block, xcd):
    R, cam = room
    w, h, spp = size
    R.set_camera(dict(cam, width=w, height=h))
    kw = dict(spp=spp, max_depth=4, seed=3)
    ref = _bits(R.render(mode="wave", **kw))
    rays = R.stats()["extension_rays"], R.stats()["shadow_rays"]
    for mult in (1, 3, 8):  # 3 x 256 workgroups: 96 to an XCD
        for mode in ("wave", "mega"):
            print("shares", size, block, xcd, mult, mode, flush=True)
            img = _staged(R, mode, flags=xcd, block=block, grid_mult=mult, **kw)
            st = R.stats()
            assert np.array_equal(img, ref)
            assert rays == (st["extension_rays"], st["shadow_rays"])


@pytest.mark.parametrize("max_leaf", [1, 3, 8])
@pytest.mark.parametrize("stack_lds", [8, 32])
@pytest.mark.parametrize("instanced", [False, True])
def test_leaves_and_stacks(max_leaf, stack_lds, instanced):
    scene = scenes.random_soup(21, 4000, extent=2.0, emissive_frac=0.05)
    inst = scenes.split_into_instances(scene, 5) if instanced else None
    cam = dict(eye=(0.0, 0.0, -6.0), target=(0, 0, 0), up=(0, 1, 0), vfov_deg=50.0, width=61, height=47)
    kw = dict(spp=2, max_depth=4, seed=5)
    R = ptmi.Renderer(scene, cam, max_leaf=max_leaf, instances=inst)
    ref = _bits(R.render(stack_lds=stack_lds, **kw))
    img, frag = oracle.Scene(scene, instances=inst).render(cam, **kw)
    assert_parity(ref.view(np.float32), img, frag, what="one launch")
    for mode, args in (("mega", {}), ("mega", dict(mega_waves=5, block=192)), ("wave", {}), ("wave", dict(tail_bounce=1)),
                       ("wave", dict(block=64, grid_mult=1)), ("wave", dict(block=192, grid_mult=1, flags=XCD)),
                       ("wave", dict(flags=ptmi.FLAG_COUNT_WORK))):
        print("leaves", max_leaf, stack_lds, instanced, mode, args, flush=True)
        assert np.array_equal(_staged(R, mode, stack_lds=stack_lds, **args, **kw), ref)
        if args.get("tail_bounce"):
            assert R.stats()["launches"]["tail"] == 1


@pytest.mark.parametrize("max_leaf", [1, 4, 8])
def test_launch_shapes(max_leaf):
    scene, cam = scenes.procedural(seed=41, n_objects=30, width=64, height=40)
    R = ptmi.Renderer(scene, cam, max_leaf=max_leaf)
    kw = dict(spp=2, max_depth=6, rr_start=2, seed=3)
    ref = _bits(R.render(**kw))
    T, S = 1 << 30, ptmi.FLAG_SERIAL_STAGES
    for args in (dict(), dict(block=64, grid_mult=1), dict(block=256, grid_mult=3), dict(block=192, grid_mult=2),
                 dict(tail_threshold=700), dict(tail_threshold=T), dict(tail_bounce=1),
                 dict(tail_bounce=3, tail_threshold=300), dict(tail_bounce=2, tail_spread=True),
                 dict(tail_threshold=T, tail_spread=True, block=64, grid_mult=1), dict(flags=XCD),
                 dict(flags=XCD, block=64, grid_mult=3, tail_bounce=3), dict(flags=S), dict(flags=S, tail_bounce=4),
                 dict(flags=S, tail_threshold=400, block=64, grid_mult=2)):
        print("shape", max_leaf, args, flush=True)
        assert np.array_equal(_staged(R, "wave", **args, **kw), ref), args
    for args in (dict(), dict(block=64, grid_mult=2), dict(mega_waves=5), dict(flags=XCD),
                 dict(flags=XCD, block=128, grid_mult=1, mega_waves=5)):
        print("shape", max_leaf, "mega", args, flush=True)
        assert np.array_equal(_staged(R, "mega", **args, **kw), ref), args


@pytest.mark.parametrize("queues", ["4", "8", "10"])
@pytest.mark.parametrize("mode,args", [("wave", {}), ("wave", dict(tail_threshold=3000, tail_bounce=4)), ("mega", {})])
def test_frames_in_flight(mode, args, queues, monkeypatch):
    # one path more than a frame in flight that runs as one launch
    scene, cam = scenes.procedural(seed=52, n_objects=30, width=241, height=272)
    assert 241 * 272 > 1 << 16
    monkeypatch.setenv("GPU_MAX_HW_QUEUES", queues)
    R = ptmi.Renderer(scene, cam)
    kw = dict(spp=1, max_depth=5, rr_start=3, **args)
    acc, ref = (torch.zeros((272, 241, 3), device="cuda") for _ in range(2))
    print("in flight", mode, args, queues, flush=True)
    img = R.render_frames(11, accum=acc, mode=mode, **kw)
    for f in range(11):
        last = R.render(accum=ref, mode=mode, frame=f, flags=P, **kw)
    assert np.array_equal(_bits(img), _bits(last)) and np.array_equal(_bits(acc), _bits(ref))


@pytest.mark.parametrize("max_leaf,stack_lds,block", [(1, 8, 192), (3, 32, 64), (8, 8, 192), (8, 32, 256)])
def test_batch(max_leaf, stack_lds, block):
    Rs, args = [], []
    for j, (w, h) in enumerate([(61, 47), (8, 8), (1, 1), (130, 70)]):
        scene, cam = scenes.procedural(seed=60 + j, n_objects=6 + 10 * j, width=w, height=h)
        Rs.append(ptmi.Renderer(scene, cam, max_leaf=max_leaf))
        args.append(dict(spp=1 + j, max_depth=5, rr_start=2 if j & 1 else -1, seed=j))
    for cap in (64, 4096):
        print("batch", max_leaf, stack_lds, block, cap, flush=True)
        imgs, ms, _ = ptmi.render_batch(Rs, args, block=block, grid_mult=1, stack_lds=stack_lds, pool_capacity=cap)
        assert (ms > 0).all()
        for j, R in enumerate(Rs):
            assert np.array_equal(_bits(imgs[j]), _staged(R, "wave", job=j, **args[j])), j


@pytest.mark.parametrize("max_leaf", [1, 8])
@pytest.mark.parametrize("block", [64, 192, 256])
def test_adjoint(max_leaf, block):
    # replay A by the stages and as one kernel, replay B tracing and from the
    # records, in workgroups of one, three and four waves: a gradient's terms
    # are the same and only their order differs, so two sums of n terms are
    # within 2 n 2^-24 of the terms' magnitudes (the oracle's) of each other
    scene, cam = scenes.procedural(seed=71, n_objects=30, width=57, height=43)
    R = ptmi.Renderer(scene, cam, max_leaf=max_leaf)
    kw = dict(spp=3, max_depth=3, seed=5, frame=1)
    d = np.random.default_rng(3).normal(size=(57 * 43, 3)).astype(np.float32)
    _, _, aa, ae = oracle.Scene(scene).backward(cam, d, **kw)
    order = 57 * 43 * 3 * (3 + 1) * 2 * 2.0 ** -24
    first = None
    for mode, flags in (("mega", P), ("mega", P | ptmi.FLAG_KEEP_HITS), ("wave", P), ("wave", P | XCD),
                        ("wave", P | ptmi.FLAG_KEEP_HITS | ptmi.FLAG_SERIAL_STAGES)):
        for mult in (1, 8):
            print("adjoint", max_leaf, block, mode, flags, mult, flush=True)
            ga, ge = torch.zeros_like(R.albedo), torch.zeros_like(R.emission)
            R.backward(torch.from_numpy(d).cuda(), ga, ge, mode=mode, flags=flags, block=block, grid_mult=mult, **kw)
            ran = R.stats()["launches"]
            assert ran["adjoint"] == 1 and ("extend" in ran) == (mode == "wave")
            g = [t.cpu().numpy()[:R.nt].astype(np.float64) for t in (ga, ge)]
            first = first or g
            for k, a in enumerate((aa, ae)):
                assert (np.abs(g[k] - first[k]) <= 2.0 * order * 1.001 * a).all(), (mode, flags)
