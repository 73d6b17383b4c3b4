"""The traversal step on the GPU against the oracle where it can go wrong:
leaves of one, three and eight triangles (the record that comes with the fetch
and the ones that follow), entries that stay in LDS or spill, axis-parallel
and shared-edge hits of a triangle soup, two-level scenes, both schedules."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _parity(img, ref, frag):
    img = img.cpu().numpy().reshape(-1, 3)
    ref = np.asarray(ref).reshape(-1, 3)
    tol = 1e-4 * np.maximum(np.abs(img), np.abs(ref)) + 1e-6 * float(np.abs(ref).mean())
    ok = (np.abs(img - ref) <= tol).all(1)
    assert not (~ok & (np.asarray(frag).reshape(-1) == 0)).any() and ok.mean() >= 0.999


@pytest.mark.parametrize("max_leaf", [1, 3, 8])
@pytest.mark.parametrize("stack_lds", [8, 32])
@pytest.mark.parametrize("instanced", [False, True])
def test_leaves_and_stacks_match_the_oracle(max_leaf, stack_lds, instanced):
    import oracle
    from paper_2605_27323_amd import ptmi, scenes
    scene = scenes.random_soup(21, 4000, extent=2.0, emissive_frac=0.05)
    inst = scenes.split_into_instances(scene, 5) if instanced else None
    cam = dict(eye=(0.0, 0.0, -6.0), target=(0, 0, 0), up=(0, 1, 0), vfov_deg=50.0, width=61, height=47)
    kw = dict(spp=2, max_depth=4, seed=5)
    ref, frag = oracle.Scene(scene, instances=inst).render(cam, **kw)
    R = ptmi.Renderer(scene, cam, max_leaf=max_leaf, instances=inst)
    mega = R.render(mode="mega", stack_lds=stack_lds, **kw)
    _parity(mega, ref, frag)
    for args in (dict(), dict(tail_bounce=1), dict(block=64, grid_mult=1)):
        wave = R.render(mode="wave", stack_lds=stack_lds, **args, **kw)
        assert np.array_equal(wave.cpu().numpy().view(np.uint32), mega.cpu().numpy().view(np.uint32))
