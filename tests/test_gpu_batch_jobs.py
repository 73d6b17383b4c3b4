"""The batch's job counters (kept per workgroup, taken off at the end of each
kernel): one job, as many as a workgroup has threads, the most a batch takes,
from workgroups of 64 and 256 threads.  Every job's image equals the job alone
bit for bit, and every job has its completion time."""
import numpy as np
import pytest

from paper_2605_27323_amd import scenes

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2605_27323_amd import ptmi  # noqa: E402


@pytest.mark.parametrize("block", [64, 256])
@pytest.mark.parametrize("n", [1, 64, 65, 255])
def test_many_jobs(n, block):
    print("jobs", n, block, flush=True)
    s, c = scenes.procedural(seed=1000, n_objects=5, width=13, height=7)
    R = ptmi.Renderer(s, c)
    args = [dict(spp=1 + j % 3, max_depth=4, seed=5, frame=j) for j in range(n)]
    imgs, ms, res = ptmi.render_batch([R] * n, args, block=block, pool_capacity=4096)
    torch.cuda.synchronize()
    for j in range(n):
        ref = R.render(mode="wave", job=j, **args[j])
        assert np.array_equal(imgs[j].cpu().numpy().view(np.uint32), ref.cpu().numpy().view(np.uint32)), j
    assert (ms > 0).all() and ms.max() <= 1e3 * res["seconds"]
