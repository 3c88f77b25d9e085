"""Camera frames of the resident kernel against the per-step kernels (tolerance
0): frames of many steps, of one, and shorter than a step, of which only the
first within a step is written."""
import pytest

from tests.test_ensemble_push_gpu import _lif

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("num,den", [(3, 1000), (7, 50), (1, 1), (3, 2), (2, 1), (5, 1)])
def test_resident_frames(num, den):
    import torch
    import paper_0908_3934_amd as gn
    spec = _lif(700, 1, 0.05)
    spec.frame_num, spec.frame_den = num, den
    a, b = gn.Net(spec, frame_capacity=300), gn.Net(spec, flags=gn.NET_BUILD_PER_STEP, frame_capacity=300)
    for T in (60, 340, 8):
        a.step(T)
        b.step(T)
        frames = min(b.info()["frames_done"], 300)
        assert a.info()["frames_done"] == b.info()["frames_done"]
        for what, kw in [(gn.NET_OBS_CALCIUM, {})] + ([(gn.NET_OBS_FRAMES, {"frames": frames})] if frames else []):
            p, q = a.observe(what, **kw), b.observe(what, **kw)
            torch.cuda.synchronize()
            assert torch.equal(p, q), (T, what)
    assert bool((q != 0).any())
    a.close()
    b.close()
