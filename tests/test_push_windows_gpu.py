"""Single-launch networks of many vertex groups whose delays need many windows
(so many words of spike bits that their number's division has to be exact,
see test_push_plan.py) against the per-step kernels (tolerance 0)."""
import pytest

from tests.test_ensemble_push_gpu import _lif

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,delays", [(4800, [1, 90, 191]), (7850, [1, 40, 71, 80]), (8060, [2, 69, 88])])
def test_many_windows_equal_per_step(n, delays):
    import torch
    import paper_0908_3934_amd as gn
    specs = [_lif(n, 1, 0.0, delays), _lif(70, 2, 0.05)]
    print(n, delays, specs[0].src.size, flush=True)
    a, b = gn.Net(specs), gn.Net(specs, flags=gn.NET_BUILD_PER_STEP)
    assert a.info()["ensemble_blocks"] == 2
    spikes = 0
    for T in (150, 33, 400):
        x, y = a.step(T, raster=True, v=True, inp=True), b.step(T, raster=True, v=True, inp=True)
        torch.cuda.synchronize()
        for key in ("raster", "v", "input"):
            assert torch.equal(x[key], y[key]), key
        spikes += int(gn.unpack_raster(y["raster"], b.n_total)[:, n - 42:n].sum())
    assert spikes > 0                                  # (of the last group, whose words stand last)
    a.close()
    b.close()
