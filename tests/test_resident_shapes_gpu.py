"""The resident kernel at the edges of the shape it really has: delays one
below, at and one beyond the window of arrivals in LDS, workgroups of one wave
up to the full 1,024 vertices; which handles use it, and which calls.  Against
the per-step kernels (tolerance 0)."""
import pytest

import synth
from tests.test_ensemble_push_gpu import _lif

pytestmark = pytest.mark.gpu


def _compare(spec, flags, calls):
    import torch
    import paper_0908_3934_amd as gn
    a, b = gn.Net(spec, flags=flags), gn.Net(spec, flags=gn.NET_BUILD_PER_STEP)
    shape, spikes = a.resident(), 0
    assert shape["workgroups"] > 0 and b.resident()["workgroups"] == 0
    for T in calls:
        x, y = a.step(T, raster=True, v=True, inp=True), b.step(T, raster=True, v=True, inp=True)
        torch.cuda.synchronize()
        for key in ("raster", "v", "input"):
            assert torch.equal(x[key], y[key]), (T, key)
        spikes += int(gn.unpack_raster(y["raster"], b.n_total).sum())
    assert a.resident()["launches"] == len(calls) and b.resident()["launches"] == 0
    assert spikes > 20
    a.close()
    b.close()
    return shape


# vertices, and per workgroup of 256 CUs' worth of them
@pytest.mark.parametrize("flag", ["default", "FUSED_STEP", "PUSH", "REORDER"])
@pytest.mark.parametrize("n,vertices", [(33000, 192), (70000, 320), (200001, 832), (245761, 1024), (262144, 1024)])
def test_delays_around_the_window(n, vertices, flag):
    import torch
    import paper_0908_3934_amd as gn
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are for 256 CUs")
    flags = 0 if flag == "default" else getattr(gn, "NET_BUILD_" + flag)
    net = gn.Net(_lif(n, 1, 0.0, [255]), flags=flags)
    shape = net.resident()
    net.close()
    W = shape["window"]
    assert shape["vertices"] == vertices and 1 < W < 254
    print(n, flag, shape, flush=True)
    got = _compare(_lif(n, 2, 0.0, [1, W - 1, W, W + 1, 255]), flags, (2 * W + 130, 128))
    assert got["window"] == W


def test_full_window_in_lds():
    """One wave per workgroup: every delay there is stays in LDS."""
    assert _compare(_lif(1500, 3, 0.05, [1, 128, 254, 255]), 0, (300, 200))["window"] == 255


@pytest.mark.parametrize("n", [64, 16384, 65535])
def test_plastic_uses_it(n):
    shape = _compare(synth.plastic(_lif(n, 4, 0.05, [1, 2, 25])), 0, (120, 60))
    assert shape["window"] == 25 and shape["vertices"] in (64, 256)


def test_which_calls():
    import paper_0908_3934_amd as gn
    for flags, want in ((0, (1, 1, 1, 2, 3, 3)), (gn.NET_BUILD_PUSH, (1, 1, 2, 3, 4, 4))):
        net = gn.Net(_lif(900, 5, 0.05), flags=flags)
        got = []
        # resident; short; too short to rebuild pull delivery's arrivals; rebuilt; resident; short
        for T in (200, 7, 40, 128, 8, 1):
            net.step(T)
            got.append(net.resident()["launches"])
        assert tuple(got) == want, flags
        net.close()


def test_which_handles():
    import paper_0908_3934_amd as gn
    lif, exc = _lif(900, 6, 0.05), gn.NET_BUILD_SINGLE_LAUNCH
    for specs, kw, uses in ((lif, {}, True), (lif, {"flags": gn.NET_BUILD_AUTOTUNE}, True), (lif, {"flags": exc}, False),
                            (lif, {"flags": gn.NET_BUILD_GRAPH}, False), (lif, {"flags": gn.NET_BUILD_DELIVER_PACKED}, False),
                            (lif, {"block_threads": 256}, False), (lif, {"blocks_per_cu": 1}, False), ([lif, lif], {}, False),
                            (synth.izhikevich(_lif(60, 7, 0.0)), {}, False), (synth.plastic(lif), {"flags": exc}, True),
                            (synth.plastic(lif), {"flags": gn.NET_BUILD_PER_STEP}, False)):
        net = gn.Net(specs, **kw)
        assert (net.resident()["workgroups"] > 0) == uses, kw
        net.close()
